"""GPU parity on seeded random shapes: every entry point against the CPU oracle, bit for bit, on
shapes and expert splits that no other test fixes by hand (tiles of 128 and 256 columns, partial
row tiles, odd split lengths, empty experts, unaligned k-rows), with guard bytes around every
output of the ragged forms; transposing conversions by the tiles of small matrices and, with the columns repeated,
by those of large ones.  MXFP4_EXTRA_SEEDS=n in the environment adds n further seeds to each test."""
import functools
import os

import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import ref
from paper_2603_02731_amd import synth
from tests.rules import times_as_wide
from tests.test_gpu_parity import UNITS, check_wide

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 1024
EXTRA = int(os.environ.get("MXFP4_EXTRA_SEEDS", "0"))


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def same(got, want, what):
    got, want = np.asarray(got).reshape(-1), np.asarray(want).reshape(-1)
    assert got.size == want.size, (what, got.size, want.size)
    if got.dtype == np.float32:
        got, want = got.view(np.uint32), want.view(np.uint32)
    bad = np.flatnonzero(got != want)
    assert bad.size == 0, f"{what}: {bad.size} mismatches, first at {int(bad[0])}"


def guarded(n, dtype, fill):
    buf = torch.full((GUARD + n + GUARD,), fill, dtype=dtype, device=DEV)
    return buf, buf[GUARD:GUARD + n]


def check_guards(buf, n, fill, what):
    b = host(buf)
    assert (b[:GUARD] == fill).all() and (b[GUARD + n:] == fill).all(), f"{what}: written outside the output"
    return b[GUARD:GUARD + n]


def random_splits(rng, total_cap):
    """Expert lengths of every kind: empty, shorter than a block, odd, multiples of 32/128/256, long."""
    kinds = [0, 1, 5, 31, 32, 33, 64, 96, 127, 128, 129, 255, 256, 257, 300, 384, 511, 513]
    n = int(rng.integers(1, 12))
    T = [int(rng.choice(kinds)) for _ in range(n)]
    while sum(T) > total_cap:
        T.pop()
    if sum(T) == 0:
        T.append(32)
    return T


def wide_experts(kind, q, sf, T, wants):
    """The grouped conversion of the same columns again and again beside each other, as often as it takes to leave the small tiles:
    every expert's k-rows are the oracle's (wants: data, scales), as often, and nothing around the outputs is written."""
    M, K = q.shape[0], 2 * q.shape[1]
    n = times_as_wide(kind, M, K, len(T), UNITS)
    off = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    units, fill = ((2, 32), (0xA5, 0x5A)) if kind == "mxfp4" else ((1, 128), (0xA5, -7.0))
    types = (torch.uint8, torch.uint8 if kind == "mxfp4" else torch.float32)
    bufs = [guarded(n * w.size, t, f) for w, t, f in zip(wants, types, fill)]
    args = dev(q).repeat(1, n), dev(sf).repeat(1, n), torch.from_numpy(off).to(DEV)
    if kind == "mxfp4":
        mx.mxfp4_row_to_col_grouped(*args, q_col=bufs[0][1], sf_col=bufs[1][1], offsets_host=off)
    else:
        mx.mxfp4_row_to_fp8_col_grouped(*args, x_col=bufs[0][1], x_col_scale=bufs[1][1], requant=kind == "requant", offsets_host=off)
    for (buf, _), w, u, f in zip(bufs, wants, units, fill):
        ends = np.cumsum([0] + [K * -(-t // u) for t in T])
        want = np.concatenate([np.tile(w.reshape(-1)[a:b], n) for a, b in zip(ends, ends[1:])])
        same(check_guards(buf, want.size, f, kind), want, f"{kind} T={T} K={n} x {K}")


@pytest.mark.parametrize("seed", range(12 + EXTRA))
def test_flat_entry_points_on_random_shapes(seed):
    rng = np.random.default_rng(1000 + seed)
    M = 32 * int(rng.integers(1, 40))            # row->col needs M % 32 == 0
    K = 128 * int(rng.integers(1, 9))
    x8, s = synth.fp8_blockwise_quantize(torch.from_numpy(
        (rng.standard_t(3, size=(M, K)) * 10.0 ** rng.uniform(-3, 3)).astype(np.float32)))
    x8, s = x8.numpy(), s.numpy()
    q, sf = mx.mxfp4_quant_from_fp8(dev(x8), dev(s))
    wq, wsf = ref.quant_from_fp8(x8, s)
    same(host(sf), wsf, f"quant scales [{M},{K}]")
    same(host(q), wq, f"quant nibbles [{M},{K}]")
    x, xs = mx.mxfp4_dequant_to_fp8(q, sf)
    wx, wxs = ref.dequant_to_fp8(wq, wsf)
    same(host(xs), wxs, f"dequant scales [{M},{K}]")
    same(host(x), wx, f"dequant bytes [{M},{K}]")
    qc, sc = mx.mxfp4_row_to_col(q, sf)
    wqc, wsc = ref.row_to_col(wq, wsf)
    same(host(sc), wsc, f"row->col scales [{M},{K}]")
    same(host(qc), wqc, f"row->col nibbles [{M},{K}]")
    check_wide("mxfp4", mx.mxfp4_row_to_col, wq, wsf, wqc, wsc)
    if M % 128 == 0:
        for requant in (False, True):
            xc, xcs = mx.mxfp4_row_to_fp8_col(q, sf, requant=requant)
            wxc, wxcs = ref.row_to_fp8_col(wq, wsf, requant=requant)
            same(host(xcs), wxcs, f"row->FP8 col scales [{M},{K}] requant={requant}")
            same(host(xc), wxc, f"row->FP8 col bytes [{M},{K}] requant={requant}")
            check_wide("requant" if requant else "align", functools.partial(mx.mxfp4_row_to_fp8_col, requant=requant), wq, wsf, wxc, wxcs)


@pytest.mark.parametrize("seed", range(12 + EXTRA))
def test_grouped_entry_points_on_random_splits(seed):
    rng = np.random.default_rng(2000 + seed)
    K = 128 * int(rng.integers(1, 7))
    T = random_splits(rng, 2400)
    off = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    M = int(off[-1])
    q, sf = synth.random_mxfp4(M, K, seed=3000 + seed, scale_center=int(rng.integers(60, 200)),
                               scale_spread=int(rng.integers(0, 12)), nan_scale_frac=0.002 * (seed % 3))
    q, sf = q.numpy(), sf.numpy()
    offd = torch.from_numpy(off).to(DEV)

    wqc, wsc = ref.row_to_col_grouped(q, sf, off)
    qbuf, qv = guarded(wqc.size, torch.uint8, 0xA5)
    sbuf, sv = guarded(wsc.size, torch.uint8, 0x5A)
    mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), offd, q_col=qv, sf_col=sv, offsets_host=off)
    same(check_guards(sbuf, wsc.size, 0x5A, "sf_col"), wsc, f"grouped row->col scales T={T} K={K}")
    same(check_guards(qbuf, wqc.size, 0xA5, "q_col"), wqc, f"grouped row->col nibbles T={T} K={K}")
    wide_experts("mxfp4", q, sf, T, (wqc, wsc))

    for requant in (False, True):
        wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off, requant=requant)
        xbuf, xv = guarded(wx.size, torch.uint8, 0xA5)
        fbuf, fv = guarded(wxs.size, torch.float32, -7.0)
        mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), offd, x_col=xv, x_col_scale=fv, requant=requant, offsets_host=off)
        same(check_guards(fbuf, wxs.size, -7.0, "x_col_scale"), wxs, f"grouped FP8 col scales T={T} K={K} requant={requant}")
        same(check_guards(xbuf, wx.size, 0xA5, "x_col"), wx, f"grouped FP8 col bytes T={T} K={K} requant={requant}")
        wide_experts("requant" if requant else "align", q, sf, T, (wx, wxs))


@pytest.mark.parametrize("seed", range(10 + EXTRA))
def test_strided_and_routed_forms_on_random_shapes(seed):
    """The non-dense kernel instances: gathered rows into padded planes and into per-token records, the
    de-quantizer reading those, the scatter form with a random fan-out, the BF16 quantizer into padded
    planes; bytes between the rows of a padded output must stay as they were."""
    rng = np.random.default_rng(4000 + seed)
    M_src = int(rng.integers(1, 700))
    K = 128 * int(rng.integers(1, 9))
    v = (rng.standard_t(3, size=(M_src, K)) * 10.0 ** rng.uniform(-3, 3)).astype(np.float32)
    x8, s = synth.fp8_blockwise_quantize(torch.from_numpy(v))
    x8, s = x8.numpy(), s.numpy()
    xd, sd = dev(x8), dev(s)

    # gather into planes whose rows are padded
    M_out = int(rng.integers(1, 1500))
    idx = rng.integers(0, M_src, M_out).astype(np.int32)
    wq, wsf = ref.quant_from_fp8(x8, s, gather_idx=idx)
    ld_q = K // 2 + 8 * int(rng.integers(0, 5))
    ld_sf = K // 32 + 4 * int(rng.integers(0, 5))
    qbuf = torch.full((M_out * ld_q,), 0xA5, dtype=torch.uint8, device=DEV)
    sbuf = torch.full((M_out * ld_sf,), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_fp8(xd, sd, gather_idx=dev(idx), q=qbuf, sf=sbuf, ld_q=ld_q, ld_sf=ld_sf)
    qh, sh = host(qbuf).reshape(M_out, ld_q), host(sbuf).reshape(M_out, ld_sf)
    same(qh[:, :K // 2], wq, f"gathered nibbles, ld_q={ld_q}")
    same(sh[:, :K // 32], wsf, f"gathered scales, ld_sf={ld_sf}")
    assert (qh[:, K // 2:] == 0xA5).all() and (sh[:, K // 32:] == 0x5A).all(), "padding between rows written"

    # one record per token (nibbles, scales, padding to 16 bytes), and the de-quantizer reading the records
    rec = (K // 2 + K // 32 + 15) // 16 * 16 + 16 * int(rng.integers(0, 3))
    rbuf = torch.full((M_out * rec,), 0xC3, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_fp8(xd, sd, gather_idx=dev(idx), q=rbuf, sf=rbuf[K // 2:], ld_q=rec, ld_sf=rec)
    rh = host(rbuf).reshape(M_out, rec)
    same(rh[:, :K // 2], wq, f"record nibbles, record of {rec} bytes")
    same(rh[:, K // 2:K // 2 + K // 32], wsf, "record scales")
    assert (rh[:, K // 2 + K // 32:] == 0xC3).all(), "padding of the records written"
    x, xs = mx.mxfp4_dequant_to_fp8(rbuf, rbuf[K // 2:], M=M_out, K=K, ld_q=rec, ld_sf=rec)
    wx, wxs = ref.dequant_to_fp8(wq, wsf)
    same(host(xs), wxs, "tile scales from records")
    same(host(x), wx, "E4M3 bytes from records")

    # the routing turned around: random fan-out, some entries pointing nowhere
    fanout = int(rng.integers(1, 10))
    M_dst = M_src * fanout + int(rng.integers(0, 50))
    slots = rng.permutation(M_dst)[:M_src * fanout].astype(np.int32).reshape(M_src, fanout)
    nowhere = rng.random(slots.shape) < 0.1
    slots[nowhere] = rng.choice(np.array([-1, M_dst, 2 ** 31 - 1], np.int32), size=int(nowhere.sum()))
    wq2, wsf2 = ref.quant_from_fp8_scatter(x8, s, slots, M_dst, q=np.full((M_dst, K // 2), 0xA5, np.uint8),
                                           sf=np.full((M_dst, K // 32), 0x5A, np.uint8))
    q2 = torch.full((M_dst, K // 2), 0xA5, dtype=torch.uint8, device=DEV)
    sf2 = torch.full((M_dst, K // 32), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_fp8_scatter(xd, sd, dev(slots), M_dst, q=q2, sf=sf2)
    same(host(sf2), wsf2, f"scattered scales, fanout {fanout}")
    same(host(q2), wq2, f"scattered nibbles, fanout {fanout}")

    # BF16 source into padded planes
    xb = torch.from_numpy(v).to(torch.bfloat16)
    wq3, wsf3 = ref.quant_from_bf16(xb.view(torch.int16).numpy().view(np.uint16))
    ld_q3 = K // 2 + 4 * int(rng.integers(0, 5))
    q3 = torch.full((M_src * ld_q3,), 0xA5, dtype=torch.uint8, device=DEV)
    s3 = torch.full((M_src * ld_sf,), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_bf16(xb.to(DEV), q=q3, sf=s3, ld_q=ld_q3, ld_sf=ld_sf)
    q3h, s3h = host(q3).reshape(M_src, ld_q3), host(s3).reshape(M_src, ld_sf)
    same(q3h[:, :K // 2], wq3, f"BF16 nibbles, ld_q={ld_q3}")
    same(s3h[:, :K // 32], wsf3, "BF16 scales")
    assert (q3h[:, K // 2:] == 0xA5).all() and (s3h[:, K // 32:] == 0x5A).all(), "padding between rows written"
