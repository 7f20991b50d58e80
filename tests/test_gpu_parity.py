"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, bit for bit.

Every comparison is exact equality of packed nibbles, scale bytes, E4M3 bytes and FP32
scale bit patterns.  Sizes span several tiles and ragged tails; the edge cases of each
conversion (zero blocks, NaN, subnormals, saturation, huge scale spreads) are included, by
the tiles of small matrices and by those of large ones.
"""
import functools

import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import ref
from paper_2603_02731_amd import synth
from oracle import parallel as par
from tests.rules import small_tiles, times_as_wide
from tests.test_oracle_quant import scale_sweep

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
UNITS = torch.cuda.get_device_properties(0).multi_processor_count if torch.cuda.is_available() else 256


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def assert_same(got, want, what):
    got, want = np.asarray(got), np.asarray(want)
    assert got.shape == want.shape, (what, got.shape, want.shape)
    if got.dtype == np.float32:
        got, want = got.view(np.uint32), want.view(np.uint32)
    bad = np.argwhere(got != want)
    assert bad.size == 0, f"{what}: {len(bad)} mismatches, first at {bad[0].tolist()}: " \
                          f"got {got[tuple(bad[0])]:#x} want {want[tuple(bad[0])]:#x}"


def check_quant(x8, s, **kw):
    q, sf = mx.mxfp4_quant_from_fp8(dev(x8), dev(s), **kw)
    wq, wsf = par.quant(x8, s)
    assert_same(host(sf), wsf, "quant scale bytes")
    assert_same(host(q), wq, "quant nibbles")
    return wq, wsf


def check_dequant(q, sf):
    x, xs = mx.mxfp4_dequant_to_fp8(dev(q), dev(sf))
    wx, wxs = par.dequant(q, sf)
    assert_same(host(xs), wxs, "dequant tile scales")
    assert_same(host(x), wx, "dequant E4M3 bytes")


def check_wide(kind, convert, q, sf, want, want_scales):
    """The same columns again and again beside each other: as often as it takes for tiles of 256 x 256, and for their nibbles to arrive
    by 16-byte loads (where the rows fill a tile).  want, want_scales: the oracle's result for the columns once."""
    M, K = q.shape[0], 2 * q.shape[1]
    staged = (3 if kind == "mxfp4" else 4) * UNITS  # tiles
    want, want_scales = dev(want), dev(want_scales)
    for n in (times_as_wide(kind, M, K, units=UNITS), -(-(-(-staged // -(-M // 256)) * 256) // K)):
        assert not small_tiles(kind, M, n * K, units=UNITS)
        data, scales = convert(dev(q).repeat(1, n), dev(sf).repeat(1, n))
        for got, w, what in ((scales, want_scales, "scales"), (data, want, "elements")):
            got, w = (t.view(torch.int32) if t.dtype == torch.float32 else t for t in (got, w))
            bad = (got.view(n, *w.shape) != w).sum().item()
            assert bad == 0, f"{kind} {what}, {n} times as wide: {bad} differ"


def check_row_to_col(q, sf):
    qc, sc = mx.mxfp4_row_to_col(dev(q), dev(sf))
    wq, ws = par.row_to_col(q, sf)
    assert_same(host(sc), ws, "row->col scale bytes")
    assert_same(host(qc), wq, "row->col nibbles")
    check_wide("mxfp4", mx.mxfp4_row_to_col, q, sf, wq, ws)


# ------------------------------------------------------------------ config 1: tiny round trip

@pytest.mark.parametrize("seed", [0, 1, 2])
def test_config1_round_trip_and_row_to_col(seed):
    x8, s = synth.tiny_roundtrip_fp8(seed=seed)
    x8, s = x8.numpy(), s.numpy()
    q, sf = check_quant(x8, s)
    check_dequant(q, sf)
    check_row_to_col(q, sf)


# ------------------------------------------------------------------ quant: exhaustive codes x scales

def test_quant_all_codes_times_scale_sweep():
    rng = np.random.default_rng(0)
    scales = scale_sweep()
    scales += [float(np.float32(rng.uniform(1e-3, 10.0)) / np.float32(448)) for _ in range(200)]
    scales += [float(np.float32(2.0 ** rng.uniform(-149, 118))) for _ in range(200)]
    rows_x, rows_s = [], []
    for s in scales:
        # every code once, shuffled over 8 blocks; then every code under small block maxima
        perm = rng.permutation(256).astype(np.uint8)
        rows_x.append(perm.reshape(2, 128))
        rows_s.append(np.full((2, 1), s, np.float32))
        small = (rng.integers(0, 256, size=(2, 128)) & 0x8F | rng.integers(0, 0x30, size=(2, 128))).astype(np.uint8)
        rows_x.append(small)
        rows_s.append(np.full((2, 1), s, np.float32))
    x8 = np.concatenate(rows_x)
    s = np.concatenate(rows_s)
    pad = (-x8.shape[0]) % 7                      # K = 128*7 so that rows hold several tiles
    x8 = np.concatenate([x8, np.zeros((pad, 128), np.uint8)]).reshape(-1, 128 * 7)
    s = np.concatenate([s, np.ones((pad, 1), np.float32)]).reshape(-1, 7)
    check_quant(x8, s)


def test_quant_every_code_under_every_block_maximum():
    rows = []
    for cmax in range(1, 0x7F):
        others = np.arange(0, cmax + 1)
        for i in range(0, len(others), 31):
            blk = np.concatenate([[cmax], others[i:i + 31]])
            blk = np.concatenate([blk, np.zeros(32 - len(blk), np.int64)])
            sign = ((np.arange(32) + cmax) % 3 == 0) * 0x80
            rows.append((blk | sign).astype(np.uint8))
    rows += [np.zeros(32, np.uint8)] * ((-len(rows)) % 4)
    x8 = np.stack(rows).reshape(-1, 128)
    for sval in [1.0, 2.0 ** -131, 2.0 ** 118, 0.0123, 3.3e-38, 1.7e36]:
        check_quant(x8, np.full((x8.shape[0], 1), sval, np.float32))


def test_quant_nan_inf_zero_blocks():
    x8, s = synth.student_t_fp8(96, 1024, seed=3)
    x8, s = x8.numpy().copy(), s.numpy().copy()
    x8[3, 5] = 0x7F
    x8[3, 700] = 0xFF
    x8[10, 32:64] = 0
    x8[11, :] = 0x80
    s[20, 2] = 0.0
    s[21, 1] = np.finfo(np.float32).max / 8      # products overflow to inf
    s[22, 0] = 2.0 ** -149
    s[23, 3] = 2.0 ** -140
    check_quant(x8, s)


def test_quant_scales_outside_the_format():
    """Tile scales no blockwise-FP8 producer emits: infinite, NaN, negative, negative zero, negative subnormal.
    The element is the IEEE-754 product, so a NaN scale and infinity times a zero code poison their blocks."""
    rng = np.random.default_rng(9)
    x8 = rng.integers(0, 256, (64, 512), dtype=np.int64).astype(np.uint8)
    x8[::2][(x8[::2] & 0x7F) == 0] = 0x21         # even rows hold no zero codes
    x8[(x8 & 0x7F) == 0x7F] = 0x42                # NaN codes have their own test
    exotic = np.array([np.inf, -np.inf, np.nan, -1.0, -0.0, -3.5e-40, -2.0 ** 100, 1.0], np.float32)
    s = exotic[rng.integers(0, len(exotic), (64, 4))]
    check_quant(x8, s)
    q, sf = check_quant(x8, np.full((64, 4), np.inf, np.float32))
    assert (sf[::2] == 254).all() and ((sf[1::2] == 254) | (sf[1::2] == 255)).all() and (sf[1::2] == 255).any()
    # the routed forms of the kernel
    idx = rng.integers(0, 64, 200).astype(np.int32)
    gq, gsf = mx.mxfp4_quant_from_fp8(dev(x8), dev(s), gather_idx=dev(idx))
    wq, wsf = ref.quant_from_fp8(x8, s, gather_idx=idx)
    assert_same(host(gsf), wsf, "gathered scale bytes")
    assert_same(host(gq), wq, "gathered nibbles")
    dst = rng.permutation(64 * 3).astype(np.int32).reshape(64, 3)
    sq, ssf = mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), 64 * 3)
    inv = np.empty(64 * 3, np.int32)
    inv[dst.reshape(-1)] = np.repeat(np.arange(64, dtype=np.int32), 3)
    wq, wsf = ref.quant_from_fp8(x8, s, gather_idx=inv)
    assert_same(host(ssf), wsf, "scattered scale bytes")
    assert_same(host(sq), wq, "scattered nibbles")


# ------------------------------------------------------------------ dequant

@pytest.mark.parametrize("center,spread,nan", [(127, 0, 0.0), (127, 3, 0.0), (120, 9, 0.01), (60, 25, 0.0),
                                              (8, 8, 0.0), (250, 4, 0.02), (127, 127, 0.0)])
def test_dequant_random_codes_and_scale_spreads(center, spread, nan):
    q, sf = synth.random_mxfp4(96, 1152, seed=center + spread, scale_center=center, scale_spread=spread,
                               nan_scale_frac=nan)
    check_dequant(q.numpy(), sf.numpy())


def test_dequant_every_shift_and_code():
    # block 1 of each tile sits d binades under the tile maximum, d = 0..40; all 16 codes
    rows_q, rows_s = [], []
    for bmax in (254, 140, 41, 20, 6, 3):
        for d in range(0, 41):
            if bmax - d < 0:
                continue
            nib = np.tile(np.arange(16, dtype=np.uint8), 8)
            rows_q.append((nib[0::2] | (nib[1::2] << 4)).astype(np.uint8))
            rows_s.append(np.array([bmax, bmax - d, max(bmax - d // 2, 0), bmax - d], np.uint8))
    pad = (-len(rows_q)) % 3
    rows_q += [np.zeros(64, np.uint8)] * pad
    rows_s += [np.zeros(4, np.uint8)] * pad
    check_dequant(np.stack(rows_q).reshape(-1, 192), np.stack(rows_s).reshape(-1, 12))


# ------------------------------------------------------------------ row -> col

@pytest.mark.parametrize("M,K,center,spread,nan", [
    (256, 256, 127, 0, 0.0), (288, 384, 127, 3, 0.0), (32, 128, 100, 8, 0.0), (544, 640, 30, 30, 0.0),
    (96, 1152, 4, 6, 0.0), (320, 256, 250, 5, 0.0), (512, 512, 127, 127, 0.0), (352, 384, 120, 4, 0.003)])
def test_row_to_col_random_codes_and_scale_spreads(M, K, center, spread, nan):
    q, sf = synth.random_mxfp4(M, K, seed=M + K + spread, scale_center=center, scale_spread=spread,
                               nan_scale_frac=nan)
    q, sf = q.numpy().copy(), sf.numpy()
    q[:, 5] = 0                                   # two all-zero columns
    q[7::32, :] &= 0x88                           # rows of signed zeros
    check_row_to_col(q, sf)


def test_row_to_col_on_quantized_swiglu():
    x8, s = synth.swiglu_fp8(1024, 2048, seed=1)
    q, sf = par.quant(x8.numpy(), s.numpy())
    check_row_to_col(q, sf)


# ------------------------------------------------------------------ grouped, gather, records

def test_grouped_variants_small():
    off, counts = synth.expert_offsets(seed=1, num_experts=7, total_tokens=1500, pad_to=32)
    M = int(off[-1])
    x8, s = synth.student_t_fp8(M, 512, seed=2)
    x8, s = synth.zero_padding_rows(x8, s, off, counts)
    x8, s = x8.numpy(), s.numpy()
    q, sf = mx.mxfp4_quant_from_fp8_grouped(dev(x8), dev(s), off.to(DEV))
    wq, wsf = ref.quant_from_fp8_grouped(x8, s, off.numpy())
    assert_same(host(q), wq, "grouped quant nibbles")
    assert_same(host(sf), wsf, "grouped quant scales")
    qc, sc = mx.mxfp4_row_to_col_grouped(dev(wq), dev(wsf), off.to(DEV))
    wqc, wsc = ref.row_to_col_grouped(wq, wsf, off.numpy())
    assert_same(host(sc)[:wsc.size], wsc, "grouped row->col scales")
    assert_same(host(qc)[:wqc.size], wqc, "grouped row->col nibbles")


def test_grouped_with_empty_experts():
    off = torch.tensor([0, 0, 320, 320, 352, 864, 864], dtype=torch.int32)
    q, sf = synth.random_mxfp4(864, 384, seed=5, scale_center=125, scale_spread=4)
    q, sf = q.numpy(), sf.numpy()
    qc, sc = mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), off.to(DEV))
    wqc, wsc = ref.row_to_col_grouped(q, sf, off.numpy())
    assert_same(host(sc)[:wsc.size], wsc, "grouped row->col scales")
    assert_same(host(qc)[:wqc.size], wqc, "grouped row->col nibbles")


def test_gather_and_token_records():
    x8, s = synth.student_t_fp8(300, 1024, seed=6)
    idx = synth.routing_indices(seed=7, num_tokens=300, top_k=8)
    x8, s = x8.numpy(), s.numpy()
    wq, wsf = ref.quant_from_fp8(x8, s, gather_idx=idx.numpy())
    q, sf = mx.mxfp4_quant_from_fp8(dev(x8), dev(s), gather_idx=idx.to(DEV))
    assert_same(host(q), wq, "gathered nibbles")
    assert_same(host(sf), wsf, "gathered scales")
    # one record per token: K/2 nibble bytes then K/32 scale bytes
    K = 1024
    rec = K // 2 + K // 32
    buf = torch.zeros(idx.shape[0] * rec, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_fp8(dev(x8), dev(s), gather_idx=idx.to(DEV), q=buf, sf=buf[K // 2:], ld_q=rec, ld_sf=rec)
    recs = host(buf).reshape(-1, rec)
    assert_same(recs[:, :K // 2], wq, "record nibbles")
    assert_same(recs[:, K // 2:], wsf, "record scales")
    # and back: dequantize straight from the records
    x, xs = mx.mxfp4_dequant_to_fp8(buf, buf[K // 2:], M=idx.shape[0], K=K, ld_q=rec, ld_sf=rec)
    wx, wxs = par.dequant(wq, wsf)
    assert_same(host(x), wx, "dequant from records")
    assert_same(host(xs), wxs, "dequant scales from records")
    # an out-of-range index yields a zero row, not a fault
    bad = idx.clone()
    bad[3], bad[11] = -1, 300
    q, sf = mx.mxfp4_quant_from_fp8(dev(x8), dev(s), gather_idx=bad.to(DEV))
    q, sf = host(q), host(sf)
    assert not q[3].any() and not sf[3].any() and not q[11].any() and not sf[11].any()
    keep = np.ones(len(bad), bool)
    keep[[3, 11]] = False
    assert_same(q[keep], wq[keep], "rows next to a bad index")


def test_empty_and_argument_errors():
    z8 = torch.empty((0, 256), dtype=torch.uint8, device=DEV)
    zs = torch.empty((0, 2), dtype=torch.float32, device=DEV)
    q, sf = mx.mxfp4_quant_from_fp8(z8, zs)
    assert q.shape == (0, 128) and sf.shape == (0, 8)
    x8 = torch.zeros((32, 256), dtype=torch.uint8, device=DEV)
    xs = torch.ones((32, 2), dtype=torch.float32, device=DEV)
    with pytest.raises(ValueError):
        mx.mxfp4_quant_from_fp8(x8[:, :192].contiguous(), xs)          # K % 128 != 0: stopped by the binding
    with pytest.raises(mx.Mxfp4Error) as e:
        mx.mxfp4_quant_from_fp8(x8.reshape(-1)[1:257].reshape(1, 256), xs[:1])   # misaligned
    assert e.value.status == -3
    q, sf = mx.mxfp4_quant_from_fp8(x8, xs)
    with pytest.raises(ValueError):
        mx.mxfp4_row_to_col(q[:16], sf[:16])                            # M % 32 != 0: stopped by the binding
    with pytest.raises(TypeError):
        mx.mxfp4_row_to_col(q, sf, q_col=torch.empty((256, 16), dtype=torch.uint8))   # an output in host memory
    with pytest.raises(ValueError):
        mx.mxfp4_row_to_col(q, sf, sf_col=torch.empty((256, 1), dtype=torch.uint8, device=DEV)[:255])


# ------------------------------------------------------------------ BF16 -> MXFP4 (the paper's row-wise kernel)

def check_quant_bf16(bits):
    x = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).to(DEV)
    q, sf = mx.mxfp4_quant_from_bf16(x)
    wq, wsf = par.quant_bf16(bits)
    assert_same(host(sf), wsf, "bf16 quant scale bytes")
    assert_same(host(q), wq, "bf16 quant nibbles")


def test_quant_bf16_every_bit_pattern():
    # all 65536 patterns (every exponent, subnormals, inf, NaN), shuffled over blocks, several seeds;
    # then each exponent's patterns together so that small values are not always flushed by a big neighbour
    rng = np.random.default_rng(0)
    rows = [rng.permutation(65536).astype(np.uint16).reshape(64, 1024) for _ in range(3)]
    by_exp = np.arange(65536, dtype=np.uint32).astype(np.uint16).reshape(2, 256, 128)   # [sign][exp][mant]
    grouped = np.concatenate([by_exp[0], by_exp[1]], axis=1)                            # one exponent per row
    rows.append(np.tile(grouped, (1, 4))[:, :1024])
    mixed = grouped.copy()
    for r in range(256):
        rng.shuffle(mixed[r])
    rows.append(np.tile(mixed, (1, 4))[:, :1024])
    check_quant_bf16(np.concatenate(rows))


def test_quant_bf16_activations_and_strides():
    g = torch.Generator().manual_seed(3)
    v = torch.randn(200, 1152, generator=g) * torch.logspace(-3, 3, 1152)
    v[5, 40:72] = 0
    v[6, 100] = float("inf")
    v[7, 300] = float("nan")
    xb = v.to(torch.bfloat16)
    bits = xb.view(torch.uint16).numpy()
    check_quant_bf16(bits)
    K = 1152
    rec = K // 2 + K // 32
    buf = torch.zeros(200 * rec, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_bf16(xb.to(DEV), q=buf, sf=buf[K // 2:], ld_q=rec, ld_sf=rec)
    wq, wsf = ref.quant_from_bf16(bits)
    recs = host(buf).reshape(200, rec)
    assert_same(recs[:, : K // 2], wq, "bf16 record nibbles")
    assert_same(recs[:, K // 2:], wsf, "bf16 record scales")


# ------------------------------------------------------------------ row-blocked MXFP4 -> column-wise FP8

def check_row_to_fp8_col(q, sf):
    x, xs = mx.mxfp4_row_to_fp8_col(dev(q), dev(sf))
    wx, wxs = ref.row_to_fp8_col(q, sf)
    assert_same(host(xs), wxs, "row->FP8 col: group scales")
    assert_same(host(x), wx, "row->FP8 col: E4M3 bytes")
    check_wide("align", mx.mxfp4_row_to_fp8_col, q, sf, wx, wxs)


@pytest.mark.parametrize("M,K,center,spread,nan", [
    (256, 256, 127, 0, 0.0), (384, 384, 127, 3, 0.0), (128, 128, 100, 8, 0.0), (640, 640, 30, 30, 0.0),
    (128, 1152, 4, 6, 0.0), (384, 256, 250, 5, 0.0), (512, 512, 127, 127, 0.0), (384, 384, 120, 4, 0.003),
    (256, 256, 120, 12, 0.05)])
def test_row_to_fp8_col_random_codes_and_scale_spreads(M, K, center, spread, nan):
    q, sf = synth.random_mxfp4(M, K, seed=M + K + spread, scale_center=center, scale_spread=spread,
                               nan_scale_frac=nan)
    q, sf = q.numpy().copy(), sf.numpy()
    q[:, 5] = 0                                   # two all-zero columns
    q[7::32, :] &= 0x88                           # rows of signed zeros
    check_row_to_fp8_col(q, sf)


def test_row_to_fp8_col_every_shift_and_code():
    # row r of each 128-row group sits d = r binades under the group maximum (d = 0..127, then the same
    # with larger steps down to byte 0); the 16 codes repeat along k; both halves of a 256-row tile differ
    K = 256
    nib = np.tile(np.arange(16, dtype=np.uint8), K // 16)
    qrow = (nib[0::2] | (nib[1::2] << 4)).astype(np.uint8)
    qs, sfs = [], []
    for bmax, step in ((254, 1), (140, 1), (254, 2), (41, 1), (20, 1), (6, 1), (3, 1), (0, 1)):
        b = np.clip(bmax - step * np.arange(128), 0, 254).astype(np.uint8)
        sf = np.repeat(b[:, None], K // 32, axis=1)
        sf[:, 1] = b[::-1]                        # the maximum at the other end of the group
        sf[:, 2] = np.roll(b, 37)
        qs.append(np.repeat(qrow[None], 128, axis=0))
        sfs.append(sf)
    check_row_to_fp8_col(np.concatenate(qs), np.concatenate(sfs))


def test_row_to_fp8_col_on_quantized_swiglu():
    x8, s = synth.swiglu_fp8(1024, 2048, seed=1)
    q, sf = par.quant(x8.numpy(), s.numpy())
    check_row_to_fp8_col(q, sf)


def test_row_to_fp8_col_grouped():
    off = torch.tensor([0, 0, 384, 384, 512, 1152, 1152], dtype=torch.int32)
    q, sf = synth.random_mxfp4(1152, 384, seed=6, scale_center=125, scale_spread=6, nan_scale_frac=0.001)
    q, sf = q.numpy(), sf.numpy()
    x, xs = mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), off.to(DEV))
    wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off.numpy())
    assert_same(host(xs)[:wxs.size], wxs, "grouped row->FP8 col: group scales")
    assert_same(host(x), wx, "grouped row->FP8 col: E4M3 bytes")
    # one expert holding everything equals the flat call
    one = torch.tensor([0, 1152], dtype=torch.int32)
    x1, xs1 = mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), one.to(DEV))
    fx, fxs = ref.row_to_fp8_col(q, sf)
    assert_same(host(xs1)[:fxs.size].reshape(fxs.shape), fxs, "single expert: group scales")
    assert_same(host(x1).reshape(fx.shape), fx, "single expert: E4M3 bytes")


def test_row_to_fp8_col_empty_and_argument_errors():
    q = torch.zeros((0, 128), dtype=torch.uint8, device=DEV)
    sf = torch.zeros((0, 8), dtype=torch.uint8, device=DEV)
    x, xs = mx.mxfp4_row_to_fp8_col(q, sf)
    assert x.shape == (256, 0) and xs.shape == (256, 0)
    q = torch.zeros((96, 128), dtype=torch.uint8, device=DEV)
    sf = torch.zeros((96, 8), dtype=torch.uint8, device=DEV)
    with pytest.raises(ValueError):
        mx.mxfp4_row_to_fp8_col(q, sf)                                  # M % 128 != 0: stopped by the binding
    q = torch.zeros((128, 128), dtype=torch.uint8, device=DEV)
    sf = torch.zeros((128, 8), dtype=torch.uint8, device=DEV)
    xbuf = torch.zeros(256 * 128 + 16, dtype=torch.uint8, device=DEV)
    with pytest.raises(mx.Mxfp4Error) as e:
        mx.mxfp4_row_to_fp8_col(q, sf, x_col=xbuf[1:1 + 256 * 128])     # misaligned output
    assert e.value.status == -3


def test_grouped_more_experts_than_a_wave():
    # 150 experts (the lookup works on 64 at a time), many empty, sizes 0..5 blocks of 128 rows
    rng = np.random.default_rng(12)
    counts = rng.integers(0, 6, size=150) * 128
    counts[rng.random(150) < 0.4] = 0
    counts[[0, 63, 64, 127, 128, 149]] = [0, 256, 128, 0, 384, 128]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    M, K = int(off[-1]), 256
    q, sf = synth.random_mxfp4(M, K, seed=13, scale_center=124, scale_spread=5)
    q, sf = q.numpy(), sf.numpy()
    offd = torch.from_numpy(off).to(DEV)
    qc, sc = mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), offd)
    wqc, wsc = ref.row_to_col_grouped(q, sf, off)
    assert_same(host(sc)[:wsc.size], wsc, "150 experts row->col scales")
    assert_same(host(qc)[:wqc.size], wqc, "150 experts row->col nibbles")
    x, xs = mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), offd)
    wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off)
    assert_same(host(xs)[:wxs.size], wxs, "150 experts row->FP8 col scales")
    assert_same(host(x), wx, "150 experts row->FP8 col bytes")


def test_grouped_tile_order_over_many_experts_and_column_tiles():
    """200 experts in four lane-parallel steps of the lookup, three column tiles, lengths from empty to more
    row tiles than a macro block of the tile order holds (9000 rows = 36 tiles): every tile of every expert has
    to be visited exactly once by the order that walks macro blocks inside each expert."""
    rng = np.random.default_rng(77)
    kinds = [0, 0, 1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 511, 513, 1025]
    counts = rng.choice(kinds, size=200)
    counts[17], counts[130] = 9000, 8192 + 256
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    M, K = int(off[-1]), 768
    q, sf = synth.random_mxfp4(M, K, seed=78, scale_center=121, scale_spread=6, nan_scale_frac=0.0005)
    q, sf = q.numpy(), sf.numpy()
    offd = torch.from_numpy(off).to(DEV)
    qc, sc = mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), offd, offsets_host=off)
    wqc, wsc = ref.row_to_col_grouped(q, sf, off)
    assert_same(host(sc), wsc, "200 experts row->col scales")
    assert_same(host(qc), wqc, "200 experts row->col nibbles")
    for requant in (False, True):
        x, xs = mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), offd, requant=requant, offsets_host=off)
        wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off, requant=requant)
        assert_same(host(xs), wxs, f"200 experts row->FP8 col scales, requant={requant}")
        assert_same(host(x), wx, f"200 experts row->FP8 col bytes, requant={requant}")


def test_grouped_with_the_largest_number_of_experts():
    # 1024 experts, the most the C ABI takes (16 lane-parallel steps of the lookup): ragged sizes 0..300,
    # many empty, the first and last experts of every step of 64 non-empty
    E = 1024
    rng = np.random.default_rng(14)
    counts = rng.integers(0, 301, size=E)
    counts[rng.random(E) < 0.5] = 0
    counts[::64] = 33
    counts[63::64] = 257
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    M, K = int(off[-1]), 128
    q, sf = synth.random_mxfp4(M, K, seed=15, scale_center=124, scale_spread=5)
    q, sf = q.numpy(), sf.numpy()
    offd = torch.from_numpy(off).to(DEV)
    qc, sc = mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), offd)
    wqc, wsc = ref.row_to_col_grouped(q, sf, off)
    assert_same(host(sc).reshape(-1)[:wsc.size], wsc, "1024 experts row->col scales")
    assert_same(host(qc).reshape(-1)[:wqc.size], wqc, "1024 experts row->col nibbles")
    for requant in (False, True):
        x, xs = mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), offd, requant=requant)
        wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off, requant=requant)
        assert_same(host(xs).reshape(-1)[:wxs.size], wxs, f"1024 experts row->FP8 col scales, requant={requant}")
        assert_same(host(x).reshape(-1)[:wx.size], wx, f"1024 experts row->FP8 col bytes, requant={requant}")
    with pytest.raises(mx.Mxfp4Error) as e:
        mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), torch.zeros(1026, dtype=torch.int32, device=DEV))
    assert e.value.status == -4


@pytest.mark.parametrize("K", [256, 384])
def test_row_to_fp8_col_ragged_splits_without_padding(K):
    # any T_e: partial last scale groups, partial tiles, unaligned rows; outputs are checked together
    # with guard bytes around them
    T = [5, 0, 128, 256, 31, 257, 1, 300, 16, 15, 17, 511, 0, 130]
    off = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    M = int(off[-1])
    q, sf = synth.random_mxfp4(M, K, seed=31 + K, scale_center=118, scale_spread=9, nan_scale_frac=0.002)
    q, sf = q.numpy(), sf.numpy()
    wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off)
    guard = 4096
    xbuf = torch.full((guard + wx.size + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    sbuf = torch.full((guard + wxs.size + guard,), -7.0, dtype=torch.float32, device=DEV)
    mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), torch.from_numpy(off).to(DEV),
                                    x_col=xbuf[guard:guard + wx.size], x_col_scale=sbuf[guard:guard + wxs.size],
                                    offsets_host=off)
    xb, sb = host(xbuf), host(sbuf)
    assert (xb[:guard] == 0xA5).all() and (xb[guard + wx.size:] == 0xA5).all(), "bytes written outside x_col"
    assert (sb[:guard] == -7.0).all() and (sb[guard + wxs.size:] == -7.0).all(), "floats written outside x_col_scale"
    assert_same(sb[guard:guard + wxs.size], wxs, "ragged row->FP8 col: group scales")
    assert_same(xb[guard:guard + wx.size], wx, "ragged row->FP8 col: E4M3 bytes")


# ------------------------------------------------------------------ the same under the re-quantization reading

def check_row_to_fp8_col_requant(q, sf):
    x, xs = mx.mxfp4_row_to_fp8_col(dev(q), dev(sf), requant=True)
    wx, wxs = ref.row_to_fp8_col(q, sf, requant=True)
    assert_same(host(xs), wxs, "row->FP8 col (requant): group scales")
    assert_same(host(x), wx, "row->FP8 col (requant): E4M3 bytes")
    check_wide("requant", functools.partial(mx.mxfp4_row_to_fp8_col, requant=True), q, sf, wx, wxs)


@pytest.mark.parametrize("M,K,center,spread,nan", [
    (256, 256, 127, 0, 0.0), (384, 384, 127, 3, 0.0), (128, 128, 100, 8, 0.0), (640, 640, 30, 30, 0.0),
    (128, 1152, 4, 6, 0.0), (384, 256, 250, 5, 0.0), (512, 512, 127, 127, 0.0), (384, 384, 120, 4, 0.003),
    (256, 256, 120, 12, 0.05), (256, 384, 9, 4, 0.0)])
def test_row_to_fp8_col_requant_random_codes_and_scale_spreads(M, K, center, spread, nan):
    q, sf = synth.random_mxfp4(M, K, seed=M + K + spread + 1, scale_center=center, scale_spread=spread,
                               nan_scale_frac=nan)
    q, sf = q.numpy().copy(), sf.numpy()
    q[:, 5] = 0                                   # two all-zero columns
    q[7::32, :] &= 0x88                           # rows of signed zeros
    q[:, 16:20] = np.where(np.random.default_rng(M).random((M, 4)) < 0.95, q[:, 16:20] & 0x88, q[:, 16:20])
    check_row_to_fp8_col_requant(q, sf)


def test_row_to_fp8_col_requant_every_shift_and_code():
    K = 256
    nib = np.tile(np.arange(16, dtype=np.uint8), K // 16)
    qrow = (nib[0::2] | (nib[1::2] << 4)).astype(np.uint8)
    qs, sfs = [], []
    for bmax, step in ((254, 1), (252, 1), (140, 1), (254, 2), (41, 1), (20, 1), (9, 1), (6, 1), (3, 1), (0, 1)):
        b = np.clip(bmax - step * np.arange(128), 0, 254).astype(np.uint8)
        sf = np.repeat(b[:, None], K // 32, axis=1)
        sf[:, 1] = b[::-1]
        sf[:, 2] = np.roll(b, 37)
        qq = np.repeat(qrow[None], 128, axis=0).copy()
        qq[::3, 40:48] &= 0x88                    # columns whose largest element is not in the largest-scale row
        qs.append(qq)
        sfs.append(sf)
    check_row_to_fp8_col_requant(np.concatenate(qs), np.concatenate(sfs))


def test_row_to_fp8_col_requant_on_quantized_swiglu():
    x8, s = synth.swiglu_fp8(1024, 2048, seed=1)
    q, sf = par.quant(x8.numpy(), s.numpy())
    check_row_to_fp8_col_requant(q, sf)


@pytest.mark.parametrize("K", [256, 384])
def test_row_to_fp8_col_requant_ragged_splits(K):
    T = [5, 0, 128, 256, 31, 257, 1, 300, 16, 15, 17, 511, 0, 130] + [0] * 60 + [128, 3]
    off = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    M = int(off[-1])
    q, sf = synth.random_mxfp4(M, K, seed=41 + K, scale_center=118, scale_spread=9, nan_scale_frac=0.002)
    q, sf = q.numpy(), sf.numpy()
    sf[40:44, 0] = 254                                                    # beyond FP32 inside a partial tile
    wx, wxs = ref.row_to_fp8_col_grouped(q, sf, off, requant=True)
    guard = 4096
    xbuf = torch.full((guard + wx.size + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    sbuf = torch.full((guard + wxs.size + guard,), -7.0, dtype=torch.float32, device=DEV)
    mx.mxfp4_row_to_fp8_col_grouped(dev(q), dev(sf), torch.from_numpy(off).to(DEV), x_col=xbuf[guard:guard + wx.size],
                                    x_col_scale=sbuf[guard:guard + wxs.size], requant=True, offsets_host=off)
    xb, sb = host(xbuf), host(sbuf)
    assert (xb[:guard] == 0xA5).all() and (xb[guard + wx.size:] == 0xA5).all(), "bytes written outside x_col"
    assert (sb[:guard] == -7.0).all() and (sb[guard + wxs.size:] == -7.0).all(), "floats written outside x_col_scale"
    assert_same(sb[guard:guard + wxs.size], wxs, "ragged row->FP8 col (requant): group scales")
    assert_same(xb[guard:guard + wx.size], wx, "ragged row->FP8 col (requant): E4M3 bytes")


# ------------------------------------------------------------------ the quantizer with the routing turned around

def test_quant_scatter_equals_gather_and_leaves_other_rows_alone():
    rng = np.random.default_rng(8)
    M, K, fan = 300, 768, 4
    x8, s = synth.student_t_fp8(M, K, seed=3)
    x8, s = x8.numpy(), s.numpy()
    M_out = M * fan + 11
    perm = rng.permutation(M_out)[:M * fan].reshape(M, fan).astype(np.int32)
    perm[5, 1] = -1
    perm[9, 0] = M_out + 3
    q0 = rng.integers(0, 256, size=(M_out, K // 2)).astype(np.uint8)
    sf0 = rng.integers(0, 255, size=(M_out, K // 32)).astype(np.uint8)
    wq, wsf = ref.quant_from_fp8_scatter(x8, s, perm, M_out, q=q0.copy(), sf=sf0.copy())
    q, sf = mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(perm), M_out, q=dev(q0), sf=dev(sf0))
    assert_same(host(sf), wsf, "scatter: scale bytes")
    assert_same(host(q), wq, "scatter: nibbles")
    # into per-token records (nibbles then scales), fan-out 1 = a permutation
    rec = K // 2 + K // 32
    one = rng.permutation(M).astype(np.int32).reshape(M, 1)
    buf = torch.zeros(M * rec, dtype=torch.uint8, device=DEV)
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(one), M, q=buf, sf=buf[K // 2:], ld_q=rec, ld_sf=rec)
    got = host(buf).reshape(M, rec)
    fq, fsf = ref.quant_from_fp8(x8, s)
    assert_same(got[one[:, 0], : K // 2], fq, "scatter into records: nibbles")
    assert_same(got[one[:, 0], K // 2:], fsf, "scatter into records: scale bytes")


@pytest.mark.parametrize("K,M,fan,pad,whole", [
    (512, 37, 8, 0, False), (7168, 133, 8, 0, False), (7168, 64, 11, 32, False), (640, 203, 3, 12, False), (1536, 50, 1, 0, False),
    (16384, 9, 2, 0, False), (32768, 5, 9, 0, False), (2048, 130, 8, 16, False),
    (7168, 233, 8, 0, True), (7168, 221, 11, 32, True), (16384, 97, 2, 0, True), (32768, 49, 9, 0, True), (6272, 255, 3, 16, True),
    (2048, 3085, 8, 16, True), (2176, 2894, 3, 0, True)])
def test_quant_scatter_whole_rows_through_lds(K, M, fan, pad, whole):
    """Outputs whose rows start on 16-byte boundaries.  From 1.5 Mi elements of rows of 6144 and longer, and from 6 Mi of shorter ones
    of 2048 on, a workgroup or a wave writes whole rows out of LDS; smaller launches, and the rest, are a lane's per chunk.  Records
    of K/2 + K/32 bytes (plus padding), scale bytes as 16-byte pieces (K % 512 == 0) or dwords, fan-outs beyond the eight
    prefetched indices, row counts that end inside a workgroup, entries that point nowhere; the bytes between and around
    the records stay as they were."""
    assert (M * K > (6 << 20 if K < 6144 else 3 << 19)) == whole
    rng = np.random.default_rng(K + M)
    x8, s = synth.student_t_fp8(M, K, seed=K % 97)
    x8, s = x8.numpy(), s.numpy()
    x8[rng.integers(0, M), rng.integers(0, K)] = 0x7F                   # a NaN block
    x8[rng.integers(0, M)] = 0                                          # a zero row
    M_out = M * fan + 7
    dst = rng.permutation(M_out)[:M * fan].reshape(M, fan).astype(np.int32)
    nowhere = rng.random(dst.shape) < 0.05
    dst[nowhere] = rng.choice(np.array([-1, -7, M_out, 2 ** 31 - 1], np.int32), size=int(nowhere.sum()))
    rec = (K // 2 + K // 32 + 15) // 16 * 16 + pad // 16 * 16
    assert rec % 16 == 0
    guard = 256
    buf = torch.full((guard + M_out * rec + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    recs = buf[guard:guard + M_out * rec]
    assert recs.data_ptr() % 16 == 0
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), M_out, q=recs, sf=recs[K // 2:], ld_q=rec, ld_sf=rec)
    got = host(buf)
    assert (got[:guard] == 0xA5).all() and (got[guard + M_out * rec:] == 0xA5).all(), "written outside the records"
    got = got[guard:guard + M_out * rec].reshape(M_out, rec)
    wq, wsf = ref.quant_from_fp8_scatter(x8, s, dst, M_out, q=np.full((M_out, K // 2), 0xA5, np.uint8),
                                         sf=np.full((M_out, K // 32), 0xA5, np.uint8))
    assert_same(got[:, K // 2:K // 2 + K // 32], wsf, "scatter through LDS: scale bytes")
    assert_same(got[:, :K // 2], wq, "scatter through LDS: nibbles")
    assert (got[:, K // 2 + K // 32:] == 0xA5).all(), "padding of the records written"


# ------------------------------------------------------------------ streams and graphs

def test_side_stream_and_graph_replays():
    # the library only enqueues kernels on the stream it is given: it runs on a side stream and under
    # HIP graph capture; every replay (with new input contents between replays) equals the eager result
    M, K = 512, 1024
    gen = [synth.student_t_fp8(M, K, seed=sd) for sd in (0, 1, 2)]
    x8 = torch.empty((M, K), dtype=torch.uint8, device=DEV)
    s = torch.empty((M, K // 128), dtype=torch.float32, device=DEV)
    q = torch.empty((M, K // 2), dtype=torch.uint8, device=DEV)
    sf = torch.empty((M, K // 32), dtype=torch.uint8, device=DEV)
    xb = torch.empty((M, K), dtype=torch.uint8, device=DEV)
    sb = torch.empty((M, K // 128), dtype=torch.float32, device=DEV)
    qc = torch.empty((K, M // 2), dtype=torch.uint8, device=DEV)
    sc = torch.empty((K, M // 32), dtype=torch.uint8, device=DEV)
    xc = torch.empty((K, M), dtype=torch.uint8, device=DEV)
    xcs = torch.empty((K, M // 128), dtype=torch.float32, device=DEV)

    def path(stream):
        mx.mxfp4_quant_from_fp8(x8, s, q=q, sf=sf, stream=stream)
        mx.mxfp4_dequant_to_fp8(q, sf, x=xb, x_scale=sb, stream=stream)
        mx.mxfp4_row_to_col(q, sf, q_col=qc, sf_col=sc, stream=stream)
        mx.mxfp4_row_to_fp8_col(q, sf, x_col=xc, x_col_scale=xcs, stream=stream)

    side = torch.cuda.Stream()
    x8.copy_(gen[0][0])
    s.copy_(gen[0][1])
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        path(side)                                      # warm-up on the side stream, eager
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        path(torch.cuda.current_stream())
    for xs8, ss in gen:
        xh, sh = xs8.numpy(), ss.numpy()
        x8.copy_(xs8)
        s.copy_(ss)
        for t in (q, sf, xb, sb, qc, sc, xc, xcs):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        wq, wsf = ref.quant_from_fp8(xh, sh)
        wx, wxs = ref.dequant_to_fp8(wq, wsf)
        wqc, wsc = ref.row_to_col(wq, wsf)
        wxc, wxcs = ref.row_to_fp8_col(wq, wsf)
        for got, want, name in ((q, wq, "q"), (sf, wsf, "sf"), (xb, wx, "x"), (sb, wxs, "x_scale"), (qc, wqc, "q_col"),
                                (sc, wsc, "sf_col"), (xc, wxc, "x_col"), (xcs, wxcs, "x_col_scale")):
            assert_same(host(got), want, f"graph replay: {name}")


@pytest.mark.parametrize("K", [256, 384])
def test_row_to_col_ragged_splits_without_padding(K):
    # any T_e: partial last blocks, partial tiles, odd lengths, unaligned k-rows; guard bytes around the outputs
    T = [5, 0, 32, 256, 31, 257, 1, 300, 16, 15, 17, 511, 0, 130, 33] + [0] * 60 + [64, 3]
    off = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    M = int(off[-1])
    q, sf = synth.random_mxfp4(M, K, seed=51 + K, scale_center=120, scale_spread=8, nan_scale_frac=0.002)
    q, sf = q.numpy(), sf.numpy()
    sf[40:44, 0] = 254                                                    # beyond FP32 inside a partial tile
    wqc, wsc = ref.row_to_col_grouped(q, sf, off)
    guard = 4096
    qbuf = torch.full((guard + wqc.size + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    sbuf = torch.full((guard + wsc.size + guard,), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_row_to_col_grouped(dev(q), dev(sf), torch.from_numpy(off).to(DEV), q_col=qbuf[guard:guard + wqc.size],
                                sf_col=sbuf[guard:guard + wsc.size], offsets_host=off)
    qb, sb = host(qbuf), host(sbuf)
    assert (qb[:guard] == 0xA5).all() and (qb[guard + wqc.size:] == 0xA5).all(), "bytes written outside q_col"
    assert (sb[:guard] == 0x5A).all() and (sb[guard + wsc.size:] == 0x5A).all(), "bytes written outside sf_col"
    assert_same(sb[guard:guard + wsc.size], wsc, "ragged row->col: column scales")
    assert_same(qb[guard:guard + wqc.size], wqc, "ragged row->col: nibbles")
