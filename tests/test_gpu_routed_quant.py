"""GPU parity of the routed quantizers on both sides of every rule that picks a kernel: a gathered or scattered row is
the oracle's flat row, and bytes that no row owns keep their contents."""
import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par
from paper_2603_02731_amd import synth
from tests.test_gpu_parity import DEV, assert_same, dev, host

pytestmark = pytest.mark.gpu
GUARD = 256


def source(M, K, seed):
    """Activations with a NaN block and a zero row, and the oracle's packed rows plus one zero row at the end."""
    rng = np.random.default_rng(seed)
    x8, s = synth.student_t_fp8(M, K, seed=seed)
    x8, s = x8.numpy(), s.numpy()
    x8[rng.integers(0, M), rng.integers(0, K)] = 0x7F
    x8[rng.integers(0, M)] = 0
    q, sf = par.quant(x8, s)
    zero = np.zeros((1, q.shape[1]), np.uint8), np.zeros((1, sf.shape[1]), np.uint8)
    return rng, x8, s, np.concatenate([q, zero[0]]), np.concatenate([sf, zero[1]])


def outputs(rows, K, layout):
    """(buffer, q, sf, ld_q, ld_sf, views): records on 16-byte boundaries with a gap, or two planes with rows on
    8- and 4-byte boundaries; guard bytes around all of it."""
    nq, ns = K // 2, K // 32
    if layout == "records":
        ld_q = ld_sf = (nq + ns + 15) // 16 * 16 + 16
        at_q, at_sf, size = GUARD, GUARD + nq, GUARD + rows * ld_q
    else:
        step = {"planes": 16, "planes8": 8}[layout]
        ld_q, ld_sf = nq + step, ns + step // 2
        at_q, at_sf = GUARD, (GUARD + rows * ld_q + 15) // 16 * 16
        size = at_sf + rows * ld_sf
    buf = torch.full((size + GUARD,), 0xA5, dtype=torch.uint8, device=DEV)
    return buf, buf[at_q:], buf[at_sf:], ld_q, ld_sf, (at_q, at_sf)


def check(buf, at, ld_q, ld_sf, K, rows, wq, wsf):
    """wq / wsf: oracle rows; rows: which output rows they are.  Everything else in buf is still 0xA5."""
    want = np.full(buf.numel(), 0xA5, np.uint8)
    for start, ld, w in ((at[0], ld_q, wq), (at[1], ld_sf, wsf)):
        place = start + rows.astype(np.int64)[:, None] * ld + np.arange(w.shape[1])[None, :]
        want[place] = w
    assert_same(host(buf), want, "routed rows")


@pytest.mark.parametrize("layout", ["records", "planes", "planes8"])
@pytest.mark.parametrize("K,M,fan", [(1920, 37, 3), (2048, 37, 3), (2048, 1023, 2), (2048, 1024, 2), (2176, 1025, 3),
                                     (2176, 9, 1), (5120, 21, 8), (6016, 6, 9), (6016, 1030, 1), (6144, 1024, 1),
                                     (6144, 13, 1), (6144, 13, 2), (6272, 5, 9), (7680, 1024, 1), (7808, 512, 1),
                                     (8192, 512, 1), (8192, 511, 1), (16896, 342, 1), (98304, 2, 2), (98304, 79, 1)])
def test_scatter_kernels(K, M, fan, layout):
    """One lane per chunk, one wave per row (from 1024 rows on; several segments of a row count, from 7681 elements on) and
    one workgroup per row; fan-outs of 1, 2 and past the eight indices read ahead; scale bytes as 16-byte pieces and as dwords."""
    rng, x8, s, wq, wsf = source(M, K, K + fan)
    M_out = M * fan + 5
    dst = rng.permutation(M_out)[: M * fan].reshape(M, fan).astype(np.int32)
    nowhere = rng.random(dst.shape) < 0.05
    dst[nowhere] = rng.choice(np.array([-1, M_out, 2 ** 31 - 1], np.int32), size=int(nowhere.sum()))
    buf, q, sf, ld_q, ld_sf, at = outputs(M_out, K, layout)
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), M_out, q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    src, _ = np.nonzero(~nowhere)
    check(buf, at, ld_q, ld_sf, K, dst[~nowhere], wq[src], wsf[src])


def index_of(kind, M, n, rng):
    """int32 [n] gather indices into M source rows."""
    idx = (np.arange(n) % M).astype(np.int32)
    rng.shuffle(idx)
    if kind == "padded":        # every fifth slot unused, some far outside
        idx[::5] = -1
        idx[7::50] = M
        idx[9::50] = 2 ** 31 - 1
    elif kind == "crowd":       # a quarter of the slots name one row: its owner's rows are dealt out
        idx[rng.random(n) < 0.25] = 5
    elif kind == "hidden":      # a crowd where no sample is taken (every sixteenth slot): the list overflows
        idx[np.arange(n) % 16 != 0] = np.where(rng.random(n) < 0.5, 3, idx)[np.arange(n) % 16 != 0]
    elif kind == "one":         # all slots name the last row
        idx[:] = M - 1
    elif kind == "sorted":
        idx.sort()
    return idx


@pytest.mark.parametrize("layout", ["records", "planes8"])
@pytest.mark.parametrize("K,M,n,kind", [
    (2048, 1024, 19175, "mixed"), (2048, 1024, 19174, "mixed"),                     # work just above and below the rule
    (2048, 1023, 21846, "mixed"), (1920, 1024, 32768, "mixed"),                     # too few rows; too short rows
    (7168, 4200, 8401, "sorted"), (7168, 4200, 8399, "sorted"),                     # two copies a row, and just under
    (2176, 1300, 30001, "padded"), (2048, 1029, 40003, "crowd"), (2048, 1024, 30010, "hidden"),
    (7808, 1030, 5003, "padded"), (8192, 1024, 5003, "mixed"), (2048, 2047, 24577, "one")])
def test_gather_by_owners(K, M, n, kind, layout):
    """Both sides of the rule for gathering by owners, ends of the index that are no whole quad, an index that starts
    at any multiple of 4 bytes, unused slots, crowds that the sample sees and ones that it does not."""
    rng, x8, s, wq, wsf = source(M, K, K + n)
    idx = index_of(kind, M, n, rng)
    buf, q, sf, ld_q, ld_sf, at = outputs(n, K, layout)
    padded = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    padded[1:] = dev(idx)
    mx.mxfp4_quant_from_fp8(dev(x8), dev(s), padded[1:], q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    src = np.where((idx >= 0) & (idx < M), idx, M)
    check(buf, at, ld_q, ld_sf, K, np.arange(n), wq[src], wsf[src])


def test_gather_by_owners_under_capture():
    """Replays of a captured gather, with the inputs changed and eager work between the replays."""
    K, M, n = 2048, 1024, 20480
    rng, x8, s, _, _ = source(M, K, 1)
    x, xs = dev(x8), dev(s)
    idx = dev(index_of("padded", M, n, rng))
    q, sf = mx.mxfp4_quant_from_fp8(x, xs, idx)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)
    for i in range(4):
        y8, ys = synth.student_t_fp8(M, K, seed=10 + i)
        x.copy_(y8)
        xs.copy_(ys)
        idx.copy_(idx.roll(i * 977))
        want = mx.mxfp4_quant_from_fp8(x, xs, idx)
        q.zero_()
        sf.fill_(7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(q, want[0]) and torch.equal(sf, want[1]), f"replay {i}"
