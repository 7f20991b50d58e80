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
@pytest.mark.parametrize("K,M,fan", [(1920, 37, 3), (2048, 37, 3), (2176, 9, 1), (5120, 21, 8), (6016, 6, 9),
                                     (6144, 13, 1), (6144, 13, 2), (6272, 5, 9), (7680, 7, 1), (7808, 7, 1),
                                     (8192, 5, 1), (16896, 3, 1), (98304, 2, 2)])
def test_scatter_kernels(K, M, fan, layout):
    """One lane per chunk, one wave per row (several segments from 7681 elements on) and one workgroup per row; fan-outs
    of 1, 2 and past the eight indices read ahead; scale bytes as 16-byte pieces and as dwords."""
    rng, x8, s, wq, wsf = source(M, K, K + fan)
    M_out = M * fan + 5
    dst = rng.permutation(M_out)[: M * fan].reshape(M, fan).astype(np.int32)
    nowhere = rng.random(dst.shape) < 0.05
    dst[nowhere] = rng.choice(np.array([-1, M_out, 2 ** 31 - 1], np.int32), size=int(nowhere.sum()))
    buf, q, sf, ld_q, ld_sf, at = outputs(M_out, K, layout)
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), M_out, q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    src, _ = np.nonzero(~nowhere)
    check(buf, at, ld_q, ld_sf, K, dst[~nowhere], wq[src], wsf[src])
