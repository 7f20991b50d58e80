"""GPU parity of the grouped row->col conversion on both sides of the sizes from which un-padded splits are launched with
three workgroups per compute unit (32768 x 7168 elements, 1024 rows per expert, total rows no multiple of 128)."""
import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par
from paper_2603_02731_amd import synth
from tests.test_gpu_parity import DEV, assert_same, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,E", [(32769, 32), (32767, 31), (33000, 33), (32896, 4)])  # above; too small; too many; padded total
def test_row_to_col_around_the_limit(M, E):
    K = 7168
    rng = np.random.default_rng(M)
    off = np.concatenate([[0], np.sort(rng.integers(0, M + 1, E - 1)), [M]]).astype(np.int32)
    q, sf = synth.random_mxfp4(M, K, seed=M, scale_spread=5, device=DEV)
    rows = np.diff(off)
    n2, n32 = K * int(((rows + 1) // 2).sum()), K * int(((rows + 31) // 32).sum())
    guard = 4096
    qc = torch.full((n2 + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    sc = torch.full((n32 + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    mx.mxfp4_row_to_col_grouped(q, sf, torch.from_numpy(off).to(DEV), q_col=qc[:n2], sf_col=sc[:n32], offsets_host=off.tolist())
    assert bool((qc[n2:] == 0xA5).all()) and bool((sc[n32:] == 0xA5).all())
    # experts of every kind against the oracle: the shortest, the longest and the last
    picks = {int(np.argmin(np.where(rows > 0, rows, M + 1))), int(rows.argmax()), E - 1}
    a2 = np.concatenate([[0], np.cumsum((rows + 1) // 2)]) * K
    a32 = np.concatenate([[0], np.cumsum((rows + 31) // 32)]) * K
    for e in sorted(picks):
        lo, T = int(off[e]), int(rows[e])
        if T == 0:
            continue
        whole = T // 32 * 32
        gq = host(qc[a2[e]:a2[e + 1]]).reshape(K, -1)
        gs = host(sc[a32[e]:a32[e + 1]]).reshape(K, -1)
        if whole:
            wq, ws = par.row_to_col(host(q[lo:lo + whole]), host(sf[lo:lo + whole]))
            assert_same(gq[:, :whole // 2], wq, f"expert {e} nibbles")
            assert_same(gs[:, :whole // 32], ws, f"expert {e} scale bytes")
        if T > whole:  # the last, shorter block: rows of zeros behind it change neither scale nor codes
            tq = np.zeros((32, K // 2), np.uint8)
            ts = np.zeros((32, K // 32), np.uint8)
            tq[:T - whole], ts[:T - whole] = host(q[lo + whole:lo + T]), host(sf[lo + whole:lo + T])
            wq, ws = par.row_to_col(tq, ts)
            assert_same(gq[:, whole // 2:], wq[:, : (T - whole + 1) // 2], f"expert {e} last nibbles")
            assert_same(gs[:, whole // 32:], ws, f"expert {e} last scale bytes")
