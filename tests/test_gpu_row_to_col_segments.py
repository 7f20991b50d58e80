"""GPU parity of row->col where tiles write whole 64-byte segments of the output (one large matrix whose k-rows are no whole
segments, on both sides of the rule), of large splits of any length, and of small launches of many un-padded splits, whose k-rows
leave in aligned pieces."""
import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par
from oracle import ref
from paper_2603_02731_amd import synth
from tests.rules import aligned_pieces
from tests.test_gpu_parity import DEV, UNITS, assert_same, host

pytestmark = pytest.mark.gpu


def special_rows(sf, at):
    """NaN bytes, bytes beyond FP32 and the smallest ones in the rows from `at` on, in some k-blocks only."""
    sf[at, 0], sf[at + 3, 2] = 255, 253
    sf[at + 40:at + 44, 1], sf[at + 70:at + 105, 3] = 254, 0


def check_matrix(q, sf, gq, gs, what):
    """One matrix or expert of any number of rows against the oracle, a last block of fewer than 32 rows included."""
    T, K = q.shape[0], 2 * q.shape[1]
    whole = T // 32 * 32
    gq, gs = gq.reshape(K, -1), gs.reshape(K, -1)
    if whole:
        wq, ws = par.row_to_col(q[:whole], sf[:whole])
        assert_same(gs[:, :whole // 32], ws, what + " scale bytes")
        assert_same(gq[:, :whole // 2], wq, what + " nibbles")
    if T > whole:
        tq, ts = np.zeros((32, K // 2), np.uint8), np.zeros((32, K // 32), np.uint8)
        tq[:T - whole], ts[:T - whole] = q[whole:], sf[whole:]
        wq, ws = par.row_to_col(tq, ts)
        assert_same(gs[:, whole // 32:], ws, what + " last scale bytes")
        assert_same(gq[:, whole // 2:], wq[:, : (T - whole + 1) // 2], what + " last nibbles")


@pytest.mark.parametrize("M,K,off", [(45088, 4096, 0), (45056, 4096, 16), (25760, 7168, 48), (180224 + 96, 1024, 0),
                                     (45024, 4096, 0), (45184, 4096, 32), (24608, 7552, 0)])
def test_one_matrix(M, K, off):
    """Above and below 176 Mi elements; k-rows on 16, 32 and 64 bytes, outputs off a segment; an odd number of 128 columns."""
    q, sf = synth.random_mxfp4(M, K, seed=M, scale_spread=5, device=DEV)
    special_rows(sf, 130)
    special_rows(sf, 256 * 40 - 60)
    n, ns = K * (M // 2), K * (M // 32)
    qb = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    sb = torch.full((ns + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_row_to_col(q, sf, q_col=qb[off:off + n].view(K, M // 2), sf_col=sb[:ns].view(K, M // 32))
    assert bool((qb[:off] == 0xA5).all()) and bool((qb[off + n:] == 0xA5).all()) and bool((sb[ns:] == 0x5A).all())
    wq, ws = par.row_to_col(host(q), host(sf))
    assert_same(host(sb)[:ns].reshape(K, -1), ws, f"scale bytes {M} {K}")
    assert_same(host(qb)[off:off + n].reshape(K, -1), wq, f"nibbles {M} {K}")


@pytest.mark.parametrize("rows,K", [([8191, 15, 0, 20001, 4999], 7168), ([33000, 7], 7552), ([9000, 9001, 257, 1, 14603], 7168),
                                    ([8192, 16400, 8208, 48], 7168)])  # the last one's total is a multiple of 16
def test_large_splits(rows, K):
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    M = int(off[-1])
    q, sf = synth.random_mxfp4(M, K, seed=M, scale_spread=5, device=DEV)
    special_rows(sf, 256 * 9 - 100)
    n, ns = K * sum((r + 1) // 2 for r in rows), K * sum((r + 31) // 32 for r in rows)
    qb = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    sb = torch.full((ns + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_row_to_col_grouped(q, sf, torch.from_numpy(off).to(DEV), q_col=qb[:n], sf_col=sb[:ns], offsets_host=off.tolist())
    assert bool((qb[n:] == 0xA5).all()) and bool((sb[ns:] == 0x5A).all())
    q, sf, qb, sb = host(q), host(sf), host(qb), host(sb)
    a = b = 0
    for e, r in enumerate(rows):
        na, nb = K * ((r + 1) // 2), K * ((r + 31) // 32)
        if r:
            check_matrix(q[off[e]:off[e + 1]], sf[off[e]:off[e + 1]], qb[a:a + na], sb[b:b + nb], f"expert {e} of {r} rows")
        a, b = a + na, b + nb


@pytest.mark.parametrize("rows", [[1, 31, 32, 33, 29, 30], [255, 256, 257, 511, 0, 513, 37], [1023, 2, 225, 226, 227, 240, 241]])
@pytest.mark.parametrize("K,more", [(384, 0), (256, 250), (128, 310)])
@pytest.mark.parametrize("off", [0, 16])
def test_small_splits_leave_in_aligned_pieces(rows, K, more, off):
    """With so many experts more that small tiles do not take them: these leave in pieces on 16-byte boundaries."""
    rows = rows + [(7 * i) % 67 for i in range(more)] + ([300, 15] if more else [])
    assert aligned_pieces(sum(rows), K, len(rows), UNITS) == (more > 0)
    o = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    q, sf = synth.random_mxfp4(int(o[-1]), K, seed=len(rows), scale_spread=5)
    q, sf = q.numpy(), sf.numpy()
    wq, ws = ref.row_to_col_grouped(q, sf, o)
    qb = torch.full((wq.size + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    sb = torch.full((ws.size + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    mx.mxfp4_row_to_col_grouped(torch.from_numpy(q).to(DEV), torch.from_numpy(sf).to(DEV), torch.from_numpy(o).to(DEV),
                                q_col=qb[off:off + wq.size], sf_col=sb[:ws.size], offsets_host=o.tolist())
    got = host(qb)
    assert (got[:off] == 0xA5).all() and (got[off + wq.size:] == 0xA5).all() and bool((sb[ws.size:] == 0x5A).all())
    assert_same(host(sb)[:ws.size], ws, "scale bytes")
    assert_same(got[off:off + wq.size], wq, "nibbles")


@pytest.mark.parametrize("M", [145592096, 145592128, 150000032])
def test_rows_on_both_sides_of_32_bit_offsets(M):
    """The longest matrix whose store offsets have 32 bits in whole segments, and longer ones: rows of a 32032-row pattern over and
    over, every byte of every k-row against the oracle's columns of the pattern."""
    K, P = 128, 32 * 1001
    pq, ps = synth.random_mxfp4(P, K, seed=31, scale_spread=5)
    wq, ws = par.row_to_col(pq.numpy(), ps.numpy())
    n, tail = M // P, M % P

    def over_and_over(t):
        t = t.to(DEV)
        return torch.cat([t.expand(n, *t.shape).reshape(n * P, -1), t[:tail]])

    q, sf = over_and_over(pq), over_and_over(ps)
    qb = torch.full((K * (M // 2) + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    sb = torch.full((K * (M // 32) + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    qc, sc = qb[:-4096].view(K, M // 2), sb[:-64].view(K, M // 32)
    mx.mxfp4_row_to_col(q, sf, q_col=qc, sf_col=sc)
    assert bool((qb[-4096:] == 0xA5).all()) and bool((sb[-64:] == 0x5A).all())
    for got, want, unit, what in ((qc, wq, 2, "nibbles"), (sc, ws, 32, "scale bytes")):
        want = torch.from_numpy(want).to(DEV)
        for k in range(K):
            whole = got[k, :n * (P // unit)].view(n, P // unit)
            assert bool((whole == want[k]).all()), f"{what} of k-row {k}, {M} rows"
            assert torch.equal(got[k, n * (P // unit):], want[k, :tail // unit]), f"last {what} of k-row {k}, {M} rows"
