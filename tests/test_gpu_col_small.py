"""GPU parity of the transposing conversions of small matrices and of ragged experts, on both sides of the rule that takes
smaller tiles."""
import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par, ref
from paper_2603_02731_amd import synth
from tests.test_gpu_fp8_col_segments import SPLITS
from tests.rules import small_tiles, times_as_wide
from tests.test_gpu_parity import DEV, UNITS, assert_same, host

pytestmark = pytest.mark.gpu

KINDS = {"mxfp4": 11, "align": 11, "requant": 12}  # quarters of a compute unit's tiles up to which tiles are small


def convert(kind, q, sf):
    """(columns, scales) into guarded buffers."""
    M, K = q.shape[0], 2 * q.shape[1]
    n, ns = (K * M // 2, K * M // 32) if kind == "mxfp4" else (K * M, K * M // 128)
    data = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device=DEV)
    scale = torch.full((ns + 16,), 0x5A, dtype=torch.uint8, device=DEV) if kind == "mxfp4" else torch.full((ns + 16,), 7.0, device=DEV)
    if kind == "mxfp4":
        mx.mxfp4_row_to_col(q, sf, q_col=data[:n].view(K, M // 2), sf_col=scale[:ns].view(K, M // 32))
    else:
        mx.mxfp4_row_to_fp8_col(q, sf, x_col=data[:n].view(K, M), x_col_scale=scale[:ns].view(K, M // 128), requant=kind == "requant")
    assert bool((data[n:] == 0xA5).all()) and bool((scale[ns:] == (0x5A if kind == "mxfp4" else 7.0)).all())
    return data[:n].view(K, -1), scale[:ns].view(K, -1)


def check(kind, q, sf, what):
    data, scale = convert(kind, q, sf)
    if kind == "mxfp4":
        want, ws = par.row_to_col(host(q), host(sf))
        assert_same(host(scale), ws, what + " scale bytes")
    else:
        want, ws = par.row_to_fp8_col(host(q), host(sf), requant=kind == "requant")
        assert_same(host(scale).view(np.uint32), ws.view(np.uint32), what + " scales")
    assert_same(host(data), want, what)


SCALES = {"real": (127, 4, 0.0), "wide": (127, 127, 0.004), "low": (4, 6, 0.0), "high": (250, 5, 0.02), "nan": (120, 3, 0.002)}


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("scales", SCALES)
def test_scales(kind, scales):
    """Row scales from the smallest to those beyond FP32, alone and mixed, NaN bytes in some blocks, whole groups of zeros."""
    center, spread, nan = SCALES[scales]
    q, sf = synth.random_mxfp4(640, 896, seed=7, scale_center=center, scale_spread=spread, nan_scale_frac=nan, device=DEV)
    q[128:256, :64] = 0x80  # zeros of either sign, a whole group of 128 columns
    q[300:340, 64:80] = 0
    check(kind, q, sf, f"{kind} {scales}")
    n = times_as_wide(kind, 640, 896, units=UNITS)  # the same by the larger tiles
    check(kind, q.repeat(1, n), sf.repeat(1, n), f"{kind} {scales}, {n} times as wide")


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("M,K", [(32, 128), (64, 256), (96, 384), (128, 128), (160, 640), (224, 128), (256, 2176), (1152, 384), (2048, 1024)])
def test_sizes(kind, M, K):
    """One tile and many, last tiles of one to three blocks of 32 rows."""
    if kind != "mxfp4" and M % 128:
        M = (M + 127) // 128 * 128
    q, sf = synth.random_mxfp4(M, K, seed=M + K, scale_spread=9, nan_scale_frac=0.001, device=DEV)
    check(kind, q, sf, f"{kind} {M} {K}")


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("over", [0, 1])
def test_sides_of_the_rule(kind, over):
    """The most tiles that are small ones, and one more: the results are the oracle's on both sides."""
    tiles = KINDS[kind] * UNITS // 4 + over
    q, sf = synth.random_mxfp4(128 * tiles, 128, seed=tiles, scale_spread=9, nan_scale_frac=0.001, device=DEV)
    check(kind, q, sf, f"{kind} {tiles} tiles")
    q, sf = synth.random_mxfp4(128, 128 * tiles, seed=tiles, scale_spread=9, nan_scale_frac=0.001, device=DEV)
    check(kind, q, sf, f"{kind} {tiles} tiles beside each other")


def small(kind, rows, K):
    """These splits go by small tiles."""
    return small_tiles(kind, sum(rows), K, len(rows), UNITS)


def check_experts(kind, rows, K, seed, q_off=0, out_off=0, **recipe):
    """The grouped call on nibbles q_off and an output out_off bytes past a 256-byte boundary, with guards around both outputs."""
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    q, sf = (t.numpy() for t in synth.random_mxfp4(int(off[-1]), K, seed=seed, **{"scale_spread": 6, **recipe}))
    src = torch.empty(q.size + 256, dtype=torch.uint8, device=DEV)[q_off:q_off + q.size].view(q.shape)
    src.copy_(torch.from_numpy(q))
    args = src, torch.from_numpy(sf).to(DEV), torch.from_numpy(off).to(DEV)
    mxfp4 = kind == "mxfp4"
    n, ns = (K * sum(-(-r // u) for r in rows) for u in ((2, 32) if mxfp4 else (1, 128)))
    data = torch.full((n + 512,), 0xA5, dtype=torch.uint8, device=DEV)
    scale = torch.full((ns + 64,), 0x5A if mxfp4 else -7.0, dtype=torch.uint8 if mxfp4 else torch.float32, device=DEV)
    out = data[out_off:out_off + n]
    if mxfp4:
        mx.mxfp4_row_to_col_grouped(*args, q_col=out, sf_col=scale[:ns], offsets_host=off.tolist())
        want, ws = ref.row_to_col_grouped(q, sf, off)
    else:
        mx.mxfp4_row_to_fp8_col_grouped(*args, x_col=out, x_col_scale=scale[:ns], requant=kind == "requant", offsets_host=off.tolist())
        want, ws = ref.row_to_fp8_col_grouped(q, sf, off, requant=kind == "requant")
    got, gs = host(data), host(scale)
    assert (got[:out_off] == 0xA5).all() and (got[out_off + n:] == 0xA5).all() and (gs[ns:] == (0x5A if mxfp4 else -7.0)).all()
    assert_same(gs[:ns].view(np.uint8), np.ascontiguousarray(ws).view(np.uint8).ravel(), f"{kind} scales")
    assert_same(got[out_off:out_off + n], np.ascontiguousarray(want).ravel(), kind)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("name", SPLITS)
def test_experts(kind, name):
    """Splits around the edges of pieces, blocks, scale groups and tiles, by small tiles."""
    rows, K = SPLITS[name], 384
    assert small(kind, rows, K)
    check_experts(kind, rows, K, seed=len(rows))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("name", SPLITS)
def test_experts_above_the_line(kind, name):
    """The same splits, as often as it takes to leave the small tiles: the kernels for larger launches keep these edges."""
    rows, K = list(SPLITS[name]), 2176
    while small(kind, rows, K):
        rows += SPLITS[name]
    assert len(rows) <= 256
    check_experts(kind, rows, K, seed=len(rows))


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("kind,each,line", [("mxfp4", 1, 336), ("align", 1, 336), ("requant", 1, 336), ("align", 32, 96)])
def test_sides_of_the_lines_for_few_rows(kind, each, line, over):
    """256 experts of one row, of 32 rows: the widest matrix that goes by small tiles, and 128 columns more."""
    rows = [each] * 256
    K = 128 * (line * UNITS // (2 * (sum(rows) // 128) + 256) + over)
    assert small(kind, rows, K) == (over == 0)
    check_experts(kind, rows, K, seed=each + over)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("E", [1, 64, 65, 256, 257])
def test_numbers_of_experts(kind, E):
    """Both lookups of the small tiles, and one expert more than they take; empty experts at either end and in between."""
    rows = [0 if e % 7 == 0 or e == E - 1 else 1 + (37 * e) % 150 for e in range(E)] if E > 1 else [77]
    check_experts(kind, rows, 256, seed=E)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("scales", SCALES)
@pytest.mark.parametrize("above", [False, True])
def test_scales_of_experts(kind, scales, above):
    """Row scales beyond FP32 and NaN bytes in last tiles that experts do not fill, and in every row that larger tiles convert."""
    center, spread, nan = SCALES[scales]
    rows, K = [33, 161, 0, 128, 7, 300], 2176 if above else 384
    while above and small(kind, rows, K):
        rows = rows + [33, 561, 0, 128, 7, 300]
    assert small(kind, rows, K) == (not above)
    check_experts(kind, rows, K, seed=5, q_off=4, out_off=16, scale_center=center, scale_spread=spread, nan_scale_frac=nan)
