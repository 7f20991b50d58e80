"""GPU parity of the flat transposing conversions of small matrices, on both sides of the rule that takes smaller tiles."""
import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par
from paper_2603_02731_amd import synth
from tests.test_gpu_parity import DEV, assert_same, host

pytestmark = pytest.mark.gpu

UNITS = torch.cuda.get_device_properties(0).multi_processor_count if torch.cuda.is_available() else 256
KINDS = {"mxfp4": 11, "align": 9, "requant": 8}  # quarters of a compute unit's tiles up to which tiles are small


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
