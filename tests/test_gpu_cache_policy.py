"""GPU parity on both sides of the size below which packed nibbles are left in the memory-side cache (64 MiB of them),
through the chain that reads them back: quantize, de-quantize, transpose."""
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par
from paper_2603_02731_amd import synth
from tests.test_gpu_parity import DEV, assert_same, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K", [(32, 4096), (6112, 4096), (6144, 4096),     # just below 12 MiB of nibbles, and exactly
                                 (32768, 4096), (32800, 4096)])              # 64 MiB exactly, and above
def test_chain_around_the_limit(M, K):
    x8, s = synth.student_t_fp8(M, K, seed=M % 7, device=DEV)
    q, sf = mx.mxfp4_quant_from_fp8(x8, s)
    x, xs = mx.mxfp4_dequant_to_fp8(q, sf)
    qc, sc = mx.mxfp4_row_to_col(q, sf)
    wq, wsf = par.quant(host(x8), host(s))
    assert_same(host(q), wq, "nibbles")
    assert_same(host(sf), wsf, "scale bytes")
    for got, want, name in zip((x, xs, qc, sc), par.dequant(wq, wsf) + par.row_to_col(wq, wsf),
                               ("E4M3 bytes", "tile scales", "column nibbles", "column scale bytes")):
        assert_same(host(got), want, name)


@pytest.mark.parametrize("M", [4096, 32800])
def test_records_around_the_limit(M):
    K = 4096
    q, sf = synth.random_mxfp4(M, K, seed=M, scale_spread=9, device=DEV)
    rec = torch.cat((q, sf), dim=1).view(-1)
    ld = K // 2 + K // 32
    x, xs = mx.mxfp4_dequant_to_fp8(rec, rec[K // 2:], M=M, K=K, ld_q=ld, ld_sf=ld)
    wx, wxs = mx.mxfp4_dequant_to_fp8(q, sf)
    assert torch.equal(x, wx) and torch.equal(xs, wxs)
    wx, wxs = par.dequant(host(q[:512].contiguous()), host(sf[:512].contiguous()))
    assert_same(host(x[:512]), wx, "E4M3 bytes")
    assert_same(host(xs[:512]), wxs, "tile scales")
