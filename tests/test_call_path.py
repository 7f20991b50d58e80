"""The native call path: what it takes gives the wrapper's results, and what it does not take it leaves to the wrapper
without a launch."""
import pytest
import torch

import paper_2603_02731_amd as mx
from paper_2603_02731_amd import binding, synth

DEV = "cuda:0"
M, K = 256, 512


def arguments(device):
    """Per wrapper: its native counterpart's name and a plain call's arguments, in the wrapper's order."""
    x8, s = synth.tiny_roundtrip_fp8(seed=1)
    x, s = x8.to(device), s.to(device)
    q, sf = (t.to(device) for t in synth.random_mxfp4(M, K, seed=2))
    off = torch.tensor([0, 96, 96, M], dtype=torch.int32, device=device)
    idx = (torch.arange(M, dtype=torch.int32, device=device) * 7) % M
    return {
        "quant_from_fp8": (mx.mxfp4_quant_from_fp8, (x, s, None, None, None, None, None, None)),
        "quant_from_fp8 gather": (mx.mxfp4_quant_from_fp8, (x, s, idx, None, None, None, None, None)),
        "quant_from_fp8_scatter": (mx.mxfp4_quant_from_fp8_scatter, (x, s, idx.view(M, 1), M + 3, None, None, None, None, None)),
        "quant_from_bf16": (mx.mxfp4_quant_from_bf16, (x.view(torch.float8_e4m3fn).float().to(torch.bfloat16), None, None, None, None, None)),
        "quant_from_fp8_grouped": (mx.mxfp4_quant_from_fp8_grouped, (x, s, off, None, None, None)),
        "dequant_to_fp8": (mx.mxfp4_dequant_to_fp8, (q, sf, None, None, None, None, None, None, None)),
        "row_to_col": (mx.mxfp4_row_to_col, (q, sf, None, None, None)),
        "row_to_col_grouped": (mx.mxfp4_row_to_col_grouped, (q, sf, off, None, None, None)),
        "row_to_fp8_col": (mx.mxfp4_row_to_fp8_col, (q, sf, None, None, None, False)),
        "row_to_fp8_col requant": (mx.mxfp4_row_to_fp8_col, (q, sf, None, None, None, True)),
        "row_to_fp8_col_grouped": (mx.mxfp4_row_to_fp8_col_grouped, (q, sf, off, None, None, None, False)),
        "row_to_fp8_col_grouped requant": (mx.mxfp4_row_to_fp8_col_grouped, (q, sf, off, None, None, None, True)),
    }


def native(name):
    mx.lib()
    assert binding._call is not None, "the native call path is not built"
    return getattr(binding._call, name.split()[0])


@pytest.mark.parametrize("name", sorted(arguments("cpu")))
def test_leaves_other_calls_to_the_wrapper(name):
    """Host tensors, alone or beside arguments of wrong types, strides and numbers: None, and nothing is raised.  (That
    each single check refuses its argument is tested against stub entry points in test_call_path_checks.)"""
    _, args = arguments("cpu")[name]
    f = native(name)

    class Sub(torch.Tensor):
        pass

    assert f(*args) is None
    assert f(*args[:-1]) is None and f(*args, None) is None and f() is None
    for wrong in (None, 3, "x", args[0].double(), args[0].t(), args[0].view(-1), args[0].as_subclass(Sub), args[0][:0],
                  args[0].to("meta")):
        assert f(wrong, *args[1:]) is None
        assert f(args[0], wrong, *args[2:]) is None
    for i, a in enumerate(args):
        if a is None:
            assert f(*args[:i], object(), *args[i + 1:]) is None


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(arguments("cpu")))
def test_same_results_as_the_wrapper(name, monkeypatch):
    wrapper, args = arguments(DEV)[name]
    got = native(name)(*args)
    assert got is not None, "a plain call is taken"
    with monkeypatch.context() as m:
        m.setattr(binding, "_call", None)
        want = wrapper(*args)
    off = args[2] if name.startswith("row_to") and "grouped" in name else None
    for a, b in zip(got, want):
        assert a.shape == b.shape and a.dtype == b.dtype and a.device == b.device and a.is_contiguous()
    n = [t.numel() for t in want]
    if off is not None:  # flat buffers of bounds: what the splits fill
        rows = [int(v) for v in (off[1:] - off[:-1]).cpu()]
        units = (2, 32) if "to_col" in name else (1, 128)
        n = [K * sum(-(-r // u) for r in rows) for u in units]
    for a, b, k in zip(got, want, n):
        assert torch.equal(a.view(-1)[:k].cpu().view(torch.uint8), b.view(-1)[:k].cpu().view(torch.uint8))
    # into the caller's buffers, which come back as they are
    mine = [torch.full_like(t, 0 if "scatter" in name else 3) for t in want]  # scatter: unnamed rows keep their contents
    slots = [i for i, a in enumerate(args) if a is None]
    if "gather" not in name and name == "quant_from_fp8":
        slots = slots[1:]  # the gather index comes first
    if name == "dequant_to_fp8":
        slots = [6, 7]
    full = list(args)
    full[slots[0]], full[slots[1]] = mine
    back = native(name)(*full)
    assert back[0] is mine[0] and back[1] is mine[1]
    for a, b, k in zip(back, want, n):
        assert torch.equal(a.view(-1)[:k].cpu().view(torch.uint8), b.view(-1)[:k].cpu().view(torch.uint8))


@pytest.mark.gpu
def test_refusals_still_raise_and_streams_are_kept():
    """Results on side streams; which stream a call is handed is tested in test_call_path_checks."""
    x8, s = synth.tiny_roundtrip_fp8(seed=1)
    x, s = x8.to(DEV), s.to(DEV)
    mx.mxfp4_quant_from_fp8(x, s)
    with pytest.raises(ValueError, match="x_scale must have shape"):
        mx.mxfp4_quant_from_fp8(x, s[:1].contiguous())
    with pytest.raises(ValueError, match="holds"):
        mx.mxfp4_quant_from_fp8(x, s, q=torch.empty(8, dtype=torch.uint8, device=DEV))
    with pytest.raises(mx.Mxfp4Error):  # a misaligned output: refused by the library itself
        mx.mxfp4_quant_from_fp8(x, s, q=torch.empty(M * K // 2 + 16, dtype=torch.uint8, device=DEV)[1:])
    with pytest.raises(ValueError, match="multiple of 32"):
        mx.mxfp4_row_to_col(torch.zeros(33, 64, dtype=torch.uint8, device=DEV), torch.zeros(33, 4, dtype=torch.uint8, device=DEV))
    want = mx.mxfp4_quant_from_fp8(x, s)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = mx.mxfp4_quant_from_fp8(x, s)
    given = mx.mxfp4_quant_from_fp8(x, s, stream=side)
    torch.cuda.synchronize()
    for r in (got, given):
        assert torch.equal(r[0], want[0]) and torch.equal(r[1], want[1])


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["quant_from_fp8", "row_to_col_grouped"])
def test_what_takes_part_in_factory_calls_still_does(name):
    """New outputs are allocated past the dispatcher only where nothing else would happen there: dispatch modes see the
    allocations, inference mode makes inference tensors, deterministic mode fills what the call does not write."""
    from torch.utils._python_dispatch import TorchDispatchMode
    wrapper, args = arguments(DEV)[name]

    class Seen(TorchDispatchMode):
        def __init__(self):
            super().__init__()
            self.ops = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.ops.append(str(func))
            return func(*args, **(kwargs or {}))

    plain = wrapper(*args)
    with Seen() as seen:
        got = wrapper(*args)
    assert sum("aten.empty" in op for op in seen.ops) == 2
    with torch.inference_mode():
        inference = wrapper(*args)
    assert all(t.is_inference() for t in inference) and not any(t.is_inference() for t in plain)
    before = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    try:
        filled = wrapper(*args)
    finally:
        torch.use_deterministic_algorithms(before)
    n = [t.numel() for t in plain]
    if name == "row_to_col_grouped":  # the outputs are upper bounds: 256 rows in three experts, the middle one empty
        n = [K * M // 2, K * M // 32]
        assert all(bool((t.view(-1)[k:] == 255).all()) for t, k in zip(filled, n))
    for other in (got, inference, filled):
        assert all(torch.equal(a.view(-1)[:k], b.view(-1)[:k]) for a, b, k in zip(other, plain, n))
