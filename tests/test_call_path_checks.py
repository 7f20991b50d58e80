"""What the native call path hands to the library: a copy of it, bound to stub entry points that record their arguments
and launch nothing, takes host tensors, so its checks and its marshalling are tested without a GPU."""
import ctypes
import importlib.machinery
import importlib.util
import shutil
import threading
import time

import pytest
import torch

import paper_2603_02731_amd as mx
from paper_2603_02731_amd import binding

M, K, FAN = 256, 512, 2
DENSE = (K // 2, K // 32)


class Stub:
    """A copy of the call path whose entry points record (name, arguments) and return `status`."""

    def __init__(self, folder, device="cpu"):
        library = mx.lib()
        path = folder / "_call_path.so"  # a file of its own: loaded beside the binding's, with its own bound addresses
        shutil.copy(binding.CALL_PATH, path)
        loader = importlib.machinery.ExtensionFileLoader("_call_path", str(path))
        self.call = importlib.util.module_from_spec(importlib.util.spec_from_loader("_call_path", loader))
        self.calls, self.status = [], binding.OK
        self.keep = []
        for name in binding._NATIVE:
            def record(*args, name=name):
                self.calls.append((name, args))
                return self.status
            self.keep.append(ctypes.CFUNCTYPE(ctypes.c_int, *getattr(library, name).argtypes)(record))
        self.call.bind(binding._check, device, *(ctypes.cast(f, ctypes.c_void_p).value for f in self.keep))

    def launches(self, name, *args):
        """(result of the native function, the calls it made)."""
        self.calls.clear()
        return getattr(self.call, name.split()[0])(*args), list(self.calls)


@pytest.fixture
def stub(tmp_path):
    return Stub(tmp_path)


def u8(*shape, device="cpu"):
    return torch.zeros(shape, dtype=torch.uint8, device=device)


def plain(device="cpu"):
    """Per native function: the entry point it calls and a plain call's arguments, in the wrapper's order."""
    x, s = u8(M, K, device=device), torch.zeros(M, K // 128, device=device)
    q, sf = u8(M, K // 2, device=device), u8(M, K // 32, device=device)
    off = torch.tensor([0, 96, 96, M], dtype=torch.int32, device=device)
    idx = torch.zeros(3 * M, dtype=torch.int32, device=device)
    dst = torch.zeros(M, FAN, dtype=torch.int32, device=device)
    return {
        "quant_from_fp8": ("mxfp4_quant_from_fp8", [x, s, None, None, None, None, None, None]),
        "quant_from_fp8 gather": ("mxfp4_quant_from_fp8", [x, s, idx, None, None, None, None, None]),
        "quant_from_fp8_scatter": ("mxfp4_quant_from_fp8_scatter", [x, s, dst, M + 3, None, None, None, None, None]),
        "quant_from_bf16": ("mxfp4_quant_from_bf16", [x.to(torch.bfloat16), None, None, None, None, None]),
        "quant_from_fp8_grouped": ("mxfp4_quant_from_fp8_grouped", [x, s, off, None, None, None]),
        "dequant_to_fp8": ("mxfp4_dequant_to_fp8", [q, sf, None, None, None, None, None, None, None]),
        "row_to_col": ("mxfp4_row_to_col", [q, sf, None, None, None]),
        "row_to_col_grouped": ("mxfp4_row_to_col_grouped", [q, sf, off, None, None, None]),
        "row_to_fp8_col": ("mxfp4_row_to_fp8_col", [q, sf, None, None, None, False]),
        "row_to_fp8_col requant": ("mxfp4_row_to_fp8_col_requant", [q, sf, None, None, None, True]),
        "row_to_fp8_col_grouped": ("mxfp4_row_to_fp8_col_grouped", [q, sf, off, None, None, None, False]),
        "row_to_fp8_col_grouped requant": ("mxfp4_row_to_fp8_col_requant_grouped", [q, sf, off, None, None, None, True]),
    }


NAMES = sorted(plain())


@pytest.mark.parametrize("name", NAMES)
def test_failed_launch_is_raised_and_not_repeated(stub, name, monkeypatch):
    """The runtime may report a failure, an older one even, of a kernel that it has queued: one call, one error."""
    entry, args = plain()[name]
    stub.status = binding.ERR_LAUNCH
    with pytest.raises(mx.Mxfp4Error, match=entry + ": kernel launch failed") as e:
        stub.launches(name, *args)
    assert e.value.status == binding.ERR_LAUNCH and [c[0] for c in stub.calls] == [entry]

    # through the wrapper: the same, and its own way to the library is not tried after it
    stub.calls.clear()
    monkeypatch.setattr(binding, "_call", stub.call)
    monkeypatch.setattr(binding, "_on_device", lambda **_: pytest.fail("the wrapper tried again"))
    with pytest.raises(mx.Mxfp4Error):
        getattr(mx, "mxfp4_" + name.split()[0])(*args)
    assert len(stub.calls) == 1


@pytest.mark.parametrize("status", [binding.ERR_NULL, binding.ERR_SHAPE, binding.ERR_ALIGN, binding.ERR_OFFSETS])
@pytest.mark.parametrize("name", NAMES)
def test_refusal_of_the_library_is_left_to_the_wrapper(stub, name, status):
    _, args = plain()[name]
    stub.status = status
    done, calls = stub.launches(name, *args)
    assert done is None and len(calls) == 1


@pytest.mark.parametrize("name", NAMES)
def test_nested_tensors_are_refused(stub, name, monkeypatch):
    """A nested tensor of equal rows has sizes and storage like a matrix; the wrapper has always refused it."""
    _, args = plain()[name]
    monkeypatch.setattr(binding, "_call", stub.call)
    for i in (0, 1):
        if not isinstance(args[i], torch.Tensor):
            continue
        nested = torch._nested_view_from_buffer(args[i].view(-1), torch.tensor([[args[i].shape[1]]] * args[i].shape[0]),
                                                torch.ones(args[i].shape[0], 1, dtype=torch.int64),
                                                torch.arange(args[i].shape[0]) * args[i].shape[1])
        bad = args[:i] + [nested] + args[i + 1:]
        done, calls = stub.launches(name, *bad)
        assert done is None and not calls
        with pytest.raises((RuntimeError, ValueError)):
            getattr(mx, "mxfp4_" + name.split()[0])(*bad)
        assert not stub.calls


def test_other_threads_run_while_outputs_are_allocated(stub):
    """Zero-filling 2 GiB takes long enough for a thread that only takes notes of the time to run many times."""
    x, s, dst = u8(1, 8192), torch.zeros(1, 64), torch.zeros(1, 1, dtype=torch.int32)
    seen, stop = [], threading.Event()

    def ticks():
        while not stop.is_set():
            seen.append(time.perf_counter())
            time.sleep(1e-3)

    t = threading.Thread(target=ticks)
    t.start()
    try:
        begin = time.perf_counter()
        done, calls = stub.launches("quant_from_fp8_scatter", x, s, dst, 1 << 19, None, None, None, None, None)
        end = time.perf_counter()
    finally:
        stop.set()
        t.join()
    assert done is not None and len(calls) == 1
    # the middle of the call: nothing runs there if the lock is held through the allocations
    fifth = (end - begin) / 5
    assert any(begin + fifth < at < end - fifth for at in seen)
