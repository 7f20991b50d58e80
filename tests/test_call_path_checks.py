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


# ---- every check, one bad argument at a time, all others as in a plain call

ROWS = {"quant_from_fp8 gather": 3 * M, "quant_from_fp8_scatter": M + 3}
FLAT = {"row_to_col_grouped": (K * (M // 2 + 3), K * (M // 32 + 3)), "row_to_fp8_col_grouped": (K * M, 4 * K * (M // 128 + 3))}


def sizes(name):
    """Bytes of the two outputs of a plain call, and where they stand among the arguments."""
    base = name.split()[0]
    if "grouped" in base and base in FLAT:
        return FLAT[base], 3
    if base == "dequant_to_fp8" or base == "row_to_fp8_col":
        return (M * K, 4 * M * (K // 128)), 6 if base == "dequant_to_fp8" else 2
    if base == "row_to_col":
        return (K * M // 2, K * M // 32), 2
    rows = ROWS.get(name, M)
    return (rows * K // 2, rows * K // 32), {"quant_from_bf16": 1, "quant_from_fp8_scatter": 4}.get(base, 3)


def second_type(name):
    return torch.float32 if "fp8_col" in name or "dequant" in name else torch.uint8


def with_outputs(name, device="cpu"):
    """A plain call's arguments with outputs of exactly the sizes needed."""
    _, args = plain(device)[name]
    (a, b), at = sizes(name)
    args[at] = u8(a, device=device)
    args[at + 1] = torch.zeros(b // 4, device=device) if second_type(name) == torch.float32 else u8(b, device=device)
    return args, at


def strided(name):
    """A call with row strides: arguments, where the strides stand, and the bytes that the two buffers need."""
    args, at = with_outputs(name)
    rows = ROWS.get(name, M)
    ld = (DENSE[0] + 48, DENSE[1] + 16)
    need = [(rows - 1) * ld[i] + DENSE[i] for i in range(2)]
    if name == "dequant_to_fp8":
        args = [u8(need[0]), u8(need[1]), M, K, *ld, None, None, None]
        return args, 0, 4, need
    args[at], args[at + 1] = u8(need[0]), u8(need[1])
    args[at + 2], args[at + 3] = ld
    return args, at, at + 2, need


STRIDED = ["quant_from_fp8", "quant_from_fp8 gather", "quant_from_fp8_scatter", "quant_from_bf16", "dequant_to_fp8"]


class Sub(torch.Tensor):
    pass


def spoilt(t):
    """The same tensor with one thing wrong, whatever it is used for."""
    other = torch.int64 if t.dtype == torch.int32 else torch.int32 if t.dtype == torch.float32 else torch.int8
    wide = torch.zeros(*t.shape[:-1], t.shape[-1] * 2, dtype=t.dtype)
    return {"type": t.to(other), "stride": wide[..., ::2], "subclass": t.as_subclass(Sub), "device": t.to("meta"),
            "not a tensor": t.numpy() if t.dtype != torch.bfloat16 else 7, "sparse": t.to_sparse(),
            "dimensions": t.view(1, 1, *t.shape), "a last dimension of one": t.unsqueeze(-1)}


@pytest.mark.parametrize("name", NAMES)
def test_plain_calls_are_taken(stub, name):
    """New outputs and the caller's, of exactly the bytes needed: one call, with the arguments in the library's order."""
    entry, args = plain()[name]
    done, calls = stub.launches(name, *args)
    assert [c[0] for c in calls] == [entry]
    (a, b), at = sizes(name)
    assert done[0].numel() * done[0].element_size() == a and done[1].numel() * done[1].element_size() == b
    assert done[1].dtype == second_type(name)
    got, tensors = calls[0][1], [t for t in args if isinstance(t, torch.Tensor)]
    assert [p for p in got if p in {t.data_ptr() for t in tensors}] == [t.data_ptr() for t in tensors]
    assert [p for p in got if p in (done[0].data_ptr(), done[1].data_ptr())] == [t.data_ptr() for t in done]
    ints = [p for p in got if p is not None and p < 1 << 20]
    rows, off = ROWS.get(name, M), "grouped" in name
    want = {"mxfp4_quant_from_fp8": [M, K, rows, *DENSE], "mxfp4_quant_from_fp8_scatter": [M, K, FAN, rows, *DENSE],
            "mxfp4_quant_from_bf16": [M, K, *DENSE], "mxfp4_dequant_to_fp8": [*DENSE, M, K]}.get(entry, [3] * off + [M, K])
    assert ints == want

    args, at = with_outputs(name)
    done, calls = stub.launches(name, *args)
    assert done[0] is args[at] and done[1] is args[at + 1] and len(calls) == 1


@pytest.mark.parametrize("name", NAMES)
def test_each_bad_tensor_is_left_to_the_wrapper(stub, name):
    args, at = with_outputs(name)
    outputs = (at, at + 1)
    first, tried = args[0].shape, 0
    for i, t in enumerate(args):
        if not isinstance(t, torch.Tensor):
            continue
        bad = spoilt(t)
        if i in outputs:  # any shape will do that holds the bytes
            del bad["dimensions"], bad["a last dimension of one"]
            bad["one short"] = t[:-1].clone()
        elif t.dtype == torch.int32:
            if "scatter" in name:
                bad["rows"], bad["one index a row"] = t[:-1].clone(), t.view(-1)
            elif "gather" not in name:
                bad["no expert"], bad["too many experts"] = t[:1].clone(), torch.zeros(1026, dtype=torch.int32)
            bad["empty"] = t[:0].clone()
        else:
            bad["empty"] = t[:0].clone()
            bad["columns"] = t[:, :-1].contiguous()
            bad["twice as wide"] = torch.cat([t, t], dim=1) if i > 0 else t[:, : t.shape[1] - 4].contiguous()
            if name != "quant_from_bf16":
                bad["rows"] = t[:-1].clone()
            elif i == 0:
                bad["more rows than the outputs hold"] = torch.cat([t, t[:1]])
        for what, value in bad.items():
            done, calls = stub.launches(name, *args[:i], value, *args[i + 1:])
            assert done is None and not calls, f"argument {i}: {what}"
            tried += 1
    assert tried >= 24 and args[0].shape == first


@pytest.mark.parametrize("name", STRIDED)
def test_each_bad_stride_is_left_to_the_wrapper(stub, name):
    args, at, ld, need = strided(name)
    done, calls = stub.launches(name, *args)
    assert done is not None and [v for v in calls[0][1] if v in (args[ld], args[ld + 1])] == [args[ld], args[ld + 1]]
    for i in range(2):
        for what, change in (("short buffer", {at + i: u8(need[i] - 1)}), ("stride below the row", {ld + i: DENSE[i] - 1}),
                             ("huge stride", {ld + i: 1 << 62}), ("beyond 64 bits", {ld + i: 1 << 70}),
                             ("negative stride", {ld + i: -args[ld + i]}), ("no integer", {ld + i: float(args[ld + i])})):
            bad = [change.get(j, a) for j, a in enumerate(args)]
            done, calls = stub.launches(name, *bad)
            assert done is None and not calls, what
        if name != "dequant_to_fp8":  # a stride without the buffer it belongs to
            bad = list(args)
            bad[at + i] = None
            done, calls = stub.launches(name, *bad)
            assert done is None and not calls


@pytest.mark.parametrize("m,k", [(M, None), (None, K), (0, K), (M, 0), (-M, K), (M, K - 64), (M, 1 << 40), (1 << 40, K), (True, K)])
def test_bad_sizes_of_records_are_left_to_the_wrapper(stub, m, k):
    args, _, _, _ = strided("dequant_to_fp8")
    done, calls = stub.launches("dequant_to_fp8", *args[:2], m, k, *args[4:])
    assert done is None and not calls


@pytest.mark.parametrize("ld", [(DENSE[0], None), (None, DENSE[1]), DENSE])
def test_strides_without_sizes_are_left_to_the_wrapper(stub, ld):
    _, args = plain()["dequant_to_fp8"]
    done, calls = stub.launches("dequant_to_fp8", *args[:4], *ld, *args[6:])
    assert done is None and not calls


@pytest.mark.parametrize("rows", [None, 0, -1, 1 << 31, 1 << 70, 5.0, True])
def test_bad_row_counts_of_the_scatter_are_left_to_the_wrapper(stub, rows):
    args, _ = with_outputs("quant_from_fp8_scatter")
    done, calls = stub.launches("quant_from_fp8_scatter", *args[:3], rows, *args[4:])
    assert done is None and not calls


@pytest.mark.parametrize("name,rows", [("row_to_col", 33), ("row_to_fp8_col", 96), ("row_to_fp8_col requant", 160)])
def test_rows_that_are_no_whole_blocks_are_left_to_the_wrapper(stub, name, rows):
    _, args = plain()[name]
    args[0], args[1] = u8(rows, K // 2), u8(rows, K // 32)
    done, calls = stub.launches(name, *args)
    assert done is None and not calls


@pytest.mark.parametrize("name", NAMES)
def test_streams_modes_and_counts_are_left_to_the_wrapper(stub, name):
    _, args = plain()[name]
    at = len(args) - (2 if "fp8_col" in name else 1)
    for stream in (0, 12345, object(), False):
        done, calls = stub.launches(name, *args[:at], stream, *args[at + 1:])
        assert done is None and not calls
    if "fp8_col" in name:
        done, calls = stub.launches(name, *args[:-1], 1)
        assert done is None and not calls
    for wrong in (args[:-1], args + [None], []):
        done, calls = stub.launches(name, *wrong)
        assert done is None and not calls
    with torch.device("meta"):  # a mode that decides where new tensors go
        done, calls = stub.launches(name, *args)
    assert done is None and not calls


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_current_stream_of_the_device_is_handed_on(tmp_path, name):
    stub = Stub(tmp_path, "cuda")
    _, args = plain("cuda:0")[name]
    side = torch.cuda.Stream()
    for s in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(s):
            done, calls = stub.launches(name, *args)
        assert done is not None and (calls[0][1][-1] or 0) == s.cuda_stream
    assert side.cuda_stream != 0
    _, host = plain()[name]
    for i, t in enumerate(host):  # and one host tensor among device tensors is not taken
        if isinstance(t, torch.Tensor):
            done, calls = stub.launches(name, *args[:i], t, *args[i + 1:])
            assert done is None and not calls
