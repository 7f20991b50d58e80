// The short way from a Python call to the C ABI (include/mxfp4.h).
//
// A conversion of a few megabytes takes the GPU less time than the Python wrappers take to check its arguments,
// allocate the outputs and marshal the call (7-9 us).  Each function here takes the arguments of one wrapper in their
// order and either does all of it natively and returns the wrapper's result, or returns None and has launched
// nothing.  It only accepts calls that the wrapper accepts: plain tensors, exact types, default stream argument,
// non-empty sizes.  Everything else -- refusals above all -- is left to the wrapper, which checks again and raises.
// Only a launch that the runtime reports as failed is raised from here: the kernel may have been queued all the same.
// Calls back to back (through Python / here): quantizing [256,512] 9.5 / 4.6 us, into the caller's outputs 6.8 / 3.3, the three flat
// conversions of that matrix 28.6 / 14.6 (quantizing 5.1 with allocations through the dispatcher).
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <string.h>

#include <algorithm>

#include "../../include/mxfp4.h"

namespace {

struct Library {
    decltype(&mxfp4_quant_from_fp8) quant;
    decltype(&mxfp4_quant_from_fp8_scatter) scatter;
    decltype(&mxfp4_quant_from_bf16) quant_bf16;
    decltype(&mxfp4_dequant_to_fp8) dequant;
    decltype(&mxfp4_row_to_col) row_to_col;
    decltype(&mxfp4_quant_from_fp8_grouped) quant_grouped;
    decltype(&mxfp4_row_to_col_grouped) row_to_col_grouped;
    decltype(&mxfp4_row_to_fp8_col) fp8_col[2];                 // alignment, re-quantization
    decltype(&mxfp4_row_to_fp8_col_grouped) fp8_col_grouped[2];
    decltype(&mxfp4_quant_from_fp8_gather_workspace) gather_workspace;
    decltype(&mxfp4_quant_from_fp8_gather) quant_gather;
} lib;
constexpr Py_ssize_t N_FUNCTIONS = sizeof(Library) / sizeof(void *);
c10::DeviceType device_type; // whose tensors are taken
PyObject *check = nullptr;   // the binding's (name, status) -> raises; nullptr: not bound yet

// Thrown (and caught in this file) where a call is left to the Python wrapper.
struct NotHere {};

// Thrown (and caught in this file) where the library could not tell that its launch succeeded.
struct LaunchFailed {
    const char *name;
    mxfp4_status status;
};

inline void need(bool ok)
{
    if (!ok)
        throw NotHere();
}

// Without the interpreter lock while it lives: an allocation may wait for the device, a launch for room in the queue.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};

// A tensor argument: torch.Tensor itself (no subclass), dense (a nested tensor has that layout too), of the given type.
inline const at::Tensor &tensor(PyObject *o, at::ScalarType type)
{
    need(THPVariable_CheckExact(o));
    const at::Tensor &t = THPVariable_Unpack(o);
    need(t.scalar_type() == type && t.layout() == at::kStrided && !t.is_nested() && t.is_contiguous() &&
         t.device().type() == device_type);
    return t;
}

inline void same_device(const at::Tensor &a, const at::Tensor &b) { need(a.get_device() == b.get_device()); }

// Rows and columns of a 2-D input whose column count is a multiple of `of`; empty ones are left to the wrapper.
inline void matrix(const at::Tensor &t, int64_t of, int64_t *rows, int64_t *cols)
{
    need(t.dim() == 2);
    *rows = t.size(0);
    *cols = t.size(1);
    need(*rows > 0 && *cols > 0 && *cols % of == 0);
}

inline void shaped(const at::Tensor &t, int64_t rows, int64_t cols)
{
    need(t.dim() == 2 && t.size(0) == rows && t.size(1) == cols);
}

inline int64_t stride_or(PyObject *o, int64_t dense)
{
    if (o == Py_None)
        return dense;
    need(PyLong_CheckExact(o));
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        throw NotHere();
    }
    return v;
}

// An output: the caller's buffer (contiguous, at least `bytes` long, on the input's device) or a tensor that `launch` allocates.
struct Output {
    at::Tensor t;
    PyObject *given = nullptr;
    at::ScalarType type = at::kByte;
    int64_t shape[2];
    size_t dims;
    bool zero;
    void *data() const { return t.data_ptr(); }
    PyObject *result() const
    {
        if (given) {
            Py_INCREF(given);
            return given;
        }
        return THPVariable_Wrap(t);
    }
};

inline Output output(PyObject *o, const at::Tensor &like, at::ScalarType type, at::IntArrayRef shape, int64_t bytes,
                     bool zero = false)
{
    Output out;
    if (o != Py_None) {
        out.t = tensor(o, type);
        need((int64_t)out.t.nbytes() >= bytes);
        same_device(out.t, like);
        out.given = o;
    } else {
        out.type = type;
        out.dims = shape.size();
        std::copy(shape.begin(), shape.end(), out.shape);
        out.zero = zero;
    }
    return out;
}

// A new tensor on the device of `like`.  Without the dispatcher (half a microsecond of a call's two outputs) where that has nothing else to do: no
// mode, trace, transform or inference mode of this thread takes part in factory calls, and no fill of uninitialized memory is asked for.
inline at::Tensor new_tensor(at::IntArrayRef shape, at::ScalarType type, const at::Tensor &like, bool zero)
{
    const auto options = at::TensorOptions().dtype(type).device(like.device());
    if (zero)
        return at::zeros(shape, options);
    const auto &context = at::globalContext();
    if (like.is_cuda() && c10::impl::tls_local_dispatch_key_set().included_ == c10::default_included_set &&
        !(context.deterministicAlgorithms() && context.deterministicFillUninitializedMemory()))
        return at::Tensor(at::detail::empty_cuda(shape, type, like.device(), std::nullopt));
    return at::empty(shape, options);
}

inline int64_t strided_bytes(int64_t rows, int64_t row_bytes, int64_t ld)
{
    need(ld >= row_bytes && ld < ((int64_t)1 << 31) && rows < ((int64_t)1 << 31));
    return (rows - 1) * ld + row_bytes;
}

// The quantizers' two outputs; a stride other than the dense one needs the caller's buffer.
inline void quant_outputs(PyObject *q, PyObject *sf, PyObject *ld_q_arg, PyObject *ld_sf_arg, const at::Tensor &x,
                          int64_t rows, int64_t K, bool zero, Output (&out)[2], int64_t ld[2])
{
    ld[0] = stride_or(ld_q_arg, K / 2);
    ld[1] = stride_or(ld_sf_arg, K / 32);
    need((q != Py_None || ld[0] == K / 2) && (sf != Py_None || ld[1] == K / 32));
    out[0] = output(q, x, at::kByte, {rows, K / 2}, strided_bytes(rows, K / 2, ld[0]), zero);
    out[1] = output(sf, x, at::kByte, {rows, K / 32}, strided_bytes(rows, K / 32, ld[1]), zero);
}

// Experts of a grouped call whose output sizes are the documented bounds.
inline int64_t experts(const at::Tensor &off, const at::Tensor &q)
{
    need(off.dim() == 1 && off.size(0) >= 2 && off.size(0) <= MXFP4_MAX_EXPERTS + 1);
    same_device(off, q);
    return off.size(0) - 1;
}

inline void *current_stream(const at::Tensor &t)
{
    return t.is_cuda() ? c10::hip::getCurrentHIPStream(t.get_device()).stream() : nullptr;
}

// What goes to that stream is recorded into a graph (or its state cannot be told).
inline bool capturing(const at::Tensor &t)
{
    hipStreamCaptureStatus status;
    if (!t.is_cuda())
        return false;
    if (hipStreamIsCapturing(static_cast<hipStream_t>(current_stream(t)), &status) == hipSuccess)
        return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError(); // not to be taken for an error of the launch
    return true;
}

inline uint8_t *bytes_of(const at::Tensor &t) { return static_cast<uint8_t *>(t.data_ptr()); }

// Runs `body` (which returns the library's status) as a wrapper's call: the pair of outputs, or None.
template <class Body>
PyObject *call(Py_ssize_t n, Py_ssize_t want, PyObject *stream, Body &&body)
{
    if (!check || n != want || stream != Py_None || at::impl::torch_function_mode_enabled())
        Py_RETURN_NONE;
    try {
        Output out[2];
        if (body(out) != MXFP4_OK)
            Py_RETURN_NONE; // refused by the library before a launch: the wrapper's own call reports it
        PyObject *a = out[0].result(), *b = out[1].result();
        PyObject *pair = a && b ? PyTuple_Pack(2, a, b) : nullptr;
        Py_XDECREF(a);
        Py_XDECREF(b);
        return pair;
    } catch (const LaunchFailed &f) {
        Py_XDECREF(PyObject_CallFunction(check, "si", f.name, (int)f.status)); // raises
        if (!PyErr_Occurred())
            PyErr_SetString(PyExc_RuntimeError, f.name);
        return nullptr;
    } catch (const NotHere &) {
    } catch (const std::exception &) { // a tensor without storage, an allocation that failed: raised by the wrapper
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

// Allocates what the caller did not give and calls the entry point `name` through f, without the interpreter lock.
template <class F>
mxfp4_status launch(const char *name, Output (&out)[2], const at::Tensor &like, F &&f)
{
    const mxfp4_status st = [&] {
        Unlocked u;
        for (Output &o : out)
            if (!o.given)
                o.t = new_tensor(at::IntArrayRef(o.shape, o.dims), o.type, like, o.zero);
        return f();
    }();
    if (st == MXFP4_ERR_LAUNCH)
        throw LaunchFailed{name, st};
    return st;
}

// x, x_scale, gather_idx, q, sf, ld_q, ld_sf, stream
PyObject *quant_from_fp8(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 8, n == 8 ? a[7] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &x = tensor(a[0], at::kByte), &s = tensor(a[1], at::kFloat);
        int64_t M, K, ld[2];
        matrix(x, 128, &M, &K);
        shaped(s, M, K / 128);
        same_device(x, s);
        const int32_t *idx = nullptr;
        int64_t rows = M;
        if (a[2] != Py_None) {
            const at::Tensor &g = tensor(a[2], at::kInt);
            same_device(x, g);
            rows = g.numel();
            need(g.dim() == 1 && rows > 0);
            idx = static_cast<const int32_t *>(g.data_ptr());
        }
        quant_outputs(a[3], a[4], a[5], a[6], x, rows, K, false, out, ld);
        return launch("mxfp4_quant_from_fp8", out, x, [&] {
            const float *scale = static_cast<const float *>(s.data_ptr());
            uint8_t *q = static_cast<uint8_t *>(out[0].data()), *sf = static_cast<uint8_t *>(out[1].data());
            // A gather that may gain by memory to work in (smaller ones do not, whatever the library's rule) gets it from the
            // allocator of the current stream, and gives it back there.
            constexpr int64_t WORTH_ASKING = (int64_t)1 << 27; // elements of output
            if (idx && rows < ((int64_t)1 << 31) && K < ((int64_t)1 << 31) && rows * K >= WORTH_ASKING) {
                const int64_t size = lib.gather_workspace(M, K, rows, q, ld[0]);
                if (size > 0) {
                    need(!capturing(x)); // whose memory a graph may keep is looked up by the wrapper
                    at::Tensor work;
                    try {
                        work = new_tensor({size}, at::kByte, x, false);
                    } catch (const c10::OutOfMemoryError &) { // it is done without; the allocator has tried hard, once is enough
                    }
                    if (work.defined())
                        return lib.quant_gather(bytes_of(x), scale, M, K, idx, rows, q, ld[0], sf, ld[1], work.data_ptr(), size,
                                                current_stream(x));
                }
            }
            return lib.quant(bytes_of(x), scale, M, K, idx, rows, q, ld[0], sf, ld[1], current_stream(x));
        });
    });
}

// x, x_scale, dst_idx, M_out, q, sf, ld_q, ld_sf, stream
PyObject *quant_from_fp8_scatter(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 9, n == 9 ? a[8] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &x = tensor(a[0], at::kByte), &s = tensor(a[1], at::kFloat), &d = tensor(a[2], at::kInt);
        int64_t M, K, fanout, rows, ld[2];
        matrix(x, 128, &M, &K);
        shaped(s, M, K / 128);
        matrix(d, 1, &rows, &fanout);
        need(rows == M && fanout < ((int64_t)1 << 31) && a[3] != Py_None);
        same_device(x, s);
        same_device(x, d);
        rows = stride_or(a[3], 0);
        need(rows > 0);
        quant_outputs(a[4], a[5], a[6], a[7], x, rows, K, true, out, ld);
        return launch("mxfp4_quant_from_fp8_scatter", out, x, [&] {
            return lib.scatter(bytes_of(x), static_cast<const float *>(s.data_ptr()), M, K,
                               static_cast<const int32_t *>(d.data_ptr()), (int32_t)fanout, rows,
                               static_cast<uint8_t *>(out[0].data()), ld[0], static_cast<uint8_t *>(out[1].data()), ld[1],
                               current_stream(x));
        });
    });
}

// x, q, sf, ld_q, ld_sf, stream
PyObject *quant_from_bf16(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 6, n == 6 ? a[5] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &x = tensor(a[0], at::kBFloat16);
        int64_t M, K, ld[2];
        matrix(x, 128, &M, &K);
        quant_outputs(a[1], a[2], a[3], a[4], x, M, K, false, out, ld);
        return launch("mxfp4_quant_from_bf16", out, x, [&] {
            return lib.quant_bf16(static_cast<const uint16_t *>(x.data_ptr()), M, K, static_cast<uint8_t *>(out[0].data()),
                                  ld[0], static_cast<uint8_t *>(out[1].data()), ld[1], current_stream(x));
        });
    });
}

// x, x_scale, expert_offsets, q, sf, stream
PyObject *quant_from_fp8_grouped(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 6, n == 6 ? a[5] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &x = tensor(a[0], at::kByte), &s = tensor(a[1], at::kFloat), &off = tensor(a[2], at::kInt);
        int64_t M, K, ld[2];
        matrix(x, 128, &M, &K);
        shaped(s, M, K / 128);
        const int64_t E = experts(off, x);
        same_device(x, s);
        quant_outputs(a[3], a[4], Py_None, Py_None, x, M, K, false, out, ld);
        return launch("mxfp4_quant_from_fp8_grouped", out, x, [&] {
            return lib.quant_grouped(bytes_of(x), static_cast<const float *>(s.data_ptr()),
                                     static_cast<const int32_t *>(off.data_ptr()), (int32_t)E, M, K,
                                     static_cast<uint8_t *>(out[0].data()), static_cast<uint8_t *>(out[1].data()),
                                     current_stream(x));
        });
    });
}

// q, sf, M, K, ld_q, ld_sf, x, x_scale, stream
PyObject *dequant_to_fp8(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 9, n == 9 ? a[8] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &q = tensor(a[0], at::kByte), &sf = tensor(a[1], at::kByte);
        int64_t M, K, ld_q, ld_sf;
        same_device(q, sf);
        if (a[2] == Py_None && a[3] == Py_None) {
            need(a[4] == Py_None && a[5] == Py_None);
            matrix(q, 64, &M, &K);
            K *= 2;
            shaped(sf, M, K / 32);
            ld_q = K / 2;
            ld_sf = K / 32;
        } else {
            need(a[2] != Py_None && a[3] != Py_None);
            M = stride_or(a[2], 0);
            K = stride_or(a[3], 0);
            need(M > 0 && K > 0 && K % 128 == 0 && M < ((int64_t)1 << 31) && K < ((int64_t)1 << 31));
            ld_q = stride_or(a[4], K / 2);
            ld_sf = stride_or(a[5], K / 32);
            need((int64_t)q.nbytes() >= strided_bytes(M, K / 2, ld_q));
            need((int64_t)sf.nbytes() >= strided_bytes(M, K / 32, ld_sf));
        }
        out[0] = output(a[6], q, at::kByte, {M, K}, M * K);
        out[1] = output(a[7], q, at::kFloat, {M, K / 128}, M * (K / 128) * 4);
        return launch("mxfp4_dequant_to_fp8", out, q, [&] {
            return lib.dequant(bytes_of(q), ld_q, bytes_of(sf), ld_sf, M, K, static_cast<uint8_t *>(out[0].data()),
                               static_cast<float *>(out[1].data()), current_stream(q));
        });
    });
}

inline void row_blocked(const at::Tensor &q, const at::Tensor &sf, int64_t *M, int64_t *K)
{
    matrix(q, 64, M, K);
    *K *= 2;
    shaped(sf, *M, *K / 32);
    same_device(q, sf);
    need(*K <= ((int64_t)1 << 24));
}

// q_row, sf_row, q_col, sf_col, stream
PyObject *row_to_col(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 5, n == 5 ? a[4] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &q = tensor(a[0], at::kByte), &sf = tensor(a[1], at::kByte);
        int64_t M, K;
        row_blocked(q, sf, &M, &K);
        need(M % 32 == 0);
        out[0] = output(a[2], q, at::kByte, {K, M / 2}, K * (M / 2));
        out[1] = output(a[3], q, at::kByte, {K, M / 32}, K * (M / 32));
        return launch("mxfp4_row_to_col", out, q, [&] {
            return lib.row_to_col(bytes_of(q), bytes_of(sf), M, K, static_cast<uint8_t *>(out[0].data()),
                                  static_cast<uint8_t *>(out[1].data()), current_stream(q));
        });
    });
}

// q_row, sf_row, expert_offsets, q_col, sf_col, stream
PyObject *row_to_col_grouped(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 6, n == 6 ? a[5] : Py_None, [&](Output (&out)[2]) {
        const at::Tensor &q = tensor(a[0], at::kByte), &sf = tensor(a[1], at::kByte), &off = tensor(a[2], at::kInt);
        int64_t M, K;
        row_blocked(q, sf, &M, &K);
        const int64_t E = experts(off, q), n2 = K * (M / 2 + E), n32 = K * (M / 32 + E);
        out[0] = output(a[3], q, at::kByte, {n2}, n2);
        out[1] = output(a[4], q, at::kByte, {n32}, n32);
        return launch("mxfp4_row_to_col_grouped", out, q, [&] {
            return lib.row_to_col_grouped(bytes_of(q), bytes_of(sf), static_cast<const int32_t *>(off.data_ptr()), (int32_t)E,
                                          M, K, static_cast<uint8_t *>(out[0].data()), static_cast<uint8_t *>(out[1].data()),
                                          current_stream(q));
        });
    });
}

inline int flag(PyObject *o)
{
    need(PyBool_Check(o));
    return o == Py_True ? 1 : 0;
}

// q_row, sf_row, x_col, x_col_scale, stream, requant
PyObject *row_to_fp8_col(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 6, n == 6 ? a[4] : Py_None, [&](Output (&out)[2]) {
        const int requant = flag(a[5]);
        const at::Tensor &q = tensor(a[0], at::kByte), &sf = tensor(a[1], at::kByte);
        int64_t M, K;
        row_blocked(q, sf, &M, &K);
        need(M % 128 == 0);
        out[0] = output(a[2], q, at::kByte, {K, M}, K * M);
        out[1] = output(a[3], q, at::kFloat, {K, M / 128}, K * (M / 128) * 4);
        return launch(requant ? "mxfp4_row_to_fp8_col_requant" : "mxfp4_row_to_fp8_col", out, q, [&] {
            return lib.fp8_col[requant](bytes_of(q), bytes_of(sf), M, K, static_cast<uint8_t *>(out[0].data()),
                                        static_cast<float *>(out[1].data()), current_stream(q));
        });
    });
}

// q_row, sf_row, expert_offsets, x_col, x_col_scale, stream, requant
PyObject *row_to_fp8_col_grouped(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(n, 7, n == 7 ? a[5] : Py_None, [&](Output (&out)[2]) {
        const int requant = flag(a[6]);
        const at::Tensor &q = tensor(a[0], at::kByte), &sf = tensor(a[1], at::kByte), &off = tensor(a[2], at::kInt);
        int64_t M, K;
        row_blocked(q, sf, &M, &K);
        const int64_t E = experts(off, q), n128 = K * (M / 128 + E);
        out[0] = output(a[3], q, at::kByte, {M * K}, M * K);
        out[1] = output(a[4], q, at::kFloat, {n128}, n128 * 4);
        return launch(requant ? "mxfp4_row_to_fp8_col_requant_grouped" : "mxfp4_row_to_fp8_col_grouped", out, q, [&] {
            return lib.fp8_col_grouped[requant](bytes_of(q), bytes_of(sf), static_cast<const int32_t *>(off.data_ptr()),
                                                (int32_t)E, M, K, static_cast<uint8_t *>(out[0].data()),
                                                static_cast<float *>(out[1].data()), current_stream(q));
        });
    });
}

// bind(check, device, address...): what raises for a status, the type of device whose tensors are taken, and the entry
// points of the loaded library in the order of Library.
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    if (n != N_FUNCTIONS + 2 || !PyCallable_Check(a[0]) || !PyUnicode_Check(a[1])) {
        PyErr_Format(PyExc_TypeError, "bind takes a callable, a device type and %zd addresses", N_FUNCTIONS);
        return nullptr;
    }
    void *at[N_FUNCTIONS];
    for (Py_ssize_t i = 0; i < N_FUNCTIONS; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i + 2]);
        if (!at[i]) {
            if (!PyErr_Occurred())
                PyErr_SetString(PyExc_ValueError, "a null address");
            return nullptr;
        }
    }
    const bool host = PyUnicode_CompareWithASCIIString(a[1], "cpu") == 0; // stub entry points, in tests
    if (!host && PyUnicode_CompareWithASCIIString(a[1], "cuda") != 0) {
        PyErr_SetString(PyExc_ValueError, "the device type is cuda or cpu");
        return nullptr;
    }
    static_assert(sizeof(at) == sizeof(lib), "one address per entry point");
    memcpy(&lib, at, sizeof(lib));
    device_type = host ? c10::DeviceType::CPU : c10::DeviceType::CUDA;
    PyObject *before = check;
    Py_INCREF(a[0]);
    check = a[0];
    Py_XDECREF(before);
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind),
                         METHOD(quant_from_fp8),
                         METHOD(quant_from_fp8_scatter),
                         METHOD(quant_from_bf16),
                         METHOD(quant_from_fp8_grouped),
                         METHOD(dequant_to_fp8),
                         METHOD(row_to_col),
                         METHOD(row_to_col_grouped),
                         METHOD(row_to_fp8_col),
                         METHOD(row_to_fp8_col_grouped),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call_path", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__call_path(void) { return PyModule_Create(&module); }
