// The calls of dq8.py for the ordinary case, without the interpreter between the arguments and the library: exact torch
// tensors on the current device, of the right type, contiguous and large enough, plain integers.  Every function here has
// the positional arguments of its namesake in dq8.py and returns what that returns, or None when anything about the call
// is out of the ordinary (another device, a tensor subclass, a transformed or traced tensor, an active torch function mode,
// an empty array, a wrong type or size): nothing has happened then, and dq8.py goes on with its own code, which is where
// errors are raised and described.  The one error raised here is the library's own, as dq8.py raises it.
//
// A call on 4096 elements took 5.0 us on the host through ctypes, 3.2 of them in the library (most of that one kernel
// launch); the same call now 2.9, a pair of compression and expansion 9.9 / 5.9, compression into new outputs 7.9 / 4.6.
//
// Outputs that are not handed in, and scratch memory, come from torch's allocator on the current stream; while that stream is
// captured into a graph there is no scratch memory.  The interpreter's lock is released while the library runs, as ctypes does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "dq8_workspace.h"

namespace {

// The library's entry points (set by bind(); null until then: every call returns None) and dq8.Dq8Error.
struct Library {
    decltype(&dq8_absmax) absmax;
    decltype(&dq8_encode_ws) encode;
    decltype(&dq8_workspace_bytes) workspace;
    decltype(&dq8_decode) decode;
    decltype(&dq8_absmax_segments) absmax_segments;
    decltype(&dq8_encode_segments_ws) encode_segments;
    decltype(&dq8_workspace_bytes_segments) workspace_segments;
    decltype(&dq8_decode_segments) decode_segments;
    decltype(&dq8_decode_accumulate_avg) avg;
    decltype(&dq8_decode_accumulate_avg_local) avg_local;
    decltype(&dq8_decode_accumulate_avg_segments) avg_segments;
    decltype(&dq8_decode_avg_encode) avg_encode;
    decltype(&dq8_error_stats_ws) error_stats;
    decltype(&dq8_workspace_bytes_stats) workspace_stats;
    decltype(&dq8_last_error) last_error;
} g_lib;
PyObject *g_error = nullptr;

// Out of the ordinary: dq8.py takes the call.
struct Decline {};

// Tensors whose data are not, or not only, what their address says.
constexpr c10::DispatchKeySet kTransformed({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::Functionalize,
                                            c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                            c10::DispatchKey::BatchedNestedTensor, c10::DispatchKey::NestedTensor,
                                            c10::DispatchKey::Conjugate, c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});

struct Buffer {
    const at::Tensor *t = nullptr;
    void *ptr = nullptr;
    size_t n = 0;
};

Buffer buffer(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) throw Decline();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.key_set().has_any(kTransformed) || t.layout() != at::kStrided || t.scalar_type() != type ||
        !t.has_storage() || !t.is_contiguous())
        throw Decline();
    Buffer b;
    b.t = &t;
    b.n = (size_t)t.numel();
    b.ptr = t.data_ptr();
    return b;
}

size_t whole(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw Decline();
    const Py_ssize_t v = PyLong_AsSsize_t(o);
    if (v < 0) {
        PyErr_Clear();
        throw Decline();
    }
    return (size_t)v;
}

int kind_of(PyObject *o)
{
    const size_t v = whole(o);
    if (v > 255) throw Decline();
    return (int)v;
}

bool flag(PyObject *o)
{
    if (o != Py_True && o != Py_False) throw Decline();
    return o == Py_True;
}

size_t n_blocks(size_t n, size_t block)
{
    const size_t b = block == 0 || block > n ? n : block;
    return (n + b - 1) / b;
}

// The launch goes to the current stream of the device that `t` is on, which has to be the current device.
void *stream_for(const at::Tensor &t)
{
    const c10::DeviceIndex index = t.get_device();
    if (index != c10::hip::current_device()) throw Decline();
    return c10::hip::getCurrentHIPStream(index).stream();
}

// An output: the one that was handed in (None: a new one of n elements on `like`'s device).  Keeps a new one alive.
struct Output {
    PyObject *given;
    at::Tensor made;
    void *ptr;

    Output(PyObject *o, size_t n, at::ScalarType type, const at::Tensor &like) : given(o)
    {
        if (o == Py_None) {
            made = at::empty({(int64_t)n}, like.options().dtype(type).requires_grad(false));
            if (made.key_set().has_any(kTransformed)) throw Decline();
            ptr = made.data_ptr();
        } else {
            const Buffer b = buffer(o, type);
            if (b.n < n) throw Decline();
            ptr = b.ptr;
        }
    }

    PyObject *result() const
    {
        if (given != Py_None) return Py_NewRef(given);
        return THPVariable_Wrap(made);
    }
};

// Whether `stream` is being captured.  (The default stream cannot be.)
bool captured(void *stream)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    return stream && (hipStreamIsCapturing(static_cast<hipStream_t>(stream), &status) != hipSuccess || status != hipStreamCaptureStatusNone);
}

// Scratch memory of one call.  It goes back to torch's allocator when the call returns; the allocator hands it to later work on
// the same stream only, which runs after this call's kernels.  That does not hold for a graph, whose kernels run again
// whenever it is replayed, and torch keeps a graph's memory apart only where it began the capture itself.  So a captured call
// allocates nothing for itself and launches the kernels that need no scratch memory (in a graph, one scale for 1 Mi elements: 8.0
// us, with scratch memory 5.9; statistics of 25 M 57 / 46).
struct Scratch {
    at::Tensor made;
    void *ptr = nullptr;
    size_t bytes;

    Scratch(size_t n, const at::Tensor &like, void *stream) : bytes(n)
    {
        if (n == 0 || captured(stream)) return;
        made = at::empty({(int64_t)n}, like.options().dtype(at::kByte).requires_grad(false));
        if (made.key_set().has_any(kTransformed)) throw Decline();
        ptr = made.data_ptr();
    }
};

PyObject *pair(const Output &a, const Output &b)
{
    PyObject *x = a.result();
    PyObject *y = x ? b.result() : nullptr;
    PyObject *r = y ? PyTuple_New(2) : nullptr;
    if (!r) {
        Py_XDECREF(x);
        Py_XDECREF(y);
        return nullptr;
    }
    PyTuple_SET_ITEM(r, 0, x);
    PyTuple_SET_ITEM(r, 1, y);
    return r;
}

// The workers' buffers of a call: exact lists or tuples of equal length, codes of n elements, at least n_scales scales each.
struct Workers {
    const uint8_t *codes[DQ8_MAX_K];
    const float *scales[DQ8_MAX_K];
    int K = 0;
    const at::Tensor *first = nullptr;

    static bool sequence(PyObject *o) { return PyList_CheckExact(o) || PyTuple_CheckExact(o); }

    Workers(PyObject *codes_list, PyObject *scales_list)
    {
        if (!sequence(codes_list) || !sequence(scales_list)) throw Decline();
        const Py_ssize_t k = PySequence_Fast_GET_SIZE(codes_list);
        if (k != PySequence_Fast_GET_SIZE(scales_list) || k > DQ8_MAX_K) throw Decline();
        K = (int)k;
    }

    // Elements of the first worker's codes.
    size_t numel(PyObject *codes_list)
    {
        if (K == 0) throw Decline();
        const Buffer b = buffer(PySequence_Fast_GET_ITEM(codes_list, 0), at::kByte);
        first = b.t;
        return b.n;
    }

    void gather(PyObject *codes_list, PyObject *scales_list, size_t n, size_t n_scales)
    {
        for (int k = 0; k < K; ++k) {
            const Buffer c = buffer(PySequence_Fast_GET_ITEM(codes_list, k), at::kByte);
            const Buffer s = buffer(PySequence_Fast_GET_ITEM(scales_list, k), at::kFloat);
            if (c.n != n || s.n < n_scales) throw Decline();
            codes[k] = static_cast<const uint8_t *>(c.ptr);
            scales[k] = static_cast<const float *>(s.ptr);
        }
    }
};

// Runs `f` without the interpreter's lock; false with dq8.Dq8Error set when the library reports an error.
template <typename F>
bool enqueue(const char *what, F f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    if (rc == 0) return true;
    PyErr_Format(g_error, "%s failed (status %d): %s", what, rc, g_lib.last_error());
    return false;
}

// A function of this module: `body` with its positional arguments, None for a call that it declines.
template <PyObject *(*BODY)(PyObject *const *), int ARGS>
PyObject *entry(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != ARGS) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", ARGS, n);
        return nullptr;
    }
    try {
        if (g_error == nullptr || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
        return BODY(args);
    } catch (const Decline &) {
    } catch (const std::exception &) {  // dq8.py meets the same and reports it
        PyErr_Clear();
    }
    Py_RETURN_NONE;
}

PyObject *absmax(PyObject *const *a)  // x, block, scales
{
    const Buffer x = buffer(a[0], at::kFloat);
    const size_t block = whole(a[1]);
    if (x.n == 0) throw Decline();
    void *stream = stream_for(*x.t);
    const Output scales(a[2], n_blocks(x.n, block), at::kFloat, *x.t);
    if (!enqueue("dq8_absmax", [&] { return g_lib.absmax(static_cast<float *>(x.ptr), x.n, block, static_cast<float *>(scales.ptr), stream); }))
        return nullptr;
    return scales.result();
}

PyObject *encode(PyObject *const *a)  // kind, x, block, scales, codes, scales_given
{
    const int kind = kind_of(a[0]);
    const Buffer x = buffer(a[1], at::kFloat);
    const size_t block = whole(a[2]);
    const bool given = flag(a[5]);
    if (x.n == 0 || (given && a[3] == Py_None)) throw Decline();
    void *stream = stream_for(*x.t);
    const Output scales(a[3], n_blocks(x.n, block), at::kFloat, *x.t), codes(a[4], x.n, at::kByte, *x.t);
    const unsigned flags = given ? DQ8_SCALES_GIVEN : 0u;
    const Scratch scratch(g_lib.workspace(x.n, block, flags), *x.t, stream);
    if (!enqueue("dq8_encode", [&] {
            return g_lib.encode(kind, static_cast<float *>(x.ptr), x.n, block, static_cast<float *>(scales.ptr),
                                static_cast<uint8_t *>(codes.ptr), flags, scratch.ptr, scratch.bytes, stream);
        }))
        return nullptr;
    return pair(codes, scales);
}

PyObject *decode(PyObject *const *a)  // kind, codes, scales, block, out
{
    const int kind = kind_of(a[0]);
    const Buffer codes = buffer(a[1], at::kByte), scales = buffer(a[2], at::kFloat);
    const size_t block = whole(a[3]);
    if (codes.n == 0 || scales.n < n_blocks(codes.n, block)) throw Decline();
    void *stream = stream_for(*codes.t);
    const Output out(a[4], codes.n, at::kFloat, *codes.t);
    if (!enqueue("dq8_decode", [&] {
            return g_lib.decode(kind, static_cast<uint8_t *>(codes.ptr), static_cast<float *>(scales.ptr), codes.n, block,
                                static_cast<float *>(out.ptr), stream);
        }))
        return nullptr;
    return out.result();
}

// Segments in `bounds`, an int64 tensor of n_seg + 1 offsets.
size_t segments(const Buffer &bounds)
{
    if (bounds.n < 2) throw Decline();
    return bounds.n - 1;
}

PyObject *absmax_segments(PyObject *const *a)  // x, bounds, scales
{
    const Buffer x = buffer(a[0], at::kFloat), bounds = buffer(a[1], at::kLong);
    const size_t n_seg = segments(bounds);
    if (x.n == 0) throw Decline();
    void *stream = stream_for(*x.t);
    const Output scales(a[2], n_seg, at::kFloat, *x.t);
    if (!enqueue("dq8_absmax_segments", [&] {
            return g_lib.absmax_segments(static_cast<float *>(x.ptr), x.n, static_cast<uint64_t *>(bounds.ptr), n_seg,
                                         static_cast<float *>(scales.ptr), stream);
        }))
        return nullptr;
    return scales.result();
}

PyObject *encode_segments(PyObject *const *a)  // kind, x, bounds, scales, codes, scales_given
{
    const int kind = kind_of(a[0]);
    const Buffer x = buffer(a[1], at::kFloat), bounds = buffer(a[2], at::kLong);
    const size_t n_seg = segments(bounds);
    const bool given = flag(a[5]);
    if (x.n == 0 || (given && a[3] == Py_None)) throw Decline();
    void *stream = stream_for(*x.t);
    const Output scales(a[3], n_seg, at::kFloat, *x.t), codes(a[4], x.n, at::kByte, *x.t);
    const unsigned flags = given ? DQ8_SCALES_GIVEN : 0u;
    const Scratch scratch(g_lib.workspace_segments(x.n, n_seg, flags), *x.t, stream);
    if (!enqueue("dq8_encode_segments", [&] {
            return g_lib.encode_segments(kind, static_cast<float *>(x.ptr), x.n, static_cast<uint64_t *>(bounds.ptr), n_seg,
                                         static_cast<float *>(scales.ptr), static_cast<uint8_t *>(codes.ptr), flags,
                                         scratch.ptr, scratch.bytes, stream);
        }))
        return nullptr;
    return pair(codes, scales);
}

PyObject *decode_segments(PyObject *const *a)  // kind, codes, scales, bounds, out
{
    const int kind = kind_of(a[0]);
    const Buffer codes = buffer(a[1], at::kByte), scales = buffer(a[2], at::kFloat), bounds = buffer(a[3], at::kLong);
    const size_t n_seg = segments(bounds);
    if (codes.n == 0 || scales.n < n_seg) throw Decline();
    void *stream = stream_for(*codes.t);
    const Output out(a[4], codes.n, at::kFloat, *codes.t);
    if (!enqueue("dq8_decode_segments", [&] {
            return g_lib.decode_segments(kind, static_cast<uint8_t *>(codes.ptr), static_cast<float *>(scales.ptr), codes.n,
                                         static_cast<uint64_t *>(bounds.ptr), n_seg, static_cast<float *>(out.ptr), stream);
        }))
        return nullptr;
    return out.result();
}

// The device of an averaging call is that of its output, as in dq8.py.
const at::Tensor &where(const Output &o) { return o.given == Py_None ? o.made : THPVariable_Unpack(o.given); }

PyObject *decode_accumulate_avg(PyObject *const *a)  // kind, codes_list, scales_list, block, out, local
{
    const int kind = kind_of(a[0]);
    const size_t block = whole(a[3]);
    Workers w(a[1], a[2]);
    Buffer local;
    if (a[5] != Py_None) local = buffer(a[5], at::kFloat);
    const size_t n = local.t ? local.n : w.numel(a[1]);
    if (n == 0) throw Decline();
    w.gather(a[1], a[2], n, n_blocks(n, block));
    const Output out(a[4], n, at::kFloat, local.t ? *local.t : *w.first);
    void *stream = stream_for(where(out));
    if (!enqueue(local.t ? "dq8_decode_accumulate_avg_local" : "dq8_decode_accumulate_avg", [&] {
            if (local.t)
                return g_lib.avg_local(kind, w.codes, w.scales, w.K, static_cast<float *>(local.ptr), n, block,
                                       static_cast<float *>(out.ptr), stream);
            return g_lib.avg(kind, w.codes, w.scales, w.K, n, block, static_cast<float *>(out.ptr), stream);
        }))
        return nullptr;
    return out.result();
}

PyObject *decode_accumulate_avg_segments(PyObject *const *a)  // kind, codes_list, scales_list, bounds, out, local
{
    const int kind = kind_of(a[0]);
    Workers w(a[1], a[2]);
    Buffer local;
    if (a[5] != Py_None) local = buffer(a[5], at::kFloat);
    const size_t n = local.t ? local.n : w.numel(a[1]);
    const Buffer bounds = buffer(a[3], at::kLong);
    const size_t n_seg = segments(bounds);
    if (n == 0) throw Decline();
    w.gather(a[1], a[2], n, n_seg);
    const Output out(a[4], n, at::kFloat, *bounds.t);
    void *stream = stream_for(where(out));
    if (!enqueue("dq8_decode_accumulate_avg_segments", [&] {
            return g_lib.avg_segments(kind, w.codes, w.scales, w.K, static_cast<float *>(local.ptr), n, static_cast<uint64_t *>(bounds.ptr),
                                      n_seg, static_cast<float *>(out.ptr), stream);
        }))
        return nullptr;
    return out.result();
}

PyObject *decode_avg_encode(PyObject *const *a)  // kind, codes_list, scales_list, block, local, scales, codes
{
    const int kind = kind_of(a[0]);
    const size_t block = whole(a[3]);
    Workers w(a[1], a[2]);
    Buffer local;
    if (a[4] != Py_None) local = buffer(a[4], at::kFloat);
    const size_t n = local.t ? local.n : w.numel(a[1]);
    if (n == 0) throw Decline();
    const size_t nb = n_blocks(n, block);
    w.gather(a[1], a[2], n, nb);
    const at::Tensor &like = local.t ? *local.t : *w.first;
    const Output scales(a[5], nb, at::kFloat, like), codes(a[6], n, at::kByte, like);
    void *stream = stream_for(where(codes));
    if (!enqueue("dq8_decode_avg_encode", [&] {
            return g_lib.avg_encode(kind, w.codes, w.scales, w.K, static_cast<float *>(local.ptr), n, block,
                                    static_cast<float *>(scales.ptr), static_cast<uint8_t *>(codes.ptr), stream);
        }))
        return nullptr;
    return pair(codes, scales);
}

PyObject *error_stats(PyObject *const *a)  // kind, x, block, scales, scales_given, stats, means
{
    const int kind = kind_of(a[0]);
    const Buffer x = buffer(a[1], at::kFloat);
    const size_t block = whole(a[2]);
    const bool given = flag(a[4]);
    if (x.n == 0 || (given && a[3] == Py_None) || a[5] == Py_None || a[6] == Py_None) throw Decline();
    void *stream = stream_for(*x.t);
    const size_t nb = n_blocks(x.n, block);
    const Output scales(a[3], nb, at::kFloat, *x.t), stats(a[5], 4 * nb, at::kDouble, *x.t), means(a[6], 2, at::kDouble, *x.t);
    const unsigned flags = given ? DQ8_SCALES_GIVEN : 0u;
    const Scratch scratch(g_lib.workspace_stats(x.n, block, flags), *x.t, stream);
    if (!enqueue("dq8_error_stats", [&] {
            return g_lib.error_stats(kind, static_cast<float *>(x.ptr), x.n, block, static_cast<float *>(scales.ptr), flags,
                                     static_cast<double *>(stats.ptr), static_cast<double *>(means.ptr), scratch.ptr, scratch.bytes, stream);
        }))
        return nullptr;
    return pair(stats, means);
}

// bind(error class, {name: address}): the entry points of the library that dq8.py has loaded.
PyObject *bind(PyObject *, PyObject *args)
{
    PyObject *error, *addresses;
    if (!PyArg_ParseTuple(args, "OO!", &error, &PyDict_Type, &addresses)) return nullptr;
    Library l;
    bool ok = true;
    auto take = [&](auto &f, const char *name) {
        PyObject *v = PyDict_GetItemString(addresses, name);  // borrowed
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p && !PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "%s", name);
        f = reinterpret_cast<std::decay_t<decltype(f)>>(p);
        ok = ok && p;
    };
    take(l.absmax, "dq8_absmax");
    take(l.encode, "dq8_encode_ws");
    take(l.workspace, "dq8_workspace_bytes");
    take(l.decode, "dq8_decode");
    take(l.absmax_segments, "dq8_absmax_segments");
    take(l.encode_segments, "dq8_encode_segments_ws");
    take(l.workspace_segments, "dq8_workspace_bytes_segments");
    take(l.decode_segments, "dq8_decode_segments");
    take(l.avg, "dq8_decode_accumulate_avg");
    take(l.avg_local, "dq8_decode_accumulate_avg_local");
    take(l.avg_segments, "dq8_decode_accumulate_avg_segments");
    take(l.avg_encode, "dq8_decode_avg_encode");
    take(l.error_stats, "dq8_error_stats_ws");
    take(l.workspace_stats, "dq8_workspace_bytes_stats");
    take(l.last_error, "dq8_last_error");
    if (!ok) return nullptr;
    g_lib = l;
    g_error = Py_NewRef(error);
    Py_RETURN_NONE;
}

template <PyObject *(*BODY)(PyObject *const *), int ARGS>
PyMethodDef method(const char *name)
{
    return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<BODY, ARGS>)), METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    method<absmax, 3>("absmax"),
    method<encode, 6>("encode"),
    method<decode, 5>("decode"),
    method<absmax_segments, 3>("absmax_segments"),
    method<encode_segments, 6>("encode_segments"),
    method<decode_segments, 5>("decode_segments"),
    method<decode_accumulate_avg, 6>("decode_accumulate_avg"),
    method<decode_accumulate_avg_segments, 6>("decode_accumulate_avg_segments"),
    method<decode_avg_encode, 7>("decode_avg_encode"),
    method<error_stats, 7>("error_stats"),
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&g_module); }
