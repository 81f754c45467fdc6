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

// Out of the ordinary: dq8.py takes the call.  Said by a return value, not by an exception: the helpers below return false, and
// to throw and catch took 2.8 us, a declined call 2.9 where it now takes 0.2.
PyObject *declined() { Py_RETURN_NONE; }

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

bool buffer(PyObject *o, at::ScalarType type, Buffer &b)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.key_set().has_any(kTransformed) || t.layout() != at::kStrided || t.scalar_type() != type ||
        !t.has_storage() || !t.is_contiguous())
        return false;
    b.t = &t;
    b.n = (size_t)t.numel();
    b.ptr = t.data_ptr();
    return true;
}

bool whole(PyObject *o, size_t &v)
{
    if (!PyLong_CheckExact(o)) return false;
    const Py_ssize_t l = PyLong_AsSsize_t(o);
    if (l < 0) PyErr_Clear();
    v = (size_t)l;
    return l >= 0;
}

bool kind_of(PyObject *o, int &kind)
{
    size_t v;
    if (!whole(o, v) || v > 255) return false;
    kind = (int)v;
    return true;
}

bool flag(PyObject *o, bool &v)
{
    v = o == Py_True;
    return v || o == Py_False;
}

size_t n_blocks(size_t n, size_t block)
{
    const size_t b = block == 0 || block > n ? n : block;
    return (n + b - 1) / b;
}

// The launch goes to the current stream of the device that `t` is on, which has to be the current device.
bool stream_for(const at::Tensor &t, void *&stream)
{
    const c10::DeviceIndex index = t.get_device();
    if (index != c10::hip::current_device()) return false;
    stream = c10::hip::getCurrentHIPStream(index).stream();
    return true;
}

// An output: the one that was handed in (None: a new one of n elements on `like`'s device).  Keeps a new one alive.
struct Output {
    PyObject *given = nullptr;
    at::Tensor made;
    void *ptr = nullptr;

    bool take(PyObject *o, size_t n, at::ScalarType type, const at::Tensor &like)
    {
        given = o;
        if (o == Py_None) {
            made = at::empty({(int64_t)n}, like.options().dtype(type).requires_grad(false));
            if (made.key_set().has_any(kTransformed)) return false;
            ptr = made.data_ptr();
            return true;
        }
        Buffer b;
        if (!buffer(o, type, b) || b.n < n) return false;
        ptr = b.ptr;
        return true;
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
    size_t bytes = 0;

    bool take(size_t n, const at::Tensor &like, void *stream)
    {
        if (n == 0 || captured(stream)) return true;
        made = at::empty({(int64_t)n}, like.options().dtype(at::kByte).requires_grad(false));
        if (made.key_set().has_any(kTransformed)) return false;
        ptr = made.data_ptr();
        bytes = n;
        return true;
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

    bool open(PyObject *codes_list, PyObject *scales_list)
    {
        if (!sequence(codes_list) || !sequence(scales_list)) return false;
        const Py_ssize_t k = PySequence_Fast_GET_SIZE(codes_list);
        if (k != PySequence_Fast_GET_SIZE(scales_list) || k > DQ8_MAX_K) return false;
        K = (int)k;
        return true;
    }

    // Elements of an average: those of the local term, or of the first worker's codes.
    bool length(PyObject *codes_list, const Buffer &local, size_t &n)
    {
        Buffer b = local;
        if (!local.t) {
            if (K == 0 || !buffer(PySequence_Fast_GET_ITEM(codes_list, 0), at::kByte, b)) return false;
            first = b.t;
        }
        n = b.n;
        return n != 0;
    }

    bool gather(PyObject *codes_list, PyObject *scales_list, size_t n, size_t n_scales)
    {
        for (int k = 0; k < K; ++k) {
            Buffer c, s;
            if (!buffer(PySequence_Fast_GET_ITEM(codes_list, k), at::kByte, c) || !buffer(PySequence_Fast_GET_ITEM(scales_list, k), at::kFloat, s) ||
                c.n != n || s.n < n_scales)
                return false;
            codes[k] = static_cast<const uint8_t *>(c.ptr);
            scales[k] = static_cast<const float *>(s.ptr);
        }
        return true;
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
        if (g_error == nullptr || at::impl::torch_function_mode_enabled()) return declined();
        return BODY(args);
    } catch (const std::exception &) {  // dq8.py meets the same and reports it
        PyErr_Clear();
    }
    return declined();
}

PyObject *absmax(PyObject *const *a)  // x, block, scales
{
    Buffer x;
    size_t block;
    void *stream;
    Output scales;
    if (!buffer(a[0], at::kFloat, x) || !whole(a[1], block) || x.n == 0 || !stream_for(*x.t, stream) ||
        !scales.take(a[2], n_blocks(x.n, block), at::kFloat, *x.t))
        return declined();
    if (!enqueue("dq8_absmax", [&] { return g_lib.absmax(static_cast<float *>(x.ptr), x.n, block, static_cast<float *>(scales.ptr), stream); }))
        return nullptr;
    return scales.result();
}

PyObject *encode(PyObject *const *a)  // kind, x, block, scales, codes, scales_given
{
    int kind;
    Buffer x;
    size_t block;
    bool given;
    void *stream;
    Output scales, codes;
    if (!kind_of(a[0], kind) || !buffer(a[1], at::kFloat, x) || !whole(a[2], block) || !flag(a[5], given) || x.n == 0 ||
        (given && a[3] == Py_None) || !stream_for(*x.t, stream) || !scales.take(a[3], n_blocks(x.n, block), at::kFloat, *x.t) ||
        !codes.take(a[4], x.n, at::kByte, *x.t))
        return declined();
    const unsigned flags = given ? DQ8_SCALES_GIVEN : 0u;
    Scratch scratch;
    if (!scratch.take(g_lib.workspace(x.n, block, flags), *x.t, stream)) return declined();
    if (!enqueue("dq8_encode", [&] {
            return g_lib.encode(kind, static_cast<float *>(x.ptr), x.n, block, static_cast<float *>(scales.ptr),
                                static_cast<uint8_t *>(codes.ptr), flags, scratch.ptr, scratch.bytes, stream);
        }))
        return nullptr;
    return pair(codes, scales);
}

PyObject *decode(PyObject *const *a)  // kind, codes, scales, block, out
{
    int kind;
    Buffer codes, scales;
    size_t block;
    void *stream;
    Output out;
    if (!kind_of(a[0], kind) || !buffer(a[1], at::kByte, codes) || !buffer(a[2], at::kFloat, scales) || !whole(a[3], block) || codes.n == 0 ||
        scales.n < n_blocks(codes.n, block) || !stream_for(*codes.t, stream) || !out.take(a[4], codes.n, at::kFloat, *codes.t))
        return declined();
    if (!enqueue("dq8_decode", [&] {
            return g_lib.decode(kind, static_cast<uint8_t *>(codes.ptr), static_cast<float *>(scales.ptr), codes.n, block,
                                static_cast<float *>(out.ptr), stream);
        }))
        return nullptr;
    return out.result();
}

// An int64 tensor of n_seg + 1 offsets.
bool segments(PyObject *o, Buffer &bounds, size_t &n_seg)
{
    if (!buffer(o, at::kLong, bounds) || bounds.n < 2) return false;
    n_seg = bounds.n - 1;
    return true;
}

PyObject *absmax_segments(PyObject *const *a)  // x, bounds, scales
{
    Buffer x, bounds;
    size_t n_seg;
    void *stream;
    Output scales;
    if (!buffer(a[0], at::kFloat, x) || !segments(a[1], bounds, n_seg) || x.n == 0 || !stream_for(*x.t, stream) ||
        !scales.take(a[2], n_seg, at::kFloat, *x.t))
        return declined();
    if (!enqueue("dq8_absmax_segments", [&] {
            return g_lib.absmax_segments(static_cast<float *>(x.ptr), x.n, static_cast<uint64_t *>(bounds.ptr), n_seg,
                                         static_cast<float *>(scales.ptr), stream);
        }))
        return nullptr;
    return scales.result();
}

PyObject *encode_segments(PyObject *const *a)  // kind, x, bounds, scales, codes, scales_given
{
    int kind;
    Buffer x, bounds;
    size_t n_seg;
    bool given;
    void *stream;
    Output scales, codes;
    if (!kind_of(a[0], kind) || !buffer(a[1], at::kFloat, x) || !segments(a[2], bounds, n_seg) || !flag(a[5], given) || x.n == 0 ||
        (given && a[3] == Py_None) || !stream_for(*x.t, stream) || !scales.take(a[3], n_seg, at::kFloat, *x.t) ||
        !codes.take(a[4], x.n, at::kByte, *x.t))
        return declined();
    const unsigned flags = given ? DQ8_SCALES_GIVEN : 0u;
    Scratch scratch;
    if (!scratch.take(g_lib.workspace_segments(x.n, n_seg, flags), *x.t, stream)) return declined();
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
    int kind;
    Buffer codes, scales, bounds;
    size_t n_seg;
    void *stream;
    Output out;
    if (!kind_of(a[0], kind) || !buffer(a[1], at::kByte, codes) || !buffer(a[2], at::kFloat, scales) || !segments(a[3], bounds, n_seg) ||
        codes.n == 0 || scales.n < n_seg || !stream_for(*codes.t, stream) || !out.take(a[4], codes.n, at::kFloat, *codes.t))
        return declined();
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
    int kind;
    size_t block, n;
    Workers w;
    Buffer local;
    void *stream;
    Output out;
    if (!kind_of(a[0], kind) || !whole(a[3], block) || !w.open(a[1], a[2]) || (a[5] != Py_None && !buffer(a[5], at::kFloat, local)) ||
        !w.length(a[1], local, n) || !w.gather(a[1], a[2], n, n_blocks(n, block)) ||
        !out.take(a[4], n, at::kFloat, local.t ? *local.t : *w.first) || !stream_for(where(out), stream))
        return declined();
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
    int kind;
    size_t n, n_seg;
    Workers w;
    Buffer local, bounds;
    void *stream;
    Output out;
    if (!kind_of(a[0], kind) || !w.open(a[1], a[2]) || (a[5] != Py_None && !buffer(a[5], at::kFloat, local)) || !w.length(a[1], local, n) ||
        !segments(a[3], bounds, n_seg) || !w.gather(a[1], a[2], n, n_seg) || !out.take(a[4], n, at::kFloat, *bounds.t) ||
        !stream_for(where(out), stream))
        return declined();
    if (!enqueue("dq8_decode_accumulate_avg_segments", [&] {
            return g_lib.avg_segments(kind, w.codes, w.scales, w.K, static_cast<float *>(local.ptr), n, static_cast<uint64_t *>(bounds.ptr),
                                      n_seg, static_cast<float *>(out.ptr), stream);
        }))
        return nullptr;
    return out.result();
}

PyObject *decode_avg_encode(PyObject *const *a)  // kind, codes_list, scales_list, block, local, scales, codes
{
    int kind;
    size_t block, n;
    Workers w;
    Buffer local;
    void *stream;
    Output scales, codes;
    if (!kind_of(a[0], kind) || !whole(a[3], block) || !w.open(a[1], a[2]) || (a[4] != Py_None && !buffer(a[4], at::kFloat, local)) ||
        !w.length(a[1], local, n))
        return declined();
    const size_t nb = n_blocks(n, block);
    const at::Tensor &like = local.t ? *local.t : *w.first;
    if (!w.gather(a[1], a[2], n, nb) || !scales.take(a[5], nb, at::kFloat, like) || !codes.take(a[6], n, at::kByte, like) ||
        !stream_for(where(codes), stream))
        return declined();
    if (!enqueue("dq8_decode_avg_encode", [&] {
            return g_lib.avg_encode(kind, w.codes, w.scales, w.K, static_cast<float *>(local.ptr), n, block,
                                    static_cast<float *>(scales.ptr), static_cast<uint8_t *>(codes.ptr), stream);
        }))
        return nullptr;
    return pair(codes, scales);
}

PyObject *error_stats(PyObject *const *a)  // kind, x, block, scales, scales_given, stats, means
{
    int kind;
    Buffer x;
    size_t block;
    bool given;
    void *stream;
    if (!kind_of(a[0], kind) || !buffer(a[1], at::kFloat, x) || !whole(a[2], block) || !flag(a[4], given) || x.n == 0 ||
        (given && a[3] == Py_None) || a[5] == Py_None || a[6] == Py_None || !stream_for(*x.t, stream))
        return declined();
    const size_t nb = n_blocks(x.n, block);
    Output scales, stats, means;
    if (!scales.take(a[3], nb, at::kFloat, *x.t) || !stats.take(a[5], 4 * nb, at::kDouble, *x.t) || !means.take(a[6], 2, at::kDouble, *x.t))
        return declined();
    const unsigned flags = given ? DQ8_SCALES_GIVEN : 0u;
    Scratch scratch;
    if (!scratch.take(g_lib.workspace_stats(x.n, block, flags), *x.t, stream)) return declined();
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
