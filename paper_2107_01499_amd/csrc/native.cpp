// The host path of an ordinary call: torch tensors in, one C entry point of libbagua_hip.so out, without a Python
// object or a ctypes conversion per argument.
//
// Every function takes exactly the arguments of the function of its name in binding.py, checks what that one checks (device,
// contiguity, dtype, size of every tensor) and launches.  It answers True when it has made the call, raises BaguaError when the
// entry point refused it, and answers False, having done nothing, whenever anything about an argument is out of the ordinary:
// binding.py's general path then decides, and words the error.  A round of short launches is bound by this path: a call
// took 5.2 .. 6.4 us of host time (20 with the forty tensors of a ring of eight, 32 with a ring of sixteen), of which the launch itself
// needs 2.5.
#include <Python.h>

#include <stddef.h>
#include <stdint.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include "bagua_hip.h"

namespace {

#define BAGUA_NATIVE(X)                                                                                                          \
    X(bagua_bucket_flatten_run) X(bagua_bucket_unflatten_run) X(bagua_compress_minmax_u8) X(bagua_sign_compress_ef)             \
    X(bagua_momentum_sign_compress_ef) X(bagua_flatten_compress_minmax_u8) X(bagua_flatten_sign_compress_ef)                    \
    X(bagua_decompress_unflatten) X(bagua_decompress_reduce_recompress) X(bagua_decompress) X(bagua_decentralized_avg)          \
    X(bagua_decentralized_avg_peers) X(bagua_decentralized_avg_peers_lp) X(bagua_lp_encode) X(bagua_lp_apply_mix)               \
    X(bagua_reduce_compress_minmax_u8) X(bagua_reduce_compress_sign_ef) X(bagua_centralized_avg_fp) X(bagua_decompress_sgd_step) \
    X(bagua_decompress_adam_step) X(bagua_compress_topk_ef) X(bagua_decompress_reduce_recompress_topk) X(bagua_decompress_topk) \
    X(bagua_decompress_sgd_step_topk) X(bagua_decompress_adam_step_topk)

// The entry points, as binding.py's library has them: the address of each, so that both paths call one and the same library.
#define X(name) decltype(&name) f_##name = nullptr;
BAGUA_NATIVE(X)
#undef X
PyObject* g_error = nullptr;        // binding.BaguaError
PyObject* g_raw_stream = nullptr;   // device index -> raw handle of its current stream
PyObject* g_device = nullptr;       // -> index of the current device

enum Kind { kAny, kF32, kU8, kI32, kI16 };
constexpr size_t kLargest = static_cast<size_t>(1) << 48;   // sizes beyond it go the general way; products of them cannot overflow

size_t chunks_of(size_t n, size_t chunk) { return chunk ? (n + chunk - 1) / chunk : 0; }

// Address of a tensor that the call reads or writes `bytes` of; nullptr for None.  False: not an ordinary one.
bool tensor_ptr(PyObject* o, Kind kind, size_t bytes, void** p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    if (!THPVariable_CheckTypeExact(Py_TYPE(o))) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return false;
    const at::ScalarType type = t.scalar_type();
    if (kind != kAny && type != (kind == kF32 ? at::kFloat : kind == kU8 ? at::kByte : kind == kI32 ? at::kInt : at::kShort)) return false;
    if (t.nbytes() < bytes) return false;
    *p = t.data_ptr();
    return true;
}

// The arguments of one call.  ok turns false at the first one that the general path has to look at.
struct Args {
    PyObject* const* a;
    bool ok;
    Args(PyObject* const* args, Py_ssize_t given, Py_ssize_t expected)
        : a(args), ok(given == expected && at::impl::PythonTorchFunctionTLS::stack_len() == 0 && !torch::jit::tracer::isTracing())
    {
    }
    void* ptr(int i, Kind kind, size_t bytes)
    {
        void* p = nullptr;
        ok = ok && tensor_ptr(a[i], kind, bytes, &p);
        return p;
    }
    bool given(int i) const { return a[i] != Py_None; }
    float* f32(int i, size_t elements) { return static_cast<float*>(ptr(i, kF32, elements * sizeof(float))); }
    size_t numel_of(PyObject* o)
    {
        ok = ok && THPVariable_CheckTypeExact(Py_TYPE(o));
        return ok ? static_cast<size_t>(THPVariable_Unpack(o).numel()) : 0;
    }
    size_t numel(int i) { return ok ? numel_of(a[i]) : 0; }
    size_t size(int i)
    {
        if (!ok || !PyLong_CheckExact(a[i])) { ok = false; return 0; }
        const size_t v = PyLong_AsSize_t(a[i]);
        if (PyErr_Occurred()) PyErr_Clear(), ok = false;
        else if (v > kLargest) ok = false;
        return v;
    }
    int small(int i)   // a codec or a mode
    {
        const size_t v = size(i);
        ok = ok && v < 256;
        return static_cast<int>(v);
    }
    float real(int i)
    {
        if (!ok || !(PyFloat_CheckExact(a[i]) || PyLong_CheckExact(a[i]))) { ok = false; return 0.0f; }
        const double v = PyFloat_AsDouble(a[i]);
        if (PyErr_Occurred()) PyErr_Clear(), ok = false;
        return static_cast<float>(v);
    }
    bool flag(int i)
    {
        ok = ok && PyBool_Check(a[i]);
        return a[i] == Py_True;
    }
    // A list of workers' tensors into p; k = how many there have to be, or -1.  The value: how many there are.
    template <typename T>
    int list(int i, Kind kind, size_t bytes, T** p, int k = -1)
    {
        if (!ok || !(PyList_CheckExact(a[i]) || PyTuple_CheckExact(a[i]))) { ok = false; return 0; }
        const Py_ssize_t count = PySequence_Fast_GET_SIZE(a[i]);
        if (count < 1 || count > BAGUA_MAX_WORKERS || (k >= 0 && count != k)) { ok = false; return 0; }
        PyObject** items = PySequence_Fast_ITEMS(a[i]);
        for (Py_ssize_t j = 0; j < count && ok; ++j) {
            void* q = nullptr;
            ok = tensor_ptr(items[j], kind, bytes, &q);
            p[j] = static_cast<T*>(q);
        }
        return static_cast<int>(count);
    }
    size_t numel_of_first(int i)
    {
        if (!ok || !(PyList_CheckExact(a[i]) || PyTuple_CheckExact(a[i])) || PySequence_Fast_GET_SIZE(a[i]) < 1) { ok = false; return 0; }
        return numel_of(PySequence_Fast_GET_ITEM(a[i], 0));
    }
    void indexes(int i, int* p, int k)
    {
        if (!ok || !(PyList_CheckExact(a[i]) || PyTuple_CheckExact(a[i])) || PySequence_Fast_GET_SIZE(a[i]) != k) { ok = false; return; }
        for (int j = 0; j < k && ok; ++j) {
            PyObject* o = PySequence_Fast_GET_ITEM(a[i], j);
            const long v = PyLong_CheckExact(o) ? PyLong_AsLong(o) : -1;
            if (PyErr_Occurred()) PyErr_Clear();
            ok = v >= 0 && v < BAGUA_MAX_WORKERS;
            p[j] = static_cast<int>(v);
        }
    }
    size_t slots(size_t keep, size_t n, size_t chunk)
    {
        ok = ok && keep <= chunk;   // (or the entry point refuses it)
        return ok ? chunks_of(n, chunk) * keep : 0;
    }
    // Per-codec sizes: bytes of the code stream, and of the per-chunk metadata.
    static size_t code_bytes(int codec, size_t n) { return codec == BAGUA_CODEC_MINMAX_U8 ? n : (n + 31) / 32 * 4; }
    static size_t meta_floats(int codec, size_t n, size_t chunk) { return chunks_of(n, chunk) * (codec == BAGUA_CODEC_MINMAX_U8 ? 2 : 1); }
};

// The raw handle of the stream argument; None is the current stream of the current device.  False: a Python error is set.
bool stream_handle(PyObject* o, void** s)
{
    PyObject* v = nullptr;
    if (o == Py_None) {
        PyObject* device = PyObject_CallNoArgs(g_device);
        if (!device) return false;
        v = PyObject_CallOneArg(g_raw_stream, device);
        Py_DECREF(device);
    } else {
        v = PyObject_GetAttrString(o, "cuda_stream");
    }
    if (!v) return false;
    const unsigned long long h = PyLong_AsUnsignedLongLongMask(v);
    Py_DECREF(v);
    if (PyErr_Occurred()) return false;
    *s = reinterpret_cast<void*>(static_cast<uintptr_t>(h));
    return true;
}

// Marshals with `prepare`, which leaves Args::ok and answers a callable that makes the call on a stream.  Other threads run
// meanwhile, as they do in a call through ctypes.
template <typename F>
PyObject* call(const char* name, PyObject* const* a, Py_ssize_t given, Py_ssize_t expected, const F& prepare)
{
    int status = 0;
    try {
        Args args(a, given, expected);
        if (!args.ok) Py_RETURN_FALSE;
        const auto launch = prepare(args);
        if (!args.ok) Py_RETURN_FALSE;
        void* s = nullptr;
        if (!stream_handle(a[expected - 1], &s)) {
            PyErr_Clear();
            Py_RETURN_FALSE;
        }
        Py_BEGIN_ALLOW_THREADS
        status = launch(s);
        Py_END_ALLOW_THREADS
    } catch (...) {   // a tensor without memory of its own, and the like (nothing has been launched: the entry points do not throw)
        if (PyErr_Occurred()) PyErr_Clear();
        Py_RETURN_FALSE;
    }
    if (status == BAGUA_OK) Py_RETURN_TRUE;
    PyObject* e = PyObject_CallFunction(g_error, "si", name, status);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

template <typename T>
struct Ptrs {
    T* p[BAGUA_MAX_WORKERS];
};
struct Indexes {
    int i[BAGUA_MAX_WORKERS];
};

#define PY(name, expected)                                                              \
    PyObject* py_##name(PyObject*, PyObject* const* a, Py_ssize_t given)                \
    {                                                                                   \
        return call(#name, a, given, expected, [](Args& v) {
#define PY_END \
        });    \
    }

// ------------------------------------------------------------------------------------------ (arguments as in binding.py)
PY(bagua_bucket_flatten_run, 4)   // workspace, T, bucket, stream
    const void* ws = v.ptr(0, kAny, 0);
    const size_t T = v.size(1), n = v.numel(2);
    float* bucket = v.f32(2, 0);
    return [=](void* s) { return f_bagua_bucket_flatten_run(ws, T, bucket, n, s); };
PY_END

PY(bagua_bucket_unflatten_run, 4)   // workspace, T, bucket, stream
    const void* ws = v.ptr(0, kAny, 0);
    const size_t T = v.size(1), n = v.numel(2);
    const float* bucket = v.f32(2, 0);
    return [=](void* s) { return f_bagua_bucket_unflatten_run(ws, T, bucket, n, s); };
PY_END

PY(bagua_compress_minmax_u8, 6)   // x, residual, chunk, codes, minmax, stream
    const size_t n = v.numel(0), chunk = v.size(2);
    const float* x = v.f32(0, 0);
    float* res = v.f32(1, n);
    uint8_t* codes = static_cast<uint8_t*>(v.ptr(3, kU8, n));
    float* mm = v.f32(4, 2 * chunks_of(n, chunk));
    return [=](void* s) { return f_bagua_compress_minmax_u8(x, res, n, chunk, codes, mm, s); };
PY_END

PY(bagua_sign_compress_ef, 6)   // x, residual, chunk, bits, scale, stream
    const size_t n = v.numel(0), chunk = v.size(2);
    const float* x = v.f32(0, 0);
    float* res = v.f32(1, n);
    uint32_t* bits = static_cast<uint32_t*>(v.ptr(3, kI32, v.code_bytes(BAGUA_CODEC_SIGN1, n)));
    float* scale = v.f32(4, chunks_of(n, chunk));
    return [=](void* s) { return f_bagua_sign_compress_ef(x, res, n, chunk, bits, scale, s); };
PY_END

PY(bagua_momentum_sign_compress_ef, 8)   // g, m, beta1, residual, chunk, bits, scale, stream
    const size_t n = v.numel(0), chunk = v.size(4);
    const float* g = v.f32(0, 0);
    const float* m = v.f32(1, n);
    const float beta1 = v.real(2);
    float* res = v.f32(3, n);
    uint32_t* bits = static_cast<uint32_t*>(v.ptr(5, kI32, v.code_bytes(BAGUA_CODEC_SIGN1, n)));
    float* scale = v.f32(6, chunks_of(n, chunk));
    return [=](void* s) { return f_bagua_momentum_sign_compress_ef(g, m, beta1, res, n, chunk, bits, scale, s); };
PY_END

PY(bagua_flatten_compress_minmax_u8, 9)   // workspace, T, residual, n, chunk, codes, minmax, bucket_out, stream
    const void* ws = v.ptr(0, kAny, 0);
    const size_t T = v.size(1), n = v.size(3), chunk = v.size(4);
    float* res = v.f32(2, n);
    uint8_t* codes = static_cast<uint8_t*>(v.ptr(5, kU8, n));
    float* mm = v.f32(6, 2 * chunks_of(n, chunk));
    float* out = v.f32(7, n);
    return [=](void* s) { return f_bagua_flatten_compress_minmax_u8(ws, T, res, n, chunk, codes, mm, out, s); };
PY_END

PY(bagua_flatten_sign_compress_ef, 9)   // workspace, T, residual, n, chunk, bits, scale, bucket_out, stream
    const void* ws = v.ptr(0, kAny, 0);
    const size_t T = v.size(1), n = v.size(3), chunk = v.size(4);
    float* res = v.f32(2, n);
    uint32_t* bits = static_cast<uint32_t*>(v.ptr(5, kI32, v.code_bytes(BAGUA_CODEC_SIGN1, n)));
    float* scale = v.f32(6, chunks_of(n, chunk));
    float* out = v.f32(7, n);
    return [=](void* s) { return f_bagua_flatten_sign_compress_ef(ws, T, res, n, chunk, bits, scale, out, s); };
PY_END

PY(bagua_decompress_unflatten, 8)   // codec, codes, meta, n, chunk, workspace, T, stream
    const int codec = v.small(0);
    const size_t n = v.size(3), chunk = v.size(4), T = v.size(6);
    const void* codes = v.ptr(1, kAny, v.code_bytes(codec, n));
    const float* meta = v.f32(2, v.meta_floats(codec, n, chunk));
    const void* ws = v.ptr(5, kAny, 0);
    return [=](void* s) { return f_bagua_decompress_unflatten(codec, codes, meta, n, chunk, ws, T, s); };
PY_END

PY(bagua_decompress_reduce_recompress, 10)   // codec, codes_in, meta_in, server_residual, n, chunk, codes_out, meta_out, out_fp32, stream
    const int codec = v.small(0);
    const size_t n = v.size(4), chunk = v.size(5);
    const size_t cb = v.code_bytes(codec, n), mf = v.meta_floats(codec, n, chunk);
    Ptrs<const void> ci;
    Ptrs<const float> mi;
    const int k = v.list(1, kAny, cb, ci.p);
    v.list(2, kF32, mf * sizeof(float), mi.p, k);
    float* eps = v.f32(3, n);
    void* co = v.ptr(6, kAny, cb);
    float* mo = v.f32(7, mf);
    float* out = v.f32(8, n);
    return [=](void* s) { return f_bagua_decompress_reduce_recompress(codec, ci.p, mi.p, k, eps, n, chunk, co, mo, out, s); };
PY_END

PY(bagua_decompress, 7)   // codec, codes, meta, n, chunk, out, stream
    const int codec = v.small(0);
    const size_t n = v.size(3), chunk = v.size(4);
    const void* codes = v.ptr(1, kAny, v.code_bytes(codec, n));
    const float* meta = v.f32(2, v.meta_floats(codec, n, chunk));
    float* out = v.f32(5, n);
    return [=](void* s) { return f_bagua_decompress(codec, codes, meta, n, chunk, out, s); };
PY_END

PY(bagua_decentralized_avg, 8)   // mode, x_in, x_out, xhat, codes, minmax, chunk, stream
    const int mode = v.small(0);
    const size_t n = v.numel_of_first(1), chunk = v.size(6), bytes = n * sizeof(float);
    Ptrs<const float> in;
    Ptrs<float> out, hat, mm;
    Ptrs<uint8_t> cd;
    const int k = v.list(1, kF32, bytes, in.p);
    v.list(2, kF32, bytes, out.p, k);
    const bool has_hat = v.given(3), has_codes = v.given(4), has_mm = v.given(5);
    if (has_hat) v.list(3, kF32, bytes, hat.p, k);
    if (has_codes) v.list(4, kU8, n, cd.p, k);
    if (has_mm) v.list(5, kF32, 2 * chunks_of(n, chunk) * sizeof(float), mm.p, k);
    return [=](void* s) {
        return f_bagua_decentralized_avg(mode, in.p, out.p, has_hat ? hat.p : nullptr, has_codes ? cd.p : nullptr, has_mm ? mm.p : nullptr, k, n,
                                         chunk, s);
    };
PY_END

PY(bagua_decentralized_avg_peers, 4)   // x_in, x_out, peer, stream
    const size_t n = v.numel_of_first(0), bytes = n * sizeof(float);
    Ptrs<const float> in;
    Ptrs<float> out;
    Indexes peer{};
    const int k = v.list(0, kF32, bytes, in.p);
    v.list(1, kF32, bytes, out.p, k);
    v.indexes(2, peer.i, k);
    return [=](void* s) { return f_bagua_decentralized_avg_peers(in.p, out.p, peer.i, k, n, s); };
PY_END

PY(bagua_decentralized_avg_peers_lp, 8)   // x_in, x_out, xhat, codes, minmax, peer, chunk, stream
    const size_t n = v.numel_of_first(0), chunk = v.size(6), bytes = n * sizeof(float);
    Ptrs<const float> in;
    Ptrs<float> out, hat, mm;
    Ptrs<uint8_t> cd;
    Indexes peer{};
    const int k = v.list(0, kF32, bytes, in.p);
    v.list(1, kF32, bytes, out.p, k);
    v.list(2, kF32, bytes, hat.p, k);
    v.list(3, kU8, n, cd.p, k);
    v.list(4, kF32, 2 * chunks_of(n, chunk) * sizeof(float), mm.p, k);
    v.indexes(5, peer.i, k);
    return [=](void* s) { return f_bagua_decentralized_avg_peers_lp(in.p, out.p, hat.p, cd.p, mm.p, peer.i, k, n, chunk, s); };
PY_END

PY(bagua_lp_encode, 6)   // x, xhat, chunk, codes, minmax, stream
    const size_t n = v.numel(0), chunk = v.size(2);
    const float* x = v.f32(0, 0);
    float* hat = v.f32(1, n);
    uint8_t* codes = static_cast<uint8_t*>(v.ptr(3, kU8, n));
    float* mm = v.f32(4, 2 * chunks_of(n, chunk));
    return [=](void* s) { return f_bagua_lp_encode(x, hat, n, chunk, codes, mm, s); };
PY_END

PY(bagua_lp_apply_mix, 11)   // x, xhat_own, xhat_left, xhat_right, codes_left, minmax_left, codes_right, minmax_right, chunk, x_out, stream
    const size_t n = v.numel(0), chunk = v.size(8), nm = 2 * chunks_of(n, chunk);
    const float *x = v.f32(0, 0), *own = v.f32(1, n);
    float *left = v.f32(2, n), *right = v.f32(3, n);
    const uint8_t* cl = static_cast<const uint8_t*>(v.ptr(4, kU8, n));
    const float* ml = v.f32(5, nm);
    const uint8_t* cr = static_cast<const uint8_t*>(v.ptr(6, kU8, n));
    const float* mr = v.f32(7, nm);
    float* out = v.f32(9, n);
    return [=](void* s) { return f_bagua_lp_apply_mix(x, own, left, right, cl, ml, cr, mr, n, chunk, out, s); };
PY_END

PY(bagua_reduce_compress_minmax_u8, 6)   // xs, residual, chunk, codes, minmax, stream
    const size_t n = v.numel_of_first(0), chunk = v.size(2);
    Ptrs<const float> xs;
    const int k = v.list(0, kF32, n * sizeof(float), xs.p);
    float* res = v.f32(1, n);
    uint8_t* codes = static_cast<uint8_t*>(v.ptr(3, kU8, n));
    float* mm = v.f32(4, 2 * chunks_of(n, chunk));
    return [=](void* s) { return f_bagua_reduce_compress_minmax_u8(xs.p, k, res, n, chunk, codes, mm, s); };
PY_END

PY(bagua_reduce_compress_sign_ef, 6)   // xs, residual, chunk, bits, scale, stream
    const size_t n = v.numel_of_first(0), chunk = v.size(2);
    Ptrs<const float> xs;
    const int k = v.list(0, kF32, n * sizeof(float), xs.p);
    float* res = v.f32(1, n);
    uint32_t* bits = static_cast<uint32_t*>(v.ptr(3, kI32, v.code_bytes(BAGUA_CODEC_SIGN1, n)));
    float* scale = v.f32(4, chunks_of(n, chunk));
    return [=](void* s) { return f_bagua_reduce_compress_sign_ef(xs.p, k, res, n, chunk, bits, scale, s); };
PY_END

PY(bagua_centralized_avg_fp, 3)   // xs, out, stream
    const size_t n = v.numel_of_first(0);
    Ptrs<const float> xs;
    const int k = v.list(0, kF32, n * sizeof(float), xs.p);
    float* out = v.f32(1, n);
    return [=](void* s) { return f_bagua_centralized_avg_fp(xs.p, k, n, out, s); };
PY_END

PY(bagua_decompress_sgd_step, 11)   // codec, codes, meta, n, chunk, param, momentum_buf, lr, momentum, weight_decay, stream
    const int codec = v.small(0);
    const size_t n = v.size(3), chunk = v.size(4);
    const void* codes = v.ptr(1, kAny, v.code_bytes(codec, n));
    const float* meta = v.f32(2, v.meta_floats(codec, n, chunk));
    float *param = v.f32(5, n), *mom = v.f32(6, n);
    const float lr = v.real(7), mu = v.real(8), wd = v.real(9);
    return [=](void* s) { return f_bagua_decompress_sgd_step(codec, codes, meta, n, chunk, param, mom, lr, mu, wd, s); };
PY_END

// codec, codes, meta, n, chunk, param, m, v, lr, beta1, beta2, eps, weight_decay, variance_frozen, stream
PY(bagua_decompress_adam_step, 15)
    const int codec = v.small(0);
    const size_t n = v.size(3), chunk = v.size(4);
    const void* codes = v.ptr(1, kAny, v.code_bytes(codec, n));
    const float* meta = v.f32(2, v.meta_floats(codec, n, chunk));
    float *param = v.f32(5, n), *m1 = v.f32(6, n), *m2 = v.f32(7, n);
    const float lr = v.real(8), b1 = v.real(9), b2 = v.real(10), eps = v.real(11), wd = v.real(12);
    const bool frozen = v.flag(13);
    return [=](void* s) { return f_bagua_decompress_adam_step(codec, codes, meta, n, chunk, param, m1, m2, lr, b1, b2, eps, wd, frozen, s); };
PY_END

PY(bagua_compress_topk_ef, 7)   // x, residual, chunk, keep, idx, val, stream
    const size_t n = v.numel(0), chunk = v.size(2), keep = v.size(3);
    const size_t slots = v.slots(keep, n, chunk);
    const float* x = v.f32(0, 0);
    float* res = v.f32(1, n);
    uint16_t* idx = static_cast<uint16_t*>(v.ptr(4, kI16, slots * sizeof(uint16_t)));
    float* val = v.f32(5, slots);
    return [=](void* s) { return f_bagua_compress_topk_ef(x, res, n, chunk, keep, idx, val, s); };
PY_END

PY(bagua_decompress_reduce_recompress_topk, 10)   // idx_in, val_in, keep, server_residual, n, chunk, idx_out, val_out, out_fp32, stream
    const size_t keep = v.size(2), n = v.size(4), chunk = v.size(5);
    const size_t slots = v.slots(keep, n, chunk);
    Ptrs<const uint16_t> ii;
    Ptrs<const float> vi;
    const int k = v.list(0, kI16, slots * sizeof(uint16_t), ii.p);
    v.list(1, kF32, slots * sizeof(float), vi.p, k);
    float* eps = v.f32(3, n);
    uint16_t* io = static_cast<uint16_t*>(v.ptr(6, kI16, slots * sizeof(uint16_t)));
    float *vo = v.f32(7, slots), *out = v.f32(8, n);
    return [=](void* s) { return f_bagua_decompress_reduce_recompress_topk(ii.p, vi.p, k, keep, eps, n, chunk, io, vo, out, s); };
PY_END

PY(bagua_decompress_topk, 7)   // idx, val, n, chunk, keep, out, stream
    const size_t n = v.size(2), chunk = v.size(3), keep = v.size(4);
    const size_t slots = v.slots(keep, n, chunk);
    const uint16_t* idx = static_cast<const uint16_t*>(v.ptr(0, kI16, slots * sizeof(uint16_t)));
    const float* val = v.f32(1, slots);
    float* out = v.f32(5, n);
    return [=](void* s) { return f_bagua_decompress_topk(idx, val, n, chunk, keep, out, s); };
PY_END

PY(bagua_decompress_sgd_step_topk, 11)   // idx, val, n, chunk, keep, param, momentum_buf, lr, momentum, weight_decay, stream
    const size_t n = v.size(2), chunk = v.size(3), keep = v.size(4);
    const size_t slots = v.slots(keep, n, chunk);
    const uint16_t* idx = static_cast<const uint16_t*>(v.ptr(0, kI16, slots * sizeof(uint16_t)));
    const float* val = v.f32(1, slots);
    float *param = v.f32(5, n), *mom = v.f32(6, n);
    const float lr = v.real(7), mu = v.real(8), wd = v.real(9);
    return [=](void* s) { return f_bagua_decompress_sgd_step_topk(idx, val, n, chunk, keep, param, mom, lr, mu, wd, s); };
PY_END

// idx, val, n, chunk, keep, param, m, v, lr, beta1, beta2, eps, weight_decay, variance_frozen, stream
PY(bagua_decompress_adam_step_topk, 15)
    const size_t n = v.size(2), chunk = v.size(3), keep = v.size(4);
    const size_t slots = v.slots(keep, n, chunk);
    const uint16_t* idx = static_cast<const uint16_t*>(v.ptr(0, kI16, slots * sizeof(uint16_t)));
    const float* val = v.f32(1, slots);
    float *param = v.f32(5, n), *m1 = v.f32(6, n), *m2 = v.f32(7, n);
    const float lr = v.real(8), b1 = v.real(9), b2 = v.real(10), eps = v.real(11), wd = v.real(12);
    const bool frozen = v.flag(13);
    return [=](void* s) { return f_bagua_decompress_adam_step_topk(idx, val, n, chunk, keep, param, m1, m2, lr, b1, b2, eps, wd, frozen, s); };
PY_END

#undef PY
#undef PY_END

// bind(library, error, raw_stream, device): library = {name of an entry point: its address}
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t given)
{
    if (given != 4 || !PyDict_Check(a[0])) {
        PyErr_SetString(PyExc_TypeError, "bind(library, error, raw_stream, device)");
        return nullptr;
    }
#define X(name)                                                            \
    {                                                                      \
        PyObject* at = PyDict_GetItemString(a[0], #name);                  \
        void* p = at ? PyLong_AsVoidPtr(at) : nullptr;                     \
        if (!p) {                                                          \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name); \
            return nullptr;                                                \
        }                                                                  \
        f_##name = reinterpret_cast<decltype(&name)>(p);                   \
    }
    BAGUA_NATIVE(X)
#undef X
    PyObject** keep[3] = {&g_error, &g_raw_stream, &g_device};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(a[1 + i]);
        Py_XSETREF(*keep[i], a[1 + i]);
    }
    Py_RETURN_NONE;
}

#define X(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
PyMethodDef g_methods[] = {BAGUA_NATIVE(X){"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(bind)), METH_FASTCALL, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
#undef X
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&g_module); }
