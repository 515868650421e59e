// The online entry points of the Python binding as native calls: the argument checks of binding.py's functions and the
// call into the C ABI, without an interpreted step in between.
//
// Why native: a decode call's kernel lasts 3-10 us, and the interpreted checks plus ctypes marshalling took 8-10 us of
// host time per call, so a stream of small calls was bound by the host (K = N = 4096, M = 1: 8.5 us per call against
// 3.5 us of kernel).  Here a tensor argument costs a type check and a few field reads.
//
// Tensors are checked as the binding promises: device tensor and data type (TypeError), contiguous and of the shape the
// handle asks for (ValueError), errors of the library as TmError.  The interpreter lock is released during the library
// call.
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPStream.h>

#include <initializer_list>

#include "tm_attn.h"
#include "tm_w4.h"

namespace {

PyObject* g_tm_error = nullptr;                          // binding.TmError
PyObject *s_h, *s_K, *s_N, *s_experts, *s_batch, *s_kv_heads, *s_stream;      // attribute names, interned

struct Failed {};                                        // a Python exception is set

[[noreturn]] void raise(PyObject* type, const char* text)
{
    PyErr_SetString(type, text);
    throw Failed{};
}

// int(o) and float(o): everything the two builtins take.
long long as_int(PyObject* o)
{
    PyObject* n = PyLong_CheckExact(o) ? (Py_INCREF(o), o) : PyNumber_Long(o);
    if (!n) throw Failed{};
    const long long v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    if (v == -1 && PyErr_Occurred()) throw Failed{};
    return v;
}

double as_double(PyObject* o)
{
    PyObject* f = PyFloat_CheckExact(o) ? (Py_INCREF(o), o) : PyNumber_Float(o);
    if (!f) throw Failed{};
    const double v = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return v;
}

PyObject* attr(PyObject* o, PyObject* name)              // new reference
{
    PyObject* v = PyObject_GetAttr(o, name);
    if (!v) throw Failed{};
    return v;
}

long long int_attr(PyObject* o, PyObject* name)
{
    PyObject* v = attr(o, name);
    const long long x = PyLong_AsLongLong(v);
    Py_DECREF(v);
    if (x == -1 && PyErr_Occurred()) throw Failed{};
    return x;
}

void* handle_of(PyObject* owner, const char* freed)
{
    const long long h = int_attr(owner, s_h);
    if (!h) raise(PyExc_ValueError, freed);
    return (void*)h;
}

const at::Tensor& tensor(PyObject* o, const char* what)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "%s must be a device tensor", what);
        throw Failed{};
    }
    return THPVariable_Unpack(o);
}

void* device_ptr(const at::Tensor& t, at::ScalarType type, const char* what)
{
    if (!t.is_cuda()) {
        PyErr_Format(PyExc_TypeError, "%s must be a device tensor", what);
        throw Failed{};
    }
    if (t.scalar_type() != type) {
        PyErr_Format(PyExc_TypeError, "%s must have dtype torch.%s, got %S", what,
                     type == at::kHalf ? "float16" : type == at::kInt ? "int32" : "uint8",
                     (PyObject*)torch::getTHPDtype(t.scalar_type()));
        throw Failed{};
    }
    if (!t.is_contiguous()) {
        PyErr_Format(PyExc_ValueError, "%s must be contiguous", what);
        throw Failed{};
    }
    return t.data_ptr();
}

uint16_t* half_ptr(const at::Tensor& t, const char* what) { return (uint16_t*)device_ptr(t, at::kHalf, what); }

bool shape_is(const at::Tensor& t, std::initializer_list<int64_t> want)
{
    const auto have = t.sizes();
    if (have.size() != want.size()) return false;
    size_t i = 0;
    for (int64_t w : want)
        if (have[i++] != w) return false;
    return true;
}

tm_stream stream_of(PyObject* stream)
{
    if (stream == Py_None) return (tm_stream)c10::hip::getCurrentHIPStream().stream();
    return (tm_stream)int_attr(stream, s_stream);
}

template <class F>
void call(F&& f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    if (rc == TM_OK) return;
    PyObject* args = Py_BuildValue("(is)", rc, tm_last_error());
    if (args) {
        PyErr_SetObject(g_tm_error, args);
        Py_DECREF(args);
    }
    throw Failed{};
}

// Shared frame of the entry points: argument count, exceptions, and the object handed back (the output tensor or None).
template <class F>
PyObject* entry(Py_ssize_t have, Py_ssize_t want, PyObject* result, F&& f)
{
    if (have != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, have);
        return nullptr;
    }
    try {
        f();
    } catch (const Failed&) {
        return nullptr;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    Py_INCREF(result);
    return result;
}

constexpr const char* kPackedFreed = "packed handle already freed";
constexpr const char* kGroupFreed = "expert group already freed";
constexpr const char* kCacheFreed = "cache already freed";
constexpr const char* kGemmShapes = "X/Y shapes do not match the packed weight";

// The product's own arguments, checked: X [M][K], Y [M][n_out].
struct GemmArgs {
    const at::Tensor &X, &Y;
    const int64_t M, N;
    GemmArgs(PyObject* x, PyObject* packed, PyObject* y, bool halved, const char* shapes)
        : X(tensor(x, "X")), Y(tensor(y, "Y")), M(X.dim() > 0 ? X.size(0) : 0), N(int_attr(packed, s_N))
    {
        if (X.dim() != 2 || X.size(1) != int_attr(packed, s_K) || !shape_is(Y, {M, halved ? N / 2 : N})) raise(PyExc_ValueError, shapes);
    }
};

PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n)          // X, packed, Y, stream
{
    return entry(n, 4, n > 2 ? a[2] : Py_None, [&] {
        GemmArgs g(a[0], a[1], a[2], false, kGemmShapes);
        if (g.M == 0) return;
        const uint16_t* x = half_ptr(g.X, "X");
        const auto* h = (const tm_packed_w4*)handle_of(a[1], kPackedFreed);
        uint16_t* y = half_ptr(g.Y, "Y");
        const tm_stream st = stream_of(a[3]);
        call([&] { return tm_gemm_w4a16(x, h, y, (int)g.M, st); });
    });
}

PyObject* gemm_static(PyObject*, PyObject* const* a, Py_ssize_t n)   // X, packed, Y, stream
{
    return entry(n, 4, n > 2 ? a[2] : Py_None, [&] {
        GemmArgs g(a[0], a[1], a[2], false, kGemmShapes);
        if (g.M == 0) return;
        const uint16_t* x = half_ptr(g.X, "X");
        const auto* h = (const tm_packed_w4*)handle_of(a[1], kPackedFreed);
        uint16_t* y = half_ptr(g.Y, "Y");
        const tm_stream st = stream_of(a[3]);
        call([&] { return tm_gemm_w4a16_static(x, h, y, (int)g.M, st); });
    });
}

PyObject* gemm_ws(PyObject*, PyObject* const* a, Py_ssize_t n)       // X, packed, Y, workspace, stream
{
    return entry(n, 5, n > 2 ? a[2] : Py_None, [&] {
        GemmArgs g(a[0], a[1], a[2], false, kGemmShapes);
        if (g.M == 0) return;
        const uint16_t* x = half_ptr(g.X, "X");
        const auto* h = (const tm_packed_w4*)handle_of(a[1], kPackedFreed);
        uint16_t* y = half_ptr(g.Y, "Y");
        const at::Tensor& w = tensor(a[3], "workspace");
        void* ws = device_ptr(w, at::kByte, "workspace");
        const size_t bytes = (size_t)w.numel();
        const tm_stream st = stream_of(a[4]);
        call([&] { return tm_gemm_w4a16_ws(x, h, y, (int)g.M, ws, bytes, st); });
    });
}

PyObject* gemm_ex(PyObject*, PyObject* const* a, Py_ssize_t n)       // X, packed, Y, bias, residual, act, stream
{
    return entry(n, 7, n > 2 ? a[2] : Py_None, [&] {
        constexpr const char* shapes = "X / Y / bias / residual shapes do not match the packed weight";
        const int act = (int)as_int(a[5]);
        GemmArgs g(a[0], a[1], a[2], act == TM_ACT_SILU_MUL, shapes);
        const at::Tensor* bias = a[3] == Py_None ? nullptr : &tensor(a[3], "bias");
        const at::Tensor* residual = a[4] == Py_None ? nullptr : &tensor(a[4], "residual");
        if ((bias && !shape_is(*bias, {g.N})) || (residual && residual->sizes() != g.Y.sizes())) raise(PyExc_ValueError, shapes);
        if (g.M == 0) return;
        tm_epilogue epi{};
        if (bias) epi.bias = half_ptr(*bias, "bias");
        if (residual) epi.residual = half_ptr(*residual, "residual");
        epi.act = act;
        const uint16_t* x = half_ptr(g.X, "X");
        const auto* h = (const tm_packed_w4*)handle_of(a[1], kPackedFreed);
        uint16_t* y = half_ptr(g.Y, "Y");
        const tm_stream st = stream_of(a[6]);
        call([&] { return tm_gemm_w4a16_ex(x, h, y, (int)g.M, &epi, st); });
    });
}

PyObject* gemm_grouped(PyObject*, PyObject* const* a, Py_ssize_t n)  // X, group, offsets, Y, act, stream
{
    return entry(n, 6, n > 3 ? a[3] : Py_None, [&] {
        constexpr const char* shapes = "X/Y/offsets shapes do not match the expert group";
        const int act = (int)as_int(a[4]);
        GemmArgs g(a[0], a[1], a[3], act == TM_ACT_SILU_MUL, shapes);
        const at::Tensor& off = tensor(a[2], "offsets");
        PyObject* experts = attr(a[1], s_experts);
        const Py_ssize_t count = PyObject_Size(experts);
        Py_DECREF(experts);
        if (count < 0) throw Failed{};
        if (off.numel() != count + 1) raise(PyExc_ValueError, shapes);
        if (g.M == 0) return;
        const uint16_t* x = half_ptr(g.X, "X");
        const auto* h = (const tm_expert_group*)handle_of(a[1], kGroupFreed);
        const auto* o = (const int32_t*)device_ptr(off, at::kInt, "offsets");
        uint16_t* y = half_ptr(g.Y, "Y");
        const tm_stream st = stream_of(a[5]);
        call([&] { return tm_gemm_w4a16_grouped_act(x, h, o, y, (int)g.M, act, st); });
    });
}

PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n)     // cache, K_new, V_new, positions, stream
{
    return entry(n, 5, Py_None, [&] {
        const at::Tensor &K = tensor(a[1], "K_new"), &V = tensor(a[2], "V_new"), &pos = tensor(a[3], "positions");
        const int64_t batch = int_attr(a[0], s_batch);
        if (K.dim() != 4 || K.sizes() != V.sizes() || K.size(0) != batch || K.size(2) != int_attr(a[0], s_kv_heads) ||
            K.size(3) != 128 || pos.numel() != batch)
            raise(PyExc_ValueError, "K_new / V_new / positions shapes do not match the cache");
        auto* h = (tm_kv_cache*)handle_of(a[0], kCacheFreed);
        const uint16_t *k = half_ptr(K, "K_new"), *v = half_ptr(V, "V_new");
        const auto* p = (const int32_t*)device_ptr(pos, at::kInt, "positions");
        const tm_stream st = stream_of(a[4]);
        call([&] { return tm_kv_append(h, k, v, p, (int)K.size(1), st); });
    });
}

PyObject* attn_decode(PyObject*, PyObject* const* a, Py_ssize_t n)   // Q, cache, lens, O, scale, max_len, stream
{
    return entry(n, 7, n > 3 ? a[3] : Py_None, [&] {
        const at::Tensor &Q = tensor(a[0], "Q"), &lens = tensor(a[2], "lens"), &O = tensor(a[3], "O");
        const int64_t batch = int_attr(a[1], s_batch);
        if (Q.dim() != 3 || Q.size(0) != batch || Q.size(2) != 128 || O.sizes() != Q.sizes() || lens.numel() != batch)
            raise(PyExc_ValueError, "Q / O / lens shapes do not match the cache");
        const uint16_t* q = half_ptr(Q, "Q");
        const auto* h = (const tm_kv_cache*)handle_of(a[1], kCacheFreed);
        const auto* l = (const int32_t*)device_ptr(lens, at::kInt, "lens");
        uint16_t* o = half_ptr(O, "O");
        const float scale = (float)as_double(a[4]);
        const int max_len = (int)as_int(a[5]);
        const tm_stream st = stream_of(a[6]);
        call([&] { return tm_attn_decode(q, h, l, o, (int)Q.size(1), scale, max_len, st); });
    });
}

PyObject* attn_prefill(PyObject*, PyObject* const* a, Py_ssize_t n)  // Q, cache, positions, O, scale, counts, stream
{
    return entry(n, 7, n > 3 ? a[3] : Py_None, [&] {
        const at::Tensor &Q = tensor(a[0], "Q"), &O = tensor(a[3], "O"), &pos = tensor(a[2], "positions");
        const at::Tensor* counts = a[5] == Py_None ? nullptr : &tensor(a[5], "counts");
        if (Q.dim() != 4 || Q.size(3) != 128 || O.sizes() != Q.sizes())
            raise(PyExc_ValueError, "Q and O must be [batch][count][q_heads][128]");
        // The launch covers every sequence of the cache, and the C ABI cannot see how long an array is: a shorter one would be
        // read, and O written, out of range.  (A longer one is fine: its first `batch` entries count.)
        const int64_t batch = int_attr(a[1], s_batch);
        if (Q.size(0) < batch || pos.numel() < batch || (counts && counts->numel() < batch))
            raise(PyExc_ValueError, "Q / O / positions / counts have fewer sequences than the cache");
        const auto* c = counts ? (const int32_t*)device_ptr(*counts, at::kInt, "counts") : nullptr;
        const uint16_t* q = half_ptr(Q, "Q");
        const auto* h = (const tm_kv_cache*)handle_of(a[1], kCacheFreed);
        const auto* p = (const int32_t*)device_ptr(pos, at::kInt, "positions");
        uint16_t* o = half_ptr(O, "O");
        const double scale_d = PyFloat_AsDouble(a[4]);                     // a number: no text here, unlike float()
        if (scale_d == -1.0 && PyErr_Occurred()) throw Failed{};
        const float scale = (float)scale_d;
        const tm_stream st = stream_of(a[6]);
        call([&] { return tm_attn_prefill(q, h, p, c, (int)Q.size(1), o, (int)Q.size(2), scale, st); });
    });
}

PyObject* set_error(PyObject*, PyObject* type)
{
    Py_INCREF(type);
    Py_XDECREF(g_tm_error);
    g_tm_error = type;
    Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
constexpr PyMethodDef fast(const char* name)
{
    return {name, (PyCFunction)(void (*)(void))F, METH_FASTCALL, nullptr};
}

PyMethodDef g_methods[] = {fast<gemm>("gemm"),
                           fast<gemm_static>("gemm_static"),
                           fast<gemm_ws>("gemm_ws"),
                           fast<gemm_ex>("gemm_ex"),
                           fast<gemm_grouped>("gemm_grouped"),
                           fast<kv_append>("kv_append"),
                           fast<attn_decode>("attn_decode"),
                           fast<attn_prefill>("attn_prefill"),
                           {"set_error", set_error, METH_O, nullptr},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "tm_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

extern "C" __attribute__((visibility("default"))) PyObject* PyInit_tm_calls()
{
    PyObject** names[] = {&s_h, &s_K, &s_N, &s_experts, &s_batch, &s_kv_heads, &s_stream};
    const char* texts[] = {"_h", "K", "N", "experts", "batch", "kv_heads", "cuda_stream"};
    for (int i = 0; i < 7; ++i)
        if (!(*names[i] = PyUnicode_InternFromString(texts[i]))) return nullptr;
    return PyModule_Create(&g_module);
}
