// CPython side of the calls a serving loop makes for every token: argument checks, current stream, call into
// libmnnq.so.  The work of such a call on the GPU is 4 - 15 us, and the marshalling used to take as long: through
// ctypes (12 converted arguments, a Python frame per check, a call to size the packed buffer) a decode call cost the
// host about 9 us, four of them - one transformer block - 36 us.  Here it is a parse of the argument vector, reads of
// tensor fields and the launch itself.  Names, arguments, defaults, checks and errors are those of the functions in
// binding.py that this module provides; nothing is computed here and nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

#include "../../include/mnnq.h"

namespace {

constexpr int kGroup = 64;
constexpr int kMaxArgs = 12;

// Thrown with a Python error already set.
struct PyError {};

[[noreturn]] void fail(PyObject* type, const char* fmt, const char* what, long long a = 0, long long b = 0)
{
    PyErr_Format(type, fmt, what, a, b);
    throw PyError{};
}

// Parameter list of one function: names interned at import, the first `required` without a default.
struct Params {
    const char* function;
    int count, required;
    const char* names[kMaxArgs];
    PyObject* interned[kMaxArgs];
};

// Positional and keyword arguments -> v[0 .. count), nullptr where the default applies.
void parse(const Params& p, PyObject* const* args, Py_ssize_t n_pos, PyObject* kwnames, PyObject** v)
{
    for (int i = 0; i < p.count; ++i) v[i] = nullptr;
    if (n_pos > p.count) fail(PyExc_TypeError, "%s() takes %lld arguments (%lld given)", p.function, p.count, n_pos);
    for (Py_ssize_t i = 0; i < n_pos; ++i) v[i] = args[i];
    const Py_ssize_t n_kw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < n_kw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        int at = 0;
        while (at < p.count && p.interned[at] != name) ++at;
        if (at == p.count)   // (a name built at run time is not interned)
            for (at = 0; at < p.count && PyUnicode_Compare(p.interned[at], name) != 0;) ++at;
        if (at == p.count) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", p.function, name);
            throw PyError{};
        }
        if (v[at]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", p.function, name);
            throw PyError{};
        }
        v[at] = args[n_pos + k];
    }
    for (int i = 0; i < p.required; ++i)
        if (!v[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", p.function, p.names[i]);
            throw PyError{};
        }
}

int64_t integer(PyObject* o)
{
    long long v = PyLong_CheckExact(o) ? PyLong_AsLongLong(o) : -1;
    if (!PyLong_CheckExact(o)) {
        PyObject* i = PyNumber_Index(o);
        if (!i) throw PyError{};
        v = PyLong_AsLongLong(i);
        Py_DECREF(i);
    }
    if (v == -1 && PyErr_Occurred()) throw PyError{};
    return v;
}

int mode_of(PyObject* o, int def) { return o ? (int)integer(o) : def; }

bool given(PyObject* o) { return o && o != Py_None; }

const at::Tensor& tensor(PyObject* o, const char* what)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "%s must be a tensor", what);
    return THPVariable_Unpack(o);
}

const char* dtype_name(at::ScalarType t)
{
    switch (t) {
        case at::kByte: return "torch.uint8";
        case at::kChar: return "torch.int8";
        case at::kHalf: return "torch.float16";
        default: return "torch.float32";
    }
}

// A contiguous tensor of the wanted type on the GPU.
const at::Tensor& on_gpu(PyObject* o, at::ScalarType type, const char* what)
{
    const at::Tensor& t = tensor(o, what);
    if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) {
        PyErr_Format(PyExc_TypeError, "%s must be a contiguous %s tensor on the GPU", what, dtype_name(type));
        throw PyError{};
    }
    return t;
}

// The C-ABI trusts the sizes it is told; a buffer smaller than the shape implies is refused here.
void need(const at::Tensor& t, int64_t n, const char* what)
{
    if (t.numel() < n) fail(PyExc_ValueError, "%s holds %lld elements, the shape needs %lld", what, t.numel(), n);
}

const void* optional_ptr(PyObject* o, int64_t n, const char* what)
{
    if (!given(o)) return nullptr;
    const at::Tensor& t = tensor(o, what);
    need(t, n, what);
    return t.data_ptr();
}

const at::Tensor& packed_arg(PyObject* o, int64_t N, int64_t K, int mode)
{
    const at::Tensor& t = on_gpu(o, at::kByte, "packed");
    const size_t size = mnnq_packed_size(N, K, kGroup, mode);
    if (size == 0) {
        PyErr_Format(PyExc_ValueError, "unsupported shape N=%lld K=%lld mode=%d", (long long)N, (long long)K, mode);
        throw PyError{};
    }
    need(t, (int64_t)size, "packed");
    return t;
}

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

[[noreturn]] void raise_status(int status, const char* what)
{
    PyObject* m = PyImport_ImportModule("paper_2506_10443_amd.binding");
    PyObject* cls = m ? PyObject_GetAttrString(m, "MnnqError") : nullptr;
    PyObject* e = cls ? PyObject_CallFunction(cls, "is", status, what) : nullptr;
    if (e) PyErr_SetObject(cls, e);
    Py_XDECREF(e);
    Py_XDECREF(cls);
    Py_XDECREF(m);
    throw PyError{};
}

// Runs a C-ABI call without the interpreter lock (a launch can wait for room in the stream's queue).
template <typename F>
void call(F&& f, const char* what)
{
    int status;
    Py_BEGIN_ALLOW_THREADS;
    status = f();
    Py_END_ALLOW_THREADS;
    if (status != 0) raise_status(status, what);
}

// The output: the caller's tensor (a new reference), or a new one of the given shape.
struct Output {
    PyObject* object = nullptr;
    void* ptr = nullptr;
    ~Output() { Py_XDECREF(object); }
    Output(PyObject* out, at::IntArrayRef shape, at::ScalarType type, const at::Tensor& like, int64_t n, bool check_type)
    {
        if (given(out)) {
            const at::Tensor& t = tensor(out, "out");
            need(t, n, "out");
            if (check_type) on_gpu(out, type, "out");
            ptr = t.data_ptr();
            Py_INCREF(out);
            object = out;
        } else {
            at::Tensor t = at::empty(shape, like.options().dtype(type));
            ptr = t.data_ptr();
            object = THPVariable_Wrap(std::move(t));
            if (!object) throw PyError{};
        }
    }
    PyObject* release()
    {
        PyObject* o = object;
        object = nullptr;
        return o;
    }
};

struct Workspace {
    void* ptr = nullptr;
    size_t bytes = 0;
    at::Tensor own;
    const bool callers;
    explicit Workspace(PyObject* o) : callers(given(o))
    {
        if (!callers) return;
        const at::Tensor& t = on_gpu(o, at::kByte, "workspace");
        ptr = t.data_ptr();
        bytes = (size_t)t.numel();
    }
    void bring(const at::Tensor& like, int64_t M, int64_t N, int64_t K, int mode)
    {
        if (callers) return;     // (too small or empty: the call says so)
        const size_t n = mnnq_workspace_size(M, N, K, kGroup, mode);
        own = at::empty({(int64_t)(n < 16 ? 16 : n)}, like.options());
        ptr = own.data_ptr();
        bytes = (size_t)own.numel();
    }
};

// M of an [M, K] array; dimensions behind the second are not looked at ([M, K, 1] is one).
int64_t rows_of(const at::Tensor& t, int64_t K, const char* message)
{
    if (t.dim() < 2) fail(PyExc_IndexError, "%s", message);
    if (t.size(1) != K) fail(PyExc_ValueError, "%s", message);
    return t.size(0);
}

template <bool OUT16>
constexpr at::ScalarType out_type() { return OUT16 ? at::kHalf : at::kFloat; }

// ---- the calls

template <bool OUT16>
PyObject* decode(const Params& p, PyObject** v)   // packed, N, K, xq, sx, bias, out, mode
{
    const int64_t N = integer(v[1]), K = integer(v[2]);
    const int mode = mode_of(v[7], MNNQ_W4_ZP_INT);
    const at::Tensor& packed = packed_arg(v[0], N, K, mode);
    const at::Tensor& xq = on_gpu(v[3], at::kChar, "xq");
    const at::Tensor& sx = on_gpu(v[4], at::kFloat, "sx");
    if (xq.numel() != K) fail(PyExc_ValueError, "%s", "xq must hold K values");
    Output y(v[6], {N}, out_type<OUT16>(), packed, N, OUT16);
    const void* w = packed.data_ptr();
    const int8_t* q = static_cast<const int8_t*>(xq.data_ptr());
    const float* s = static_cast<const float*>(sx.data_ptr());
    const float* bias = static_cast<const float*>(optional_ptr(v[5], N, "bias"));
    void* st = stream();
    call([&] {
        return OUT16 ? mnnq_linear_decode_o16(w, N, K, kGroup, mode, q, s, bias, static_cast<uint16_t*>(y.ptr), st)
                     : mnnq_linear_decode(w, N, K, kGroup, mode, q, s, bias, static_cast<float*>(y.ptr), nullptr, 0, st);
    }, p.function);
    return y.release();
}

template <bool OUT16>
PyObject* decode_fused(const Params& p, PyObject** v)   // packed, N, K, x, bias, out, workspace, mode
{
    const int64_t N = integer(v[1]), K = integer(v[2]);
    const int mode = mode_of(v[7], MNNQ_W4_ZP_INT);
    const at::Tensor& packed = packed_arg(v[0], N, K, mode);
    const at::Tensor& x = on_gpu(v[3], at::kFloat, "x");
    if (x.numel() != K) fail(PyExc_ValueError, "%s", "x must hold K values");
    Output y(v[5], {N}, out_type<OUT16>(), packed, N, OUT16);
    const Workspace ws(v[6]);
    const void* w = packed.data_ptr();
    const float* xp = static_cast<const float*>(x.data_ptr());
    const float* bias = static_cast<const float*>(optional_ptr(v[4], N, "bias"));
    void* st = stream();
    call([&] {
        return OUT16 ? mnnq_linear_decode_fused_o16(w, N, K, kGroup, mode, xp, bias, static_cast<uint16_t*>(y.ptr), ws.ptr,
                                                    ws.bytes, st)
                     : mnnq_linear_decode_fused(w, N, K, kGroup, mode, xp, bias, static_cast<float*>(y.ptr), ws.ptr,
                                                ws.bytes, st);
    }, p.function);
    return y.release();
}

template <bool OUT16>
PyObject* prefill(const Params& p, PyObject** v)   // packed, N, K, xq, sx, bias, out, mode[, workspace]
{
    const int64_t N = integer(v[1]), K = integer(v[2]);
    const int mode = mode_of(v[7], MNNQ_W4_ZP_INT);
    const at::Tensor& packed = packed_arg(v[0], N, K, mode);
    const at::Tensor& xq = on_gpu(v[3], at::kChar, "xq");
    const at::Tensor& sx = on_gpu(v[4], at::kFloat, "sx");
    const int64_t M = rows_of(xq, K, "xq must be [M,K] and sx [M]");
    if (sx.numel() != M) fail(PyExc_ValueError, "%s", "xq must be [M,K] and sx [M]");
    const Workspace ws(OUT16 ? nullptr : v[8]);
    Output y(v[6], {M, N}, out_type<OUT16>(), packed, M * N, OUT16);
    const void* w = packed.data_ptr();
    const int8_t* q = static_cast<const int8_t*>(xq.data_ptr());
    const float* s = static_cast<const float*>(sx.data_ptr());
    const float* bias = static_cast<const float*>(optional_ptr(v[5], N, "bias"));
    void* st = stream();
    call([&] {
        return OUT16 ? mnnq_linear_prefill_o16(w, M, N, K, kGroup, mode, q, s, bias, static_cast<uint16_t*>(y.ptr), st)
                     : mnnq_linear_prefill(w, M, N, K, kGroup, mode, q, s, bias, static_cast<float*>(y.ptr), ws.ptr,
                                           ws.bytes, st);
    }, p.function);
    return y.release();
}

template <bool OUT16>
PyObject* prefill_fused(const Params& p, PyObject** v)   // packed, N, K, x, bias, out, workspace, mode
{
    const int64_t N = integer(v[1]), K = integer(v[2]);
    const int mode = mode_of(v[7], MNNQ_W4_ZP_INT);
    const at::Tensor& packed = packed_arg(v[0], N, K, mode);
    const at::Tensor& x = on_gpu(v[3], at::kFloat, "x");
    const int64_t M = rows_of(x, K, "x must be [M,K]");
    Workspace ws(v[6]);
    ws.bring(packed, M, N, K, mode);
    Output y(v[5], {M, N}, out_type<OUT16>(), packed, M * N, OUT16);
    const void* w = packed.data_ptr();
    const float* xp = static_cast<const float*>(x.data_ptr());
    const float* bias = static_cast<const float*>(optional_ptr(v[4], N, "bias"));
    void* st = stream();
    call([&] {
        return OUT16 ? mnnq_linear_prefill_fused_o16(w, M, N, K, kGroup, mode, xp, bias, static_cast<uint16_t*>(y.ptr),
                                                     ws.ptr, ws.bytes, st)
                     : mnnq_linear_prefill_fused(w, M, N, K, kGroup, mode, xp, bias, static_cast<float*>(y.ptr), ws.ptr,
                                                 ws.bytes, st);
    }, p.function);
    return y.release();
}

template <bool OUT16>
PyObject* decode_f16(const Params& p, PyObject** v)   // packed, N, K, x16, bias, out, mode
{
    const int64_t N = integer(v[1]), K = integer(v[2]);
    const int mode = mode_of(v[6], MNNQ_W4_ZP_INT);
    const at::Tensor& packed = packed_arg(v[0], N, K, mode);
    const at::Tensor& x = on_gpu(v[3], at::kHalf, "x16");
    if (x.numel() != K) fail(PyExc_ValueError, "%s", "x16 must hold K values");
    Output y(v[5], {N}, out_type<OUT16>(), packed, N, OUT16);
    const void* w = packed.data_ptr();
    const uint16_t* xp = static_cast<const uint16_t*>(x.data_ptr());
    const float* bias = static_cast<const float*>(optional_ptr(v[4], N, "bias"));
    void* st = stream();
    call([&] {
        return OUT16 ? mnnq_linear_decode_f16_o16(w, N, K, kGroup, mode, xp, bias, static_cast<uint16_t*>(y.ptr), st)
                     : mnnq_linear_decode_f16(w, N, K, kGroup, mode, xp, bias, static_cast<float*>(y.ptr), nullptr, 0, st);
    }, p.function);
    return y.release();
}

template <bool OUT16>
PyObject* prefill_f16(const Params& p, PyObject** v)   // packed, N, K, x16, bias, out, row_scale, mode
{
    const int64_t N = integer(v[1]), K = integer(v[2]);
    const int mode = mode_of(v[7], MNNQ_W4_ZP_INT);
    const at::Tensor& packed = packed_arg(v[0], N, K, mode);
    const at::Tensor& x = on_gpu(v[3], at::kHalf, "x16");
    const int64_t M = rows_of(x, K, "x16 must be [M,K]");
    Output y(v[5], {M, N}, out_type<OUT16>(), packed, M * N, OUT16);
    const void* w = packed.data_ptr();
    const uint16_t* xp = static_cast<const uint16_t*>(x.data_ptr());
    const float* bias = static_cast<const float*>(optional_ptr(v[4], N, "bias"));
    const float* rs = static_cast<const float*>(optional_ptr(v[6], 0, "row_scale"));
    void* st = stream();
    call([&] {
        return OUT16 ? mnnq_linear_prefill_f16_o16(w, M, N, K, kGroup, mode, xp, rs, bias, static_cast<uint16_t*>(y.ptr), st)
                     : mnnq_linear_prefill_f16(w, M, N, K, kGroup, mode, xp, rs, bias, static_cast<float*>(y.ptr), nullptr,
                                               0, st);
    }, p.function);
    return y.release();
}

PyObject* pack_weights(const Params& p, PyObject** v)   // W, out, mode
{
    const at::Tensor& W = on_gpu(v[0], at::kFloat, "W");
    if (W.dim() != 2) fail(PyExc_ValueError, "%s", "W must be [N, K]");
    const int64_t N = W.size(0), K = W.size(1);
    const int mode = mode_of(v[2], MNNQ_W4_ZP_INT);
    const float* wp = static_cast<const float*>(W.data_ptr());
    void* st = stream();
    const int64_t size = (int64_t)mnnq_packed_size(N, K, kGroup, mode);
    if (size == 0)   // the call says what is wrong with the shape (its checks run before it touches the buffer)
        call([&] { return mnnq_pack_weights(wp, N, K, kGroup, mode, const_cast<float*>(wp), 0, st); }, p.function);
    PyObject* out = v[1];
    if (given(out)) tensor(out, "out");
    // (the size of a caller's buffer is checked by the call itself: a status, not a ValueError)
    Output packed(out, {size}, at::kByte, W, 0, false);
    const size_t bytes = given(out) ? (size_t)THPVariable_Unpack(out).numel() : (size_t)size;
    call([&] { return mnnq_pack_weights(wp, N, K, kGroup, mode, packed.ptr, bytes, st); }, p.function);
    return packed.release();
}

typedef PyObject* (*Body)(const Params&, PyObject**);

PyObject* run(Params& p, Body body, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
{
    PyObject* v[kMaxArgs];
    try {
        parse(p, args, nargs, kwnames, v);
        return body(p, v);
    } catch (const PyError&) {
    } catch (...) {     // torch's own errors as its Python calls raise them (OutOfMemoryError among them)
        torch::translate_exception_to_python(std::current_exception());
    }
    return nullptr;
}

#define MNNQ_FUNCTION(NAME, BODY, REQUIRED, ...)                                                                        \
    Params params_##NAME{#NAME, (int)(sizeof((const char*[]){__VA_ARGS__}) / sizeof(char*)), REQUIRED, {__VA_ARGS__}, {}}; \
    PyObject* py_##NAME(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)                          \
    {                                                                                                                   \
        return run(params_##NAME, BODY, args, nargs, kwnames);                                                          \
    }

MNNQ_FUNCTION(mnnq_linear_decode, decode<false>, 5, "packed", "N", "K", "xq", "sx", "bias", "out", "mode")
MNNQ_FUNCTION(mnnq_linear_decode_o16, decode<true>, 5, "packed", "N", "K", "xq", "sx", "bias", "out", "mode")
MNNQ_FUNCTION(mnnq_linear_decode_fused, decode_fused<false>, 4, "packed", "N", "K", "x", "bias", "out", "workspace", "mode")
MNNQ_FUNCTION(mnnq_linear_decode_fused_o16, decode_fused<true>, 4, "packed", "N", "K", "x", "bias", "out", "workspace",
              "mode")
MNNQ_FUNCTION(mnnq_linear_prefill, prefill<false>, 5, "packed", "N", "K", "xq", "sx", "bias", "out", "mode", "workspace")
MNNQ_FUNCTION(mnnq_linear_prefill_o16, prefill<true>, 5, "packed", "N", "K", "xq", "sx", "bias", "out", "mode")
MNNQ_FUNCTION(mnnq_linear_prefill_fused, prefill_fused<false>, 4, "packed", "N", "K", "x", "bias", "out", "workspace",
              "mode")
MNNQ_FUNCTION(mnnq_linear_prefill_fused_o16, prefill_fused<true>, 4, "packed", "N", "K", "x", "bias", "out", "workspace",
              "mode")
MNNQ_FUNCTION(mnnq_linear_decode_f16, decode_f16<false>, 4, "packed", "N", "K", "x16", "bias", "out", "mode")
MNNQ_FUNCTION(mnnq_linear_decode_f16_o16, decode_f16<true>, 4, "packed", "N", "K", "x16", "bias", "out", "mode")
MNNQ_FUNCTION(mnnq_linear_prefill_f16, prefill_f16<false>, 4, "packed", "N", "K", "x16", "bias", "out", "row_scale", "mode")
MNNQ_FUNCTION(mnnq_linear_prefill_f16_o16, prefill_f16<true>, 4, "packed", "N", "K", "x16", "bias", "out", "row_scale",
              "mode")
MNNQ_FUNCTION(mnnq_pack_weights, pack_weights, 1, "W", "out", "mode")

#define MNNQ_METHOD(NAME, SIGNATURE, DOC)                                                                  \
    {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_##NAME)),                    \
     METH_FASTCALL | METH_KEYWORDS, #NAME "(" SIGNATURE ")\n--\n\n" DOC}

PyMethodDef methods[] = {
    MNNQ_METHOD(mnnq_linear_decode, "packed, N, K, xq, sx, bias=None, out=None, mode=0",
                "One token: xq i8 [K] (or [1,K]), sx f32 [1] -> y f32 [N]."),
    MNNQ_METHOD(mnnq_linear_decode_o16, "packed, N, K, xq, sx, bias=None, out=None, mode=0",
                "One token: xq i8 [K], sx f32 [1] -> y fp16 [N]."),
    MNNQ_METHOD(mnnq_linear_decode_fused, "packed, N, K, x, bias=None, out=None, workspace=None, mode=0",
                "One token, activation quantizer fused in: x f32 [K] (or [1,K]) -> y f32 [N].\n"
                "workspace: optional uint8 tensor of mnnq_workspace_size(1, N, K) bytes."),
    MNNQ_METHOD(mnnq_linear_decode_fused_o16, "packed, N, K, x, bias=None, out=None, workspace=None, mode=0",
                "One token, activation quantizer fused in: x f32 [K] -> y fp16 [N]."),
    MNNQ_METHOD(mnnq_linear_prefill, "packed, N, K, xq, sx, bias=None, out=None, mode=0, workspace=None",
                "M tokens: xq i8 [M,K], sx f32 [M] -> y f32 [M,N].  workspace: optional uint8 tensor\n"
                "(mnnq_workspace_size bytes); with the matrix-core plane in `packed` it selects the fp6 GEMM."),
    MNNQ_METHOD(mnnq_linear_prefill_o16, "packed, N, K, xq, sx, bias=None, out=None, mode=0",
                "M tokens: xq i8 [M,K], sx f32 [M] -> y fp16 [M,N]."),
    MNNQ_METHOD(mnnq_linear_prefill_fused, "packed, N, K, x, bias=None, out=None, workspace=None, mode=0",
                "M tokens, activation quantizer inside the call: x f32 [M,K] -> y f32 [M,N].\n"
                "workspace: uint8 tensor of at least mnnq_workspace_size(M, N, K) bytes (required by the library;\n"
                "this wrapper brings one along when none is given)."),
    MNNQ_METHOD(mnnq_linear_prefill_fused_o16, "packed, N, K, x, bias=None, out=None, workspace=None, mode=0",
                "M tokens, activation quantizer inside the call: x f32 [M,K] -> y fp16 [M,N]."),
    MNNQ_METHOD(mnnq_linear_decode_f16, "packed, N, K, x16, bias=None, out=None, mode=0",
                "One token, fp16 activations (W4A16; W8A16 with MODE_W8_MIN_FLOAT): x16 fp16 [K] -> y f32 [N]."),
    MNNQ_METHOD(mnnq_linear_decode_f16_o16, "packed, N, K, x16, bias=None, out=None, mode=0",
                "One token, fp16 activations: x16 fp16 [K] -> y fp16 [N]."),
    MNNQ_METHOD(mnnq_linear_prefill_f16, "packed, N, K, x16, bias=None, out=None, row_scale=None, mode=0",
                "M tokens, fp16 activations (W4A16; W8A16 with MODE_W8_MIN_FLOAT): x16 fp16 [M,K] -> y f32 [M,N];\n"
                "row_scale f32 [M] optional."),
    MNNQ_METHOD(mnnq_linear_prefill_f16_o16, "packed, N, K, x16, bias=None, out=None, row_scale=None, mode=0",
                "M tokens, fp16 activations: x16 fp16 [M,K] -> y fp16 [M,N]; row_scale f32 [M] optional."),
    MNNQ_METHOD(mnnq_pack_weights, "W, out=None, mode=0", "W fp32 [N, K] on the GPU -> packed uint8 buffer."),
    {nullptr, nullptr, 0, nullptr}};

Params* const all_params[] = {
    &params_mnnq_linear_decode, &params_mnnq_linear_decode_o16, &params_mnnq_linear_decode_fused,
    &params_mnnq_linear_decode_fused_o16, &params_mnnq_linear_prefill, &params_mnnq_linear_prefill_o16,
    &params_mnnq_linear_prefill_fused, &params_mnnq_linear_prefill_fused_o16, &params_mnnq_linear_decode_f16,
    &params_mnnq_linear_decode_f16_o16, &params_mnnq_linear_prefill_f16, &params_mnnq_linear_prefill_f16_o16,
    &params_mnnq_pack_weights};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native",
                      "The per-token calls of libmnnq.so as CPython functions; see binding.py.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void)
{
    for (Params* p : all_params)
        for (int i = 0; i < p->count; ++i)
            if (!(p->interned[i] = PyUnicode_InternFromString(p->names[i]))) return nullptr;
    return PyModule_Create(&module);
}
