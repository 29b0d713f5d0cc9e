// The hot entry points of binding.py as a CPython extension: the online calls of include/abq.h with torch tensors in
// and out.  Argument marshalling only, like the ctypes functions it stands beside.
//
// What bounds it: a decode step is one kernel of 3-7 us, and the interpreter's share of such a call was larger than the
// kernel (one step of W4A8 M = 1, 4096 x 4096, call after call: 9.4 us, of which the kernel 3.6).  Measured parts of the
// Python version: torch.empty 1.7 us, torch.cuda.current_stream 2.8, the size query through ctypes 0.4, the call through
// ctypes with 15 converted arguments 3.3 with its launch.  Here arguments arrive by vectorcall and are matched by position
// (or by interned keyword), the stream is read from c10 directly, and the tensors come from ATen without the argument
// parser of torch.empty.  The GIL is released around allocations and the library call, as torch and ctypes do.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../../include/abq.h"

namespace {

PyObject* g_error = nullptr;           // binding.AbqError(status, where)
PyObject* g_make_problems = nullptr;   // binding.make_problems(list of dicts) -> ctypes array
PyObject* g_array = nullptr;           // ctypes.Array

// ---- arguments -----------------------------------------------------------------------------------
// Parameter names of one function; the first `required` have no default (an argument not given stays null).
template <int N>
struct Signature {
    const char* function;
    int required;
    const char* names[N];
    PyObject* interned[N];

    bool parse(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, PyObject** out)
    {
        if (nargs > N) {
            PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", function, N, nargs);
            return false;
        }
        for (int i = 0; i < N; ++i) out[i] = i < nargs ? args[i] : nullptr;
        const Py_ssize_t nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
        for (Py_ssize_t k = 0; k < nkw; ++k) {
            PyObject* name = PyTuple_GET_ITEM(kwnames, k);
            int at = -1;
            for (int i = 0; i < N && at < 0; ++i)
                if (name == interned[i]) at = i;
            for (int i = 0; i < N && at < 0; ++i)
                if (PyUnicode_Compare(name, interned[i]) == 0) at = i;
            if (at < 0) {
                PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", function, name);
                return false;
            }
            if (out[at]) {
                PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", function, names[at]);
                return false;
            }
            out[at] = args[nargs + k];
        }
        for (int i = 0; i < required; ++i)
            if (!out[i]) {
                PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", function, names[i]);
                return false;
            }
        return true;
    }
    bool intern()
    {
        for (int i = 0; i < N; ++i)
            if (!(interned[i] = PyUnicode_InternFromString(names[i]))) return false;
        return true;
    }
};

// a 64-bit value as an int; nothing is cut off
bool fits_int(int64_t v, int* out)
{
    *out = (int)v;
    if (*out == v) return true;
    PyErr_Format(PyExc_OverflowError, "%lld does not fit a 32-bit integer", (long long)v);
    return false;
}
bool to_int(PyObject* o, int* out)
{
    const long v = PyLong_AsLong(o);
    return !(v == -1 && PyErr_Occurred()) && fits_int(v, out);
}
// `count` leading arguments as integers
bool to_ints(PyObject* const* a, int count, int* out)
{
    for (int i = 0; i < count; ++i)
        if (!to_int(a[i], out + i)) return false;
    return true;
}
bool is_none(PyObject* o) { return !o || o == Py_None; }

const at::Tensor* tensor(PyObject* o)
{
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
        return nullptr;
    }
    return &THPVariable_Unpack(o);
}
// address of an operand's data: a tensor, or an object with a data_ptr() of its own (a storage); None (or an argument not
// given) is the null pointer
bool pointer(PyObject* o, void** out)
{
    *out = nullptr;
    if (is_none(o)) return true;
    if (THPVariable_Check(o)) {
        *out = THPVariable_Unpack(o).data_ptr();
        return true;
    }
    PyObject* address = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (!address) return false;
    *out = PyLong_AsVoidPtr(address);
    Py_DECREF(address);
    return *out || !PyErr_Occurred();
}
// the packed weights: their address, and the device they live on, where the outputs go
struct Weights {
    void* ptr = nullptr;
    c10::optional<at::Device> on;

    bool arg(PyObject* o)
    {
        if (THPVariable_Check(o)) {
            const at::Tensor& t = THPVariable_Unpack(o);
            ptr = t.data_ptr();
            on = t.device();
            return true;
        }
        PyObject* d = PyObject_GetAttrString(o, "device");
        if (!d) return false;
        const bool is_device = THPDevice_Check(d);
        if (is_device) on = ((THPDevice*)d)->device;
        else PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
        Py_DECREF(d);
        return is_device && pointer(o, &ptr);
    }
    at::Device device() const { return *on; }
};
// the same for an argument that has to be a contiguous device tensor of this type and shape
bool checked(PyObject* o, at::ScalarType type, at::IntArrayRef shape, void** out)
{
    const at::Tensor* t = tensor(o);
    if (!t) return false;
    if (!t->is_cuda() || !t->is_contiguous() || t->scalar_type() != type || t->sizes() != shape) {
        PyErr_SetString(PyExc_AssertionError, (std::string("expected a contiguous device tensor of ") + c10::toString(type) + ", got " + c10::toString(t->scalar_type()) +
                                               " on " + t->device().str() + (t->is_contiguous() ? "" : " (not contiguous)") +
                                               (t->sizes() != shape ? " of another shape" : "")).c_str());
        return false;
    }
    *out = t->data_ptr();
    return true;
}
bool rows_cols(const at::Tensor* t, int* M, int* K)
{
    if (t->dim() != 2) {
        PyErr_SetString(PyExc_ValueError, "expected a tensor of two dimensions");
        return false;
    }
    return fits_int(t->size(0), M) && fits_int(t->size(1), K);
}

// The GIL given up for a scope, taken back however the scope is left.
struct NoGil {
    PyThreadState* const state = PyEval_SaveThread();
    NoGil() = default;
    NoGil(const NoGil&) = delete;
    ~NoGil() { PyEval_RestoreThread(state); }
};

// Memory the call makes itself: a buffer the caller may have given (its address then), or a new one where it is wanted.  Made without
// the GIL, in the same scope as the library call: an allocation may wait for the device, and torch.empty gives the GIL up too.
struct Buffer {
    at::Tensor made;
    void* ptr = nullptr;
    bool wanted = false;

    bool arg(PyObject* given, bool want)
    {
        wanted = want && is_none(given);
        return pointer(given, &ptr);
    }
    void* make(at::IntArrayRef shape, at::ScalarType type, at::Device device)
    {
        if (wanted) {
            made = at::empty(shape, at::TensorOptions().dtype(type).device(device));
            ptr = made.data_ptr();
        }
        return ptr;
    }
    uint16_t* half(int rows, int cols, at::Device device) { return (uint16_t*)make({rows, cols}, at::kHalf, device); }
    int32_t* i32(int rows, int cols, at::Device device) { return (int32_t*)make({rows, cols}, at::kInt, device); }
};
// A workspace: the caller's, or a new one where none was given and some is needed.
struct Workspace : Buffer {
    size_t bytes = 0;

    bool arg(PyObject* given, size_t need)
    {
        wanted = is_none(given) && need;
        bytes = need;
        if (is_none(given)) return true;
        if (THPVariable_Check(given)) {
            bytes = (size_t)THPVariable_Unpack(given).numel();
        } else {
            PyObject* n = PyObject_CallMethod(given, "numel", nullptr);
            if (!n) return false;
            bytes = PyLong_AsSize_t(n);
            Py_DECREF(n);
            if (bytes == (size_t)-1 && PyErr_Occurred()) return false;
        }
        return pointer(given, &ptr);
    }
    void* make(at::Device device) { return Buffer::make({(int64_t)bytes}, at::kByte, device); }
};
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }

// ---- results -------------------------------------------------------------------------------------
// new reference: the caller's own object where one was given, else the tensor made here (None if neither)
PyObject* result(PyObject* given, Buffer& b)
{
    if (!is_none(given)) { Py_INCREF(given); return given; }
    if (!b.made.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(std::move(b.made));
}
PyObject* result(Buffer& b) { return result(nullptr, b); }
PyObject* pack(std::initializer_list<PyObject*> items)
{
    PyObject* t = PyTuple_New((Py_ssize_t)items.size());
    bool ok = t != nullptr;
    Py_ssize_t i = 0;
    for (PyObject* o : items) {
        ok = ok && o;
        if (t) PyTuple_SET_ITEM(t, i++, o);
        else Py_XDECREF(o);
    }
    if (!ok) { Py_XDECREF(t); return nullptr; }
    return t;
}
PyObject* fail(int status, const char* where)
{
    if (PyObject* e = PyObject_CallFunction(g_error, "is", status, where)) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

// The allocations and the library call, without the GIL; false (with the exception set) on an error status.
template <class F>
bool call(const char* where, F&& f)
{
    const int status = [&] { NoGil no_gil; return f(); }();
    if (status == ABQ_OK) return true;
    fail(status, where);
    return false;
}

// ---- activations ---------------------------------------------------------------------------------
Signature<4> sig_quant_pack{"abq_quant_pack_act", 2, {"q", "x_fp16", "layout", "out"}};
PyObject* quant_pack_act(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS   // (torch's errors as the Python exceptions torch itself raises)
    PyObject* a[4];
    int q, layout = ABQ_LAYOUT_AUTO, M, K;
    if (!sig_quant_pack.parse(args, nargs, kw, a) || !to_int(a[0], &q) || (a[2] && !to_int(a[2], &layout))) return nullptr;
    const at::Tensor* x = tensor(a[1]);
    void* xp;
    if (!x || !rows_cols(x, &M, &K) || !checked(a[1], at::kHalf, x->sizes(), &xp)) return nullptr;
    Workspace out;
    if (!out.arg(a[3], std::max<size_t>(abq_packed_act_bytes(q, M, K, layout), 16))) return nullptr;
    if (!call("abq_quant_pack_act", [&] {
            void* o = out.make(x->device());
            return abq_quant_pack_act(q, M, K, (const uint16_t*)xp, layout, o, out.bytes, stream());
        }))
        return nullptr;
    return result(a[3], out);
    END_HANDLE_TH_ERRORS
}

Signature<6> sig_pack_codes{"abq_pack_act_codes", 4, {"q", "a_codes", "a_scale", "a_zero", "layout", "out"}};
PyObject* pack_act_codes(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[6];
    int q, layout = ABQ_LAYOUT_AUTO, M, K;
    if (!sig_pack_codes.parse(args, nargs, kw, a) || !to_int(a[0], &q) || (a[4] && !to_int(a[4], &layout))) return nullptr;
    const at::Tensor* c = tensor(a[1]);
    void *cp, *sp, *zp;
    if (!c || !rows_cols(c, &M, &K) || !checked(a[1], at::kByte, c->sizes(), &cp) || !checked(a[2], at::kFloat, {M}, &sp) ||
        !checked(a[3], at::kInt, {M}, &zp))
        return nullptr;
    Workspace out;
    if (!out.arg(a[5], std::max<size_t>(abq_packed_act_bytes(q, M, K, layout), 16))) return nullptr;
    if (!call("abq_pack_act_codes", [&] {
            void* o = out.make(c->device());
            return abq_pack_act_codes(q, M, K, (const uint8_t*)cp, (const float*)sp, (const int32_t*)zp, layout, o, out.bytes, stream());
        }))
        return nullptr;
    return result(a[5], out);
    END_HANDLE_TH_ERRORS
}

Signature<5> sig_f4_pack{"abq_f4_pack_codes", 4, {"bits", "codes", "scale", "zero", "out"}};
PyObject* f4_pack_codes(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[5];
    int bits, R, K;
    if (!sig_f4_pack.parse(args, nargs, kw, a) || !to_int(a[0], &bits)) return nullptr;
    const at::Tensor* c = tensor(a[1]);
    void *cp, *sp, *zp;
    if (!c || !rows_cols(c, &R, &K) || !checked(a[1], at::kByte, c->sizes(), &cp) || !checked(a[2], at::kFloat, {R}, &sp) ||
        !checked(a[3], at::kInt, {R}, &zp))
        return nullptr;
    Workspace out;
    if (!out.arg(a[4], std::max<size_t>(abq_f4_packed_bytes(bits, R, K), 16))) return nullptr;
    if (!call("abq_f4_pack_codes", [&] {
            void* o = out.make(c->device());
            return abq_f4_pack_codes(bits, R, K, (const uint8_t*)cp, (const float*)sp, (const int32_t*)zp, o, out.bytes, stream());
        }))
        return nullptr;
    return result(a[4], out);
    END_HANDLE_TH_ERRORS
}

// RMSNorm (with or without the residual add) and SiLU * up with the quantizer fused in
struct QuantOutputs {
    at::Tensor codes, scale, zero;
    void make(int M, int K, at::Device device)   // (without the GIL)
    {
        const auto options = at::TensorOptions().device(device);
        codes = at::empty({M, K}, options.dtype(at::kByte));
        scale = at::empty({M}, options.dtype(at::kFloat));
        zero = at::empty({M}, options.dtype(at::kInt));
    }
    uint8_t* c() { return (uint8_t*)codes.data_ptr(); }
    float* s() { return (float*)scale.data_ptr(); }
    int32_t* z() { return (int32_t*)zero.data_ptr(); }
};

Signature<5> sig_rmsnorm{"abq_rmsnorm_quant_act", 4, {"q", "x_fp16", "gamma_fp16", "eps", "want_y"}};
PyObject* rmsnorm_quant_act(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[5];
    int q, M, K;
    if (!sig_rmsnorm.parse(args, nargs, kw, a) || !to_int(a[0], &q)) return nullptr;
    const at::Tensor* x = tensor(a[1]);
    void* gp;
    if (!x || !rows_cols(x, &M, &K) || !pointer(a[2], &gp)) return nullptr;
    const double eps = PyFloat_AsDouble(a[3]);
    if (eps == -1.0 && PyErr_Occurred()) return nullptr;
    const int want = a[4] ? PyObject_IsTrue(a[4]) : 0;
    if (want < 0) return nullptr;
    QuantOutputs o;
    Buffer y;
    y.arg(nullptr, want);
    const void* xp = x->data_ptr();
    if (!call("abq_rmsnorm_quant_act", [&] {
            o.make(M, K, x->device());
            uint16_t* yp = y.half(M, K, x->device());
            return abq_rmsnorm_quant_act(q, M, K, (const uint16_t*)xp, (const uint16_t*)gp, (float)eps, o.c(), o.s(), o.z(), yp, stream());
        }))
        return nullptr;
    return pack({THPVariable_Wrap(std::move(o.codes)), THPVariable_Wrap(std::move(o.scale)), THPVariable_Wrap(std::move(o.zero)), result(y)});
    END_HANDLE_TH_ERRORS
}

Signature<7> sig_add_rmsnorm{"abq_add_rmsnorm_quant_act", 5, {"q", "x_fp16", "residual_fp16", "gamma_fp16", "eps", "want_y", "sum_out"}};
PyObject* add_rmsnorm_quant_act(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[7];
    int q, M, K;
    if (!sig_add_rmsnorm.parse(args, nargs, kw, a) || !to_int(a[0], &q)) return nullptr;
    const at::Tensor* x = tensor(a[1]);
    void *rp, *gp;
    if (!x || !rows_cols(x, &M, &K) || !pointer(a[2], &rp) || !pointer(a[3], &gp)) return nullptr;
    const double eps = PyFloat_AsDouble(a[4]);
    if (eps == -1.0 && PyErr_Occurred()) return nullptr;
    const int want = a[5] ? PyObject_IsTrue(a[5]) : 0;
    if (want < 0) return nullptr;
    QuantOutputs o;
    Buffer h, y;
    if (!h.arg(a[6], true) || !y.arg(nullptr, want)) return nullptr;
    const void* xp = x->data_ptr();
    if (!call("abq_add_rmsnorm_quant_act", [&] {
            o.make(M, K, x->device());
            uint16_t *hp = h.half(M, K, x->device()), *yp = y.half(M, K, x->device());
            return abq_add_rmsnorm_quant_act(q, M, K, (const uint16_t*)xp, (const uint16_t*)rp, (const uint16_t*)gp, (float)eps, o.c(), o.s(), o.z(),
                                             hp, yp, stream());
        }))
        return nullptr;
    return pack({THPVariable_Wrap(std::move(o.codes)), THPVariable_Wrap(std::move(o.scale)), THPVariable_Wrap(std::move(o.zero)), result(a[6], h), result(y)});
    END_HANDLE_TH_ERRORS
}

Signature<4> sig_silu{"abq_silu_mul_quant_act", 3, {"q", "gate_fp16", "up_fp16", "want_h"}};
PyObject* silu_mul_quant_act(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[4];
    int q, M, K;
    if (!sig_silu.parse(args, nargs, kw, a) || !to_int(a[0], &q)) return nullptr;
    const at::Tensor* g = tensor(a[1]);
    void* up;
    if (!g || !rows_cols(g, &M, &K) || !pointer(a[2], &up)) return nullptr;
    const int want = a[3] ? PyObject_IsTrue(a[3]) : 0;
    if (want < 0) return nullptr;
    QuantOutputs o;
    Buffer h;
    h.arg(nullptr, want);
    const void* gp = g->data_ptr();
    if (!call("abq_silu_mul_quant_act", [&] {
            o.make(M, K, g->device());
            uint16_t* hp = h.half(M, K, g->device());
            return abq_silu_mul_quant_act(q, M, K, (const uint16_t*)gp, (const uint16_t*)up, o.c(), o.s(), o.z(), hp, stream());
        }))
        return nullptr;
    return pack({THPVariable_Wrap(std::move(o.codes)), THPVariable_Wrap(std::move(o.scale)), THPVariable_Wrap(std::move(o.zero)), result(h)});
    END_HANDLE_TH_ERRORS
}

// ---- matmul --------------------------------------------------------------------------------------
Signature<13> sig_gemm{"abq_gemm", 9, {"p", "q", "M", "N", "K", "packed_act", "a_layout", "packed_w", "w_layout", "y", "acc", "want_acc", "workspace"}};
PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[13];
    int d[5], a_layout, w_layout;   // p, q, M, N, K
    if (!sig_gemm.parse(args, nargs, kw, a) || !to_ints(a, 5, d) || !to_int(a[6], &a_layout) || !to_int(a[8], &w_layout)) return nullptr;
    Weights w;
    const int want = a[11] ? PyObject_IsTrue(a[11]) : 0;
    if (want < 0 || !w.arg(a[7])) return nullptr;
    Buffer y, acc;
    Workspace ws;
    void* ap;
    if (!pointer(a[5], &ap) || !y.arg(a[9], true) || !acc.arg(a[10], want) || !ws.arg(a[12], abq_gemm_workspace_bytes(d[0], d[1], d[2], d[3], d[4]))) return nullptr;
    if (!call("abq_gemm", [&] {
            uint16_t* yp = y.half(d[2], d[3], w.device());
            int32_t* cp = acc.i32(d[2], d[3], w.device());
            void* wsp = ws.make(w.device());
            return abq_gemm(d[0], d[1], d[2], d[3], d[4], ap, a_layout, w.ptr, w_layout, yp, cp, wsp, ws.bytes, stream());
        }))
        return nullptr;
    return pack({result(a[9], y), result(a[10], acc)});
    END_HANDLE_TH_ERRORS
}

Signature<14> sig_act_codes{"abq_gemm_act_codes", 10, {"p", "q", "M", "N", "K", "a_codes", "a_scale", "a_zero", "packed_w", "w_layout", "y", "acc", "want_acc", "workspace"}};
PyObject* gemm_act_codes(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[14];
    int d[5], w_layout;
    if (!sig_act_codes.parse(args, nargs, kw, a) || !to_ints(a, 5, d) || !to_int(a[9], &w_layout)) return nullptr;
    Weights w;
    const int want = a[12] ? PyObject_IsTrue(a[12]) : 0;
    if (want < 0 || !w.arg(a[8])) return nullptr;
    Buffer y, acc;
    Workspace ws;
    void *ap, *sp, *zp;
    if (!pointer(a[5], &ap) || !pointer(a[6], &sp) || !pointer(a[7], &zp) || !y.arg(a[10], true) || !acc.arg(a[11], want) ||
        !ws.arg(a[13], abq_gemm_act_codes_workspace_bytes(d[0], d[1], d[2], d[3], d[4], w_layout)))
        return nullptr;
    if (!call("abq_gemm_act_codes", [&] {
            uint16_t* yp = y.half(d[2], d[3], w.device());
            int32_t* cp = acc.i32(d[2], d[3], w.device());
            void* wsp = ws.make(w.device());
            return abq_gemm_act_codes(d[0], d[1], d[2], d[3], d[4], (const uint8_t*)ap, (const float*)sp, (const int32_t*)zp, w.ptr, w_layout, yp, cp, wsp,
                                      ws.bytes, stream());
        }))
        return nullptr;
    return pack({result(a[10], y), result(a[11], acc)});
    END_HANDLE_TH_ERRORS
}

Signature<15> sig_requant{"abq_gemm_act_codes_requant", 13, {"p", "q", "M", "N", "K", "a_codes", "a_scale", "a_zero", "packed_w", "w_layout", "q_out", "out_scale", "out_zero", "want_y", "workspace"}};
PyObject* gemm_act_codes_requant(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[15];
    int d[5], w_layout, q_out;
    if (!sig_requant.parse(args, nargs, kw, a) || !to_ints(a, 5, d) || !to_int(a[9], &w_layout) || !to_int(a[10], &q_out)) return nullptr;
    Weights w;
    const int want = a[13] ? PyObject_IsTrue(a[13]) : 1;
    if (want < 0 || !w.arg(a[8])) return nullptr;
    void *ap, *sp, *zp, *osp, *ozp;
    if (!checked(a[11], at::kFloat, {d[2]}, &osp) || !checked(a[12], at::kInt, {d[2]}, &ozp)) return nullptr;
    Buffer codes, y;
    Workspace ws;
    if (!pointer(a[5], &ap) || !pointer(a[6], &sp) || !pointer(a[7], &zp) || !codes.arg(nullptr, true) || !y.arg(nullptr, want) ||
        !ws.arg(a[14], abq_gemm_act_codes_workspace_bytes(d[0], d[1], d[2], d[3], d[4], w_layout)))
        return nullptr;
    if (!call("abq_gemm_act_codes_requant", [&] {
            void* kp = codes.make({d[2], d[3]}, at::kByte, w.device());
            uint16_t* yp = y.half(d[2], d[3], w.device());
            void* wsp = ws.make(w.device());
            return abq_gemm_act_codes_requant(d[0], d[1], d[2], d[3], d[4], (const uint8_t*)ap, (const float*)sp, (const int32_t*)zp, w.ptr, w_layout, q_out,
                                              (const float*)osp, (const int32_t*)ozp, (uint8_t*)kp, yp, wsp, ws.bytes, stream());
        }))
        return nullptr;
    return pack({result(codes), result(y)});
    END_HANDLE_TH_ERRORS
}

Signature<12> sig_static{"abq_gemm_act_codes_static", 11, {"p", "q", "M", "N", "K", "a_codes", "a_scale", "a_zero", "packed_w", "w_layout", "y", "acc"}};
PyObject* gemm_act_codes_static(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[12];
    int d[5], w_layout;
    if (!sig_static.parse(args, nargs, kw, a) || !to_ints(a, 5, d) || !to_int(a[9], &w_layout)) return nullptr;
    void *ap, *sp, *zp, *wp, *yp, *cp;
    if (!pointer(a[5], &ap) || !pointer(a[6], &sp) || !pointer(a[7], &zp) || !pointer(a[8], &wp) || !pointer(a[10], &yp) || !pointer(a[11], &cp)) return nullptr;
    if (!call("abq_gemm_act_codes_static", [&] {
            return abq_gemm_act_codes_static(d[0], d[1], d[2], d[3], d[4], (const uint8_t*)ap, (const float*)sp, (const int32_t*)zp, wp, w_layout,
                                             (uint16_t*)yp, (int32_t*)cp, stream());
        }))
        return nullptr;
    Buffer none;
    return pack({result(a[10], none), result(a[11], none)});
    END_HANDLE_TH_ERRORS
}

Signature<10> sig_f4_gemm{"abq_f4_gemm", 7, {"p", "q", "M", "N", "K", "packed_act", "packed_w", "y", "acc", "want_acc"}};
PyObject* f4_gemm(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[10];
    int d[5];
    if (!sig_f4_gemm.parse(args, nargs, kw, a) || !to_ints(a, 5, d)) return nullptr;
    Weights w;
    const int want = a[9] ? PyObject_IsTrue(a[9]) : 0;
    if (want < 0 || !w.arg(a[6])) return nullptr;
    Buffer y, acc;
    void* ap;
    if (!pointer(a[5], &ap) || !y.arg(a[7], true) || !acc.arg(a[8], want)) return nullptr;
    if (!call("abq_f4_gemm", [&] {
            uint16_t* yp = y.half(d[2], d[3], w.device());
            int32_t* cp = acc.i32(d[2], d[3], w.device());
            return abq_f4_gemm(d[0], d[1], d[2], d[3], d[4], ap, w.ptr, yp, cp, stream());
        }))
        return nullptr;
    return pack({result(a[7], y), result(a[8], acc)});
    END_HANDLE_TH_ERRORS
}

Signature<7> sig_grouped{"abq_gemm_grouped", 6, {"p", "q", "M", "problems", "a_layout", "w_layout", "workspace"}};
PyObject* gemm_grouped(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kw)
{
    HANDLE_TH_ERRORS
    PyObject* a[7];
    int d[3], a_layout, w_layout;
    if (!sig_grouped.parse(args, nargs, kw, a) || !to_ints(a, 3, d) || !to_int(a[4], &a_layout) || !to_int(a[5], &w_layout)) return nullptr;
    PyObject* arr = a[3];   // the ctypes array of make_problems, or what make_problems takes
    Py_INCREF(arr);
    const int is_array = PyObject_IsInstance(arr, g_array);
    if (is_array < 0) { Py_DECREF(arr); return nullptr; }
    if (!is_array) {
        PyObject* made = PyObject_CallOneArg(g_make_problems, arr);
        Py_DECREF(arr);
        if (!(arr = made)) return nullptr;
    }
    Py_buffer view;
    const int got = PyObject_GetBuffer(arr, &view, PyBUF_SIMPLE);
    Py_DECREF(arr);   // (the view holds it)
    if (got != 0) return nullptr;
    struct Release { Py_buffer* v; ~Release() { PyBuffer_Release(v); } } release{&view};
    if (view.len % (Py_ssize_t)sizeof(abq_problem) != 0) {
        PyErr_SetString(PyExc_TypeError, "problems: an array of make_problems, or a list of dicts");
        return nullptr;
    }
    const int count = (int)(view.len / (Py_ssize_t)sizeof(abq_problem));
    const abq_problem* pr = (const abq_problem*)view.buf;
    Workspace ws;
    if (!ws.arg(a[6], is_none(a[6]) ? abq_gemm_grouped_workspace_bytes(d[0], d[1], d[2], count, pr, a_layout, w_layout) : 0)) return nullptr;
    if (!call("abq_gemm_grouped", [&] {
            void* wsp = ws.make(at::kCUDA);
            return abq_gemm_grouped(d[0], d[1], d[2], count, pr, a_layout, w_layout, wsp, ws.bytes, stream());
        }))
        return nullptr;
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

// binding.py hands over its exception class, make_problems and ctypes.Array once
PyObject* init(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs != 3) {
        PyErr_SetString(PyExc_TypeError, "init(error, make_problems, array)");
        return nullptr;
    }
    for (int i = 0; i < 3; ++i) Py_INCREF(args[i]);
    g_error = args[0];
    g_make_problems = args[1];
    g_array = args[2];
    Py_RETURN_NONE;
}

#define ABQ_METHOD(NAME, FN, DOC) {NAME, (PyCFunction)(void (*)(void))FN, METH_FASTCALL | METH_KEYWORDS, DOC}
PyMethodDef methods[] = {
    ABQ_METHOD("abq_quant_pack_act", quant_pack_act,
               "abq_quant_pack_act(q, x_fp16, layout=0, out=None)\n--\n\nx_fp16 float16 [M,K] (device) -> packed activation blob."),
    ABQ_METHOD("abq_pack_act_codes", pack_act_codes,
               "abq_pack_act_codes(q, a_codes, a_scale, a_zero, layout=0, out=None)\n--\n\na_codes uint8 [M,K], a_scale float32 [M], a_zero int32 [M] (device) -> packed activation blob."),
    ABQ_METHOD("abq_f4_pack_codes", f4_pack_codes,
               "abq_f4_pack_codes(bits, codes, scale, zero, out=None)\n--\n\ncodes uint8 [rows,K] (weights: rows = N; activations: rows = M) -> blob of the 4-bit floating-point MFMA path."),
    ABQ_METHOD("abq_rmsnorm_quant_act", rmsnorm_quant_act,
               "abq_rmsnorm_quant_act(q, x_fp16, gamma_fp16, eps, want_y=False)\n--\n\n-> (codes uint8 [M,K], a_scale float32 [M], a_zero int32 [M], y float16 [M,K] or None)."),
    ABQ_METHOD("abq_add_rmsnorm_quant_act", add_rmsnorm_quant_act,
               "abq_add_rmsnorm_quant_act(q, x_fp16, residual_fp16, gamma_fp16, eps, want_y=False, sum_out=None)\n--\n\n-> (codes, a_scale, a_zero, h = x + residual as float16 [M,K], y float16 [M,K] or None)."),
    ABQ_METHOD("abq_silu_mul_quant_act", silu_mul_quant_act,
               "abq_silu_mul_quant_act(q, gate_fp16, up_fp16, want_h=False)\n--\n\n-> (codes uint8 [M,K], a_scale float32 [M], a_zero int32 [M], h float16 [M,K] or None)."),
    ABQ_METHOD("abq_gemm", gemm,
               "abq_gemm(p, q, M, N, K, packed_act, a_layout, packed_w, w_layout, y=None, acc=None, want_acc=False, workspace=None)\n--\n\n-> (y float16 [M,N], acc int32 [M,N] or None).  Buffers are allocated when not given."),
    ABQ_METHOD("abq_gemm_act_codes", gemm_act_codes,
               "abq_gemm_act_codes(p, q, M, N, K, a_codes, a_scale, a_zero, packed_w, w_layout, y=None, acc=None, want_acc=False, workspace=None)\n--\n\nActivation packing fused into the matmul -> (y float16 [M,N], acc int32 [M,N] or None)."),
    ABQ_METHOD("abq_gemm_act_codes_requant", gemm_act_codes_requant,
               "abq_gemm_act_codes_requant(p, q, M, N, K, a_codes, a_scale, a_zero, packed_w, w_layout, q_out, out_scale, out_zero, want_y=True, workspace=None)\n--\n\n-> (codes uint8 [M,N] of the next layer under (out_scale, out_zero), y float16 [M,N] or None)."),
    ABQ_METHOD("abq_gemm_act_codes_static", gemm_act_codes_static,
               "abq_gemm_act_codes_static(p, q, M, N, K, a_codes, a_scale, a_zero, packed_w, w_layout, y, acc=None)\n--\n\nabq_gemm_act_codes without a workspace and without any allocation: the caller passes every buffer."),
    ABQ_METHOD("abq_f4_gemm", f4_gemm,
               "abq_f4_gemm(p, q, M, N, K, packed_act, packed_w, y=None, acc=None, want_acc=False)\n--\n\n-> (y float16 [M,N], acc int32 [M,N] or None)."),
    ABQ_METHOD("abq_gemm_grouped", gemm_grouped,
               "abq_gemm_grouped(p, q, M, problems, a_layout, w_layout, workspace=None)\n--\n\nOne call for a list of independent problems that share p, q, M (see make_problems); outputs are written to\nthe y / acc tensors of each problem."),
    {"init", (PyCFunction)(void (*)(void))init, METH_FASTCALL, "init(error, make_problems, array)"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "abq_native", "The online entry points of libabq with torch tensors in and out.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_abq_native()
{
    if (!(sig_quant_pack.intern() && sig_pack_codes.intern() && sig_f4_pack.intern() && sig_rmsnorm.intern() && sig_add_rmsnorm.intern() && sig_silu.intern() &&
          sig_gemm.intern() && sig_act_codes.intern() && sig_requant.intern() && sig_static.intern() && sig_f4_gemm.intern() && sig_grouped.intern()))
        return nullptr;
    return PyModule_Create(&module_def);
}
