// The Python binding's plain calls, natively: take the tensors apart, allocate the outputs, call the C ABI on torch's current stream.
// What such a call costs the host bounds every small shape (quantize Q, K, V of one 128 x 64 head and attend: 26.1 us a pass with the
// arguments taken apart and the seven outputs allocated in Python, 11.1 like this, of which the two kernels take 6.6; a first pass on new inputs 38 and 24).
//
// Every function returns None for anything but the plain case -- a tensor subclass, an active torch function or dispatch mode, a tensor
// that is not contiguous, not on the current device or of another type, shapes that do not agree, a call that the C ABI refuses -- and
// the binding then takes its general path, which handles or refuses it.  An error of the HIP runtime is raised from here.  The C ABI is
// reached through the addresses that init() is given, those of the library the binding has loaded.  The GIL is released around a call, as ctypes does.
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include <climits>
#include <cstring>

#include "intfa.h"

namespace {

struct Abi {
    decltype(&::quantize_tokenwise_ex) tokenwise;
    decltype(&::quantize_headwise_ex) headwise;
    decltype(&::quantize_blockwise) blockwise;
    decltype(&::quantize_qkv) qkv;
    decltype(&::quantize_qk) qk;
    decltype(&::int_flash_attn_fwd_rect) fwd;
    decltype(&::int_flash_attn_fwd_vblock_rect) vblock;
    decltype(&::int_flash_attn_fwd_half_rect) half;
    decltype(&::int_flash_attn_fwd_splitk) splitk;
    decltype(&::int_flash_attn_fwd_splitk_static) splitk_static;
    decltype(&::ifa_block_cols) block_cols;
} abi;
constexpr int ABI_FUNCTIONS = sizeof(Abi) / sizeof(void *);
PyObject *check = nullptr;                                       // the binding's: check(status, name of the call) raises what such a status raises

// init(check, address of every function of Abi)
PyObject *init(PyObject *, PyObject *const *args, Py_ssize_t n) {
    if (n != 1 + ABI_FUNCTIONS) { PyErr_SetString(PyExc_TypeError, "init: check() and one address per function of the C ABI"); return nullptr; }
    void *p[ABI_FUNCTIONS];
    for (int i = 0; i < ABI_FUNCTIONS; ++i) {
        p[i] = PyLong_AsVoidPtr(args[1 + i]);
        if (!p[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "init: null address"); return nullptr; }
    }
    memcpy(&abi, p, sizeof p);
    Py_INCREF(args[0]);
    Py_XSETREF(check, args[0]);
    Py_RETURN_NONE;
}

// A plain tensor: contiguous, with storage of its own kind on the current device
const at::Tensor *plain(PyObject *o, c10::DeviceIndex device) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && !t.is_neg() && !t.is_conj() && t.numel() > 0 &&
           t.device().index() == device && t.is_contiguous() ? &t : nullptr;
}
bool modes() { return at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set(); }
int dtype_enum(at::ScalarType t) { return t == at::kFloat ? IFA_F32 : t == at::kHalf ? IFA_F16 : t == at::kBFloat16 ? IFA_BF16 : -1; }
signed char *i8(const at::Tensor &t) { return static_cast<signed char *>(t.data_ptr()); }
float *f32(const at::Tensor &t) { return static_cast<float *>(t.data_ptr()); }
// Outputs, straight from the caching allocator: nothing between here and there (autograd of integers, a mode, a subclass) has anything to do for a
// plain call, and every output is written whole.  The six outputs of quantize_qkv: 2.9 us of host, 4.9 through the dispatcher.
at::Tensor like(const at::Tensor &x, at::ScalarType dtype) { return at::detail::empty_strided_cuda(x.sizes(), x.strides(), dtype, x.device()); }
at::Tensor codes(const at::Tensor &x) { return like(x, at::kChar); }
at::Tensor scales(const at::Tensor &x, at::IntArrayRef shape) { return at::detail::empty_cuda(shape, at::kFloat, x.device(), std::nullopt); }
// One call of the C ABI (which does not throw) without the GIL.  The arguments, data_ptr() among them, which can throw, are evaluated before it is released.
template <typename... P, typename... A> int unlocked(int (*fn)(P...), A... a) {
    PyThreadState *const state = PyEval_SaveThread();
    const int rc = fn(a...);
    PyEval_RestoreThread(state);
    return rc;
}
// False for a refusal, which comes before anything is enqueued and which the general path repeats and reports; a HIP error is raised at once:
// the runtime has forgotten it by the time of a second call, which would enqueue again what the first one has.
bool succeeded(int rc, const char *what) {
    if (rc == IFA_ERR_HIP) Py_XDECREF(PyObject_CallFunction(check, "is", rc, what));
    return rc == IFA_OK;
}
// C++ exceptions end here: the general path meets the same condition and says so
template <typename F> PyObject *guarded(F f) {
    try {
        if (modes()) Py_RETURN_NONE;
        PyObject *r = f(c10::hip::current_device());
        if (r || PyErr_Occurred()) return r;
    } catch (const std::exception &) {
    }
    Py_RETURN_NONE;
}
PyObject *tuple(std::initializer_list<at::Tensor> ts) {
    PyObject *t = PyTuple_New(static_cast<Py_ssize_t>(ts.size()));
    if (!t) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor &x : ts) {
        PyObject *o = THPVariable_Wrap(x);
        if (!o) { Py_DECREF(t); return nullptr; }
        PyTuple_SET_ITEM(t, i++, o);
    }
    return t;
}
bool number(PyObject *o, double &v) {                            // a plain Python float or int; anything else goes the general way
    if (PyFloat_CheckExact(o)) { v = PyFloat_AS_DOUBLE(o); return true; }
    if (!PyLong_CheckExact(o)) return false;
    v = PyLong_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); return false; }
    return true;
}
hipStream_t stream(c10::DeviceIndex device) { return c10::hip::getCurrentHIPStream(device).stream(); }

// quantize_tokenwise(X, scale_mul)
PyObject *tokenwise(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        double mul;
        const at::Tensor *x = n == 2 ? plain(a[0], dev) : nullptr;
        if (!x || x->dim() < 1 || !number(a[1], mul) || dtype_enum(x->scalar_type()) < 0) return nullptr;
        const auto shape = x->sizes();
        const long d = shape.back();
        at::Tensor q = codes(*x), s = scales(*x, shape.slice(0, shape.size() - 1));
        const hipStream_t st = stream(dev);
        const int rc = unlocked(abi.tokenwise, x->data_ptr(), dtype_enum(x->scalar_type()), x->numel() / d, static_cast<int>(d), i8(q), f32(s), static_cast<float>(mul), st);
        return succeeded(rc, "quantize_tokenwise") ? tuple({q, s}) : nullptr;
    });
}

// quantize_headwise(X)
PyObject *headwise(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        const at::Tensor *x = n == 1 ? plain(a[0], dev) : nullptr;
        if (!x || x->dim() < 2 || dtype_enum(x->scalar_type()) < 0) return nullptr;
        const auto shape = x->sizes();
        const long d = shape.back(), N = shape[shape.size() - 2];
        at::Tensor q = codes(*x), s = scales(*x, shape.slice(0, shape.size() - 2));
        const hipStream_t st = stream(dev);
        const int rc = unlocked(abi.headwise, x->data_ptr(), dtype_enum(x->scalar_type()), x->numel() / (N * d), N, d, i8(q), f32(s), 0, st);
        return succeeded(rc, "quantize_headwise_ex") ? tuple({q, s}) : nullptr;
    });
}

// quantize_blockwise(X, block_keys)
PyObject *blockwise(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        const at::Tensor *x = n == 2 ? plain(a[0], dev) : nullptr;
        if (!x || x->dim() < 2 || dtype_enum(x->scalar_type()) < 0 || !PyLong_CheckExact(a[1])) return nullptr;
        int overflow = 0;
        const long block = PyLong_AsLongAndOverflow(a[1], &overflow);
        if (overflow || block <= 0 || block > INT_MAX) return nullptr;
        const auto shape = x->sizes();
        const long d = shape.back(), N = shape[shape.size() - 2];
        if (d > INT_MAX) return nullptr;
        c10::SmallVector<int64_t, 5> sshape(shape.begin(), shape.end() - 1);
        sshape.back() = (N + block - 1) / block;
        at::Tensor q = codes(*x), s = scales(*x, sshape);
        const hipStream_t st = stream(dev);
        const int rc = unlocked(abi.blockwise, x->data_ptr(), dtype_enum(x->scalar_type()), x->numel() / (N * d), N, static_cast<int>(d), static_cast<int>(block), i8(q), f32(s), st);
        return succeeded(rc, "quantize_blockwise") ? tuple({q, s}) : nullptr;
    });
}

// quantize_qkv(Q, K, V, s_Q_mul)
PyObject *qkv(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        double mul;
        const at::Tensor *q = n == 4 ? plain(a[0], dev) : nullptr, *k = q ? plain(a[1], dev) : nullptr, *v = k ? plain(a[2], dev) : nullptr;
        if (!v || q->dim() < 2 || !number(a[3], mul)) return nullptr;
        const int dt = dtype_enum(q->scalar_type());
        if (dt < 0 || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() || k->sizes() != q->sizes() || v->sizes() != q->sizes()) return nullptr;
        const auto shape = q->sizes();
        const long d = shape.back(), N = shape[shape.size() - 2];
        at::Tensor q8 = codes(*q), k8 = codes(*q), v8 = codes(*q);
        at::Tensor sq = scales(*q, shape.slice(0, shape.size() - 1)), sk = scales(*q, shape.slice(0, shape.size() - 1)), sv = scales(*q, shape.slice(0, shape.size() - 2));
        const hipStream_t st = stream(dev);
        const int rc = unlocked(abi.qkv, q->data_ptr(), k->data_ptr(), v->data_ptr(), dt, q->numel() / (N * d), N, static_cast<int>(d), i8(q8), i8(k8), i8(v8), f32(sq), f32(sk), f32(sv), static_cast<float>(mul), st);
        return succeeded(rc, "quantize_qkv") ? tuple({q8, k8, v8, sq, sk, sv}) : nullptr;
    });
}

// quantize_qk(Q, K, s_Q_mul, hadamard)
PyObject *qk(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        double mul;
        const at::Tensor *q = n == 4 ? plain(a[0], dev) : nullptr, *k = q ? plain(a[1], dev) : nullptr;
        if (!k || q->dim() < 1 || !number(a[2], mul) || !PyBool_Check(a[3])) return nullptr;
        const int dt = dtype_enum(q->scalar_type()), had = a[3] == Py_True;
        if (dt < 0 || k->scalar_type() != q->scalar_type() || k->sizes() != q->sizes()) return nullptr;
        const auto shape = q->sizes();
        const long d = shape.back();
        at::Tensor q8 = codes(*q), k8 = codes(*q), sq = scales(*q, shape.slice(0, shape.size() - 1)), sk = scales(*q, shape.slice(0, shape.size() - 1));
        const hipStream_t st = stream(dev);
        const int rc = unlocked(abi.qk, q->data_ptr(), k->data_ptr(), dt, q->numel() / d, static_cast<int>(d), i8(q8), i8(k8), f32(sq), f32(sk), static_cast<float>(mul), had, st);
        return succeeded(rc, "quantize_qk") ? tuple({q8, k8, sq, sk}) : nullptr;
    });
}

// The operands of an attention call: int8 Q [B, H, Nq, d], K, V [B, H, Nk, d] (V of `vtype`), s_Q, s_K, and the output type
struct Call {
    const at::Tensor *q, *k, *v, *sq, *sk, *sv = nullptr;
    int B, H, Nq, Nk, d, causal, o_dtype;
    at::Tensor out;
    bool take(PyObject *const *a, c10::DeviceIndex dev, at::ScalarType vtype, PyObject *s_v, PyObject *causal_, PyObject *out_dtype) {
        if (!(q = plain(a[0], dev)) || !(k = plain(a[1], dev)) || !(v = plain(a[2], dev)) || !(sq = plain(a[3], dev)) || !(sk = plain(a[4], dev))) return false;
        if (s_v && (!(sv = plain(s_v, dev)) || sv->scalar_type() != at::kFloat)) return false;
        if (q->scalar_type() != at::kChar || k->scalar_type() != at::kChar || v->scalar_type() != vtype || sq->scalar_type() != at::kFloat || sk->scalar_type() != at::kFloat) return false;
        if (q->dim() != 4 || k->dim() != 4 || v->sizes() != k->sizes() || sq->sizes() != q->sizes().slice(0, 3) || sk->sizes() != k->sizes().slice(0, 3)) return false;
        if (k->size(0) != q->size(0) || k->size(1) != q->size(1) || k->size(3) != q->size(3)) return false;
        for (const at::Tensor *t : {q, k})
            for (const auto s : t->sizes()) if (s > INT_MAX) return false;
        B = static_cast<int>(q->size(0)), H = static_cast<int>(q->size(1)), Nq = static_cast<int>(q->size(2)), Nk = static_cast<int>(k->size(2)), d = static_cast<int>(q->size(3));
        if (!PyBool_Check(causal_)) return false;
        causal = causal_ == Py_True;
        const at::ScalarType ot = out_dtype == Py_None ? at::kHalf : THPDtype_Check(out_dtype) ? reinterpret_cast<THPDtype *>(out_dtype)->scalar_type : at::kChar;
        if ((o_dtype = dtype_enum(ot)) < 0) return false;
        out = like(*q, ot);
        return true;
    }
};

// fwd(Q, K, V, s_Q, s_K, s_V, causal, out_dtype)
PyObject *fwd(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        Call c;
        if (n != 8 || !c.take(a, dev, at::kChar, a[5], a[6], a[7])) return nullptr;
        const bool vb = c.sv->dim() == 3;
        if (vb) {
            const int bc = abi.block_cols(c.d, c.causal);
            if (bc <= 0 || c.sv->size(0) != c.B || c.sv->size(1) != c.H || c.sv->size(2) != (c.Nk + bc - 1) / bc) return nullptr;
        } else if (c.sv->numel() < static_cast<int64_t>(c.B) * c.H) return nullptr;              // a scale of every head is read
        const hipStream_t st = stream(dev);
        const int rc = unlocked(vb ? abi.vblock : abi.fwd, i8(*c.q), i8(*c.k), i8(*c.v), f32(*c.sq), f32(*c.sk), f32(*c.sv), c.B, c.H, c.Nq, c.Nk, c.d, c.causal, c.out.data_ptr(), c.o_dtype, st);
        return succeeded(rc, "int_flash_attn_fwd") ? THPVariable_Wrap(c.out) : nullptr;
    });
}

// half(Q, K, V, s_Q, s_K, causal, out_dtype)
PyObject *half(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        Call c;
        if (n != 7 || !c.take(a, dev, at::kHalf, nullptr, a[5], a[6])) return nullptr;
        const hipStream_t st = stream(dev);
        const int rc = unlocked(abi.half, i8(*c.q), i8(*c.k), c.v->data_ptr(), f32(*c.sq), f32(*c.sk), c.B, c.H, c.Nq, c.Nk, c.d, c.causal, c.out.data_ptr(), c.o_dtype, st);
        return succeeded(rc, "int_flash_attn_fwd_half") ? THPVariable_Wrap(c.out) : nullptr;
    });
}

// splitk(Q, K, V, s_Q, s_K, s_V, causal, out_dtype, workspace or None for the built-in one)
PyObject *splitk(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return guarded([&](c10::DeviceIndex dev) -> PyObject * {
        Call c;
        const at::Tensor *ws = nullptr;
        if (n != 9 || (a[8] != Py_None && (!(ws = plain(a[8], dev)) || ws->scalar_type() != at::kByte))) return nullptr;
        if (!c.take(a, dev, at::kChar, a[5], a[6], a[7]) || c.sv->dim() != 2 || c.sv->size(0) != c.B || c.sv->size(1) != c.H) return nullptr;
        const hipStream_t st = stream(dev);
        const int rc = ws ? unlocked(abi.splitk, i8(*c.q), i8(*c.k), i8(*c.v), f32(*c.sq), f32(*c.sk), f32(*c.sv), c.B, c.H, c.Nq, c.Nk, c.d, c.causal, c.out.data_ptr(), c.o_dtype, ws->data_ptr(), ws->numel(), st)
                          : unlocked(abi.splitk_static, i8(*c.q), i8(*c.k), i8(*c.v), f32(*c.sq), f32(*c.sk), f32(*c.sv), c.B, c.H, c.Nq, c.Nk, c.d, c.causal, c.out.data_ptr(), c.o_dtype, st);
        return succeeded(rc, ws ? "int_flash_attn_fwd_splitk" : "int_flash_attn_fwd_splitk_static") ? THPVariable_Wrap(c.out) : nullptr;
    });
}

#define FASTCALL(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FASTCALL(init), FASTCALL(tokenwise), FASTCALL(headwise), FASTCALL(blockwise), FASTCALL(qkv), FASTCALL(qk), FASTCALL(fwd), FASTCALL(half), FASTCALL(splitk), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_intfa_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__intfa_host() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", INTFA_TORCH_VERSION) < 0) Py_CLEAR(m);      // the one whose internals it was built for
    return m;
}
