// Argument marshalling of the Python binding's per-step calls (binding.py holds their signatures and
// documentation): tensors to pointers and strides, missing outputs allocated, the current stream, one call
// of the C ABI with the interpreter lock released.  A call of a few microseconds of device work spent 8 us
// in interpreted marshalling and ctypes (2.8 of them in asking for the current stream); here it is 4, of
// which 3.3 are the launch itself.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/device_lazy_init.h>
#include <torch/types.h>

#include "../../include/osc.h"

namespace {

PyObject* g_error = nullptr;  // OscError

struct PyFailed {};  // a Python exception is set

int64_t num(PyObject* o) {
    const int64_t v = PyLong_AsLongLong(o);
    if (v == -1 && PyErr_Occurred()) throw PyFailed();
    return v;
}
float real(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw PyFailed();
    return (float)v;
}
bool none(PyObject* o) { return o == Py_None; }
bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw PyFailed();
    return v != 0;
}
const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a torch tensor, got %s", Py_TYPE(o)->tp_name);
        throw PyFailed();
    }
    return THPVariable_Unpack(o);
}
void* ptr(PyObject* o) { return none(o) ? nullptr : tensor(o).data_ptr(); }
// a 2-D tensor of 16-bit elements with contiguous rows
const at::Tensor& rows16(PyObject* o) {
    const at::Tensor& t = tensor(o);
    if (!(t.dim() == 2 && t.stride(1) == 1 && t.element_size() == 2)) {
        PyErr_SetString(PyExc_AssertionError, "need a 2-D bf16 tensor");
        throw PyFailed();
    }
    return t;
}
int32_t count(PyObject* o) { return none(o) ? 0 : (int32_t)tensor(o).numel(); }
int64_t pitch(PyObject* o) { return none(o) ? 0 : tensor(o).stride(0); }
int64_t up64(int64_t n) { return (n + 63) / 64 * 64; }

// What torch.empty and torch.cuda.current_stream() do first: initialise the device, or raise torch's own error (no
// GPU; a process forked after the GPU was used).  Torch's check takes 0.1 us, so it is made once, and
// afterwards only whether this is such a forked process.
void device_ready() {
    static bool checked = false;  // under the interpreter lock
    if (checked && !torch::utils::is_device_in_bad_fork(at::kCUDA)) return;
    torch::utils::device_lazy_init(at::kCUDA);
    checked = true;
}

// an owned reference to a new tensor on t's device
PyObject* fresh(const at::Tensor& t, at::IntArrayRef size, at::ScalarType dtype) {
    if (t.is_cuda()) device_ready();
    PyObject* o = THPVariable_Wrap(at::empty(size, t.options().dtype(dtype)));
    if (!o) throw PyFailed();
    return o;
}

// owned references that die with the call unless given away
struct Ref {
    PyObject* o = nullptr;
    Ref() = default;
    Ref(const Ref&) = delete;
    Ref& operator=(const Ref&) = delete;
    ~Ref() { Py_XDECREF(o); }
    void own(PyObject* p) { o = p; }
    void share(PyObject* p) {
        Py_INCREF(p);
        o = p;
    }
    PyObject* give() {
        PyObject* p = o;
        o = nullptr;
        return p;
    }
};

void* stream() {
    device_ready();
    return c10::hip::getCurrentHIPStream().stream();
}

template <class F>
void enqueue(F&& call) {
    void* st = stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call(st);
    Py_END_ALLOW_THREADS
    if (rc == OSC_OK) return;
    PyObject* args = Py_BuildValue("(is)", rc, osc_last_error());
    if (args) {
        PyErr_SetObject(g_error, args);
        Py_DECREF(args);
    }
    throw PyFailed();
}

PyObject* tuple(std::initializer_list<Ref*> refs) {
    PyObject* t = PyTuple_New((Py_ssize_t)refs.size());
    if (!t) throw PyFailed();
    Py_ssize_t i = 0;
    for (Ref* r : refs) PyTuple_SET_ITEM(t, i++, r->give());
    return t;
}

template <PyObject* (*F)(PyObject* const*)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n, Py_ssize_t want) {
    if (n != want) {
        PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
        return nullptr;
    }
    HANDLE_TH_ERRORS
    try {
        return F(a);
    } catch (const PyFailed&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// outputs: the caller's (a sequence of `n`) or null
struct Outs {
    Ref seq;
    PyObject** item = nullptr;
    Outs(PyObject* out, Py_ssize_t n) {
        if (none(out)) return;
        seq.own(PySequence_Fast(out, "`out` is a tuple of tensors"));
        if (!seq.o) throw PyFailed();
        if (PySequence_Fast_GET_SIZE(seq.o) != n) {
            PyErr_Format(PyExc_ValueError, "`out` holds %zd tensors, expected %zd", PySequence_Fast_GET_SIZE(seq.o), n);
            throw PyFailed();
        }
        item = PySequence_Fast_ITEMS(seq.o);
    }
    explicit operator bool() const { return item != nullptr; }
};

void give_y(Ref& y, PyObject* out, int64_t M, int64_t N, int y_dtype, const at::Tensor& like) {
    if (!none(out)) y.share(out);
    else y.own(fresh(like, {M, N}, y_dtype == OSC_DT_F32 ? at::kFloat : at::kBFloat16));
}

// MXFP4 quantiser outputs (codes, scales, B): the caller's or new ones; returns the leading dimension of B
int64_t mx4_outputs(const Outs& outs, PyObject* ldb_, int32_t K_o, const at::Tensor& X, int64_t M, int64_t K, Ref& q, Ref& s, Ref& b) {
    if (outs) {
        q.share(outs.item[0]);
        s.share(outs.item[1]);
        b.share(outs.item[2]);
        return pitch(b.o);
    }
    const int64_t ldb = none(ldb_) ? up64(K_o) : num(ldb_);
    q.own(fresh(X, {M, K / 2}, at::kByte));
    s.own(fresh(X, {(int64_t)osc_act_scale_bytes(M, K)}, at::kByte));
    if (ldb) b.own(fresh(X, {M, ldb}, at::kUInt16));
    else b.share(Py_None);
    return ldb;
}

// X, oidx, fmt, ldb, out
PyObject* quantize_act(PyObject* const* a) {
    const at::Tensor& X = rows16(a[0]);
    const int64_t M = X.size(0), K = X.size(1), ldx = X.stride(0);
    const int fmt = (int)num(a[2]);
    Ref q, s, b;
    if (fmt == OSC_FMT_MXFP8 || fmt == OSC_FMT_FP8_E4M3_TOKEN) {
        const Outs outs(a[4], 2);
        if (outs) {
            q.share(outs.item[0]);
            s.share(outs.item[1]);
        } else {
            q.own(fresh(X, {M, K}, at::kByte));
            if (fmt == OSC_FMT_MXFP8) s.own(fresh(X, {(int64_t)osc_act_scale_bytes(M, K)}, at::kByte));
            else s.own(fresh(X, {M}, at::kFloat));
        }
        void *x = X.data_ptr(), *pq = ptr(q.o), *ps = ptr(s.o);
        enqueue([&](void* st) { return osc_quantize_act(x, M, K, ldx, nullptr, 0, fmt, (uint8_t*)pq, ps, nullptr, 0, st); });
        return tuple({&q, &s});
    }
    const int32_t K_o = count(a[1]);
    const Outs outs(a[4], 3);
    const int64_t ldb = mx4_outputs(outs, a[3], K_o, X, M, K, q, s, b);
    void *x = X.data_ptr(), *pi = K_o ? ptr(a[1]) : nullptr, *pq = ptr(q.o), *ps = ptr(s.o), *pb = ptr(b.o);
    enqueue([&](void* st) { return osc_quantize_act(x, M, K, ldx, (const int32_t*)pi, K_o, fmt, (uint8_t*)pq, ps, pb, ldb, st); });
    return tuple({&q, &s, &b});
}

// Xq, Xs, B, Wpack, N, K, K_o, y_dtype, out
PyObject* dual_gemm(PyObject* const* a) {
    const at::Tensor& Xq = tensor(a[0]);
    const int64_t M = Xq.size(0), N = num(a[4]), K = num(a[5]), ldb = pitch(a[2]);
    const int32_t K_o = (int32_t)num(a[6]);
    const int dt = (int)num(a[7]);
    Ref y;
    give_y(y, a[8], M, N, dt, Xq);
    const int64_t ldy = M ? tensor(y.o).stride(0) : N;
    void *q = Xq.data_ptr(), *s = ptr(a[1]), *b = ptr(a[2]), *w = ptr(a[3]), *py = ptr(y.o);
    enqueue([&](void* st) { return osc_dual_gemm((const uint8_t*)q, (const uint8_t*)s, b, ldb, w, M, N, K, K_o, py, dt, ldy, st); });
    return y.give();
}

// Xq, Xs, B, row_map, expert_offsets, T, Wpack, N, K, K_o, y_dtype, out
PyObject* grouped_dual_gemm(PyObject* const* a) {
    const int64_t T = num(a[5]), N = num(a[7]), K = num(a[8]), ldb = pitch(a[2]);
    const int32_t K_o = (int32_t)num(a[9]), E = count(a[4]) - 1;
    const int dt = (int)num(a[10]);
    Ref y;
    give_y(y, a[11], T, N, dt, tensor(a[0]));
    const int64_t ldy = T ? tensor(y.o).stride(0) : N;
    void *q = ptr(a[0]), *s = ptr(a[1]), *b = ptr(a[2]), *rm = ptr(a[3]), *off = ptr(a[4]), *w = ptr(a[6]), *py = ptr(y.o);
    enqueue([&](void* st) {
        return osc_grouped_dual_gemm((const uint8_t*)q, (const uint8_t*)s, b, ldb, (const int32_t*)rm, (const int32_t*)off, E, T, w, N, K,
                                     K_o, py, dt, ldy, st);
    });
    return y.give();
}

// X8, scales, pack, N, K, expert_offsets, y_dtype, out
template <bool MX>
PyObject* gemm8(PyObject* const* a) {
    const at::Tensor& X8 = tensor(a[0]);
    const int64_t M = X8.size(0), N = num(a[3]), K = num(a[4]);
    const int32_t E = none(a[5]) ? 0 : count(a[5]) - 1;
    const int dt = (int)num(a[6]);
    Ref y;
    give_y(y, a[7], M, N, dt, X8);
    const int64_t ldy = M ? tensor(y.o).stride(0) : N;
    void *q = X8.data_ptr(), *s = ptr(a[1]), *w = ptr(a[2]), *off = ptr(a[5]), *py = ptr(y.o);
    enqueue([&](void* st) {
        if (MX) return osc_mxfp8_gemm((const uint8_t*)q, (const uint8_t*)s, w, M, N, K, (const int32_t*)off, E, py, dt, ldy, st);
        return osc_fp8_gemm((const uint8_t*)q, (const float*)s, w, M, N, K, (const int32_t*)off, E, py, dt, ldy, st);
    });
    return y.give();
}

// X, gamma, eps, oidx, ldb, want_norm, out
PyObject* rmsnorm_quantize_act(PyObject* const* a) {
    const at::Tensor& X = rows16(a[0]);
    const int64_t M = X.size(0), K = X.size(1), ldx = X.stride(0);
    const float eps = real(a[2]);
    const int32_t K_o = count(a[3]);
    const Outs outs(a[6], 4);
    Ref q, s, b, xn;
    const int64_t ldb = mx4_outputs(outs, a[4], K_o, X, M, K, q, s, b);
    if (outs) xn.share(outs.item[3]);
    else if (truth(a[5])) xn.own(fresh(X, {M, K}, at::kUInt16));
    else xn.share(Py_None);
    void *x = X.data_ptr(), *g = ptr(a[1]), *pi = ptr(a[3]), *pq = ptr(q.o), *ps = ptr(s.o), *pb = ptr(b.o), *pn = ptr(xn.o);
    enqueue([&](void* st) {
        return osc_rmsnorm_quantize_act(x, g, eps, M, K, ldx, (const int32_t*)pi, K_o, (uint8_t*)pq, ps, pb, ldb, pn, st);
    });
    return tuple({&q, &s, &b, &xn});
}

// G, U, want_y, out
template <bool MX>
PyObject* swiglu(PyObject* const* a) {
    const at::Tensor &G = rows16(a[0]), &U = rows16(a[1]);
    if (U.sizes() != G.sizes()) {
        PyErr_SetString(PyExc_AssertionError, "gate and up differ in shape");
        throw PyFailed();
    }
    const int64_t M = G.size(0), K = G.size(1), ldg = G.stride(0), ldu = U.stride(0);
    const Outs outs(a[3], 3);
    Ref q, s, y;
    if (outs) {
        q.share(outs.item[0]);
        s.share(outs.item[1]);
        y.share(outs.item[2]);
    } else {
        q.own(fresh(G, {M, K}, at::kByte));
        if (MX) s.own(fresh(G, {(int64_t)osc_act_scale_bytes(M, K)}, at::kByte));
        else s.own(fresh(G, {M}, at::kFloat));
        if (truth(a[2])) y.own(fresh(G, {M, K}, at::kUInt16));
        else y.share(Py_None);
    }
    void *g = G.data_ptr(), *u = U.data_ptr(), *pq = ptr(q.o), *ps = ptr(s.o), *py = ptr(y.o);
    enqueue([&](void* st) {
        if (MX) return osc_swiglu_quantize_act(g, u, M, K, ldg, ldu, (uint8_t*)pq, ps, py, st);
        return osc_swiglu_quantize_act_fp8(g, u, M, K, ldg, ldu, (uint8_t*)pq, (float*)ps, py, st);
    });
    return tuple({&q, &s, &y});
}

// X, oidx, fmt16, tensor_scale, ldb, out
PyObject* quantize_act_g16(PyObject* const* a) {
    const at::Tensor& X = rows16(a[0]);
    const int64_t M = X.size(0), K = X.size(1), ldx = X.stride(0);
    const int32_t K_o = count(a[1]);
    const int fmt = (int)num(a[2]);
    const float ts = real(a[3]);
    const int64_t ldb = none(a[4]) ? up64(K_o) : num(a[4]);
    const Outs outs(a[5], 3);
    Ref q, s, b;
    if (outs) {
        q.share(outs.item[0]);
        s.share(outs.item[1]);
        b.share(outs.item[2]);
    } else {
        q.own(fresh(X, {M, K / 2}, at::kByte));
        s.own(fresh(X, {M, K / 16}, at::kByte));
        if (ldb) b.own(fresh(X, {M, ldb}, at::kUInt16));
        else b.share(Py_None);
    }
    void *x = X.data_ptr(), *pi = ptr(a[1]), *pq = ptr(q.o), *ps = ptr(s.o), *pb = ptr(b.o);
    enqueue([&](void* st) {
        return osc_quantize_act_g16(x, M, K, ldx, (const int32_t*)pi, K_o, fmt, ts, (uint8_t*)pq, (uint8_t*)ps, pb, ldb, st);
    });
    return tuple({&q, &s, &b});
}

// Xq, Xs16, B, Wpack, N, K, K_o, fmt16, x_tensor_scale, w_tensor_scale, y_dtype, out
PyObject* dual_gemm_g16(PyObject* const* a) {
    const at::Tensor& Xq = tensor(a[0]);
    const int64_t M = Xq.size(0), N = num(a[4]), K = num(a[5]), ldb = pitch(a[2]);
    const int32_t K_o = (int32_t)num(a[6]);
    const int fmt = (int)num(a[7]), dt = (int)num(a[10]);
    const float xts = real(a[8]), wts = real(a[9]);
    Ref y;
    give_y(y, a[11], M, N, dt, Xq);
    const int64_t ldy = tensor(y.o).stride(0);
    void *q = Xq.data_ptr(), *s = ptr(a[1]), *b = ptr(a[2]), *w = ptr(a[3]), *py = ptr(y.o);
    enqueue([&](void* st) {
        return osc_dual_gemm_g16((const uint8_t*)q, (const uint8_t*)s, xts, b, ldb, w, wts, M, N, K, K_o, fmt, py, dt, ldy, st);
    });
    return y.give();
}

// X, ldb, want_idx, out
PyObject* quantize_act_dynamic(PyObject* const* a) {
    const at::Tensor& X = rows16(a[0]);
    const int64_t M = X.size(0), K = X.size(1), ldx = X.stride(0);
    const int64_t ldb = none(a[1]) ? K : num(a[1]);
    const Outs outs(a[3], 4);
    Ref q, s, b, idx;
    if (outs) {
        q.share(outs.item[0]);
        s.share(outs.item[1]);
        b.share(outs.item[2]);
        idx.share(outs.item[3]);
    } else {
        q.own(fresh(X, {M, K / 2}, at::kByte));
        s.own(fresh(X, {(int64_t)osc_act_scale_bytes(M, K)}, at::kByte));
        b.own(fresh(X, {M, ldb}, at::kUInt16));
        if (truth(a[2])) idx.own(fresh(X, {M, K / 32}, at::kByte));
        else idx.share(Py_None);
    }
    void *x = X.data_ptr(), *pq = ptr(q.o), *ps = ptr(s.o), *pb = ptr(b.o), *pi = ptr(idx.o);
    enqueue([&](void* st) { return osc_quantize_act_dynamic(x, M, K, ldx, (uint8_t*)pq, ps, pb, ldb, (uint8_t*)pi, st); });
    return tuple({&q, &s, &b, &idx});
}

PyObject* current_stream(PyObject* const*) { return PyLong_FromVoidPtr(stream()); }

PyObject* bind_error(PyObject* const* a) {
    Py_INCREF(a[0]);
    Py_XSETREF(g_error, a[0]);
    Py_RETURN_NONE;
}

#define OSC_NATIVE(NAME_, FN_, N_)                                                                                          \
    {NAME_, (PyCFunction)(void (*)(void))(PyObject * (*)(PyObject*, PyObject* const*, Py_ssize_t))[](                       \
                PyObject* self, PyObject* const* a, Py_ssize_t n) -> PyObject* { return guarded<FN_>(self, a, n, N_); },    \
     METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    OSC_NATIVE("bind_error", bind_error, 1),
    OSC_NATIVE("current_stream", current_stream, 0),
    OSC_NATIVE("quantize_act", quantize_act, 5),
    OSC_NATIVE("dual_gemm", dual_gemm, 9),
    OSC_NATIVE("grouped_dual_gemm", grouped_dual_gemm, 12),
    OSC_NATIVE("fp8_gemm", gemm8<false>, 8),
    OSC_NATIVE("mxfp8_gemm", gemm8<true>, 8),
    OSC_NATIVE("rmsnorm_quantize_act", rmsnorm_quantize_act, 7),
    OSC_NATIVE("swiglu_quantize_act", swiglu<true>, 4),
    OSC_NATIVE("swiglu_quantize_act_fp8", swiglu<false>, 4),
    OSC_NATIVE("quantize_act_g16", quantize_act_g16, 6),
    OSC_NATIVE("dual_gemm_g16", dual_gemm_g16, 12),
    OSC_NATIVE("quantize_act_dynamic", quantize_act_dynamic, 4),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "argument marshalling of the per-step calls", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() { return PyModule_Create(&module); }
