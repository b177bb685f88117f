// The calls a program makes most, marshalled natively: plain tensors on the current GPU and its current stream, outputs and
// workspace allocated here.  Every function returns None for anything else (another type, layout, device, a stream or a
// buffer of the caller's, a mode or transform of torch's that is active, a status that is not success); binding.py then
// takes its own path, which says what is wrong or does what this one does not.
//
// A call of a small problem is as long as its host side: hyena_se_fwd of 1 x 1024 x 256 fp32 took 6.9 us through ctypes, of
// which the checks, the output and the conversions were 3.3 and the launch 3; through here 4.1, where the kernel bounds it.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/VirtualGuardImpl.h>

#include "hyena.h"

namespace {

using Gated = decltype(&hyena_se_fwd);
using GatedBwd = decltype(&hyena_se_bwd);

// addresses in the loaded library (init), and torch's current raw stream by device index
struct Entries {
    Gated gated[2];
    GatedBwd bwd[2];
    decltype(&hyena_bwd_workspace_bytes) bwd_workspace;
    decltype(&hyena_chain_fwd) chain_fwd;
    decltype(&hyena_chain_workspace_bytes) chain_workspace;
    decltype(&hyena_chain_bwd) chain_bwd;
    decltype(&hyena_chain_bwd_workspace_bytes) chain_bwd_workspace;
    decltype(&hyena_li_fwd) li_fwd;
    decltype(&hyena_li_workspace_bytes) li_workspace;
} e;
constexpr int kEntries = 11;
static_assert(sizeof(Entries) == kEntries * sizeof(void*), "a table of addresses");
PyObject* raw_stream = nullptr;

// Nothing that would have a say in the calls this file makes: torch function and dispatch modes, functorch transforms.
bool plain_context() {
    static const c10::DispatchKeySet usual({c10::DispatchKey::BackendSelect, c10::DispatchKey::ADInplaceOrView});
    return (c10::impl::tls_local_dispatch_key_set().included_ - usual).empty() && !at::impl::torch_function_mode_enabled();
}

const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    static const c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                              c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                              c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || t.key_set().has_any(wrapped) || !t.is_contiguous())
        return nullptr;
    return &t;
}

struct Problem {
    int64_t B, L, D, group;
    int code;
    const at::Tensor* x[4];
    void* stream;
};

// n activations of one shape, on the current GPU
bool activations(PyObject* const* a, int n, PyObject* group, Problem& p) {
    if (!raw_stream || !plain_context() || !PyLong_CheckExact(group)) return false;
    for (int i = 0; i < n; ++i) {
        p.x[i] = plain(a[i]);
        if (!p.x[i]) return false;
    }
    const at::Tensor& x = *p.x[0];
    if (x.dim() != 3 || x.numel() == 0) return false;
    const auto type = x.scalar_type();
    if (type != at::kFloat && type != at::kBFloat16) return false;
    for (int i = 1; i < n; ++i)
        if (p.x[i]->sizes() != x.sizes() || p.x[i]->scalar_type() != type || p.x[i]->device() != x.device()) return false;
    if (c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice() != x.device()) return false;
    p.B = x.size(0);
    p.L = x.size(1);
    p.D = x.size(2);
    p.code = type == at::kFloat ? HY_F32 : HY_BF16;
    int overflow = 0;
    p.group = PyLong_AsLongLongAndOverflow(group, &overflow);
    if (overflow || p.group < 1 || p.group > 0x7fffffff) return false;
    PyObject* index = PyLong_FromLong(x.device().index());
    if (!index) throw python_error();
    PyObject* s = PyObject_CallOneArg(raw_stream, index);
    Py_DECREF(index);
    if (!s) throw python_error();
    p.stream = PyLong_AsVoidPtr(s);
    Py_DECREF(s);
    if (PyErr_Occurred()) throw python_error();
    return true;
}

// taps per filter of a [D / group, taps] table beside the activations, or 0
int32_t filter(PyObject* o, const Problem& p, int64_t group, const at::Tensor*& t) {
    t = plain(o);
    if (!t || t->scalar_type() != at::kFloat || t->dim() != 2 || t->device() != p.x[0]->device() || p.D % group != 0 ||
        t->size(0) != p.D / group || t->size(1) < 1 || t->size(1) > 0x7fffffff)
        return 0;
    return (int32_t)t->size(1);
}

at::Tensor workspace(const Problem& p, int64_t bytes) {
    return bytes > 0 ? at::empty({bytes}, p.x[0]->options().dtype(at::kByte)) : at::Tensor();
}
void* address(const at::Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }

template <typename F>
bool launched(F&& call) {
    hy_status rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return rc == HY_OK;
}

PyObject* tuple_of(std::initializer_list<at::Tensor> ts) {
    PyObject* r = PyTuple_New((Py_ssize_t)ts.size());
    if (!r) throw python_error();
    Py_ssize_t i = 0;
    for (const at::Tensor& t : ts) {
        PyObject* o = THPVariable_Wrap(t);
        if (!o) {
            Py_DECREF(r);
            throw python_error();
        }
        PyTuple_SET_ITEM(r, i++, o);
    }
    return r;
}

// (0: hyena_se_fwd, 1: hyena_mr_fwd; q, k, v, h, group)
PyObject* gated(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Problem p;
    const at::Tensor* h;
    if (n != 6 || !activations(a + 1, 3, a[5], p)) Py_RETURN_NONE;
    const int32_t lh = filter(a[4], p, p.group, h);
    if (!lh) Py_RETURN_NONE;
    const Gated fn = e.gated[PyLong_AsLong(a[0]) != 0];
    at::Tensor y = at::empty_like(*p.x[0]);
    void *q = p.x[0]->data_ptr(), *k = p.x[1]->data_ptr(), *v = p.x[2]->data_ptr(), *out = y.data_ptr();
    const float* hp = static_cast<const float*>(h->data_ptr());
    if (!launched([&] { return fn(q, k, v, hp, out, p.B, p.L, p.D, lh, (int32_t)p.group, p.code, p.stream); })) Py_RETURN_NONE;
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// (0: hyena_se_bwd, 1: hyena_mr_bwd; dy, q, k, v, h, group)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Problem p;
    const at::Tensor* h;
    if (n != 7 || !activations(a + 1, 4, a[6], p)) Py_RETURN_NONE;
    const int32_t lh = filter(a[5], p, p.group, h), group = (int32_t)p.group;
    if (!lh) Py_RETURN_NONE;
    const GatedBwd fn = e.bwd[PyLong_AsLong(a[0]) != 0];
    const int64_t need = e.bwd_workspace(p.B, p.L, p.D, lh, group, p.code);
    if (need < 0) Py_RETURN_NONE;
    const at::Tensor ws = workspace(p, need);
    const at::Tensor &dy = *p.x[0], dq = at::empty_like(dy), dk = at::empty_like(dy), dv = at::empty_like(dy), dh = at::empty_like(*h);
    void *yp = dy.data_ptr(), *q = p.x[1]->data_ptr(), *k = p.x[2]->data_ptr(), *v = p.x[3]->data_ptr(), *hp = h->data_ptr();
    void *o0 = dq.data_ptr(), *o1 = dk.data_ptr(), *o2 = dv.data_ptr(), *o3 = dh.data_ptr(), *wp = address(ws);
    if (!launched([&] {
            return fn(yp, q, k, v, static_cast<float*>(hp), o0, o1, o2, static_cast<float*>(o3), wp, need, p.B, p.L, p.D, lh, group,
                      p.code, p.stream);
        }))
        Py_RETURN_NONE;
    return tuple_of({dq, dk, dv, dh});
    END_HANDLE_TH_ERRORS
}

struct Chain {
    Problem p;
    const at::Tensor *f[3], *h;
    int32_t lf, lh, group, feat_group;
};
// n activations, hq, hk, hv, h, group, feat_group
bool chain(PyObject* const* a, int n, Chain& c) {
    if (!PyLong_CheckExact(a[n + 5]) || !activations(a, n, a[n + 4], c.p)) return false;
    int overflow = 0;
    const int64_t fg = PyLong_AsLongLongAndOverflow(a[n + 5], &overflow);
    if (overflow || fg < 1 || fg > 0x7fffffff) return false;
    c.feat_group = (int32_t)fg;
    c.group = (int32_t)c.p.group;
    c.lf = filter(a[n], c.p, fg, c.f[0]);
    if (!c.lf || filter(a[n + 1], c.p, fg, c.f[1]) != c.lf || filter(a[n + 2], c.p, fg, c.f[2]) != c.lf) return false;
    c.lh = filter(a[n + 3], c.p, c.group, c.h);
    return c.lh > 0;
}

// (q, k, v, hq, hk, hv, h, group, feat_group)
PyObject* chain_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Chain c;
    if (n != 9 || !chain(a, 3, c)) Py_RETURN_NONE;
    const Problem& p = c.p;
    const int64_t need = e.chain_workspace(p.B, p.L, p.D, c.lf, c.feat_group, c.lh, c.group, p.code);
    if (need < 0) Py_RETURN_NONE;
    const at::Tensor y = at::empty_like(*p.x[0]), ws = workspace(p, need);
    void* in[8];
    for (int i = 0; i < 3; ++i) {
        in[i] = p.x[i]->data_ptr();
        in[3 + i] = c.f[i]->data_ptr();
    }
    in[6] = c.h->data_ptr();
    in[7] = y.data_ptr();
    void* wp = address(ws);
    auto f = [&](int i) { return static_cast<const float*>(in[i]); };
    if (!launched([&] {
            return e.chain_fwd(in[0], in[1], in[2], f(3), f(4), f(5), f(6), in[7], wp, need, p.B, p.L, p.D, c.lf, c.feat_group,
                               c.lh, c.group, p.code, p.stream);
        }))
        Py_RETURN_NONE;
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// (dy, q, k, v, hq, hk, hv, h, group, feat_group)
PyObject* chain_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Chain c;
    if (n != 10 || !chain(a, 4, c)) Py_RETURN_NONE;
    const Problem& p = c.p;
    const int64_t need = e.chain_bwd_workspace(p.B, p.L, p.D, c.lf, c.feat_group, c.lh, c.group, p.code);
    if (need < 0) Py_RETURN_NONE;
    const at::Tensor ws = workspace(p, need);
    const at::Tensor dq = at::empty_like(*p.x[0]), dk = at::empty_like(*p.x[0]), dv = at::empty_like(*p.x[0]);
    const at::Tensor dhq = at::empty_like(*c.f[0]), dhk = at::empty_like(*c.f[1]), dhv = at::empty_like(*c.f[2]),
                     dh = at::empty_like(*c.h);
    void *in[8], *out[7] = {dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), dhq.data_ptr(), dhk.data_ptr(), dhv.data_ptr(), dh.data_ptr()};
    for (int i = 0; i < 4; ++i) in[i] = p.x[i]->data_ptr();
    for (int i = 0; i < 3; ++i) in[4 + i] = c.f[i]->data_ptr();
    in[7] = c.h->data_ptr();
    void* wp = address(ws);
    auto f = [&](int i) { return static_cast<const float*>(in[i]); };
    auto g = [&](int i) { return static_cast<float*>(out[i]); };
    if (!launched([&] {
            return e.chain_bwd(in[0], in[1], in[2], in[3], f(4), f(5), f(6), f(7), out[0], out[1], out[2], g(3), g(4), g(5), g(6),
                               wp, need, p.B, p.L, p.D, c.lf, c.feat_group, c.lh, c.group, p.code, p.stream);
        }))
        Py_RETURN_NONE;
    return tuple_of({dq, dk, dv, dhq, dhk, dhv, dh});
    END_HANDLE_TH_ERRORS
}

// (q, k, v, R, lam, group)
PyObject* li(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Problem p;
    const at::Tensor *R, *lam;
    if (n != 6 || !activations(a, 3, a[5], p)) Py_RETURN_NONE;
    const int32_t order = filter(a[3], p, p.group, R), group = (int32_t)p.group;
    if (!order || filter(a[4], p, p.group, lam) != order) Py_RETURN_NONE;
    const int64_t need = e.li_workspace(p.B, p.L, p.D, order, group, p.code);
    if (need < 0) Py_RETURN_NONE;
    const at::Tensor y = at::empty_like(*p.x[0]), ws = workspace(p, need);
    void *q = p.x[0]->data_ptr(), *k = p.x[1]->data_ptr(), *v = p.x[2]->data_ptr(), *rp = R->data_ptr(), *lp = lam->data_ptr(),
         *out = y.data_ptr(), *wp = address(ws);
    if (!launched([&] {
            return e.li_fwd(q, k, v, static_cast<float*>(rp), static_cast<float*>(lp), out, wp, need, p.B, p.L, p.D, order, group,
                            p.code, p.stream);
        }))
        Py_RETURN_NONE;
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// (addresses in the order of Entries, callable: device index -> raw stream)
PyObject* init(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != 2 || !PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != kEntries || !PyCallable_Check(a[1])) {
        PyErr_SetString(PyExc_TypeError, "init(addresses, raw_stream)");
        return nullptr;
    }
    void* p[kEntries];
    for (int i = 0; i < kEntries; ++i) {
        p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(a[0], i));
        if (PyErr_Occurred()) return nullptr;
    }
    memcpy(&e, p, sizeof e);
    Py_INCREF(a[1]);
    Py_XSETREF(raw_stream, a[1]);
    Py_RETURN_NONE;
}

#define FAST(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(gated), FAST(bwd), FAST(chain_fwd), FAST(chain_bwd), FAST(li), FAST(init), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
