// Host path of the per-call entry points: a CPython module that takes the binding's arguments as they are (the configuration, tensors,
// numbers), checks them and calls the C ABI on the current stream.  Through ctypes the same work is 12 to 20 interpreted attribute reads and the
// conversion of every argument: 2.7 us of a call beside the 2.6 us of its launch, more than the kernels of a small call take.
//
// A function returns the library's status when it has made the call, and -1, with nothing done, for every argument that is not of the
// ordinary kind (no buffer given, another type, tensor subclasses and wrapped tensors, an active torch-function mode, of which
// torch.set_default_device is one, a failed check); the binding then goes through its own checks and ctypes, which raise what they raise.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "lq.h"

namespace {

constexpr int NOT_HERE = -1;
PyTypeObject* config_type = nullptr;  // binding.lq_config, a ctypes.Structure laid out as lq_config

// An ordinary GPU tensor: exactly torch.Tensor or Parameter, strided, with memory of its own.
const at::Tensor* tensor(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage()) return nullptr;
    if (t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                                 c10::DispatchKey::Functionalize, c10::DispatchKey::Python})))
        return nullptr;
    return &t;
}
bool dense(const at::Tensor* t, c10::ScalarType ty, int64_t rows, int64_t cols)  // contiguous rows x cols
{
    return t && t->scalar_type() == ty && t->dim() == 2 && t->size(0) == rows && t->size(1) == cols && t->is_contiguous();
}
bool row_major(const at::Tensor* t, c10::ScalarType ty, int64_t cols)  // rows may be further apart than cols
{
    return t && t->scalar_type() == ty && t->dim() == 2 && t->stride(1) == 1 && t->size(1) == cols;
}
bool integer(PyObject* o, int64_t* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    *v = PyLong_AsLongLongAndOverflow(o, &over);
    return over == 0;
}
bool number(PyObject* o, float* v)
{
    if (!PyFloat_CheckExact(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}

// The configuration's bytes, held for the duration of a call.
struct Config {
    Py_buffer view{};
    const lq_config* p = nullptr;
    explicit Config(PyObject* o)
    {
        if (!config_type || Py_TYPE(o) != config_type) return;
        if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return;
        }
        if (view.len == (Py_ssize_t)sizeof(lq_config)) p = (const lq_config*)view.buf;
    }
    ~Config()
    {
        if (view.obj) PyBuffer_Release(&view);
    }
    Config(const Config&) = delete;
    Config& operator=(const Config&) = delete;
};

// Runs f (which returns a status, or NOT_HERE before it has called anything) for n arguments; a C++ exception is NOT_HERE as well: only
// the tensors' accessors throw, all of them before the call.
template <typename F>
PyObject* guarded(Py_ssize_t nargs, Py_ssize_t n, F f)
{
    int st = NOT_HERE;
    if (nargs == n && !at::impl::torch_function_mode_enabled()) {
        try {
            st = f();
        } catch (...) {
            st = NOT_HERE;
        }
    }
    return PyLong_FromLong(st);
}
template <typename F>
int on_stream(F call)  // the launch without the interpreter lock, as ctypes makes it
{
    void* s = (void*)c10::hip::getCurrentHIPStream().stream();
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = (int)call(s);
    Py_END_ALLOW_THREADS
    return st;
}

PyObject* set_config_type(PyObject*, PyObject* type)
{
    if (!PyType_Check(type)) {
        PyErr_SetString(PyExc_TypeError, "a type is needed");
        return nullptr;
    }
    Py_INCREF(type);
    Py_XDECREF((PyObject*)config_type);
    config_type = (PyTypeObject*)type;
    Py_RETURN_NONE;
}

PyObject* quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n)  // cfg, packed, X, act
{
    return guarded(n, 4, [&] {
        const Config c(a[0]);
        const at::Tensor *packed = tensor(a[1]), *X = tensor(a[2]), *act = tensor(a[3]);
        if (!c.p || !packed || !act || !row_major(X, c.p->x_dtype == LQ_BF16 ? at::kBFloat16 : at::kFloat, c.p->K) || X->size(0) == 0) return NOT_HERE;
        const void *pp = packed->data_ptr(), *xp = X->data_ptr();
        void* ap = act->data_ptr();
        const int64_t pn = packed->numel(), M = X->size(0), ld = X->stride(0), an = act->numel();
        return on_stream([&](void* s) { return lq_quantize_act(c.p, pp, (size_t)pn, xp, M, ld, ap, (size_t)an, nullptr, s); });
    });
}

PyObject* linear_lowrank_fwd(PyObject*, PyObject* const* a, Py_ssize_t n)  // cfg, packed, act, M, Y
{
    return guarded(n, 5, [&] {
        const Config c(a[0]);
        const at::Tensor *packed = tensor(a[1]), *act = tensor(a[2]), *Y = tensor(a[4]);
        int64_t M;
        if (!c.p || !packed || !act || !integer(a[3], &M) || !row_major(Y, at::kBFloat16, c.p->N) || Y->size(0) != M) return NOT_HERE;
        const void *pp = packed->data_ptr(), *ap = act->data_ptr();
        void* yp = Y->data_ptr();
        const int64_t pn = packed->numel(), an = act->numel(), ld = Y->stride(0);
        return on_stream([&](void* s) { return lq_linear_lowrank_fwd(c.p, pp, (size_t)pn, ap, (size_t)an, M, yp, ld, nullptr, s); });
    });
}

PyObject* linear_lowrank_fwd_handoff(PyObject*, PyObject* const* a, Py_ssize_t n)  // cfg, packed, act, M, next_cfg, act_next, codes, Y or None
{
    return guarded(n, 8, [&] {
        const Config c(a[0]), cn(a[4]);
        const at::Tensor *packed = tensor(a[1]), *act = tensor(a[2]), *next = tensor(a[5]), *codes = tensor(a[6]);
        const at::Tensor* Y = a[7] == Py_None ? nullptr : tensor(a[7]);
        int64_t M;
        if (!c.p || !cn.p || !packed || !act || !next || !codes || !integer(a[3], &M)) return NOT_HERE;
        if (a[7] != Py_None && (!row_major(Y, at::kBFloat16, c.p->N) || Y->size(0) != M)) return NOT_HERE;
        const void *pp = packed->data_ptr(), *ap = act->data_ptr();
        void *np = next->data_ptr(), *cp = codes->data_ptr(), *yp = Y ? Y->data_ptr() : nullptr;
        const int64_t pn = packed->numel(), an = act->numel(), nn = next->numel(), kn = codes->numel(), ld = Y ? Y->stride(0) : 0;
        return on_stream([&](void* s) {
            return lq_linear_lowrank_fwd_handoff(c.p, pp, (size_t)pn, ap, (size_t)an, M, yp, ld, cn.p, np, (size_t)nn, cp, (size_t)kn, s);
        });
    });
}

PyObject* branch_from_codes(PyObject*, PyObject* const* a, Py_ssize_t n)  // next_cfg, packed_next, codes, M, act_next
{
    return guarded(n, 5, [&] {
        const Config c(a[0]);
        const at::Tensor *packed = tensor(a[1]), *codes = tensor(a[2]), *act = tensor(a[4]);
        int64_t M;
        if (!c.p || !packed || !codes || !act || !integer(a[3], &M)) return NOT_HERE;
        const void *pp = packed->data_ptr(), *cp = codes->data_ptr();
        void* ap = act->data_ptr();
        const int64_t pn = packed->numel(), kn = codes->numel(), an = act->numel();
        return on_stream([&](void* s) { return lq_branch_from_codes(c.p, pp, (size_t)pn, cp, (size_t)kn, M, ap, (size_t)an, s); });
    });
}

PyObject* pack_weights(PyObject*, PyObject* const* a, Py_ssize_t n)  // cfg, W, L, R, packed
{
    return guarded(n, 5, [&] {
        const Config c(a[0]);
        const at::Tensor *W = tensor(a[1]), *L = tensor(a[2]), *R = tensor(a[3]), *packed = tensor(a[4]);
        if (!c.p || !packed || !dense(W, at::kFloat, c.p->N, c.p->K) || !dense(L, at::kFloat, c.p->N, c.p->rank) || !dense(R, at::kFloat, c.p->rank, c.p->K))
            return NOT_HERE;
        const float *wp = (const float*)W->data_ptr(), *lp = (const float*)L->data_ptr(), *rp = (const float*)R->data_ptr();
        void* pp = packed->data_ptr();
        const int64_t pn = packed->numel();
        return on_stream([&](void* s) { return lq_pack_weights(c.p, wp, lp, rp, pp, (size_t)pn, s); });
    });
}

bool loss_arg(PyObject* o, void** p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    const at::Tensor* t = tensor(o);
    if (!t) return false;
    *p = t->data_ptr();
    return true;
}

PyObject* calib_step(PyObject*, PyObject* const* a, Py_ssize_t n)  // cfg, W, state, step, lr, beta1, beta2, eps, loss or None
{
    return guarded(n, 9, [&] {
        const Config c(a[0]);
        const at::Tensor *W = tensor(a[1]), *state = tensor(a[2]);
        int64_t step;
        lq_adam ad;
        void* loss;
        if (!c.p || !state || !dense(W, at::kFloat, c.p->N, c.p->K) || !integer(a[3], &step) || step < INT32_MIN || step > INT32_MAX) return NOT_HERE;
        if (!number(a[4], &ad.lr) || !number(a[5], &ad.beta1) || !number(a[6], &ad.beta2) || !number(a[7], &ad.eps) || !loss_arg(a[8], &loss)) return NOT_HERE;
        const float* wp = (const float*)W->data_ptr();
        void* sp = state->data_ptr();
        const int64_t sn = state->numel();
        return on_stream([&](void* s) { return lq_calib_step(c.p, wp, sp, (size_t)sn, (int32_t)step, &ad, (float*)loss, s); });
    });
}

PyObject* rot_step(PyObject*, PyObject* const* a, Py_ssize_t n)  // cfg, L, R, state, lr, beta, eps, q, s, grad_scale, loss or None
{
    return guarded(n, 11, [&] {
        const Config c(a[0]);
        const at::Tensor *L = tensor(a[1]), *R = tensor(a[2]), *state = tensor(a[3]);
        int64_t passes;
        lq_cayley cs;
        void* loss;
        if (!c.p || !state || !dense(L, at::kFloat, c.p->N, c.p->rank) || !dense(R, at::kFloat, c.p->rank, c.p->K)) return NOT_HERE;
        if (!number(a[4], &cs.lr) || !number(a[5], &cs.beta) || !number(a[6], &cs.eps) || !number(a[7], &cs.q) || !integer(a[8], &passes) ||
            passes < INT32_MIN || passes > INT32_MAX || !number(a[9], &cs.grad_scale) || !loss_arg(a[10], &loss))
            return NOT_HERE;
        cs.s = (int32_t)passes;
        const float *lp = (const float*)L->data_ptr(), *rp = (const float*)R->data_ptr();
        void* sp = state->data_ptr();
        const int64_t sn = state->numel();
        return on_stream([&](void* s) { return lq_rot_step(c.p, lp, rp, sp, (size_t)sn, &cs, (float*)loss, s); });
    });
}

#define FAST(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"set_config_type", set_config_type, METH_O, nullptr},
                         FAST(quantize_act),
                         FAST(linear_lowrank_fwd),
                         FAST(linear_lowrank_fwd_handoff),
                         FAST(branch_from_codes),
                         FAST(pack_weights),
                         FAST(calib_step),
                         FAST(rot_step),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call() { return PyModule_Create(&module); }
