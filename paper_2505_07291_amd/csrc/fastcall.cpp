// The binding's ordinary calls without the interpreter: tensors checked, outputs allocated and libgrpo called from
// here.  What bounds a call on a few thousand values is the host: of 35 us for the shaping of a rollout step
// (four calls, four launches, 13 us on the GPU) two thirds were attribute lookups, nine torch.empty and ctypes
// conversions in Python.
//
// A function returns None when a call is not an ordinary one - another tensor class, dtype, device or layout, a
// number that is not a plain int or float, a mode or transform that wants to see the allocations - and binding.py then
// takes its general path, which checks everything and raises what there is to raise (it does not ask at all where a
// stream, or an output other than the gradient, is given); an int is a grpo_status other than GRPO_OK.  Nothing is kept
// between calls but the library's addresses.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "grpo.h"

namespace {

decltype(&grpo_workspace_bytes) f_workspace_bytes;
decltype(&grpo_group_advantages) f_group_advantages;
decltype(&grpo_logprobs_fwd) f_logprobs_fwd;
decltype(&grpo_loss_fwd_bwd) f_loss_fwd_bwd;
decltype(&grpo_loss_aux_fwd_bwd) f_loss_aux_fwd_bwd;
decltype(&grpo_total_rewards) f_total_rewards;
decltype(&grpo_filter_groups) f_filter_groups;
decltype(&grpo_packed_layout) f_packed_layout;
bool bound = false;

// Are all functionalities of `keys` among the usual ones?  (Which backends the keys name is not looked at.)
bool only(c10::DispatchKeySet keys, c10::DispatchKeySet usual)
{
    return (keys.raw_repr() & ~usual.raw_repr()) >> c10::num_backends == 0;
}

// Nothing but plain eager execution: no Python function or dispatch mode, no transform, tracing or functionalisation.
bool plain_mode()
{
    using c10::DispatchKey;
    if (!bound || at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) return false;
    return only(c10::impl::tls_local_dispatch_key_set().included_,
                c10::autocast_dispatch_keyset | c10::DispatchKeySet({DispatchKey::BackendSelect, DispatchKey::ADInplaceOrView}));
}

// A torch.Tensor or Parameter over ordinary device memory, or nullptr.
const at::Tensor *plain(PyObject *o)
{
    using c10::DispatchKey;
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    const auto usual = c10::autocast_dispatch_keyset |
                       c10::DispatchKeySet({DispatchKey::CUDA, DispatchKey::AutogradCUDA, DispatchKey::ADInplaceOrView});
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !only(t.key_set(), usual)) return nullptr;
    return &t;
}
// the same, one-dimensional and contiguous, of this type, length (-1: any) and device
const at::Tensor *row(PyObject *o, at::ScalarType type, int64_t n, const c10::Device *dev)
{
    const at::Tensor *t = plain(o);
    if (!t || t->scalar_type() != type || t->dim() != 1 || (n >= 0 && t->size(0) != n) || !t->is_contiguous() ||
        (dev && t->device() != *dev))
        return nullptr;
    return t;
}
// an optional one: false if it is neither None nor such a tensor
bool row_or_none(PyObject *o, at::ScalarType type, int64_t n, const c10::Device *dev, const at::Tensor **out)
{
    *out = o == Py_None ? nullptr : row(o, type, n, dev);
    return o == Py_None || *out;
}
bool number(PyObject *o, double *out)
{
    if (PyFloat_CheckExact(o)) {
        *out = PyFloat_AS_DOUBLE(o);
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    *out = PyLong_AsDouble(o);
    if (*out == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}
bool whole(PyObject *o, int64_t *out)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *out = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0;
}

at::Tensor make(int64_t n, at::ScalarType type, const c10::Device &dev)
{
    return at::empty({n}, at::TensorOptions().dtype(type).device(dev));
}
void *ptr(const at::Tensor *t) { return t ? t->data_ptr() : nullptr; }
void *ptr(const at::Tensor &t) { return t.data_ptr(); }
template <typename T>
T *as(const at::Tensor *t)
{
    return (T *)ptr(t);
}
template <typename T>
T *as(const at::Tensor &t)
{
    return (T *)ptr(t);
}
void *current_stream() { return (void *)c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream(); }

// The call itself without the interpreter's lock, as ctypes makes it.  Its arguments are values by then: what may
// throw (data_ptr() of a tensor whose memory is gone) is evaluated with the lock held, and the lock is taken again
// however the block is left.
struct Unlocked {
    PyThreadState *state = PyEval_SaveThread();
    ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename... T>
grpo_status call(grpo_status (*f)(T...), std::common_type_t<T>... args)
{
    Unlocked no_lock;
    return f(args...);
}
// (None for a tensor that is not defined.)  last: an object of the caller's, or None, and then made_last's.
PyObject *tuple_of(std::initializer_list<at::Tensor> made, PyObject *last = nullptr, const at::Tensor &made_last = {})
{
    PyObject *out = PyTuple_New((Py_ssize_t)made.size() + (last ? 1 : 0));
    if (!out) return nullptr;
    Py_ssize_t i = 0;
    for (const at::Tensor &t : made) {
        PyObject *o = THPVariable_Wrap(t);
        if (!o) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i++, o);
    }
    if (last) {
        if (last == Py_None)
            last = THPVariable_Wrap(made_last);
        else
            Py_INCREF(last);
        if (!last) {
            Py_DECREF(out);
            return nullptr;
        }
        PyTuple_SET_ITEM(out, i, last);
    }
    return out;
}

struct Logits {
    const at::Tensor *t;
    c10::Device dev = c10::Device(c10::kCPU);
    grpo_dtype dtype;
    int64_t n, v, stride;
};
bool logits_of(PyObject *o, Logits *l)
{
    l->t = plain(o);
    if (!l->t || l->t->dim() != 2 || l->t->stride(1) != 1) return false;
    if (l->t->scalar_type() == at::kBFloat16)
        l->dtype = GRPO_BF16;
    else if (l->t->scalar_type() == at::kFloat)
        l->dtype = GRPO_F32;
    else
        return false;
    l->dev = l->t->device();
    l->n = l->t->size(0);
    l->v = l->t->size(1);
    l->stride = l->n > 1 ? l->t->stride(0) : std::max<int64_t>(l->t->stride(0), l->v);
    return true;
}
// Where the gradient goes: the caller's tensor, of the logits' type, shape and strides (it may be the logits), or, for
// None, a new one of that kind, made by grad_made when the other arguments have been looked at.
bool grad_ok(PyObject *o, const Logits &l)
{
    if (o == Py_None) return true;
    const at::Tensor *g = plain(o);
    return g && g->scalar_type() == l.t->scalar_type() && g->device() == l.dev && g->sizes() == l.t->sizes() &&
           g->strides() == l.t->strides();
}
at::Tensor grad_made(PyObject *o, const Logits &l)
{
    if (o != Py_None) return THPVariable_Unpack(o);
    return at::empty_strided(l.t->sizes(), l.t->strides(), at::TensorOptions().dtype(l.t->scalar_type()).device(l.dev));
}

#define ORDINARY(cond) \
    if (!(cond)) Py_RETURN_NONE

// total_rewards(task_rewards, lengths, target_lengths, alpha)
PyObject *total_rewards(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    double alpha;
    ORDINARY(n_args == 4 && plain_mode() && number(a[3], &alpha));
    const at::Tensor *task = row(a[0], at::kFloat, -1, nullptr);
    ORDINARY(task);
    const c10::Device dev = task->device();
    const int64_t n = task->size(0);
    const at::Tensor *len = row(a[1], at::kInt, n, &dev), *target = row(a[2], at::kInt, n, &dev);
    ORDINARY(len && target);
    at::Tensor out = make(n, at::kFloat, dev);
    void *st = current_stream();
    const grpo_status rc = call(f_total_rewards, as<const float>(task), as<const int32_t>(len), as<const int32_t>(target),
                                n, (float)alpha, as<float>(out), st);
    return rc == GRPO_OK ? THPVariable_Wrap(out) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// filter_groups(rewards, group_size)
PyObject *filter_groups(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    int64_t size;
    ORDINARY(n_args == 2 && plain_mode() && whole(a[1], &size) && size > 0);
    const at::Tensor *rewards = row(a[0], at::kFloat, -1, nullptr);
    ORDINARY(rewards);
    const c10::Device dev = rewards->device();
    const int64_t n = rewards->size(0), groups = n / size;
    ORDINARY(groups > 0);
    at::Tensor keep = make(groups, at::kByte, dev), kept = make(groups, at::kInt, dev), n_kept = make(1, at::kInt, dev),
               rollouts = make(n, at::kByte, dev);
    void *st = current_stream();
    const grpo_status rc = call(f_filter_groups, as<const float>(rewards), n, nullptr, groups, size, as<uint8_t>(keep),
                                as<int32_t>(kept), as<int32_t>(n_kept), as<uint8_t>(rollouts), st);
    return rc == GRPO_OK ? tuple_of({keep, kept, n_kept, rollouts}) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// packed_layout(cu_seqlens, n_tokens, sample_level)
PyObject *packed_layout(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    int64_t n;
    ORDINARY(n_args == 3 && plain_mode() && whole(a[1], &n) && n >= 0 && PyBool_Check(a[2]));
    const at::Tensor *cu = row(a[0], at::kLong, -1, nullptr);
    ORDINARY(cu);
    const c10::Device dev = cu->device();
    at::Tensor weights = make(n, at::kFloat, dev), rollout = make(n, at::kInt, dev);
    void *st = current_stream();
    const grpo_status rc = call(f_packed_layout, as<const int64_t>(cu), cu->size(0) - 1, n, a[2] == Py_True ? 1 : 0,
                                as<float>(weights), as<int32_t>(rollout), st);
    return rc == GRPO_OK ? tuple_of({weights, rollout}) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// group_advantages(rewards, group_size, eps_std, ddof, rollout_of_token or None)
PyObject *group_advantages(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    int64_t size, ddof;
    double eps;
    ORDINARY(n_args == 5 && plain_mode() && whole(a[1], &size) && size > 0 && number(a[2], &eps) && whole(a[3], &ddof) &&
             ddof >= 0 && ddof <= 1);
    const at::Tensor *rewards = row(a[0], at::kFloat, -1, nullptr), *rollout;
    ORDINARY(rewards);
    const c10::Device dev = rewards->device();
    ORDINARY(row_or_none(a[4], at::kInt, -1, &dev, &rollout));
    const int64_t n = rewards->size(0), tokens = rollout ? rollout->size(0) : 0;
    at::Tensor adv = make(n, at::kFloat, dev), adv_tok;
    if (rollout) adv_tok = make(tokens, at::kFloat, dev);
    void *st = current_stream();
    const grpo_status rc = call(f_group_advantages, as<const float>(rewards), n, nullptr, n / size, size, (float)eps,
                                (int)ddof, as<float>(adv), as<const int32_t>(rollout), tokens, rollout ?
                                as<float>(adv_tok) : nullptr, st);
    return rc == GRPO_OK ? tuple_of({adv, adv_tok}) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// logprobs_fwd(logits, tokens, mask or None, temperature, workspace)
PyObject *logprobs_fwd(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    double temperature;
    Logits l;
    ORDINARY(n_args == 5 && plain_mode() && number(a[3], &temperature) && logits_of(a[0], &l));
    const at::Tensor *tokens = row(a[1], at::kLong, l.n, &l.dev), *mask, *ws = row(a[4], at::kByte, -1, &l.dev);
    ORDINARY(tokens && ws && row_or_none(a[2], at::kByte, l.n, &l.dev, &mask));
    at::Tensor lp = make(l.n, at::kFloat, l.dev);
    void *st = current_stream();
    const grpo_status rc = call(f_logprobs_fwd, ptr(l.t), l.dtype, l.n, l.v, l.stride, as<const int64_t>(tokens),
                                as<const uint8_t>(mask), (float)temperature, as<float>(lp), ptr(ws), (size_t)ws->numel(), st);
    return rc == GRPO_OK ? THPVariable_Wrap(lp) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// loss_fwd_bwd(logits, tokens, old_logprobs, advantages, mask or None, eps_low, eps_high, delta, temperature, denom,
//              grad_scale, grad_logits or None, workspace or None)
PyObject *loss_fwd_bwd(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    Logits l;
    double f[6];
    ORDINARY(n_args == 13 && plain_mode() && logits_of(a[0], &l));
    for (int i = 0; i < 6; ++i) ORDINARY(number(a[5 + i], &f[i]));
    const at::Tensor *tokens = row(a[1], at::kLong, l.n, &l.dev), *old = row(a[2], at::kFloat, l.n, &l.dev),
                     *adv = row(a[3], at::kFloat, l.n, &l.dev), *mask, *given;
    ORDINARY(tokens && old && adv && grad_ok(a[11], l) && row_or_none(a[4], at::kByte, l.n, &l.dev, &mask) &&
             row_or_none(a[12], at::kByte, -1, &l.dev, &given));
    at::Tensor loss = make(1, at::kFloat, l.dev), lp = make(l.n, at::kFloat, l.dev), counts = make(5, at::kLong, l.dev);
    const at::Tensor grad = grad_made(a[11], l), ws = given ? *given : make((int64_t)f_workspace_bytes(l.n), at::kByte, l.dev);
    void *st = current_stream();
    const grpo_status rc = call(f_loss_fwd_bwd, ptr(l.t), l.dtype, l.n, l.v, l.stride, as<const int64_t>(tokens),
                                as<const float>(old), as<const float>(adv), as<const uint8_t>(mask), (float)f[0], (float)f[1],
                                (float)f[2], (float)f[3], f[4], (float)f[5], as<float>(loss), as<float>(lp),
                                as<int64_t>(counts), ptr(grad), ptr(ws), (size_t)ws.numel(), st);
    return rc == GRPO_OK ? tuple_of({loss, lp, counts}, a[11], grad) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// loss_aux_fwd_bwd(logits, tokens, old_logprobs, ref_logprobs or None, advantages, mask or None, token_weights or None,
//                  eps_low, eps_high, delta, temperature, kl_coef, entropy_coef, denom, grad_scale,
//                  grad_logits or None, workspace or None, want_entropy)
PyObject *loss_aux_fwd_bwd(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    Logits l;
    double f[8];
    ORDINARY(n_args == 18 && plain_mode() && PyBool_Check(a[17]) && logits_of(a[0], &l));
    for (int i = 0; i < 8; ++i) ORDINARY(number(a[7 + i], &f[i]));
    const at::Tensor *tokens = row(a[1], at::kLong, l.n, &l.dev), *old = row(a[2], at::kFloat, l.n, &l.dev),
                     *adv = row(a[4], at::kFloat, l.n, &l.dev), *ref, *mask, *weights, *given;
    ORDINARY(tokens && old && adv && grad_ok(a[15], l) && row_or_none(a[3], at::kFloat, l.n, &l.dev, &ref) &&
             row_or_none(a[5], at::kByte, l.n, &l.dev, &mask) && row_or_none(a[6], at::kFloat, l.n, &l.dev, &weights) &&
             row_or_none(a[16], at::kByte, -1, &l.dev, &given));
    at::Tensor loss = make(4, at::kFloat, l.dev), lp = make(l.n, at::kFloat, l.dev), counts = make(5, at::kLong, l.dev), entropy;
    if (a[17] == Py_True) entropy = make(l.n, at::kFloat, l.dev);
    const at::Tensor grad = grad_made(a[15], l), ws = given ? *given : make((int64_t)f_workspace_bytes(l.n), at::kByte, l.dev);
    void *st = current_stream();
    const grpo_status rc = call(f_loss_aux_fwd_bwd, ptr(l.t), l.dtype, l.n, l.v, l.stride, as<const int64_t>(tokens),
                                as<const float>(old), as<const float>(ref), as<const float>(adv), as<const uint8_t>(mask),
                                as<const float>(weights), (float)f[0], (float)f[1], (float)f[2], (float)f[3], (float)f[4],
                                (float)f[5], f[6], (float)f[7], as<float>(loss), as<float>(lp), entropy.defined() ?
                                as<float>(entropy) : nullptr, as<int64_t>(counts), ptr(grad), ptr(ws), (size_t)ws.numel(),
                                st);
    return rc == GRPO_OK ? tuple_of({loss, lp, entropy, counts}, a[15], grad) : PyLong_FromLong(rc);
    END_HANDLE_TH_ERRORS
}

// bind(addresses in the order below): the library that calls go to from now on
PyObject *bind(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    void *at[8];
    if (n_args != 8) {
        PyErr_SetString(PyExc_TypeError, "bind takes eight addresses");
        return nullptr;
    }
    for (int i = 0; i < 8; ++i) {
        at[i] = PyLong_AsVoidPtr(a[i]);
        if (!at[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function's address is not null");
            return nullptr;
        }
    }
    f_workspace_bytes = (decltype(f_workspace_bytes))at[0];
    f_group_advantages = (decltype(f_group_advantages))at[1];
    f_logprobs_fwd = (decltype(f_logprobs_fwd))at[2];
    f_loss_fwd_bwd = (decltype(f_loss_fwd_bwd))at[3];
    f_loss_aux_fwd_bwd = (decltype(f_loss_aux_fwd_bwd))at[4];
    f_total_rewards = (decltype(f_total_rewards))at[5];
    f_filter_groups = (decltype(f_filter_groups))at[6];
    f_packed_layout = (decltype(f_packed_layout))at[7];
    bound = true;
    Py_RETURN_NONE;
}

#define METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {METHOD(bind),           METHOD(total_rewards), METHOD(filter_groups), METHOD(packed_layout),
                         METHOD(group_advantages), METHOD(logprobs_fwd),  METHOD(loss_fwd_bwd),  METHOD(loss_aux_fwd_bwd),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&module); }
