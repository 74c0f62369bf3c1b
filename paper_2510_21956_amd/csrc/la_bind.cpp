// Argument marshalling of the small, frequent calls (binding.py) in native code: the checks, addresses
// and conversions that the Python functions of the same names make, one tensor at a time, took most
// of a decode step's 7 us.  Takes plain tensors only, without a trace; everything else stays with the Python
// functions, which are also what a build without this file runs.
//
// Refuses nothing itself: what does not pass the checks (a tensor without storage or a functorch wrapper, whose
// C++ exception ends up here, included) goes back to the Python functions, which refuse or take it.  The library
// is called without the interpreter lock, as ctypes does.
#include <ATen/FuncTorchTLS.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_cpp_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include "la.h"

namespace {

PyObject *raw_stream = nullptr;       // device index -> stream handle of its current stream
PyObject *python_backward = nullptr;  // the wrapper's backward pass in Python

// Entry points of libla.so, as addresses (binding.py has loaded the library).
decltype(&la_forward_traced) fwd_plain, fwd_qknorm;
decltype(&la_forward_save) fwd_save, fwd_qknorm_save;
decltype(&la_backward_traced) bwd_plain, bwd_qknorm;
decltype(&la_backward_saved) bwd_saved, bwd_qknorm_saved;
decltype(&la_decode_step) dec_step;
decltype(&la_decode_prefill) dec_prefill;
decltype(&la_workspace_bytes) workspace_bytes;
decltype(&la_saved_state_bytes) saved_state_bytes;

struct Decline {};  // the Python function takes over; a Python exception may be set
void require(bool ok)
{
    if (!ok) throw Decline();
}

bool is_none(PyObject *o) { return o == Py_None; }
// Tensors and parameters; a subclass may answer is_contiguous, data_ptr and the rest in its own way, which
// the Python functions ask it for.
bool plain(PyObject *o) { return THPVariable_CheckExact(o); }
bool plain_or_none(PyObject *o) { return is_none(o) || plain(o); }
const at::Tensor &tensor(PyObject *o) { return THPVariable_Unpack(o); }
void *address(PyObject *o) { return is_none(o) ? nullptr : tensor(o).data_ptr(); }
size_t bytes(const at::Tensor &t) { return (size_t)t.numel() * t.element_size(); }

// Packed device tensors, all on one device (None is left out).
void check_packed(std::initializer_list<PyObject *> ts)
{
    const at::Tensor &ref = tensor(*ts.begin());
    for (PyObject *o : ts) {
        if (is_none(o)) continue;
        const at::Tensor &t = tensor(o);
        require(t.is_cuda() && t.is_contiguous() && t.get_device() == ref.get_device());
    }
}
void check_like(const at::Tensor &ref, std::initializer_list<PyObject *> ts)
{
    for (PyObject *o : ts)
        require(is_none(o) || (tensor(o).sizes() == ref.sizes() && tensor(o).scalar_type() == ref.scalar_type()));
}
void check_rows(const at::Tensor &ref, PyObject *g)
{
    if (is_none(g)) return;
    const at::Tensor &t = tensor(g);
    require(t.sizes() == ref.sizes().slice(0, 3) && t.scalar_type() == at::kFloat);
}
la_dtype dtype_code(const at::Tensor &t)
{
    require(t.scalar_type() == at::kFloat || t.scalar_type() == at::kBFloat16);
    return t.scalar_type() == at::kFloat ? LA_F32 : LA_BF16;
}
double real(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return PyFloat_AS_DOUBLE(o);
    PyObject *f = PyNumber_Float(o);  // what float(o) gives
    require(f);
    const double x = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return x;
}
float number(PyObject *o) { return (float)real(o); }
int truth(PyObject *o)
{
    const int x = PyObject_IsTrue(o);
    require(x >= 0);
    return x;
}
void *stream_of(PyObject *stream, const at::Tensor &ref)
{
    PyObject *h = is_none(stream) ? PyObject_CallFunction(raw_stream, "i", (int)ref.get_device())
                                  : PyObject_GetAttrString(stream, "cuda_stream");
    require(h);
    void *p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    require(p || !PyErr_Occurred());
    return p;
}

// Runs body, which returns the library's status, on n arguments.  None: the Python function takes over.
template <typename Body>
PyObject *guarded(Py_ssize_t given, Py_ssize_t n, Body body)
{
    if (given != n) return PyErr_Format(PyExc_TypeError, "%zd arguments expected", n);
    try {
        return body();
    } catch (const Decline &) {
    } catch (const std::exception &) {
    }
    if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;  // an interrupt
    PyErr_Clear();
    Py_RETURN_NONE;
}
template <typename Call>
PyObject *status(Call call)
{
    la_status s;
    Py_BEGIN_ALLOW_THREADS s = call();
    Py_END_ALLOW_THREADS return PyLong_FromLong(s);
}
bool ours(PyObject *const *a, int first, int last)
{
    if (!plain(a[first])) return false;
    for (int i = first + 1; i <= last; ++i)
        if (!plain_or_none(a[i])) return false;
    return true;
}

// kind (0 plain, 1 save, 2 qknorm, 3 qknorm_save), Q, K, V, O, G, a, b, causal, workspace, saved, stream
PyObject *forward(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    return guarded(n, 12, [&]() -> PyObject * {
        if (!ours(x, 1, 5) || !plain(x[9]) || !plain_or_none(x[10]) || is_none(x[2]) ||
            is_none(x[3]) || is_none(x[4]))
            Py_RETURN_NONE;
        const long kind = PyLong_AsLong(x[0]);
        const at::Tensor &Q = tensor(x[1]), &ws = tensor(x[9]);
        require(Q.dim() == 4);
        check_packed({x[1], x[2], x[3], x[4], x[5], x[9]});
        check_like(Q, {x[2], x[3], x[4]});
        check_rows(Q, x[5]);
        const float a = number(x[6]), b = number(x[7]);
        const int causal = truth(x[8]), B = Q.size(0), H = Q.size(1), N = Q.size(2), D = Q.size(3);
        const la_dtype dt = dtype_code(Q);
        void *sv = nullptr;
        size_t sb = 0;
        if (kind % 2 && !is_none(x[10])) {
            check_packed({x[1], x[10]});
            sv = address(x[10]);
            sb = bytes(tensor(x[10]));
        }
        void *st = stream_of(x[11], Q), *q = address(x[1]), *k = address(x[2]), *v = address(x[3]),
             *o = address(x[4]), *w = address(x[9]);
        float *g = (float *)address(x[5]);
        const size_t wb = bytes(ws);
        return status([&] {
            if (kind == 0) return fwd_plain(q, k, v, o, g, B, H, N, D, a, b, causal, dt, w, wb, st, nullptr);
            if (kind == 2) return fwd_qknorm(q, k, v, o, g, B, H, N, D, a, b, causal, dt, w, wb, st, nullptr);
            return (kind == 1 ? fwd_save : fwd_qknorm_save)(q, k, v, o, g, B, H, N, D, a, b, causal, dt, w, wb, sv,
                                                            sb, st, nullptr);
        });
    });
}

// kind, Q, K, V, O, G, dO, dQ, dK, dV, a, b, causal, workspace, saved, stream
PyObject *backward(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    return guarded(n, 16, [&]() -> PyObject * {
        if (!ours(x, 1, 9) || !plain(x[13]) || !plain_or_none(x[14])) Py_RETURN_NONE;
        for (int i : {2, 3, 6, 7, 8, 9})
            if (is_none(x[i])) Py_RETURN_NONE;
        const long kind = PyLong_AsLong(x[0]);
        const at::Tensor &Q = tensor(x[1]), &ws = tensor(x[13]);
        require(Q.dim() == 4);
        check_packed({x[1], x[2], x[3], x[4], x[5], x[6], x[7], x[8], x[9], x[13]});
        check_like(Q, {x[2], x[3], x[4], x[6], x[7], x[8], x[9]});
        check_rows(Q, x[5]);
        const float a = number(x[10]), b = number(x[11]);
        const int causal = truth(x[12]), B = Q.size(0), H = Q.size(1), N = Q.size(2), D = Q.size(3);
        const la_dtype dt = dtype_code(Q);
        void *sv = nullptr;
        size_t sb = 0;
        if (kind % 2 && !is_none(x[14])) {
            check_packed({x[1], x[14]});
            sv = address(x[14]);
            sb = bytes(tensor(x[14]));
        }
        void *st = stream_of(x[15], Q), *p[10], *w = address(x[13]);
        for (int i = 1; i <= 9; ++i) p[i] = address(x[i]);
        const size_t wb = bytes(ws);
        return status([&] {
            if (kind % 2 == 0)
                return (kind == 0 ? bwd_plain : bwd_qknorm)(p[1], p[2], p[3], p[4], (const float *)p[5], p[6], p[7],
                                                            p[8], p[9], B, H, N, D, a, b, causal, dt, w, wb, st,
                                                            nullptr);
            return (kind == 1 ? bwd_saved : bwd_qknorm_saved)(p[1], p[2], p[3], p[4], (const float *)p[5], p[6], p[7],
                                                              p[8], p[9], B, H, N, D, a, b, causal, dt, w, wb, sv, sb,
                                                              st, nullptr);
        });
    });
}

// q, k, v, o, g, state, a, b, stream
PyObject *decode_step(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    return guarded(n, 9, [&]() -> PyObject * {
        if (!ours(x, 0, 5)) Py_RETURN_NONE;
        for (int i : {1, 2, 3, 5})
            if (is_none(x[i])) Py_RETURN_NONE;
        const at::Tensor &q = tensor(x[0]), &state = tensor(x[5]);
        require(q.dim() == 4);
        check_packed({x[0], x[1], x[2], x[3], x[4], x[5]});
        check_like(q, {x[1], x[2], x[3]});
        require(state.scalar_type() == at::kFloat);
        check_rows(q, x[4]);
        const float a = number(x[6]), b = number(x[7]);
        const int B = q.size(0), H = q.size(1), T = q.size(2), D = q.size(3);
        const la_dtype dt = dtype_code(q);
        void *st = stream_of(x[8], q), *p[6];
        for (int i = 0; i < 6; ++i) p[i] = address(x[i]);
        const size_t sb = (size_t)state.numel() * 4;
        return status([&] {
            return dec_step(p[0], p[1], p[2], p[3], (float *)p[4], (float *)p[5], sb, B, H, T, D, a, b, dt, st);
        });
    });
}

// K, V, state, accumulate, workspace, stream
PyObject *decode_prefill(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    return guarded(n, 6, [&]() -> PyObject * {
        for (int i : {0, 1, 2, 4})
            if (!plain(x[i])) Py_RETURN_NONE;
        const at::Tensor &K = tensor(x[0]), &V = tensor(x[1]), &state = tensor(x[2]), &ws = tensor(x[4]);
        require(K.dim() == 4);
        check_packed({x[0], x[1], x[2], x[4]});
        check_like(K, {x[1]});
        require(state.scalar_type() == at::kFloat);
        const int B = K.size(0), H = K.size(1), N = K.size(2), D = K.size(3), add = truth(x[3]);
        const la_dtype dt = dtype_code(K);
        void *st = stream_of(x[5], K), *k = address(x[0]), *v = address(x[1]), *s = address(x[2]), *w = address(x[4]);
        const size_t sb = (size_t)state.numel() * 4, wb = bytes(ws);
        return status([&] { return dec_prefill(k, v, (float *)s, sb, B, H, N, D, dt, add, w, wb, st); });
    });
}

// ---- the autograd wrapper ------------------------------------------------------------------------------------
// linear_attention on plain tensors as an autograd node in native code: LinearAttentionFunction (autograd.py) step by
// step, without the interpreter, whose lock the engine's thread otherwise waits for in the backward pass.  Forward
// and backward pass of a toy layer (1 slice of 256 rows, D = 16): 117 -> 83 us, nearly all of it host.

at::Tensor buffer(size_t n, const at::Tensor &ref)
{
    return at::empty({(int64_t)(n < 256 ? 256 : n)}, ref.options().dtype(at::kByte));
}
void *current_stream(const at::Tensor &ref) { return c10::hip::getCurrentHIPStream(ref.get_device()).stream(); }

struct Status {  // what the library answered
    int rc;
};
struct Attention : torch::autograd::Function<Attention> {
    static at::Tensor forward(torch::autograd::AutogradContext *ctx, const at::Tensor &Q0, const at::Tensor &K0,
                              const at::Tensor &V0, double a, double b, bool causal, bool norm)
    {
        const at::Tensor Q = Q0.contiguous(), K = K0.contiguous(), V = V0.contiguous();
        const int B = Q.size(0), H = Q.size(1), N = Q.size(2), D = Q.size(3);
        const la_dtype dt = dtype_code(Q);
        const at::Tensor O = at::empty_like(Q), G = at::empty({B, H, N}, Q.options().dtype(at::kFloat));
        const at::Tensor ws = buffer(workspace_bytes(B, H, N, D, dt, causal, 0), Q);
        const size_t ns = saved_state_bytes(B, H, N, D, dt, causal);
        at::Tensor saved;
        if (ns) saved = buffer(ns, Q);
        // everything that can throw, while the interpreter lock is held
        void *const q = Q.data_ptr(), *const k = K.data_ptr(), *const v = V.data_ptr(), *const o = O.data_ptr(),
                   *const w = ws.data_ptr(), *const sv = ns ? saved.data_ptr() : nullptr, *const st = current_stream(Q);
        float *const g = (float *)G.data_ptr();
        const size_t wb = bytes(ws), sb = ns ? bytes(saved) : 0;
        int rc;
        Py_BEGIN_ALLOW_THREADS rc = (norm ? fwd_qknorm_save : fwd_save)(
            q, k, v, o, g, B, H, N, D, (float)a, (float)b, causal, dt, w, wb, sv, sb, st, nullptr);
        Py_END_ALLOW_THREADS
        if (rc != 0) throw Status{rc};
        ctx->save_for_backward({Q, K, V, O, G});
        ctx->saved_data["a"] = a;
        ctx->saved_data["b"] = b;
        ctx->saved_data["causal"] = causal;
        ctx->saved_data["norm"] = norm;
        if (ns) ctx->saved_data["sums"] = saved;
        return O;
    }
    static torch::autograd::variable_list backward(torch::autograd::AutogradContext *ctx,
                                                   torch::autograd::variable_list grads)
    {
        const auto s = ctx->get_saved_variables();
        const at::Tensor &Q = s[0], dO = grads[0].contiguous();
        const double a = ctx->saved_data["a"].toDouble(), b = ctx->saved_data["b"].toDouble();
        const bool causal = ctx->saved_data["causal"].toBool(), norm = ctx->saved_data["norm"].toBool();
        const auto it = ctx->saved_data.find("sums");
        const at::Tensor sums = it == ctx->saved_data.end() ? at::Tensor() : it->second.toTensor();
        torch::autograd::variable_list out(7);
        const bool ordinary = [&] {
            for (const at::Tensor *t : {&s[0], &s[1], &s[2], &s[3], &s[4], &dO})
                if (!t->is_cuda() || !t->is_contiguous() || t->unsafeGetTensorImpl()->is_python_dispatch() ||
                    t->get_device() != Q.get_device() || (t != &s[4] && t->sizes() != Q.sizes()) ||
                    t->scalar_type() != (t == &s[4] ? at::kFloat : Q.scalar_type()))
                    return false;
            return true;
        }();
        if (ordinary) {
            const int B = Q.size(0), H = Q.size(1), N = Q.size(2), D = Q.size(3);
            const la_dtype dt = dtype_code(Q);
            for (int i = 0; i < 3; ++i) out[i] = at::empty_like(Q);
            const at::Tensor ws = buffer(workspace_bytes(B, H, N, D, dt, causal, 1), Q);
            const int rc = (norm ? bwd_qknorm_saved : bwd_saved)(
                Q.data_ptr(), s[1].data_ptr(), s[2].data_ptr(), s[3].data_ptr(), (const float *)s[4].data_ptr(),
                dO.data_ptr(), out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(), B, H, N, D, (float)a, (float)b,
                causal, dt, ws.data_ptr(), bytes(ws), sums.defined() ? sums.data_ptr() : nullptr,
                sums.defined() ? bytes(sums) : 0, current_stream(Q), nullptr);
            if (rc == 0) return out;
        }
        // gradients of another kind, or a call that the library refuses: the Python code takes or words it
        pybind11::gil_scoped_acquire gil;
        PyObject *none = Py_None;
        Py_INCREF(none);
        PyObject *got = PyObject_CallFunction(
            python_backward, "NNNNNNNddii", THPVariable_Wrap(Q), THPVariable_Wrap(s[1]), THPVariable_Wrap(s[2]),
            THPVariable_Wrap(s[3]), THPVariable_Wrap(s[4]), THPVariable_Wrap(dO),
            sums.defined() ? (Py_DECREF(none), THPVariable_Wrap(sums)) : none, a, b, (int)causal, (int)norm);
        if (!got) {
            python_error e;
            e.persist();
            throw e;
        }
        for (int i = 0; i < 3; ++i) out[i] = tensor(PyTuple_GET_ITEM(got, i));
        Py_DECREF(got);
        return out;
    }
};

// What grad_fn shows of LinearAttentionFunction's own: saved_tensors, la_args and la_saved.
using AttentionNode = torch::autograd::CppNode<Attention>;
AttentionNode &node(PyObject *self)
{
    return static_cast<AttentionNode &>(*reinterpret_cast<torch::autograd::THPCppFunction *>(self)->cdata);
}
PyObject *saved_tensors(PyObject *self, void *)
{
    HANDLE_TH_ERRORS
    const auto saved = node(self).ctx_.get_saved_variables();
    PyObject *t = PyTuple_New((Py_ssize_t)saved.size());
    for (size_t i = 0; t && i < saved.size(); ++i) PyTuple_SET_ITEM(t, (Py_ssize_t)i, THPVariable_Wrap(saved[i]));
    return t;
    END_HANDLE_TH_ERRORS
}
PyObject *la_args(PyObject *self, void *)
{
    HANDLE_TH_ERRORS
    auto &d = node(self).ctx_.saved_data;
    return Py_BuildValue("ddNN", d["a"].toDouble(), d["b"].toDouble(), PyBool_FromLong(d["causal"].toBool()),
                         PyBool_FromLong(d["norm"].toBool()));
    END_HANDLE_TH_ERRORS
}
PyObject *la_saved(PyObject *self, void *)
{
    HANDLE_TH_ERRORS
    const auto &d = node(self).ctx_.saved_data;
    const auto it = d.find("sums");
    if (it == d.end()) Py_RETURN_NONE;
    return THPVariable_Wrap(it->second.toTensor());
    END_HANDLE_TH_ERRORS
}
void show_node()
{
    using namespace torch::autograd;
    static PyTypeObject type;
    if (type.tp_name) return;
    static PyMethodDef functions[] = {{"name", THPCppFunction_name, METH_NOARGS, nullptr},
                                      {"register_hook", THPCppFunction_register_hook, METH_O, nullptr},
                                      {"register_prehook", THPCppFunction_register_prehook, METH_O, nullptr},
                                      {"_register_hook_dict", THPCppFunction_register_hook_dict, METH_O, nullptr},
                                      {"_sequence_nr", THPCppFunction_sequence_nr, METH_NOARGS, nullptr},
                                      {nullptr}};
    static PyGetSetDef properties[] = {{"next_functions", THPCppFunction_next_functions, nullptr, nullptr, nullptr},
                                       {"requires_grad", THPCppFunction_requires_grad, nullptr, nullptr, nullptr},
                                       {"metadata", THPCppFunction_metadata, nullptr, nullptr, nullptr},
                                       {"_input_metadata", THPCppFunction_input_metadata, nullptr, nullptr, nullptr},
                                       {"saved_tensors", saved_tensors, nullptr, nullptr, nullptr},
                                       {"la_args", la_args, nullptr, nullptr, nullptr},
                                       {"la_saved", la_saved, nullptr, nullptr, nullptr},
                                       {nullptr}};
    registerCppFunction(typeid(AttentionNode),
                        _initFunctionPyTypeObject(type, "LinearAttention", properties, functions));
}

// Q, K, V, a, b, causal, normalise -> O, or the library's status.  None: LinearAttentionFunction takes over, which is
// where modes, transforms and traces that look into Python functions find what they look for.
PyObject *attention(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    at::Tensor O;
    double a = 0, b = 0;
    PyObject *declined = guarded(n, 7, [&]() -> PyObject * {
        for (int i = 0; i < 3; ++i)
            if (!plain(x[i])) Py_RETURN_NONE;
        const at::Tensor &Q = tensor(x[0]);
        require(Q.dim() == 4 && Q.is_cuda());
        dtype_code(Q);
        check_like(Q, {x[1], x[2]});
        for (int i = 0; i < 3; ++i)
            require(tensor(x[i]).is_cuda() && tensor(x[i]).get_device() == Q.get_device() &&
                    !tensor(x[i])._fw_grad(0).defined());
        for (int i = 0; i < 3; ++i) tensor(x[i]).const_data_ptr();  // throws where there is no storage
        require(!at::impl::torch_function_mode_enabled() && !c10::impl::TorchDispatchModeTLS::any_modes_set() &&
                !torch::jit::tracer::isTracing());
        if (const auto &transforms = at::functorch::functorchTLSAccessor())
            transforms->checkSupportsCppAutogradFunction();  // throws inside of vmap, grad and the like
        // a tensor among the coefficients and switches is an input of the Python node: its grad makes O require one
        for (int i = 3; i < 7; ++i)
            require(PyFloat_CheckExact(x[i]) || PyLong_Check(x[i]) || !THPVariable_Check(x[i]));
        a = real(x[3]);
        b = real(x[4]);
        return PyBool_FromLong(1);
    });
    if (declined != Py_True) return declined;
    Py_DECREF(declined);
    const int causal = PyObject_IsTrue(x[5]), norm = PyObject_IsTrue(x[6]);
    if (PyErr_Occurred()) return nullptr;
    try {
        O = Attention::apply(tensor(x[0]), tensor(x[1]), tensor(x[2]), a, b, causal != 0, norm != 0);
    } catch (const Status &s) {
        return PyLong_FromLong(s.rc);
    }
    return THPVariable_Wrap(std::move(O));
    END_HANDLE_TH_ERRORS
}

// python_backward, raw_stream, then the addresses of the entry points in the order of the pointers above
PyObject *init(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    void **const to[] = {(void **)&fwd_plain, (void **)&fwd_qknorm, (void **)&fwd_save, (void **)&fwd_qknorm_save,
                         (void **)&bwd_plain, (void **)&bwd_qknorm, (void **)&bwd_saved, (void **)&bwd_qknorm_saved,
                         (void **)&dec_step, (void **)&dec_prefill, (void **)&workspace_bytes,
                         (void **)&saved_state_bytes};
    constexpr Py_ssize_t COUNT = sizeof(to) / sizeof(to[0]);
    if (n != 2 + COUNT) {
        PyErr_SetString(PyExc_TypeError, "init takes two callables and the entry points' addresses");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < COUNT; ++i) {
        *to[i] = PyLong_AsVoidPtr(x[2 + i]);
        if (!*to[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    Py_INCREF(x[0]);
    Py_XSETREF(python_backward, x[0]);
    Py_INCREF(x[1]);
    Py_XSETREF(raw_stream, x[1]);
    HANDLE_TH_ERRORS
    show_node();
    Py_RETURN_NONE;
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"init", (PyCFunction)(void (*)())init, METH_FASTCALL, nullptr},
                         {"forward", (PyCFunction)(void (*)())forward, METH_FASTCALL, nullptr},
                         {"backward", (PyCFunction)(void (*)())backward, METH_FASTCALL, nullptr},
                         {"attention", (PyCFunction)(void (*)())attention, METH_FASTCALL, nullptr},
                         {"decode_step", (PyCFunction)(void (*)())decode_step, METH_FASTCALL, nullptr},
                         {"decode_prefill", (PyCFunction)(void (*)())decode_prefill, METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", LA_BUILT_FOR) < 0) Py_CLEAR(m);
    return m;
}
