// Argument marshalling of the small, frequent calls (binding.py) in native code: the checks, addresses
// and conversions that the Python functions of the same names make, one tensor at a time, took most
// of a decode step's 7 us.  Takes plain tensors only, without a trace; everything else stays with the Python
// functions, which are also what a build without this file runs.
//
// Refuses nothing itself: what does not pass the checks (a tensor without storage or a functorch wrapper, whose
// C++ exception ends up here, included) goes back to the Python functions, which refuse or take it.  The library
// is called without the interpreter lock, as ctypes does.
#include <torch/csrc/autograd/python_variable.h>

#include "la.h"

namespace {

PyObject *raw_stream = nullptr;  // device index -> stream handle of its current stream

// Entry points of libla.so, as addresses (binding.py has loaded the library).
decltype(&la_forward_traced) fwd_plain, fwd_qknorm;
decltype(&la_forward_save) fwd_save, fwd_qknorm_save;
decltype(&la_backward_traced) bwd_plain, bwd_qknorm;
decltype(&la_backward_saved) bwd_saved, bwd_qknorm_saved;
decltype(&la_decode_step) dec_step;
decltype(&la_decode_prefill) dec_prefill;

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
float number(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    PyObject *f = PyNumber_Float(o);  // what float(o) gives
    require(f);
    const double x = PyFloat_AS_DOUBLE(f);
    Py_DECREF(f);
    return (float)x;
}
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

// raw_stream, then the addresses of the entry points in the order of the pointers above
PyObject *init(PyObject *, PyObject *const *x, Py_ssize_t n)
{
    void **const to[] = {(void **)&fwd_plain, (void **)&fwd_qknorm, (void **)&fwd_save, (void **)&fwd_qknorm_save,
                         (void **)&bwd_plain, (void **)&bwd_qknorm, (void **)&bwd_saved, (void **)&bwd_qknorm_saved,
                         (void **)&dec_step, (void **)&dec_prefill};
    constexpr Py_ssize_t COUNT = sizeof(to) / sizeof(to[0]);
    if (n != 1 + COUNT) {
        PyErr_SetString(PyExc_TypeError, "init takes a callable and the entry points' addresses");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < COUNT; ++i) {
        *to[i] = PyLong_AsVoidPtr(x[1 + i]);
        if (!*to[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    Py_INCREF(x[0]);
    Py_XSETREF(raw_stream, x[0]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"init", (PyCFunction)(void (*)())init, METH_FASTCALL, nullptr},
                         {"forward", (PyCFunction)(void (*)())forward, METH_FASTCALL, nullptr},
                         {"backward", (PyCFunction)(void (*)())backward, METH_FASTCALL, nullptr},
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
