// The shuffle's calls for binding.py without the interpreter in between: one call from Python per library call that checks the
// tensors, takes their pointers and the current stream, and enqueues.  A call of the ctypes path spends 2 to 3 us on the checks and on
// building arguments, as much as the launch itself takes (2.3 us), and a decode batch of a few tokens is bound by that: 4 tokens, two
// calls, 11.5 us with ctypes.
//
// Only the plain case is handled: exact torch.Tensor objects that satisfy every check, no stream argument, no torch function mode.
// Anything else returns None and the caller goes its own way through the checks of binding.py, which accept or refuse it as
// they do without this module.  Otherwise the library's return code is returned.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include "fusco.h"

namespace {

// the library's entry points, by bind(): this module is not linked against it
decltype(&fusco_plan) p_plan = nullptr;
decltype(&fusco_dispatch) p_dispatch = nullptr;
decltype(&fusco_plan_dispatch) p_plan_dispatch = nullptr;
decltype(&fusco_combine) p_combine = nullptr;
decltype(&fusco_combine_two_hop) p_combine_two_hop = nullptr;

PyObject *s_c, *s_scratch;   // attribute names of Layout

// The C struct of a Layout object, held by the buffer of its ctypes structure for the duration of the call.
struct LayoutRef {
    PyObject *c = nullptr;
    Py_buffer view{};
    bool ok = false;
    explicit LayoutRef(PyObject *layout)
    {
        c = PyObject_GetAttr(layout, s_c);
        if (!c || PyObject_GetBuffer(c, &view, PyBUF_WRITABLE) != 0) {
            PyErr_Clear();
            return;
        }
        ok = view.len == (Py_ssize_t)sizeof(fusco_layout);
    }
    ~LayoutRef()
    {
        if (view.obj) PyBuffer_Release(&view);
        Py_XDECREF(c);
    }
    LayoutRef(const LayoutRef &) = delete;
    fusco_layout *operator->() const { return (fusco_layout *)view.buf; }
    fusco_layout *get() const { return (fusco_layout *)view.buf; }
};

const at::Tensor *tensor(PyObject *o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

// binding.py's _rows: contiguous 2-D device tensor of at least min_rows rows; its row size in bytes, -1 otherwise
int64_t rows(const at::Tensor &t, int64_t min_rows)
{
    if (!t.is_cuda() || t.dim() != 2 || !t.is_contiguous() || t.size(0) < min_rows) return -1;
    return t.size(1) * (int64_t)t.element_size();
}

bool matrix_of(const at::Tensor &t, at::ScalarType type, int64_t n, int64_t k)
{
    return t.is_cuda() && t.scalar_type() == type && t.is_contiguous() && t.dim() == 2 && t.size(0) == n && t.size(1) == k;
}

int dtype_code(const at::Tensor &t)
{
    return t.scalar_type() == at::kBFloat16 ? FUSCO_BF16 : t.scalar_type() == at::kFloat ? FUSCO_F32 : -1;
}

void *current_stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// f() either returns a code of the library (with the interpreter released around the call) or kElsewhere
constexpr int kElsewhere = 1;

template <typename F>
PyObject *guarded(F f)
{
    int rc = kElsewhere;
    try {
        if (!at::impl::torch_function_mode_enabled()) rc = f();
    } catch (...) {   // a tensor without storage, for instance: the caller's own path raises what it raises
        rc = kElsewhere;
    }
    if (rc == kElsewhere) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

template <typename F>
int released(F f)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

// plan(layout, topk_idx)
PyObject *plan(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2 || !p_plan) Py_RETURN_NONE;
    return guarded([&]() -> int {
        LayoutRef L(args[0]);
        const at::Tensor *A = tensor(args[1]);
        if (!L.ok || !A || !matrix_of(*A, at::kInt, L->N, L->k)) return kElsewhere;
        PyObject *so = PyObject_GetAttr(args[0], s_scratch);
        const at::Tensor *s = so ? tensor(so) : nullptr;
        int rc = kElsewhere;
        if (s) {
            void *a = A->data_ptr(), *m = s->data_ptr(), *stream = current_stream();
            const int64_t bytes = s->numel();
            rc = released([&] { return p_plan(L.get(), (const int32_t *)a, m, (size_t)bytes, stream); });
        }
        Py_XDECREF(so);
        return rc;
    });
}

struct Plane {
    void *p = nullptr;
    int64_t row = 0;
};

// a plane that may be absent (None): false where it is neither that nor fit
bool plane(PyObject *o, int64_t min_rows, Plane &out)
{
    if (o == Py_None) return true;
    const at::Tensor *t = tensor(o);
    if (!t || (out.row = rows(*t, min_rows)) < 0) return false;
    out.p = t->data_ptr();
    return true;
}

// dispatch(layout, x, expert_buf, x_aux, expert_aux, send_buf, send_aux, flags)
PyObject *dispatch(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 8 || !p_dispatch || !PyLong_CheckExact(args[7])) Py_RETURN_NONE;
    return guarded([&]() -> int {
        const long flags = PyLong_AsLong(args[7]);
        if (flags < 0 || flags > 15) return kElsewhere;
        LayoutRef L(args[0]);
        if (!L.ok) return kElsewhere;
        long which = flags & ~(long)FUSCO_DISPATCH_STREAMING;
        if (which == 0) which = FUSCO_DISPATCH_EXPERT;
        if (which & FUSCO_DISPATCH_TWO_HOP) which |= FUSCO_DISPATCH_EXPERT | FUSCO_DISPATCH_WIRE;
        const bool expert = which & FUSCO_DISPATCH_EXPERT, wire = which & FUSCO_DISPATCH_WIRE;
        Plane x, xa, e, ea, w, wa;
        if (args[1] == Py_None || !plane(args[1], L->N, x) || !plane(args[3], L->N, xa)) return kElsewhere;
        // tensors that the flags do not ask for are passed on as they are, unchecked, by the other path
        if (!expert && (args[2] != Py_None || args[4] != Py_None)) return kElsewhere;
        if (!wire && (args[5] != Py_None || args[6] != Py_None)) return kElsewhere;
        if (!plane(args[2], L->P, e) || !plane(args[4], L->P, ea) || !plane(args[5], L->send_cap, w) || !plane(args[6], L->send_cap, wa))
            return kElsewhere;
        if (expert && (args[2] == Py_None || e.row != x.row || (xa.row ? ea.row != xa.row || args[4] == Py_None : args[4] != Py_None))) return kElsewhere;
        if (wire && (args[5] == Py_None || w.row != x.row || (xa.row ? wa.row != xa.row || args[6] == Py_None : args[6] != Py_None))) return kElsewhere;
        void *stream = current_stream();
        return released([&] {
            return p_dispatch(L.get(), x.p, (size_t)x.row, xa.p, (size_t)xa.row, e.p, ea.p, w.p, wa.p, (uint32_t)flags, stream);
        });
    });
}

// plan_dispatch(layout, topk_idx, x, expert_buf, x_aux, expert_aux)
PyObject *plan_dispatch(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 6 || !p_plan_dispatch) Py_RETURN_NONE;
    return guarded([&]() -> int {
        LayoutRef L(args[0]);
        const at::Tensor *A = tensor(args[1]);
        if (!L.ok || !A || !matrix_of(*A, at::kInt, L->N, L->k)) return kElsewhere;
        Plane x, e, xa, ea;
        if (args[2] == Py_None || args[3] == Py_None || !plane(args[2], L->N, x) || !plane(args[3], L->P, e) || e.row != x.row) return kElsewhere;
        if (!plane(args[4], L->N, xa) || !plane(args[5], L->P, ea)) return kElsewhere;
        if (xa.row ? args[5] == Py_None || ea.row != xa.row : args[5] != Py_None) return kElsewhere;
        void *a = A->data_ptr(), *stream = current_stream();
        return released([&] {
            return p_plan_dispatch(L.get(), (const int32_t *)a, x.p, (size_t)x.row, xa.p, (size_t)xa.row, e.p, ea.p, stream);
        });
    });
}

// what combine and two-hop combine share: y, w, out
struct Sums {
    const at::Tensor *y, *w, *out;
    int yt, ot;
    int64_t H;
    bool ok;
    Sums(const LayoutRef &L, PyObject *oy, PyObject *ow, PyObject *oo) : y(tensor(oy)), w(tensor(ow)), out(tensor(oo)), yt(-1), ot(-1), H(0), ok(false)
    {
        if (!L.ok || !y || !w || !out || rows(*y, L->P) < 0 || rows(*out, L->N) < 0) return;
        H = y->size(1);
        yt = dtype_code(*y);
        ot = dtype_code(*out);
        ok = out->size(1) == H && H <= INT32_MAX && yt >= 0 && ot >= 0 && matrix_of(*w, at::kFloat, L->N, L->k);
    }
};

// combine(layout, y, w, out)
PyObject *combine(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 4 || !p_combine) Py_RETURN_NONE;
    return guarded([&]() -> int {
        LayoutRef L(args[0]);
        Sums s(L, args[1], args[2], args[3]);
        if (!s.ok) return kElsewhere;
        void *y = s.y->data_ptr(), *w = s.w->data_ptr(), *out = s.out->data_ptr(), *stream = current_stream();
        return released([&] { return p_combine(L.get(), y, s.yt, (const float *)w, out, s.ot, (int32_t)s.H, 0, stream); });
    });
}

// combine_two_hop(layout, y, w, partial, out)
PyObject *combine_two_hop(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5 || !p_combine_two_hop) Py_RETURN_NONE;
    return guarded([&]() -> int {
        LayoutRef L(args[0]);
        Sums s(L, args[1], args[2], args[4]);
        const at::Tensor *p = tensor(args[3]);
        if (!s.ok || !p || s.H % 4 != 0 || p->scalar_type() != at::kFloat || rows(*p, L->send_cap) != 4 * s.H) return kElsewhere;
        void *y = s.y->data_ptr(), *w = s.w->data_ptr(), *part = p->data_ptr(), *out = s.out->data_ptr(), *stream = current_stream();
        return released([&] { return p_combine_two_hop(L.get(), y, s.yt, (const float *)w, (float *)part, out, s.ot, (int32_t)s.H, stream); });
    });
}

// bind(plan, dispatch, plan_dispatch, combine, combine_two_hop): addresses of the library's entry points
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long a[5];
    if (!PyArg_ParseTuple(args, "KKKKK", a, a + 1, a + 2, a + 3, a + 4)) return nullptr;
    p_plan = (decltype(p_plan))(uintptr_t)a[0];
    p_dispatch = (decltype(p_dispatch))(uintptr_t)a[1];
    p_plan_dispatch = (decltype(p_plan_dispatch))(uintptr_t)a[2];
    p_combine = (decltype(p_combine))(uintptr_t)a[3];
    p_combine_two_hop = (decltype(p_combine_two_hop))(uintptr_t)a[4];
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)bind, METH_VARARGS, nullptr},
    {"plan", (PyCFunction)(void (*)())plan, METH_FASTCALL, nullptr},
    {"dispatch", (PyCFunction)(void (*)())dispatch, METH_FASTCALL, nullptr},
    {"plan_dispatch", (PyCFunction)(void (*)())plan_dispatch, METH_FASTCALL, nullptr},
    {"combine", (PyCFunction)(void (*)())combine, METH_FASTCALL, nullptr},
    {"combine_two_hop", (PyCFunction)(void (*)())combine_two_hop, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods};

}   // namespace

PyMODINIT_FUNC PyInit__fastcall()
{
    s_c = PyUnicode_InternFromString("c");
    s_scratch = PyUnicode_InternFromString("scratch");
    return s_c && s_scratch ? PyModule_Create(&module) : nullptr;
}
