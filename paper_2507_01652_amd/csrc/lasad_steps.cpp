// The decode steps' marshalling as a CPython extension (module _steps): what binding.py does for them in Python (shape, type
// and layout checks, pointers, the current stream), for plain GPU tensors.  A decode step is one short kernel, so a loop of them is
// bound by the host: one image through twelve layers 79 us a token with the checks in Python and ctypes, 48 with these.
//
// Every function returns the output tensor, a status of the library (an int other than 0), or None where an argument is not what
// it expects: binding.py then goes through its own checks, so that a wrong call fails there as it always did.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/lasad.h"

namespace {

// An argument that does not fit ends the call (None to the caller).
struct NotHandled {};

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw NotHandled();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided || t.numel() == 0 || !t.is_contiguous()) throw NotHandled();
    return t;
}

int code(const at::Tensor &t)
{
    if (t.scalar_type() == at::kBFloat16) return LASAD_BF16;
    if (t.scalar_type() == at::kFloat) return LASAD_F32;
    throw NotHandled();
}

int integer(PyObject *o)
{
    if (!PyLong_CheckExact(o)) throw NotHandled();
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow || v != (int)v) throw NotHandled();
    return (int)v;
}

float real(PyObject *o)
{
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    return (float)integer(o);
}

void *stream(PyObject *o)                          // a handle, or None: the current stream
{
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    if (!PyLong_CheckExact(o)) throw NotHandled();
    void *p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) { PyErr_Clear(); throw NotHandled(); }
    return p;
}

// What all steps have: q [B, Hh, d] and its like, the fp32 state [B, Hh, d, d], the output.
struct Step {
    const at::Tensor &q;
    int B, Hh, d, io;
    explicit Step(PyObject *o) : q(tensor(o))
    {
        if (q.dim() != 3) throw NotHandled();
        B = (int)q.size(0); Hh = (int)q.size(1); d = (int)q.size(2);
        if (q.size(0) != B || q.size(1) != Hh || q.size(2) != d) throw NotHandled();
        io = code(q);
    }
    const void *like(PyObject *o, bool optional = false) const      // a tensor like q
    {
        if (optional && o == Py_None) return nullptr;
        const at::Tensor &t = tensor(o);
        if (t.scalar_type() != q.scalar_type() || t.sizes() != q.sizes()) throw NotHandled();
        return t.data_ptr();
    }
    float *state(PyObject *o) const
    {
        const at::Tensor &t = tensor(o);
        if (t.scalar_type() != at::kFloat || t.dim() != 4 || t.size(0) != B || t.size(1) != Hh || t.size(2) != d || t.size(3) != d) throw NotHandled();
        return (float *)t.data_ptr();
    }
    const float *floats(PyObject *o, int64_t n, bool optional) const
    {
        if (optional && o == Py_None) return nullptr;
        const at::Tensor &t = tensor(o);
        if (t.scalar_type() != at::kFloat || t.numel() != n) throw NotHandled();
        return (const float *)t.data_ptr();
    }
    void *out(PyObject *o, int &type, at::Tensor &made) const       // None: a new one like q
    {
        if (o == Py_None) made = at::empty_like(q);
        const at::Tensor &t = o == Py_None ? made : tensor(o);
        if (t.sizes() != q.sizes()) throw NotHandled();
        type = code(t);
        return t.data_ptr();
    }
};

template <typename F>
PyObject *call(PyObject *const *args, Py_ssize_t got, Py_ssize_t want, int out_arg, F step)
{
    if (got != want) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    at::Tensor made;
    try {
        const int status = step(made);
        if (status != 0) return PyLong_FromLong(status);
    } catch (const NotHandled &) {
        Py_RETURN_NONE;
    } catch (const std::exception &) {             // (of torch, on a tensor that has no memory to point at)
        Py_RETURN_NONE;
    }
    if (made.defined()) return THPVariable_Wrap(made);
    Py_INCREF(args[out_arg]);
    return args[out_arg];
}

#define WITHOUT_GIL(expr) [&] { int rc_; Py_BEGIN_ALLOW_THREADS rc_ = (expr); Py_END_ALLOW_THREADS return rc_; }()

// q, k, v, gamma, state, grid_h, grid_w, pos, boundary_mode, q_scale, out, stream
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 12, 10, [&](at::Tensor &made) {
        const Step s(a[0]);
        const void *k = s.like(a[1]), *v = s.like(a[2]);
        const at::Tensor &g = tensor(a[3]);
        if (g.dim() != 1) throw NotHandled();
        const float *gamma = s.floats(a[3], s.Hh, false);
        float *state = s.state(a[4]);
        const int gh = integer(a[5]), gw = integer(a[6]), pos = integer(a[7]), mode = integer(a[8]);
        const float scale = real(a[9]);
        int ot;
        void *o = s.out(a[10], ot, made), *st = stream(a[11]);
        return WITHOUT_GIL(lasad_decode_step(s.q.data_ptr(), k, v, o, s.io, ot, s.B, s.Hh, s.d, gh, gw, pos, gamma, mode, scale, state, st));
    });
}

// q, lam, v, state, grid_h, grid_w, pos, k, boundary_mode, q_scale, out, stream
PyObject *decode_step_gated(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 12, 10, [&](at::Tensor &made) {
        const Step s(a[0]);
        const void *lam = s.like(a[1]), *v = s.like(a[2]);
        float *state = s.state(a[3]);
        const int gh = integer(a[4]), gw = integer(a[5]), pos = integer(a[6]), mode = integer(a[8]);
        const void *k = s.like(a[7], true);
        const float scale = real(a[9]);
        int ot;
        void *o = s.out(a[10], ot, made), *st = stream(a[11]);
        return WITHOUT_GIL(lasad_decode_step_gated(s.q.data_ptr(), lam, k, v, o, s.io, ot, s.B, s.Hh, s.d, gh, gw, pos, mode, scale, state, st));
    });
}

// q_pre, z, v, state, grid_h, grid_w, pos, norm_weight, norm_eps, boundary_mode, q_scale, out, stream
PyObject *decode_step_layer(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 13, 11, [&](at::Tensor &made) {
        const Step s(a[0]);
        const void *z = s.like(a[1]), *v = s.like(a[2]);
        float *state = s.state(a[3]);
        const int gh = integer(a[4]), gw = integer(a[5]), pos = integer(a[6]), mode = integer(a[9]);
        const float *w = s.floats(a[7], (int64_t)s.Hh * s.d, true);
        const float eps = real(a[8]), scale = real(a[10]);
        int ot;
        void *o = s.out(a[11], ot, made), *st = stream(a[12]);
        return WITHOUT_GIL(lasad_decode_step_layer(s.q.data_ptr(), z, v, o, s.io, ot, s.B, s.Hh, s.d, gh, gw, pos, mode, scale, w, eps, state, st));
    });
}

// q, v, state, pos_rows, grid_h, grid_w, k, lam, gamma, boundary_mode, q_scale, out, stream
PyObject *decode_step_rows(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 13, 11, [&](at::Tensor &made) {
        const Step s(a[0]);
        const void *v = s.like(a[1]);
        float *state = s.state(a[2]);
        const at::Tensor &p = tensor(a[3]);
        if (p.scalar_type() != at::kInt || p.numel() != s.B) throw NotHandled();
        const int gh = integer(a[4]), gw = integer(a[5]), mode = integer(a[9]);
        const void *k = s.like(a[6], true), *lam = s.like(a[7], true);
        const float *gamma = s.floats(a[8], s.Hh, true);
        const float scale = real(a[10]);
        int ot;
        void *o = s.out(a[11], ot, made), *st = stream(a[12]);
        return WITHOUT_GIL(lasad_decode_step_rows(s.q.data_ptr(), lam, k, v, o, s.io, ot, s.B, s.Hh, s.d, gh, gw, (const int32_t *)p.data_ptr(),
                                                  gamma, mode, scale, state, st));
    });
}

PyMethodDef methods[] = {
    {"decode_step", (PyCFunction)(void (*)(void))decode_step, METH_FASTCALL, nullptr},
    {"decode_step_gated", (PyCFunction)(void (*)(void))decode_step_gated, METH_FASTCALL, nullptr},
    {"decode_step_layer", (PyCFunction)(void (*)(void))decode_step_layer, METH_FASTCALL, nullptr},
    {"decode_step_rows", (PyCFunction)(void (*)(void))decode_step_rows, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_steps", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__steps() { return PyModule_Create(&module); }
