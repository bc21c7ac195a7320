// The marshalling of the decode steps, the forwards and the backwards as a CPython extension (module _steps): what binding.py does for
// them in Python (shape, type and layout checks, pointers, new outputs and workspaces, the current stream), for plain GPU tensors.  A
// decode step is one short kernel, so a loop of them is bound by the host: one image through twelve layers 79 us a token with the
// checks in Python and ctypes, 48 with these; so is a prefill of few sequences: 96 of 256
// tokens 11.5 us a call with the checks in Python, 6.7 with these, 60 of 311 with carried states 11.9 and 6.2.
//
// Every function returns the output tensor (the backwards: a tuple of gradients), a status of the library (an int other than 0), or
// None where an argument is not what it expects: binding.py then goes through its own checks, so that a wrong call fails there as it
// always did.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/lasad.h"

namespace {

// An argument that does not fit ends the call (None to the caller).
struct NotHandled {};

const at::Tensor &any_strides(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) throw NotHandled();
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided || t.numel() == 0) throw NotHandled();
    return t;
}

const at::Tensor &tensor(PyObject *o)
{
    const at::Tensor &t = any_strides(o);
    if (!t.is_contiguous()) throw NotHandled();
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

// What the calls over a token axis have: q [B, n, Hh, d] with unit stride along d, its like in shape, strides and type, states.
lasad_layout_t layout(const at::Tensor &t)
{
    if (t.dim() != 4 || (t.size(3) > 1 && t.stride(3) != 1)) throw NotHandled();
    return {t.stride(0), t.stride(1), t.stride(2)};
}

struct Sequences {
    const at::Tensor &q;
    lasad_layout_t in;
    int B, n, Hh, d, io;
    explicit Sequences(PyObject *o) : q(any_strides(o)), in(layout(q))
    {
        B = (int)q.size(0); n = (int)q.size(1); Hh = (int)q.size(2); d = (int)q.size(3);
        if (q.size(0) != B || q.size(1) != n || q.size(2) != Hh || q.size(3) != d) throw NotHandled();
        io = code(q);
    }
    const void *like(PyObject *o, bool optional = false) const
    {
        if (optional && o == Py_None) return nullptr;
        const at::Tensor &t = any_strides(o);
        if (t.scalar_type() != q.scalar_type() || t.sizes() != q.sizes() || t.strides() != q.strides()) throw NotHandled();
        return t.data_ptr();
    }
    float *state(PyObject *o) const                                 // or None
    {
        if (o == Py_None) return nullptr;
        const at::Tensor &t = tensor(o);
        if (t.scalar_type() != at::kFloat || t.dim() != 4 || t.size(0) != B || t.size(1) != Hh || t.size(2) != d || t.size(3) != d) throw NotHandled();
        return (float *)t.data_ptr();
    }
    const float *floats(PyObject *o, int64_t count, bool optional) const
    {
        if (optional && o == Py_None) return nullptr;
        const at::Tensor &t = tensor(o);
        if (t.scalar_type() != at::kFloat || t.numel() != count) throw NotHandled();
        return (const float *)t.data_ptr();
    }
    void *out(PyObject *o, int &type, lasad_layout_t &l, at::Tensor &made) const       // None: a new one like q
    {
        if (o == Py_None) made = at::empty_like(q);
        const at::Tensor &t = o == Py_None ? made : any_strides(o);
        if (t.sizes() != q.sizes()) throw NotHandled();
        type = code(t);
        l = layout(t);
        return t.data_ptr();
    }
    at::Tensor fp32(at::IntArrayRef sizes) const { return at::empty(sizes, q.options().dtype(at::kFloat)); }
    at::Tensor bytes(size_t n_bytes) const { return at::empty({(int64_t)n_bytes}, q.options().dtype(at::kByte)); }
};

// q, k, v, gamma, grid_h, grid_w, start_pos, boundary_mode, q_scale, state_in, state_out, out
PyObject *forward_chunked(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 12, 11, [&](at::Tensor &made) {
        const Sequences s(a[0]);
        const void *k = s.like(a[1]), *v = s.like(a[2]);
        if (tensor(a[3]).dim() != 1) throw NotHandled();
        const float *gamma = s.floats(a[3], s.Hh, false);
        const int gh = integer(a[4]), gw = integer(a[5]), start = integer(a[6]), mode = integer(a[7]);
        const float scale = real(a[8]);
        const float *s0 = s.state(a[9]);
        float *s1 = s.state(a[10]);
        int ot;
        lasad_layout_t lo;
        void *o = s.out(a[11], ot, lo, made), *st = stream(Py_None);
        const size_t need = lasad_forward_workspace_bytes(s.B, s.Hh, s.n, s.d, s.io);
        at::Tensor ws;
        if (need) ws = s.bytes(need);
        return WITHOUT_GIL(lasad_forward_chunked(s.q.data_ptr(), k, v, o, &s.in, &lo, s.io, ot, s.B, s.Hh, s.d, gh, gw, start, s.n, gamma, mode,
                                                 scale, s0, s1, need ? ws.data_ptr() : nullptr, need, st));
    });
}

// q, lam, v, grid_h, grid_w, k, start_pos, boundary_mode, q_scale, state_in, state_out, out
PyObject *forward_gated(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 12, 11, [&](at::Tensor &made) {
        const Sequences s(a[0]);
        const void *lam = s.like(a[1]), *v = s.like(a[2]), *k = s.like(a[5], true);
        const int gh = integer(a[3]), gw = integer(a[4]), start = integer(a[6]), mode = integer(a[7]);
        const float scale = real(a[8]);
        const float *s0 = s.state(a[9]);
        float *s1 = s.state(a[10]);
        int ot;
        lasad_layout_t lo;
        void *o = s.out(a[11], ot, lo, made), *st = stream(Py_None);
        return WITHOUT_GIL(lasad_forward_gated(s.q.data_ptr(), lam, k, v, o, &s.in, &lo, s.io, ot, s.B, s.Hh, s.d, gh, gw, start, s.n, mode, scale,
                                               s0, s1, st));
    });
}

// q_pre, z, v, grid_h, grid_w, norm_weight, norm_eps, start_pos, boundary_mode, q_scale, state_in, state_out, out
PyObject *forward_layer(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return call(a, n, 13, 12, [&](at::Tensor &made) {
        const Sequences s(a[0]);
        const void *z = s.like(a[1]), *v = s.like(a[2]);
        const int gh = integer(a[3]), gw = integer(a[4]), start = integer(a[7]), mode = integer(a[8]);
        const float *w = s.floats(a[5], (int64_t)s.Hh * s.d, true);
        const float eps = real(a[6]), scale = real(a[9]);
        const float *s0 = s.state(a[10]);
        float *s1 = s.state(a[11]);
        int ot;
        lasad_layout_t lo;
        void *o = s.out(a[12], ot, lo, made), *st = stream(Py_None);
        return WITHOUT_GIL(lasad_forward_layer(s.q.data_ptr(), z, v, o, &s.in, &lo, s.io, ot, s.B, s.Hh, s.d, gh, gw, start, s.n, mode, scale, w, eps,
                                               s0, s1, st));
    });
}

// The backwards: new gradients like q, and what comes with them, as a tuple.
template <typename F>
PyObject *gradients(Py_ssize_t got, Py_ssize_t want, F step)
{
    if (got != want) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    at::Tensor made[4];                            // (an undefined one: None)
    int count = 0;
    try {
        const int status = step(made, count);
        if (status != 0) return PyLong_FromLong(status);
    } catch (const NotHandled &) {
        Py_RETURN_NONE;
    } catch (const std::exception &) {
        Py_RETURN_NONE;
    }
    PyObject *all = PyTuple_New(count);
    if (!all) return nullptr;
    for (int i = 0; i < count; ++i) {
        PyObject *x = made[i].defined() ? THPVariable_Wrap(made[i]) : Py_None;
        if (!x) { Py_DECREF(all); return nullptr; }
        if (x == Py_None) Py_INCREF(x);
        PyTuple_SET_ITEM(all, i, x);
    }
    return all;
}

// q, k, v, d_o, gamma, grid_h, grid_w, start_pos, boundary_mode, q_scale
PyObject *backward_chunked(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return gradients(n, 10, [&](at::Tensor (&g)[4], int &count) {
        const Sequences s(a[0]);
        const void *k = s.like(a[1]), *v = s.like(a[2]), *d_o = s.like(a[3]);
        const float *gamma = s.floats(a[4], s.Hh, false);
        const int gh = integer(a[5]), gw = integer(a[6]), start = integer(a[7]), mode = integer(a[8]);
        const float scale = real(a[9]);
        count = 4;
        for (int i = 0; i < 3; ++i) g[i] = at::empty_like(s.q);
        g[3] = s.fp32({s.Hh});
        const lasad_layout_t lg = layout(g[0]);
        const size_t need = lasad_backward_workspace_bytes(s.B, s.Hh, s.n, s.d, s.io);
        at::Tensor ws = s.bytes(need);
        void *st = stream(Py_None);
        return WITHOUT_GIL(lasad_backward_chunked(s.q.data_ptr(), k, v, d_o, g[0].data_ptr(), g[1].data_ptr(), g[2].data_ptr(), (float *)g[3].data_ptr(),
                                                  &s.in, &lg, s.io, s.io, s.B, s.Hh, s.d, gh, gw, start, s.n, gamma, mode, scale, ws.data_ptr(),
                                                  need, st));
    });
}

// q, lam, v, d_o, grid_h, grid_w, k, start_pos, boundary_mode, q_scale
PyObject *backward_gated(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return gradients(n, 10, [&](at::Tensor (&g)[4], int &count) {
        const Sequences s(a[0]);
        const void *lam = s.like(a[1]), *v = s.like(a[2]), *d_o = s.like(a[3]), *k = s.like(a[6], true);
        const int gh = integer(a[4]), gw = integer(a[5]), start = integer(a[7]), mode = integer(a[8]);
        const float scale = real(a[9]);
        count = k ? 4 : 3;                         // dq, dlam, dv, dk
        for (int i = 0; i < count; ++i) g[i] = at::empty_like(s.q);
        const lasad_layout_t lg = layout(g[0]);
        const size_t need = lasad_backward_gated_workspace_bytes(s.B, s.Hh, s.n, s.d);
        at::Tensor ws = s.bytes(need);
        void *st = stream(Py_None);
        return WITHOUT_GIL(lasad_backward_gated(s.q.data_ptr(), lam, k, v, d_o, g[0].data_ptr(), g[1].data_ptr(), k ? g[3].data_ptr() : nullptr,
                                                g[2].data_ptr(), &s.in, &lg, s.io, s.io, s.B, s.Hh, s.d, gh, gw, start, s.n, mode, scale,
                                                ws.data_ptr(), need, st));
    });
}

// q_pre, z, v, d_out, grid_h, grid_w, norm_weight, norm_eps, start_pos, boundary_mode, q_scale, want_dweight
PyObject *backward_layer(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    return gradients(n, 12, [&](at::Tensor (&g)[4], int &count) {
        const Sequences s(a[0]);
        const void *z = s.like(a[1]), *v = s.like(a[2]);
        const at::Tensor &d_out = any_strides(a[3]);
        if (d_out.sizes() != s.q.sizes() || d_out.scalar_type() != s.q.scalar_type()) throw NotHandled();
        const lasad_layout_t lo = layout(d_out);
        const int gh = integer(a[4]), gw = integer(a[5]), start = integer(a[8]), mode = integer(a[9]);
        const float *w = s.floats(a[6], (int64_t)s.Hh * s.d, true);
        const float eps = real(a[7]), scale = real(a[10]);
        count = 4;
        for (int i = 0; i < 3; ++i) g[i] = at::empty_like(s.q);
        if (a[11] == Py_True) g[3] = s.fp32({s.Hh, s.d});
        else if (a[11] != Py_False) throw NotHandled();
        const lasad_layout_t lg = layout(g[0]);
        const size_t need = lasad_backward_layer_workspace_bytes(s.B, s.Hh, s.n, s.d, s.io, &s.in);
        at::Tensor ws = s.bytes(need);
        void *st = stream(Py_None);
        return WITHOUT_GIL(lasad_backward_layer(s.q.data_ptr(), z, v, d_out.data_ptr(), g[0].data_ptr(), g[1].data_ptr(), g[2].data_ptr(),
                                                g[3].defined() ? (float *)g[3].data_ptr() : nullptr, &s.in, &lo, &lg, s.io, s.io, s.B, s.Hh, s.d, gh,
                                                gw, start, s.n, mode, scale, w, eps, ws.data_ptr(), need, st));
    });
}

PyMethodDef methods[] = {
    {"decode_step", (PyCFunction)(void (*)(void))decode_step, METH_FASTCALL, nullptr},
    {"decode_step_gated", (PyCFunction)(void (*)(void))decode_step_gated, METH_FASTCALL, nullptr},
    {"decode_step_layer", (PyCFunction)(void (*)(void))decode_step_layer, METH_FASTCALL, nullptr},
    {"decode_step_rows", (PyCFunction)(void (*)(void))decode_step_rows, METH_FASTCALL, nullptr},
    {"forward_chunked", (PyCFunction)(void (*)(void))forward_chunked, METH_FASTCALL, nullptr},
    {"forward_gated", (PyCFunction)(void (*)(void))forward_gated, METH_FASTCALL, nullptr},
    {"forward_layer", (PyCFunction)(void (*)(void))forward_layer, METH_FASTCALL, nullptr},
    {"backward_chunked", (PyCFunction)(void (*)(void))backward_chunked, METH_FASTCALL, nullptr},
    {"backward_gated", (PyCFunction)(void (*)(void))backward_gated, METH_FASTCALL, nullptr},
    {"backward_layer", (PyCFunction)(void (*)(void))backward_layer, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_steps", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__steps() { return PyModule_Create(&module); }
