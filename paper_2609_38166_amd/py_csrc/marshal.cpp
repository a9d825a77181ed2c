// Argument marshalling of the Python binding's per-token calls.
//
// A call made of regular arguments (an lq_dims, a binding.State, contiguous
// device tensors of the right type and size, the current stream) takes 15.7 us of
// host time when its 16 tensors are checked and unpacked from Python (7.7 us of
// it the checks), against 3 to 6 us for the kernel it launches on a small batch.
// The same checks here take 0.3 us, the call 4.0 (the C entry with its launch
// 3.9).  Anything else -- another type, raw addresses, a stream of the
// caller's, an argument that fails a check -- returns None before anything is
// enqueued, and the Python path takes the call: it accepts what it accepts and
// words what it refuses.  Nothing is kept from one call for the next.
#include <Python.h>

#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "leapquant.h"

namespace {

PyTypeObject *g_dims_type = nullptr, *g_state_type = nullptr;
PyObject *g_names[10];      // attribute names of the state buffers, in lq_state's order
int32_t (*g_state_bytes)(const lq_dims *, size_t *) = nullptr;

enum { ANY = -1 };

// The address of a contiguous device tensor of scalar type `type` (ANY: any)
// with at least `bytes` bytes; false for anything else.
bool tensor_ptr(PyObject *o, size_t bytes, int type, void **p) {
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return false;
    if (type != ANY && t.scalar_type() != static_cast<at::ScalarType>(type)) return false;
    if (t.nbytes() < bytes) return false;
    *p = t.data_ptr();
    return true;
}

struct Call {
    lq_dims dims;
    lq_state st;
    size_t tiles, ktiles, gate;
};

bool unpack(PyObject *dims, PyObject *state, Call &c) {
    if (Py_TYPE(dims) != g_dims_type || Py_TYPE(state) != g_state_type) return false;
    Py_buffer v;
    if (PyObject_GetBuffer(dims, &v, PyBUF_SIMPLE) != 0) return false;
    const bool whole = v.len == (Py_ssize_t)sizeof(lq_dims);
    if (whole) memcpy(&c.dims, v.buf, sizeof(lq_dims));
    PyBuffer_Release(&v);
    if (!whole) return false;
    size_t need[10];
    if (g_state_bytes(&c.dims, need) != LQ_OK) return false;
    void **field[10] = {&c.st.codes, (void **)&c.st.scale, (void **)&c.st.smooth, (void **)&c.st.comp_k,
                        (void **)&c.st.comp_u, (void **)&c.st.rec_k, (void **)&c.st.rec_u, (void **)&c.st.rec_a,
                        (void **)&c.st.rec_len, (void **)&c.st.err};
    for (int i = 0; i < 10; ++i) {
        PyObject *o = PyObject_GetAttr(state, g_names[i]);
        if (!o) return false;
        bool ok;
        if ((i == 3 || i == 4) && c.dims.n_comp == 0) {     // the tokens of a state without any: only addressed
            ok = THPVariable_CheckExact(o);
            if (ok) *field[i] = THPVariable_Unpack(o).data_ptr();
        } else {
            ok = tensor_ptr(o, need[i], ANY, field[i]);
        }
        Py_DECREF(o);                                       // (the state holds it)
        if (!ok) return false;
    }
    c.tiles = (size_t)c.dims.batch * c.dims.heads_v;
    c.ktiles = (size_t)c.dims.batch * c.dims.heads_k;
    c.gate = c.dims.gate == LQ_GATE_DIAG ? c.dims.d_k : 1;
    return true;
}

// Runs body, which enqueues on the current stream and sets `status`; None where
// it returns false or throws.
template <typename F>
PyObject *guarded(F body) {
    int32_t status = 0;
    bool ok = false;
    try {
        ok = body(status);
    } catch (...) {
    }
    if (!ok) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(status);
}

void *current_stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

constexpr int F32 = (int)at::ScalarType::Float;

// step(fn, dims, state, q, k, v, alpha, beta, o)
PyObject *step(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 9) Py_RETURN_NONE;
    return guarded([&](int32_t &status) {
        Call c;
        if (!unpack(a[1], a[2], c)) return false;
        const size_t vec = c.tiles * c.dims.d_v * 4, key = c.ktiles * c.dims.d_k * 4;
        const size_t need[6] = {key, key, vec, c.tiles * c.gate * 4, c.tiles * 4, vec};
        void *p[6];
        for (int i = 0; i < 6; ++i)
            if (!tensor_ptr(a[3 + i], need[i], F32, &p[i])) return false;
        using Fn = int32_t (*)(const lq_dims *, lq_state *, void *, void *, void *, void *, void *, void *, void *);
        const Fn fn = (Fn)PyLong_AsVoidPtr(a[0]);
        void *s = current_stream();
        Py_BEGIN_ALLOW_THREADS
        status = fn(&c.dims, &c.st, p[0], p[1], p[2], p[3], p[4], p[5], s);
        Py_END_ALLOW_THREADS
        return true;
    });
}

// step_general(fn, dims, state, q, k, b, v, alpha, beta, o)
PyObject *step_general(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 10) Py_RETURN_NONE;
    return guarded([&](int32_t &status) {
        Call c;
        if (!unpack(a[1], a[2], c)) return false;
        const size_t vec = c.tiles * c.dims.d_v * 4, key = c.ktiles * c.dims.d_k * 4;
        const size_t need[7] = {key, key, c.tiles * c.dims.d_k * 4, vec, c.tiles * c.gate * 4, c.tiles * 4, vec};
        void *p[7];
        for (int i = 0; i < 7; ++i)
            if (!tensor_ptr(a[3 + i], need[i], F32, &p[i])) return false;
        using Fn = int32_t (*)(const lq_dims *, lq_state *, void *, void *, void *, void *, void *, void *, void *, void *);
        const Fn fn = (Fn)PyLong_AsVoidPtr(a[0]);
        void *s = current_stream();
        Py_BEGIN_ALLOW_THREADS
        status = fn(&c.dims, &c.st, p[0], p[1], p[2], p[3], p[4], p[5], p[6], s);
        Py_END_ALLOW_THREADS
        return true;
    });
}

// commit(fn, dims, state, mask or None)
PyObject *commit(PyObject *, PyObject *const *a, Py_ssize_t n) {
    if (n != 4) Py_RETURN_NONE;
    return guarded([&](int32_t &status) {
        Call c;
        if (!unpack(a[1], a[2], c)) return false;
        void *mask = nullptr;
        if (a[3] != Py_None && !tensor_ptr(a[3], (size_t)c.dims.batch * 4, ANY, &mask)) return false;
        using Fn = int32_t (*)(const lq_dims *, lq_state *, void *, void *);
        const Fn fn = (Fn)PyLong_AsVoidPtr(a[0]);
        void *s = current_stream();
        Py_BEGIN_ALLOW_THREADS
        status = fn(&c.dims, &c.st, mask, s);
        Py_END_ALLOW_THREADS
        return true;
    });
}

// setup(lq_dims type, State type, field names, address of leapquant_state_bytes)
PyObject *setup(PyObject *, PyObject *args) {
    PyObject *dims, *state, *names, *fn;
    if (!PyArg_ParseTuple(args, "OOOO", &dims, &state, &names, &fn)) return nullptr;
    if (!PyType_Check(dims) || !PyType_Check(state) || !PyTuple_Check(names) || PyTuple_Size(names) != 10) {
        PyErr_SetString(PyExc_TypeError, "setup(type, type, ten names, address)");
        return nullptr;
    }
    void *addr = PyLong_AsVoidPtr(fn);
    if (!addr) return PyErr_Occurred() ? nullptr : (PyErr_SetString(PyExc_ValueError, "no address"), nullptr);
    for (int i = 0; i < 10; ++i) {
        PyObject *s = PyTuple_GetItem(names, i);
        Py_INCREF(s);
        PyUnicode_InternInPlace(&s);
        Py_XSETREF(g_names[i], s);
    }
    Py_INCREF(dims);
    Py_XSETREF(g_dims_type, (PyTypeObject *)dims);
    Py_INCREF(state);
    Py_XSETREF(g_state_type, (PyTypeObject *)state);
    g_state_bytes = (int32_t(*)(const lq_dims *, size_t *))addr;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"setup", setup, METH_VARARGS, "types, field names and leapquant_state_bytes of the binding"},
    {"step", (PyCFunction)(void (*)(void))step, METH_FASTCALL, "decode step: status, or None for the Python path"},
    {"step_general", (PyCFunction)(void (*)(void))step_general, METH_FASTCALL, "decode step with read vectors"},
    {"commit", (PyCFunction)(void (*)(void))commit, METH_FASTCALL, "window commit"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// (the binding uses the extension with the torch that it was built against only)
PyMODINIT_FUNC PyInit__marshal(void) {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", LQ_TORCH_VERSION) != 0) Py_CLEAR(m);
    return m;
}
