// cf_args.cpp -- the argument checks of the Python binding in native code
// (CPython module _cf_args, built beside libconvfirst.so).  A call passes a
// dozen tensors, and checking each one's type, shape, layout and device from
// Python takes longer than many of the kernels; here it is one pass over the
// parameter dict.  Host time of a block call: 21 -> 5 us on one CPU core; a
// block on one 14x14x64 image, whose kernel runs 10.6 us, from 15.7 to 10.6 us
// a call.  These functions only say yes: with anything other than what
// a call wants they return None, and the binding's own checks then raise the
// error that names it.  Nothing is remembered between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdint.h>

#include <string>
#include <vector>

namespace {

// One parameter: its key, whether it is a weight (x's dtype, required) or an
// fp32 vector (optional), and its shape as indices into the call's sizes.
struct Param {
    PyObject *key;  // interned
    bool weight;
    std::vector<int> dims;
};
typedef std::vector<Param> Spec;

constexpr const char *SPEC = "cf_args.spec";
constexpr int MAX_SIZES = 8;

Spec *spec_of(PyObject *o) { return static_cast<Spec *>(PyCapsule_GetPointer(o, SPEC)); }

void free_spec(PyObject *o) {
    Spec *s = spec_of(o);
    for (const Param &p : *s)
        Py_DECREF(p.key);
    delete s;
}

// spec(((key, weight, (size index, ..)), ..)) -> capsule
PyObject *make_spec(PyObject *, PyObject *arg) {
    PyObject *seq = PySequence_Fast(arg, "spec: a sequence of (key, weight, sizes)");
    if (!seq)
        return nullptr;
    Spec *s = new Spec;
    bool ok = true;
    for (Py_ssize_t i = 0; ok && i < PySequence_Fast_GET_SIZE(seq); i++) {
        PyObject *key = nullptr, *sizes = nullptr;
        int weight = 0;
        ok = PyArg_ParseTuple(PySequence_Fast_GET_ITEM(seq, i), "UpO!", &key, &weight, &PyTuple_Type, &sizes);
        if (!ok)
            break;
        Param p{key, weight != 0, {}};
        for (Py_ssize_t d = 0; ok && d < PyTuple_GET_SIZE(sizes); d++) {
            const long v = PyLong_AsLong(PyTuple_GET_ITEM(sizes, d));
            ok = v >= 0 && v < MAX_SIZES;
            p.dims.push_back((int)v);
        }
        Py_INCREF(key);
        PyUnicode_InternInPlace(&key);
        p.key = key;
        s->push_back(p);
    }
    Py_DECREF(seq);
    PyObject *c = ok ? PyCapsule_New(s, SPEC, free_spec) : nullptr;
    if (!c) {
        for (const Param &p : *s)
            Py_DECREF(p.key);
        delete s;
        if (!PyErr_Occurred())
            PyErr_SetString(PyExc_ValueError, "spec: size index out of range");
    }
    return c;
}

// A strided GPU tensor whose memory the library can use as it is.  Callers let
// only torch.Tensor and Parameter themselves through, no other subclass.
bool plain(const at::Tensor &t) {
    return t.defined() && t.layout() == at::kStrided && t.is_cuda() && t.is_contiguous() && !t.is_conj() && !t.is_neg();
}

// tensor4(x) -> (N, H, W, C, dtype code, address) of a contiguous 4-D fp16 or
// bf16 GPU tensor, else None
PyObject *tensor4(PyObject *, PyObject *o) {
    if (!THPVariable_CheckExact(o))
        Py_RETURN_NONE;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!plain(t) || t.dim() != 4 || (t.scalar_type() != at::kHalf && t.scalar_type() != at::kBFloat16))
        Py_RETURN_NONE;
    return Py_BuildValue("LLLLiK", (long long)t.size(0), (long long)t.size(1), (long long)t.size(2),
                         (long long)t.size(3), t.scalar_type() == at::kHalf ? 0 : 1,
                         (unsigned long long)(uintptr_t)t.data_ptr());
}

// like(x, t, shape) -> address of t when it has x's dtype and device and this
// shape, contiguous, else None
PyObject *like(PyObject *, PyObject *args) {
    PyObject *xo, *to, *shape;
    if (!PyArg_ParseTuple(args, "OOO!", &xo, &to, &PyTuple_Type, &shape))
        return nullptr;
    if (!THPVariable_CheckExact(xo) || !THPVariable_CheckExact(to))
        Py_RETURN_NONE;
    const at::Tensor &x = THPVariable_Unpack(xo), &t = THPVariable_Unpack(to);
    if (!plain(t) || t.scalar_type() != x.scalar_type() || t.device() != x.device() ||
        t.dim() != PyTuple_GET_SIZE(shape))
        Py_RETURN_NONE;
    for (int64_t d = 0; d < t.dim(); d++) {
        const long long v = PyLong_AsLongLong(PyTuple_GET_ITEM(shape, d));
        if (v != t.size(d)) {
            PyErr_Clear();
            Py_RETURN_NONE;
        }
    }
    return PyLong_FromUnsignedLongLong((unsigned long long)(uintptr_t)t.data_ptr());
}

// shape(p, key) -> shape of the tensor p[key], else None
PyObject *shape(PyObject *, PyObject *args) {
    PyObject *p, *key;
    if (!PyArg_ParseTuple(args, "OO", &p, &key))
        return nullptr;
    PyObject *o = PyDict_CheckExact(p) ? PyDict_GetItem(p, key) : nullptr;
    if (!o || !THPVariable_CheckExact(o))
        Py_RETURN_NONE;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined())
        Py_RETURN_NONE;
    PyObject *r = PyTuple_New(t.dim());
    for (int64_t d = 0; r && d < t.dim(); d++)
        PyTuple_SET_ITEM(r, d, PyLong_FromLongLong(t.size(d)));
    return r;
}

// collect(spec, x, p, sizes) -> the parameters' addresses as the bytes of the
// C struct, when p holds exactly what the spec says for these sizes, in x's
// dtype (weights) or fp32, contiguous and on x's device; else None
PyObject *collect(PyObject *, PyObject *args) {
    PyObject *so, *xo, *p, *sizes;
    if (!PyArg_ParseTuple(args, "OOOO!", &so, &xo, &p, &PyTuple_Type, &sizes))
        return nullptr;
    Spec *spec = spec_of(so);
    if (!spec)
        return nullptr;
    if (!THPVariable_CheckExact(xo) || !PyDict_CheckExact(p) || PyTuple_GET_SIZE(sizes) > MAX_SIZES)
        Py_RETURN_NONE;
    const at::Tensor &x = THPVariable_Unpack(xo);
    long long sz[MAX_SIZES] = {0};
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(sizes); i++)
        sz[i] = PyLong_AsLongLong(PyTuple_GET_ITEM(sizes, i));
    if (PyErr_Occurred())
        return nullptr;
    uint64_t out[32] = {0};
    Py_ssize_t seen = 0;
    if (spec->size() > 32)
        Py_RETURN_NONE;
    for (size_t i = 0; i < spec->size(); i++) {
        const Param &q = (*spec)[i];
        PyObject *o = PyDict_GetItem(p, q.key);
        if (o)
            seen++;
        if (!o || o == Py_None) {
            if (q.weight)
                Py_RETURN_NONE;
            continue;
        }
        if (!THPVariable_CheckExact(o))
            Py_RETURN_NONE;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!plain(t) || t.device() != x.device() || t.scalar_type() != (q.weight ? x.scalar_type() : at::kFloat) ||
            t.dim() != (int64_t)q.dims.size())
            Py_RETURN_NONE;
        for (size_t d = 0; d < q.dims.size(); d++)
            if (t.size(d) != sz[q.dims[d]])
                Py_RETURN_NONE;
        out[i] = (uint64_t)(uintptr_t)t.data_ptr();
    }
    if (seen != PyDict_GET_SIZE(p))
        Py_RETURN_NONE;  // a key that is none of the spec's
    return PyBytes_FromStringAndSize(reinterpret_cast<const char *>(out), (Py_ssize_t)(8 * spec->size()));
}

// C++ exceptions (a tensor without storage, say) end here: the binding's own
// checks take over
template <PyObject *(*F)(PyObject *, PyObject *)>
PyObject *guarded(PyObject *self, PyObject *arg) {
    try {
        return F(self, arg);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

PyMethodDef methods[] = {{"spec", guarded<make_spec>, METH_O, nullptr},
                         {"tensor4", guarded<tensor4>, METH_O, nullptr},
                         {"like", guarded<like>, METH_VARARGS, nullptr},
                         {"shape", guarded<shape>, METH_VARARGS, nullptr},
                         {"collect", guarded<collect>, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_cf_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__cf_args() { return PyModule_Create(&module); }
