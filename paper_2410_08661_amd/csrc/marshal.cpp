// The calls a training or decode loop makes, from torch tensors to libqeft's C functions without the interpreter in between:
// binding.py's functions pass their arguments here first.  The smallest calls are bound by the host: one row through a 512 x 512 layer took
// 5.9 us with ctypes (a struct of four pointers, ten conversions, two lookups of the stream), of which a bare launch of an empty kernel with as many
// arguments is 3.8; it takes 4.0 now, 0.25 of them here.  A group call 5.1 -> 3.9.
//
// Only plain cases are taken: exact tensors on one GPU, the current one, and this package's own argument objects.  Anything else - a subclass,
// host memory, a missing output - makes the functions return None, and binding.py goes the way it describes itself.  Nothing is kept
// between calls: pointers, pitches and the stream are read off the objects each time.  The interpreter's lock is released around the C call.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include "qeft.h"

namespace {

struct Fns {
    decltype(&qeft_linear_fwd) fwd;
    decltype(&qeft_linear_fwd_group) fwd_group;
    decltype(&qeft_linear_bwd_dx) bwd_dx;
    decltype(&qeft_linear_bwd) bwd;
    decltype(&qeft_linear_fwd_irregular) fwd_irregular;
    decltype(&qeft_linear_bwd_dx_irregular) bwd_dx_irregular;
    decltype(&qeft_weak_grad) weak_grad;
} fns;
PyTypeObject *desc_type, *weight_type;
PyObject *n_desc, *n_qweight, *n_scales, *n_zeros, *n_weak;

// the bytes of a ctypes object (which owns them for its lifetime)
template <class T>
const T* bytes_of(PyObject* o) {
    Py_buffer b;
    if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) != 0) {
        PyErr_Clear();
        return nullptr;
    }
    const T* p = b.len >= (Py_ssize_t)sizeof(T) ? (const T*)b.buf : nullptr;
    PyBuffer_Release(&b);
    return p;
}

struct Call {
    int device = -1;
    bool ok = true;
    const at::Tensor* tensor(PyObject* o) {
        if (!ok || !THPVariable_CheckExact(o)) {
            ok = false;
            return nullptr;
        }
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.defined() || !t.is_cuda()) ok = false;
        else if (device < 0) device = t.get_device();
        else if (device != t.get_device()) ok = false;
        return ok ? &t : nullptr;
    }
    void* ptr(PyObject* o) {
        const at::Tensor* t = tensor(o);
        return t ? t->data_ptr() : nullptr;
    }
    void* matrix(PyObject* o, int64_t& rows, int64_t& pitch) {
        const at::Tensor* t = tensor(o);
        if (!t || t->dim() != 2) {
            ok = false;
            return nullptr;
        }
        rows = t->size(0);
        pitch = t->stride(0);
        return t->data_ptr();
    }
    void* workspace(PyObject* o, size_t& n) {   // None: none
        n = 0;
        if (o == Py_None) return nullptr;
        const at::Tensor* t = tensor(o);
        if (!t) return nullptr;
        n = (size_t)t->numel();
        return t->data_ptr();
    }
    int number(PyObject* o) {
        const long v = PyLong_AsLong(o);
        if (v == -1 && PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        return (int)v;
    }
    const qeft_desc_t* desc(PyObject* o) {
        const qeft_desc_t* d = Py_TYPE(o) == desc_type ? bytes_of<qeft_desc_t>(o) : nullptr;
        if (!d) ok = false;
        return d;
    }
    void weight(PyObject* o, qeft_weight_t& w) {
        w = {};
        if (!ok || Py_TYPE(o) != weight_type) {
            ok = false;
            return;
        }
        PyObject* own = PyObject_GetAttr(o, n_desc);
        const qeft_desc_t* d = own ? desc(own) : nullptr;
        auto take = [&](PyObject* name) -> void* {
            PyObject* t = ok ? PyObject_GetAttr(o, name) : nullptr;
            if (!t) {
                ok = false;
                return nullptr;
            }
            void* p = ptr(t);
            Py_DECREF(t);
            return p;
        };
        if (d && d->in_features > d->n_weak) {
            w.qweight = (decltype(w.qweight))take(n_qweight);
            w.scales = (decltype(w.scales))take(n_scales);
            w.zeros = (decltype(w.zeros))take(n_zeros);
        }
        if (d && d->n_weak > 0) w.weak = (decltype(w.weak))take(n_weak);
        if (!d) ok = false;
        Py_XDECREF(own);
        if (PyErr_Occurred()) PyErr_Clear();
    }
    // the current stream, if the tensors' GPU is the current one (binding.py takes the current GPU's)
    void* stream() {
        if (!ok || device < 0 || c10::hip::current_device() != device) {
            ok = false;
            return nullptr;
        }
        return c10::hip::getCurrentHIPStream((c10::DeviceIndex)device).stream();
    }
};

// Runs f(call) with torch's exceptions as Python's; f returns false where the call is not a plain one.
template <class F>
PyObject* guarded(F&& f) {
    int status = 0;
    try {
        Call c;
        if (!f(c, status)) Py_RETURN_NONE;
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    return PyLong_FromLong(status);
}
template <class F>
int unlocked(F&& f) {
    PyThreadState* s = PyEval_SaveThread();
    const int st = f();
    PyEval_RestoreThread(s);
    return st;
}

// (desc, w, X, Y, ws)
PyObject* linear_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Call& c, int& st) {
        if (n != 5) return false;
        const qeft_desc_t* d = c.desc(a[0]);
        qeft_weight_t w;
        c.weight(a[1], w);
        if (!c.ok) return false;
        int64_t M, ldx, my, ldy;
        size_t nws;
        const void* x = c.matrix(a[2], M, ldx);
        void* y = c.matrix(a[3], my, ldy);
        void* ws = c.workspace(a[4], nws);
        void* s = c.stream();
        if (!c.ok) return false;
        if (!M) ldx = d->in_features, ldy = d->out_features;   // (an empty matrix's pitch says nothing)
        st = unlocked([&] { return fns.fwd(d, &w, x, M, ldx, y, ldy, ws, nws, s); });
        return true;
    });
}
// (n, descs, weights, X, ys, ldys): the arrays of a Group
PyObject* linear_fwd_group(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Call& c, int& st) {
        if (n != 6) return false;
        const int layers = c.number(a[0]);
        const qeft_desc_t* d = bytes_of<qeft_desc_t>(a[1]);
        const qeft_weight_t* w = bytes_of<qeft_weight_t>(a[2]);
        void* const* ys = bytes_of<void*>(a[4]);
        const int64_t* ldy = bytes_of<int64_t>(a[5]);
        int64_t M, ldx;
        const void* x = c.matrix(a[3], M, ldx);
        void* s = c.stream();
        if (!c.ok || !d || !w || !ys || !ldy) return false;
        if (!M) ldx = d->in_features;
        st = unlocked([&] { return fns.fwd_group(layers, d, w, x, M, ldx, ys, ldy, s); });
        return true;
    });
}
// (desc, w, dY, dX, ws)
PyObject* linear_bwd_dx(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Call& c, int& st) {
        if (n != 5) return false;
        const qeft_desc_t* d = c.desc(a[0]);
        qeft_weight_t w;
        c.weight(a[1], w);
        if (!c.ok) return false;
        int64_t M, ldy, mx, ldx;
        size_t nws;
        const void* y = c.matrix(a[2], M, ldy);
        void* x = c.matrix(a[3], mx, ldx);
        void* ws = c.workspace(a[4], nws);
        void* s = c.stream();
        if (!c.ok) return false;
        if (!M) ldy = d->out_features, ldx = d->in_features;
        st = unlocked([&] { return fns.bwd_dx(d, &w, y, M, ldy, x, ldx, ws, nws, s); });
        return true;
    });
}
// (desc, w, perm, X or dY, Y or dX, ws)
template <bool FWD>
PyObject* irregular(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Call& c, int& st) {
        if (n != 6) return false;
        const qeft_desc_t* d = c.desc(a[0]);
        qeft_weight_t w;
        c.weight(a[1], w);
        if (!c.ok) return false;
        const int32_t* perm = (const int32_t*)c.ptr(a[2]);
        int64_t M, ldi, mo, ldo;
        size_t nws;
        const void* in = c.matrix(a[3], M, ldi);
        void* out = c.matrix(a[4], mo, ldo);
        void* ws = c.workspace(a[5], nws);
        void* s = c.stream();
        if (!c.ok) return false;
        if (!M) ldi = FWD ? d->in_features : d->out_features, ldo = FWD ? d->out_features : d->in_features;
        st = unlocked([&] { return (FWD ? fns.fwd_irregular : fns.bwd_dx_irregular)(d, &w, perm, in, M, ldi, out, ldo, ws, nws, s); });
        return true;
    });
}
// (desc, dY, Xw, dW, dtype, accumulate, ws)
PyObject* weak_grad(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Call& c, int& st) {
        if (n != 7) return false;
        const qeft_desc_t* d = c.desc(a[0]);
        if (!c.ok) return false;
        int64_t M, ldy, mx, ldx;
        size_t nws;
        const void* y = c.matrix(a[1], M, ldy);
        const void* x = c.matrix(a[2], mx, ldx);
        void* dw = c.ptr(a[3]);
        const int dtype = c.number(a[4]), accumulate = c.number(a[5]);
        void* ws = c.workspace(a[6], nws);
        void* s = c.stream();
        if (!c.ok || mx != M) return false;
        if (!M) ldy = d->out_features, ldx = d->n_weak > 8 ? d->n_weak : 8;
        st = unlocked([&] { return fns.weak_grad(d, y, M, ldy, x, ldx, dw, dtype, accumulate, ws, nws, s); });
        return true;
    });
}
// (desc, w, dY, dX, Xw, dW, dtype, accumulate, ws)
PyObject* linear_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&](Call& c, int& st) {
        if (n != 9) return false;
        const qeft_desc_t* d = c.desc(a[0]);
        qeft_weight_t w;
        c.weight(a[1], w);
        if (!c.ok) return false;
        int64_t M, ldy, mx, ldx, mw, ldw;
        size_t nws;
        const void* y = c.matrix(a[2], M, ldy);
        void* x = c.matrix(a[3], mx, ldx);
        const void* xw = c.matrix(a[4], mw, ldw);
        void* dw = c.ptr(a[5]);
        const int dtype = c.number(a[6]), accumulate = c.number(a[7]);
        void* ws = c.workspace(a[8], nws);
        void* s = c.stream();
        if (!c.ok || mw != M) return false;
        if (!M) ldy = d->out_features, ldx = d->in_features, ldw = d->n_weak > 8 ? d->n_weak : 8;
        st = unlocked([&] { return fns.bwd(d, &w, y, M, ldy, x, ldx, xw, ldw, dw, dtype, accumulate, ws, nws, s); });
        return true;
    });
}
// (addresses of the seven C functions in the order of Fns, qeft_desc_t, Weight)
PyObject* init(PyObject*, PyObject* args) {
    unsigned long long f[7];
    PyObject *d, *w;
    if (!PyArg_ParseTuple(args, "(KKKKKKK)O!O!", f, f + 1, f + 2, f + 3, f + 4, f + 5, f + 6, &PyType_Type, &d, &PyType_Type, &w)) return nullptr;
    fns = {(decltype(fns.fwd))f[0], (decltype(fns.fwd_group))f[1], (decltype(fns.bwd_dx))f[2], (decltype(fns.bwd))f[3],
           (decltype(fns.fwd_irregular))f[4], (decltype(fns.bwd_dx_irregular))f[5], (decltype(fns.weak_grad))f[6]};
    Py_INCREF(d);
    Py_INCREF(w);
    desc_type = (PyTypeObject*)d;
    weight_type = (PyTypeObject*)w;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"init", init, METH_VARARGS, nullptr},
    {"linear_fwd", (PyCFunction)(void (*)())linear_fwd, METH_FASTCALL, nullptr},
    {"linear_fwd_group", (PyCFunction)(void (*)())linear_fwd_group, METH_FASTCALL, nullptr},
    {"linear_bwd_dx", (PyCFunction)(void (*)())linear_bwd_dx, METH_FASTCALL, nullptr},
    {"linear_fwd_irregular", (PyCFunction)(void (*)())irregular<true>, METH_FASTCALL, nullptr},
    {"linear_bwd_dx_irregular", (PyCFunction)(void (*)())irregular<false>, METH_FASTCALL, nullptr},
    {"weak_grad", (PyCFunction)(void (*)())weak_grad, METH_FASTCALL, nullptr},
    {"linear_bwd", (PyCFunction)(void (*)())linear_bwd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
    n_desc = PyUnicode_InternFromString("desc");
    n_qweight = PyUnicode_InternFromString("qweight");
    n_scales = PyUnicode_InternFromString("scales");
    n_zeros = PyUnicode_InternFromString("zeros");
    n_weak = PyUnicode_InternFromString("weak");
    return PyModule_Create(&module);
}
