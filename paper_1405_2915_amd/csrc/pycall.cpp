// _skelcall: the Python binding's skeleton calls without ctypes.
//
// A skeleton call on 2^20 elements runs for 3 to 6 us on the GPU, and the host
// issues it in about 3 us through the C ABI; marshalling its arguments in Python
// and ctypes added 2 us (5 for the 2D maps, whose weight arrays went through
// numpy), which made short sequences of calls host-bound.  Each function here
// takes the arguments of the Python wrapper of the same name in order, converts
// the plain ones (containers, numbers, contiguous float32 weight arrays) and calls
// the C entry point with the GIL released.  It returns the status, or None when
// an argument is of any other kind: the wrapper then takes its general path,
// which converts or rejects it.  The entry points come from the library that the
// binding loaded (bind()), so this module links to none.
// Measured: the four calls of the small configuration on 2^20 elements 20.3 -> 17.2
// us (now the GPU's time), a 5-point map and its transpose on 24 fields of 121 x
// 163 14.5 -> 9.5 us.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <type_traits>

#include "skel.h"

namespace {

decltype(&skel_map) f_map;
decltype(&skel_reduce) f_reduce;
decltype(&skel_mapreduce) f_mapreduce;
decltype(&skel_mapoverlap1d) f_ov1;
decltype(&skel_mapoverlap1d_backward) f_ov1b;
decltype(&skel_mapoverlap2d_fields) f_ov2;
decltype(&skel_mapoverlap2d_fields_backward) f_ov2b;
decltype(&skel_scan) f_scan;
decltype(&skel_scan_rows) f_scan_rows;
decltype(&skel_reduce_segments) f_segments;
PyTypeObject* g_container;     // the binding's Container class
PyObject* g_current_stream;    // callable: the current stream as an integer
PyObject* s_handle;

constexpr int kMax = 8;  // operands or parameters of one call

// The converters return false for an argument that is not plain; an error of a
// conversion is dropped, since the general path raises its own.  An exception from
// the query of the current stream (an interrupt, say) stays set and is raised.

bool plain_int(PyObject* o, int64_t* v) {
    if (!PyLong_Check(o)) return false;
    *v = PyLong_AsLongLong(o);
    if (*v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool plain_int(PyObject* o, int* v) {
    int64_t x;
    if (!plain_int(o, &x) || x < INT32_MIN || x > INT32_MAX) return false;
    *v = (int)x;
    return true;
}

bool plain_double(PyObject* o, double* v) {
    if (PyFloat_CheckExact(o)) {
        *v = PyFloat_AS_DOUBLE(o);
        return true;
    }
    if (!PyLong_CheckExact(o)) return false;
    *v = PyLong_AsDouble(o);
    if (*v == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

bool container(PyObject* o, skel_container** c) {
    if (Py_TYPE(o) != g_container) return false;
    PyObject* h = PyObject_GetAttr(o, s_handle);
    if (!h) {
        PyErr_Clear();
        return false;
    }
    const bool ok = PyLong_CheckExact(h);
    *c = ok ? static_cast<skel_container*>(PyLong_AsVoidPtr(h)) : nullptr;
    Py_DECREF(h);
    if (PyErr_Occurred()) PyErr_Clear();
    return ok && *c;
}

bool containers(PyObject* o, skel_container* (&c)[kMax], int* n) {
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(o);
    if (k > kMax) return false;
    for (Py_ssize_t i = 0; i < k; ++i)
        if (!container(PySequence_Fast_GET_ITEM(o, i), &c[i])) return false;
    *n = (int)k;
    return true;
}

bool parameters(PyObject* o, double (&p)[kMax], int* n) {
    *n = 0;
    if (o == Py_None) return true;
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(o);
    if (k > kMax) return false;
    for (Py_ssize_t i = 0; i < k; ++i)
        if (!plain_double(PySequence_Fast_GET_ITEM(o, i), &p[i])) return false;
    *n = (int)k;
    return true;
}

bool stream_of(PyObject* o, void** s) {
    if (o != Py_None) {
        if (!PyLong_CheckExact(o)) return false;
        *s = PyLong_AsVoidPtr(o);
    } else {
        PyObject* v = PyObject_CallNoArgs(g_current_stream);
        if (!v) return false;
        const bool ok = PyLong_Check(v);
        *s = ok ? PyLong_AsVoidPtr(v) : nullptr;
        Py_DECREF(v);
        if (!ok) return false;
    }
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

// a C-contiguous float32 array, held for the duration of the call
struct Weights {
    Py_buffer b;
    bool held = false;
    ~Weights() {
        if (held) PyBuffer_Release(&b);
    }
    bool take(PyObject* o) {
        if (PyObject_GetBuffer(o, &b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
            PyErr_Clear();
            return false;
        }
        held = true;
        return b.format && b.format[0] == 'f' && b.format[1] == 0 && b.itemsize == 4;
    }
    const float* data() const { return held ? static_cast<const float*>(b.buf) : nullptr; }
    int64_t count() const { return b.len / 4; }
};

// the 2D weights and radii of _weights_2d's plain cases
struct Weights2 {
    Weights w2d, wy, wx;
    int ry = 0, rx = 0;
    bool take(PyObject* o2, PyObject* oy, PyObject* ox, PyObject* ory, PyObject* orx) {
        if (o2 != Py_None) {
            if (oy != Py_None || ox != Py_None || !w2d.take(o2)) return false;
            if (ory == Py_None || orx == Py_None) {
                if (w2d.b.ndim != 2) return false;
                ry = (int)((w2d.b.shape[0] - 1) / 2);
                rx = (int)((w2d.b.shape[1] - 1) / 2);
            }
            if (ory != Py_None && !plain_int(ory, &ry)) return false;
            if (orx != Py_None && !plain_int(orx, &rx)) return false;
            return w2d.count() == (2 * (int64_t)ry + 1) * (2 * (int64_t)rx + 1);
        }
        if (oy == Py_None || ox == Py_None || !wy.take(oy) || !wx.take(ox)) return false;
        ry = (int)((wy.count() - 1) / 2);
        rx = (int)((wx.count() - 1) / 2);
        if (ory != Py_None && !plain_int(ory, &ry)) return false;
        if (orx != Py_None && !plain_int(orx, &rx)) return false;
        return wy.count() == 2 * (int64_t)ry + 1 && wx.count() == 2 * (int64_t)rx + 1;
    }
};

template <class F>
PyObject* enter(F&& call) {
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

#define SKEL_PY(name, args) \
    PyObject* name(PyObject*, PyObject* const* a, Py_ssize_t n) { \
        if (n != (args)) { \
            PyErr_SetString(PyExc_TypeError, #name ": wrong number of arguments"); \
            return nullptr; \
        }
#define SKEL_PLAIN(cond) \
    if (!(cond)) { \
        if (PyErr_Occurred()) return nullptr; \
        Py_RETURN_NONE; \
    }

// (op, params, ins, out, variant, stream)
SKEL_PY(py_map, 6)
    int op, np, ni, variant;
    double p[kMax];
    skel_container *in[kMax], *out;
    void* s;
    SKEL_PLAIN(plain_int(a[0], &op) && parameters(a[1], p, &np) && containers(a[2], in, &ni) &&
               container(a[3], &out) && plain_int(a[4], &variant) && stream_of(a[5], &s));
    return enter([&] {
        return (int)f_map((skel_map_op)op, np ? p : nullptr, np, in, ni, out, variant, s);
    });
}

// (op, in, out, variant, stream)
SKEL_PY(py_reduce, 5)
    int op, variant;
    skel_container *in, *out;
    void* s;
    SKEL_PLAIN(plain_int(a[0], &op) && container(a[1], &in) && container(a[2], &out) &&
               plain_int(a[3], &variant) && stream_of(a[4], &s));
    return enter([&] { return (int)f_reduce((skel_reduce_op)op, in, out, variant, s); });
}

// (map_op, params, ins, op, out, variant, stream)
SKEL_PY(py_mapreduce, 7)
    int mop, np, ni, op, variant;
    double p[kMax];
    skel_container *in[kMax], *out;
    void* s;
    SKEL_PLAIN(plain_int(a[0], &mop) && parameters(a[1], p, &np) && containers(a[2], in, &ni) &&
               plain_int(a[3], &op) && container(a[4], &out) && plain_int(a[5], &variant) &&
               stream_of(a[6], &s));
    return enter([&] {
        return (int)f_mapreduce((skel_map_op)mop, np ? p : nullptr, np, in, ni,
                                (skel_reduce_op)op, out, variant, s);
    });
}

// (in, out, w, radius, edge, pad, variant, stream)
SKEL_PY(py_mapoverlap1d, 8)
    int r, edge, variant;
    double pad;
    skel_container *in, *out;
    Weights w;
    void* s;
    SKEL_PLAIN(container(a[0], &in) && container(a[1], &out) && plain_int(a[3], &r) &&
               plain_int(a[4], &edge) && plain_double(a[5], &pad) && plain_int(a[6], &variant) &&
               w.take(a[2]) && w.count() == 2 * (int64_t)r + 1 && stream_of(a[7], &s));
    return enter([&] {
        return (int)f_ov1(in, out, w.data(), r, (skel_edge)edge, (float)pad, variant, s);
    });
}

// (g, grad_in, w, radius, edge, variant, stream)
SKEL_PY(py_mapoverlap1d_backward, 7)
    int r, edge, variant;
    skel_container *g, *gi;
    Weights w;
    void* s;
    SKEL_PLAIN(container(a[0], &g) && container(a[1], &gi) && plain_int(a[3], &r) &&
               plain_int(a[4], &edge) && plain_int(a[5], &variant) && w.take(a[2]) &&
               w.count() == 2 * (int64_t)r + 1 && stream_of(a[6], &s));
    return enter([&] { return (int)f_ov1b(g, gi, w.data(), r, (skel_edge)edge, variant, s); });
}

// (in, out, fields, w2d, wy, wx, ry, rx, edge, pad, variant, stream)
SKEL_PY(py_mapoverlap2d_fields, 12)
    int edge, variant;
    int64_t fields;
    double pad;
    skel_container *in, *out;
    Weights2 w;
    void* s;
    SKEL_PLAIN(container(a[0], &in) && container(a[1], &out) && plain_int(a[2], &fields) &&
               plain_int(a[8], &edge) && plain_double(a[9], &pad) && plain_int(a[10], &variant) &&
               w.take(a[3], a[4], a[5], a[6], a[7]) && stream_of(a[11], &s));
    return enter([&] {
        return (int)f_ov2(in, out, fields, w.w2d.data(), w.wy.data(), w.wx.data(), w.ry, w.rx,
                          (skel_edge)edge, (float)pad, variant, s);
    });
}

// (g, grad_in, fields, w2d, wy, wx, ry, rx, edge, variant, stream)
SKEL_PY(py_mapoverlap2d_fields_backward, 11)
    int edge, variant;
    int64_t fields;
    skel_container *g, *gi;
    Weights2 w;
    void* s;
    SKEL_PLAIN(container(a[0], &g) && container(a[1], &gi) && plain_int(a[2], &fields) &&
               plain_int(a[8], &edge) && plain_int(a[9], &variant) &&
               w.take(a[3], a[4], a[5], a[6], a[7]) && stream_of(a[10], &s));
    return enter([&] {
        return (int)f_ov2b(g, gi, fields, w.w2d.data(), w.wy.data(), w.wx.data(), w.ry, w.rx,
                           (skel_edge)edge, variant, s);
    });
}

// (in, out, kind, op, variant, stream)
template <class F>
PyObject* scan_call(F f, PyObject* const* a) {
    int kind, op, variant;
    skel_container *in, *out;
    void* s;
    SKEL_PLAIN(container(a[0], &in) && container(a[1], &out) && plain_int(a[2], &kind) &&
               plain_int(a[3], &op) && plain_int(a[4], &variant) && stream_of(a[5], &s));
    return enter([&] {
        return (int)f(in, out, (skel_scan_kind)kind, (skel_reduce_op)op, variant, s);
    });
}
SKEL_PY(py_scan, 6)
    return scan_call(f_scan, a);
}
SKEL_PY(py_scan_rows, 6)
    return scan_call(f_scan_rows, a);
}

// (op, in, offsets, out, variant, stream)
SKEL_PY(py_reduce_segments, 6)
    int op, variant;
    skel_container *in, *off, *out;
    void* s;
    SKEL_PLAIN(plain_int(a[0], &op) && container(a[1], &in) && container(a[2], &off) &&
               container(a[3], &out) && plain_int(a[4], &variant) && stream_of(a[5], &s));
    return enter([&] { return (int)f_segments((skel_reduce_op)op, in, off, out, variant, s); });
}

// bind(Container, current_stream, {name: address})
PyObject* py_bind(PyObject*, PyObject* args) {
    PyObject *cls, *cur, *addr;
    if (!PyArg_ParseTuple(args, "O!OO!", &PyType_Type, &cls, &cur, &PyDict_Type, &addr))
        return nullptr;
    const auto get = [&](const char* name, auto& f) {
        PyObject* v = PyDict_GetItemString(addr, name);
        void* p = v ? PyLong_AsVoidPtr(v) : nullptr;
        if (!p) {
            if (!PyErr_Occurred()) PyErr_Format(PyExc_KeyError, "no address of %s", name);
            return false;
        }
        f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(p);
        return true;
    };
    if (!get("skel_map", f_map) || !get("skel_reduce", f_reduce) ||
        !get("skel_mapreduce", f_mapreduce) || !get("skel_mapoverlap1d", f_ov1) ||
        !get("skel_mapoverlap1d_backward", f_ov1b) || !get("skel_mapoverlap2d_fields", f_ov2) ||
        !get("skel_mapoverlap2d_fields_backward", f_ov2b) || !get("skel_scan", f_scan) ||
        !get("skel_scan_rows", f_scan_rows) || !get("skel_reduce_segments", f_segments))
        return nullptr;
    Py_INCREF(cls);
    Py_XSETREF(g_container, reinterpret_cast<PyTypeObject*>(cls));
    Py_INCREF(cur);
    Py_XSETREF(g_current_stream, cur);
    Py_RETURN_NONE;
}

#define SKEL_FAST(name, fn) \
    {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(fn)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr},
    SKEL_FAST("map", py_map),
    SKEL_FAST("reduce", py_reduce),
    SKEL_FAST("mapreduce", py_mapreduce),
    SKEL_FAST("mapoverlap1d", py_mapoverlap1d),
    SKEL_FAST("mapoverlap1d_backward", py_mapoverlap1d_backward),
    SKEL_FAST("mapoverlap2d_fields", py_mapoverlap2d_fields),
    SKEL_FAST("mapoverlap2d_fields_backward", py_mapoverlap2d_fields_backward),
    SKEL_FAST("scan", py_scan),
    SKEL_FAST("scan_rows", py_scan_rows),
    SKEL_FAST("reduce_segments", py_reduce_segments),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_skelcall", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__skelcall(void) {
    s_handle = PyUnicode_InternFromString("handle");
    return s_handle ? PyModule_Create(&module) : nullptr;
}
