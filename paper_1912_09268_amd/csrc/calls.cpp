// CPython extension module: the device calls of Context (binding.py), argument conversion in native code.
//
// A device call enqueues a kernel and returns, and a training loop makes one per group or per tensor, so what the
// binding adds to each counts: ctypes took 0.85 us (pack_tensors) to 1.15 us (group_pipeline) beside the 2.5 us the
// HIP runtime needs for a launch; the conversions below take about 0.1 us.  The module has no link to the library:
// binding.py loads that through ctypes and hands over the addresses of its entry points.  Each device call of the class
// Context is a DeviceCall in front of the plain ctypes method; `_handle` of an instance is the address of the context, 0 after close().
//
// Conversions are those of the ctypes signatures: integers through int(), kept to 32 bits; addresses and streams
// from an int or None; floats through float().  The interpreter lock is released during a call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstddef>
#include <cstdint>
#include <cstring>

namespace {

enum Kind : char { I32, PTR, PTR_OR_NONE, F32 };      // PTR_OR_NONE: 0 counts as None
struct Arg { const char* name; Kind kind; };
struct Value { int32_t i; void* p; float f; };
constexpr int MAX_ARGS = 10;

struct Call { const char* fn; int n; Arg arg[MAX_ARGS]; };     // the last argument is the stream and may be left out
enum { PACK, PACK_TENSORS, REDUCE, UNPACK_UPDATE, REDUCE_UPDATE, GROUP_PIPELINE, DIRECT_UPDATE, GROUP_PIPELINE_SPAN,
       GROUP_PIPELINE_STATIC, N_CALLS };

#define GRADS {"d_grad_ptrs", PTR}
#define MERGE {"d_merge_bufs", PTR}
#define WEIGHTS {"d_w_ptrs", PTR}, {"d_v_ptrs", PTR}, {"lr", F32}, {"momentum", F32}
#define STREAM {"stream", PTR}
const Call CALLS[N_CALLS] = {
    {"mgwfbp_pack", 4, {{"group", I32}, GRADS, MERGE, STREAM}},
    {"mgwfbp_pack_tensors", 5, {{"first_tensor", I32}, {"last_tensor", I32}, GRADS, MERGE, STREAM}},
    {"mgwfbp_reduce", 4, {{"group", I32}, MERGE, {"d_reduced", PTR}, STREAM}},
    {"mgwfbp_unpack_update", 7, {{"group", I32}, {"d_reduced", PTR}, WEIGHTS, STREAM}},
    {"mgwfbp_reduce_update", 7, {{"group", I32}, MERGE, WEIGHTS, STREAM}},
    {"mgwfbp_group_pipeline", 9, {{"group", I32}, GRADS, MERGE, {"d_reduced", PTR_OR_NONE}, WEIGHTS, STREAM}},
    {"mgwfbp_direct_update", 8, {{"group", I32}, GRADS, {"d_reduced", PTR_OR_NONE}, WEIGHTS, STREAM}},
    {"mgwfbp_group_pipeline_span", 10,
     {{"group_first", I32}, {"group_count", I32}, GRADS, MERGE, {"d_reduced", PTR_OR_NONE}, WEIGHTS, STREAM}},
    {"mgwfbp_group_pipeline_static", 9, {{"group", I32}, GRADS, MERGE, {"d_reduced", PTR_OR_NONE}, WEIGHTS, STREAM}},
};

void* g_entry[N_CALLS];          // written by set_functions, under the interpreter lock
PyObject* g_raise = nullptr;     // binding._check
PyObject* g_handle = nullptr;    // "_handle"

bool convert(PyObject* o, Kind kind, Value& v) {
    if (kind == F32) {
        if (PyFloat_Check(o)) {
            v.f = static_cast<float>(PyFloat_AS_DOUBLE(o));
            return true;
        }
        PyObject* f = PyNumber_Float(o);
        if (f == nullptr) return false;
        v.f = static_cast<float>(PyFloat_AS_DOUBLE(f));
        Py_DECREF(f);
        return true;
    }
    if (kind == I32) {
        PyObject* n = PyLong_Check(o) ? (Py_INCREF(o), o) : PyNumber_Long(o);
        if (n == nullptr) return false;
        v.i = static_cast<int32_t>(static_cast<uint32_t>(PyLong_AsUnsignedLongLongMask(n)));
        Py_DECREF(n);
        return !PyErr_Occurred();
    }
    if (PyLong_Check(o)) {
        v.p = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o)));
        return v.p != nullptr || !PyErr_Occurred();
    }
    v.p = nullptr;
    if (o == Py_None) return true;
    if (kind == PTR_OR_NONE) {
        const int truth = PyObject_IsTrue(o);
        if (truth <= 0) return truth == 0;
    }
    PyErr_SetString(PyExc_TypeError, "cannot be converted to pointer");
    return false;
}

// Positional and keyword arguments into v[0 .. c.n).
bool parse(const Call& c, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, Value* v) {
    const Py_ssize_t nkw = kwnames == nullptr ? 0 : PyTuple_GET_SIZE(kwnames);
    if (nargs > c.n) {
        PyErr_Format(PyExc_TypeError, "%s() takes %d arguments but %zd were given", c.fn + 7, c.n, nargs);
        return false;
    }
    PyObject* got[MAX_ARGS] = {};
    for (Py_ssize_t i = 0; i < nargs; ++i) got[i] = args[i];
    for (Py_ssize_t k = 0; k < nkw; ++k) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, k);
        int at = 0;
        while (at < c.n && PyUnicode_CompareWithASCIIString(name, c.arg[at].name) != 0) ++at;
        if (at == c.n) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", c.fn + 7, name);
            return false;
        }
        if (got[at] != nullptr) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%U'", c.fn + 7, name);
            return false;
        }
        got[at] = args[nargs + k];
    }
    for (int i = 0; i < c.n; ++i) {
        if (got[i] == nullptr) {
            if (i + 1 == c.n) {
                v[i].p = nullptr;
                continue;
            }
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", c.fn + 7, c.arg[i].name);
            return false;
        }
        if (!convert(got[i], c.arg[i].kind, v[i])) return false;
    }
    return true;
}

// The entry points by shape: c = context, then the values in order.
int enter(int which, void* fn, void* c, const Value* v) {
    switch (which) {
        case PACK: return reinterpret_cast<int (*)(void*, int32_t, void*, void*, void*)>(fn)(c, v[0].i, v[1].p, v[2].p, v[3].p);
        case PACK_TENSORS:
            return reinterpret_cast<int (*)(void*, int32_t, int32_t, void*, void*, void*)>(fn)(c, v[0].i, v[1].i, v[2].p, v[3].p, v[4].p);
        case REDUCE: return reinterpret_cast<int (*)(void*, int32_t, void*, void*, void*)>(fn)(c, v[0].i, v[1].p, v[2].p, v[3].p);
        case UNPACK_UPDATE:
        case REDUCE_UPDATE:
            return reinterpret_cast<int (*)(void*, int32_t, void*, void*, void*, float, float, void*)>(fn)(
                c, v[0].i, v[1].p, v[2].p, v[3].p, v[4].f, v[5].f, v[6].p);
        case DIRECT_UPDATE:
            return reinterpret_cast<int (*)(void*, int32_t, void*, void*, void*, void*, float, float, void*)>(fn)(
                c, v[0].i, v[1].p, v[2].p, v[3].p, v[4].p, v[5].f, v[6].f, v[7].p);
        case GROUP_PIPELINE_SPAN:
            return reinterpret_cast<int (*)(void*, int32_t, int32_t, void*, void*, void*, void*, void*, float, float, void*)>(fn)(
                c, v[0].i, v[1].i, v[2].p, v[3].p, v[4].p, v[5].p, v[6].p, v[7].f, v[8].f, v[9].p);
        default:         // GROUP_PIPELINE, GROUP_PIPELINE_STATIC
            return reinterpret_cast<int (*)(void*, int32_t, void*, void*, void*, void*, void*, float, float, void*)>(fn)(
                c, v[0].i, v[1].p, v[2].p, v[3].p, v[4].p, v[5].p, v[6].f, v[7].f, v[8].p);
    }
}

// A device call as an attribute of the class: a function of its own, bound like one (the calls of an instance pass it as
// first argument, without a bound method in between).  Where the native way is not open -- the library not loaded yet, its
// entry point replaced -- the plain Python function it stands for is called instead.
struct DeviceCall {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    int which;
    PyObject* plain;
    PyObject* dict;           // what functools.update_wrapper sets: name, docstring, annotations, __wrapped__
};

PyObject* call(PyObject* callable, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
    const DeviceCall* self = reinterpret_cast<DeviceCall*>(callable);
    const int which = self->which;
    void* const fn = g_entry[which];
    const Py_ssize_t nargs = PyVectorcall_NARGS(nargsf);
    if (fn == nullptr || nargs == 0) return PyObject_Vectorcall(self->plain, args, nargsf, kwnames);
    Value v[MAX_ARGS];
    if (!parse(CALLS[which], args + 1, nargs - 1, kwnames, v)) return nullptr;
    PyObject* handle = PyObject_GetAttr(args[0], g_handle);
    if (handle == nullptr) return nullptr;
    const unsigned long long address = PyLong_AsUnsignedLongLongMask(handle);
    Py_DECREF(handle);
    if (address == static_cast<unsigned long long>(-1) && PyErr_Occurred()) return nullptr;
    void* const ctx = reinterpret_cast<void*>(static_cast<uintptr_t>(address));
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = enter(which, fn, ctx, v);
    Py_END_ALLOW_THREADS
    if (status == 0) Py_RETURN_NONE;
    return PyObject_CallFunction(g_raise, "si", CALLS[which].fn, status);     // raises
}

int call_index(const char* fn) {
    for (int i = 0; i < N_CALLS; ++i)
        if (std::strcmp(fn, CALLS[i].fn) == 0) return i;
    return -1;
}

// DeviceCall(name of the entry point, plain function)
PyObject* device_call_new(PyTypeObject* type, PyObject* args, PyObject* kwargs) {
    const char* fn;
    PyObject* plain;
    if (kwargs != nullptr && PyDict_GET_SIZE(kwargs) > 0) {
        PyErr_SetString(PyExc_TypeError, "DeviceCall() takes no keyword arguments");
        return nullptr;
    }
    if (!PyArg_ParseTuple(args, "sO", &fn, &plain)) return nullptr;
    const int which = call_index(fn);
    if (which < 0) {
        PyErr_Format(PyExc_KeyError, "%s", fn);
        return nullptr;
    }
    DeviceCall* self = reinterpret_cast<DeviceCall*>(type->tp_alloc(type, 0));
    if (self == nullptr) return nullptr;
    self->vectorcall = call;
    self->which = which;
    Py_INCREF(plain);
    self->plain = plain;
    return reinterpret_cast<PyObject*>(self);
}
int device_call_traverse(PyObject* o, visitproc visit, void* arg) {
    Py_VISIT(reinterpret_cast<DeviceCall*>(o)->plain);
    Py_VISIT(reinterpret_cast<DeviceCall*>(o)->dict);
    return 0;
}
int device_call_clear(PyObject* o) {
    Py_CLEAR(reinterpret_cast<DeviceCall*>(o)->plain);
    Py_CLEAR(reinterpret_cast<DeviceCall*>(o)->dict);
    return 0;
}
void device_call_dealloc(PyObject* o) {
    PyObject_GC_UnTrack(o);
    device_call_clear(o);
    Py_TYPE(o)->tp_free(o);
}
PyObject* device_call_get(PyObject* o, PyObject* obj, PyObject*) {
    if (obj == nullptr || obj == Py_None) {
        Py_INCREF(o);
        return o;
    }
    return PyMethod_New(o, obj);
}
PyGetSetDef device_call_getset[] = {{"__dict__", PyObject_GenericGetDict, PyObject_GenericSetDict, nullptr, nullptr},
                                    {nullptr, nullptr, nullptr, nullptr, nullptr}};
PyTypeObject DeviceCallType = {PyVarObject_HEAD_INIT(nullptr, 0)};

bool ready_device_call() {
    PyTypeObject& t = DeviceCallType;
    t.tp_name = "paper_1912_09268_amd._calls.DeviceCall";
    t.tp_basicsize = sizeof(DeviceCall);
    t.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_METHOD_DESCRIPTOR;
    t.tp_new = device_call_new;
    t.tp_call = PyVectorcall_Call;
    t.tp_vectorcall_offset = offsetof(DeviceCall, vectorcall);
    t.tp_dictoffset = offsetof(DeviceCall, dict);
    t.tp_getset = device_call_getset;
    t.tp_descr_get = device_call_get;
    t.tp_traverse = device_call_traverse;
    t.tp_clear = device_call_clear;
    t.tp_dealloc = device_call_dealloc;
    return PyType_Ready(&t) == 0;
}

// set_functions(check, {name: address})
PyObject* set_functions(PyObject*, PyObject* args) {
    PyObject *check, *table;
    if (!PyArg_ParseTuple(args, "OO!", &check, &PyDict_Type, &table)) return nullptr;
    void* entry[N_CALLS];
    for (int i = 0; i < N_CALLS; ++i) {
        PyObject* a = PyDict_GetItemString(table, CALLS[i].fn);
        if (a == nullptr || !PyLong_Check(a)) {
            PyErr_Format(PyExc_KeyError, "%s", CALLS[i].fn);
            return nullptr;
        }
        entry[i] = reinterpret_cast<void*>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(a)));
    }
    Py_INCREF(check);
    Py_XSETREF(g_raise, check);
    std::memcpy(g_entry, entry, sizeof entry);
    Py_RETURN_NONE;
}

// set_entry(name, address): one entry point, 0 for the plain function in its place
PyObject* set_entry(PyObject*, PyObject* args) {
    const char* fn;
    unsigned long long address;
    if (!PyArg_ParseTuple(args, "sK", &fn, &address)) return nullptr;
    const int which = call_index(fn);
    if (which >= 0) g_entry[which] = reinterpret_cast<void*>(static_cast<uintptr_t>(address));
    Py_RETURN_NONE;
}

PyMethodDef functions[] = {{"set_functions", set_functions, METH_VARARGS, "set_functions(check, {name: address})"},
                           {"set_entry", set_entry, METH_VARARGS, "set_entry(name, address)"},
                           {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", "device calls of Context", -1, functions,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
    if (g_handle == nullptr) g_handle = PyUnicode_InternFromString("_handle");
    if (g_handle == nullptr || !ready_device_call()) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m == nullptr) return nullptr;
    Py_INCREF(&DeviceCallType);
    if (PyModule_AddObject(m, "DeviceCall", reinterpret_cast<PyObject*>(&DeviceCallType)) < 0) {
        Py_DECREF(&DeviceCallType);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
