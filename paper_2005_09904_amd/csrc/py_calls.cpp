// Calls from Python into libbiq.so without ctypes (module paper_2005_09904_amd._calls).
//
// Bound by the host: a small layer's kernel takes 3 us, its launch 2.5 us, and marshalling a dozen
// arguments through ctypes took 1.2-2 us of what was left.  Here a call converts its
// arguments itself (tensors by their data_ptr(), as the ctypes binding did) or has them converted once
// (Prepared), and only crosses the C ABI.  The functions' addresses come from the library that
// binding.load_library() holds; nothing is linked against it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "biq.h"

namespace {

// The entry points and the callables of binding.py that a call needs.
enum { GEMM, QUERY, GEMM_NOALLOC, PACK, QUANTIZE, BUILD_LUT, GROUPED, LSTM, ENTRIES };
const char* const kNames[ENTRIES] = {"biq_gemm",     "biq_query",     "biq_gemm_noalloc", "biq_pack",
                                     "biq_quantize", "biq_build_lut", "biq_gemm_grouped", "biq_lstm_cell"};

struct Calls {
    PyObject_HEAD
    void* fn[ENTRIES];
    PyObject* check;      // (status, name): raises BiqError
    PyObject* as_int;     // integers that are no Python int
    PyObject* stream;     // () -> handle of the current stream
};

PyObject *str_data_ptr, *str_numel, *str_element_size, *str_cuda_stream;

constexpr int kMaxArgs = 13;

// Arguments of one call in the order of its C function, whatever their width.
struct Args {
    uint64_t v[kMaxArgs];
    void* p(int i) const { return reinterpret_cast<void*>(static_cast<uintptr_t>(v[i])); }
    int i(int k) const { return static_cast<int>(static_cast<uint32_t>(v[k])); }
    size_t z(int i) const { return static_cast<size_t>(v[i]); }
};

// Python int -> its low 64 bits (as ctypes: no overflow check); others through as_int.
bool integer(const Calls* c, PyObject* o, uint64_t& out) {
    if (PyLong_Check(o)) {
        out = PyLong_AsUnsignedLongLongMask(o);
        return !(out == ~0ull && PyErr_Occurred());
    }
    PyObject* r = PyObject_CallOneArg(c->as_int, o);
    if (!r) return false;
    out = PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return !(out == ~0ull && PyErr_Occurred());
}

bool method_integer(PyObject* o, PyObject* name, uint64_t& out) {
    PyObject* r = PyObject_CallMethodNoArgs(o, name);
    if (!r) return false;
    out = PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return !(out == ~0ull && PyErr_Occurred());
}

bool pointer(PyObject* o, uint64_t& out) {
    out = 0;
    return o == Py_None || method_integer(o, str_data_ptr, out);
}

bool bytes(PyObject* o, uint64_t& out) {
    out = 0;
    if (o == Py_None) return true;
    uint64_t count, size;
    if (!method_integer(o, str_numel, count) || !method_integer(o, str_element_size, size)) return false;
    out = count * size;
    return true;
}

bool stream_of(const Calls* c, PyObject* o, uint64_t& out) {
    PyObject* r = o == Py_None ? PyObject_CallNoArgs(c->stream) : PyObject_GetAttr(o, str_cuda_stream);
    if (!r) return false;
    out = 0;
    if (r != Py_None) out = PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
    return !(out == ~0ull && PyErr_Occurred());
}

// `tensors` pointers, `ints` integers, a workspace and its size if the function takes one, the stream.
bool convert(const Calls* c, PyObject* const* a, Py_ssize_t nargs, int tensors, int ints, bool workspace, Args& out) {
    if (nargs != tensors + ints + workspace + 1) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return false;
    }
    int k = 0;
    for (int i = 0; i < tensors; ++i, ++k)
        if (!pointer(a[k], out.v[k])) return false;
    for (int i = 0; i < ints; ++i, ++k)
        if (!integer(c, a[k], out.v[k])) return false;
    int j = k;
    if (workspace) {
        if (!pointer(a[k], out.v[j]) || !bytes(a[k], out.v[j + 1])) return false;
        ++k;
        j += 2;
    }
    return stream_of(c, a[k], out.v[j]);
}

// What a function takes before the stream: tensors, integers, a workspace.
struct Form { int tensors, ints; bool workspace; };
constexpr Form kForms[ENTRIES] = {{4, 5, true}, {4, 5, true}, {4, 5, false}, {2, 4, false},
                                  {3, 3, false}, {2, 3, false}, {1, 2, false}, {7, 5, false}};

// The call itself, without the interpreter lock (as ctypes): a launch can wait for room in the queue.
biq_status enter(int entry, void* fn, const Args& a) {
    biq_status s = BIQ_EINVAL;
    Py_BEGIN_ALLOW_THREADS
    auto in = [&](int i) { return static_cast<const float*>(a.p(i)); };
    auto out = [&](int i) { return static_cast<float*>(a.p(i)); };
    auto keys = [&](int i) { return static_cast<uint8_t*>(a.p(i)); };
    switch (entry) {
        case GEMM:
        case QUERY:
            s = reinterpret_cast<decltype(&biq_gemm)>(fn)(keys(0), in(1), in(2), out(3), a.i(4), a.i(5), a.i(6), a.i(7),
                                                          a.i(8), a.p(9), a.z(10), a.p(11));
            break;
        case GEMM_NOALLOC:
            s = reinterpret_cast<decltype(&biq_gemm_noalloc)>(fn)(keys(0), in(1), in(2), out(3), a.i(4), a.i(5), a.i(6),
                                                                  a.i(7), a.i(8), a.p(9));
            break;
        case PACK:
            s = reinterpret_cast<decltype(&biq_pack)>(fn)(static_cast<const int8_t*>(a.p(0)), keys(1), a.i(2), a.i(3),
                                                          a.i(4), a.i(5), a.p(6));
            break;
        case QUANTIZE:
            s = reinterpret_cast<decltype(&biq_quantize)>(fn)(in(0), keys(1), out(2), a.i(3), a.i(4), a.i(5), a.p(6));
            break;
        case BUILD_LUT:
            s = reinterpret_cast<decltype(&biq_build_lut)>(fn)(in(0), out(1), a.i(2), a.i(3), a.i(4), a.p(5));
            break;
        case GROUPED:
            s = reinterpret_cast<decltype(&biq_gemm_grouped)>(fn)(static_cast<const biq_problem*>(a.p(0)), a.i(1), a.i(2),
                                                                  a.p(3));
            break;
        case LSTM:
            s = reinterpret_cast<decltype(&biq_lstm_cell)>(fn)(keys(0), in(1), in(2), in(3), in(4), out(5), out(6), a.i(7),
                                                               a.i(8), a.i(9), a.i(10), a.i(11), a.p(12));
            break;
    }
    Py_END_ALLOW_THREADS
    return s;
}

PyObject* finish(PyObject* check, int entry, biq_status s) {
    if (s == BIQ_OK) Py_RETURN_NONE;
    return PyObject_CallFunction(check, "is", static_cast<int>(s), kNames[entry]);
}

template <int ENTRY>
PyObject* call(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    Args args;
    if (!convert(c, a, nargs, kForms[ENTRY].tensors, kForms[ENTRY].ints, kForms[ENTRY].workspace, args)) return nullptr;
    return finish(c->check, ENTRY, enter(ENTRY, c->fn[ENTRY], args));
}

// ---- a call whose arguments were converted once; the caller keeps the tensors -------------------------
struct Prepared {
    PyObject_HEAD
    int entry;
    void* fn;
    PyObject* check;
    Args args;
};

PyObject* prepared_call(PyObject* self, PyObject* args, PyObject* kwargs) {
    if (PyTuple_GET_SIZE(args) != 0 || (kwargs && PyDict_GET_SIZE(kwargs) != 0)) {
        PyErr_SetString(PyExc_TypeError, "a prepared call takes no arguments");
        return nullptr;
    }
    const Prepared* p = reinterpret_cast<Prepared*>(self);
    return finish(p->check, p->entry, enter(p->entry, p->fn, p->args));
}

void prepared_dealloc(PyObject* self) {
    Py_XDECREF(reinterpret_cast<Prepared*>(self)->check);
    Py_TYPE(self)->tp_free(self);
}

PyTypeObject prepared_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

template <int ENTRY>
PyObject* prepare(PyObject* self, PyObject* const* a, Py_ssize_t nargs) {
    const Calls* c = reinterpret_cast<Calls*>(self);
    Args args{};
    if constexpr (ENTRY == GROUPED) {      // (address of the descriptors, count, mu, stream)
        if (nargs != 4) {
            PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
            return nullptr;
        }
        for (int i = 0; i < 3; ++i)
            if (!integer(c, a[i], args.v[i])) return nullptr;
        if (!stream_of(c, a[3], args.v[3])) return nullptr;
    } else {
        if (!convert(c, a, nargs, kForms[ENTRY].tensors, kForms[ENTRY].ints, kForms[ENTRY].workspace, args)) return nullptr;
    }
    Prepared* p = PyObject_New(Prepared, &prepared_type);
    if (!p) return nullptr;
    p->entry = ENTRY;
    p->fn = c->fn[ENTRY];
    p->check = c->check;
    Py_INCREF(p->check);
    p->args = args;
    return reinterpret_cast<PyObject*>(p);
}

// Calls({name: address}, check, as_int, stream)
PyObject* calls_new(PyTypeObject* type, PyObject* args, PyObject*) {
    PyObject *table, *check, *as_int, *stream;
    if (!PyArg_ParseTuple(args, "O!OOO", &PyDict_Type, &table, &check, &as_int, &stream)) return nullptr;
    Calls* c = reinterpret_cast<Calls*>(type->tp_alloc(type, 0));
    if (!c) return nullptr;
    Py_INCREF(check); Py_INCREF(as_int); Py_INCREF(stream);
    c->check = check; c->as_int = as_int; c->stream = stream;
    for (int e = 0; e < ENTRIES; ++e) {
        PyObject* address = PyDict_GetItemString(table, kNames[e]);
        c->fn[e] = address ? PyLong_AsVoidPtr(address) : nullptr;
        if (!c->fn[e]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, kNames[e]);
            Py_DECREF(c);
            return nullptr;
        }
    }
    return reinterpret_cast<PyObject*>(c);
}

void calls_dealloc(PyObject* self) {
    Calls* c = reinterpret_cast<Calls*>(self);
    Py_XDECREF(c->check); Py_XDECREF(c->as_int); Py_XDECREF(c->stream);
    Py_TYPE(self)->tp_free(self);
}

#define BIQ_METHOD(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef calls_methods[] = {
    BIQ_METHOD("gemm", call<GEMM>), BIQ_METHOD("query", call<QUERY>), BIQ_METHOD("gemm_noalloc", call<GEMM_NOALLOC>),
    BIQ_METHOD("pack", call<PACK>), BIQ_METHOD("quantize", call<QUANTIZE>), BIQ_METHOD("build_lut", call<BUILD_LUT>),
    BIQ_METHOD("lstm_cell", call<LSTM>), BIQ_METHOD("prepare_gemm", prepare<GEMM>),
    BIQ_METHOD("prepare_grouped", prepare<GROUPED>), BIQ_METHOD("prepare_lstm_cell", prepare<LSTM>),
    {nullptr, nullptr, 0, nullptr}};
#undef BIQ_METHOD

PyTypeObject calls_type = {PyVarObject_HEAD_INIT(nullptr, 0)};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
    prepared_type.tp_name = "paper_2005_09904_amd._calls.Prepared";
    prepared_type.tp_basicsize = sizeof(Prepared);
    prepared_type.tp_flags = Py_TPFLAGS_DEFAULT;
    prepared_type.tp_dealloc = prepared_dealloc;
    prepared_type.tp_call = prepared_call;
    calls_type.tp_name = "paper_2005_09904_amd._calls.Calls";
    calls_type.tp_basicsize = sizeof(Calls);
    calls_type.tp_flags = Py_TPFLAGS_DEFAULT;
    calls_type.tp_dealloc = calls_dealloc;
    calls_type.tp_new = calls_new;
    calls_type.tp_methods = calls_methods;
    if (PyType_Ready(&prepared_type) < 0 || PyType_Ready(&calls_type) < 0) return nullptr;
    str_data_ptr = PyUnicode_InternFromString("data_ptr");
    str_numel = PyUnicode_InternFromString("numel");
    str_element_size = PyUnicode_InternFromString("element_size");
    str_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    PyObject* m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    Py_INCREF(&calls_type);
    if (PyModule_AddObject(m, "Calls", reinterpret_cast<PyObject*>(&calls_type)) < 0) return nullptr;
    return m;
}
