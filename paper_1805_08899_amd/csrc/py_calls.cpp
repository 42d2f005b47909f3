// The Python binding's argument marshalling in native code: builtin functions with the names, parameters and defaults
// of the launching calls in binding.py, on top of the C ABI.
//
// What bounds a small call is the host: through ctypes a call with a dozen tensors spends 3 to 6 us on two Python-level
// method calls and one c_void_p object per tensor, more than the launch behind it (2.2 us here).  In native code a tensor
// argument costs a type check and two loads: 6.2 -> 0.6 us for the arguments of echo_attn_bwd; host time of a forward +
// backward pass 18.6 -> 14.5 us (its three launches are 7 of them), of a 50-step decoder sentence 609 -> 468 us.
//
// Arguments are matched by position or keyword; a device pointer is a torch tensor (contiguous), an integer address, None, or
// any object (tensor subclasses among them) with is_contiguous() and data_ptr().  The interpreter lock is released around the library call, as ctypes
// does.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>
#include <tuple>
#include <utility>

#include "../../include/echodropout.h"
#include "../../include/echolstm.h"

namespace {

PyTypeObject *g_desc_type = nullptr;                       // binding.echo_attn_desc_t
PyObject *g_s_data_ptr, *g_s_is_contiguous, *g_s_cuda_stream, *g_s_numel, *g_s_element_size;

bool int_value(PyObject *o, unsigned long long &out) {     // two's complement bits of any integer, as ctypes takes them
    if (!PyLong_Check(o)) {
        PyErr_Format(PyExc_TypeError, "an integer is required, not %.100s", Py_TYPE(o)->tp_name);
        return false;
    }
    out = PyLong_AsUnsignedLongLongMask(o);
    return !(out == (unsigned long long)-1 && PyErr_Occurred());
}

bool address_from_attribute(PyObject *o, PyObject *attr, bool call, void *&out) {
    PyObject *r = call ? PyObject_CallMethodNoArgs(o, attr) : PyObject_GetAttr(o, attr);
    if (!r) return false;
    unsigned long long x = 0;
    const bool ok = int_value(r, x);
    Py_DECREF(r);
    out = reinterpret_cast<void *>(x);
    return ok;
}

// ---- one parameter kind each: how many Python parameters it takes, what it holds, how it is read ----------------
struct Desc {                                              // echo_attn_desc_t, a ctypes structure
    using C = const echo_attn_desc_t *;
    Py_buffer view{};
    bool read(PyObject *o) {
        if (!PyObject_TypeCheck(o, g_desc_type)) {
            PyErr_Format(PyExc_TypeError, "expected echo_attn_desc_t, got %.100s", Py_TYPE(o)->tp_name);
            return false;
        }
        return PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) == 0;
    }
    C value() const { return static_cast<C>(view.buf); }
    ~Desc() {
        if (view.obj) PyBuffer_Release(&view);
    }
};
template <typename T> struct Ptr {
    using C = T *;
    void *p = nullptr;
    bool read(PyObject *o) {
        if (THPVariable_CheckExact(o)) {                    // subclasses may override the two methods: they go through them below
            try {                                           // tensors without storage (fake, functional, under a transform) throw
                const at::Tensor &t = THPVariable_Unpack(o);
                if (!t.is_contiguous()) {
                    PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
                    return false;
                }
                p = t.data_ptr();
            } catch (const c10::Error &e) {
                PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
                return false;
            } catch (const std::exception &e) {
                PyErr_SetString(PyExc_RuntimeError, e.what());
                return false;
            }
            return true;
        }
        if (o == Py_None) return true;
        if (PyLong_Check(o)) {
            unsigned long long x = 0;
            if (!int_value(o, x)) return false;
            p = reinterpret_cast<void *>(x);
            return true;
        }
        PyObject *c = PyObject_CallMethodNoArgs(o, g_s_is_contiguous);
        if (!c) return false;
        const int yes = PyObject_IsTrue(c);
        Py_DECREF(c);
        if (yes == 0) PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
        return yes > 0 && address_from_attribute(o, g_s_data_ptr, true, p);
    }
    C value() const { return static_cast<C>(p); }
};
struct Stream {
    using C = void *;
    void *p = nullptr;
    bool read(PyObject *o) {
        if (o == Py_None) return true;
        if (PyLong_Check(o)) {
            unsigned long long x = 0;
            if (!int_value(o, x)) return false;
            p = reinterpret_cast<void *>(x);
            return true;
        }
        return address_from_attribute(o, g_s_cuda_stream, false, p);
    }
    C value() const { return p; }
};
template <typename T> struct Int {
    using C = T;
    T x = 0;
    bool read(PyObject *o) {
        unsigned long long u = 0;
        if (!int_value(o, u)) return false;
        x = static_cast<T>(u);
        return true;
    }
    C value() const { return x; }
};
struct Float {
    using C = float;
    float x = 0.f;
    bool read(PyObject *o) {
        const double d = PyFloat_AsDouble(o);
        if (d == -1.0 && PyErr_Occurred()) return false;
        x = static_cast<float>(d);
        return true;
    }
    C value() const { return x; }
};
struct Bytes {                                             // workspace_bytes; None: what the workspace tensor holds
    using C = size_t;
    size_t x = 0;
    bool given = false;
    bool read(PyObject *o) {
        if (o == Py_None) return true;
        unsigned long long u = 0;
        if (!int_value(o, u)) return false;
        x = u;
        given = true;
        return true;
    }
    // `ws`: the argument in front of this one
    bool resolve(PyObject *ws) {
        if (given || ws == Py_None || PyLong_Check(ws)) return true;
        if (THPVariable_CheckExact(ws)) {                   // Ptr::read has accepted it: strided, with storage
            try {
                x = THPVariable_Unpack(ws).nbytes();
            } catch (const c10::Error &e) {
                PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
                return false;
            } catch (const std::exception &e) {
                PyErr_SetString(PyExc_RuntimeError, e.what());
                return false;
            }
            return true;
        }
        void *n = nullptr, *e = nullptr;
        if (!address_from_attribute(ws, g_s_numel, true, n) || !address_from_attribute(ws, g_s_element_size, true, e)) return false;
        x = reinterpret_cast<uintptr_t>(n) * reinterpret_cast<uintptr_t>(e);
        return true;
    }
    C value() const { return x; }
};

// ---- a call: parameter kinds in the order of the C prototype, parameter names in the same order ----------------
constexpr int kMaxParams = 20;
struct Names {
    const char *fn;
    const char *param[kMaxParams];                         // nullptr-terminated
    int required;                                          // the rest default to None
    PyObject *interned[kMaxParams];
    int count;
    void *target;                                          // the library's function, set by bind()
};

bool collect(Names &n, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames, PyObject **slot) {
    if (!n.target) {
        PyErr_Format(PyExc_RuntimeError, "%s: the library is not loaded", n.fn);
        return false;
    }
    if (nargs > n.count) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", n.fn, n.count, nargs);
        return false;
    }
    for (int i = 0; i < n.count; ++i) slot[i] = i < nargs ? args[i] : nullptr;
    const Py_ssize_t nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t k = 0; k < nk; ++k) {
        PyObject *key = PyTuple_GET_ITEM(kwnames, k);
        int at = 0;
        while (at < n.count && n.interned[at] != key) ++at;          // keywords in source code are interned
        if (at == n.count)
            for (at = 0; at < n.count && PyUnicode_Compare(n.interned[at], key) != 0;) ++at;
        if (at == n.count || slot[at]) {
            PyErr_Format(PyExc_TypeError, at == n.count ? "%s() got an unexpected keyword argument '%U'"
                                                        : "%s() got multiple values for argument '%U'", n.fn, key);
            return false;
        }
        slot[at] = args[nargs + k];
    }
    for (int i = 0; i < n.count; ++i) {
        if (slot[i]) continue;
        if (i < n.required) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", n.fn, n.param[i]);
            return false;
        }
        slot[i] = Py_None;
    }
    return true;
}

template <typename P> bool resolve_bytes(P &, PyObject *) { return true; }
bool resolve_bytes(Bytes &b, PyObject *ws) { return b.resolve(ws); }

template <typename... K, size_t... I>
PyObject *call_with(Names &n, PyObject **slot, std::index_sequence<I...>) {
    std::tuple<K...> a;
    if (!(std::get<I>(a).read(slot[I]) && ...)) return nullptr;
    if (!(resolve_bytes(std::get<I>(a), slot[I > 0 ? I - 1 : 0]) && ...)) return nullptr;
    const auto fn = reinterpret_cast<echo_status_t (*)(typename K::C...)>(n.target);
    echo_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(std::get<I>(a).value()...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

template <int ID, typename... K> struct Call {
    static Names names;
    static PyObject *run(PyObject *, PyObject *const *args, Py_ssize_t nargs, PyObject *kwnames) {
        PyObject *slot[kMaxParams];
        if (!collect(names, args, nargs, kwnames, slot)) return nullptr;
        return call_with<K...>(names, slot, std::index_sequence_for<K...>{});
    }
};

using In = Ptr<const void>;
using InF = Ptr<const float>;
using Len = Ptr<const int32_t>;
using OutF = Ptr<float>;
using Work = Ptr<void>;
using I32 = Int<int32_t>;
using I64 = Int<int64_t>;
using U64 = Int<uint64_t>;
using Size = Int<size_t>;

// every launching call of the headers
using Fwd = Call<0, Desc, In, In, In, In, Len, OutF, OutF, Work, Bytes, Stream>;
using Bwd = Call<1, Desc, InF, InF, In, In, In, In, Len, OutF, OutF, OutF, OutF, Work, Bytes, Stream>;
using BwdStatic = Call<2, Desc, InF, InF, In, In, In, In, Len, OutF, OutF, OutF, OutF, Stream>;
using BwdAccumulate = Call<3, Desc, InF, InF, In, In, In, In, Len, OutF, OutF, OutF, OutF, Work, Bytes, Stream>;
using StepFwd = Call<4, Desc, In, In, In, In, Len, OutF, OutF, Stream>;
using StepBwd = Call<5, Desc, InF, InF, In, In, In, In, Len, OutF, OutF, OutF, OutF, Stream>;
using StepFinish = Call<6, Desc, InF, OutF, Stream>;
using StepBwdQuery = Call<7, Desc, I32, I32, InF, InF, In, In, In, In, Len, OutF, Work, Stream>;
using StepsBwdKeys = Call<8, Desc, InF, InF, In, In, In, Len, In, OutF, OutF, OutF, Work, Bytes, Stream>;
using FwdStash = Call<9, Desc, In, In, In, In, Len, OutF, OutF, OutF, Work, Bytes, Stream>;
using BwdStash = Call<10, Desc, InF, InF, InF, In, In, Len, OutF, OutF, OutF, OutF, Work, Bytes, Stream>;
using DropoutFwd = Call<11, InF, Size, Float, U64, U64, OutF, Ptr<uint32_t>, Stream>;
using DropoutBwd = Call<12, InF, Ptr<const uint32_t>, Size, Float, OutF, Stream>;
using LstmFwd = Call<13, I64, I64, InF, InF, InF, OutF, OutF, OutF, Stream>;
using LstmBwd = Call<14, I64, I64, InF, InF, InF, InF, OutF, OutF, Stream>;
using LstmFwdStash = Call<15, I64, I64, InF, InF, InF, OutF, OutF, OutF, OutF, Stream>;
using LstmBwdStash = Call<16, I64, I64, InF, InF, InF, InF, InF, OutF, OutF, Stream>;

#define NAMES(CALL, FN, REQUIRED, ...) template <> Names CALL::names = {FN, {__VA_ARGS__, nullptr}, REQUIRED, {}, 0, nullptr}
NAMES(Fwd, "echo_attn_fwd", 9, "desc", "Qp", "Kp", "V", "v", "key_len", "context", "P", "workspace", "workspace_bytes", "stream");
NAMES(Bwd, "echo_attn_bwd", 13, "desc", "dContext", "P", "Qp", "Kp", "V", "v", "key_len", "dQp", "dKp", "dV", "dv", "workspace",
      "workspace_bytes", "stream");
NAMES(BwdStatic, "echo_attn_bwd_static", 12, "desc", "dContext", "P", "Qp", "Kp", "V", "v", "key_len", "dQp", "dKp", "dV", "dv",
      "stream");
NAMES(BwdAccumulate, "echo_attn_bwd_accumulate", 13, "desc", "dContext", "P", "Qp", "Kp", "V", "v", "key_len", "dQp", "dKp", "dV",
      "dv", "workspace", "workspace_bytes", "stream");
NAMES(StepFwd, "echo_attn_step_fwd", 8, "desc", "Qp", "Kp", "V", "v", "key_len", "context", "P", "stream");
NAMES(StepBwd, "echo_attn_step_bwd", 12, "desc", "dContext", "P", "Qp", "Kp", "V", "v", "key_len", "dQp", "dKp", "dV", "dv_part",
      "stream");
NAMES(StepFinish, "echo_attn_step_finish", 3, "desc", "dv_part", "dv", "stream");
NAMES(StepBwdQuery, "echo_attn_step_bwd_query", 12, "desc", "step", "steps", "dContext", "P", "Qp", "Kp", "V", "v", "key_len", "dQp",
      "ds_rows", "stream");
NAMES(StepsBwdKeys, "echo_attn_steps_bwd_keys", 12, "desc", "dContext", "P", "Qp", "Kp", "v", "key_len", "ds_rows", "dKp", "dV", "dv",
      "workspace", "workspace_bytes", "stream");
NAMES(FwdStash, "echo_attn_fwd_stash", 10, "desc", "Qp", "Kp", "V", "v", "key_len", "context", "P", "tanh_map", "workspace",
      "workspace_bytes", "stream");
NAMES(BwdStash, "echo_attn_bwd_stash", 12, "desc", "dContext", "P", "tanh_map", "V", "v", "key_len", "dQp", "dKp", "dV", "dv",
      "workspace", "workspace_bytes", "stream");
NAMES(DropoutFwd, "echo_dropout_fwd", 7, "x", "n", "p", "seed", "offset", "y", "mask_bits", "stream");
NAMES(DropoutBwd, "echo_dropout_bwd", 5, "dy", "mask_bits", "n", "p", "dx", "stream");
NAMES(LstmFwd, "echo_lstm_cell_fwd", 8, "B", "H", "Gx", "Gh", "c_prev", "h", "c", "a", "stream");
NAMES(LstmBwd, "echo_lstm_cell_bwd", 8, "B", "H", "dh", "dc", "a", "c_prev", "da", "dc_prev", "stream");
NAMES(LstmFwdStash, "echo_lstm_cell_fwd_stash", 9, "B", "H", "Gx", "Gh", "c_prev", "h", "c", "acts", "tanh_c", "stream");
NAMES(LstmBwdStash, "echo_lstm_cell_bwd_stash", 9, "B", "H", "dh", "dc", "acts", "tanh_c", "c_prev", "da", "dc_prev", "stream");
#undef NAMES

Names *const kAll[] = {&Fwd::names, &Bwd::names, &BwdStatic::names, &BwdAccumulate::names, &StepFwd::names, &StepBwd::names,
                       &StepFinish::names, &StepBwdQuery::names, &StepsBwdKeys::names, &FwdStash::names, &BwdStash::names,
                       &DropoutFwd::names, &DropoutBwd::names, &LstmFwd::names, &LstmBwd::names, &LstmFwdStash::names,
                       &LstmBwdStash::names};

// bind(desc_type, {name: address of the loaded library's function}): the names that are not in the dict raise when called
PyObject *bind(PyObject *, PyObject *args) {
    PyObject *type = nullptr, *addresses = nullptr;
    if (!PyArg_ParseTuple(args, "O!O!", &PyType_Type, &type, &PyDict_Type, &addresses)) return nullptr;
    for (Names *n : kAll) {
        PyObject *a = PyDict_GetItemString(addresses, n->fn);        // borrowed
        unsigned long long x = 0;
        if (a && !int_value(a, x)) return nullptr;
        n->target = reinterpret_cast<void *>(x);
    }
    Py_INCREF(type);
    Py_XDECREF(reinterpret_cast<PyObject *>(g_desc_type));
    g_desc_type = reinterpret_cast<PyTypeObject *>(type);
    Py_RETURN_NONE;
}

#define METHOD(CALL) \
    {CALL::names.fn, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&CALL::run)), METH_FASTCALL | METH_KEYWORDS, nullptr}
PyMethodDef g_methods[] = {METHOD(Fwd), METHOD(Bwd), METHOD(BwdStatic), METHOD(BwdAccumulate), METHOD(StepFwd), METHOD(StepBwd),
                           METHOD(StepFinish), METHOD(StepBwdQuery), METHOD(StepsBwdKeys), METHOD(FwdStash), METHOD(BwdStash),
                           METHOD(DropoutFwd), METHOD(DropoutBwd), METHOD(LstmFwd), METHOD(LstmBwd), METHOD(LstmFwdStash),
                           METHOD(LstmBwdStash), {"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
#undef METHOD

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_py_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__py_calls() {
    for (Names *n : kAll)
        for (n->count = 0; n->param[n->count]; ++n->count) {
            n->interned[n->count] = PyUnicode_InternFromString(n->param[n->count]);
            if (!n->interned[n->count]) return nullptr;
        }
    g_s_data_ptr = PyUnicode_InternFromString("data_ptr");
    g_s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
    g_s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    g_s_numel = PyUnicode_InternFromString("numel");
    g_s_element_size = PyUnicode_InternFromString("element_size");
    if (!g_s_data_ptr || !g_s_is_contiguous || !g_s_cuda_stream || !g_s_numel || !g_s_element_size) return nullptr;
    return PyModule_Create(&g_module);
}
