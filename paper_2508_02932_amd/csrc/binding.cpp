// Argument marshalling of the Python binding (plora.py) in C++: pointers out of tensors, lists of tensors into the host tables
// of device pointers that the C entry points take, the current stream, and the call.  No arithmetic, no state of a call is kept.
// In Python the marshalling was most of a short call: the optimizer step of 16 adapters took the host 36.5 us (7.8 now), a
// forward and a backward call of two fp32 adapters 28.9 (17.5, most of it the four launches), a forward of eight adapters 17.6 (12.8).
#include <torch/csrc/autograd/python_variable.h>

#include <Python.h>

#include <deque>
#include <string>
#include <unordered_map>
#include <vector>

#include "plora.h"

namespace {

struct PythonError {};                                         // a Python exception is set

struct Ref {                                                   // an owned reference
    PyObject *o;
    explicit Ref(PyObject *p) : o(p) { if (!o) throw PythonError(); }
    ~Ref() { Py_DECREF(o); }
    Ref(const Ref &) = delete;
    Ref &operator=(const Ref &) = delete;
};

uint64_t integer(PyObject *o)
{
    const Ref i(PyNumber_Long(o));
    const unsigned long long v = PyLong_AsUnsignedLongLong(i.o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) throw PythonError();
    return v;
}

uint64_t method_integer(PyObject *o, const char *name)
{
    const Ref r(PyObject_CallMethod(o, name, nullptr));
    return integer(r.o);
}

// Device pointer of a tensor (0 for None).  Anything but a plain tensor is asked for it as Python would.
uint64_t pointer(PyObject *o)
{
    if (o == Py_None) return 0;
    if (THPVariable_CheckExact(o)) {
        try {
            return (uint64_t)(uintptr_t)THPVariable_Unpack(o).data_ptr();
        } catch (const std::exception &) {                     // no storage: let the method raise its own error
        }
    }
    return method_integer(o, "data_ptr");
}

uint64_t byte_size(PyObject *o)
{
    if (THPVariable_CheckExact(o)) {
        const at::Tensor &t = THPVariable_Unpack(o);
        return (uint64_t)t.numel() * (uint64_t)t.element_size();
    }
    return method_integer(o, "numel") * method_integer(o, "element_size");
}

// Host arrays of one call; a deque keeps them where they are.
using Arrays = std::deque<std::vector<uint64_t>>;

uint64_t table(PyObject *list, Arrays &keep, bool none_allowed)
{
    if (list == Py_None) return 0;
    if (PyObject_Size(list) < 0) throw PythonError();          // (an iterator has no length)
    const Ref seq(PySequence_Fast(list, "a sequence of tensors is expected"));
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq.o);
    keep.emplace_back((size_t)(n > 0 ? n : 1), 0);
    std::vector<uint64_t> &out = keep.back();
    for (Py_ssize_t i = 0; i < n; ++i) {
        PyObject *o = PySequence_Fast_GET_ITEM(seq.o, i);
        out[(size_t)i] = o == Py_None && !none_allowed ? method_integer(o, "data_ptr") : pointer(o);
    }
    return (uint64_t)(uintptr_t)out.data();
}

uint64_t table_of_tables(PyObject *lists, Arrays &keep)
{
    if (lists == Py_None) return 0;
    if (PyObject_Size(lists) < 0) throw PythonError();
    const Ref seq(PySequence_Fast(lists, "a sequence of sequences of tensors is expected"));
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq.o);
    std::vector<uint64_t> out((size_t)(n > 0 ? n : 1), 0);
    for (Py_ssize_t i = 0; i < n; ++i) out[(size_t)i] = table(PySequence_Fast_GET_ITEM(seq.o, i), keep, false);
    keep.push_back(std::move(out));
    return (uint64_t)(uintptr_t)keep.back().data();
}

PyObject *g_device = nullptr, *g_raw_stream = nullptr;        // torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream

uint64_t stream_of(PyObject *s)
{
    if (s != Py_None) {
        const Ref h(PyObject_GetAttrString(s, "cuda_stream"));
        return integer(h.o);
    }
    const Ref dev(PyObject_CallNoArgs(g_device));
    const Ref h(PyObject_CallOneArg(g_raw_stream, dev.o));
    return integer(h.o);
}

struct Side { uint64_t t[5]; };

Side side_of(PyObject *dict, Arrays &keep)
{
    static const char *const names[5] = {"param", "master", "grad", "m", "v"};
    Side s{};
    for (int i = 0; i < 5; ++i) {
        const Ref v(PyObject_CallMethod(dict, "get", "s", names[i]));
        s.t[i] = table(v.o, keep, false);
    }
    return s;
}

std::vector<plora_adamw_hparams> hparams_of(PyObject *list)
{
    if (PyObject_Size(list) < 0) throw PythonError();
    const Ref seq(PySequence_Fast(list, "a sequence of hyperparameter tuples is expected"));
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq.o);
    std::vector<plora_adamw_hparams> out((size_t)(n > 0 ? n : 1));
    for (Py_ssize_t i = 0; i < n; ++i) {
        const Ref h(PySequence_Tuple(PySequence_Fast_GET_ITEM(seq.o, i)));
        const Py_ssize_t m = PyTuple_GET_SIZE(h.o);
        if (m < 6) { PyErr_SetString(PyExc_TypeError, "hyperparameters: (lr, beta1, beta2, eps, weight_decay, step[, grad_scale])"); throw PythonError(); }
        float f[7] = {0, 0, 0, 0, 0, 0, 1.f};                  // grad_scale may be left out
        int32_t step = 0;
        for (Py_ssize_t j = 0; j < m && j < 7; ++j) {
            PyObject *v = PyTuple_GET_ITEM(h.o, j);
            if (j == 5) {
                if (!PyLong_Check(v)) { PyErr_SetString(PyExc_TypeError, "step: an int is expected"); throw PythonError(); }
                const unsigned long k = PyLong_AsUnsignedLongMask(v);
                if (k == (unsigned long)-1 && PyErr_Occurred()) throw PythonError();
                step = (int32_t)(uint32_t)k;
            } else {
                const double d = PyFloat_AsDouble(v);
                if (d == -1.0 && PyErr_Occurred()) throw PythonError();
                f[j] = (float)d;
            }
        }
        out[(size_t)i] = plora_adamw_hparams{f[0], f[1], f[2], f[3], f[4], step, f[6]};
    }
    return out;
}

template <size_t... I> int invoke(void *fn, const uint64_t *a, std::index_sequence<I...>)
{
    return reinterpret_cast<int (*)(decltype((void)I, (uint64_t)0)...)>(fn)(a[I]...);
}
template <size_t N> int invoke_words(void *fn, const uint64_t *a) { return invoke(fn, a, std::make_index_sequence<N>()); }

// Integers and pointers all travel as 64-bit words in this platform's calling convention.  Looked up with the interpreter lock
// held: what a number of words that no entry point takes leads to is a Python error.
using Invoke = int (*)(void *, const uint64_t *);
Invoke invoke_for(size_t n_words)
{
    switch (n_words) {
    case 5: return invoke_words<5>;
    case 8: return invoke_words<8>;
    case 9: return invoke_words<9>;
    case 10: return invoke_words<10>;
    case 11: return invoke_words<11>;
    case 12: return invoke_words<12>;
    case 13: return invoke_words<13>;
    case 14: return invoke_words<14>;
    }
    PyErr_SetString(PyExc_RuntimeError, "no entry point takes this many arguments");
    throw PythonError();
}

struct Unlocked {                                              // the interpreter lock is given up for this scope, however it is left
    PyThreadState *state = PyEval_SaveThread();
    Unlocked() = default;
    ~Unlocked() { PyEval_RestoreThread(state); }
    Unlocked(const Unlocked &) = delete;
    Unlocked &operator=(const Unlocked &) = delete;
};

// call(address, form, argument, ...): one letter of the form per argument:
//   d  address of a description            p  tensor or None               t  list of tensors or None
//   P  list of tensors or Nones, or None   T  list of lists of tensors or None
//   w  workspace tensor (pointer, bytes)   s  stream or None (the current one)
//   a  optimizer side (dict of lists)      h  hyperparameters (list of tuples)
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    try {
        if (n_args < 2) { PyErr_SetString(PyExc_TypeError, "call(address, form, ...)"); return nullptr; }
        void *fn = reinterpret_cast<void *>((uintptr_t)integer(args[0]));
        Py_ssize_t n_form = 0;
        const char *form = PyUnicode_AsUTF8AndSize(args[1], &n_form);
        if (!form) return nullptr;
        if (!fn || n_form != n_args - 2) { PyErr_SetString(PyExc_TypeError, "call: form and arguments differ"); return nullptr; }
        Arrays keep;
        std::deque<Side> sides;
        std::vector<plora_adamw_hparams> hp;
        std::vector<uint64_t> a;
        a.reserve(16);
        for (Py_ssize_t i = 0; i < n_form; ++i) {
            PyObject *o = args[i + 2];
            switch (form[i]) {
            case 'd': a.push_back(integer(o)); break;
            case 'p': a.push_back(pointer(o)); break;
            case 't': a.push_back(table(o, keep, false)); break;
            case 'P': a.push_back(table(o, keep, true)); break;
            case 'T': a.push_back(table_of_tables(o, keep)); break;
            case 'w': a.push_back(pointer(o)); a.push_back(byte_size(o)); break;
            case 's': a.push_back(stream_of(o)); break;
            case 'a': sides.push_back(side_of(o, keep)); a.push_back((uint64_t)(uintptr_t)&sides.back()); break;
            case 'h': hp = hparams_of(o); a.push_back((uint64_t)(uintptr_t)hp.data()); break;
            default: PyErr_SetString(PyExc_TypeError, "call: unknown letter in the form"); return nullptr;
            }
        }
        int code = 0;
        const Invoke call_it = invoke_for(a.size());
        {
            const Unlocked unlocked;
            code = call_it(fn, a.data());
        }
        return PyLong_FromLong(code);
    } catch (const PythonError &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

PyMethodDef kMethods[] = {{"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(call)), METH_FASTCALL,
                           "call(address, form, argument, ...) -> status"},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_plora_binding", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__plora_binding()
{
    try {
        const Ref c(PyImport_ImportModule("torch._C"));
        g_device = PyObject_GetAttrString(c.o, "_cuda_getDevice");
        g_raw_stream = g_device ? PyObject_GetAttrString(c.o, "_cuda_getCurrentRawStream") : nullptr;
        if (!g_raw_stream) return nullptr;
        return PyModule_Create(&kModule);
    } catch (const PythonError &) {
        return nullptr;
    }
}
