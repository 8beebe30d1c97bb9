// Python calls of the entry points without ctypes: torch tensors, numbers and ctypes structures in, the C ABI called, its
// status out.  A decode round makes dozens of calls of up to 20 arguments, and the commit takes the caches of every layer: the
// three attribute lookups per tensor from Python took 22 us for 96 caches, more than the kernels of the call.
//
// Every wrapper follows from the entry point's own signature (one template).  A pointer is a device pointer: it takes a contiguous
// tensor on the GPU or None, and nothing else, so that host memory never reaches a kernel as one.  The exceptions have types of
// their own: the descriptor (a ctypes structure), host out-parameters (ENTRY_HOST names their position) and the stream (always the
// last argument, a raw handle).  An array of pointers takes a sequence of tensors, the projection jobs a sequence of sequences; size_t
// takes an integer or a tensor (its bytes); the rest are numbers.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <cstdint>
#include <exception>
#include <tuple>
#include <utility>
#include <vector>
#include "dream.h"

namespace {

struct Failed {};     // a Python exception has been set

void *device_pointer(PyObject *o)
{
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda()) {
        PyErr_SetString(PyExc_ValueError, "device tensor expected");
        throw Failed();
    }
    if (!t.is_contiguous()) {
        PyErr_SetString(PyExc_ValueError, "contiguous tensor expected");
        throw Failed();
    }
    return t.data_ptr();
}

// One argument of type T, alive as long as the call.
template <class T>
struct Arg {
    static_assert(std::is_integral_v<T>, "numbers");
    T value;
    explicit Arg(PyObject *o)
    {
        if (std::is_same_v<T, size_t> && THPVariable_Check(o)) {
            value = (T)THPVariable_Unpack(o).nbytes();
            return;
        }
        const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
        if (PyErr_Occurred())
            throw Failed();
        value = (T)v;
    }
};
template <>
struct Arg<float> {
    float value;
    explicit Arg(PyObject *o) : value((float)PyFloat_AsDouble(o))
    {
        if (PyErr_Occurred())
            throw Failed();
    }
};
template <class T>
struct Arg<T *> {
    T *value = nullptr;
    explicit Arg(PyObject *o)
    {
        if (o == Py_None)
            return;
        if (!THPVariable_Check(o)) {
            PyErr_Format(PyExc_TypeError, "device tensor or None expected, not %.100s", Py_TYPE(o)->tp_name);
            throw Failed();
        }
        value = static_cast<T *>(device_pointer(o));
    }
};

// Host memory of exactly one T, through the buffer interface (ctypes structures and numbers are writable buffers).
template <class T>
struct HostObject {
    T *value = nullptr;
    Py_buffer view = {};
    explicit HostObject(PyObject *o, bool nullable)
    {
        if (nullable && o == Py_None)
            return;
        if (PyObject_GetBuffer(o, &view, PyBUF_WRITABLE))
            throw Failed();
        if (view.len != (Py_ssize_t)sizeof(T)) {
            PyBuffer_Release(&view);
            PyErr_Format(PyExc_TypeError, "an object of %d bytes is expected", (int)sizeof(T));
            throw Failed();
        }
        value = static_cast<T *>(view.buf);
    }
    ~HostObject()
    {
        if (view.obj)
            PyBuffer_Release(&view);
    }
    HostObject(const HostObject &) = delete;
};
template <>
struct Arg<const dream_attn_desc *> : HostObject<dream_attn_desc> {
    explicit Arg(PyObject *o) : HostObject(o, false) {}
};
struct HostInt : HostObject<int32_t> {
    explicit HostInt(PyObject *o) : HostObject(o, true) {}
};
struct Stream {
    void *value;
    explicit Stream(PyObject *o) : value(PyLong_AsVoidPtr(o))
    {
        if (PyErr_Occurred())
            throw Failed();
    }
};

template <>
struct Arg<void *const *> {
    std::vector<void *> pointers;
    void *const *value;
    explicit Arg(PyObject *o)
    {
        PyObject *seq = PySequence_Fast(o, "a sequence of tensors is expected");
        if (!seq)
            throw Failed();
        try {
            const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
            pointers.reserve(n);
            for (Py_ssize_t i = 0; i < n; i++) {
                PyObject *t = PySequence_Fast_GET_ITEM(seq, i);
                if (!THPVariable_Check(t)) {
                    PyErr_SetString(PyExc_TypeError, "a sequence of tensors is expected");
                    throw Failed();
                }
                pointers.push_back(device_pointer(t));
            }
        } catch (...) {
            Py_DECREF(seq);
            throw;
        }
        Py_DECREF(seq);
        value = pointers.data();
    }
};

// A sequence of (x, w, n_heads, row_base, row_index, out).
template <>
struct Arg<const dream_proj_job *> {
    std::vector<dream_proj_job> jobs;
    const dream_proj_job *value;
    explicit Arg(PyObject *o)
    {
        PyObject *seq = PySequence_Fast(o, "a sequence of jobs is expected");
        if (!seq)
            throw Failed();
        try {
            const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
            for (Py_ssize_t i = 0; i < n; i++) {
                // (a tuple of its own: converting a field may run Python code, which must not take the others away)
                struct Owned {
                    PyObject *o;
                    ~Owned() { Py_XDECREF(o); }
                } job = {PySequence_Tuple(PySequence_Fast_GET_ITEM(seq, i))};
                if (!job.o)
                    throw Failed();
                if (PyTuple_GET_SIZE(job.o) != 6) {
                    PyErr_SetString(PyExc_ValueError, "a job is (x, w, n_heads, row_base, row_index, out)");
                    throw Failed();
                }
                auto pointer = [&](int k) { return Arg<void *>(PyTuple_GET_ITEM(job.o, k)).value; };
                jobs.push_back({pointer(0), pointer(1), Arg<int32_t>(PyTuple_GET_ITEM(job.o, 2)).value, static_cast<int32_t *>(pointer(3)),
                                static_cast<int32_t *>(pointer(4)), pointer(5)});
            }
        } catch (...) {
            Py_DECREF(seq);
            throw;
        }
        Py_DECREF(seq);
        value = jobs.data();
    }
};

struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// HOST: position of the host out-parameter, or -1
template <auto F, int HOST>
struct Entry;
template <class... A, int (*F)(A...), int HOST>
struct Entry<F, HOST> {
    template <class T, int I>
    using ArgAt = std::conditional_t<I == (int)sizeof...(A) - 1, Stream, std::conditional_t<I == HOST, HostInt, Arg<T>>>;
    template <size_t... I>
    static int run(PyObject *const *args, std::index_sequence<I...>)
    {
        const std::tuple<ArgAt<A, I>...> a(args[I]...);     // (converted in place: some are neither copied nor moved)
        const WithoutGil unlocked;
        return F(std::get<I>(a).value...);
    }
    static PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n)
    {
        if (n != (Py_ssize_t)sizeof...(A))
            return PyErr_Format(PyExc_TypeError, "%d arguments expected, got %d", (int)sizeof...(A), (int)n);
        try {
            return PyLong_FromLong(run(args, std::index_sequence_for<A...>{}));
        } catch (const Failed &) {
        } catch (...) {     // torch's own errors (a sparse tensor has no bytes) and the allocator's: nothing may leave a C function
            torch::translate_exception_to_python(std::current_exception());
        }
        return nullptr;
    }
};

#define ENTRY_HOST(name, host) {#name, (PyCFunction)(void (*)(void))&Entry<&name, host>::call, METH_FASTCALL, nullptr}
#define ENTRY(name) ENTRY_HOST(name, -1)
PyMethodDef methods[] = {
    ENTRY(dream_tree_verify_attn), ENTRY(dream_draft_xattn), ENTRY_HOST(dream_visual_compress, 14), ENTRY(dream_accept_path), ENTRY(dream_accept_path_static),
    ENTRY(dream_kv_commit), ENTRY(dream_project_rows), ENTRY(dream_project_rows_multi), ENTRY(dream_spec_accept), ENTRY(dream_attention_entropy),
    ENTRY(dream_tree_expand_level), ENTRY_HOST(dream_tree_finalize, 9), {nullptr, nullptr, 0, nullptr}};
#undef ENTRY
#undef ENTRY_HOST
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__call(void) { return PyModule_Create(&module); }
