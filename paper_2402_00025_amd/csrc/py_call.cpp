// Python calls of the GEMM entry points, without an interpreter's work around them.
//
// A decode step makes one call per linear layer, and on small matrices the GPU is done with a call
// in 3 to 5 us.  Marshalling the same arguments through ctypes and asking torch.cuda for the current
// stream took 4.6 us of host time per call on top of the launch (m = 1, n = k = 4096: 7.8 us per call
// where the C entry point called in a loop gives 4.1 us), so the host set the pace.  Here a call reads
// the tensors' addresses and the stream from torch's own C++ objects and goes straight into the
// library; the argument rules (names, defaults, tensors or raw addresses, stream None = the current
// stream) are those of the functions' signatures below, and of `_p`, `_stream` and ctypes' c_int for what
// is no plain tensor, address or integer: such arguments take the slow way through their own methods.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <ATen/PythonTorchFunctionTLS.h>

#include <pthread.h>

#include "../../include/w4a16.h"

namespace {

constexpr int kMaxPtrs = 7, kMaxInts = 5, kMaxArgs = kMaxPtrs + kMaxInts + 1;

// One entry point: its pointer arguments, then its integers, then the stream (optional).  `required`
// counts the arguments without a default; an integer left out is 0.
struct Entry {
    const char* name;
    int ptrs, ints, required;
    const char* args[kMaxArgs];
};

struct Values {
    void* p[kMaxPtrs];
    int i[kMaxInts];
    void* stream;
};

// The address of an int (its low 64 bits, as a void* argument of ctypes takes it) or of None.
bool to_address(PyObject* o, void** out)
{
    if (o == Py_None) {
        *out = nullptr;
        return true;
    }
    if (!PyLong_Check(o)) {
        PyErr_SetString(PyExc_TypeError, "cannot be converted to pointer");
        return false;
    }
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == ~0ull && PyErr_Occurred()) return false;
    *out = (void*)(uintptr_t)v;
    return true;
}

// The address a pointer argument names: a tensor's data, a raw address, None, or what data_ptr() says: also of a
// tensor's subclass, which may have its own, and while a mode looks on at the calls of tensors' methods.
bool to_pointer(PyObject* o, void** out)
{
    if (THPVariable_CheckExact(o) && !at::impl::torch_function_mode_enabled()) {
        *out = THPVariable_Unpack(o).data_ptr();
        return true;
    }
    if (o == Py_None || PyLong_Check(o)) return to_address(o, out);
    PyObject* address = PyObject_CallMethod(o, "data_ptr", nullptr);
    if (!address) return false;
    const bool ok = to_address(address, out);
    Py_DECREF(address);
    return ok;
}

bool to_int(PyObject* o, int position, int* out)
{
    unsigned long v = PyLong_AsUnsignedLongMask(o);
    if (v == (unsigned long)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        PyObject* binding = PyImport_ImportModule("paper_2402_00025_amd.binding");
        if (!binding) return false;
        PyObject* i = PyObject_CallMethod(binding, "_int", "Oi", o, position);
        Py_DECREF(binding);
        if (!i) return false;
        v = PyLong_AsUnsignedLongMask(i);
        Py_DECREF(i);
        if (v == (unsigned long)-1 && PyErr_Occurred()) return false;
    }
    *out = (int)v;
    return true;
}

// Has torch set the GPU up in this process?  It does so when it is first asked for a stream, and refuses in a child
// forked from a process that has used the GPU.
bool torch_ready = false;

bool to_stream(PyObject* o, void** out)
{
    if (!o || o == Py_None) {
        if (!torch_ready) {
            PyObject* cuda = PyImport_ImportModule("torch.cuda");
            if (!cuda) return false;
            PyObject* current = PyObject_CallMethod(cuda, "current_stream", nullptr);
            Py_DECREF(cuda);
            if (!current) return false;
            Py_DECREF(current);
            torch_ready = true;
        }
        *out = (void*)c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    if (PyLong_Check(o)) return to_address(o, out);
    PyObject* handle = PyObject_GetAttrString(o, "cuda_stream");
    if (!handle) return false;
    const bool ok = to_address(handle, out);
    Py_DECREF(handle);
    return ok;
}

bool parse(const Entry& e, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, Values* v)
{
    const int total = e.ptrs + e.ints + 1;
    if (nargs > total) {
        PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", e.name, total, nargs);
        return false;
    }
    PyObject* slot[kMaxArgs] = {};
    for (Py_ssize_t i = 0; i < nargs; ++i) slot[i] = args[i];
    const Py_ssize_t named = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
    for (Py_ssize_t i = 0; i < named; ++i) {
        PyObject* name = PyTuple_GET_ITEM(kwnames, i);
        int at = 0;
        while (at < total && PyUnicode_CompareWithASCIIString(name, e.args[at]) != 0) ++at;
        if (at == total) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", e.name, name);
            return false;
        }
        if (slot[at]) {
            PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", e.name, e.args[at]);
            return false;
        }
        slot[at] = args[nargs + i];
    }
    for (int i = 0; i < e.required; ++i)
        if (!slot[i]) {
            PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", e.name, e.args[i]);
            return false;
        }
    for (int i = 0; i < e.ptrs; ++i)
        if (!to_pointer(slot[i], &v->p[i])) return false;
    if (!to_stream(slot[total - 1], &v->stream)) return false;
    for (int i = 0; i < e.ints; ++i) {
        v->i[i] = 0;
        if (slot[e.ptrs + i] && !to_int(slot[e.ptrs + i], e.ptrs + i + 1, &v->i[i])) return false;
    }
    return true;
}

// None, or the exception that binding._check raises for a negative return code.
PyObject* result_of(int rc, const char* name)
{
    if (rc == W4A16_OK) Py_RETURN_NONE;
    PyObject* binding = PyImport_ImportModule("paper_2402_00025_amd.binding");
    if (!binding) return nullptr;
    PyObject* none = PyObject_CallMethod(binding, "_check", "is", rc, name);
    Py_DECREF(binding);
    return none;
}

template <class Call>
PyObject* call_entry(const Entry& e, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames, Call&& call)
{
    Values v;
    try {
        if (!parse(e, args, nargs, kwnames, &v)) return nullptr;
    } catch (const c10::Error& x) {
        PyErr_SetString(PyExc_RuntimeError, x.what_without_backtrace());
        return nullptr;
    } catch (const std::exception& x) {
        PyErr_SetString(PyExc_RuntimeError, x.what());
        return nullptr;
    }
    int rc;
    // (a launch can block while the queue is full: other threads go on meanwhile)
    Py_BEGIN_ALLOW_THREADS
    rc = call(v);
    Py_END_ALLOW_THREADS
    return result_of(rc, e.name);
}

#define GEMM_ARGS "A", "qweight", "scales", "qzeros", "C", "m", "n", "k", "group_size"

// name(A, qweight, scales, qzeros, C, m, n, k, group_size, split_k, stream=None)
#define SPLITK_ENTRY(name, required)                                                                                  \
    const Entry name##_entry = {#name, 5, 5, required, {GEMM_ARGS, "split_k", "stream"}};                             \
    PyObject* name##_py(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)                        \
    {                                                                                                                 \
        return call_entry(name##_entry, args, nargs, kwnames, [](const Values& v) {                                   \
            return name(v.p[0], v.p[1], v.p[2], v.p[3], v.p[4], v.i[0], v.i[1], v.i[2], v.i[3], v.i[4], v.stream);     \
        });                                                                                                           \
    }

// name(A, qweight, scales, qzeros, C, m, n, k, group_size, stream=None)
#define DP_ENTRY(name)                                                                                                \
    const Entry name##_entry = {#name, 5, 4, 9, {GEMM_ARGS, "stream"}};                                               \
    PyObject* name##_py(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)                        \
    {                                                                                                                 \
        return call_entry(name##_entry, args, nargs, kwnames, [](const Values& v) {                                   \
            return name(v.p[0], v.p[1], v.p[2], v.p[3], v.p[4], v.i[0], v.i[1], v.i[2], v.i[3], v.stream);             \
        });                                                                                                           \
    }

SPLITK_ENTRY(w4a16_gemm, 10)
SPLITK_ENTRY(w4a16_gemm_static, 10)
SPLITK_ENTRY(w8a16_gemm, 9)
SPLITK_ENTRY(w3a16_gemm, 9)
SPLITK_ENTRY(w2a16_gemm, 9)
DP_ENTRY(w4a16_gemm_dp)
DP_ENTRY(w8a16_gemm_dp)
DP_ENTRY(w3a16_gemm_dp)
DP_ENTRY(w2a16_gemm_dp)

const Entry actorder_entry = {
    "w4a16_gemm_actorder", 7, 5, 11,
    {"A", "qweight_sorted", "scales", "qzeros", "perm", "A_work", "C", "m", "n", "k", "group_size", "split_k", "stream"}};
PyObject* w4a16_gemm_actorder_py(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
{
    return call_entry(actorder_entry, args, nargs, kwnames, [](const Values& v) {
        return w4a16_gemm_actorder(v.p[0], v.p[1], v.p[2], v.p[3], v.p[4], v.p[5], v.p[6], v.i[0], v.i[1], v.i[2],
                                   v.i[3], v.i[4], v.stream);
    });
}

#define METHOD(name, signature) \
    {#name, (PyCFunction)(void (*)(void))name##_py, METH_FASTCALL | METH_KEYWORDS, #name signature "\n--\n\n"}
#define GEMM_SIGNATURE "(A, qweight, scales, qzeros, C, m, n, k, group_size, "

PyMethodDef methods[] = {
    METHOD(w4a16_gemm, GEMM_SIGNATURE "split_k, stream=None)"),
    METHOD(w4a16_gemm_static, GEMM_SIGNATURE "split_k, stream=None)"),
    METHOD(w8a16_gemm, GEMM_SIGNATURE "split_k=0, stream=None)"),
    METHOD(w3a16_gemm, GEMM_SIGNATURE "split_k=0, stream=None)"),
    METHOD(w2a16_gemm, GEMM_SIGNATURE "split_k=0, stream=None)"),
    METHOD(w4a16_gemm_dp, GEMM_SIGNATURE "stream=None)"),
    METHOD(w8a16_gemm_dp, GEMM_SIGNATURE "stream=None)"),
    METHOD(w3a16_gemm_dp, GEMM_SIGNATURE "stream=None)"),
    METHOD(w2a16_gemm_dp, GEMM_SIGNATURE "stream=None)"),
    METHOD(w4a16_gemm_actorder,
           "(A, qweight_sorted, scales, qzeros, perm, A_work, C, m, n, k, group_size, split_k=0, stream=None)"),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", "The GEMM entry points of libw4a16.so.", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__call(void)
{
    pthread_atfork(nullptr, nullptr, [] { torch_ready = false; });
    return PyModule_Create(&module);
}
