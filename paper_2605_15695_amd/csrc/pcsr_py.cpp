// The per-call part of the Python binding: what binding.py does around pcsr_spmm - check two
// tensors, take their addresses and the stream's handle, call - done on the tensors' C++
// objects.  A 4 us product is bound by the host, and ctypes with a dozen attribute lookups took
// 2.5 us of the call's 5.3.  Anything but plain fp32 device tensors is left to the Python code
// (by returning NotImplemented), which knows the errors.
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using ReleaseFn = int64_t (*)(void *);
ReleaseFn g_release = nullptr;

} // namespace

namespace c10 { // where the registry is declared

// torch's allocator asks before it takes more memory from the driver: what the library keeps for
// reuse goes first where the device is low
struct PcsrGiveBack : FreeMemoryCallback {
    bool Execute() override { return g_release && g_release(hip::getCurrentHIPStream().stream()) > 0; }
};
REGISTER_FREE_MEMORY_CALLBACK("pcsr", PcsrGiveBack)

} // namespace c10

namespace {

using SpmmFn = int (*)(void *, const float *, float *, int32_t, void *);
SpmmFn g_spmm = nullptr;
PyObject *s_raw, *s_rows, *s_cols, *s_stream;

// int64 attribute; false (no exception set) if it is something else
bool int_attr(PyObject *o, PyObject *name, int64_t *v)
{
    PyObject *a = PyObject_GetAttr(o, name);
    if (!a) {
        PyErr_Clear();
        return false;
    }
    const bool ok = PyLong_Check(a);
    if (ok) *v = PyLong_AsLongLong(a);
    Py_DECREF(a);
    if (ok && *v == -1 && PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return ok;
}

inline bool usable(const at::Tensor &t, int64_t numel)
{
    return t.defined() && t.is_cuda() && t.scalar_type() == at::kFloat && t.is_contiguous() && t.numel() == numel;
}

// spmm(handle, B, C, K, stream) -> error code, or NotImplemented
PyObject *spmm(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 5 || !g_spmm || !THPVariable_Check(args[1]) || !THPVariable_Check(args[2]) || !PyLong_Check(args[3]))
        Py_RETURN_NOTIMPLEMENTED;
    int64_t raw, rows, cols, stream = 0;
    const int64_t K = PyLong_AsLongLong(args[3]);
    if (K <= 0 || K > INT32_MAX || !int_attr(args[0], s_raw, &raw) || !int_attr(args[0], s_rows, &rows) ||
        !int_attr(args[0], s_cols, &cols)) {
        PyErr_Clear();
        Py_RETURN_NOTIMPLEMENTED;
    }
    if (args[4] != Py_None) {
        if (PyLong_Check(args[4])) {
            stream = PyLong_AsLongLong(args[4]);
            if (PyErr_Occurred()) {
                PyErr_Clear();
                Py_RETURN_NOTIMPLEMENTED;
            }
        } else if (!int_attr(args[4], s_stream, &stream)) {
            Py_RETURN_NOTIMPLEMENTED;
        }
    }
    const at::Tensor &B = THPVariable_Unpack(args[1]), &C = THPVariable_Unpack(args[2]);
    if (!usable(B, cols * K) || !usable(C, rows * K)) Py_RETURN_NOTIMPLEMENTED;
    const float *b = static_cast<const float *>(B.const_data_ptr());
    float *c = static_cast<float *>(C.data_ptr());
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_spmm(reinterpret_cast<void *>(raw), b, c, (int32_t)K, reinterpret_cast<void *>(stream));
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// init(address of pcsr_spmm, address of pcsr_release_cached_if_low)
PyObject *init(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "init(spmm, release)");
        return nullptr;
    }
    void *spmm = PyLong_AsVoidPtr(args[0]), *release = PyErr_Occurred() ? nullptr : PyLong_AsVoidPtr(args[1]);
    if (PyErr_Occurred()) return nullptr;
    g_spmm = reinterpret_cast<SpmmFn>(spmm);
    g_release = reinterpret_cast<ReleaseFn>(release);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"spmm", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(spmm)), METH_FASTCALL, nullptr},
    {"init", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(init)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pcsr_py", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__pcsr_py(void)
{
    s_raw = PyUnicode_InternFromString("raw");
    s_rows = PyUnicode_InternFromString("n_rows");
    s_cols = PyUnicode_InternFromString("n_cols");
    s_stream = PyUnicode_InternFromString("cuda_stream");
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", PCSR_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
