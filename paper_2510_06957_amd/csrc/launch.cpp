// Python module _launch: the binding's calls on torch tensors, for the arguments that calls ordinarily have.  A short call is
// bound by the host: of the 7.0 us that Y = X W + b took from Python (M = 1, 512 x 512), 1.7 went into looking the tensors over,
// 1.4 into torch.empty and 0.7 into ctypes; here the whole call takes 4.0 us, 3.4 with Y given, of which the launch is 2.5.
//
// launch() returns None, without having done anything, for whatever is not plain -- a tensor of another class, type, layout or
// device, a shape that does not fit, a dispatch or function mode, a call that the library refuses -- and the caller goes the long
// way, which refuses what it refuses with the message that belongs to it.  An error of the GPU, which kernels of the call may have
// gone before, is raised here: nothing is launched twice.
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>

#include "tstgemm.h"

namespace {

typedef int (*Gemm)(const float *, const void *, const float *, float *, int, int, int, void *);
typedef int (*Prelu)(const float *, const void *, const float *, const float *, int, float *, int, int, int, void *);

enum Entry { kGemm, kPacked, kSigned, kNoalloc, kEntries };
Gemm g_entry[kEntries];
Prelu g_prelu;
PyObject *g_error;   // TstgemmError
PyObject *s_raw, *s_n, *s_device_index, *s_cuda_stream;

// An attribute that is an int; false (no error set) if it is not there or something else.
bool int_attr(PyObject *o, PyObject *name, unsigned long long *out)
{
    PyObject *v = PyObject_GetAttr(o, name);
    const bool ok = v != nullptr && PyLong_CheckExact(v);
    if (ok) *out = PyLong_AsUnsignedLongLong(v);
    Py_XDECREF(v);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return ok;
}

// A float32 tensor with memory of its own on device `dev`, contiguous, of torch's own class.
const at::Tensor *plain(PyObject *o, int dev)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != at::kFloat || t.layout() != at::kStrided || !t.has_storage() ||
        !t.is_contiguous() || (dev >= 0 && t.get_device() != dev))
        return nullptr;
    return &t;
}

struct WithoutGil {
    PyThreadState *state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// launch(entry, X, t, b, Y, stream, alpha) -> Y or None
PyObject *launch(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    if (n_args != 7) {
        PyErr_SetString(PyExc_TypeError, "launch(entry, X, t, b, Y, stream, alpha)");
        return nullptr;
    }
    try {
        const long entry = PyLong_AsLong(a[0]);
        unsigned long long raw = 0, n = 0, index = 0, stream = 0;
        if (entry < 0 || entry >= kEntries || g_prelu == nullptr || at::impl::PythonTorchFunctionTLS::stack_len() > 0 ||
            c10::impl::TorchDispatchModeTLS::any_modes_set() || !int_attr(a[2], s_raw, &raw) || !int_attr(a[2], s_n, &n) ||
            !int_attr(a[2], s_device_index, &index))
            Py_RETURN_NONE;
        const at::Tensor *x = plain(a[1], (int)index);
        if (x == nullptr || raw == 0 || x->dim() != 2 || x->size(0) > INT_MAX || x->size(1) > INT_MAX ||
            c10::hip::current_device() != (int)index)
            Py_RETURN_NONE;
        const int M = (int)x->size(0), K = (int)x->size(1), N = (int)n;
        const float *bias = nullptr, *alpha = nullptr;
        int alpha_count = 0;
        if (a[3] != Py_None) {
            const at::Tensor *b = plain(a[3], (int)index);
            if (b == nullptr || b->numel() != N) Py_RETURN_NONE;
            bias = static_cast<const float *>(b->data_ptr());
        }
        if (a[6] != Py_None) {
            const at::Tensor *t = plain(a[6], (int)index);
            if (t == nullptr || entry != kGemm || (t->numel() != 1 && t->numel() != N)) Py_RETURN_NONE;
            alpha = static_cast<const float *>(t->data_ptr());
            alpha_count = (int)t->numel();
        }
        if (a[5] == Py_None)
            stream = reinterpret_cast<unsigned long long>(c10::hip::getCurrentHIPStream((c10::DeviceIndex)index).stream());
        else if (!int_attr(a[5], s_cuda_stream, &stream))
            Py_RETURN_NONE;
        at::Tensor y;
        if (a[4] != Py_None) {
            const at::Tensor *t = plain(a[4], (int)index);
            if (t == nullptr || t->dim() != 2 || t->size(0) != M || t->size(1) != N) Py_RETURN_NONE;
            y = *t;
        }
        int rc;
        {
            WithoutGil released;
            if (!y.defined()) y = at::empty({M, N}, at::TensorOptions().dtype(at::kFloat).device(x->device()));
            const float *xp = static_cast<const float *>(x->data_ptr());
            float *yp = static_cast<float *>(y.data_ptr());
            const void *handle = reinterpret_cast<const void *>(raw);
            void *s = reinterpret_cast<void *>(stream);
            rc = alpha ? g_prelu(xp, handle, bias, alpha, alpha_count, yp, M, K, N, s)
                       : g_entry[entry](xp, handle, bias, yp, M, K, N, s);
        }
        if (rc == TSTGEMM_EHIP) {
            static const char *const names[kEntries] = {"tstgemm", "tstgemm_packed", "tstgemm_signed", "tstgemm_noalloc"};
            PyObject *e = PyObject_CallFunction(g_error, "is", rc, names[entry]);
            if (e != nullptr) PyErr_SetObject(g_error, e);
            Py_XDECREF(e);
            return nullptr;
        }
        if (rc != 0) Py_RETURN_NONE;
        if (a[4] != Py_None) {
            Py_INCREF(a[4]);
            return a[4];
        }
        return THPVariable_Wrap(std::move(y));
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// bind(tstgemm, tstgemm_packed, tstgemm_signed, tstgemm_noalloc, tstgemm_prelu, TstgemmError): addresses in the loaded library
PyObject *bind(PyObject *, PyObject *args)
{
    unsigned long long p[kEntries + 1];
    PyObject *error;
    if (!PyArg_ParseTuple(args, "KKKKKO", &p[0], &p[1], &p[2], &p[3], &p[4], &error)) return nullptr;
    Py_INCREF(error);
    Py_XSETREF(g_error, error);
    for (int i = 0; i < kEntries; ++i) g_entry[i] = reinterpret_cast<Gemm>(p[i]);
    g_prelu = reinterpret_cast<Prelu>(p[kEntries]);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"launch", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(launch)), METH_FASTCALL, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_launch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__launch()
{
    s_raw = PyUnicode_InternFromString("_raw");
    s_n = PyUnicode_InternFromString("N");
    s_device_index = PyUnicode_InternFromString("device_index");
    s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
    PyObject *module = PyModule_Create(&module_def);
    // what it reads of a tensor is laid out as in the torch it was built for
    if (module != nullptr && PyModule_AddStringConstant(module, "torch_version", BUILT_FOR_TORCH) < 0) Py_CLEAR(module);
    return module;
}
