// rsr_matvec_ex for Python callers who want a new result on the current stream: the checks, the result
// and the call in one native function.  A small product is bound by what happens on the host: of
// 5.3 us for a 1024 x 1024 product the launch takes 2.7, and ctypes, torch.empty from Python and the
// attribute reads around them took 2.6.  With this function 5.8 -> 4.9 us (on a slower host), three vectors on
// 1001 x 2999 6.5 -> 4.9, one on 4488 x 3946 6.2 -> 5.0: what the launch and the kernel take.
//
// It decides nothing: whatever is not a plain strided float32 or bf16 tensor on a GPU with the shape that the handle
// asks for, and whatever fails, is left to the Python path (None), which does the same work and raises; only errors of
// Python code that torch runs underneath are passed on as they are.
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "rsr.h"

namespace {

typedef int (*Matvec)(rsr_handle_t, const void *, int, float, void *, int, int64_t, int64_t, void *);
Matvec matvec = nullptr;

PyObject *bind(PyObject *, PyObject *address) {
    matvec = reinterpret_cast<Matvec>(PyLong_AsVoidPtr(address));
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}

// product(handle, rows, cols, v, scale)
PyObject *product(PyObject *, PyObject *const *arg, Py_ssize_t n) {
    if (n != 5 || !matvec || !THPVariable_CheckExact(arg[3])) Py_RETURN_NONE;
    void *handle = PyLong_AsVoidPtr(arg[0]);
    const int64_t rows = PyLong_AsLongLong(arg[1]), cols = PyLong_AsLongLong(arg[2]);
    const double scale = PyFloat_AsDouble(arg[4]);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
    try {
        const at::Tensor &v = THPVariable_Unpack(arg[3]);
        const bool wide = v.scalar_type() == at::kFloat;
        const int64_t dim = v.dim();
        if (!v.is_cuda() || v.layout() != at::kStrided || (!wide && v.scalar_type() != at::kBFloat16) || dim < 1 ||
            dim > 2 || v.size(dim - 1) != cols || v.stride(dim - 1) != 1)
            Py_RETURN_NONE;
        const int64_t batch = dim == 2 ? v.size(0) : 1, ldv = dim == 2 ? v.stride(0) : cols;
        if (batch < 1 || batch > 65535) Py_RETURN_NONE;
        const at::TensorOptions options = at::TensorOptions().dtype(at::kFloat).device(v.device());
        at::Tensor out = dim == 2 ? at::empty({batch, rows}, options) : at::empty({rows}, options);
        const void *in = v.data_ptr();
        void *to = out.data_ptr(), *stream = c10::hip::getCurrentHIPStream().stream();
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = matvec(static_cast<rsr_handle_t>(handle), in, wide ? RSR_F32 : RSR_BF16, (float)scale, to, (int)batch,
                    ldv, rows, stream);
        Py_END_ALLOW_THREADS
        if (rc == RSR_OK) return THPVariable_Wrap(std::move(out));
    } catch (python_error &e) {  // of Python code under a call of torch, a dispatch mode's: the caller's
        e.restore();
        return nullptr;
    } catch (...) {
    }
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_O, "address of rsr_matvec_ex"},
    {"product", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(product)), METH_FASTCALL,
     "product(handle, rows, cols, v, scale): a new tensor, or None"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_rsr_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The attribute `torch` names the torch that this was compiled against; the binding compares it before the first call.
PyMODINIT_FUNC PyInit__rsr_call() {
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch", RSR_TORCH) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
