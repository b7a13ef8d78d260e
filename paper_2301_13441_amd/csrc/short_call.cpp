// predict() and predict_leaves() with a buffer of their own, as one native call: the checks of X, the output tensor,
// the current stream, the launch and the views.  A small batch is a few microseconds of GPU time, and the same steps
// one by one in Python were what a call took (1,000 rows, 10 trees of depth 4: 9.3 us, 5 of them on the GPU).
//
// A CPython extension on torch's C++ interface.  It knows nothing of the library but the address of the entry point it
// is given, forest_predict, forest_predict_leaves or linear_predict, which share a signature.  What it does not take
// (anything but a plain contiguous float32 device tensor, batches of `max_rows` rows or more, active torch function or
// dispatch modes) it declines, and the caller goes the general way, whose checks raise the errors.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using Predict = int (*)(const void *handle, const void *X, int64_t n_rows, void *out, void *stream);

// What a call returns: bits of `parts`.
enum { SCORES = 1, LABELS = 2, LEAVES = 4 };

// call(entry point, handle, X, n_features, columns, parts, max_rows): columns are a model's outputs, or its trees for
// leaf ids.  Returns (scores, labels), the leaf ids, the entry point's error code, or None where it declines.
PyObject *call(PyObject *, PyObject *const *args, Py_ssize_t n_args)
{
    HANDLE_TH_ERRORS
    if (n_args != 7) {
        PyErr_SetString(PyExc_TypeError, "call takes 7 arguments");
        return nullptr;
    }
    PyObject *x = args[2];
    const auto predict = reinterpret_cast<Predict>(PyLong_AsVoidPtr(args[0]));
    const void *handle = PyLong_AsVoidPtr(args[1]);
    const int64_t n_features = PyLong_AsLongLong(args[3]), columns = PyLong_AsLongLong(args[4]);
    const long parts = PyLong_AsLong(args[5]);
    const int64_t max_rows = PyLong_AsLongLong(args[6]);
    if (PyErr_Occurred()) return nullptr;
    if (!predict || !THPVariable_CheckExact(x) || at::impl::PythonTorchFunctionTLS::stack_len() > 0 ||
        c10::impl::TorchDispatchModeTLS::any_modes_set())
        Py_RETURN_NONE;
    const at::Tensor &X = THPVariable_Unpack(x);
    if (!X.is_cuda() || X.scalar_type() != at::kFloat || X.layout() != at::kStrided || !X.has_storage() || X.dim() != 2)
        Py_RETURN_NONE;
    const int64_t n = X.size(0);
    if (X.size(1) != n_features || n < 1 || n >= max_rows || !X.is_contiguous()) Py_RETURN_NONE;

    const at::TensorOptions floats = at::TensorOptions().device(X.device()).dtype(at::kFloat);
    at::Tensor out;
    if (parts == SCORES) out = at::empty({n, columns}, floats);
    else if (parts == LABELS) out = at::empty({n}, floats.dtype(at::kInt));
    else if (parts == LEAVES) out = at::empty({n, columns}, floats.dtype(at::kInt));
    else out = at::empty({n * (columns + 1)}, floats);  // scores, then labels, as the entry point lays them out
    const void *from = X.data_ptr();
    void *to = out.data_ptr(), *stream = c10::hip::getCurrentHIPStream(X.get_device()).stream();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = predict(handle, from, n, to, stream);
    Py_END_ALLOW_THREADS
    if (rc != 0) return PyLong_FromLong(rc);
    if (parts == LEAVES) return THPVariable_Wrap(std::move(out));
    at::Tensor scores, labels;
    if (parts == SCORES) {
        scores = std::move(out);
    } else if (parts == LABELS) {
        labels = std::move(out);
    } else {
        scores = out.as_strided({n, columns}, {columns, 1}, 0);
        labels = out.view(at::kInt).as_strided({n}, {1}, n * columns);
    }
    PyObject *pair = PyTuple_New(2);
    if (!pair) return nullptr;
    const at::Tensor *part[2] = {&scores, &labels};
    for (int i = 0; i < 2; ++i) {
        PyObject *o = part[i]->defined() ? THPVariable_Wrap(*part[i]) : Py_NewRef(Py_None);
        if (!o) {
            Py_DECREF(pair);
            return nullptr;
        }
        PyTuple_SET_ITEM(pair, i, o);
    }
    return pair;
    END_HANDLE_TH_ERRORS
}

PyMethodDef METHODS[] = {
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(call)), METH_FASTCALL,
     "call(entry point, handle, X, n_features, columns, parts, max_rows)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef MODULE = {PyModuleDef_HEAD_INIT, "_short_call", nullptr, -1, METHODS, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__short_call() { return PyModule_Create(&MODULE); }
