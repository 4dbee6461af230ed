// Test helper, host code only: tensors that say they are on the device but lie in host memory, for the binding's argument
// checks without a GPU, and an entry point that throws.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdlib>
#include <new>

namespace {

int throwing_entry(...) { throw std::bad_alloc(); }

PyObject* tensor(PyObject*, PyObject* sizes)     // float32, contiguous, zeros
{
    std::vector<int64_t> shape;
    int64_t n = 1;
    for (Py_ssize_t i = 0; i < PyTuple_Size(sizes); ++i) {
        shape.push_back(PyLong_AsLongLong(PyTuple_GetItem(sizes, i)));
        n *= shape.back();
    }
    void* p = std::calloc((size_t)n, sizeof(float));
    c10::DataPtr data(p, p, [](void* q) { std::free(q); }, c10::Device(c10::DeviceType::CUDA, 0));
    c10::Storage storage(c10::Storage::use_byte_size_t(), n * sizeof(float), std::move(data), nullptr, false);
    auto impl = c10::make_intrusive<c10::TensorImpl>(std::move(storage), c10::DispatchKeySet(c10::DispatchKey::CUDA),
                                                     caffe2::TypeMeta::fromScalarType(at::kFloat));
    impl->set_sizes_contiguous(shape);
    return THPVariable_Wrap(at::Tensor(std::move(impl)));
}
PyObject* throwing(PyObject*, PyObject*) { return PyLong_FromVoidPtr(reinterpret_cast<void*>(throwing_entry)); }

PyMethodDef methods[] = {{"tensor", tensor, METH_VARARGS, nullptr}, {"throwing", throwing, METH_NOARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "device_tensor_stub", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_device_tensor_stub(void) { return PyModule_Create(&module); }
