// The part of the binding's native marshalling that reads torch tensors, a module of its own: loaded when a call brings a
// tensor, and torch is there for certain.
#include "dmi_python.h"

#include <torch/csrc/autograd/python_variable.h>

namespace {

bool read_tensor(PyObject *o, dmi_py_tensor *t)
{
    if (!THPVariable_CheckExact(o)) return false;
    try {
        const at::Tensor &x = THPVariable_Unpack(o);
        t->data = x.data_ptr();
        t->bytes = (uint64_t)x.numel() * x.element_size();
        t->dim = (int32_t)x.dim();
        switch (x.scalar_type()) {
        case at::kBFloat16: t->dtype = DMI_DTYPE_BF16; break;
        case at::kHalf: t->dtype = DMI_DTYPE_FP16; break;
        case at::kFloat: t->dtype = DMI_DTYPE_FP32; break;
        default: t->dtype = 0;
        }
        for (int i = 0; i < 2 && t->dim == 2; i++) { t->shape[i] = x.size(i); t->stride[i] = x.stride(i); }
        return true;
    } catch (...) {             // (no storage, no plain sizes: the general function says what is wrong)
        return false;
    }
}

PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_dmi_python_torch", "reads torch tensors for _dmi_python", -1, nullptr,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dmi_python_torch(void)
{
    PyObject *m = PyModule_Create(&module_def);
    if (m && PyModule_AddObject(m, "reader", PyCapsule_New(reinterpret_cast<void *>(read_tensor), DMI_PY_READER, nullptr)) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
