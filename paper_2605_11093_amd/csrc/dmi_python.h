// Between the two halves of the binding's native marshalling: _dmi_python (arguments, calls; no torch) and _dmi_python_torch
// (reads tensors).
#pragma once
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "dmi.h"

#ifndef DMI_HEADER_DIGEST
#define DMI_HEADER_DIGEST 0     // of the dmi.h this was built with; the build sets it
#endif

struct dmi_py_tensor {
    void *data;
    uint64_t bytes;             // elements times their size
    uint32_t dtype;             // DMI_DTYPE_* of a source, 0: none of them
    int32_t dim;
    int64_t shape[2], stride[2];        // of a matrix
};

// False: not exactly a torch.Tensor, or one without an address or plain sizes (no Python error is left behind).
typedef bool (*dmi_py_reader)(PyObject *o, dmi_py_tensor *t);
#define DMI_PY_READER "dmi_py_reader"
