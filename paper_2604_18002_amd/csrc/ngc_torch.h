// Between the CPython front (ngc_host.cpp, which knows no torch) and its reader of tensors (ngc_torch.cpp).
#pragma once
#include <Python.h>
#include <stdint.h>

struct ngc_tensor {
    void *data;
    const int64_t *sizes;      // the tensor's own, while it is not changed
    int64_t numel;
    int32_t dims;
    int32_t contiguous;
};

// 1: *out is filled.  0: ask the object's methods; no Python error is set.
typedef int (*ngc_read_tensor_fn)(PyObject *o, ngc_tensor *out);

// The torch that the reader was compiled against, as torch_identity() in _build.py writes it: it reads torch's structures
// where that one has them, so it serves no other.
typedef const char *(*ngc_torch_identity_fn)(void);
