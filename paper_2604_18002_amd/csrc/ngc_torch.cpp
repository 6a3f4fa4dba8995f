// What the CPython front reads of a tensor, from the tensor itself instead of through its Python methods.  A decode step
// reads nine tensors with some twenty method calls, each 40-90 ns (is_contiguous() parses arguments): 0.8 us of the 1.25 us that
// the front and the binding took of a call of 3.8-4.5 us.  Read here they take 0.65 us of 3.2-3.9 (a paged append 1.4 of 4.1-4.7, now
// 0.65 of 3.4-4.1): call after call decode of one small sequence 4.6 -> 4.2 us, a paged period of 32 tokens over 16 x 28 layers,
// two calls a layer-step, 8.12 -> 8.01 ms, over 4 x 8 layers 2.5 -> 2.1.
//
// Only plain tensors are read here: of torch's own class (or a Parameter), with a storage, dense, ordinary sizes, in no
// wrapper of functorch or of functionalisation, and with no torch-function mode that might want to see the method calls.
// All others, and whatever torch refuses, go back to the front, which asks the object's own methods.
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/DispatchKeySet.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ngc_torch.h"

extern "C" __attribute__((visibility("default"))) const char *ngc_torch_identity(void) noexcept { return NGC_TORCH_IDENTITY; }

extern "C" __attribute__((visibility("default"))) int ngc_read_tensor(PyObject *o, ngc_tensor *out) noexcept
{
    try {
        if (!THPVariable_CheckExact(o) || at::impl::torch_function_mode_enabled()) return 0;
        const at::Tensor &t = THPVariable_Unpack(o);
        if (!t.defined()) return 0;
        const c10::TensorImpl *const impl = t.unsafeGetTensorImpl();
        constexpr c10::DispatchKeySet wrapped({c10::DispatchKey::Python, c10::DispatchKey::Functionalize,
                                               c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                               c10::DispatchKey::BatchedNestedTensor});
        if (impl->key_set().has_any(wrapped) || impl->layout() != c10::kStrided || !impl->has_storage() ||
            impl->has_symbolic_sizes_strides() || t.is_nested())
            return 0;
        const c10::IntArrayRef sizes = t.sizes();
        out->data = t.data_ptr();
        out->sizes = sizes.data();
        out->dims = (int32_t)sizes.size();
        out->contiguous = t.is_contiguous();
        out->numel = t.numel();
        return 1;
    } catch (...) {          // torch says the same, as a Python error, to the front's own question
        return 0;
    }
}
