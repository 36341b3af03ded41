// Included ahead of csrc_host/fsa_host.cpp by tests/test_host_path.py: CPU tensors stand in for those on a GPU, and every
// output allocation is counted, those made while the interpreter lock is held also on their own.
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <torch/csrc/autograd/python_variable.h>

extern "C" {
int allocations = 0;
int allocations_with_gil = 0;
}

namespace at {
inline Tensor counted_empty(IntArrayRef size, TensorOptions options) {
    ++allocations;
    allocations_with_gil += PyGILState_Check();
    return at::empty(size, options);
}
}  // namespace at

#define empty counted_empty
#define is_cuda is_cpu
