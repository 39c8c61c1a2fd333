// csrc/binding.cpp for tensors in host memory: its headers as they are, then the few queries of the device that it makes replaced,
// so that a test can see on the CPU what it calls, and what it does where the wrapping of a new output fails.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <new>

extern "C" {
int wraps_until_failure = 0;  // the n-th output to be wrapped fails; 0: none
}

namespace c10::hip {
struct HostStream {
    void *stream() const { return nullptr; }
};
inline HostStream host_stream(DeviceIndex) { return {}; }
inline DeviceIndex host_device() { return -1; }  // what a host tensor's get_device() answers
}  // namespace c10::hip

static PyObject *wrap_or_fail(const at::Tensor &t) {
    if (wraps_until_failure > 0 && --wraps_until_failure == 0) throw std::bad_alloc();
    return THPVariable_Wrap(t);
}

#define is_cuda is_cpu
#define current_device host_device
#define getCurrentHIPStream host_stream
#define THPVariable_Wrap wrap_or_fail
#define PyInit__binding PyInit_binding_on_host
#include "../paper_2311_09550_amd/csrc/binding.cpp"
