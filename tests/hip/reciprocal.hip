// The z update's reciprocal (evx_rcp) on its own: out[i] = evx_rcp(x_i), x_i the float whose bits are
// first + i.  Built beside the library, loaded by tests/test_gpu_reciprocal.py.
#include <hip/hip_runtime.h>

#include "evx_device.hpp"

__global__ __launch_bounds__(256) void reciprocal_kernel(unsigned first, unsigned count, float* out) {
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  if (i < count) out[i] = evx_rcp(__uint_as_float(first + i));
}

extern "C" int evx_test_reciprocal(unsigned first, unsigned count, float* out, void* stream) {
  if (!out || count == 0 || count > (1u << 24)) return int(hipErrorInvalidValue);
  hipLaunchKernelGGL(reciprocal_kernel, dim3((count + 255) / 256), dim3(256), 0,
                     static_cast<hipStream_t>(stream), first, count, out);
  return int(hipGetLastError());
}
