// Frozen two-level emitters (the paper's Bloch-equation comparison in the
// section on molecular mapping), one thread per emitter, classical RK4 with
// the field held over the step.  In atomic units, V = -mu E:
//   d rho_ee/dt = 2 V Im(rho_ge) - g1 rho_ee
//   d rho_ge/dt = (i w0 - g2) rho_ge - i V (2 rho_ee - 1)
// State planes [3][n] (structure of arrays: each plane is read with unit
// stride across the wavefront).
#include <hip/hip_runtime.h>

#include "bloch.h"

namespace msqd {

template <typename T>
__global__ __launch_bounds__(256) void bloch_kernel(BlochArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.n) bloch_emitter<T>(a, i);
}

int launch_bloch(const BlochArgs& a, bool f32, hipStream_t s) {
  if (a.n <= 0) return 0;
  const int blocks = (a.n + 255) / 256;
  if (f32)
    hipLaunchKernelGGL(bloch_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(bloch_kernel<double>, dim3(blocks), dim3(256), 0, s, a);
  return static_cast<int>(hipGetLastError());
}

}  // namespace msqd
