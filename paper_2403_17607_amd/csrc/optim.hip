// Optimizer step on fp32 master weights, then the bf16 weights the fused
// kernels read.  The paper leaves the optimizer out of its training step
// (section III-A); applications need one.  SGD, and Adam as defined by
// Kingma and Ba (2015, Algorithm 1) with bias-corrected moments; one
// thread per parameter, all state in the weights' own layout.  With a packed
// buffer the same launch re-packs the weights: a parameter's thread writes its
// bf16 value to its two packed places, and one thread per packed element
// writes the zero padding.  A launch bounds these steps (a few us for tens of
// thousands of parameters): as two kernels, update then pack, they took 2.8 us
// each and the gap between them.
#include "device.h"
#include "pack.h"

namespace ffmlp {

__global__ __launch_bounds__(256) void optim_kernel(const OptArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.n) {
    const int64_t e = i - a.n;
    if (e < a.pack.total && packed_param(a.pack, e) < 0) a.pack.dst[e] = 0;
    return;
  }
  const float g = a.G[i];
  float w = a.master[i];
  if (a.adam) {
    const float m = a.beta1 * a.m[i] + (1.f - a.beta1) * g;
    const float v = a.beta2 * a.v[i] + (1.f - a.beta2) * g * g;
    a.m[i] = m;
    a.v[i] = v;
    // lr (m / (1 - beta1^t)) / (sqrt(v / (1 - beta2^t)) + eps)
    w -= a.step_size * m / (__builtin_sqrtf(v) * a.inv_sqrt_bc2 + a.eps);
  } else {
    w -= a.lr * g;
  }
  a.master[i] = w;
  const uint16_t wb = __builtin_bit_cast(uint16_t, (__bf16)w);  // round to nearest even
  a.W[i] = wb;
  if (a.pack.total > 0) {
    int64_t fwd, bwd;
    param_packed(a.pack, i, fwd, bwd);
    a.pack.dst[fwd] = wb;
    a.pack.dst[bwd] = wb;
  }
}

hipError_t launch_optim(const OptArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(optim_kernel, dim3((unsigned)((a.n + a.pack.total + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace ffmlp
