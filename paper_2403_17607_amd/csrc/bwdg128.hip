// Fused backward kernel for width 128: which nets it covers, and its
// instantiations (the kernel is in bwdg_kernel.h).
#include "bwdg_kernel.h"

namespace ffmlp {

bool backward_fused_supported(int width, int L, int act, int out_dim) {
  return width == 128 && L >= 2 && L <= kBwdgMaxL && act == ACT_RELU && out_dim <= 16;  // register budget
}

hipError_t launch_backward_fused(int L, int seeded, const BwdgArgs& a, hipStream_t s, int* grid_out) {
  return bwdg_by_l<128, 1>(L, seeded, a, s, grid_out);
}

}  // namespace ffmlp
