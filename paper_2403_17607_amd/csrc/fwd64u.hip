// Forward kernel instantiations for width 64, other input widths (the kernel is in fwd_kernel.h).
#include "fwd_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_forward_w<64, 1>(int act, int mode, const FwdArgs& a, hipStream_t s, int* grid_out) {
  return by_act<64, 1>(act, mode, a, s, grid_out);
}

}  // namespace ffmlp
