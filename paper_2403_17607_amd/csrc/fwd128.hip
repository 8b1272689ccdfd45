// Forward kernel instantiations for width 128, X rows of whole 16-byte pieces (the kernel is in fwd_kernel.h).
#include "fwd_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_forward_w<128, 0>(int act, int mode, const FwdArgs& a, hipStream_t s, int* grid_out) {
  return by_act<128, 0>(act, mode, a, s, grid_out);
}

}  // namespace ffmlp
