// Segmented backward kernel instantiations for width 16 (the kernel is in
// bwdsn_kernel.h).
#include "bwdsn_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_bwds_w<16>(const BwdsArgs& a, hipStream_t s) {
  return bwds_by_len<16>(a, s);
}

}  // namespace ffmlp
