// Segmented backward kernel instantiations for width 64 (the kernel is in
// bwds_kernel.h).
#include "bwds_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_bwds_w<64>(const BwdsArgs& a, hipStream_t s) {
  return bwds_by_len<64>(a, s);
}

}  // namespace ffmlp
