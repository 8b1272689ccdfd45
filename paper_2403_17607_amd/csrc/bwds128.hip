// Segmented backward kernel instantiations for width 128 (the kernel is in
// bwds_kernel.h).
#include "bwds_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_bwds_w<128>(const BwdsArgs& a, hipStream_t s) {
  return bwds_by_len<128>(a, s);
}

}  // namespace ffmlp
