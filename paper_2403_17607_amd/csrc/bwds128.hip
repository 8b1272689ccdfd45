// Segmented backward kernel instantiations for width 128 (the kernel is in
// bwds_kernel.h): segments of up to 3 layers, of 2 or 3 in deeper nets.
#include "bwds_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_bwds_w<128>(const BwdsArgs& a, hipStream_t s) {
  switch (a.hi - a.lo + 1) {
    case 1: return bwds_by_pos<128, 1, 0>(a, s);
    case 2: return bwds_by_pos<128, 2, 1>(a, s);
    case 3: return bwds_by_pos<128, 3, 1>(a, s);
    default: return hipErrorNotSupported;
  }
}

}  // namespace ffmlp
