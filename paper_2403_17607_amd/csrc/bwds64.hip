// Segmented backward kernel instantiations for width 64 (the kernel is in
// bwds_kernel.h): segments of up to 5 layers, of 3 to 5 in deeper nets.
#include "bwds_kernel.h"

namespace ffmlp {

template <>
hipError_t launch_bwds_w<64>(const BwdsArgs& a, hipStream_t s) {
  switch (a.hi - a.lo + 1) {
    case 1: return bwds_by_pos<64, 1, 0>(a, s);
    case 2: return bwds_by_pos<64, 2, 0>(a, s);
    case 3: return bwds_by_pos<64, 3, 1>(a, s);
    case 4: return bwds_by_pos<64, 4, 1>(a, s);
    case 5: return bwds_by_pos<64, 5, 1>(a, s);
    default: return hipErrorNotSupported;
  }
}

}  // namespace ffmlp
