// Fused backward kernel entry: which calls it covers, and dispatch on the
// width; each width's instantiations are compiled in their own translation
// unit (bwdg64.hip, bwdg128.hip), the kernel itself is in bwdg_kernel.h.
#include "bwdg_kernel.h"

namespace ffmlp {

// Without the input gradient, 2 to 5 matrices.  Width 128: ReLU nets with one
// output strip (register budget).  Width 64: seeded passes with X rows of whole
// 8-byte pieces.  There the segments (bwds_kernel.h) have some 2 us more before
// their first tile, and this kernel more registers from 3 matrices on (one
// workgroup per CU), so the segments take large batches.  Backward and reduce,
// segments against this kernel (us): ReLU, out 3: 2 matrices 1024 rows 8.2 /
// 6.7, 10^6 rows 64 / 60; 3 matrices 1024 rows 9.7 / 8.6, 2^17 rows 23.2 / 22.4,
// 2^18 rows 32 / 35; 5 matrices 1024 rows 12.8 / 10.9, 2^17 rows 34.3 / 33.7; sine: 3
// matrices 1024 rows 10.1 / 8.9, 2^16 rows 18.3 / 17.1, 10^5 rows equal.  Input
// widths that are no multiple of 4 gain less than 5% at 1024 rows and lose from
// 40000 on.  dY of several strips that are not whole is loaded by element, which
// costs large batches more than they gain (2 matrices, out 26, 65536 rows 1.09 of
// the segments' time, 10^6 rows 1.2-1.3).
bool backward_fused_supported(int width, int L, int act, int in_dim, int out_dim, bool seeded, int64_t M) {
  if (L < 2 || L > kBwdgMaxL) return false;
  if (width == 128) return act == ACT_RELU && out_dim <= 16;
  if (width != 64 || !seeded || in_dim % 4 != 0) return false;
  if (out_dim > 16 && out_dim % 4 != 0 && M > 1 << 15) return false;
  if (L == 2) return true;
  return M <= (act == ACT_RELU ? 1 << 17 : 1 << 16);
}

hipError_t launch_backward_fused(int width, int L, int out_dim, int seeded, const BwdgArgs& a, hipStream_t s,
                                 int* grid_out) {
  switch (width) {
    case 64: return launch_backward_fused_w<64>(L, out_dim, seeded, a, s, grid_out);
    case 128: return launch_backward_fused_w<128>(L, out_dim, seeded, a, s, grid_out);
    default: return hipErrorNotSupported;
  }
}

}  // namespace ffmlp
