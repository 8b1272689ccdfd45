// Segmented backward pass entry: the plan of a net, and dispatch on the
// width; each width's instantiations are compiled in their own translation
// unit (bwds64.hip, bwds128.hip), the kernel is in bwds_kernel.h.
#include "bwds_kernel.h"

namespace ffmlp {

hipError_t bwds_plan(int width, int L, int act, int64_t M, BwdsPlan* out) {
  (void)act;
  if (width < 64) return hipErrorNotSupported;
  DeviceInfo di;
  hipError_t e = device_info(&di);
  if (e != hipSuccess) return e;
  const int most = bwds_max(width);
  const int64_t rows = kBwdsWaves * 16 * (width == 64 ? bwds_nt<64>() : bwds_nt<128>());
  BwdsPlan p;
  p.nseg = (L + most - 1) / most;
  p.base = L / p.nseg;
  p.rem = L % p.nseg;
  p.ntiles = (int)((M + rows - 1) / rows);
  // One workgroup per CU (LDS), and no more of them than the tiles need:
  // every workgroup writes a whole partial G (270 KB at width 128, 5
  // matrices), so 403 tiles run on 202 workgroups of two, not on 256.
  int64_t most_wg = di.cus < kBwdgMaxBlocks ? di.cus : kBwdgMaxBlocks;
  const int64_t per = (p.ntiles + most_wg - 1) / most_wg;
  p.grid = (int)((p.ntiles + per - 1) / per);
  *out = p;
  return hipSuccess;
}

hipError_t launch_bwds(int width, const BwdsArgs& a, hipStream_t s) {
  switch (width) {
    case 64: return launch_bwds_w<64>(a, s);
    case 128: return launch_bwds_w<128>(a, s);
    default: return hipErrorNotSupported;
  }
}

}  // namespace ffmlp
