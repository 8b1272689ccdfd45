// Segmented backward pass entry: the plan of a net, and dispatch on the
// width; each width's instantiations are compiled in their own translation
// unit (bwds16.hip .. bwds128.hip), the kernels are in bwds_kernel.h (widths
// 64 and 128) and bwdsn_kernel.h (widths 16 and 32).
#include "bwds_kernel.h"

namespace ffmlp {

int bwds_segments(int width, int L) { return (L + bwds_max(width) - 1) / bwds_max(width); }

hipError_t bwds_plan(int width, int L, int64_t M, BwdsPlan* out) {
  DeviceInfo di;
  hipError_t e = device_info(&di);
  if (e != hipSuccess) return e;
  const int64_t rows = kBwdsWaves * 16 * (width >= 64 ? 1 : 2);
  BwdsPlan p;
  p.nseg = bwds_segments(width, L);
  p.base = L / p.nseg;
  p.rem = L % p.nseg;
  p.ntiles = (int)((M + rows - 1) / rows);
  // One workgroup per CU (LDS or registers); two at widths 16 and 64, where
  // that leaves each at least two tiles (a first tile runs on cold caches).
  // And no more of them than the tiles need: every workgroup writes a whole
  // partial G (270 KB at width 128, 5 matrices), so 403 tiles run on 202
  // workgroups of two, not on 256.
  const int64_t two = (width == 16 || width == 64) && p.ntiles >= 4 * (int64_t)di.cus;
  const int64_t fit = (int64_t)di.cus * (two ? 2 : 1);
  const int64_t most_wg = fit < kBwdgMaxBlocks ? fit : kBwdgMaxBlocks;
  const int64_t per = (p.ntiles + most_wg - 1) / most_wg;
  p.grid = (int)((p.ntiles + per - 1) / per);
  *out = p;
  return hipSuccess;
}

hipError_t launch_bwds(int width, const BwdsArgs& a, hipStream_t s) {
  switch (width) {
    case 16: return launch_bwds_w<16>(a, s);
    case 32: return launch_bwds_w<32>(a, s);
    case 64: return launch_bwds_w<64>(a, s);
    case 128: return launch_bwds_w<128>(a, s);
    default: return hipErrorNotSupported;
  }
}

}  // namespace ffmlp
