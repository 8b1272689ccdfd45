// The delta and gradient kernel pair (bwd_kernel.h, wgrad.hip): when it is
// used, and dispatch on the width; each width's instantiations are compiled in
// their own translation unit (bwd16.hip .. bwd128.hip).
#include "bwd_kernel.h"

namespace ffmlp {

// Small batches of nets of several segments.  Each segment of bwds_kernel.h is
// a launch with some 3 us of its own (arguments, weights, first loads, the
// write of its partial G) before and after a tile, where the delta kernel
// walks all layers in one launch and the gradient kernel runs them side by
// side; and at width 128 a segment net's partial G of every workgroup (1.1 MB at
// 17 matrices) is more to reduce.  From some rows on, what the segments save
// (every delta stored and read, every activation read again) is more.
// Measured, backward and reduce of ReLU nets of 17 matrices, the segments' time
// over the pair's:
//   32 wide:  4096 rows 25 / 20 us, 32768 rows 0.97, 2^17 rows 0.58
//   64 wide:  4096 rows 41 / 29 us, 60000 rows 0.98, 2^17 rows 0.74
//   128 wide: 1024 rows 91 / 80 us, 32768 rows 1.26, 2^17 rows 0.93
// Between, over 6 to 33 matrices, the crossing moves with the number of
// segments and the activation (sigmoid's and sine's delta kernels read a value
// where ReLU's reads a mask bit; dX adds as much to both; input widths that are
// no multiple of 8 cost the pair 5% more; a seeded top with a nonlinear output
// activation, act_top, costs it up to a quarter more, most with many outputs and
// right after the forward pass: 64 wide, out 64, sigmoid outputs, 1024 rows,
// forward and backward, 11 sigmoid matrices 49 / 59 us, 11 ReLU 40 / 44, 17 ReLU
// 0.95; 128 wide, 17 sine 242 / 266, 11 ReLU, 11224 rows 152 / 166): the lines
// below lie where the two are within some 5%.  One segment only at width 32, 7
// sine matrices, whose segment spills: seeded pass, in 32, 1024 rows 17 / 14 us,
// in 3, 16384 rows 19.6 / 16.7.
bool backward_pair(int width, int L, int act, bool dx, bool act_top, int64_t M) {
  const int n = bwds_segments(width, L);
  const bool sine = act == ACT_SINE, sigmoid = act == ACT_SIGMOID;
  if (act_top && (sigmoid ? (width == 16 && n == 3) || width == 64 : sine && width == 128)) return false;
  if (width == 16) return n >= 3 && M <= (sine ? 24576 : (sigmoid ? 4096 : 8192) * (int64_t)(n - (act_top ? 2 : 1)));
  if (width == 32 && n == 1) return L == 7 && sine && M <= 16384;
  if (width == 32) return M <= (n == 2 ? (sine ? 24576 : 8192) : (sigmoid ? 16384 : 32768));
  if (width == 64 && n < 3) return n == 2 && L >= 8 && !sigmoid && !act_top && M <= 16384;
  if (width == 64) return act_top ? n >= 4 && M <= 8192 : M <= (sigmoid ? 24576 : 40960);
  return !sigmoid && n >= (sine || act_top ? 6 : (dx ? 5 : 4)) && M <= 16384 * (int64_t)(n < 8 ? n : 8);
}

hipError_t launch_backward(int width, int act, int seeded, const BwdArgs& a, hipStream_t s) {
  switch (width) {
    case 16: return launch_backward_w<16>(act, seeded, a, s);
    case 32: return launch_backward_w<32>(act, seeded, a, s);
    case 64: return launch_backward_w<64>(act, seeded, a, s);
    case 128: return launch_backward_w<128>(act, seeded, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ffmlp
