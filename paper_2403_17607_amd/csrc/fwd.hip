// Forward kernel entry: dispatch on the width and on how X is loaded; the
// instantiations are compiled in translation units of their own (fwd16.hip ..
// fwd128u.hip), the kernel itself is in fwd_kernel.h.
#include "fwd_kernel.h"

namespace ffmlp {

template <int W>
static hipError_t by_pieces(int act, int mode, const FwdArgs& a, hipStream_t s, int* g) {
  return a.in_dim % 8 == 0 ? launch_forward_w<W, 0>(act, mode, a, s, g) : launch_forward_w<W, 1>(act, mode, a, s, g);
}

hipError_t launch_forward(int width, int act, int mode, const FwdArgs& a,
                          hipStream_t s, int* grid_out) {
  switch (width) {
    case 16: return by_pieces<16>(act, mode, a, s, grid_out);
    case 32: return by_pieces<32>(act, mode, a, s, grid_out);
    case 64: return by_pieces<64>(act, mode, a, s, grid_out);
    case 128: return by_pieces<128>(act, mode, a, s, grid_out);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ffmlp
