// The packed-weight layout: which parameter a packed element holds, and
// where a parameter goes.  The buffer holds the forward layers 0 .. L-1, then
// the backward layers 1 .. L-1, then the backward layer 0 (for the input
// gradient), each as fragments [strip][k-block][lane][slot]; see common.h for
// the two orientations and the contraction orders.
#pragma once

#include "common.h"

namespace ffmlp {

// bf16 elements of one strip, of one hidden segment, of the forward output
// layer, and of the L - 1 hidden segments of one orientation.  A segment holds
// strips(rows) fragments of 512 elements per k-block, rows being the fan_out
// (forward) or fan_in (backward) of its layer, so every hidden segment has the
// same size and positions follow in closed form, whatever the depth.
struct PackSizes {
  int64_t per, nW, nO, nH;
  __device__ __forceinline__ PackSizes(const PackArgs& a) {
    per = (int64_t)((a.width + 31) / 32) * 512;
    nW = per * ((a.width + 15) / 16);
    nO = per * ((a.out_dim + 15) / 16);
    nH = (int64_t)(a.L - 1) * nW;
  }
};
__device__ __forceinline__ int64_t layer_offset(const PackArgs& a, int l) {
  return l == 0 ? 0 : (int64_t)a.in_dim * a.width + (int64_t)(l - 1) * a.width * a.width;
}

// Index of the parameter that packed element e holds, or -1 (zero padding).
__device__ __forceinline__ int64_t packed_param(const PackArgs& a, int64_t e) {
  const PackSizes z(a);
  int dir, l;
  if (e < z.nH) {
    dir = 0;
    l = (int)(e / z.nW);
    e -= (int64_t)l * z.nW;
  } else if ((e -= z.nH) < z.nO) {
    dir = 0;
    l = a.L - 1;
  } else if ((e -= z.nO) < z.nH) {
    dir = 1;
    l = 1 + (int)(e / z.nW);
    e -= (int64_t)(l - 1) * z.nW;
  } else {
    e -= z.nH;  // < strips(in_dim) strips: e < total
    dir = 1;
    l = 0;
  }
  const int fi = l == 0 ? a.in_dim : a.width, fo = l == a.L - 1 ? a.out_dim : a.width;
  const int kblocks = (a.width + 31) / 32;  // every layer is padded to the width's k-blocks
  const int slot = (int)(e & 7), lane = (int)((e >> 3) & 63);
  const int frag = (int)(e >> 9);
  const int s = frag / kblocks, kb = frag - s * kblocks;
  const int g = lane >> 4, row = 16 * s + (lane & 15);
  int pos;  // contraction index the (g, slot) pair stands for
  if (dir == 0 && l == 0)
    pos = 32 * kb + 8 * g + slot;
  else
    pos = 32 * kb + (slot < 4 ? 4 * g + slot : 16 + 4 * g + (slot - 4));
  const int f = dir == 0 ? pos : row, j = dir == 0 ? row : pos;  // W_l[f][j]
  return f < fi && j < fo ? layer_offset(a, l) + (int64_t)f * fo + j : -1;
}

// The two packed elements that hold parameter i (the inverse of the above).
__device__ __forceinline__ void param_packed(const PackArgs& a, int64_t i, int64_t& fwd, int64_t& bwd) {
  const PackSizes z(a);
  const int64_t n0 = (int64_t)a.in_dim * (a.L == 1 ? a.out_dim : a.width), nh = (int64_t)a.width * a.width;
  int l = 0;
  if (i >= n0) {
    l = 1 + (int)((i - n0) / nh);
    if (l > a.L - 1) l = a.L - 1;  // an output layer is at most that large
    i -= layer_offset(a, l);
  }
  const int fo = l == a.L - 1 ? a.out_dim : a.width;
  const int f = (int)(i / fo), j = (int)(i - (int64_t)f * fo);
  const int kblocks = (a.width + 31) / 32;
  auto at = [&](int row, int pos, bool input) -> int64_t {
    const int q = pos & 31;
    const int g = input ? q >> 3 : (q & 15) >> 2;
    const int slot = input ? q & 7 : (q & 3) + ((q >> 4) << 2);
    return ((int64_t)((row >> 4) * kblocks + (pos >> 5)) * 64 + g * 16 + (row & 15)) * 8 + slot;
  };
  fwd = (int64_t)l * z.nW + at(j, f, l == 0);
  bwd = z.nH + z.nO + (l == 0 ? z.nH : (int64_t)(l - 1) * z.nW) + at(f, j, false);
}

}  // namespace ffmlp
