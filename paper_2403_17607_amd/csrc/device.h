// Device-side helpers shared by the fused kernels.
#pragma once

#include <type_traits>

#include "common.h"

namespace ffmlp {

// Compile-time loop: f(std::integral_constant<int, I>) for I = B .. E-1.  Used
// where register arrays are indexed by the loop variable, so the index is a
// constant even when the body is too large for the unroller's heuristics.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Two fp32 values to packed bf16 (low half = a), round-to-nearest-even
// (gfx950 v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  bf16x2 r = __builtin_convertvector(f32x2{a, b}, bf16x2);
  return __builtin_bit_cast(uint32_t, r);
}

// Keep the computation of v at this point of the program: an empty asm
// that claims to change v, so the compiler can neither sink the work that
// produced v towards v's later uses nor drop it.  A layer's activations
// are otherwise converted only at the end of the layer, which keeps every
// strip's fp32 accumulators alive until then.
__device__ __forceinline__ void pin(uint32_t& v) { asm volatile("" : "+v"(v)); }

// ReLU of two packed bf16 values: a bf16 value is <= 0 exactly when its bit
// pattern read as int16 is <= 0, so a packed int16 max with 0 is ReLU.  It
// commutes with rounding (rounding keeps the sign), so ReLU may be applied
// after the conversion.
typedef short s16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t p) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, p), (s16x2){0, 0}));
}

// Each half of p (a non-negative bf16 value) as 0 or 1 in that half.  The
// constant 1 in both halves comes from a register: an inline constant of a
// packed instruction would give the high half 0.
__device__ __forceinline__ uint32_t nonzero_halves(uint32_t p) {
  uint32_t m;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(m) : "v"(p), "v"(0x00010001u));
  return m;
}

// p with each 16-bit half multiplied by the 0 or 1 in the same half of m.
__device__ __forceinline__ uint32_t mask_halves(uint32_t p, uint32_t m) {
  uint32_t r;
  asm("v_pk_mul_lo_u16 %0, %1, %2" : "=v"(r) : "v"(p), "v"(m));
  return r;
}

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// out += A * B on the matrix cores: 16x16 fp32 result, 32 bf16 contraction
// positions per lane group (see common.h for the lane layout).
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(
      __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ float act_apply(int act, float c) {
  switch (act) {
    case ACT_RELU: return c > 0.f ? c : 0.f;
    case ACT_SIGMOID: return 1.f / (1.f + __expf(-c));
    case ACT_SINE: return __sinf(c);
    default: return c;
  }
}

// Derivative of the output activation, from the pre-activation c and the
// fp32 output y = act(c) (both still in registers at the output layer).
__device__ __forceinline__ float act_out_grad(int act, float c, float y) {
  switch (act) {
    case ACT_RELU: return c > 0.f ? 1.f : 0.f;
    case ACT_SIGMOID: return y * (1.f - y);
    case ACT_SINE: return __cosf(c);
    default: return 1.f;
  }
}

// The training epilogue of one 16-row block of an output strip, OA the
// output activation: acc holds the pre-activations C (lane (g, i): row i,
// columns j0 .. j0 + 3), t the targets, `valid` which of the four are real
// (row < M, column < out_dim).  Returns Y as two packed bf16 pairs in y and
// the output delta scale (Y - T) sigma_out'(C) in d (0 where not valid), and
// adds (Y - T)^2 of the valid ones to loss.  Y and the loss use the fp32 Y.
template <int OA>
__device__ __forceinline__ void train_epilogue(const f32x4& acc, const u32x4& t, const bool (&valid)[4],
                                               float scale, float& loss, u32x2& y, u32x2& d) {
  float yv[4], dv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    yv[q] = act_apply(OA, acc[q]);
    const float diff = yv[q] - __uint_as_float(t[q]);
    if (valid[q]) loss += diff * diff;
    dv[q] = valid[q] ? (scale * diff) * act_out_grad(OA, acc[q], yv[q]) : 0.f;
  }
  y = u32x2{pack_bf16x2(yv[0], yv[1]), pack_bf16x2(yv[2], yv[3])};
  d = u32x2{pack_bf16x2(dv[0], dv[1]), pack_bf16x2(dv[2], dv[3])};
}

// f(std::integral_constant<int, act>{}) for a run-time activation.
template <typename F>
__device__ __forceinline__ void by_act_value(int act, F&& f) {
  if (act == ACT_LINEAR) f(std::integral_constant<int, ACT_LINEAR>{});
  else if (act == ACT_RELU) f(std::integral_constant<int, ACT_RELU>{});
  else if (act == ACT_SIGMOID) f(std::integral_constant<int, ACT_SIGMOID>{});
  else f(std::integral_constant<int, ACT_SINE>{});
}

// Derivative of a hidden activation from what the forward pass stored: the
// bf16 activation a (ReLU: a > 0, sigmoid: a (1 - a)) or, for sine, the
// stored bf16 cos(c) passed in as a.
template <int ACT>
__device__ __forceinline__ float act_hidden_grad(float a) {
  if constexpr (ACT == ACT_RELU) return a > 0.f ? 1.f : 0.f;
  else if constexpr (ACT == ACT_SIGMOID) return a * (1.f - a);
  else if constexpr (ACT == ACT_SINE) return a;
  else return 1.f;
}

template <int ACT>
__device__ __forceinline__ float act_hidden(float c) {
  if constexpr (ACT == ACT_RELU) return c > 0.f ? c : 0.f;
  else if constexpr (ACT == ACT_SIGMOID) return 1.f / (1.f + __expf(-c));
  else if constexpr (ACT == ACT_SINE) return __sinf(c);
  else return c;
}

// Buffer descriptor over [base, base + bytes) (gfx9 raw buffer, no
// swizzle).  The hardware range check makes loads past the end return 0 and
// drops stores past the end, so a wave can address its whole tile with
// 32-bit offsets and no per-row branches.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOOB = 0x80000000u;  // an offset past any descriptor's end

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, int64_t bytes) {
  const int n = bytes <= 0 ? 0 : (bytes > 0x7fffffff ? 0x7fffffff : (int)bytes);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, n, 0x00020000);
}
__device__ __forceinline__ u32x2 bload64(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ u32x4 bload128(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ uint32_t bload32(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
}
__device__ __forceinline__ uint32_t bload16(rsrc_t r, uint32_t voff, uint32_t soff) {
  return (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
}
// Stores are non-temporal (cache policy nt) by default: everything the
// forward and backward kernels store (outputs, the activation and delta
// stash, masks, dX) is read at most once, by a later kernel, so keeping it
// in L2 and the last-level cache would only evict lines that are still in
// use.  Measured on the training step: 4.7% faster at width 128 and 9% at
// width 64 (2^20 rows).  NT = false gives the default policy, whose stores
// are acknowledged sooner: a kernel that waits for all its stores at every
// layer (streamed weights) and gains nothing later uses it for inference.
constexpr int kStoreNT = 2;  // the nt bit of the buffer instructions' cache policy
template <bool NT = true>
__device__ __forceinline__ void bstore32(uint32_t v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b32(v, r, voff, soff, NT ? kStoreNT : 0);
}
template <bool NT = true>
__device__ __forceinline__ void bstore16(uint32_t v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, r, voff, soff, NT ? kStoreNT : 0);
}
template <bool NT = true>
__device__ __forceinline__ void bstore64(u32x2 v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b64(v, r, voff, soff, NT ? kStoreNT : 0);
}
template <bool NT = true>
__device__ __forceinline__ void bstore128(u32x4 v, rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, soff, NT ? kStoreNT : 0);
}

// A_1 = X of NT 16-row blocks from row0 on, in input order: lane (g, i) of
// block n gets features 32 kb + 8 g .. + 7 of row 16 n + i.  in_dim a
// multiple of 8: aligned 16-byte buffer loads, 0 past the row and past M.
template <int NT, int KBW>
__device__ __forceinline__ void load_x_aligned(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                               u32x4 (&dst)[NT][KBW]) {
  int64_t vr = M - row0;
  vr = vr < 0 ? 0 : (vr > NT * 16 ? NT * 16 : vr);
  const rsrc_t xr = make_rsrc(X + row0 * in_dim, vr * in_dim * 2);
#pragma unroll
  for (int kb = 0; kb < KBW; ++kb) {
    const int f0 = kb * 32 + lg * 8;
    const uint32_t voff = f0 < in_dim ? (uint32_t)((li * in_dim + f0) * 2) : kOOB;
#pragma unroll
    for (int n = 0; n < NT; ++n) dst[n][kb] = bload128(xr, voff, (uint32_t)(n * 32 * in_dim));
  }
}
// Other widths: rows start at any 2-byte address, so a lane's P features
// (P = 8, or 4 of a strip) come in one unaligned load.  It may read on into
// the next row; a load that would pass the end of X is moved back to end
// there.  x_piece_fix, called when the values are first used (the loads stay
// in flight until then), shifts such a piece into place and clears what is
// past in_dim or M.  XPieces holds what both need for a wave's rows.
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
template <int P>
struct XPieces {
  const uint16_t* p;  // first element of row0 (or, past M, of X's last P elements)
  int rem;            // largest element offset from p that a load may start at
  int rows;           // rows of X from row0 on, as far as they matter
  bool tiny;          // X has fewer than P elements: loaded one by one
  __device__ __forceinline__ XPieces(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int max_rows) {
    const int64_t left = M - row0;
    rows = (int)(left < 0 ? 0 : (left > max_rows + P ? max_rows + P : left));
    p = rows > 0 ? X + row0 * in_dim : X + M * in_dim - P;
    rem = rows > 0 ? rows * in_dim - P : 0;
    tiny = M * in_dim < P;
  }
};
// One lane's P features, as P / 2 dwords, from feature f0 of row r (0-based
// from row0).
template <int P, typename V, typename VU>
__device__ __forceinline__ V x_piece_load(const XPieces<P>& x, int r, int f0, int in_dim) {
  if (x.tiny) {
    V v = {};
#pragma unroll 1
    for (int q = P - 1; q >= 0; --q) {
      const uint32_t e = r < x.rows && f0 + q < in_dim ? (uint32_t)x.p[r * in_dim + f0 + q] : 0u;
#pragma unroll
      for (int d = P / 2 - 1; d > 0; --d) v[d] = (v[d] << 16) | (v[d - 1] >> 16);
      v[0] = (v[0] << 16) | e;
    }
    return v;
  }
  const int e = r * in_dim + (f0 < in_dim ? f0 : 0);
  return *reinterpret_cast<const VU*>(x.p + (e < x.rem ? e : x.rem));
}
template <int P, typename V>
__device__ __forceinline__ void x_piece_fix(const XPieces<P>& x, int r, int f0, int in_dim, bool tail, V& v) {
  if (tail) {  // wave-uniform
    const int e = r * in_dim + (f0 < in_dim ? f0 : 0), k = e - (e < x.rem ? e : x.rem);
#pragma unroll
    for (int d = 0; d < P / 2; ++d) {
      const uint32_t up = d + 1 < P / 2 ? v[d + 1 < P / 2 ? d + 1 : 0] : 0u;
      v[d] = (k & 1) ? (v[d] >> 16) | (up << 16) : v[d];
    }
#pragma unroll
    for (int h = 1; h < P / 2; h *= 2)
#pragma unroll
      for (int d = 0; d < P / 2; ++d) {
        const uint32_t up = d + h < P / 2 ? v[d + h < P / 2 ? d + h : 0] : 0u;
        v[d] = (k & (2 * h)) ? up : v[d];
      }
#pragma unroll
    for (int d = 0; d < P / 2; ++d) v[d] = (r < x.rows && k < P) ? v[d] : 0u;
  }
  const int n = in_dim - f0;  // features of this piece
#pragma unroll
  for (int d = 0; d < P / 2; ++d) v[d] &= n >= 2 * d + 2 ? 0xffffffffu : (n == 2 * d + 1 ? 0xffffu : 0u);
}
template <int NT, int KBW>
__device__ __forceinline__ void load_x_unaligned(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                                 u32x4 (&dst)[NT][KBW]) {
  const XPieces<8> x(X, row0, M, in_dim, NT * 16);
#pragma unroll
  for (int kb = 0; kb < KBW; ++kb) {
    if (32 * kb >= in_dim) {  // wave-uniform: nothing of this k-block to load
#pragma unroll
      for (int n = 0; n < NT; ++n) dst[n][kb] = u32x4{0u, 0u, 0u, 0u};
      continue;
    }
#pragma unroll
    for (int n = 0; n < NT; ++n)
      dst[n][kb] = x_piece_load<8, u32x4, u32x4_a2>(x, 16 * n + li, kb * 32 + lg * 8, in_dim);
  }
}
template <int NT, int KBW>
__device__ __forceinline__ void load_x_rows(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                            u32x4 (&dst)[NT][KBW]) {
  if ((in_dim & 7) == 0) load_x_aligned<NT, KBW>(X, row0, M, in_dim, li, lg, dst);
  else load_x_unaligned<NT, KBW>(X, row0, M, in_dim, li, lg, dst);
}
// Completes load_x_unaligned (nothing to do for multiples of 8).
template <int NT, int KBW>
__device__ __forceinline__ void mask_x_rows(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                            u32x4 (&v)[NT][KBW]) {
  if ((in_dim & 7) == 0) return;
  const XPieces<8> x(X, row0, M, in_dim, NT * 16);
  // past the end of X only in the last wave tile
  const bool tail = !x.tiny && (x.rows < NT * 16 || x.rem < (NT * 16 - 1) * in_dim + ((in_dim - 1) & ~7));
#pragma unroll
  for (int kb = 0; kb < KBW; ++kb) {
    if (32 * kb >= in_dim || (!tail && 32 * kb + 32 <= in_dim)) continue;
#pragma unroll
    for (int n = 0; n < NT; ++n) x_piece_fix<8>(x, 16 * n + li, kb * 32 + lg * 8, in_dim, tail, v[n][kb]);
  }
}

// One load per feature, for rows of few features: an unaligned 16-byte load
// takes as long as several of these.  0 past in_dim and past M.
template <int NT, int KBW>
__device__ __forceinline__ void load_x_features(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                                u32x4 (&dst)[NT][KBW]) {
  int64_t vr = M - row0;
  vr = vr < 0 ? 0 : (vr > NT * 16 ? NT * 16 : vr);
  const rsrc_t xr = make_rsrc(X + row0 * in_dim, vr * in_dim * 2);
#pragma unroll
  for (int kb = 0; kb < KBW; ++kb) {
    const int f0 = kb * 32 + lg * 8;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      uint32_t e[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        e[q] = bload16(xr, f0 + q < in_dim ? (uint32_t)((li * in_dim + f0 + q) * 2) : kOOB, (uint32_t)(n * 32 * in_dim));
      dst[n][kb] = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
  }
}

// The same in strip order: lane (g, i) of block n gets features
// 16 s + 4 g .. + 3 of row 16 n + i (the order of a tile image's strips), as
// two strips of one 32-feature operand (k-block kb: strips 2 kb, 2 kb + 1);
// W = 16 has one strip, the other half is 0.  XU 0: in_dim is known to be a
// multiple of 4; 1: not known; 2: one load per feature (see load_x_features).
template <int W, int XU, int NT, int KBW>
__device__ __forceinline__ void load_x_strips(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                              u32x4 (&dst)[NT][KBW]) {
  auto put = [&](int n, auto sc, u32x2 v) {
    constexpr int s = decltype(sc)::value;
    if constexpr (W == 16) {
      dst[n][0] = u32x4{v.x, v.y, 0u, 0u};
    } else if constexpr (s & 1) {
      dst[n][s >> 1].z = v.x;
      dst[n][s >> 1].w = v.y;
    } else {
      dst[n][s >> 1].x = v.x;
      dst[n][s >> 1].y = v.y;
    }
  };
  if constexpr (XU == 2) {
    int64_t vr = M - row0;
    vr = vr < 0 ? 0 : (vr > NT * 16 ? NT * 16 : vr);
    const rsrc_t xr = make_rsrc(X + row0 * in_dim, vr * in_dim * 2);
    static_for<0, W / 16>([&](auto sc) {
      const int f0 = 16 * decltype(sc)::value + 4 * lg;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        uint32_t e[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          e[q] = bload16(xr, f0 + q < in_dim ? (uint32_t)((li * in_dim + f0 + q) * 2) : kOOB, (uint32_t)(n * 32 * in_dim));
        put(n, sc, u32x2{e[0] | (e[1] << 16), e[2] | (e[3] << 16)});
      }
    });
  } else if (XU == 0 || (in_dim & 3) == 0) {
    int64_t vr = M - row0;
    vr = vr < 0 ? 0 : (vr > NT * 16 ? NT * 16 : vr);
    const rsrc_t xr = make_rsrc(X + row0 * in_dim, vr * in_dim * 2);
    static_for<0, W / 16>([&](auto sc) {
      const int f0 = 16 * decltype(sc)::value + 4 * lg;
#pragma unroll
      for (int n = 0; n < NT; ++n)
        put(n, sc, bload64(xr, f0 < in_dim ? (uint32_t)((li * in_dim + f0) * 2) : kOOB, (uint32_t)(n * 32 * in_dim)));
    });
  } else {
    const XPieces<4> x(X, row0, M, in_dim, NT * 16);
    static_for<0, W / 16>([&](auto sc) {
#pragma unroll
      for (int n = 0; n < NT; ++n)
        put(n, sc, x_piece_load<4, u32x2, u32x2_a2>(x, 16 * n + li, 16 * decltype(sc)::value + 4 * lg, in_dim));
    });
  }
}
template <int W, int NT, int KBW>
__device__ __forceinline__ void mask_x_strips(const uint16_t* X, int64_t row0, int64_t M, int in_dim, int li, int lg,
                                              u32x4 (&v)[NT][KBW]) {
  if ((in_dim & 3) == 0) return;
  const XPieces<4> x(X, row0, M, in_dim, NT * 16);
  const bool tail = !x.tiny && (x.rows < NT * 16 || x.rem < (NT * 16 - 1) * in_dim + ((in_dim - 1) & ~3));
#pragma unroll
  for (int s = 0; s < W / 16; ++s) {
    if (!tail && 16 * s + 16 <= in_dim) continue;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      u32x2 t = {v[n][s >> 1][2 * (s & 1)], v[n][s >> 1][2 * (s & 1) + 1]};
      x_piece_fix<4>(x, 16 * n + li, 16 * s + 4 * lg, in_dim, tail, t);
      v[n][s >> 1][2 * (s & 1)] = t.x;
      v[n][s >> 1][2 * (s & 1) + 1] = t.y;
    }
  }
}

// LDS tile of batch rows, [row][W] bf16, from which a contraction over the
// batch reads its MFMA operands: such an operand needs eight rows of one
// feature per lane, which ds_read_b64_tr_b16 gathers from row-major LDS (the
// 16 lanes of a group read four rows of 16 values, 8 bytes each, and get back
// four rows of one value each).  The waves store the operands they hold as
// they are, one 16-byte chunk c = 4 kb + g per k-block and row, so bringing
// a row block to the contraction's layout costs no arithmetic (against two
// selection-matrix MFMAs and four conversions per pair of strips).
// Position 8 c + e of a row holds, for activations and deltas (chain order),
// feature chain_feature(8 c + e); for X (input order) feature 8 c + e.
// A 16-value piece q of row r is stored at piece q ^ (r mod pieces) with its
// two chunks swapped where the next bit of r is set, so that the 16-byte stores
// of one chunk in 8 (16) rows and the reads of one piece in 4 rows per lane group
// spread over the banks.  Counted over the segmented kernels that use it, bank
// conflicts still take 6-7% of the active cycles at width 128 and 15% at 64.
template <int W>
struct RowTile {
  static constexpr int RB = W * 2, NQ = W / 16;  // bytes per row, pieces
  static constexpr int QS = NQ == 8 ? 3 : 2;
  static __device__ __forceinline__ uint32_t chunk_off(int row, int c) {
    return (uint32_t)(row * RB + ((((c >> 1) ^ (row & (NQ - 1))) << 1) | ((c & 1) ^ ((row >> QS) & 1))) * 16);
  }
  // NT blocks of 16 rows from row0 on, as MFMA operands (lane (g, i): row i).
  template <int NT, int KBW>
  static __device__ __forceinline__ void put(uint8_t* tile, int row0, int li, int lg, const u32x4 (&x)[NT][KBW]) {
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int kb = 0; kb < KBW; ++kb)
        *reinterpret_cast<u32x4*>(tile + chunk_off(row0 + 16 * n + li, 4 * kb + lg)) = x[n][kb];
  }
  // This lane's byte offset for piece q of the first 16 rows.
  static __device__ __forceinline__ uint32_t read_off(int li, int lg, int q) {
    return chunk_off(4 * lg + (li >> 2), 2 * q + ((li >> 1) & 1)) + 8 * (li & 1);
  }
  static __device__ __forceinline__ u32x2 read4(const uint8_t* p) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(
        u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p)));
  }
  // Operand of 32-row step ks: lane (g, n) gets value n of the piece, rows
  // 32 ks + 4 g + r in slots r and 32 ks + 16 + 4 g + r in slots 4 + r.
  static __device__ __forceinline__ u32x4 read(const uint8_t* tile, uint32_t off, int ks) {
    const u32x2 a = read4(tile + off + (32 * ks) * RB), b = read4(tile + off + (32 * ks + 16) * RB);
    return u32x4{a.x, a.y, b.x, b.y};
  }
};
// Feature at position p of a chain-order row.
__device__ __forceinline__ int chain_feature(int p) {
  return (p & ~31) + 16 * ((p >> 2) & 1) + 4 * ((p >> 3) & 3) + (p & 3);
}

// Asynchronous copy of nfrag 1 KiB fragments from global memory into LDS
// with direct-to-LDS loads (no registers): wave w copies fragments w,
// w + nwaves, ...; lane l of a load writes bytes 16 l .. 16 l + 15 of the
// fragment.  The data is in LDS once the issuing wave has waited for its
// vector memory counter; other waves may read it after a barrier.
__device__ __forceinline__ void stage_frags(u32x4* dst, const u32x4* src, uint32_t nfrag,
                                            int wave, int nwaves, int lane) {
  for (uint32_t f = wave; f < nfrag; f += nwaves)
    __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(src + (size_t)f * 64 + lane),
                                     (void __attribute__((address_space(3)))*)(dst + (size_t)f * 64), 16, 0, 0);
}

// Wait for every vector memory operation of this wave (direct-to-LDS loads
// included), then synchronize the workgroup.
__device__ __forceinline__ void drain_and_sync() {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
}

// Deterministic wave-wide sum (fixed butterfly order).
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace ffmlp
