// Segmented backward pass for widths 16 and 32 (see bwds_kernel.h for the
// segments): here a whole layer's G is one (width 16) or four (width 32)
// 16x16 tiles, so every wave keeps the segment's G in registers and contracts
// over its own two 16-row blocks only.  No LDS tile and no barrier in the
// tile loop; LDS holds the segment's weights, and at the end the waves' G is
// added through it in a fixed order.  The inputs of the next three layers (of
// this tile or the next) are in flight while a layer computes.
#pragma once

#include "bwds_kernel.h"

namespace ffmlp {

template <int W, int NL>
struct BwdsnGeom {
  static constexpr int NW = kBwdsWaves, NT = 2, SW = W / 16;
  static constexpr int ROWS = NW * NT * 16;
  static constexpr int LF = SW;        // 1 KiB fragments of one layer (one k-block)
  static constexpr int TPW = SW * SW;  // G tiles of one layer
  static constexpr int RL = NW / TPW;                // layers per pass of the final sum: a tile per wave
  static constexpr int RT = (NL < RL ? NL : RL) * TPW;  // tiles of a pass
  static constexpr size_t red_bytes() { return (size_t)NW * RT * 1024; }
  static constexpr size_t lds_bytes() {
    return (size_t)NL * LF * 1024 > red_bytes() ? (size_t)NL * LF * 1024 : red_bytes();
  }
  static_assert(W <= 32, "narrow segmented backward");
};

// The seeded kernel of whole 16-wide sine nets of 4 matrices takes 133 registers
// by itself and is held to the 128 that let two workgroups share a CU: 500000
// rows 0.81-0.92 of the time.  (The 6-layer top segment, 132 registers, spills 2
// and loses up to 5%.)
template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
constexpr int bwdsn_min_waves() {
  return W == 16 && AC == BWDS_SINE && NL == 4 && TOP && BOT && SEEDED ? 4 : 2;
}

template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
__global__ __launch_bounds__(kBwdsWaves * 64, (bwdsn_min_waves<W, NL, TOP, BOT, SEEDED, AC>()))
void bwdsn_kernel(const BwdsArgs a) {
  using Gm = BwdsnGeom<W, NL>;
  constexpr int NW = Gm::NW, NT = Gm::NT, SW = Gm::SW, LF = Gm::LF, TPW = Gm::TPW;
  static_assert(TOP || !SEEDED, "dY enters at the output layer");
  constexpr int AHEAD = NL < 4 ? NL - 1 : 3;  // layers whose inputs are in flight while one computes
  extern __shared__ u32x4 smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int li = lane & 15, lg = lane >> 4;
  const int64_t M = a.M;
  const int in_dim = a.in_dim, out_dim = a.out_dim, act = a.act, out_act = a.out_act;
  const int hi = a.hi;
  const int SO = TOP ? (out_dim + 15) >> 4 : SW;  // strips of the delta entering the segment

  // Weights of the segment's layers, slot i layer hi - i; at the bottom the
  // last slot holds layer 0's, which only the input gradient reads.
  static_for<0, NL>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (BOT && i == NL - 1) {
      if (a.dX != nullptr)
        stage_frags(smem + (size_t)i * LF * 64, a.packed0, (uint32_t)((in_dim + 15) >> 4), wave, NW, lane);
    } else {
      stage_frags(smem + (size_t)i * LF * 64, a.packed + (size_t)(hi - i - 1) * LF * 64, (uint32_t)LF, wave, NW, lane);
    }
  });
  // Selection matrices: an MFMA of an operand whose lane (g, i) holds row i
  // with one of these 0/1 matrices transposes its strip 0 or 1 exactly.
  u32x4 sel0 = {0u, 0u, 0u, 0u}, sel1 = {0u, 0u, 0u, 0u};
  {
    const int q = li - 4 * lg;
    if (q >= 0 && q < 4) {
      const uint32_t one = 0x3F80u << (16 * (q & 1));
      if (q < 2) {
        sel0.x = one;
        sel1.z = one;
      } else {
        sel0.y = one;
        sel1.w = one;
      }
    }
  }
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 gacc[NL * TPW];
#pragma unroll
  for (int i = 0; i < NL * TPW; ++i) gacc[i] = zero4;

  struct Rows {
    int64_t row0, vr;
    int vblk;
  };
  auto rows_of = [&](int tile) {
    Rows r;
    r.row0 = ((int64_t)tile * NW + wave) * NT * 16;
    int64_t v = M - r.row0;
    r.vr = v < 0 ? 0 : (v > NT * 16 ? NT * 16 : v);
    r.vblk = (int)((r.vr + 15) / 16);
    return r;
  };
  // The wave's rows of an [M16][16 S] tile image; both strips form one
  // operand (width 16: the second half stays 0).
  auto load_img = [&](const uint16_t* base, int S, const Rows& r, u32x4 (&dst)[NT][1]) {
    const rsrc_t d = make_rsrc(base + r.row0 * (16 * S), base ? (int64_t)r.vblk * 512 * S : 0);
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const u32x2 lo = bload64(d, lane * 8, (uint32_t)(n * S * 512));
      u32x2 up = {0u, 0u};
      if constexpr (SW == 2) up = bload64(d, lane * 8, S > 1 ? (uint32_t)((n * S + 1) * 512) : kOOB);
      dst[n][0] = u32x4{lo.x, lo.y, up.x, up.y};
    }
  };
  u32x4 ab[NL][NT][1];                              // A of every layer
  u32x4 cq[AC == BWDS_SINE ? NL : 1][NT][1];        // sine: the cos of every product's layer
  u32x4 dN[NT][1];                                  // the next tile's D_{hi+1}
  u32x4 gq[SEEDED ? SW : 1][NT], oq[SEEDED ? SW : 1][NT];  // seeded: its dY and C_L
  auto load_layer = [&](auto ic, int tile) {
    constexpr int i = decltype(ic)::value;
    const Rows r = rows_of(tile);
    if constexpr (BOT && i == NL - 1) {
      load_x_strips<W, 1, NT, 1>(a.X, r.row0, M, in_dim, li, lg, ab[i]);
    } else {
      load_img(a.stashA + (size_t)(hi - i - 1) * a.M16 * W, SW, r, ab[i]);
      if constexpr (AC == BWDS_SINE) load_img(a.stashS + (size_t)(hi - i - 1) * a.M16 * W, SW, r, cq[i]);
    }
  };
  auto fetch_top = [&](int tile) {
    const Rows r = rows_of(tile);
    if constexpr (SEEDED) {
      const rsrc_t gr = make_rsrc(a.dY + r.row0 * out_dim, r.vr * out_dim * 4);
      const rsrc_t cr = make_rsrc(a.cOut + r.row0 * (16 * SO), a.cOut ? (int64_t)r.vblk * 1024 * SO : 0);
#pragma unroll
      for (int s = 0; s < SW; ++s) {
        if (s >= SO) break;
        const int j0 = s * 16 + lg * 4;
        const uint32_t eo = j0 < out_dim ? (uint32_t)((li * out_dim + j0) * 4) : kOOB;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          gq[s][n] = bload128(gr, eo, (uint32_t)(n * 64 * out_dim));
          if (out_act != ACT_LINEAR) oq[s][n] = bload128(cr, lane * 16, (uint32_t)((n * SO + s) * 1024));
        }
      }
    } else {
      load_img(a.deltaIn, SO, r, dN);
    }
  };
  auto der = [&](uint32_t half) -> float {  // sigmoid a (1 - a), sine the stored cos, linear 1
    const float v = __uint_as_float(half);
    if constexpr (AC == BWDS_SINE) return v;
    else return act == ACT_SIGMOID ? v * (1.f - v) : 1.f;
  };

  const int G = gridDim.x;
#pragma unroll
  for (int s = 0; s < (SEEDED ? SW : 1); ++s)
#pragma unroll
    for (int n = 0; n < NT; ++n) gq[s][n] = oq[s][n] = u32x4{0u, 0u, 0u, 0u};
  fetch_top(blockIdx.x);
  static_for<0, AHEAD + 1>([&](auto ic) { load_layer(ic, blockIdx.x); });
  drain_and_sync();  // weights in LDS

  for (int tile = blockIdx.x; tile < a.ntiles; tile += G) {
    const Rows r = rows_of(tile);
    u32x4 dA[NT], dB[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      if constexpr (!SEEDED) {
        dA[n] = dN[n][0];
      } else {
        dA[n] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int s = 0; s < SW; ++s) {
          float d[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // past out_dim the load holds the next row's values
            d[q] = s * 16 + lg * 4 + q < out_dim ? __uint_as_float(gq[s][n][q]) : 0.f;
            if (out_act != ACT_LINEAR) {
              const float c = __uint_as_float(oq[s][n][q]);
              d[q] *= act_out_grad(out_act, c, act_apply(out_act, c));
            }
          }
          dA[n][2 * s] = pack_bf16x2(d[0], d[1]);
          dA[n][2 * s + 1] = pack_bf16x2(d[2], d[3]);
        }
      }
    }

    // Layer i of the segment (l = hi - i): G_l += A_l^T D_{l+1} over the
    // wave's rows (slot q of both operands: row 4 g + q of block 0, slot
    // 4 + q the same row of block 1), then D_l = (D_{l+1} W_l^T) sigma'(a_l).
    auto layer_step = [&](auto ic, const u32x4 (&cur)[NT], u32x4 (&nxt)[NT]) {
      constexpr int i = decltype(ic)::value;
      constexpr bool BOTL = BOT && i == NL - 1;
      if constexpr (BOTL) mask_x_strips<W, NT, 1>(a.X, r.row0, M, in_dim, li, lg, ab[i]);
      u32x4 dop[SW];
#pragma unroll
      for (int j = 0; j < SW; ++j) {
        const f32x4 o0 = mfma16(cur[0], j ? sel1 : sel0, zero4), o1 = mfma16(cur[1], j ? sel1 : sel0, zero4);
        dop[j] = u32x4{pack_bf16x2(o0[0], o0[1]), pack_bf16x2(o0[2], o0[3]), pack_bf16x2(o1[0], o1[1]),
                       pack_bf16x2(o1[2], o1[3])};
      }
#pragma unroll
      for (int t = 0; t < SW; ++t) {
        const f32x4 o0 = mfma16(ab[i][0][0], t ? sel1 : sel0, zero4), o1 = mfma16(ab[i][1][0], t ? sel1 : sel0, zero4);
        const u32x4 aop = {pack_bf16x2(o0[0], o0[1]), pack_bf16x2(o0[2], o0[3]), pack_bf16x2(o1[0], o1[1]),
                           pack_bf16x2(o1[2], o1[3])};
#pragma unroll
        for (int j = 0; j < SW; ++j) gacc[i * TPW + t * SW + j] = mfma16(aop, dop[j], gacc[i * TPW + t * SW + j]);
      }
      const u32x4* wl = smem + (size_t)i * LF * 64;
      if constexpr (!BOTL) {
#pragma unroll
        for (int s = 0; s < SW; ++s) {
          const u32x4 af = wl[s * 64 + lane];
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const f32x4 acc = mfma16(af, cur[n], zero4);
            const u32x4 av = AC == BWDS_SINE ? cq[AC == BWDS_SINE ? i : 0][n][0] : ab[i][n][0];
            const u32x2 dv = s ? u32x2{av.z, av.w} : u32x2{av.x, av.y};
            if constexpr (AC == BWDS_RELU) {
              nxt[n][2 * s] = mask_halves(pack_bf16x2(acc[0], acc[1]), nonzero_halves(dv.x));
              nxt[n][2 * s + 1] = mask_halves(pack_bf16x2(acc[2], acc[3]), nonzero_halves(dv.y));
            } else {
              nxt[n][2 * s] = pack_bf16x2(acc[0] * der(dv.x << 16), acc[1] * der(dv.x & 0xffff0000u));
              nxt[n][2 * s + 1] = pack_bf16x2(acc[2] * der(dv.y << 16), acc[3] * der(dv.y & 0xffff0000u));
            }
          }
        }
        if constexpr (SW == 1) {
#pragma unroll
          for (int n = 0; n < NT; ++n) nxt[n].z = nxt[n].w = 0u;
        }
      }
      // The inputs that are needed AHEAD + 1 layers from here, of this tile or the next.
      load_layer(std::integral_constant<int, (i + 1 + AHEAD) % NL>{}, i + 1 + AHEAD < NL ? tile : tile + G);
      if constexpr (i == NL - 1) {
        fetch_top(tile + G);
        if constexpr (BOTL) {
          // dX^T = W_0 D_1^T, no activation derivative, fp32 out.
          if (a.dX != nullptr) {
            const rsrc_t xr = make_rsrc(a.dX + r.row0 * in_dim, r.vr * in_dim * 4);
#pragma unroll
            for (int s = 0; s < SW; ++s) {
              if (16 * s >= in_dim) break;
              const u32x4 af = wl[s * 64 + lane];
              const int f0 = 16 * s + 4 * lg;
#pragma unroll
              for (int n = 0; n < NT; ++n) {
                const f32x4 acc = mfma16(af, cur[n], zero4);
                const uint32_t eo = (uint32_t)((li * in_dim + f0) * 4), so = (uint32_t)(n * 64 * in_dim);
                if ((in_dim & 3) == 0 || f0 + 4 <= in_dim) {
                  bstore128(__builtin_bit_cast(u32x4, acc), xr, f0 < in_dim ? eo : kOOB, so);
                } else {
#pragma unroll
                  for (int q = 0; q < 4; ++q)
                    bstore32(__float_as_uint(acc[q]), xr, f0 + q < in_dim ? eo + 4 * q : kOOB, so);
                }
              }
            }
          }
        } else {
          // D_lo for the segment below
          const rsrc_t dr = make_rsrc(a.deltaNext + r.row0 * W, (int64_t)r.vblk * 32 * W);
#pragma unroll
          for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int s = 0; s < SW; ++s)
              bstore64(u32x2{nxt[n][2 * s], nxt[n][2 * s + 1]}, dr, lane * 8, (uint32_t)((n * SW + s) * 512));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    static_for<0, NL>([&](auto ic) {
      if constexpr ((decltype(ic)::value & 1) == 0) layer_step(ic, dA, dB);
      else layer_step(ic, dB, dA);
    });
  }

  // The waves' G added in a fixed order through LDS (the weights are no
  // longer read), RL layers at a time so that every thread adds one piece of
  // four; the workgroup writes one partial in the weights' layout.  One layer
  // at a time, with a branch per element, took two barriers and a fifth of
  // a small batch's whole time (backward and reduce, 1024 rows: 16
  // wide, 9 matrices 10.2 -> 8.2 us; 32 wide, 11 matrices 20.7 -> 17.0).
  f32x4* red = reinterpret_cast<f32x4*>(smem);
  float* part = a.partial + (size_t)blockIdx.x * (size_t)a.params;
  constexpr int RL = Gm::RL, RT = Gm::RT;
  static_for<0, (NL + RL - 1) / RL>([&](auto pc) {
    constexpr int i0 = decltype(pc)::value * RL, ni = NL - i0 < RL ? NL - i0 : RL;
    __syncthreads();
    static_for<0, ni * TPW>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      red[(wave * RT + t) * 64 + lane] = gacc[i0 * TPW + t];
    });
    __syncthreads();
    const int i = i0 + wave / TPW, t = wave % TPW;
    if (i < NL) {
      f32x4 s = zero4;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[(w * RT + wave) * 64 + lane];
      const int l = hi - i;
      const int fi = l == 0 ? in_dim : W, fo = l == a.L - 1 ? out_dim : W;
      const rsrc_t pr = make_rsrc(part + g_offset(l, in_dim, W), (int64_t)fi * fo * 4);
      const int k = 16 * (t / SW) + 4 * lg, j = 16 * (t % SW) + li;
      const uint32_t vo = j < fo ? (uint32_t)(k * fo + j) * 4 : kOOB;
#pragma unroll
      for (int q = 0; q < 4; ++q) bstore32<false>(__float_as_uint(s[q]), pr, vo + (uint32_t)(q * fo * 4), 0u);
    }
  });
}

template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
struct BwdsnKernel {
  static constexpr auto kern = bwdsn_kernel<W, NL, TOP, BOT, SEEDED, AC>;
  static constexpr size_t lds = BwdsnGeom<W, NL>::lds_bytes();
};

}  // namespace ffmlp
