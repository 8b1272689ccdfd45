// Segmented backward pass: the delta loop of Algorithm 2 and the weight
// gradients G_l = A_l^T D_{l+1} (arXiv 2403.17607, section III-A) of the
// layers hi .. lo of a net of any depth, with the input gradient when asked.
//
// A net's G does not fit the registers of one workgroup beyond a few
// matrices, so the layers are cut into segments of NL, run as one kernel
// each: the delta D_{hi+1} enters from memory (from the caller's dY, the
// training forward's output delta, or the segment above), the deltas inside
// the segment never leave the chip, and only D_lo is written.  Against a
// delta kernel that stores every delta and a gradient kernel that reads
// every activation and delta, the traffic per layer falls from 3 W bf16
// values written and read per row (4 W for sigmoid) to W plus 2 W / NL.
//
// A workgroup of eight waves owns tiles of 128 NT rows (persistent loop).
// Each wave carries the deltas of its own 16 NT rows through the layers in
// VGPRs (chain order, weights resident in LDS).  Per layer it stores its rows
// of D_{l+1} and A_l as they are into the LDS row tiles DT and AT; after a
// barrier every wave accumulates its fixed slice of G_l from them (transposing
// LDS reads), interleaved with the delta product of its own rows, whose
// derivative sigma'(A_l) comes from the same registers.  The activations of
// the next two layers (of this tile or the next) are in flight while a layer
// computes, so the kernel streams the stash.
#pragma once

#include "device.h"

namespace ffmlp {

enum { BWDS_RELU = 0, BWDS_SINE = 1, BWDS_OTHER = 2 };

// First element of matrix l in a buffer of all weights or gradients.
__device__ __forceinline__ int64_t g_offset(int l, int in_dim, int W) {
  return l == 0 ? 0 : (int64_t)in_dim * W + (int64_t)(l - 1) * W * W;
}

// One 16-row block per wave.  At width 64 two fit, but with one the kernel
// takes 128 registers and two workgroups share a CU: the same speed on large
// batches (training step of 9 matrices, 683354 rows: 499 us both), and twice
// the workgroups on small ones (17 matrices, 20000 rows: 109 -> 94 us).
template <int W> constexpr int bwds_nt() { return 1; }

template <int W, int NL>
struct BwdsGeom {
  static constexpr int NW = kBwdsWaves, NT = bwds_nt<W>(), SW = W / 16, KBW = (W + 31) / 32;
  static constexpr int ROWS = NW * NT * 16, KS = ROWS / 32;
  static constexpr int LF = SW * KBW;  // 1 KiB fragments of one layer
  // G slices: TK x TJ tiles of 16x16 per wave and layer.
  static constexpr int TK = W == 128 ? 2 : 1, TJ = W == 128 ? 4 : 2;
  static constexpr int JG = SW / TJ;   // waves that share a k-strip group
  static constexpr int TPW = TK * TJ;
  static constexpr size_t tiles_off() { return (size_t)NL * LF * 1024; }
  static constexpr size_t lds_bytes() { return tiles_off() + (size_t)2 * ROWS * W * 2; }
  static_assert(W >= 64 && (SW / TK) * JG == NW, "slices cover G");
};

template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
__global__ __launch_bounds__(kBwdsWaves * 64, (W == 64 ? 4 : 2)) void bwds_kernel(const BwdsArgs a) {
  using Gm = BwdsGeom<W, NL>;
  constexpr int NW = Gm::NW, NT = Gm::NT, SW = Gm::SW, KBW = Gm::KBW, KS = Gm::KS;
  constexpr int LF = Gm::LF, TK = Gm::TK, TJ = Gm::TJ, TPW = Gm::TPW;
  static_assert(TOP || !SEEDED, "dY enters at the output layer");
  constexpr int AHEAD = NL < 3 ? NL - 1 : 2;  // layers whose A is in flight while one computes
  constexpr bool XLATE = BOT && NL > (W == 128 ? 1 : 3);
  extern __shared__ u32x4 smem[];
  using RT = RowTile<W>;
  uint8_t* DT = reinterpret_cast<uint8_t*>(smem) + Gm::tiles_off();
  uint8_t* AT = DT + (size_t)Gm::ROWS * W * 2;
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
        stage_frags(smem + (size_t)i * LF * 64, a.packed0, (uint32_t)(((in_dim + 15) >> 4) * KBW), wave, NW, lane);
    } else {
      stage_frags(smem + (size_t)i * LF * 64, a.packed + (size_t)(hi - i - 1) * LF * 64, (uint32_t)LF, wave, NW, lane);
    }
  });
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 gacc[NL * TPW];
#pragma unroll
  for (int i = 0; i < NL * TPW; ++i) gacc[i] = zero4;
  const int kt0 = (wave / Gm::JG) * TK, jt0 = (wave % Gm::JG) * TJ;

  uint32_t offK[TK], offJ[TJ];  // tile read offsets of the wave's pieces
#pragma unroll
  for (int t = 0; t < TK; ++t) offK[t] = RT::read_off(li, lg, kt0 + t);
#pragma unroll
  for (int t = 0; t < TJ; ++t) offJ[t] = RT::read_off(li, lg, jt0 + t);

  struct Rows {
    int64_t row0, vr;
    int vblk;
  };
  auto rows_of = [&](int tile) {
    Rows r;
    r.row0 = (int64_t)tile * Gm::ROWS + wave * NT * 16;
    int64_t v = M - r.row0;
    r.vr = v < 0 ? 0 : (v > NT * 16 ? NT * 16 : v);
    r.vblk = (int)((r.vr + 15) / 16);
    return r;
  };
  // One [M16][F] tile image, the wave's rows of a tile, `S` strips, as
  // chain-order operands (k-block kb: strips 2 kb, 2 kb + 1).
  auto load_img = [&](const uint16_t* base, int S, const Rows& r, u32x4 (&dst)[NT][KBW]) {
    const rsrc_t d = make_rsrc(base + r.row0 * (16 * S), base ? (int64_t)r.vblk * 512 * S : 0);
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int kb = 0; kb < KBW; ++kb) {
        const u32x2 lo = bload64(d, lane * 8, 2 * kb < S ? (uint32_t)((n * S + 2 * kb) * 512) : kOOB);
        const u32x2 up = bload64(d, lane * 8, 2 * kb + 1 < S ? (uint32_t)((n * S + 2 * kb + 1) * 512) : kOOB);
        dst[n][kb] = u32x4{lo.x, lo.y, up.x, up.y};
      }
  };
  u32x4 ab[NL][NT][KBW];               // A of every layer of the segment
  u32x4 cq[NT][KBW];                   // sine: cos of the next product's layer
  u32x4 dN[SEEDED ? 1 : NT][SEEDED ? 1 : KBW];  // the next tile's D_{hi+1}
  u32x4 gq[SEEDED ? NT : 1], oq[SEEDED ? NT : 1];  // seeded: its first strip's dY and C_L
  auto load_a = [&](auto ic, int tile) {
    constexpr int i = decltype(ic)::value;
    const Rows r = rows_of(tile);
    if constexpr (BOT && i == NL - 1) {
      load_x_rows<NT, KBW>(a.X, r.row0, M, in_dim, li, lg, ab[i]);
    } else {
      load_img(a.stashA + (size_t)(hi - i - 1) * a.M16 * W, SW, r, ab[i]);
    }
  };
  auto load_cos = [&](int i, int tile) {
    if constexpr (AC == BWDS_SINE) load_img(a.stashS + (size_t)(hi - i - 1) * a.M16 * W, SW, rows_of(tile), cq);
  };
  // Seeded: strip s of dY (columns 16 s + 4 g .. + 3 of row i; fp32 rows,
  // 4-byte aligned) and of C_L.
  auto load_seed = [&](int s, const Rows& r, u32x4 (&gv)[SEEDED ? NT : 1], u32x4 (&cv)[SEEDED ? NT : 1]) {
    if constexpr (SEEDED) {
      const rsrc_t gr = make_rsrc(a.dY + r.row0 * out_dim, r.vr * out_dim * 4);
      const rsrc_t cr = make_rsrc(a.cOut + r.row0 * (16 * SO), a.cOut ? (int64_t)r.vblk * 1024 * SO : 0);
      const int j0 = s * 16 + lg * 4;
      const uint32_t eo = j0 < out_dim ? (uint32_t)((li * out_dim + j0) * 4) : kOOB;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        gv[n] = bload128(gr, eo, (uint32_t)(n * 64 * out_dim));
        cv[n] = out_act != ACT_LINEAR ? bload128(cr, lane * 16, (uint32_t)((n * SO + s) * 1024)) : u32x4{0u, 0u, 0u, 0u};
      }
    }
  };
  // What a tile's top needs, requested one tile ahead.
  auto fetch_top = [&](int tile) {
    const Rows r = rows_of(tile);
    if constexpr (SEEDED) load_seed(0, r, gq, oq);
    else load_img(a.deltaIn, SO, r, dN);
    if constexpr (!(BOT && NL == 1)) load_cos(0, tile);
  };
  auto der = [&](uint32_t half) -> float {  // sigmoid a (1 - a), sine the stored cos, linear 1
    const float v = __uint_as_float(half);
    if constexpr (AC == BWDS_SINE) return v;
    else return act == ACT_SIGMOID ? v * (1.f - v) : 1.f;
  };

  const int G = gridDim.x;
  fetch_top(blockIdx.x);
  static_for<0, AHEAD + 1>([&](auto ic) {
    if constexpr (!XLATE || decltype(ic)::value != NL - 1) load_a(ic, blockIdx.x);
  });
  drain_and_sync();  // weights in LDS

  for (int tile = blockIdx.x; tile < a.ntiles; tile += G) {
    const Rows r = rows_of(tile);
    u32x4 dA[NT][KBW], dB[NT][KBW];
    if constexpr (!SEEDED) {
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int kb = 0; kb < KBW; ++kb) dA[n][kb] = dN[n][kb];
    } else {
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int kb = 0; kb < KBW; ++kb) dA[n][kb] = u32x4{0u, 0u, 0u, 0u};
      static_for<0, SW>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if (s >= SO) return;
        u32x4 gv[NT], cv[NT];
        if constexpr (s == 0) {
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            gv[n] = gq[n];
            cv[n] = oq[n];
          }
        } else {
          load_seed(s, r, gv, cv);
        }
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          float d[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // past out_dim the load holds the next row's values
            d[q] = s * 16 + lg * 4 + q < out_dim ? __uint_as_float(gv[n][q]) : 0.f;
            if (out_act != ACT_LINEAR) {
              const float c = __uint_as_float(cv[n][q]);
              d[q] *= act_out_grad(out_act, c, act_apply(out_act, c));
            }
          }
          const uint32_t p0 = pack_bf16x2(d[0], d[1]), p1 = pack_bf16x2(d[2], d[3]);
          if constexpr (s & 1) {
            dA[n][s >> 1].z = p0;
            dA[n][s >> 1].w = p1;
          } else {
            dA[n][s >> 1].x = p0;
            dA[n][s >> 1].y = p1;
          }
        }
      });
    }

    // Layer i of the segment (l = hi - i).  Phase 1: D_{l+1} (in `cur`) and
    // A_l of the wave's rows into DT and AT.  Phase 2 (after a barrier): the
    // wave's G_l slice over the tile's rows, interleaved strip by strip with
    // D_l = (D_{l+1} W_l^T) sigma'(a_l) of its own rows into `nxt`.  A
    // barrier then frees both tiles.
    auto layer_step = [&](auto ic, const u32x4 (&cur)[NT][KBW], u32x4 (&nxt)[NT][KBW]) {
      constexpr int i = decltype(ic)::value;
      constexpr bool OUTL = TOP && i == 0;       // the output layer: SO strips of delta
      constexpr bool BOTL = BOT && i == NL - 1;  // layer 0: A is X, no further delta
      if constexpr (BOTL) mask_x_rows<NT, KBW>(a.X, r.row0, M, in_dim, li, lg, ab[i]);
      RT::template put<NT, KBW>(DT, wave * NT * 16, li, lg, cur);
      RT::template put<NT, KBW>(AT, wave * NT * 16, li, lg, ab[i]);
      __syncthreads();  // DT and AT hold the tile's rows

      constexpr int NG = KS * TPW, NS = BOTL ? 1 : SW;
      const u32x4* wl = smem + (size_t)i * LF * 64;
      u32x4 ao[TK], bo[TJ];
      static_for<0, NS>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        static_for<s * NG / NS, (s + 1) * NG / NS>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          constexpr int ks = q / TPW, u = (q % TPW) / TJ, v = q % TJ;
          if constexpr (q % TPW == 0) {
#pragma unroll
            for (int t = 0; t < TK; ++t) ao[t] = RT::read(AT, offK[t], ks);
#pragma unroll
            for (int t = 0; t < TJ; ++t)
              if (!OUTL || ((jt0 + t) & ~1) < SO) bo[t] = RT::read(DT, offJ[t], ks);
          }
          if (!OUTL || ((jt0 + v) & ~1) < SO)  // pieces 2 kb, 2 kb + 1 hold strips 2 kb, 2 kb + 1
            gacc[i * TPW + u * TJ + v] = mfma16(ao[u], bo[v], gacc[i * TPW + u * TJ + v]);
        });
        if constexpr (!BOTL) {
          u32x4 af[KBW];
#pragma unroll
          for (int kb = 0; kb < KBW; ++kb)
            if (!OUTL || 2 * kb < SO) af[kb] = wl[(s * KBW + kb) * 64 + lane];
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            f32x4 acc = zero4;
#pragma unroll
            for (int kb = 0; kb < KBW; ++kb)
              if (!OUTL || 2 * kb < SO) acc = mfma16(af[kb], cur[n][kb], acc);
            const u32x4 av = AC == BWDS_SINE ? cq[n][s >> 1] : ab[i][n][s >> 1];
            const u32x2 dv = (s & 1) ? u32x2{av.z, av.w} : u32x2{av.x, av.y};
            uint32_t p0, p1;
            if constexpr (AC == BWDS_RELU) {
              p0 = mask_halves(pack_bf16x2(acc[0], acc[1]), nonzero_halves(dv.x));
              p1 = mask_halves(pack_bf16x2(acc[2], acc[3]), nonzero_halves(dv.y));
            } else {
              p0 = pack_bf16x2(acc[0] * der(dv.x << 16), acc[1] * der(dv.x & 0xffff0000u));
              p1 = pack_bf16x2(acc[2] * der(dv.y << 16), acc[3] * der(dv.y & 0xffff0000u));
            }
            if constexpr (s & 1) {
              nxt[n][s >> 1].z = p0;
              nxt[n][s >> 1].w = p1;
            } else {
              nxt[n][s >> 1].x = p0;
              nxt[n][s >> 1].y = p1;
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      // The A that is needed AHEAD + 1 layers from here, of this tile or the
      // next, and the cos of the layer below.  In long segments X is requested
      // one layer ahead only (register budget).
      if constexpr (!XLATE || (i + 1 + AHEAD) % NL != NL - 1)
        load_a(std::integral_constant<int, (i + 1 + AHEAD) % NL>{}, i + 1 + AHEAD < NL ? tile : tile + G);
      if constexpr (XLATE && i == NL - 2) load_a(std::integral_constant<int, NL - 1>{}, tile);
      if constexpr (AC == BWDS_SINE) {
        if constexpr (i + 1 < NL && !(BOT && i + 1 == NL - 1)) load_cos(i + 1, tile);
      }
      if constexpr (i == NL - 1) {
        fetch_top(tile + G);
        if constexpr (BOTL) {
          // dX^T = W_0 D_1^T, no activation derivative, fp32 out.
          if (a.dX != nullptr) {
            const rsrc_t xr = make_rsrc(a.dX + r.row0 * in_dim, r.vr * in_dim * 4);
#pragma unroll 1
            for (int s = 0; 16 * s < in_dim; ++s) {
              u32x4 af[KBW];
#pragma unroll
              for (int kb = 0; kb < KBW; ++kb) af[kb] = wl[(s * KBW + kb) * 64 + lane];
              const int f0 = 16 * s + 4 * lg;
#pragma unroll
              for (int n = 0; n < NT; ++n) {
                f32x4 acc = zero4;
#pragma unroll
                for (int kb = 0; kb < KBW; ++kb) acc = mfma16(af[kb], cur[n][kb], acc);
                const uint32_t eo = (uint32_t)((li * in_dim + f0) * 4), so = (uint32_t)(n * 64 * in_dim);
                // four features in one store (4-byte aligned), or the last
                // few of the row one by one
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
              bstore64((s & 1) ? u32x2{nxt[n][s >> 1].z, nxt[n][s >> 1].w} : u32x2{nxt[n][s >> 1].x, nxt[n][s >> 1].y},
                       dr, lane * 8, (uint32_t)((n * SW + s) * 512));
        }
      }
      __syncthreads();  // every wave is done reading DT and AT
    };
    static_for<0, NL>([&](auto ic) {
      if constexpr ((decltype(ic)::value & 1) == 0) layer_step(ic, dA, dB);
      else layer_step(ic, dB, dA);
    });
  }

  // The workgroup's partial G, in the weights' layout (each element of G is
  // in exactly one wave's slice).  One descriptor per layer drops what is past
  // its matrix: with a branch per element this took 1300 cycles a layer, a
  // quarter of the kernel in a batch of one tile per workgroup (64 wide, 5
  // matrices, 1024 rows, backward and reduce: 13.0 -> 12.0 us; 128 wide, 17
  // matrices: 103 -> 91).
  float* part = a.partial + (size_t)blockIdx.x * (size_t)a.params;
  static_for<0, NL>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr bool BOTL = BOT && i == NL - 1;
    const int l = hi - i;
    const int fi = BOTL ? in_dim : W, fo = TOP && i == 0 ? out_dim : W;
    const rsrc_t pr = make_rsrc(part + g_offset(l, in_dim, W), (int64_t)fi * fo * 4);
#pragma unroll
    for (int u = 0; u < TK; ++u)
#pragma unroll
      for (int v = 0; v < TJ; ++v) {
        const int p = 16 * (kt0 + u) + 4 * lg, k = BOTL ? p : chain_feature(p);
        const int j = chain_feature(16 * (jt0 + v) + li);
        const uint32_t vo = j < fo ? (uint32_t)(k * fo + j) * 4 : kOOB;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          bstore32<false>(__float_as_uint(gacc[i * TPW + u * TJ + v][q]), pr, vo + (uint32_t)(q * fo * 4), 0u);
      }
  });
}

template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
struct BwdsKernel {
  static constexpr auto kern = bwds_kernel<W, NL, TOP, BOT, SEEDED, AC>;
  static constexpr size_t lds = BwdsGeom<W, NL>::lds_bytes();
};
template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
struct BwdsnKernel;  // widths 16 and 32, bwdsn_kernel.h

template <int W, int NL, bool TOP, bool BOT, bool SEEDED, int AC>
static hipError_t bwds_launch_t(const BwdsArgs& a, hipStream_t stream) {
  using K = std::conditional_t<(W <= 32), BwdsnKernel<W, NL, TOP, BOT, SEEDED, AC>,
                               BwdsKernel<W, NL, TOP, BOT, SEEDED, AC>>;
  int occ = 0;  // raises the kernel's LDS limit
  hipError_t e = kernel_occupancy(reinterpret_cast<const void*>(K::kern), kBwdsWaves * 64, K::lds, &occ);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(K::kern, dim3(a.grid), dim3(kBwdsWaves * 64), K::lds, stream, a);
  return hipGetLastError();
}

template <int W, int NL, bool TOP, bool BOT, bool SEEDED>
static hipError_t bwds_by_act(const BwdsArgs& a, hipStream_t s) {
  switch (a.act) {
    case ACT_RELU: return bwds_launch_t<W, NL, TOP, BOT, SEEDED, BWDS_RELU>(a, s);
    case ACT_SINE: return bwds_launch_t<W, NL, TOP, BOT, SEEDED, BWDS_SINE>(a, s);
    default: return bwds_launch_t<W, NL, TOP, BOT, SEEDED, BWDS_OTHER>(a, s);
  }
}

// One segment of NL layers: the whole net, its top, its bottom or its
// middle.  A training step reaches a whole net only where no one-kernel step
// covers it (one matrix, or width 128).
template <int W, int NL, bool MULTI>
static hipError_t bwds_by_pos(const BwdsArgs& a, hipStream_t s) {
  const bool top = a.hi == a.L - 1, bot = a.lo == 0, seeded = a.dY != nullptr;
  if (top && bot) {
    if (seeded) return bwds_by_act<W, NL, true, true, true>(a, s);
    if constexpr (W == 128 || NL == 1 || NL > kTrainfMaxL) return bwds_by_act<W, NL, true, true, false>(a, s);
    return hipErrorNotSupported;
  }
  if constexpr (MULTI) {
    if (top) return seeded ? bwds_by_act<W, NL, true, false, true>(a, s) : bwds_by_act<W, NL, true, false, false>(a, s);
    if (bot) return bwds_by_act<W, NL, false, true, false>(a, s);
    return bwds_by_act<W, NL, false, false, false>(a, s);
  }
  return hipErrorNotSupported;
}

// Longest segment.  Width 128: three layers' weights (96 KiB) and the two row
// tiles (64 KiB) are all of LDS.  Width 64: five layers' G and operands take the
// 128 registers that let two workgroups share a CU.  Width 32: seven layers' G
// alone is 112 registers per lane.  Width 16: nine layers' kernels take 108 to
// 165.  The sine kernels of the longest segments hold a second source value per
// element and spill (width 32, 7 matrices, up to 64 registers; width 64, 5
// matrices, 12); from some 20000 rows on they are faster all the same than the
// delta and gradient kernels (32 wide, 7 sine matrices, 50000 rows 0.98 of their
// time, 2^17 rows 0.7-0.9), below that backward_pair takes those.
// The shortest segment of a net of several: with n segments of at most
// bwds_max layers for more than (n - 1) bwds_max, each has at least
// (bwds_max + 1) / 2.
constexpr int bwds_max(int width) { return width == 128 ? 3 : (width == 64 ? 5 : (width == 32 ? 7 : 9)); }

template <int W, int NL = 1>
static hipError_t bwds_by_len(const BwdsArgs& a, hipStream_t s) {
  if constexpr (NL <= bwds_max(W)) {
    if (a.hi - a.lo + 1 == NL) return bwds_by_pos<W, NL, (2 * NL >= bwds_max(W))>(a, s);
    return bwds_by_len<W, NL + 1>(a, s);
  }
  return hipErrorNotSupported;
}

template <int W>
hipError_t launch_bwds_w(const BwdsArgs& a, hipStream_t s);

}  // namespace ffmlp
