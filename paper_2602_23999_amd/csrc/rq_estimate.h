// The first stage of the cluster-local search on the matrix cores (Sections 3.3.4, 3.4.1(2)): 1-bit estimates of a 64-vector tile
// for up to 16 pairs of its cluster and their comparison with the pairs' thresholds, by one wavefront.  Shared by the
// group scan, which refines the survivors itself, and the estimate kernel of the split search, which leaves them as bits.
//
// I - S/2 = <x_b, qhat> - S/2 is v_mfma_f32_16x16x128_f8f6f4 with qhat as 8-bit floats (integers up to 14, exact) against the
// sign bits as 4-bit floats: a bit in place 0, 1 or 2 of a nibble IS the 4-bit float 0.5, 1 or 2, so a word of 32 sign
// bits becomes 32 operands in five instructions (eight for 16 operands as bytes), and the query's values carry the factors 2,
// 1, 0.5, 2 that make every product x_b * qhat.  All partial sums are multiples of 0.5 below 2^13: exact.
// The part of tau - bound that is a product of pair and vector terms, (tau - G) - f_add + f_err * radius, is a
// v_mfma_f32_16x16x4_f32 over (pair coefficients) x (vector factors).  What is left per (pair, vector) are three vector
// instructions: times delta, times f_rescale plus that, sign bit shifted into the lane's word.  (207 vector instructions per 16 x
// 64 estimates of 128 dimensions when all of it but the product of bytes was done on the vector units, now 89.)
//
// Lane (lj, g) = (lane % 16, lane / 16) works on vectors 4 lj + cb (cb = 0..3) of the tile and pairs 4 g + r (r = 0..3); its codes
// and factors are 16-byte loads, requested a tile ahead.
#pragma once
#include "rq_device.h"
#include "rq_scan_args.h"

namespace rq {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int ESTIMATE_SCRATCH = QM * 128;  // bytes of LDS

template <int W, bool DBG>
struct TileEstimator {
  static constexpr int KC = (W + 3) / 4;  // 128-dimension steps
  v8i qa[KC];
  float ta, al[4];
  v4f c0;
  uint32_t present;  // bits of the pairs there are
  uint4 cw[KC];
  float4 fx, fr;     // f_add (lanes g = 0) or f_err (the others); f_rescale

  // codes and factors of a tile
  __device__ __forceinline__ void codes(const ScanArgs& a, int kc, int tile, int lj, int g) {
    cw[kc] = *reinterpret_cast<const uint4*>(a.short_codes + ((int64_t)tile * W + min(4 * kc + g, W - 1)) * TILE + 4 * lj);
  }
  __device__ __forceinline__ float4 factors(const ScanArgs& a, int plane, int tile, int lj) const {
    return *reinterpret_cast<const float4*>(a.short_factors + ((int64_t)tile * 3 + plane) * TILE + 4 * lj);
  }
  __device__ __forceinline__ void fetch(const ScanArgs& a, int tile, int lj, int g) {
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) codes(a, kc, tile, lj, g);
    fx = factors(a, g == 0 ? 0 : 2, tile, lj);
    fr = factors(a, 1, tile, lj);
  }

  // The A operand.  Lane group g holds elements 16 g .. 16 g + 15 of the first and of the second 64 of a step (8-bit operands),
  // while the B operand's group g holds all 32 elements of word g (4-bit operands); element 8 s + n of a word is dimension
  // 4 n + s (place s of nibble n).  Words past the code's last are zero here and need not be there.
  __device__ __forceinline__ void operand(int kc, const int8_t* row, int g) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v4i v = v4i{0, 0, 0, 0};
      if (4 * kc + 2 * h < W) v = *reinterpret_cast<const v4i*>(row + 64 * h + 16 * g);
#pragma unroll
      for (int i = 0; i < 4; ++i) qa[kc][4 * h + i] = v[i];
    }
  }

  // the pairs: lane lj's pair is `pp` of query q (an absent one repeats the last); `scratch`: ESTIMATE_SCRATCH bytes of LDS
  __device__ __forceinline__ void pairs(const ScanArgs& a, int pp, int q, int np, int8_t* scratch, int lane, float& G, float& dl) {
    const int lj = lane & 15, g = lane >> 4;
    if (a.qhat_fp8) {  // (a search has the operand ready in this order: qhat_fp8_pos)
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) operand(kc, a.qhat8 + (int64_t)q * a.Dp + 128 * kc, g);
    } else {  // (the stage entry points' callers hand in bytes)
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        constexpr int LAST = (W + 1) / 2 * 64 - 128 * (KC - 1);  // bytes of the last step: the row has no more
        wave_sync();
#pragma unroll 1
        for (int r = 0; r < QM; ++r) {
          const int8_t* src = a.qhat8 + (int64_t)__builtin_amdgcn_readlane(q, r) * a.Dp + 128 * kc;
          for (int i = lane; i < (kc == KC - 1 ? LAST : 128); i += 64)
            scratch[128 * r + qhat_fp8_pos(i)] = (int8_t)qhat_fp8(src[qhat_mfma_pos(i)], i & 3);
        }
        wave_sync();
        operand(kc, scratch + 128 * lj, g);
      }
      wave_sync();
    }
    dl = a.delta[q];
    G = a.probe_G[pp];
    const float E = a.probe_E[pp], tau = a.tau[q];
    const float radius = sqrtf(fmaf(a.qerr, dl * dl, E * E));  // ||q'-c'|| widened by the rounding error of the 4-bit query
    const float half_S = 0.5f * (float)a.sum_qhat[q];
    // row lj of the product that gives (tau - G) - f_add + f_err * radius; k = g
    ta = g == 0 ? -1.f : (g == 1 ? radius : (g == 2 ? fminf(tau - G, 3.402823466e+38f) : 0.f));
    // scalars of this lane's four pairs 4 g + r, which lanes 4 g + r have
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      al[r] = __shfl(dl, 4 * g + r, 64);
      c0[r] = -__shfl(half_S, 4 * g + r, 64);
    }
    present = 0x1111u * ((1u << min(max(np - 4 * g, 0), 4)) - 1u);
  }

  // 32 sign bits as 4-bit floats
  __device__ static __forceinline__ v8i sign_operand(uint32_t w) {
    return v8i{(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u), (int)((w >> 3) & 0x11111111u), 0, 0, 0, 0};
  }

  // Bit 4 cb + r of lane (lj, g): vector 4 lj + cb of the fetched tile is NOT dropped for pair 4 g + r (padding, whose f_add is
  // +inf, is, and so are pairs that are absent).  The registers of `next` are requested as soon as this tile's are used
  // up.  (DBG: `dbg` is where the integers of this tile go, per pair)
  template <typename Dbg>
  __device__ __forceinline__ uint32_t scan(const ScanArgs& a, int next, int lj, int g, Dbg dbg) {
    v4f tt[4], acc[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const float f = one_of(cb, fx.x, fx.y, fx.z, fx.w);
      tt[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ta, g == 3 ? 0.f : (g == 2 ? 1.f : f), v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    fx = factors(a, g == 0 ? 0 : 2, next, lj);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        acc[cb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(qa[kc], sign_operand(one_of(cb, cw[kc].x, cw[kc].y, cw[kc].z, cw[kc].w)),
                                                                   kc == 0 ? c0 : acc[cb], 0, 4, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
      codes(a, kc, next, lj, g);
    }
    // the sign of tau - bound: set where the bound is above the threshold; the last comparison ends up in bit 0
    uint32_t bits = 0u;
#pragma unroll
    for (int cb = 3; cb >= 0; --cb) {
      const float f = one_of(cb, fr.x, fr.y, fr.z, fr.w);
#pragma unroll
      for (int r = 3; r >= 0; --r) {
        if (DBG) dbg(4 * g + r, 4 * lj + cb, (int)(acc[cb][r] - c0[r]));
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(fmaf(-f, al[r] * acc[cb][r], tt[cb][r])), 31);
      }
    }
    fr = factors(a, 1, next, lj);
    return ~bits & present;
  }
};

}  // namespace rq
