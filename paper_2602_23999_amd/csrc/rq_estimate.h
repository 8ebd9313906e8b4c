// The first stage of the cluster-local search on the matrix cores (Sections 3.3.4, 3.4.1(2)): 1-bit estimates of a 64-vector tile
// for up to 16 pairs of its cluster and their comparison with the pairs' thresholds, by one wavefront.  Shared by the
// group scan, which refines the survivors itself, and the estimate kernel of the split search, which leaves them as bits.
//
// I = <x_b, qhat> is v_mfma_f32_16x16x128_f8f6f4 with qhat as 8-bit floats (integers up to 14, exact) against the
// sign bits as 4-bit floats: a bit in place 0, 1 or 2 of a nibble IS the 4-bit float 0.5, 1 or 2, so a word of 32 sign
// bits becomes 32 operands in five instructions (eight for 16 operands as bytes), and the query's values carry the factors 2,
// 1, 0.5, 2 that make every product x_b * qhat.  All partial sums are multiples of 0.5 below 2^13: exact.
// G + f_add of every (pair, vector) is a v_mfma_f32_16x16x4_f32 over (1, G) x (f_add, 1).  What is left are five vector
// instructions each: an FMA for delta * (I - S/2), one for the estimate and one for its bound, the comparison with the threshold,
// and the addition with carry that shifts its outcome into the lane's word.  They are the operations of the kernels for
// single work items, in their order and rounding: where a threshold is met exactly, where an estimate is infinite and where
// it is not a number (such a vector is dropped), every scan keeps the same vectors.  (207 vector instructions per 16 x 64
// estimates of 128 dimensions with the sum on the vector units and a subtraction's sign for the comparison, now 107.  89, and
// searches 0 to 2 % shorter, with tau - G as one more factor of the matrix product: but then a vector whose distance ties
// with the k-th may be dropped by a rounding, and the sign of a NaN decides about it.)
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
  float ga;      // row lj of the product that gives G + f_add; k = g
  uint32_t present;  // bits of the pairs there are
  const float4* pair;  // [QM] in LDS: delta, delta * S / 2, radius of the bound, threshold (16 registers otherwise)
  uint4 cw[KC];
  float4 fa, fr, fe;  // f_add (lanes g = 0; the B operand of G + f_add in the others), f_rescale, f_err

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
    const float one = g == 1 ? 1.f : 0.f;
    fa = make_float4(one, one, one, one);
    if (g == 0) fa = factors(a, 0, tile, lj);
    fr = factors(a, 1, tile, lj);
    fe = factors(a, 2, tile, lj);
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

  // the pairs: lane lj's pair is `pp` of query q (an absent one repeats the last); `scratch`: ESTIMATE_SCRATCH bytes of LDS,
  // `table`: room for `pair` (a wave_sync follows before the first scan)
  __device__ __forceinline__ void pairs(const ScanArgs& a, int pp, int q, int np, int8_t* scratch, float4* table, int lane, float& G, float& dl) {
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
    if (lane < QM) table[lane] = make_float4(dl, 0.5f * dl * (float)a.sum_qhat[q], radius, tau);
    pair = table;
    ga = g == 0 ? 1.f : (g == 1 ? G : 0.f);
    present = 0x1111u * ((1u << min(max(np - 4 * g, 0), 4)) - 1u);
  }

  // 32 sign bits as 4-bit floats
  __device__ static __forceinline__ v8i sign_operand(uint32_t w) {
    return v8i{(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u), (int)((w >> 3) & 0x11111111u), 0, 0, 0, 0};
  }

  // Bit 4 cb + r of lane (lj, g): the bound of vector 4 lj + cb of the fetched tile is at most pair 4 g + r's threshold
  // (padding's, whose f_add is +inf, is not, and pairs that are absent have no bits).  The registers of `next` are requested as
  // soon as this tile's are used up.  (DBG: `dbg` is where the integers of this tile go, per pair)
  // (Four comparisons' masks are shifted in together, behind the two wait states that a mask needs before it is a carry.)
  template <typename Dbg>
  __device__ __forceinline__ uint32_t scan(const ScanArgs& a, int next, int lj, int g, Dbg dbg) {
    v4f base[4], acc[4];
    int mine = 4 * g;
    asm volatile("" : "+v"(mine));  // (the table is read for every tile)
    float4 p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = pair[mine + r];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const float f = one_of(cb, fa.x, fa.y, fa.z, fa.w);
      base[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ga, f, v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    if (g == 0) fa = factors(a, 0, next, lj);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        acc[cb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(qa[kc], sign_operand(one_of(cb, cw[kc].x, cw[kc].y, cw[kc].z, cw[kc].w)),
                                                                   kc == 0 ? v4f{0.f, 0.f, 0.f, 0.f} : acc[cb], 0, 4, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
      codes(a, kc, next, lj, g);
    }
    uint32_t bits = 0u;  // (the last comparison ends up in bit 0)
#pragma unroll
    for (int cb = 3; cb >= 0; --cb) {
      const float f = one_of(cb, fr.x, fr.y, fr.z, fr.w), err = one_of(cb, fe.x, fe.y, fe.z, fe.w);
      uint64_t keep[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (DBG) dbg(4 * g + r, 4 * lj + cb, (int)acc[cb][r]);
        const float est = fmaf(f, fmaf(p[r].x, acc[cb][r], -p[r].y), base[cb][r]);
        keep[r] = __builtin_amdgcn_fcmpf(fmaf(-err, p[r].z, est), p[r].w, 5);  // at most the threshold; false for a NaN
      }
      asm("s_nop 1\n\t"
          "v_addc_co_u32_e64 %0, vcc, %0, %0, %1\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\t"
          "v_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %4"
          : "+v"(bits) : "s"(keep[3]), "s"(keep[2]), "s"(keep[1]), "s"(keep[0]) : "vcc");
    }
    fr = factors(a, 1, next, lj);
    fe = factors(a, 2, next, lj);
    return bits & present;
  }
};

}  // namespace rq
