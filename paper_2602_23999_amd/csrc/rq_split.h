// fp32 products on the bf16 matrix cores (coarse scores).  A number is the sum of three bf16 pieces, x = x1 + x2 + x3 with
// |x2| <= 2^-9 |x| and |x3| <= 2^-18 |x| (24 bits are in them), and of the nine products of two numbers the six that are not below
// 2^-26 of the result are summed in fp32, small ones first.  Six v_mfma_f32_32x32x16_bf16 do the work of eight
// v_mfma_f32_32x32x2_f32 in less than half their time.
// Every score is accumulated over k in steps of 16 in this order, whatever kernel computes it, so that it does not depend on
// the batch it is computed in.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rq {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

struct Split8 { bf16x8 p[3]; };  // eight numbers in pieces

__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{a, b}), bf16x2));
}
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  uint4 w[3];
  uint32_t* o[3] = {&w[0].x, &w[1].x, &w[2].x};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const uint32_t v = bf16_pair(a, b);
      o[p][i] = v;
      a -= __uint_as_float(v << 16);
      b -= __uint_as_float(v & 0xffff0000u);
    }
  }
  Split8 s;
#pragma unroll
  for (int p = 0; p < 3; ++p) s.p[p] = __builtin_bit_cast(bf16x8, w[p]);
  return s;
}

// [list][query] += 16 steps of k of 32 lists x 32 queries, in two sums, which are independent chains of matrix instructions (one
// chain of six waited for itself half of the time)
struct SplitSum { floatx16 lo, hi; };
__device__ __forceinline__ void split_mma(const bf16x8 (&c)[3], const Split8& q, SplitSum& s) {
  s.lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[2], q.p[0], s.lo, 0, 0, 0);
  s.hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[1], q.p[0], s.hi, 0, 0, 0);
  s.lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[0], q.p[2], s.lo, 0, 0, 0);
  s.hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[0], q.p[1], s.hi, 0, 0, 0);
  s.lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[1], q.p[1], s.lo, 0, 0, 0);
  s.hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[0], q.p[0], s.hi, 0, 0, 0);
}

}  // namespace rq
