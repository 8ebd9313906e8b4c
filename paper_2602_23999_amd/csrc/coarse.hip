// Coarse scores (Section 3.3.2): s_q 1^T + 1 s_c^T - 2 Q' C^T, or -Q' C^T, with the products of rq_split.h, and the smallest
// score of every 32 lists, which lets the probe selection read a few percent of the matrix instead of all of it.
#include "rq_device.h"
#include "rq_split.h"

namespace rq {

// Centroid pieces in the order the matrix instruction takes them: [tile of 32 lists][16 dimensions][piece][lane], 16 bytes
// each, lane l holding list l % 32, dimensions 8 (l / 32) .. + 7 of the step.  Lists past the last are zero.  Behind them
// the squared norms, padded to whole tiles.
__global__ __launch_bounds__(64) void centroid_pieces_kernel(const float* __restrict__ ct, const float* __restrict__ csq, int nlist,
                                                            int steps, uint4* __restrict__ out) {
  const int tile = blockIdx.x, lane = threadIdx.x, c = 32 * tile + (lane & 31);
  if (blockIdx.y == 0 && lane < 32) reinterpret_cast<float*>(out + (int64_t)gridDim.x * steps * 3 * 64)[c] = c < nlist ? csq[c] : 0.f;
  for (int s = blockIdx.y; s < steps; s += gridDim.y) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = c < nlist ? ct[(int64_t)(16 * s + 8 * (lane >> 5) + i) * nlist + c] : 0.f;
    const Split8 p = split8(x);
#pragma unroll
    for (int j = 0; j < 3; ++j) out[(((int64_t)tile * steps + s) * 3 + j) * 64 + lane] = __builtin_bit_cast(uint4, p.p[j]);
  }
}

constexpr int TROW = 36;  // floats of a query's row of a tile in LDS (padded: 8 rows of a 16-byte column lie in different banks)

// One 32-list tile's scores of 32 queries: the lane has those of its query, register r of list 8 (r / 4) + 4 (lane / 32) + r % 4.
// They go out through `lds` (32 rows of TROW floats of this wavefront's own), 128 contiguous bytes per query (16 bytes at a time,
// as the registers have them: 1.7 TB/s).  Returns the query's smallest.
struct TileNorms { float4 v[4]; };  // of the lane's 16 lists
__device__ __forceinline__ TileNorms tile_norms(const float* __restrict__ norms, int tile, int half) {
  TileNorms t;
#pragma unroll
  for (int g = 0; g < 4; ++g) t.v[g] = *reinterpret_cast<const float4*>(norms + 32 * tile + 8 * g + 4 * half);
  return t;
}
template <bool L2>
__device__ __forceinline__ float put_scores(const SplitSum& sum, const TileNorms& norms, int tile, int nlist, int lane, int64_t m0,
                                            int64_t nq, float rv, float* __restrict__ scores, float* lds) {
  const int half = lane >> 5;
  float least = INFINITY;
  wave_sync();
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int n = 32 * tile + 8 * g + 4 * half;
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a = sum.hi[4 * g + i] + sum.lo[4 * g + i];
      v[i] = L2 ? rv + one_of(i, norms.v[g].x, norms.v[g].y, norms.v[g].z, norms.v[g].w) - 2.0f * a : -a;
      least = n + i < nlist ? fminf(least, v[i]) : least;
    }
    *reinterpret_cast<float4*>(lds + (lane & 31) * TROW + 8 * g + 4 * half) = make_float4(v[0], v[1], v[2], v[3]);
  }
  wave_sync();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 8 * i + (lane >> 3), n = 32 * tile + 4 * (lane & 7);
    const float4 v = *reinterpret_cast<const float4*>(lds + r * TROW + 4 * (lane & 7));
    float* to = scores + (m0 + r) * nlist + n;
    if (m0 + r < nq) {
      if ((nlist & 3) == 0 && n + 3 < nlist) {
        *reinterpret_cast<float4*>(to) = v;
      } else {
        if (n < nlist) to[0] = v.x;
        if (n + 1 < nlist) to[1] = v.y;
        if (n + 2 < nlist) to[2] = v.z;
        if (n + 3 < nlist) to[3] = v.w;
      }
    }
  }
  return fminf(least, __shfl_xor(least, 32, 64));
}

// A wavefront has 32 queries, their pieces of S steps (16 S dimensions) in registers.  SHARE (many queries): the four wavefronts
// of a workgroup have 128 queries and go through the same lists, whose pieces come through LDS, a tile ahead; otherwise they
// have the same 32 queries and every fourth tile each, straight from memory.  ONE: the S steps are the whole contraction, so
// the queries' pieces are made once per workgroup; else NT tiles are accumulated together, over chunks of S steps.
// What bounds it: the matrix cores (6 x 32 cycles per 32 x 32 x 16), then the write of the scores.  6000 x 8192 x 128: the fp32
// kernel took 175 us.
template <bool L2, int S, bool ONE, bool SHARE>
__global__ __launch_bounds__(256) void coarse_kernel(const float* __restrict__ q_rot, const v4i* __restrict__ pieces, int64_t nq,
                                                    int nlist, int D, int tiles_per_block, const float* __restrict__ rowv,
                                                    float* __restrict__ scores, float* __restrict__ tmin) {
  constexpr int NT = ONE ? 1 : 2, STAGE = S * 3 * 64;  // 16-byte words of a tile's chunk
  __shared__ v4i buf[SHARE ? 2 : 1][SHARE ? STAGE : 1];
  __shared__ __align__(16) float rows[4][32 * TROW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int n_tiles = (nlist + 31) / 32, steps = D / 16, chunks = ONE ? 1 : steps / S;
  const int64_t m = SHARE ? (int64_t)blockIdx.x * 128 + 32 * wave + (lane & 31) : (int64_t)blockIdx.x * 32 + (lane & 31);
  const bool row_ok = m < nq;
  const float* src = q_rot + (row_ok ? m : 0) * D + 8 * half;
  const int tile0 = (int)blockIdx.y * tiles_per_block + (SHARE ? 0 : wave), tile1 = min(((int)blockIdx.y + 1) * tiles_per_block, n_tiles);
  constexpr int TSTEP = SHARE ? 1 : 4;
  const float rv = L2 && row_ok ? rowv[m] : 0.f;
  const int64_t m0 = m - (lane & 31);
  float* lds = &rows[wave][0];
  float* mins = tmin != nullptr ? tmin + (row_ok ? m : 0) * n_tiles : nullptr;

  const float* norms = reinterpret_cast<const float*>(pieces + (int64_t)n_tiles * steps * 3 * 64);
  Split8 qp[S];
  auto load_queries = [&](int chunk) {
    float x[S][8];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const float* p = src + (chunk * S + s) * 16;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(p + 4 * i);
        x[s][4 * i] = v.x; x[s][4 * i + 1] = v.y; x[s][4 * i + 2] = v.z; x[s][4 * i + 3] = v.w;
      }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) qp[s] = split8(x[s]);
  };
  auto chunk_at = [&](int tile, int chunk) { return pieces + ((int64_t)min(tile, n_tiles - 1) * steps + chunk * S) * 3 * 64; };
  auto multiply = [&](const v4i* from, SplitSum& acc) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      bf16x8 c[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) c[p] = __builtin_bit_cast(bf16x8, from[(s * 3 + p) * 64 + lane]);
      split_mma(c, qp[s], acc);
    }
    if (SHARE) {
      // (a step's pieces are read from LDS while the step before is multiplied: left alone, the compiler reads them where it
      // needs them and waits)
      __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (s + 1 < S) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
      }
    }
  };
  if (ONE) load_queries(0);
  if constexpr (SHARE) {
    constexpr int PER = (STAGE + 255) / 256;
    v4i ahead[PER];
    auto request = [&](int tile, int chunk) {
      const v4i* p = chunk_at(tile, chunk);
#pragma unroll
      for (int i = 0; i < PER; ++i) ahead[i] = p[(i + 1) * 256 <= STAGE ? i * 256 + tid : min(i * 256 + tid, STAGE - 1)];
    };
    auto stash = [&](int b) {
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if ((i + 1) * 256 <= STAGE || i * 256 + tid < STAGE) buf[b][i * 256 + tid] = ahead[i];
    };
    request(tile0, 0);
    stash(0);
    __syncthreads();
    int b = 0;
    float4 least4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int t = tile0; t < tile1; t += NT) {
      SplitSum acc[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[j].lo = acc[j].hi = floatx16{0};
      TileNorms cn;
      if (L2 && ONE) cn = tile_norms(norms, t, half);
      for (int ch = 0; ch < chunks; ++ch) {
        if (!ONE) load_queries(ch);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          // the stage after this one: the next tile of the group, the group's first at the next chunk, the next group's first
          const bool group_done = j + 1 == NT, chunk_done = group_done && ch + 1 == chunks;
          request(chunk_done ? t + NT : (group_done ? t : t + j + 1), chunk_done ? 0 : (group_done ? ch + 1 : ch));
          // (the requests stay ahead of the products and the stores behind them: left alone, both end up at the end)
          __builtin_amdgcn_sched_barrier(0);
          multiply(buf[b], acc[j]);
          __builtin_amdgcn_sched_barrier(0);
          stash(b ^ 1);  // (last read before the previous barrier)
          __syncthreads();
          b ^= 1;
        }
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (t + j >= tile1) break;
        if (L2 && !ONE) cn = tile_norms(norms, t + j, half);
        const float least = put_scores<L2>(acc[j], cn, t + j, nlist, lane, m0, nq, rv, scores, lds);
        // (four tiles' minima are written together)
        least4 = make_float4(least4.y, least4.z, least4.w, least);
        if (mins != nullptr && row_ok && half == 0) {
          if ((n_tiles & 3) == 0 && ((t + j) & 3) == 3 && t + j >= tile0 + 3) *reinterpret_cast<float4*>(mins + t + j - 3) = least4;
          else if ((n_tiles & 3) != 0 || t + j + 4 - ((t + j) & 3) > tile1 || ((t + j) & ~3) < tile0) mins[t + j] = least;
        }
      }
    }
  } else {
    for (int t = tile0; t < tile1; t += TSTEP) {
      SplitSum acc;
      acc.lo = acc.hi = floatx16{0};
      TileNorms cn;
      if (L2) cn = tile_norms(norms, t, half);
      for (int ch = 0; ch < chunks; ++ch) {
        if (!ONE) load_queries(ch);
        multiply(chunk_at(t, ch), acc);
      }
      const float least = put_scores<L2>(acc, cn, t, nlist, lane, m0, nq, rv, scores, lds);
      if (mins != nullptr && row_ok && half == 0) mins[t] = least;
    }
  }
}

// 16-byte words of the centroid pieces and the norms behind them
int64_t centroid_pieces_words(int nlist, int D) { return (int64_t)((nlist + 31) / 32) * ((D / 16) * 3 * 64 + 8); }

int launch_centroid_pieces(const float* ct, const float* csq, int nlist, int D, uint4* pieces, hipStream_t st) {
  hipLaunchKernelGGL(centroid_pieces_kernel, dim3((unsigned)((nlist + 31) / 32), (unsigned)std::min(D / 16, 64)), dim3(64), 0, st, ct,
                     csq, nlist, D / 16, pieces);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

template <bool L2, int S, bool ONE>
static int launch_coarse_s(const rabitq_index* ix, const float* q_rot, const float* sq_norm, int64_t nq, float* scores, float* tmin,
                           hipStream_t st) {
  const int nlist = ix->nlist, n_tiles = (nlist + 31) / 32;
  // A workgroup of 128 queries re-reads the lists' pieces a quarter as often; with fewer queries than give 512 of them (at two
  // tiles each) the chip is better filled by workgroups of 32 queries.
  const int64_t rows = (nq + 127) / 128;
  const bool share = rows * ((n_tiles + 1) / 2) >= 512;
  if (share) {
    // about 1536 workgroups (three times what runs at once), at least two tiles each
    int tpb = (int)std::max<int64_t>(2, (int64_t)n_tiles * rows / 1536);
    if (!ONE) tpb = (tpb + 1) / 2 * 2;
    if (rows > 0x7fffffff || (n_tiles + tpb - 1) / tpb > 65535) { set_error("coarse scores: matrix too large"); return RABITQ_EINVAL; }
    hipLaunchKernelGGL((coarse_kernel<L2, S, ONE, true>), dim3((unsigned)rows, (unsigned)((n_tiles + tpb - 1) / tpb)), dim3(256), 0, st,
                       q_rot, reinterpret_cast<const v4i*>(ix->centroid_pieces), nq, nlist, ix->dim, tpb, sq_norm, scores, tmin);
  } else {
    const int64_t rows32 = (nq + 31) / 32;
    hipLaunchKernelGGL((coarse_kernel<L2, S, ONE, false>), dim3((unsigned)rows32, (unsigned)((n_tiles + 3) / 4)), dim3(256), 0, st, q_rot,
                       reinterpret_cast<const v4i*>(ix->centroid_pieces), nq, nlist, ix->dim, 4, sq_norm, scores, tmin);
  }
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

int launch_coarse(const rabitq_index* ix, const float* q_rot, const float* sq_norm, int64_t nq, float* scores, float* tmin,
                  hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
#define RQ_C(S_, ONE_)                                                                                      \
  return ix->metric == RABITQ_L2 ? launch_coarse_s<true, S_, ONE_>(ix, q_rot, sq_norm, nq, scores, tmin, st) \
                                 : launch_coarse_s<false, S_, ONE_>(ix, q_rot, sq_norm, nq, scores, tmin, st)
  switch (ix->dim / 16) {
    case 2: RQ_C(2, true);
    case 4: RQ_C(4, true);
    case 6: RQ_C(6, true);
    case 8: RQ_C(8, true);
    case 60: RQ_C(6, false);
    default: RQ_C(8, false);  // 16, 32, 48, 64
  }
#undef RQ_C
}

}  // namespace rq
