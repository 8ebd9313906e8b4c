// Device-side index construction (Section 3.2): k-means in the rotated space, assignment,
// normalisation with respect to the centroid, RaBitQ quantisation by the two-phase grid
// search over the rescaling factor, factors, and the tiled index layout.
#include <vector>

#include "rq_device.h"

namespace rq {

__device__ inline float wave_sum_f32(float v) {
  const uint32_t r = wave_reduce_u32(__builtin_bit_cast(uint32_t, v), [](uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b));
  });
  return __builtin_bit_cast(float, r);
}
__device__ inline float wave_max_f32(float v) {
  const uint32_t r = wave_reduce_u32(__builtin_bit_cast(uint32_t, v), [](uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)));
  });
  return __builtin_bit_cast(float, r);
}

// rows[i] = src[(i * stride_num) / stride_den]  (strided training subset / initial centroids)
__global__ void gather_rows_kernel(const float* __restrict__ src, int64_t n_src, int64_t n_dst, int D,
                                   float* __restrict__ dst) {
  const int64_t total = n_dst * D;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / D;
    const int64_t s = (r * n_src) / n_dst;
    dst[i] = src[s * D + (i - r * D)];
  }
}

// ct[d][c] = c_rows[c][d], csq[c] = ||c||^2 (summed in the order of the dimensions).  A thread's row arrives 32 values at a time
// (D is a multiple of 32): the chain of dependent loads was all its time.  (512 x 128: 21 us -> 4.3)
__global__ __launch_bounds__(64) void transpose_centroids_kernel(const float* __restrict__ c_rows, int nlist, int D,
                                                                 float* __restrict__ ct, float* __restrict__ csq) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  if (c >= nlist) return;
  float s = 0.f;
  for (int d0 = 0; d0 < D; d0 += 32) {
    float4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(c_rows + (int64_t)c * D + d0 + 4 * u);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ct[(int64_t)(d0 + 4 * u + i) * nlist + c] = x[i];
        s += x[i] * x[i];
      }
    }
  }
  csq[c] = s;
}

// nearest centroid of each row from the best of every 32 or 64 (launch_gemm_nearest), ties to the lower id; 16 lanes a row
__global__ __launch_bounds__(256) void nearest_of_parts_kernel(const uint64_t* __restrict__ keys, int64_t rows, int parts,
                                                              int32_t* __restrict__ out) {
  const int l = threadIdx.x & 15;
  const int64_t r = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const uint64_t* row = keys + min(r, rows - 1) * parts;
  uint64_t best = KEY_NONE;
  for (int p = l; p < parts; p += 16) best = min(best, row[p]);
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) best = min(best, (uint64_t)__shfl_xor(best, d, 16));
  if (l == 0 && r < rows) out[r] = (int32_t)(uint32_t)best;
}

// Lloyd update: one wavefront per cluster and 64 dimensions sums the members in list order (deterministic); an empty cluster keeps
// its centroid.  The order makes every sum a chain, so the longest list decides: its rows are asked for 32 ahead of the additions.
// (128-d, 512 lists: 43 us a pass over 50 000 rows with one row in flight -> 6)
__global__ __launch_bounds__(64) void centroid_update_kernel(const float* __restrict__ x, const int32_t* __restrict__ off,
                                                             const int32_t* __restrict__ members, int D,
                                                             float* __restrict__ c_rows) {
  constexpr int AHEAD = 32;
  const int c = blockIdx.x, lane = threadIdx.x;
  const int s = off[c], e = off[c + 1];
  if (e == s) return;
  const float inv = 1.0f / (float)(e - s);
  const int d = blockIdx.y * 64 + lane;
  const int dl = min(d, D - 1);
  float acc = 0.f;
  for (int i0 = s; i0 < e; i0 += 64) {
    const int32_t mem = members[min(i0 + lane, e - 1)];
#pragma unroll
    for (int h = 0; h < 64; h += AHEAD) {
      if (i0 + h >= e) break;
      float v[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) v[u] = x[(int64_t)__builtin_amdgcn_readlane(mem, h + u) * D + dl];  // (past the end: the last member)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (i0 + h + u < e) acc += v[u];
    }
  }
  if (d < D) c_rows[(int64_t)c * D + d] = acc * inv;
}

__global__ void cluster_layout_kernel(const int32_t* __restrict__ off, int nlist, int32_t* __restrict__ csize) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < nlist) csize[c] = off[c + 1] - off[c];
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// f_add planes of the short factors start at +inf (padding), everything else at 0
__global__ void init_short_factors_kernel(float* p, int64_t n_tiles) {
  const int64_t total = n_tiles * 3 * TILE;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = ((i / TILE) % 3 == 0) ? INFINITY : 0.f;
}

struct EncodeArgs {
  const float* xr;          // [N][D] rotated vectors
  const float* c_rows;      // [nlist][D] rotated centroids
  const int32_t* off;       // [nlist+1] CSR over stored vectors
  const int32_t* members;   // [N] vector ids in cluster order
  const int32_t* tile_off;  // [nlist+1]
  int64_t n;
  int64_t p0;               // first position of this launch
  int D, B, F, LW, nlist, metric;
  float eps0;
  uint32_t* short_codes;
  float* short_factors;
  uint32_t* long_codes;
  float* long_factors;
  int32_t* ids;
};

// ---------------------------------------------------------------------------------
// One wavefront per two stored vectors (Section 3.2.2 maps a thread block to a vector).  Phase 1, for each: lanes =
// dimensions (residual, norm, o').  Phase 2: lanes = sampled rescaling factors — every lane walks all dimensions for
// its own t, so the N_coarse = 64 samples need no cross-lane reduction until the arg-max; then the N_fine = 32 samples
// around the best one, half a wavefront for each of the two vectors, against the coarse winner itself.  Phase 3, for
// each: lanes = dimensions again (codes, factor sums, packing).
// Bound by the vector instructions of phase 2 (about 6.5 per dimension and sample).  (250 000 x 128: 696 us when a
// wavefront had one vector, half of its lanes idle in the fine search -> 563)
// ---------------------------------------------------------------------------------
template <int DPL>  // dimensions per lane = ceil(D / 64)
__global__ __launch_bounds__(256) void encode_kernel(EncodeArgs a) {
  extern __shared__ unsigned char smem_raw[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int D = a.D, B = a.B;
  float* obuf = reinterpret_cast<float*>(smem_raw) + (size_t)wave * 2 * D;                        // [2][D] o'
  unsigned char* ubuf = smem_raw + 8 * (size_t)D * sizeof(float) + (size_t)wave * D;              // [D] codes
  const int64_t p = a.p0 + 2 * ((int64_t)blockIdx.x * 4 + wave);  // positions in cluster order: this one and the next
  if (p >= a.n) return;
  const int half = 1 << (B - 1), L = half - 1;
  const float Lf = (float)L;

  int cluster[2];
  int32_t vid[2];
  float r[2], r2[2], cdotres[2], t_end[2], t_c[2];
  bool ok[2];
  uint32_t coarse[2];  // best objective of the coarse samples, as ordered bits
  auto wave_fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto objective = [&](const float* o, float t) -> float {
    float num = 0.f, den = 0.f;
    for (int d = 0; d < D; d += 4) {
      const float4 y = *reinterpret_cast<const float4*>(o + d);
      const float y0 = fabsf(y.x), y1 = fabsf(y.y), y2 = fabsf(y.z), y3 = fabsf(y.w);
      const float m0 = fminf(floorf(t * y0), Lf) + 0.5f, m1 = fminf(floorf(t * y1), Lf) + 0.5f;
      const float m2 = fminf(floorf(t * y2), Lf) + 0.5f, m3 = fminf(floorf(t * y3), Lf) + 0.5f;
      num += m0 * y0 + m1 * y1 + m2 * y2 + m3 * y3;
      den += m0 * m0 + m1 * m1 + m2 * m2 + m3 * m3;
    }
    return num * rsqrtf(den);
  };
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int64_t pv = p + v < a.n ? p + v : p;
    // cluster of this position: largest c with off[c] <= p
    int lo = 0, hi = a.nlist;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.off[mid] <= pv) lo = mid; else hi = mid;
    }
    cluster[v] = lo;
    vid[v] = a.members[pv];
    float res[DPL];
    r2[v] = 0.f;
    cdotres[v] = 0.f;
#pragma unroll
    for (int k = 0; k < DPL; ++k) {
      const int d = k * 64 + lane;
      res[k] = 0.f;
      float cr = 0.f;
      if (d < D) {
        cr = a.c_rows[(int64_t)lo * D + d];
        res[k] = a.xr[(int64_t)vid[v] * D + d] - cr;
      }
      r2[v] += res[k] * res[k];
      cdotres[v] += cr * res[k];
    }
    r2[v] = wave_sum_f32(r2[v]);
    cdotres[v] = wave_sum_f32(cdotres[v]);
    r[v] = sqrtf(r2[v]);
    ok[v] = r[v] > 0.f;
    const float inv_r = ok[v] ? 1.0f / r[v] : 0.f;
    float ymax = 0.f;
#pragma unroll
    for (int k = 0; k < DPL; ++k) {
      const float o = res[k] * inv_r;
      const int d = k * 64 + lane;
      if (d < D) obuf[v * D + d] = o;
      ymax = fmaxf(ymax, fabsf(o));
    }
    ymax = wave_max_f32(ymax);
    // search range: the best factor lies below range_mult * 2^(B-1) / max|o'| (the fewer
    // levels, the further the bulk of the coordinates may be pushed past the largest one)
    const float range_mult = (B >= 5) ? 1.5f : (B == 4 ? 2.5f : (B == 3 ? 4.5f : 6.0f));
    t_end[v] = range_mult * (float)half / ymax;
    t_c[v] = 0.f;
    coarse[v] = 0u;
  }
  wave_fence();
  float t_best[2] = {0.f, 0.f};
  if (L > 0 && (ok[0] || ok[1])) {
    // coarse: t_k = (k+1)/64 * t_end, one sample per lane; ties go to the smaller t
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      if (!ok[v]) continue;
      const float tc = (float)(lane + 1) * (1.0f / 64.0f) * t_end[v];
      uint64_t key = ((uint64_t)f2ord(objective(obuf + v * D, tc)) << 32) | (uint32_t)(63 - lane);
      key = wave_reduce_u64(key, [](uint64_t x, uint64_t y) { return x > y ? x : y; });
      const int kc = 63 - (int)(uint32_t)key;
      t_c[v] = (float)(kc + 1) * (1.0f / 64.0f) * t_end[v];
      coarse[v] = (uint32_t)(key >> 32);
    }
    // fine: 32 samples uniform over t_c -+ t_end/64, a half of the wavefront for each vector, and t_c itself after them
    const int mine = lane >> 5, sample = lane & 31;
    const float my_t_c = mine ? t_c[1] : t_c[0];
    const float width = (mine ? t_end[1] : t_end[0]) * (1.0f / 64.0f);
    const float tf = fmaxf(my_t_c + width * (-1.0f + 2.0f * (float)sample * (1.0f / 31.0f)), 0.f);
    uint64_t key = ((uint64_t)f2ord(objective(obuf + mine * D, tf)) << 32) | (uint32_t)(63 - sample);
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
      const uint64_t other = (uint64_t)__shfl_xor((unsigned long long)key, d, 64);
      key = other > key ? other : key;
    }
    const uint64_t at_c = ((uint64_t)(mine ? coarse[1] : coarse[0]) << 32) | 31u;
    const float t_fine = __shfl(tf, 32 * mine + ((63 - (int)(uint32_t)key) & 31), 64);
    const float t_mine = at_c > key ? my_t_c : t_fine;
    t_best[0] = __shfl(t_mine, 0, 64);
    t_best[1] = __shfl(t_mine, 32, 64);
  }
  // codes and factor sums (lanes = dimensions)
  const float cB = (float)((1 << B) - 1) * 0.5f;
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    if (p + v >= a.n) break;
    const int64_t slot = (int64_t)a.tile_off[cluster[v]] * TILE + (p + v - a.off[cluster[v]]);
    float xo = 0.f, xc = 0.f, xx = 0.f, bo = 0.f, bc = 0.f;
    uint32_t u[DPL];
#pragma unroll
    for (int k = 0; k < DPL; ++k) {
      const int d = k * 64 + lane;
      const float o = d < D ? obuf[v * D + d] : 0.f, cr = d < D ? a.c_rows[(int64_t)cluster[v] * D + d] : 0.f;
      const float y = fabsf(o);
      const int m = (L > 0 && ok[v]) ? (int)fminf(floorf(t_best[v] * y), Lf) : 0;
      const bool pos = o >= 0.f;
      u[k] = ok[v] ? (uint32_t)(pos ? half + m : half - 1 - m) : (uint32_t)half;
      if (d < D) {
        ubuf[d] = (unsigned char)u[k];
        const float x = (float)u[k] - cB;
        const float xb = (float)(u[k] >> (B - 1)) - 0.5f;
        xo += x * o; xc += x * cr; xx += x * x;
        bo += xb * o; bc += xb * cr;
      }
    }
    xo = wave_sum_f32(xo); xc = wave_sum_f32(xc); xx = wave_sum_f32(xx);
    bo = wave_sum_f32(bo); bc = wave_sum_f32(bc);
    // short code: sign bits, 64 dimensions per ballot
    const int W = D >> 5;
    const int64_t tile = slot >> 6;
    const int ln = (int)(slot & 63);
#pragma unroll
    for (int k = 0; k < DPL; ++k) {
      const int d = k * 64 + lane;
      const uint64_t m = __ballot(d < D && ((u[k] >> (B - 1)) & 1u));
      if (lane == 0) {
        const int w = 2 * k;
        if (w < W) a.short_codes[(tile * W + w) * TILE + ln] = (uint32_t)m;
        if (w + 1 < W) a.short_codes[(tile * W + w + 1) * TILE + ln] = (uint32_t)(m >> 32);
      }
    }
    if (lane == 0) {
      const float Df = (float)D;
      float f1[3] = {0.f, 0.f, 0.f}, fB[2] = {0.f, 0.f};
      if (ok[v]) {
        const float scale = (a.metric == RABITQ_L2) ? 2.0f : 1.0f;
        const float lead = (a.metric == RABITQ_L2) ? r2[v] : -cdotres[v];
        const float a1 = fminf(fmaxf(bo / (0.5f * sqrtf(Df)), 0.f), 1.f);
        f1[0] = lead + scale * r[v] * bc / bo;
        f1[1] = -scale * r[v] / bo;
        f1[2] = scale * r[v] * a.eps0 * sqrtf(fmaxf(1.f - a1 * a1, 0.f)) / (a1 * sqrtf(Df - 1.f));
        fB[0] = lead + scale * r[v] * xc / xo;
        fB[1] = -scale * r[v] / xo;
      }
      a.short_factors[(tile * 3 + 0) * TILE + ln] = f1[0];
      a.short_factors[(tile * 3 + 1) * TILE + ln] = f1[1];
      a.short_factors[(tile * 3 + 2) * TILE + ln] = f1[2];
      if (B > 1) {
        a.long_factors[2 * slot] = fB[0];
        a.long_factors[2 * slot + 1] = fB[1];
      }
      a.ids[slot] = vid[v];
    }
    if (B > 1) {
      wave_fence();
      const int per = 32 / a.F;
      for (int w = lane; w < a.LW; w += 64) {
        uint32_t word = 0;
        for (int j = 0; j < per; ++j) word |= (uint32_t)ubuf[w * per + j] << (a.F * j);
        a.long_codes[slot * a.LW + w] = word;
      }
      wave_fence();  // (the next vector's codes take the same place)
    }
  }
}

// The scratch of a build: one allocation that is cut into arrays and freed on return.  (Allocating and freeing the nine arrays one by one
// cost the host 1.2 ms of the 4.1 that a build of 250 000 x 128 vectors takes with its first batch.)
struct Scratch {
  char* base = nullptr;
  int64_t used = 0;
  ~Scratch() { if (base) (void)hipFree(base); }
  static int64_t place(int64_t bytes) { return (std::max<int64_t>(bytes, 1) + 255) / 256 * 256; }
  int alloc(int64_t bytes) {
    const hipError_t e = hipMalloc(reinterpret_cast<void**>(&base), (size_t)std::max<int64_t>(bytes, 256));
    if (e != hipSuccess) {
      (void)hipGetLastError();
      base = nullptr;
      set_error("index build: hipMalloc failed: " + std::string(hipGetErrorString(e)));
      return RABITQ_ENOMEM;
    }
    return RABITQ_OK;
  }
  template <typename T>
  T* take(int64_t count) {
    T* p = reinterpret_cast<T*>(base + used);
    used += place(count * (int64_t)sizeof(T));
    return p;
  }
};

// Column means of a row-major [n][D] matrix in two fixed-order passes (deterministic): every
// workgroup sums its own block of rows per column in fp64, then one workgroup adds the
// partial sums in block order.
// Both are chains of additions: the next 16 rows and 64 partial sums are on their way meanwhile.  (250 000 x 128: 109 + 39 us -> 34 + 14)
constexpr int MEAN_BLOCKS = 1024;
__global__ __launch_bounds__(256) void column_partial_kernel(const float* __restrict__ x, int64_t n, int D,
                                                            double* __restrict__ partial) {
  constexpr int AHEAD = 16;
  const int64_t rows_per = (n + MEAN_BLOCKS - 1) / MEAN_BLOCKS;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per, r1 = r0 + rows_per < n ? r0 + rows_per : n;
  for (int d = threadIdx.x; d < D; d += blockDim.x) {
    double acc = 0.0;
    for (int64_t r = r0; r < r1; r += AHEAD) {
      float v[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) v[u] = x[(r + u < r1 ? r + u : r1 - 1) * D + d];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (r + u < r1) acc += (double)v[u];
    }
    partial[(int64_t)blockIdx.x * D + d] = acc;
  }
}
__global__ __launch_bounds__(64) void column_mean_kernel(const double* __restrict__ partial, int64_t n, int D,
                                                         float* __restrict__ mean) {
  constexpr int AHEAD = 64;
  const int d = blockIdx.x * 64 + threadIdx.x;
  if (d >= D) return;
  double acc = 0.0;
  for (int b = 0; b < MEAN_BLOCKS; b += AHEAD) {
    double v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[u] = partial[(int64_t)(b + u) * D + d];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) acc += v[u];
  }
  mean[d] = (float)(acc / (double)n);
}

static unsigned grid_for(int64_t n, int block = 256, int64_t cap = 65535) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + block - 1) / block, cap));
}

// ---- rows grouped by cluster -------------------------------------------------------------------
// A stable counting sort of row ids by cluster id whose memory grows with rows + blocks * nlist (the
// search path's builder keeps one bit per (cluster, query), which is right for 10^4 queries and far
// too much for 10^7 vectors).  The rows are cut into `nb` contiguous blocks; a wavefront counts its
// block per cluster, the counts are scanned block-major per cluster, and the same wavefront then places
// its rows 64 by 64 in row order, so every list holds its rows in ascending order whatever the
// scheduling.  A block is a chain of round trips to its counters, so there are as many blocks as the
// counters' memory allows: 16 MiB of them, or one block per 4096 rows where that is more.
constexpr int GROUP_TILE = 64;
struct GroupPlan {
  int nb;       // wavefronts = row blocks
  int64_t ch;   // rows per block, a multiple of GROUP_TILE
};
static GroupPlan group_plan(int64_t rows, int nlist) {
  GroupPlan g;
  const int64_t few = std::min<int64_t>((rows + 4095) / 4096, 1024);
  const int64_t many = std::min<int64_t>({(rows + 4 * GROUP_TILE - 1) / (4 * GROUP_TILE), ((int64_t)1 << 22) / nlist, 4096});
  const int64_t want = std::max<int64_t>({1, few, many});
  g.ch = ((rows + want - 1) / want + GROUP_TILE - 1) / GROUP_TILE * GROUP_TILE;
  if (g.ch < GROUP_TILE) g.ch = GROUP_TILE;
  g.nb = (int)std::max<int64_t>(1, (rows + g.ch - 1) / g.ch);
  return g;
}

__global__ __launch_bounds__(GROUP_TILE) void group_count_kernel(const int32_t* __restrict__ asg, int64_t rows, int64_t ch,
                                                                 int nlist, int32_t* __restrict__ hist) {
  const int64_t r0 = (int64_t)blockIdx.x * ch, r1 = r0 + ch < rows ? r0 + ch : rows;
  int32_t* h = hist + (int64_t)blockIdx.x * nlist;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += GROUP_TILE) atomicAdd(&h[asg[i]], 1);
}

// per cluster: counts of the row blocks -> exclusive prefix over the blocks (in place) and the list length.  32 clusters a
// workgroup, the blocks of each in 32 segments, whose sums are exchanged through LDS.
__global__ __launch_bounds__(1024) void group_block_prefix_kernel(int32_t* __restrict__ hist, int nb, int nlist,
                                                                  int32_t* __restrict__ total) {
  constexpr int AHEAD = 8;
  __shared__ int32_t s_sum[32][32];
  const int cl = threadIdx.x & 31, seg = threadIdx.x >> 5;
  const int c = blockIdx.x * 32 + cl;
  const int per = (nb + 31) / 32, b0 = min(seg * per, nb), b1 = min(b0 + per, nb);
  int32_t* col = hist + min(c, nlist - 1);
  int32_t sum = 0;
  for (int b = b0; b < b1; b += AHEAD) {
    int32_t v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[u] = col[(int64_t)min(b + u, b1 - 1) * nlist];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) sum += b + u < b1 ? v[u] : 0;
  }
  s_sum[seg][cl] = sum;
  __syncthreads();
  if (c >= nlist) return;
  int32_t run = 0;
  for (int t = 0; t < seg; ++t) run += s_sum[t][cl];
  if (seg == 31) total[c] = run + sum;
  for (int b = b0; b < b1; b += AHEAD) {
    int32_t v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[u] = col[(int64_t)min(b + u, b1 - 1) * nlist];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      if (b + u < b1) col[(int64_t)(b + u) * nlist] = run;
      run += v[u];
    }
  }
}

// off[c] = sum of total[0..c), off[nlist] = rows; one workgroup walks the lists in order
__global__ __launch_bounds__(1024) void group_offsets_kernel(const int32_t* __restrict__ total, int nlist,
                                                             int32_t* __restrict__ off) {
  __shared__ int32_t s_part[1024];
  __shared__ int32_t s_base;
  if (threadIdx.x == 0) s_base = 0;
  __syncthreads();
  for (int c0 = 0; c0 < nlist; c0 += 1024) {
    const int c = c0 + threadIdx.x;
    const int32_t v = c < nlist ? total[c] : 0;
    s_part[threadIdx.x] = v;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {  // inclusive scan of the 1024 values
      const int32_t add = threadIdx.x >= d ? s_part[threadIdx.x - d] : 0;
      __syncthreads();
      s_part[threadIdx.x] += add;
      __syncthreads();
    }
    if (c < nlist) off[c] = s_base + s_part[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 1023) s_base += s_part[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) off[nlist] = s_base;
}

// A tile of 64 rows: the lanes whose rows fall into the same list find each other by one ballot per bit of the list id, the last of
// them advances the list's counter by their number, and all of them take their places behind its old value.  (50 000 rows, 512
// lists: 94 us a pass when a workgroup of 256 rows compared each with all others -> 5.4)
__global__ __launch_bounds__(GROUP_TILE) void group_scatter_kernel(const int32_t* __restrict__ asg, int64_t rows, int64_t ch,
                                                                   int nlist, int bits, int32_t* __restrict__ hist,
                                                                   const int32_t* __restrict__ off,
                                                                   int32_t* __restrict__ members) {
  const int64_t r0 = (int64_t)blockIdx.x * ch, r1 = r0 + ch < rows ? r0 + ch : rows;
  int32_t* h = hist + (int64_t)blockIdx.x * nlist;  // rows of this cluster placed so far, by earlier blocks and tiles
  const int lane = threadIdx.x;
  int32_t next = asg[min(r0 + lane, r1 - 1)];
  for (int64_t t0 = r0; t0 < r1; t0 += GROUP_TILE) {
    const int64_t i = t0 + lane;
    const bool valid = i < r1;
    const int32_t key = next;
    next = asg[min(i + GROUP_TILE, r1 - 1)];
    uint64_t same = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool set = (key >> b) & 1;
      const uint64_t m = __ballot(set);
      same &= set ? m : ~m;
    }
    const int last = valid ? 63 - __builtin_clzll(same) : lane;
    int32_t base = 0;
    if (valid && lane == last) base = atomicAdd(&h[key], (int32_t)__builtin_popcountll(same));
    base = __shfl(base, last, 64);
    if (valid) members[off[key] + base + __builtin_popcountll(same & ((1ull << lane) - 1ull))] = (int32_t)i;
  }
}

// rows [0, rows) grouped by asg[] into off[nlist + 1] / members[rows]; hist holds group_plan(rows, nlist).nb * nlist words
static int launch_group_rows(const int32_t* asg, int64_t rows, int nlist, int32_t* off, int32_t* members, int32_t* hist,
                             int32_t* total, hipStream_t st) {
  const GroupPlan g = group_plan(rows, nlist);
  const int64_t hw = (int64_t)g.nb * nlist;
  hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(hw)), dim3(256), 0, st, hist, hw, 0);
  if (rows > 0)
    hipLaunchKernelGGL(group_count_kernel, dim3(g.nb), dim3(GROUP_TILE), 0, st, asg, rows, g.ch, nlist, hist);
  hipLaunchKernelGGL(group_block_prefix_kernel, dim3((nlist + 31) / 32), dim3(1024), 0, st, hist, g.nb, nlist, total);
  hipLaunchKernelGGL(group_offsets_kernel, dim3(1), dim3(1024), 0, st, total, nlist, off);
  int bits = 0;
  while (((int64_t)1 << bits) < nlist) ++bits;
  if (rows > 0)
    hipLaunchKernelGGL(group_scatter_kernel, dim3(g.nb), dim3(GROUP_TILE), 0, st, asg, rows, g.ch, nlist, bits, hist, off, members);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

// nearest rotated centroid of every row of `x` [rows][D]; `keys` holds chunk x ceil(nlist / 32) words
static int assign_rows(const float* x, int64_t rows, int D, int nlist, const float* ct, const float* csq, uint64_t* keys,
                       int64_t chunk, int32_t* out, hipStream_t st) {
  for (int64_t s = 0; s < rows; s += chunk) {
    const int64_t m = std::min(chunk, rows - s);
    int parts = 0;
    int rc = launch_gemm_nearest(x + s * D, ct, keys, m, nlist, D, csq, &parts, st);
    if (rc) return rc;
    hipLaunchKernelGGL(nearest_of_parts_kernel, dim3((unsigned)((m + 15) / 16)), dim3(256), 0, st, keys, m, parts, out + s);
  }
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

int build_index_device(rabitq_index* ix, const float* data, const float* rotation_host, int kmeans_iters,
                       int64_t train_size, float eps0, int center, hipStream_t st) {
  const int D = ix->dim, nlist = ix->nlist, B = ix->total_bits;
  const int64_t N = ix->n;
  int rc;
#define RQ_TRY(x) do { if ((rc = (x)) != RABITQ_OK) return rc; } while (0)
  // rotation to the device, rotate all vectors once (distances are rotation invariant, so
  // clustering and residuals are taken in the rotated space)
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->rotation), (size_t)D * D * sizeof(float)));
  RQ_HIP(hipMemcpyAsync(ix->rotation, rotation_host, (size_t)D * D * sizeof(float), hipMemcpyHostToDevice, st));
  const int64_t nt = std::max<int64_t>(nlist, std::min<int64_t>(train_size > 0 ? train_size : N, N));
  const int nearest_words = (nlist + 31) / 32;
  const int64_t rows = std::max(N, nt);
  const int64_t chunk = std::max<int64_t>(1024, ((int64_t)1 << 23) / nearest_words);  // 64 MiB of keys
  const int64_t n_keys = std::min<int64_t>(chunk, rows) * nearest_words;
  const int64_t n_hist = (int64_t)std::max(group_plan(N, nlist).nb, group_plan(nt, nlist).nb) * nlist;
  const int64_t n_partial = center && N > 0 ? (int64_t)MEAN_BLOCKS * D : 0;
  Scratch mem;
  RQ_TRY(mem.alloc(Scratch::place(N * D * 4) + Scratch::place(nt * D * 4) + Scratch::place((int64_t)nlist * D * 4) +
                   Scratch::place(n_keys * 8) + 2 * Scratch::place(rows * 4) + Scratch::place((nlist + 1) * (int64_t)4) +
                   Scratch::place(n_hist * 4) + Scratch::place(nlist * (int64_t)4) + Scratch::place(n_partial * 8) +
                   Scratch::place(D * (int64_t)4)));
  float* const xr = mem.take<float>(N * D);
  float* const tr = mem.take<float>(nt * D);
  float* const c_rows = mem.take<float>((int64_t)nlist * D);
  uint64_t* const keys = mem.take<uint64_t>(n_keys);
  int32_t* const asg = mem.take<int32_t>(rows);
  int32_t* const members = mem.take<int32_t>(rows);
  int32_t* const off = mem.take<int32_t>(nlist + 1);
  int32_t* const hist = mem.take<int32_t>(n_hist);
  int32_t* const total = mem.take<int32_t>(nlist);
  if (center && N > 0) {
    // mean of the raw vectors; every later step sees (x - mean) P = x P - mean P
    double* const partial = mem.take<double>(n_partial);
    float* const mean_dev = mem.take<float>(D);
    hipLaunchKernelGGL(column_partial_kernel, dim3(MEAN_BLOCKS), dim3(std::min(256, (D + 63) / 64 * 64)), 0, st, data, N, D, partial);
    hipLaunchKernelGGL(column_mean_kernel, dim3((D + 63) / 64), dim3(64), 0, st, partial, N, D, mean_dev);
    std::vector<float> mean(D);
    RQ_HIP(hipMemcpyAsync(mean.data(), mean_dev, (size_t)D * sizeof(float), hipMemcpyDeviceToHost, st));
    RQ_HIP(hipStreamSynchronize(st));
    RQ_TRY(set_index_mean(ix, mean.data(), rotation_host, st));
  }
  RQ_TRY(launch_rotate(ix, data, xr, N, st));
  hipLaunchKernelGGL(gather_rows_kernel, dim3(grid_for(nt * D)), dim3(256), 0, st, xr, N, nt, D, tr);
  hipLaunchKernelGGL(gather_rows_kernel, dim3(grid_for((int64_t)nlist * D)), dim3(256), 0, st, tr, nt, (int64_t)nlist,
                     D, c_rows);
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->centroids_t), (size_t)D * nlist * sizeof(float)));
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->centroid_sq), (size_t)nlist * sizeof(float)));
  for (int it = 0; it < kmeans_iters; ++it) {
    hipLaunchKernelGGL(transpose_centroids_kernel, dim3((nlist + 63) / 64), dim3(64), 0, st, c_rows, nlist, D,
                       ix->centroids_t, ix->centroid_sq);
    RQ_TRY(assign_rows(tr, nt, D, nlist, ix->centroids_t, ix->centroid_sq, keys, chunk, asg, st));
    RQ_TRY(launch_group_rows(asg, nt, nlist, off, members, hist, total, st));
    hipLaunchKernelGGL(centroid_update_kernel, dim3(nlist, (D + 63) / 64), dim3(64), 0, st, tr, off, members, D, c_rows);
  }
  hipLaunchKernelGGL(transpose_centroids_kernel, dim3((nlist + 63) / 64), dim3(64), 0, st, c_rows, nlist, D,
                     ix->centroids_t, ix->centroid_sq);
  RQ_TRY(assign_rows(xr, N, D, nlist, ix->centroids_t, ix->centroid_sq, keys, chunk, asg, st));
  RQ_TRY(launch_group_rows(asg, N, nlist, off, members, hist, total, st));
  // layout: cluster sizes, tile offsets (the total is needed on the host to size the arrays)
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->cluster_size), (size_t)nlist * sizeof(int32_t)));
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->tile_off), (size_t)tile_off_words(nlist) * sizeof(int32_t)));
  RQ_HIP(hipMemsetAsync(ix->tile_off, 0, (size_t)tile_off_words(nlist) * sizeof(int32_t), st));
  hipLaunchKernelGGL(cluster_layout_kernel, dim3((nlist + 255) / 256), dim3(256), 0, st, off, nlist, ix->cluster_size);
  std::vector<int32_t> h_off(nlist + 1), h_tile(nlist + 1);
  RQ_HIP(hipMemcpyAsync(h_off.data(), off, (size_t)(nlist + 1) * sizeof(int32_t), hipMemcpyDeviceToHost, st));
  RQ_HIP(hipStreamSynchronize(st));
  int64_t tiles = 0;
  for (int c = 0; c < nlist; ++c) {
    h_tile[c] = (int32_t)tiles;
    tiles += (h_off[c + 1] - h_off[c] + TILE - 1) / TILE;
  }
  h_tile[nlist] = (int32_t)tiles;
  ix->host_tiles.resize(nlist);
  for (int c = 0; c < nlist; ++c) ix->host_tiles[c] = h_tile[c + 1] - h_tile[c];
  if (tiles > (0x7fffffff / TILE)) { set_error("index build: too many slots"); return RABITQ_EINVAL; }
  ix->n_tiles = tiles;
  ix->n_slots = tiles * TILE;
  RQ_HIP(hipMemcpyAsync(ix->tile_off, h_tile.data(), (size_t)(nlist + 1) * sizeof(int32_t), hipMemcpyHostToDevice, st));
  const int W = ix->W, LW = ix->LW;
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->short_codes), (size_t)std::max<int64_t>(1, tiles * W * TILE) * 4));
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->short_factors), (size_t)std::max<int64_t>(1, tiles * 3 * TILE) * 4));
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->ids), (size_t)std::max<int64_t>(1, tiles * TILE) * 4));
  hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(tiles * W * TILE)), dim3(256), 0, st,
                     reinterpret_cast<int32_t*>(ix->short_codes), tiles * W * TILE, 0);
  hipLaunchKernelGGL(init_short_factors_kernel, dim3(grid_for(tiles * 3 * TILE)), dim3(256), 0, st, ix->short_factors, tiles);
  hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(tiles * TILE)), dim3(256), 0, st, ix->ids, tiles * TILE, -1);
  if (B > 1) {
    RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->long_codes), (size_t)std::max<int64_t>(1, tiles * TILE * LW) * 4));
    RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->long_factors), (size_t)std::max<int64_t>(1, tiles * TILE * 2) * 4));
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(tiles * TILE * LW)), dim3(256), 0, st,
                       reinterpret_cast<int32_t*>(ix->long_codes), tiles * TILE * LW, 0);
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(tiles * TILE * 2)), dim3(256), 0, st,
                       reinterpret_cast<int32_t*>(ix->long_factors), tiles * TILE * 2, 0);
  }
  EncodeArgs a{};
  a.xr = xr; a.c_rows = c_rows; a.off = off; a.members = members; a.tile_off = ix->tile_off;
  a.n = N; a.D = D; a.B = B; a.F = ix->F; a.LW = LW; a.nlist = nlist; a.metric = ix->metric; a.eps0 = eps0;
  a.short_codes = ix->short_codes; a.short_factors = ix->short_factors; a.long_codes = ix->long_codes;
  a.long_factors = ix->long_factors; a.ids = ix->ids;
  // (a launch may hold fewer than 2^32 work-items: the positions are encoded in slices)
  constexpr int64_t SLICE = (int64_t)1 << 24;
  for (int64_t p0 = 0; p0 < N; p0 += SLICE) {
    a.p0 = p0;
    const unsigned grid = (unsigned)((std::min(SLICE, N - p0) + 7) / 8);
    const size_t smem = 4 * (size_t)D * (2 * sizeof(float) + 1);
    const int dpl = (D + 63) / 64;
    if (dpl <= 2) hipLaunchKernelGGL(encode_kernel<2>, dim3(grid), dim3(256), smem, st, a);
    else if (dpl <= 4) hipLaunchKernelGGL(encode_kernel<4>, dim3(grid), dim3(256), smem, st, a);
    else if (dpl <= 8) hipLaunchKernelGGL(encode_kernel<8>, dim3(grid), dim3(256), smem, st, a);
    else if (dpl <= 16) hipLaunchKernelGGL(encode_kernel<16>, dim3(grid), dim3(256), smem, st, a);
    else hipLaunchKernelGGL(encode_kernel<32>, dim3(grid), dim3(256), smem, st, a);
  }
  RQ_HIP(hipGetLastError());
  RQ_HIP(hipStreamSynchronize(st));  // temporaries are freed on return
#undef RQ_TRY
  return RABITQ_OK;
}

}  // namespace rq
