// Device-side building blocks shared by the selection, seeding, scan and merge kernels.
#pragma once
#include "rq_internal.h"

namespace rq {

constexpr uint64_t KEY_NONE = ~0ull;

// (by value: a conditional on variables selects among their addresses, which puts them into memory)
template <typename T>
__device__ inline T one_of(int i, T a, T b, T c, T d) { return i == 0 ? a : (i == 1 ? b : (i == 2 ? c : d)); }

__device__ inline uint64_t make_key(float v, uint32_t lo) { return ((uint64_t)f2ord(v) << 32) | lo; }

// ---------------------------------------------------------------------------------
// Bitonic sort (ascending) of n = 2^m u64 keys in LDS by the whole workgroup.
// Ends with a barrier.
// ---------------------------------------------------------------------------------
__device__ inline void block_bitonic_sort(uint64_t* keys, int n) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int k = 2; k <= n; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      __syncthreads();
      for (int t = tid; t < (n >> 1); t += nt) {
        const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
        const int l = i | j;
        const uint64_t a = keys[i], b = keys[l];
        const bool up = (i & k) == 0;
        if ((a > b) == up) {
          keys[i] = b;
          keys[l] = a;
        }
      }
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------
// Workgroup-wide selection of the K smallest of n u64 keys produced by key_at(i),
// written in ascending order to out[0..Kpad) (Kpad = power of two >= K, the tail is
// KEY_NONE).  key_at may return KEY_NONE for an absent entry.  Keys are distinct (their
// low word is an index or id), so the result is unique.
//
// MSB-first radix select that (1) skips the bits all keys share (estimates of one query lie
// in a narrow range, so their exponent bits are equal and would all hit one histogram bin),
// (2) stops as soon as the bucket holding the K-th key is taken whole, and (3) finishes a
// bucket of at most 64 keys inside one wavefront by ranking them against each other.
// blockDim.x must be a multiple of 64, at most 1024.
// ---------------------------------------------------------------------------------
// Wavefront reductions on the VALU's data-parallel primitives (no LDS round trips).
// After the four row steps every lane of a 16-lane row holds the row's result; the four
// rows are then combined through scalar lane reads.
template <typename Op>
__device__ inline uint32_t wave_reduce_u32(uint32_t v, Op op) {
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));  // row_half_mirror
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));  // row_mirror
  const uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
  return op(op(a, b), op(c, d));
}

template <typename Op>
__device__ inline uint64_t wave_reduce_u64(uint64_t v, Op op) {
  auto step = [&](int ctrl_id) {
    int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    int olo, ohi;
    switch (ctrl_id) {
      case 0: olo = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, true); ohi = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, true); break;
      case 1: olo = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, true); ohi = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, true); break;
      case 2: olo = __builtin_amdgcn_update_dpp(0, lo, 0x141, 0xF, 0xF, true); ohi = __builtin_amdgcn_update_dpp(0, hi, 0x141, 0xF, 0xF, true); break;
      default: olo = __builtin_amdgcn_update_dpp(0, lo, 0x140, 0xF, 0xF, true); ohi = __builtin_amdgcn_update_dpp(0, hi, 0x140, 0xF, 0xF, true); break;
    }
    v = op(v, ((uint64_t)(uint32_t)ohi << 32) | (uint32_t)olo);
  };
  step(0); step(1); step(2); step(3);
  auto rd = [&](int l) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  };
  return op(op(rd(0), rd(16)), op(rd(32), rd(48)));
}

struct SelectScratch {
  uint64_t lo, hi, bound;
  uint64_t small[64];
  uint64_t wlo[16], whi[16];
  uint32_t hist[256];
  uint32_t wcnt[16];
  uint32_t digit, need, bucket, cnt, nvalid;
};

template <typename KeyFn>
__device__ inline void block_select_smallest(int n, int K, int Kpad, KeyFn key_at, uint64_t* out, SelectScratch* sh) {
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  // range and count of the present keys
  uint64_t lo = KEY_NONE, hi = 0ull;
  uint32_t nv = 0;
  for (int i = tid; i < n; i += nt) {
    const uint64_t key = key_at(i);
    if (key != KEY_NONE) {
      lo = key < lo ? key : lo;
      hi = key > hi ? key : hi;
      ++nv;
    }
  }
  lo = wave_reduce_u64(lo, [](uint64_t a, uint64_t b) { return a < b ? a : b; });
  hi = wave_reduce_u64(hi, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
  nv = wave_reduce_u32(nv, [](uint32_t a, uint32_t b) { return a + b; });
  if (lane == 0) {
    sh->wlo[wave] = lo;
    sh->whi[wave] = hi;
    sh->wcnt[wave] = nv;
  }
  __syncthreads();
  if (tid == 0) {
    uint64_t l = KEY_NONE, h = 0ull;
    uint32_t c = 0;
    for (int w = 0; w < nw; ++w) {
      l = sh->wlo[w] < l ? sh->wlo[w] : l;
      h = sh->whi[w] > h ? sh->whi[w] : h;
      c += sh->wcnt[w];
    }
    sh->lo = l;
    sh->hi = h;
    sh->nvalid = c;
  }
  __syncthreads();
  uint64_t bound = KEY_NONE;  // select present keys <= bound
  if (sh->nvalid > (uint32_t)K && sh->lo != sh->hi) {
    lo = sh->lo;
    hi = sh->hi;
    const int top = 63 - __clzll((long long)(lo ^ hi));  // highest bit in which two keys differ
    int width = min(8, top + 1);
    int shift = top + 1 - width;
    uint64_t pmask = (top == 63) ? 0ull : (~0ull << (top + 1));
    uint64_t prefix = lo & pmask;
    uint32_t need = (uint32_t)K;
    while (true) {
      for (int i = tid; i < 256; i += nt) sh->hist[i] = 0;
      __syncthreads();
      const uint32_t dmask = (1u << width) - 1u;
      for (int i = tid; i < n; i += nt) {
        const uint64_t key = key_at(i);
        if (key != KEY_NONE && (key & pmask) == prefix) atomicAdd(&sh->hist[(uint32_t)(key >> shift) & dmask], 1u);
      }
      __syncthreads();
      if (tid < 64) {
        const uint32_t c0 = sh->hist[4 * tid], c1 = sh->hist[4 * tid + 1], c2 = sh->hist[4 * tid + 2],
                       c3 = sh->hist[4 * tid + 3];
        const uint32_t s = c0 + c1 + c2 + c3;
        uint32_t incl = s;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t o = __shfl_up(incl, d, 64);
          if (tid >= d) incl += o;
        }
        const uint32_t excl = incl - s;
        if (excl < need && need <= incl) {
          uint32_t rem = need - excl, digit, cnt;
          if (rem <= c0) { digit = 0; cnt = c0; }
          else if (rem <= c0 + c1) { digit = 1; cnt = c1; rem -= c0; }
          else if (rem <= c0 + c1 + c2) { digit = 2; cnt = c2; rem -= c0 + c1; }
          else { digit = 3; cnt = c3; rem -= c0 + c1 + c2; }
          sh->digit = 4 * tid + digit;
          sh->need = rem;
          sh->bucket = cnt;
          sh->cnt = 0;
        }
      }
      __syncthreads();
      prefix |= (uint64_t)sh->digit << shift;
      pmask |= (uint64_t)dmask << shift;
      need = sh->need;
      const uint32_t bucket = sh->bucket;
      if (bucket == need || shift == 0) {  // the whole bucket is selected
        bound = prefix | (shift == 0 ? 0ull : ((1ull << shift) - 1ull));
        break;
      }
      if (bucket <= 64u) {  // rank the bucket's keys against each other in one wavefront
        for (int i = tid; i < n; i += nt) {
          const uint64_t key = key_at(i);
          if (key != KEY_NONE && (key & pmask) == prefix) sh->small[atomicAdd(&sh->cnt, 1u)] = key;
        }
        __syncthreads();
        if (tid < (int)bucket) {
          const uint64_t mine = sh->small[tid];
          uint32_t rank = 0;
          for (uint32_t m = 0; m < bucket; ++m) rank += (sh->small[m] < mine) ? 1u : 0u;
          if (rank == need - 1u) sh->bound = mine;
        }
        __syncthreads();
        bound = sh->bound;
        break;
      }
      width = min(8, shift);
      shift -= width;
      __syncthreads();
    }
  }
  __syncthreads();
  if (tid == 0) sh->cnt = 0;
  for (int i = tid; i < Kpad; i += nt) out[i] = KEY_NONE;
  __syncthreads();
  for (int i = tid; i < n; i += nt) {
    const uint64_t key = key_at(i);
    if (key <= bound && key != KEY_NONE) {
      const uint32_t pos = atomicAdd(&sh->cnt, 1u);
      if (pos < (uint32_t)Kpad) out[pos] = key;
    }
  }
  block_bitonic_sort(out, Kpad);
}

// ---------------------------------------------------------------------------------
// Wavefront-wide selection with the keys in registers: every lane holds R keys (KEY_NONE =
// absent).  Returns a bound such that exactly min(K, #present) present keys are <= bound.
// MSB-first bisection: one bit per step, counting the keys of the current bucket whose
// next bit is 0; the bits all keys share are skipped and the search stops as soon as the
// bucket holding the K-th key is taken whole.  No LDS, no barriers.
// ---------------------------------------------------------------------------------
template <int R>
__device__ inline uint64_t wave_kth_bound(const uint64_t (&key)[R], int K) {
  uint64_t lo = KEY_NONE, hi = 0ull;
  uint32_t nv = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (key[r] != KEY_NONE) {
      lo = key[r] < lo ? key[r] : lo;
      hi = key[r] > hi ? key[r] : hi;
      ++nv;
    }
  }
  lo = wave_reduce_u64(lo, [](uint64_t a, uint64_t b) { return a < b ? a : b; });
  hi = wave_reduce_u64(hi, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
  nv = wave_reduce_u32(nv, [](uint32_t a, uint32_t b) { return a + b; });
  if (nv <= (uint32_t)K) return KEY_NONE - 1ull;
  if (lo == hi) return hi;
  const int top = 63 - __clzll((long long)(lo ^ hi));
  uint64_t prefix = (top == 63) ? 0ull : (hi & (~0ull << (top + 1)));
  uint32_t need = (uint32_t)K, cmatch = nv;
  for (int b = top; b >= 0; --b) {
    const uint64_t mask_hi = ~0ull << b;
    uint32_t c0 = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) c0 += ((key[r] & mask_hi) == prefix) ? 1u : 0u;
    c0 = wave_reduce_u32(c0, [](uint32_t a, uint32_t x) { return a + x; });
    if (need <= c0) {
      cmatch = c0;
    } else {
      need -= c0;
      cmatch -= c0;
      prefix |= 1ull << b;
    }
    if (cmatch == need) return prefix | ((b == 0) ? 0ull : ((1ull << b) - 1ull));
  }
  return prefix;
}

// ---------------------------------------------------------------------------------
// The same with 32-bit words (order-preserving float bits; all ones = absent) whose order of arrival, r then lane, is
// the order of their positions, so that a tie goes to the earlier one.  Bisection of the value range; a step is one
// compare per word on the vector unit and its bits counted on the scalar unit, and it ends as soon as a value splits
// off exactly K words: about 10 steps where the words lie within an octave or two, more where they straddle zero, and the
// whole bit length of the range (32 at most) where the K-th word has equals.  (Drawing the range in to the words that are
// in it every 12 steps ends that case sooner, 4 queries on a list of 20000 mostly equal vectors: seeding 28 us against 33, but
// costs every search of a few queries 1 %.)
// Returns a bound with count(words <= bound) = *n_le >= K, where *n_le > K only if the bound is the K-th smallest
// word itself and has equals.  If fewer than K words are present (1 <= K), the largest of them and their number.
// ---------------------------------------------------------------------------------
template <int R>
__device__ inline uint32_t wave_kth_ord(const uint32_t (&ord)[R], uint32_t K, uint32_t* n_le) {
  uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    mn = min(mn, ord[r]);
    mx = max(mx, ord[r] == 0xffffffffu ? 0u : ord[r]);
  }
  uint32_t lo = wave_reduce_u32(mn, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
  uint32_t hi = wave_reduce_u32(mx, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
  auto count = [&](uint32_t v) {
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) c += (uint32_t)__popcll(__ballot(ord[r] <= v));
    return c;
  };
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    const uint32_t c = count(mid);
    if (c == K) {
      *n_le = K;
      return mid;
    }
    if (c > K) hi = mid;
    else lo = mid + 1;
  }
  *n_le = count(hi);
  return hi;
}

// Value of the K-th smallest word (the bound above may lie between two words); all ones if fewer than K are present
// (an estimate that is a NaN of all ones reads as absent).
template <int R>
__device__ inline uint32_t wave_kth_value(const uint32_t (&ord)[R], uint32_t K) {
  uint32_t n_le;
  const uint32_t bound = wave_kth_ord<R>(ord, K, &n_le);
  uint32_t mx = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) mx = max(mx, ord[r] <= bound ? ord[r] : 0u);
  mx = wave_reduce_u32(mx, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
  return n_le < K ? 0xffffffffu : mx;
}

// Hands the selected words out in their order, put(place, r) for every word <= bound, or, where more than K words are
// (n_le > K), for those below it and the first equals.  Returns K.  (the caller orders its own LDS accesses)
template <int R, typename Put>
__device__ inline int wave_put_smallest(const uint32_t (&ord)[R], uint32_t bound, uint32_t n_le, uint32_t K, int lane, Put put) {
  uint32_t equals = 0xffffffffu;  // how many words equal to the bound may still be taken
  if (n_le > K) {
    uint32_t below = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) below += (uint32_t)__popcll(__ballot(ord[r] < bound));
    equals = K - below;
  }
  const uint64_t lower = (1ull << lane) - 1ull;
  uint32_t base = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    bool take = ord[r] <= bound;
    if (n_le > K) {
      const uint64_t eq = __ballot(ord[r] == bound);
      if (ord[r] == bound) take = (uint32_t)__popcll(eq & lower) < equals;
      equals -= min(equals, (uint32_t)__popcll(eq));
    }
    const uint64_t m = __ballot(take);
    if (take) put((int)(base + (uint32_t)__popcll(m & lower)), r);
    base += (uint32_t)__popcll(m);
  }
  return (int)base;
}

// The k best of more than k keys in registers (KEY_NONE = absent), put(place, key) for places 0 .. k - 1 in any order, by one
// wavefront.  Keys may repeat: of several at the last place only as many are kept as there is room for.  *cnt = k; returns a
// limit that only keys at or below it can be among the k best: the k-th key, or a value between it and the next one up.
// (the caller orders its own memory accesses)
template <int R, typename Put>
__device__ __forceinline__ uint64_t wave_keep_best(const uint64_t (&key)[R], int k, int lane, int* cnt, Put put) {
  uint32_t ord[R], n_le;
#pragma unroll
  for (int r = 0; r < R; ++r) ord[r] = (uint32_t)(key[r] >> 32);
  const uint32_t bound = wave_kth_ord<R>(ord, (uint32_t)k, &n_le);
  uint64_t last = ((uint64_t)bound << 32) | 0xffffffffu;
  // (equal distances at the last place: the lower ids)
  if (n_le != (uint32_t)k) last = wave_kth_bound<R>(key, k);
  const uint64_t lower = (1ull << lane) - 1ull;
  int at = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t m = __ballot(key[r] < last);
    if (key[r] < last) put(at + __popcll(m & lower), key[r]);
    at += __popcll(m);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t m = __ballot(key[r] == last);
    const int place = at + __popcll(m & lower);
    if (key[r] == last && place < k) put(place, key[r]);
    at += __popcll(m);
  }
  *cnt = min(at, k);
  return at > k ? last - 1ull : last;
}

// ---------------------------------------------------------------------------------
// Streaming selection of the K <= 64 smallest 64-bit keys by one wavefront, entirely in
// registers: lane l holds the l-th smallest key seen so far.  The first 64 keys are sorted
// across the lanes (bitonic network); afterwards a tile of 64 keys is compared with the
// current K-th key and only the few that beat it are inserted, one at a time.  Keys are
// unique (their low word is an index), so the result does not depend on the order of
// arrival.  All control flow is wave-uniform.
// ---------------------------------------------------------------------------------
__device__ inline uint64_t shfl_u64(uint64_t v, int src) {
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src, 64);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src, 64);
  return ((uint64_t)hi << 32) | lo;
}
__device__ inline uint64_t readlane_u64(uint64_t v, int src) {  // src must be wave-uniform
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}

// Keeps a loaded value where it is: without it the compiler moves a load whose value is only used under a
// condition back under that condition, into a block of its own, and then waits for every such load before it
// issues the next one.
__device__ inline float pinned(float v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ inline uint64_t pinned(uint64_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

struct WaveTopK {
  uint64_t v;  // lane l: l-th smallest key so far (KEY_NONE where there is none yet)

  // the first tile: ascending bitonic sort of one key per lane
  __device__ inline void init_sorted(uint64_t key, int lane) {
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
      for (int j = k >> 1; j > 0; j >>= 1) {
        const uint64_t other = shfl_u64(key, lane ^ j);
        const bool asc = (lane & k) == 0;
        const bool low = (lane & j) == 0;
        const bool take_min = (asc == low);
        const uint64_t mn = key < other ? key : other, mx = key < other ? other : key;
        key = take_min ? mn : mx;
      }
    }
    v = key;
  }

  // a further tile: one key per lane
  __device__ inline void push_tile(uint64_t key, int K, int lane) {
    uint64_t kth = readlane_u64(v, K - 1);
    uint64_t m = __ballot(key < kth);
    while (m != 0ull) {
      const int src = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)m) - 1);
      m &= m - 1ull;
      const uint64_t x = readlane_u64(key, src);
      if (x < kth) {  // the K-th key may have dropped since the ballot
        const int p = __popcll(__ballot(v < x));  // keys below x; x goes to position p (< K)
        // every lane's left neighbour through the data-parallel primitive that shifts the whole wavefront by one
        // lane (lane 0 keeps its own value, which it never needs: it takes x or stays)
        const uint32_t ulo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)v, (int)(uint32_t)v, 0x138, 0xF, 0xF, false);
        const uint32_t uhi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(v >> 32), (int)(uint32_t)(v >> 32), 0x138, 0xF, 0xF, false);
        const uint64_t up = ((uint64_t)uhi << 32) | ulo;
        v = lane < p ? v : (lane == p ? x : up);
        kth = readlane_u64(v, K - 1);
      }
    }
  }
};

template <int F>
__host__ __device__ inline int stage_index(int d);  // position of dimension d in the refinement's query order (below)
__device__ inline float digit_factor(float delta);
__device__ inline uint4 digit_quad(float4 q, float factor);

// Position of dimension d in the qhat8 array (the matrix-core scan's query operand).  Within every chunk of 64
// dimensions, dimension r = 32 w + 8 b + 4 h + i (w: word of the chunk, b = 0..3, h = 0..1, i = 0..3) sits at byte
// 16 (2 w + h) + 4 i + b: the order in which (word >> (4h + i)) & 0x01010101 delivers the sign bits of a code word.
__host__ __device__ inline int qhat_mfma_pos(int d) {
  const int c = d >> 6, r = d & 63, w = r >> 5, x = r & 31;
  return 64 * c + 16 * (2 * w + ((x >> 2) & 1)) + 4 * (x & 3) + (x >> 3);
}

// The same digit in the group scan's operand, an 8-bit float (e4m3) of qhat times the 2, 1, 0.5 or 2 that undoes the 0.5, 1,
// 2 or 0.5 a sign bit in place s of a nibble stands for, and its byte.
__device__ inline uint32_t qhat_fp8(int qh, int s) {
  const uint32_t m = (uint32_t)abs(qh);
  const uint32_t lo = s == 1 ? 0x44403800u : (s == 2 ? 0x3c383000u : 0x4c484000u);  // for |qhat| = 0..3
  const uint32_t hi = s == 1 ? 0x4e4c4a48u : (s == 2 ? 0x46444240u : 0x56545250u);  // 4..7
  return (((m < 4 ? lo : hi) >> (8 * (m & 3))) & 255u) | (qh < 0 ? 128u : 0u);
}
__host__ __device__ inline int qhat_fp8_pos(int d) {
  const int w = d >> 5, n = (d & 31) >> 2, s = d & 3;
  return 64 * (w >> 1) + 16 * (2 * (w & 1) + (s >> 1)) + 8 * (s & 1) + n;
}

// ---------------------------------------------------------------------------------
// Section 3.3.3 / 3.4.1(2): the per-query representation of one rotated query x[0..D), by one wavefront:
// 4-bit signed quantisation and its bit-planes, sums, the query in refinement order, lookup tables.
// delta = max|q'|/7 and q'/delta use IEEE fp32 division and round-half-even, because they decide integers.
// prep_reduce is the first half on its own (max |x|, sum, squared norm, each the same in every lane afterwards);
// whoever needs only the squared norm calls it and gets the very bits query_prep_row stores.
// ---------------------------------------------------------------------------------
__device__ inline void prep_reduce(const float* x, int D, int lane, float& amax, float& s1, float& s2) {
  amax = 0.f; s1 = 0.f; s2 = 0.f;
  for (int i = lane; i < D; i += 64) {
    const float v = x[i];
    amax = fmaxf(amax, fabsf(v));
    s1 += v;
    s2 += v * v;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    amax = fmaxf(amax, __shfl_xor(amax, d, 64));
    s1 += __shfl_xor(s1, d, 64);
    s2 += __shfl_xor(s2, d, 64);
  }
}

// form (QueryForm): what a search's own scans read, in the same space: the refinement's digits (below) instead of q' in
// q_stage, the group scan's operand instead of bytes in qhat8.
template <int F>
__device__ inline void query_prep_row(const float* x, int64_t q, int D, const rabitq_query_repr& o, int lane, int form) {
  const int W = D >> 5;
  const int Dp = (D + 63) / 64 * 64;
  float amax, s1, s2;
  prep_reduce(x, D, lane, amax, s1, s2);
  const float dl = (amax == 0.f) ? 1.0f : __fdiv_rn(amax, 7.0f);
  if ((form & QUERY_DIGITS) != 0 && F > 0) {
    constexpr int FF = F == 0 ? 8 : F, DPW = 32 / FF, SPB = 8 / FF;
    const float factor = digit_factor(dl);
    uint32_t* out = reinterpret_cast<uint32_t*>(o.q_stage) + q * D;
    for (int i = lane; i < D / 4; i += 64) {  // positions 4i .. 4i+3 of the refinement order
      const float* src = x + i / SPB * DPW + i % SPB;
      const uint4 d = digit_quad(make_float4(src[0], src[SPB], src[2 * SPB], src[3 * SPB]), factor);
      out[i] = d.x; out[D / 4 + i] = d.y; out[D / 2 + i] = d.z; out[3 * (D / 4) + i] = d.w;
    }
  } else {
    for (int i = lane; i < D; i += 64) o.q_stage[q * D + (F == 0 ? i : stage_index<(F == 0 ? 8 : F)>(i))] = x[i];
  }
  int S = 0;
  uint32_t* pl = o.planes + q * 4 * W;
  for (int base = 0; base < Dp; base += 64) {
    const int i = base + lane;
    int qh = 0;
    if (i < D && amax != 0.f) {
      const float t = rintf(__fdiv_rn(x[i], dl));
      qh = (int)fminf(fmaxf(t, -7.f), 7.f);
    }
    S += qh;
    if ((form & QUERY_FP8) != 0) o.qhat8[q * Dp + qhat_fp8_pos(i)] = (int8_t)qhat_fp8(qh, i & 3);
    else o.qhat8[q * Dp + qhat_mfma_pos(i)] = (int8_t)qh;
    const uint32_t tc = (uint32_t)qh & 15u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint64_t m = __ballot((tc >> j) & 1u);
      const int w = base >> 5;
      if (lane == 0 && w < W) pl[j * W + w] = (uint32_t)m;
      if (lane == 0 && w + 1 < W) pl[j * W + w + 1] = (uint32_t)(m >> 32);
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) S += __shfl_xor(S, d, 64);
  // Section 3.4.1(1): lookup tables, one entry per (block of 4 dimensions, 4-bit pattern); the sum runs in
  // fp32 over the set bits in ascending dimension order and is rounded to binary16
  if (o.lut != nullptr) {
    _Float16* lut = reinterpret_cast<_Float16*>(o.lut) + q * (int64_t)D * 4;
    for (int e = lane; e < D * 4; e += 64) {
      const int j = e >> 4, b = e & 15;
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((b >> i) & 1) acc += x[4 * j + i];
      lut[e] = (_Float16)acc;
    }
  }
  if (lane == 0) {
    o.delta[q] = dl;
    o.sum_qhat[q] = S;
    o.sum_q[q] = s1;
    o.sq_norm[q] = s2;
  }
}

// ---------------------------------------------------------------------------------
// Section 3.3.2: the K <= 64 smallest of row[0..n) as (order-preserving score bits << 32 | index), by one
// wavefront that reads the row once through a register-resident sorted list.
// ---------------------------------------------------------------------------------
__device__ inline WaveTopK stream_select_smallest(const float* __restrict__ row, int nlist, int nprobe, int lane) {
  WaveTopK top;
  // The first 16 tiles (1024 scores) are held in registers: the 64 per-lane minima start the sorted list, so
  // its nprobe-th key is small from the outset and few of the remaining scores have to be inserted.
  constexpr int R = 16;
  {
    // (unconditional loads of clamped indices, all requested before the first value is touched: a load whose value
    // is only used under a condition would otherwise be waited for before the next one is issued)
    float sv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) sv[r] = __builtin_nontemporal_load(row + min(r * 64 + lane, nlist - 1));
#pragma unroll
    for (int r = 0; r < R; ++r) sv[r] = pinned(sv[r]);
    uint32_t ord[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ord[r] = (r * 64 + lane < nlist) ? f2ord(sv[r]) : 0xffffffffu;
    uint32_t mo = ord[0];
    int mr = 0;
#pragma unroll
    for (int r = 1; r < R; ++r)
      if (ord[r] < mo) { mo = ord[r]; mr = r; }  // ties keep the lower index, as the key order does
    top.init_sorted(mo == 0xffffffffu ? KEY_NONE : (((uint64_t)mo << 32) | (uint32_t)(mr * 64 + lane)), lane);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (r * 64 < nlist) {
        const bool take = r != mr && ord[r] != 0xffffffffu;
        top.push_tile(take ? (((uint64_t)ord[r] << 32) | (uint32_t)(r * 64 + lane)) : KEY_NONE, nprobe, lane);
      }
    }
  }
  // the rest of the row, eight tiles of scores in flight; a tile is only looked at closely when its smallest
  // score beats the current nprobe-th key
  for (int tb = R * 64; tb < nlist; tb += 512) {
    float sc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) sc[u] = __builtin_nontemporal_load(row + min(tb + u * 64 + lane, nlist - 1));
#pragma unroll
    for (int u = 0; u < 8; ++u) sc[u] = pinned(sc[u]);
#pragma unroll
    for (int u = 0; u < 8; ++u) sc[u] = (tb + u * 64 + lane < nlist) ? sc[u] : INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (tb + u * 64 < nlist) {
        const int i = tb + u * 64 + lane;
        top.push_tile((i < nlist) ? make_key(sc[u], (uint32_t)i) : KEY_NONE, nprobe, lane);
      }
    }
  }
  return top;
}

// Largest c in [0, n) with off[c] <= v, for a non-decreasing array off[0..n] with off[0] <= v < off[n]
// (any v >= off[n] gives n - 1).  One wavefront, 64-ary: every level is a single coalesced load and a ballot,
// so the chain of dependent loads is ceil(log64(n + 1)) long.  Every index read is within [0, n].
__device__ inline int wave_upper_cluster(const int32_t* __restrict__ off, int n, int v, int lane) {
  int stride = 1;
  while ((int64_t)stride * 64 < (int64_t)n + 1) stride *= 64;
  int base = 0;
  for (; stride >= 1; stride >>= 6) {
    const int64_t idx = (int64_t)base + (int64_t)lane * stride;
    const bool in = idx < n;
    const int val = off[in ? idx : n];
    const uint64_t m = __ballot(in && val <= v);
    const int cnt = __popcll(m);
    base += (cnt > 0 ? cnt - 1 : 0) * stride;
  }
  return base;
}

// ---------------------------------------------------------------------------------
// Running sums over the lists of an index (pair offsets, work-item tables) by ONE workgroup of NT threads.
// A thread takes SCAN_PER consecutive entries of a chunk, whose loads are independent of one another, so that a
// chunk of 8192 lists costs one round of memory latency and two barriers; the sums of NV values travel together.
// NT: 256 where one chunk of 2048 holds all lists (a launch of 1024 threads starts about 1 us later), 1024 otherwise.
// excl[v] becomes the sum of all entries before this thread's, carry[v] the sum up to the end of the chunk.
// ---------------------------------------------------------------------------------
constexpr int SCAN_PER = 8, SCAN_SMALL = 256, SCAN_LARGE = 1024;

template <int NT, int NV>
__device__ inline void block_chunk_scan(const uint32_t (&sum)[NV], uint32_t (&excl)[NV], uint32_t (&carry)[NV],
                                        uint32_t (*s_wave)[NT / 64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) incl[v] = sum[v];
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const uint32_t o = __shfl_up(incl[v], d, 64);
      if (lane >= d) incl[v] += o;
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v)
    if (lane == 63) s_wave[v][wave] = incl[v];
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    // (lanes 0..15 hold the wavefronts' totals; every wavefront adds up those before it and all of them)
    const uint32_t t = lane < NT / 64 ? s_wave[v][lane] : 0u;
    const uint32_t before = wave_reduce_u32(lane < wave ? t : 0u, [](uint32_t a, uint32_t b) { return a + b; });
    const uint32_t all = wave_reduce_u32(t, [](uint32_t a, uint32_t b) { return a + b; });
    excl[v] = carry[v] + before + incl[v] - sum[v];
    carry[v] += all;
  }
  __syncthreads();  // s_wave is free for the next chunk
}

__host__ __device__ inline int next_pow2(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

// ---------------------------------------------------------------------------------
// Section 3.4.1(2): <x_b, qhat> = -8 pc(x&q3) + 4 pc(x&q2) + 2 pc(x&q1) + pc(x&q0),
// 32 dimensions per AND + popcount.  `pl` points at the query's planes [4][W]; it is
// wave-uniform, so the compiler keeps the plane words in scalar registers.
// ---------------------------------------------------------------------------------
typedef const uint32_t __attribute__((address_space(4)))* const_u32_ptr;
typedef const uint64_t __attribute__((address_space(4)))* const_u64_ptr;

// popcount(x) + acc in one VALU instruction (the compiler otherwise splits the add off)
__device__ inline uint32_t bcnt_acc(uint32_t x, uint32_t acc) {
  uint32_t d;
  asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(d) : "v"(x), "v"(acc));
  return d;
}

template <int W>
__device__ inline int ip_bitplanes(const uint32_t (&cw)[W], const_u32_ptr pl) {
  uint32_t p0 = 0, p1 = 0, p2 = 0, p3 = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    p0 = bcnt_acc(cw[w] & pl[0 * W + w], p0);
    p1 = bcnt_acc(cw[w] & pl[1 * W + w], p1);
    p2 = bcnt_acc(cw[w] & pl[2 * W + w], p2);
    p3 = bcnt_acc(cw[w] & pl[3 * W + w], p3);
  }
  // p0 + 2 p1 + 4 p2 - 8 p3 in three instructions
  uint32_t t;
  asm("v_lshl_add_u32 %0, %1, 1, %2" : "=v"(t) : "v"(p1), "v"(p0));
  asm("v_lshl_add_u32 %0, %1, 2, %2" : "=v"(t) : "v"(p2), "v"(t));
  int r;
  asm("v_mad_i32_i24 %0, %1, -8, %2" : "=v"(r) : "v"(p3), "v"(t));
  return r;
}

// ---------------------------------------------------------------------------------
// Refinement (Section 3.4.2: lanes cooperate on one candidate).  The long code holds the
// whole B-bit code of every dimension in F-bit fields (F = 2, 4, 8), LW = D*F/32 words per
// vector.  <u, q'> of 16 candidates against 4 queries is one chain of v_mfma_i32_16x16x64_i8: the fields u are bytes
// as they come (masked out of a word four at a time), and q' is a 30-bit fixed-point number cut into four signed bytes
// ("digits"), so that the 16 rows of the left operand are 4 queries x 4 digits and a lane's four results are the four
// digit sums of ONE query, exact integers, whatever the order of the sum.  Lane (lj, g) = (lane % 16, lane / 16) feeds
// part g of candidate lj and receives candidate lj against query g.
// What bounds it: nothing in the arithmetic (2 matrix and ~50 vector instructions per 16 candidates of 128 x 4 bits,
// about 190 when each of 4 lanes converted and multiplied 32 fields in fp32 and the partial sums were added across lanes).
//
// Digits.  With 2^x <= delta < 2^(x+1) (delta = max|q'|/7, so |q'| < 2^(x+4)), Q = rint(q' * 2^(26-x)) < 2^30, an error of
// at most 2^(x-27) <= max|q'| * 2^-29.8 per dimension, below the rounding of the 32-bit sum it replaces;
// Q = d0 + 2^8 d1 + 2^16 d2 + 2^24 d3 with -128 <= d <= 127.  Stored [query][digit][D/4] dwords, four consecutive
// positions of the refinement order (stage_index) per dword.
// ---------------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));

template <int F>
__host__ __device__ inline int stage_index(int d) {
  constexpr int DPW = 32 / F, SPB = 8 / F;
  const int w = d / DPW, r = d % DPW;
  return w * DPW + (r % SPB) * 4 + (r / SPB);
}

// biased exponent of delta, kept where both powers of two below are normal numbers
__device__ inline uint32_t digit_exponent(float delta) { return min(max((__float_as_uint(delta) >> 23) & 255u, 27u), 253u); }
__device__ inline float digit_factor(float delta) { return __uint_as_float((280u - digit_exponent(delta)) << 23); }  // 2^(26-x)
__device__ inline float digit_unit(float delta) { return __uint_as_float((digit_exponent(delta) - 26u) << 23); }     // 2^(x-26)

// the four digits of one value, a byte each (the largest byte sum is 0x7f7f7f7f)
__device__ inline uint32_t digits_of(float q, float factor) {
  const float v = fminf(fmaxf(rintf(q * factor), -2139062016.f), 2139062016.f);
  return ((uint32_t)(int)v + 0x80808080u) ^ 0x80808080u;
}

__device__ inline float4 four_floats(const float* p) { return make_float4(p[0], p[1], p[2], p[3]); }  // (any alignment)

// four values -> a dword per digit, value i in byte i
__device__ inline uint4 digit_quad(float4 q, float factor) {
  const uint32_t a = digits_of(q.x, factor), b = digits_of(q.y, factor), c = digits_of(q.z, factor), d = digits_of(q.w, factor);
  const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x05010400u), cd = __builtin_amdgcn_perm(d, c, 0x05010400u);
  const uint32_t ab2 = __builtin_amdgcn_perm(b, a, 0x07030602u), cd2 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  return make_uint4(__builtin_amdgcn_perm(cd, ab, 0x05040100u), __builtin_amdgcn_perm(cd, ab, 0x07060302u),
                    __builtin_amdgcn_perm(cd2, ab2, 0x05040100u), __builtin_amdgcn_perm(cd2, ab2, 0x07060302u));
}

// one digit of them, from memory
__device__ inline uint32_t digit_of_quad(const float* p, float factor, int digit) {
  const uint4 d = digit_quad(four_floats(p), factor);
  uint32_t v = digit == 0 ? d.x : (digit == 1 ? d.y : (digit == 2 ? d.z : d.w));
  asm volatile("" : "+v"(v)::"memory");  // (one after the other: many of them in flight would cost every kernel registers)
  return v;
}

// How the words of a long-code row are dealt to the four lanes of a candidate: 16 words at a time, four consecutive ones
// per lane (so that the four lanes read 64 contiguous bytes), and the last LW % 16 in four runs of RW.
template <int F, int LW>
struct RefineShape {
  static constexpr int UNITS = LW / 16, RW = (LW % 16 + 3) / 4;
  static constexpr int WPL = 4 * UNITS + RW;      // words per lane
  static constexpr int QPW = 8 / F;               // operand dwords a word expands to
  static constexpr int DW = WPL * QPW;            // operand dwords per lane
  static constexpr int KC = (DW + 3) / 4;         // matrix instructions per 16 candidates
  static constexpr int NS = 16;                   // candidates per round
  static constexpr bool EVEN = 16 * UNITS + 4 * RW == LW;  // the last part's runs end with the row
  static constexpr bool IN_REGS = KC <= 4;        // the query operand of a work item lives in registers (else in LDS)
  static constexpr int ROW = LW * QPW + 4;        // ... dwords of a digit row there (padded: rows start in other banks)
  static constexpr int LDS_WORDS = IN_REGS ? 0 : 4 * ROW;  // ... dwords per query
  __device__ static inline int word(int i, int g) { return i < 4 * UNITS ? 16 * (i / 4) + 4 * g + i % 4 : 16 * UNITS + RW * g + i - 4 * UNITS; }
};

// the words of one candidate this lane feeds (every address is inside the row)
template <int F, int LW>
__device__ inline void refine_load(const uint32_t* __restrict__ row, int g, uint32_t (&w)[RefineShape<F, LW>::WPL]) {
  using S = RefineShape<F, LW>;
#pragma unroll
  for (int u = 0; u < S::UNITS; ++u) {
    if (LW % 4 == 0) {  // rows start at multiples of 16 bytes
      const uint4 v = *reinterpret_cast<const uint4*>(row + 16 * u + 4 * g);
      w[4 * u] = v.x; w[4 * u + 1] = v.y; w[4 * u + 2] = v.z; w[4 * u + 3] = v.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) w[4 * u + i] = row[16 * u + 4 * g + i];
    }
  }
#pragma unroll
  for (int i = 0; i < S::RW; ++i) {
    const int at = 16 * S::UNITS + S::RW * g + i;
    w[4 * S::UNITS + i] = row[S::EVEN ? at : min(at, LW - 1)];
  }
}

// dword c of the candidate operand.  (8-bit codes: flip turns 0..255 into -128..127; it is 0 for shorter codes)
template <int F>
__device__ inline uint32_t refine_field(uint32_t word, int s, uint32_t flip) {
  if (F == 8) return word ^ flip;
  return (word >> (F * s)) & (((1u << F) - 1u) * 0x01010101u);
}

// dword c of the query operand of lane (., g), whose left row of digits is at `row`
template <int F, int LW>
__device__ __forceinline__ uint32_t query_operand(const uint32_t* row, int c, int g) {
  using S = RefineShape<F, LW>;
  const int w = S::word(c / S::QPW, g);
  const bool whole = c / S::QPW < 4 * S::UNITS;  // (a word of the last, incomplete part may lie past the row)
  const uint32_t v = row[(whole ? w : min(w, LW - 1)) * S::QPW + c % S::QPW];
  return whole || w < LW ? v : 0u;
}
// the whole of it in registers
template <int F, int LW>
__device__ __forceinline__ void load_query_operand(const uint32_t* row, int g, v4i (&qa)[RefineShape<F, LW>::KC]) {
  using S = RefineShape<F, LW>;
#pragma unroll
  for (int kc = 0; kc < S::KC; ++kc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) qa[kc][i] = 4 * kc + i < S::DW ? (int)query_operand<F, LW>(row, 4 * kc + i, g) : 0;
  }
}
// The four digit rows of one query, `stride` dwords apart, written by one wavefront: copied from the digits, or made from
// q' (the stage entry points, whose callers hand in q' and no digits).
template <int D>
__device__ __forceinline__ void stage_digits(uint32_t* dst, int stride, const uint32_t* digits, const float* q_stage, float factor, int64_t q, int lane) {
  constexpr int NQ = D / 4;
  if (digits != nullptr) {
#pragma unroll
    for (int i0 = 0; i0 < NQ; i0 += 64) {
      const int i = i0 + lane;
      if (i < NQ) {
        const uint32_t* src = digits + q * D + i;
        dst[i] = src[0]; dst[stride + i] = src[NQ]; dst[2 * stride + i] = src[2 * NQ]; dst[3 * stride + i] = src[3 * NQ];
      }
    }
  } else {
#pragma unroll 1
    for (int i = lane; i < NQ; i += 64) {
      const uint4 d = digit_quad(four_floats(q_stage + q * D + 4 * i), factor);
      dst[i] = d.x; dst[stride + i] = d.y; dst[2 * stride + i] = d.z; dst[3 * stride + i] = d.w;
    }
  }
}

// digit sums of candidate lane % 16 against query lane / 16; operand(kc) gives the query operand of step kc
template <int F, int LW, typename Operand>
__device__ __forceinline__ v4i refine_mfma(const uint32_t (&w)[RefineShape<F, LW>::WPL], uint32_t flip, Operand operand) {
  using S = RefineShape<F, LW>;
  v4i acc = v4i{0, 0, 0, 0};
#pragma unroll
  for (int kc = 0; kc < S::KC; ++kc) {
    v4i x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = 4 * kc + i;
      x[i] = c < S::DW ? (int)refine_field<F>(w[c < S::DW ? c / S::QPW : 0], c % S::QPW, flip) : 0;
    }
    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(operand(kc), x, acc, 0, 0, 0);
  }
  return acc;
}

// One of a query's four digit rows.
struct DigitRow {
  const uint32_t* row;
  __device__ __forceinline__ v4i four(int at) const { return *reinterpret_cast<const v4i*>(row + at); }
  __device__ __forceinline__ uint32_t one(int at) const { return row[at]; }
};
// The same, or made from q' where there are no digits: again for every candidate, which a stage entry point only does where it
// may not allocate the memory for them (launch_scan).
struct DigitRowOrQuery {
  const uint32_t* row;  // nullptr: none
  const float* q_stage;
  float factor;
  int digit;
  __device__ __forceinline__ DigitRowOrQuery(const uint32_t* digits, const float* q, float f, int64_t index, int d, int D)
      : row(digits != nullptr ? digits + index * D + d * (D / 4) : nullptr), q_stage(q + index * D), factor(f), digit(d) {}
  __device__ __forceinline__ v4i four(int at) const {
    if (row != nullptr) return *reinterpret_cast<const v4i*>(row + at);
    v4i v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (int)digit_of_quad(q_stage + 4 * (at + i), factor, digit);
    return v;
  }
  __device__ __forceinline__ uint32_t one(int at) const { return row != nullptr ? row[at] : digit_of_quad(q_stage + 4 * at, factor, digit); }
};

// The same sums with both operands read where they are needed: for kernels that refine little and have better uses for their
// registers meanwhile (seeding, the matrix-core scans' lists of wide codes), U units of both in flight.  `row`: this lane's candidate;
// `query`: its left row (DigitRow, or what else gives four dwords and one).
template <int F, int LW, int U = 16, typename Query>
__device__ __forceinline__ v4i refine_mfma_from_memory(const uint32_t* __restrict__ row, const Query query, int g, uint32_t flip) {
  using S = RefineShape<F, LW>;
  v4i acc = v4i{0, 0, 0, 0};
  auto unit = [&](int u) __attribute__((always_inline)) {
    uint32_t w[4];
    if (LW % 4 == 0) {
      const uint4 v = *reinterpret_cast<const uint4*>(row + 16 * u + 4 * g);
      w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = row[16 * u + 4 * g + i];
    }
#pragma unroll
    for (int h = 0; h < S::QPW; ++h) {  // 4 / QPW words per instruction
      const int at = (16 * u + 4 * g) * S::QPW + 4 * h;
      const v4i qa = query.four(at);
      v4i x;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = (int)refine_field<F>(w[(4 * h + i) / S::QPW], (4 * h + i) % S::QPW, flip);
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(qa, x, acc, 0, 0, 0);
    }
  };
  if (S::UNITS <= U) {
#pragma unroll
    for (int u = 0; u < S::UNITS; ++u) unit(u);
  } else {
    constexpr int STEP = S::UNITS % 5 == 0 ? 5 : (S::UNITS % 4 == 0 ? 4 : (S::UNITS % 3 == 0 ? 3 : 1));
#pragma unroll 1
    for (int u0 = 0; u0 < S::UNITS; u0 += STEP) {
#pragma unroll
      for (int u = 0; u < STEP; ++u) unit(u0 + u);
    }
  }
  if (S::RW > 0) {
    constexpr int W0 = 4 * S::UNITS, RD = S::RW * S::QPW;  // words before the last part, its operand dwords
    uint32_t w[S::RW > 0 ? S::RW : 1];
#pragma unroll
    for (int i = 0; i < S::RW; ++i) w[i] = row[min(16 * S::UNITS + S::RW * g + i, LW - 1)];
#pragma unroll
    for (int kc = 0; kc < (RD + 3) / 4; ++kc) {
      v4i qa, x;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = 4 * kc + i;
        const int at = min(16 * S::UNITS + S::RW * g + (c < RD ? c / S::QPW : 0), LW - 1) * S::QPW + c % S::QPW;
        uint32_t v = 0u;
        if (c < RD) v = query.one(at);
        qa[i] = 16 * S::UNITS + S::RW * g + (c < RD ? c / S::QPW : 0) < LW ? (int)v : 0;
        x[i] = c < RD ? (int)refine_field<F>(w[c < RD ? c / S::QPW : 0], c % S::QPW, flip) : 0;
      }
      acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(qa, x, acc, 0, 0, 0);
    }
  }
  return acc;
}

// <u, q'> (u: fields as the operand has them) from the four digit sums, none larger than 2^24
__device__ inline float digit_sum(v4i d, float unit) {
  return unit * fmaf(256.f, fmaf(256.f, fmaf(256.f, (float)d[3], (float)d[2]), (float)d[1]), (float)d[0]);
}

// ---------------------------------------------------------------------------------
// Shared by the matrix-core variants of the scan.
// ---------------------------------------------------------------------------------
// 16 sign bits of a code word -> 16 bytes of 0/1 for the matrix instruction's B operand, at two instructions per
// four bytes: (word >> s) & 0x01010101 leaves bits s, s+8, s+16, s+24 of the word in the four bytes.  The lane
// group with half h (0 / 1) of a word takes the shifts s = 4h .. 4h+3, so byte b of its i-th operand word is dimension
// 4h + i + 8b of the code word, and the query's qhat bytes are stored in that same order (qhat_mfma_pos).
__device__ inline v4i expand_half(uint32_t word, int h) {
  const uint32_t v = word >> (4 * h);
  v4i x;
  x.x = (int)(v & 0x01010101u);
  x.y = (int)((v >> 1) & 0x01010101u);
  x.z = (int)((v >> 2) & 0x01010101u);
  x.w = (int)((v >> 3) & 0x01010101u);
  return x;
}

__device__ inline void wave_sync() {  // orders LDS traffic among the lanes of one wavefront
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// bitonic sort of n = 2^m keys in LDS by ONE wavefront of a larger workgroup (no workgroup barrier)
__device__ inline void wave_bitonic_sort(uint64_t* keys, int n, int lane) {
  for (int k = 2; k <= n; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      wave_sync();
      for (int t = lane; t < (n >> 1); t += 64) {
        const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
        const int l = i | j;
        const uint64_t x = keys[i], y = keys[l];
        const bool up = (i & k) == 0;
        if ((x > y) == up) {
          keys[i] = y;
          keys[l] = x;
        }
      }
    }
  }
  wave_sync();
}

__device__ inline int wave_pool_compact(uint64_t* pool, int pool_n, int cnt, int k, int lane) {
  wave_sync();
  for (int i = cnt + lane; i < pool_n; i += 64) pool[i] = KEY_NONE;
  wave_bitonic_sort(pool, pool_n, lane);
  return min(cnt, k);
}

}  // namespace rq
