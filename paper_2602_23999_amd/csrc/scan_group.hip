// Cluster-local search of 16 pairs per wavefront, estimates and refinement both on the matrix cores (Sections 3.3.4, 3.4.1(2),
// 3.4.2): the form of the scan for batches in which many queries share a list.
//
// A work item is a group of up to 16 pairs of one cluster (NARROW: codes of up to 256 dimensions) or that times a segment of its
// tiles (wide codes); one wavefront does all of it: estimates (TileEstimator), survivors to four lists in LDS, one per 4
// pairs, a list's candidates refined 16 at a time against its 4 queries (RefineShape).
// NARROW: four times 16 candidates in flight together, from whichever lists are longest; the queries' digits are read
// from LDS, 64 rows, the four-dword pieces of a row permuted by its number so that 16 rows spread over the banks.  (In
// registers, 32 of them, they allow three wavefronts per SIMD instead of four, and four candidates' worth of every list had to
// be taken at a time, full or not.)  The keys go straight to the pair's region of the candidate array, which is cut to the k
// best when it is full.  (Pools in LDS, cut to the k best when full, cost a third of the wavefronts in flight at k = 100 and a cut
// every 28 keys.)  A list is not cut into segments: group_wanted keeps out the indices whose longest list would outlast the
// rest of the launch.
// Wide codes: 16 queries' digits would leave room for two or three wavefronts per compute unit; they are read from memory with
// the candidates, which pays where few vectors survive (960 dimensions).  LDS is free for pools, so a list may be scanned in
// segments by several items, each contributing at most k keys to the pair's region.
#include <algorithm>

#include "rq_estimate.h"

namespace rq {

constexpr int GLISTS = 4;
constexpr int GROUNDS = 4;                          // times 16 candidates in flight
// A list holds less than 16 GROUNDS entries before a tile, and a tile is filed in parts of at most 16 vectors x 4 pairs when it
// might add more than there is room for.
constexpr int GLIST_CAP = 16 * GROUNDS + 64;

template <int W, int F, bool DBG>
__device__ __forceinline__ void scan_group_item(const ScanArgs& a, const int item) {
  constexpr int LW = W * F, D = 32 * W;
  constexpr bool NARROW = group_narrow(W);
  using RS = RefineShape<F, LW>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int NQ = D / 4;                                                       // dwords of a digit row
  float4* scal = reinterpret_cast<float4*>(smem_raw);                             // [QM] G, cB * sum(q'), unit of the digits, pair
  float4* est_pair = scal + QM;                                                   // [QM] TileEstimator's
  uint64_t* s_kth = reinterpret_cast<uint64_t*>(est_pair + QM);                     // [QM] only keys up to this one count
  uint32_t* lists = reinterpret_cast<uint32_t*>(s_kth + QM);                      // [GLISTS][GLIST_CAP]
  uint32_t* qdig = lists + GLISTS * GLIST_CAP;                                    // [QM * 4][NQ] (NARROW)
  uint64_t* pools = reinterpret_cast<uint64_t*>(qdig);                            // [QM][pool] (wide codes)
  static_assert(GLISTS * GLIST_CAP * 4 >= ESTIMATE_SCRATCH, "the lists' memory serves the estimator's set-up");
  int lane = threadIdx.x;
  asm volatile("" : "+v"(lane));  // (opaque: what follows from the lane would be kept in registers from one item to the next)
  const int lj = lane & 15, g = lane >> 4;

  typedef const ItemDesc __attribute__((address_space(4)))* const_desc_ptr;
  const_desc_ptr ds = (const_desc_ptr)(a.item_desc + item);
  const int pbeg = ds->pbeg, np = ds->np_mg & 255, t0 = ds->t0, ts = ds->ts, te = ds->te, nseg = ds->nseg;

  TileEstimator<W, DBG> est;
  if (ts < te) est.fetch(a, ts, lj, g);
  // pair lj of the group (an absent one repeats the last)
  const int pp = a.pair_ids[pbeg + min(lj, np - 1)];
  const int q = pair_query(a, pp);
  float G, dl;
  est.pairs(a, pp, q, np, reinterpret_cast<int8_t*>(lists), est_pair, lane, G, dl);
  if (lane < QM) scal[lane] = make_float4(G, a.cB * a.sum_q[q], digit_unit(dl), __int_as_float(pp));

  // The digits: row 4 j + d is digit d of query j, and piece c (four dwords) of row x is kept at place c ^ (x % 8) % pieces.
  constexpr int PIECES = NQ / 4, PMASK = (PIECES < 8 ? PIECES & -PIECES : 8) - 1;
  if (!NARROW) {
  } else if (a.q_digits != nullptr) {
#pragma unroll
    for (int i0 = 0; i0 < 64 * PIECES; i0 += 64) {
      const int i = i0 + lane, row = i / PIECES, c = i % PIECES;
      const uint4 v = *reinterpret_cast<const uint4*>(a.q_digits + (int64_t)__shfl(q, row >> 2, 64) * D + (row & 3) * NQ + 4 * c);
      *reinterpret_cast<uint4*>(qdig + row * NQ + 4 * (c ^ (row & PMASK))) = v;
    }
  } else {
#pragma unroll 1
    for (int j = 0; j < QM; ++j) {
      const int qj = __builtin_amdgcn_readlane(q, j);
      for (int i = lane; i < NQ; i += 64) {
        const uint4 d = digit_quad(four_floats(a.q_stage + (int64_t)qj * D + 4 * i), digit_factor(a.delta[qj]));
        const uint32_t v[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) qdig[(4 * j + r) * NQ + 4 * ((i >> 2) ^ ((4 * j + r) & PMASK)) + (i & 3)] = v[r];
      }
    }
  }

  // keys that pair 4 l + g holds, and the length of list g, in every lane of the group
  int pcnt[GLISTS], lcnt = 0;
#pragma unroll
  for (int l = 0; l < GLISTS; ++l) pcnt[l] = 0;
  if (lane < QM) s_kth[lane] = KEY_NONE;
  if (lj == 0) lists[g * GLIST_CAP] = 0u;  // (an empty list's first entry is read below, for a candidate that does not count)
  wave_sync();

  const int room = NARROW ? a.cand_stride : a.pool;  // keys a pair can hold, at least k + 16 ROUNDS
  // cuts every pair that holds more than `limit` >= k keys to its k best
  auto cut_above = [&](int limit) {
    if (__ballot(max(max(pcnt[0], pcnt[1]), max(pcnt[2], pcnt[3])) > limit) == 0ull) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll 1
    for (int p = 0; p < np; ++p) {
      const int l = p >> 2, gg = p & 3;
      const int c = __builtin_amdgcn_readlane(one_of(l, pcnt[0], pcnt[1], pcnt[2], pcnt[3]), 16 * gg);
      if (c <= limit) continue;
      uint64_t* region = a.cand_keys + (int64_t)__builtin_amdgcn_readlane(pp, p) * a.cand_stride;
      uint64_t* pool = pools + (size_t)p * a.pool;
      constexpr int RB = 4;  // (at most 256 keys)
      uint64_t key[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int i = r * 64 + lane;
        key[r] = KEY_NONE;
        if (i < c) key[r] = NARROW ? region[i] : pool[i];
      }
      wave_sync();
      int left = 0;
      const uint64_t last = wave_keep_best<RB>(key, a.k, lane, &left, [&](int at, uint64_t v) { (NARROW ? region : pool)[at] = v; });
      if (lane == 0) s_kth[p] = last;
#pragma unroll
      for (int u = 0; u < GLISTS; ++u) pcnt[u] = u == l && g == gg ? left : pcnt[u];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };

  constexpr int ROUNDS = NARROW ? GROUNDS : 1;  // times 16 candidates in flight
  // Refines ROUNDS times the last 16 entries of the longest list, as long as there are so many (everything: until the lists
  // are empty).  The rounds' candidates are fetched together; nothing is fetched under a condition.
  auto refine = [&](bool everything) {
    while (true) {
      int c[GLISTS];
#pragma unroll
      for (int l = 0; l < GLISTS; ++l) c[l] = __builtin_amdgcn_readlane(lcnt, 16 * l);
      if (everything ? c[0] + c[1] + c[2] + c[3] == 0 : (c[0] >> 4) + (c[1] >> 4) + (c[2] >> 4) + (c[3] >> 4) < GROUNDS) break;
      wave_sync();
      cut_above(room - 16 * ROUNDS);
      uint32_t w[ROUNDS][RS::WPL], e[ROUNDS];
      float2 lf[ROUNDS];
      int64_t slot[ROUNDS];
      int id[ROUNDS], list[ROUNDS], n[ROUNDS];
#pragma unroll
      for (int d = 0; d < ROUNDS; ++d) {
        const int m01 = max(c[0], c[1]), m23 = max(c[2], c[3]);
        list[d] = m01 >= m23 ? (c[0] >= c[1] ? 0 : 1) : (c[2] >= c[3] ? 2 : 3);
        n[d] = min(max(m01, m23), 16);
        const int from = max(m01, m23) - n[d];
#pragma unroll
        for (int l = 0; l < GLISTS; ++l) c[l] = list[d] == l ? from : c[l];
        e[d] = lists[list[d] * GLIST_CAP + max(from + min(lj, n[d] - 1), 0)];
        slot[d] = (int64_t)t0 * TILE + (e[d] & 0x3fffffffu);
        if (NARROW) refine_load<F, LW>(a.long_codes + slot[d] * LW, g, w[d]);
        lf[d] = *reinterpret_cast<const float2*>(a.long_factors + 2 * slot[d]);
        id[d] = a.ids[slot[d]];
      }
      lcnt = one_of(g, c[0], c[1], c[2], c[3]);
      // (all rounds' keys before the first is stored: one block without branches, in which the chains overlap)
      uint64_t key[ROUNDS];
      uint64_t* to[ROUNDS];
      bool take[ROUNDS];
#pragma unroll
      for (int d = 0; d < ROUNDS; ++d) {
        const float4 sc = scal[4 * list[d] + g];
        v4i sums;
        if (NARROW) {
          const uint32_t* row = qdig + (16 * list[d] + lj) * NQ;
          sums = refine_mfma<F, LW>(w[d], a.flip, [&](int kc) {
            v4i x;
            if (4 * kc / RS::QPW < 4 * RS::UNITS || RS::RW * RS::QPW % 4 == 0) {  // a step's four dwords are one piece
              const int word = RS::word(4 * kc / RS::QPW, g);
              x = *reinterpret_cast<const v4i*>(row + 4 * ((min(word, LW - 1) * RS::QPW / 4) ^ (lj & PMASK)));
              if (!RS::EVEN && word >= LW) x = v4i{0, 0, 0, 0};
            } else {
  #pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int cc = 4 * kc + i, word = RS::word(cc < RS::DW ? cc / RS::QPW : 0, g), at = min(word, LW - 1) * RS::QPW + cc % RS::QPW;
                x[i] = cc < RS::DW && word < LW ? (int)row[4 * ((at >> 2) ^ (lj & PMASK)) + (at & 3)] : 0;
              }
            }
            return x;
          });
        } else {
          const int j = 4 * list[d] + (lj >> 2);  // the query this lane's left row is of
          const DigitRowOrQuery query(a.q_digits, a.q_stage, digit_factor(__shfl(dl, j, 64)), __shfl(q, j, 64), lj & 3, D);
          sums = refine_mfma_from_memory<F, LW, 7>(a.long_codes + slot[d] * LW, query, g, a.flip);
        }
        const float ip = digit_sum(sums, sc.z);
        const float eB = sc.x + lf[d].x + lf[d].y * (ip - sc.y);
        key[d] = make_key(eB, (uint32_t)id[d]);
        take[d] = lj < n[d] && (int)(e[d] >> 30) == g && key[d] <= s_kth[4 * list[d] + g];
        const uint32_t m = (uint32_t)(__ballot(take[d]) >> (16 * g)) & 0xffffu;  // of this lane's pair
        const int cnt = one_of(list[d], pcnt[0], pcnt[1], pcnt[2], pcnt[3]);
        const int place = cnt + __popc(m & ((1u << lj) - 1u));
        to[d] = NARROW ? a.cand_keys + (int64_t)__float_as_int(sc.w) * a.cand_stride + place
                       : pools + (size_t)(4 * list[d] + g) * a.pool + place;
#pragma unroll
        for (int l = 0; l < GLISTS; ++l) pcnt[l] = list[d] == l ? cnt + __popc(m) : pcnt[l];
      }
#pragma unroll
      for (int d = 0; d < ROUNDS; ++d)
        if (take[d]) *to[d] = key[d];
    }
  };

  uint32_t rest = 0u, pos0 = 0u;  // survivors that are in no list yet
  for (int tile = ts;;) {
    if (__ballot(rest != 0u) == 0ull && tile < te) {
      pos0 = (uint32_t)((tile - t0) * TILE + 4 * lj);
      rest = est.scan(a, min(tile + 1, te - 1), lj, g, [&](int pair, int v, int I) {  // (past the end: a harmless re-read)
        if (pair < np) a.dbg_ip[a.dbg_off[pbeg + pair] + (int64_t)(tile - t0) * TILE + v] = I;
      });
      ++tile;
    }
    if (__ballot(rest != 0u) != 0ull) {
      // all of them, or, where a list might overflow, the first column block's that has any
      uint32_t now = rest;
      int incl, total;
      auto sums = [&]() {  // running sum over the 16 lanes of the group
        incl = __popc(now);
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xF, 0xF, true);  // row_shr:1
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xF, 0xF, true);
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xF, 0xF, true);
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xF, 0xF, true);
        total = __builtin_amdgcn_update_dpp(0, incl, 0x15F, 0xF, 0xF, true);  // row_newbcast:15
      };
      sums();
      if (__ballot(lcnt + total > GLIST_CAP) != 0ull) {
        uint32_t block = 15u;
        while (__ballot((rest & block) != 0u) == 0ull) block <<= 4;
        now = rest & block;
        sums();
      }
      uint32_t* at = lists + g * GLIST_CAP + lcnt + incl - __popc(now);
      rest &= ~now;
      lcnt += total;
      while (now != 0u) {
        const uint32_t b = (uint32_t)__ffs(now) - 1u;
        *at++ = (b << 30) | (pos0 + (b >> 2));
        now &= now - 1u;
      }
    }
    const bool done = tile >= te && __ballot(rest != 0u) == 0ull;
    refine(done);
    if (done) break;
  }

  if (!NARROW && nseg > 1) cut_above(a.k);  // (the segments of a list share the pair's region)
  // lane 16 i + l counts the keys of pair 4 l + i (and reserves their place: the atomics of an item are in flight together)
  const int pair = 4 * (lj & 3) + g;
  const int mine = one_of(lj & 3, pcnt[0], pcnt[1], pcnt[2], pcnt[3]);
  const int pair_pp = __shfl(pp, pair, 64);
  int base = 0;
  if (lj < 4 && pair < np && mine > 0) {
    if (!NARROW && nseg > 1) base = atomicAdd(&a.cand_cnt[pair_pp], mine);
    else a.cand_cnt[pair_pp] = mine;
  }
  if (NARROW) return;
  wave_sync();
#pragma unroll 1
  for (int p = 0; p < np; ++p) {
    const int from = 16 * (p & 3) + (p >> 2);
    const int c = __builtin_amdgcn_readlane(mine, from);
    uint64_t* out = a.cand_keys + (int64_t)__builtin_amdgcn_readlane(pp, p) * a.cand_stride + __builtin_amdgcn_readlane(base, from);
    for (int i = lane; i < c; i += 64) out[i] = pools[(size_t)p * a.pool + i];
  }
}

// Workgroups are dealt round-robin to the 8 XCDs.  Lists are dealt to the XCDs by length, every eighth to the same one (the
// items of one list share an L2), and each XCD takes its own longest first, so that the items that end the launch are short.
// The number of items is only known on the device: the grid is sized for the usual one, and a workgroup goes on to a
// further item of its XCD while there is one.
template <int W, int F, bool DBG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(W <= 4 ? 4 : 2))) void scan_group_kernel(ScanArgs a) {
  const int x = (int)(blockIdx.x & 7);
  const int first = a.item_off[xcd_first(a.nlist, x)], last = a.item_off[xcd_first(a.nlist, x + 1)];
  for (int item = first + (int)(blockIdx.x >> 3); item < last; item += (int)(gridDim.x >> 3)) {
    scan_group_item<W, F, DBG>(a, item);
    wave_sync();  // (the next item starts by overwriting what this one read from LDS last)
  }
}

static size_t group_smem(int W, int pool) {
  return QM * (2 * sizeof(float4) + sizeof(uint64_t)) + GLISTS * GLIST_CAP * sizeof(uint32_t) +
         (group_narrow(W) ? (size_t)QM * 4 * 8 * W * sizeof(uint32_t) : (size_t)QM * pool * sizeof(uint64_t));
}

// Keys of a pair's pool (wide codes): at least 64, and the k best, the 16 that a round may add and 24 more, so that a cut pays for itself.
// (960 dimensions, 5 bits, 965 groups, k = 40: 826 us with 8 more, 749 with 24)
int group_pool(int k) { return std::max(64, (k + 40 + 15) / 16 * 16); }

template <int W, int F>
static void launch_wf(const ScanArgs& a, unsigned grid, bool dbg, hipStream_t st) {
  if (dbg)
    hipLaunchKernelGGL((scan_group_kernel<W, F, true>), dim3(grid), dim3(64), group_smem(W, a.pool), st, a);
  else
    hipLaunchKernelGGL((scan_group_kernel<W, F, false>), dim3(grid), dim3(64), group_smem(W, a.pool), st, a);
}

template <int W>
static void launch_w(const ScanArgs& a, int F, unsigned grid, bool dbg, hipStream_t st) {
  switch (F) {
    case 2: launch_wf<W, 2>(a, grid, dbg, st); break;
    case 4: launch_wf<W, 4>(a, grid, dbg, st); break;
    default: launch_wf<W, 8>(a, grid, dbg, st); break;
  }
}

// Returns false when the kernel is not built for the code width W.
bool scan_group(const ScanArgs& a, int W, int F, unsigned grid, bool dbg, hipStream_t st) {
  switch (W) {
    case 1: launch_w<1>(a, F, grid, dbg, st); return true;
    case 2: launch_w<2>(a, F, grid, dbg, st); return true;
    case 3: launch_w<3>(a, F, grid, dbg, st); return true;
    case 4: launch_w<4>(a, F, grid, dbg, st); return true;
    case 8: launch_w<8>(a, F, grid, dbg, st); return true;
    case 30: launch_w<30>(a, F, grid, dbg, st); return true;
    case 32: launch_w<32>(a, F, grid, dbg, st); return true;
    default: return false;
  }
}

}  // namespace rq
