// Small stages of the search path: per-query representation, probe selection,
// probe-list regrouping and the per-query merge.
#include "rq_device.h"

namespace rq {


// ---------------------------------------------------------------------------------
// Section 3.3.3 / 3.4.1(2): 4-bit signed quantisation of q' and its bit-planes, once
// per query.  One wavefront per query.  delta = max|q'|/7 and q'/delta use IEEE fp32
// division and round-half-even, because they decide integers.
// ---------------------------------------------------------------------------------
template <int F>
__global__ __launch_bounds__(256) void query_prep_kernel(const float* __restrict__ q_rot, int64_t nq, int D,
                                                        rabitq_query_repr o, int form, PrepClear clear) {
  const int lane = threadIdx.x & 63;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < clear.n_bitmap; i += (int64_t)gridDim.x * 256) clear.bitmap[i] = 0u;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < clear.n_counters; i += (int64_t)gridDim.x * 256) clear.counters[i] = 0;
  const int64_t q = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (q >= nq) return;
  query_prep_row<F>(q_rot + q * D, q, D, o, lane, form);
}

// A batch that is too small for a stream of its own to clear the list builder's bitmap and the candidate counters lets its query
// preparation do it: two launches of 3-5 us fewer in a chain of fourteen.  Up to 8 words per thread of that kernel (a few us; beyond
// it the launches of their own have more workgroups to do it with).
PrepClear prep_clear(int64_t nq, int nlist, int nprobe, uint32_t* bitmap, int32_t* counters) {
  const int64_t n_bitmap = (int64_t)nlist * ((nq + 31) / 32), n_counters = nq * nprobe;
  if (n_bitmap + n_counters > 8 * 64 * nq) return PrepClear{};
  return PrepClear{bitmap, n_bitmap, counters, n_counters};
}

int launch_query_prep(const float* q_rot, int64_t nq, int D, int F, const rabitq_query_repr& out, int form,
                      const PrepClear& clear, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  const unsigned grid = (unsigned)((nq + 3) / 4);
  switch (F) {
    case 0: hipLaunchKernelGGL(query_prep_kernel<0>, dim3(grid), dim3(256), 0, st, q_rot, nq, D, out, form, clear); break;
    case 2: hipLaunchKernelGGL(query_prep_kernel<2>, dim3(grid), dim3(256), 0, st, q_rot, nq, D, out, form, clear); break;
    case 4: hipLaunchKernelGGL(query_prep_kernel<4>, dim3(grid), dim3(256), 0, st, q_rot, nq, D, out, form, clear); break;
    default: hipLaunchKernelGGL(query_prep_kernel<8>, dim3(grid), dim3(256), 0, st, q_rot, nq, D, out, form, clear); break;
  }
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

// ---------------------------------------------------------------------------------
// Section 3.3.2: the nprobe best clusters of one score row, best first, ties to the
// lower cluster id (the key's low word).  One workgroup per query.
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void select_probes_kernel(const float* __restrict__ scores,
                                                           const float* __restrict__ sq_norm,
                                                           const float* __restrict__ centroid_sq, int nlist,
                                                           int nprobe, int npad, int metric,
                                                           int32_t* __restrict__ probe_ids,
                                                           float* __restrict__ probe_G,
                                                           float* __restrict__ probe_E) {
  extern __shared__ uint64_t sel_out[];  // [npad]
  __shared__ SelectScratch sh;
  const int64_t q = blockIdx.x;
  const float* row = scores + q * nlist;
  auto key_at = [&](int i) -> uint64_t { return make_key(row[i], (uint32_t)i); };
  block_select_smallest(nlist, nprobe, npad, key_at, sel_out, &sh);
  for (int r = threadIdx.x; r < nprobe; r += blockDim.x) {
    const uint64_t key = sel_out[r];
    const int c = (int)(uint32_t)key;
    const float s = ord2f((uint32_t)(key >> 32));
    probe_ids[q * nprobe + r] = c;
    probe_G[q * nprobe + r] = s;
    const float d2 = (metric == RABITQ_L2) ? s : (sq_norm[q] + centroid_sq[c] + 2.0f * s);
    probe_E[q * nprobe + r] = sqrtf(fmaxf(d2, 0.f));
  }
}

// The same selection with one wavefront per query and the whole score row in registers
// (nlist <= 64*R): no LDS histogram, no workgroup barriers.
template <int R>
__global__ __launch_bounds__(64) void select_probes_wave_kernel(const float* __restrict__ scores,
                                                               const float* __restrict__ sq_norm,
                                                               const float* __restrict__ centroid_sq, int nlist,
                                                               int nprobe, int npad, int metric,
                                                               int32_t* __restrict__ probe_ids,
                                                               float* __restrict__ probe_G,
                                                               float* __restrict__ probe_E) {
  extern __shared__ uint64_t sel_out[];  // [npad]
  const int lane = threadIdx.x;
  const int64_t q = blockIdx.x;
  const float* row = scores + q * nlist;
  uint32_t ord[R];
  float sv[R];
#pragma unroll
  for (int r = 0; r < R; ++r) sv[r] = row[min(r * 64 + lane, nlist - 1)];  // unconditional: R requests in flight together
#pragma unroll
  for (int r = 0; r < R; ++r) sv[r] = pinned(sv[r]);
#pragma unroll
  for (int r = 0; r < R; ++r) ord[r] = (r * 64 + lane < nlist) ? min(f2ord(sv[r]), 0xfffffffeu) : 0xffffffffu;
  // (32-bit words bisected with ballots; 64-bit keys counted per lane and reduced at every step are slower: 3001
  // queries, 1024 lists, 128 probes: the kernel 19 us against 25.  Where every list is probed there is nothing to bisect:
  // no value short of the largest splits off all words, so the search would go through the whole range: 10 us of 65 for the
  // coarse stage of one query and 1024 lists.)
  uint32_t n_le = (uint32_t)nlist, bound = 0xfffffffeu;
  if (nprobe < nlist) bound = wave_kth_ord<R>(ord, (uint32_t)nprobe, &n_le);
  const int got = wave_put_smallest<R>(ord, bound, n_le, (uint32_t)nprobe, lane, [&](int at, int r) {
    sel_out[at] = ((uint64_t)ord[r] << 32) | (uint32_t)(r * 64 + lane);
  });
  for (int i = got + lane; i < npad; i += 64) sel_out[i] = KEY_NONE;
  block_bitonic_sort(sel_out, npad);
  for (int r = lane; r < nprobe; r += 64) {
    const uint64_t k2 = sel_out[r];
    const int c = (int)(uint32_t)k2;
    const float s = ord2f((uint32_t)(k2 >> 32));
    probe_ids[q * nprobe + r] = c;
    probe_G[q * nprobe + r] = s;
    const float d2 = (metric == RABITQ_L2) ? s : (sq_norm[q] + centroid_sq[c] + 2.0f * s);
    probe_E[q * nprobe + r] = sqrtf(fmaxf(d2, 0.f));
  }
}

// The selection for nprobe <= 64 and any nlist, one wavefront per query: the score row is read
// once through a register-resident sorted list of the best.
__global__ __launch_bounds__(256) void select_probes_stream_kernel(const float* __restrict__ scores,
                                                                  const float* __restrict__ sq_norm,
                                                                  const float* __restrict__ centroid_sq, int64_t nq,
                                                                  int nlist, int nprobe, int metric,
                                                                  int32_t* __restrict__ probe_ids,
                                                                  float* __restrict__ probe_G,
                                                                  float* __restrict__ probe_E) {
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= nq) return;
  const float* row = scores + q * nlist;
  const WaveTopK top = stream_select_smallest(row, nlist, nprobe, lane);
  if (lane < nprobe) {
    const uint64_t key = top.v;
    const int c = (int)(uint32_t)key;
    const float s = ord2f((uint32_t)(key >> 32));
    probe_ids[q * nprobe + lane] = c;
    probe_G[q * nprobe + lane] = s;
    const float d2 = (metric == RABITQ_L2) ? s : (sq_norm[q] + centroid_sq[c] + 2.0f * s);
    probe_E[q * nprobe + lane] = sqrtf(fmaxf(d2, 0.f));
  }
}

// The same from the smallest score of every 32 lists: the nprobe best scores lie in the nprobe tiles of 32 with the smallest
// minima, so only those tiles are read.  Tiles and scores are selected by bisection of values in registers (wave_kth_ord): RT words
// per lane for the minima, RS for the scores of at most 2 RS tiles.  What bounds it is the read of the minima and of nprobe
// scattered 128-byte tiles.  (10^4 queries, 8192 lists, 32 probes: 87 us for the whole rows, 30.5 for this, and 71 when the
// second selection inserted one score after another into a sorted list; 6000 queries, 4096 lists, 8 probes: 42 -> 9.5.  The
// minima cost the GEMM that writes them nothing that shows: 212 us and 169 against 212 and 175.)
template <int RT, int RS>
__global__ __launch_bounds__(256) void select_probes_tiles_kernel(const float* __restrict__ scores, const uint32_t* __restrict__ tmin,
                                                                 const float* __restrict__ sq_norm,
                                                                 const float* __restrict__ centroid_sq, int64_t nq,
                                                                 int nlist, int nprobe, int metric,
                                                                 int32_t* __restrict__ probe_ids,
                                                                 float* __restrict__ probe_G,
                                                                 float* __restrict__ probe_E) {
  __shared__ uint64_t s_sel[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t q = (int64_t)blockIdx.x * 4 + wave;
  if (q >= nq) return;
  uint64_t* sel = s_sel[wave];
  const float* row = scores + q * nlist;
  const int n_t = (nlist + 31) / 32;  // more than nprobe
  uint32_t n_le;
  {
    float v[RT];
    uint32_t ord[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) v[r] = __uint_as_float(tmin[q * n_t + min(r * 64 + lane, n_t - 1)]);
#pragma unroll
    for (int r = 0; r < RT; ++r) v[r] = pinned(v[r]);
#pragma unroll
    for (int r = 0; r < RT; ++r) ord[r] = r * 64 + lane < n_t ? min(__float_as_uint(v[r]), 0xfffffffeu) : 0xffffffffu;
    const uint32_t bound = wave_kth_ord<RT>(ord, (uint32_t)nprobe, &n_le);
    wave_put_smallest<RT>(ord, bound, n_le, (uint32_t)nprobe, lane, [&](int at, int r) { sel[at] = (uint64_t)(r * 64 + lane); });
  }
  wave_sync();
  int at[RS];
  float sc[RS];
  uint32_t ord[RS];
#pragma unroll
  for (int u = 0; u < RS; ++u) {
    const int t = 2 * u + (lane >> 5);
    at[u] = 32 * (int)sel[min(t, nprobe - 1)] + (lane & 31);
    sc[u] = __builtin_nontemporal_load(row + min(at[u], nlist - 1));
    if (t >= nprobe) at[u] = nlist;
  }
#pragma unroll
  for (int u = 0; u < RS; ++u) sc[u] = pinned(sc[u]);
#pragma unroll
  for (int u = 0; u < RS; ++u) ord[u] = at[u] < nlist ? min(f2ord(sc[u]), 0xfffffffeu) : 0xffffffffu;
  wave_sync();
  // (the selected tiles are in ascending order, so equals are taken in the order of their lists)
  const uint32_t bound = wave_kth_ord<RS>(ord, (uint32_t)nprobe, &n_le);
  const int got = wave_put_smallest<RS>(ord, bound, n_le, (uint32_t)nprobe, lane, [&](int place, int r) {
    sel[place] = ((uint64_t)ord[r] << 32) | (uint32_t)at[r];
  });
  wave_sync();
  WaveTopK top;
  top.init_sorted(lane < got ? sel[lane] : KEY_NONE, lane);
  if (lane < nprobe) {
    const uint64_t key = top.v;
    const int c = (int)(uint32_t)key;
    const float s = ord2f((uint32_t)(key >> 32));
    probe_ids[q * nprobe + lane] = c;
    probe_G[q * nprobe + lane] = s;
    const float d2 = (metric == RABITQ_L2) ? s : (sq_norm[q] + centroid_sq[c] + 2.0f * s);
    probe_E[q * nprobe + lane] = sqrtf(fmaxf(d2, 0.f));
  }
}

// From how many lists the minima of 32 pay: at least four times as many tiles as are read, so that at most a quarter of the row
// and of the minima's 1/32 are (1024 lists, 32 probes: 15.5 us for the whole rows, whose tiles would all be read); no more minima
// than 16 words a lane hold.
bool select_by_minima(int nlist, int nprobe) {
  const int n_t = (nlist + 31) / 32;
  return nprobe <= 64 && n_t >= 4 * nprobe && n_t <= 1024;
}

// Which selection kernel a given (nlist, nprobe) takes: 0 = one wavefront per query streaming the score row through
// a register-resident sorted list (nprobe <= 64, any nlist); 1, 2, 3 = one wavefront per query with the whole row
// in registers, 8 / 16 / 32 scores per lane (nprobe > 64, nlist <= 512 / 1024 / 2048); 4 = one workgroup per
// query, radix select in LDS (nprobe > 64, nlist > 2048).
int probe_select_variant(int nlist, int nprobe) {
  if (nprobe <= 64) return 0;
  if (nlist <= 64 * 8) return 1;
  if (nlist <= 64 * 16) return 2;
  if (nlist <= 64 * 32) return 3;
  return 4;
}

int launch_select_probes(const float* scores, const uint32_t* tmin, const float* sq_norm, const float* centroid_sq, int64_t nq, int nlist,
                         int nprobe, int metric, int32_t* probe_ids, float* probe_G, float* probe_E, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  const int npad = next_pow2(nprobe);
  const size_t smem = npad * sizeof(uint64_t);
  switch (probe_select_variant(nlist, nprobe)) {
    case 0:
      if (tmin != nullptr) {
        const bool many = nlist > 32 * 256;
        auto kernel = nprobe <= 8    ? (many ? select_probes_tiles_kernel<16, 4> : select_probes_tiles_kernel<4, 4>)
                      : nprobe <= 32 ? (many ? select_probes_tiles_kernel<16, 16> : select_probes_tiles_kernel<4, 16>)
                                     : (many ? select_probes_tiles_kernel<16, 32> : select_probes_tiles_kernel<4, 32>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, st, scores, tmin, sq_norm, centroid_sq, nq, nlist,
                           nprobe, metric, probe_ids, probe_G, probe_E);
        break;
      }
      hipLaunchKernelGGL(select_probes_stream_kernel, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, st, scores, sq_norm,
                         centroid_sq, nq, nlist, nprobe, metric, probe_ids, probe_G, probe_E);
      break;
    case 1:
      hipLaunchKernelGGL(select_probes_wave_kernel<8>, dim3((unsigned)nq), dim3(64), smem, st, scores, sq_norm,
                         centroid_sq, nlist, nprobe, npad, metric, probe_ids, probe_G, probe_E);
      break;
    case 2:
      hipLaunchKernelGGL(select_probes_wave_kernel<16>, dim3((unsigned)nq), dim3(64), smem, st, scores, sq_norm,
                         centroid_sq, nlist, nprobe, npad, metric, probe_ids, probe_G, probe_E);
      break;
    case 3:
      hipLaunchKernelGGL(select_probes_wave_kernel<32>, dim3((unsigned)nq), dim3(64), smem, st, scores, sq_norm,
                         centroid_sq, nlist, nprobe, npad, metric, probe_ids, probe_G, probe_E);
      break;
    default:
      hipLaunchKernelGGL(select_probes_kernel, dim3((unsigned)nq), dim3(256), smem, st, scores, sq_norm, centroid_sq,
                         nlist, nprobe, npad, metric, probe_ids, probe_G, probe_E);
  }
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

// ---------------------------------------------------------------------------------
// Section 3.3.3: regroup (query, cluster) pairs by cluster, stable in query id.
// A query probes a cluster at most once, so membership is one bit per (cluster, query):
//   1. clear and set the bitmap  M[c][q]
//   2. per cluster: running popcount of its bitmap row -> rank of every 32-query word
//   3. exclusive scan of the cluster totals -> pair_off
//   4. every pair computes its own destination: pair_off[c] + rank of q in row c
// All integer, no order-dependent atomics: the output is unique.
// scratch: bitmap [nlist][QWORDS] | word_rank [nlist][QWORDS] | total [nlist]
// ---------------------------------------------------------------------------------
__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void bitmap_set_kernel(const int32_t* __restrict__ probe_ids, int64_t npairs, int nprobe, int qwords,
                                  uint32_t* __restrict__ bitmap) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npairs; p += (int64_t)gridDim.x * blockDim.x) {
    const int c = probe_ids[p];
    const int64_t q = p / nprobe;
    atomicOr(&bitmap[(int64_t)c * qwords + (q >> 5)], 1u << (q & 31));
  }
}

__global__ __launch_bounds__(64) void row_rank_kernel(const uint32_t* __restrict__ bitmap, int qwords,
                                                      uint32_t* __restrict__ word_rank,
                                                      uint32_t* __restrict__ total) {
  const int c = blockIdx.x, lane = threadIdx.x;
  const uint32_t* row = bitmap + (int64_t)c * qwords;
  uint32_t* out = word_rank + (int64_t)c * qwords;
  uint32_t carry = 0;
  for (int base = 0; base < qwords; base += 64) {
    const int w = base + lane;
    const uint32_t pc = (w < qwords) ? __popc(row[w]) : 0u;
    uint32_t incl = pc;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(incl, d, 64);
      if (lane >= d) incl += o;
    }
    if (w < qwords) out[w] = carry + incl - pc;
    carry += __shfl(incl, 63, 64);
  }
  if (lane == 0) total[c] = carry;
}

// out[0] = 0, out[i+1] = sum_{j<=i} in[j].  One workgroup, bound by its latencies: 8 entries per thread whose loads
// are in flight together (one entry after the other, 32 per thread, took 27 us for 8192 lists).
template <int NT>
__global__ __launch_bounds__(NT) void exclusive_scan_kernel(const uint32_t* __restrict__ in, int n,
                                                                     int32_t* __restrict__ out) {
  __shared__ uint32_t s_wave[1][NT / 64];
  uint32_t carry[1] = {0};
  for (int base = 0; base < n; base += NT * SCAN_PER) {
    const int s = base + (int)threadIdx.x * SCAN_PER;
    uint32_t x[SCAN_PER], sum[1] = {0}, run[1];
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) x[e] = in[min(s + e, n - 1)];
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
      if (s + e >= n) x[e] = 0;
      sum[0] += x[e];
    }
    block_chunk_scan<NT, 1>(sum, run, carry, s_wave);
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
      if (s + e < n) out[s + e] = (int32_t)run[0];
      run[0] += x[e];
    }
  }
  if (threadIdx.x == 0) out[n] = (int32_t)carry[0];
}

__global__ void scatter_pairs_kernel(const int32_t* __restrict__ probe_ids, int64_t npairs, int nprobe, int qwords,
                                     const uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ word_rank,
                                     const int32_t* __restrict__ pair_off, int32_t* __restrict__ pair_ids) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npairs; p += (int64_t)gridDim.x * blockDim.x) {
    const int c = probe_ids[p];
    const int64_t q = p / nprobe;
    const int64_t wi = (int64_t)c * qwords + (q >> 5);
    const uint32_t below = bitmap[wi] & ((1u << (q & 31)) - 1u);
    pair_ids[pair_off[c] + word_rank[wi] + __popc(below)] = (int32_t)p;
  }
}

int64_t probe_list_scratch_words(int32_t nlist, int64_t nq) {
  const int64_t qwords = (nq + 31) / 32;
  return 2 * (int64_t)nlist * qwords + nlist;
}

// step 1 on its own: it needs no probes, so a search can clear the bitmap while the probes are still being computed
int launch_clear_list_bitmap(int64_t nq, int nlist, uint32_t* scratch, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  const int64_t bm_words = (int64_t)nlist * ((nq + 31) / 32);
  const unsigned g1 = (unsigned)std::min<int64_t>((bm_words + 255) / 256, 4096);
  hipLaunchKernelGGL(fill_u32_kernel, dim3(g1), dim3(256), 0, st, scratch, bm_words, 0u);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

int launch_build_lists(const int32_t* probe_ids, int64_t nq, int nprobe, int nlist, int32_t* pair_off,
                       int32_t* pair_ids, uint32_t* scratch, hipStream_t st, bool bitmap_is_clear) {
  if (nq <= 0) return RABITQ_OK;
  const int qwords = (int)((nq + 31) / 32);
  const int64_t npairs = nq * nprobe;
  uint32_t* bitmap = scratch;
  uint32_t* word_rank = scratch + (int64_t)nlist * qwords;
  uint32_t* total = word_rank + (int64_t)nlist * qwords;
  if (!bitmap_is_clear) {
    if (int rc = launch_clear_list_bitmap(nq, nlist, scratch, st)) return rc;
  }
  const unsigned g2 = (unsigned)std::min<int64_t>((npairs + 255) / 256, 8192);
  hipLaunchKernelGGL(bitmap_set_kernel, dim3(g2), dim3(256), 0, st, probe_ids, npairs, nprobe, qwords, bitmap);
  hipLaunchKernelGGL(row_rank_kernel, dim3(nlist), dim3(64), 0, st, bitmap, qwords, word_rank, total);
  if (nlist <= SCAN_SMALL * SCAN_PER)
    hipLaunchKernelGGL(exclusive_scan_kernel<SCAN_SMALL>, dim3(1), dim3(SCAN_SMALL), 0, st, total, nlist, pair_off);
  else
    hipLaunchKernelGGL(exclusive_scan_kernel<SCAN_LARGE>, dim3(1), dim3(SCAN_LARGE), 0, st, total, nlist, pair_off);
  hipLaunchKernelGGL(scatter_pairs_kernel, dim3(g2), dim3(256), 0, st, probe_ids, npairs, nprobe, qwords, bitmap,
                     word_rank, pair_off, pair_ids);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

// ---------------------------------------------------------------------------------
// Section 3.3.5: merge the nprobe cluster-local lists of one query into its top-k, any k.
// The lists are short and ragged: 64 of them at a time are laid end to end (a scan of their lengths), so that every
// lane fetches a key that exists, four at a time.  Keys that can still be among the k best go to a buffer in LDS,
// which is cut to its k best by bisection when it is full; the k that are left are sorted.  (10^4 queries, 32 lists, k = 100:
// 27 us, a workgroup per query with a radix select 87; 3001 queries, 128 lists, k = 50: 21 us, one serial insertion per
// key into a sorted register list 43.)
// SHARED: the four wavefronts of a workgroup take every fourth step of one query, each with its own buffer, and the first
// one selects from what they kept; otherwise each has a query of its own.
// ---------------------------------------------------------------------------------
constexpr int MERGE_BUF = 512;
static_assert(RABITQ_MAX_K <= 128 && RABITQ_MAX_K + TILE <= MERGE_BUF, "k keys and a step of 64 fit the buffer; k are sorted in 128 places");

template <bool SHARED>
__global__ __launch_bounds__(256) void merge_kernel(const uint64_t* __restrict__ cand_keys,
                                                   const int32_t* __restrict__ cand_cnt, int64_t nq, int k, int cap,
                                                   int nprobe, int metric, int64_t* __restrict__ out_ids,
                                                   float* __restrict__ out_dists) {
  __shared__ uint64_t s_buf[4][MERGE_BUF];
  __shared__ int s_off[4][64];
  __shared__ int s_cnt[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t q = SHARED ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + wave;
  if (q >= nq) return;
  uint64_t* buf = s_buf[wave];
  int* off = s_off[wave];
  const uint64_t* keys = cand_keys + q * nprobe * (int64_t)cap;
  const int32_t* counts = cand_cnt + q * nprobe;
  const uint64_t lower = (1ull << lane) - 1ull;
  int cnt = 0;
  uint64_t limit = KEY_NONE;  // only keys below this can be among the k best
  constexpr int RB = MERGE_BUF / 64;
  // Leaves the k best of more than k keys in the buffer.  Keys may repeat (a caller of the stage may hand in what it likes):
  // of several at the last place only as many stay as there is room for, and another copy of them is no better, so
  // the limit excludes it.
  auto keep_best = [&](const uint64_t (&key)[RB]) {
    wave_sync();
    const uint64_t next = wave_keep_best<RB>(key, k, lane, &cnt, [&](int at, uint64_t v) { buf[at] = v; }) + 1ull;
    limit = next < limit ? next : limit;
    wave_sync();
  };
  auto cut = [&]() {
    uint64_t key[RB];
    wave_sync();
#pragma unroll
    for (int r = 0; r < RB; ++r) key[r] = r * 64 + lane < cnt ? buf[r * 64 + lane] : KEY_NONE;
    keep_best(key);
  };
  for (int jb = 0; jb < nprobe; jb += 64) {
    const int n = jb + lane < nprobe ? min(counts[jb + lane], cap) : 0;
    int incl = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int o = __shfl_up(incl, d, 64);
      if (lane >= d) incl += o;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    wave_sync();
    off[lane] = incl - n;  // first place of list jb + lane
    wave_sync();
    for (int i0 = SHARED ? wave * 256 : 0; i0 < total; i0 += SHARED ? 1024 : 256) {
      uint64_t kk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = min(i0 + u * 64 + lane, total - 1);
        int j = 0;  // the last list that starts at or before place i (lists of length 0 start where the next one does)
#pragma unroll
        for (int d = 32; d > 0; d >>= 1)
          if (off[j + d] <= i) j += d;
        kk[u] = keys[(int64_t)(jb + j) * cap + (i - off[j])];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) kk[u] = pinned(kk[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i0 + u * 64 >= total) break;
        if (i0 + u * 64 + lane >= total) kk[u] = KEY_NONE;
        uint64_t m = __ballot(kk[u] < limit);
        if (m == 0ull) continue;
        if (cnt + __popcll(m) > MERGE_BUF) {
          cut();  // (k keys are left: a step of 64 always fits)
          m = __ballot(kk[u] < limit);
        }
        if (kk[u] < limit) buf[cnt + __popcll(m & lower)] = kk[u];
        cnt += __popcll(m);
      }
    }
  }
  if (!SHARED) {
    if (cnt > k) cut();
  } else {
    // the first wavefront takes the k best of the four buffers, which fit its registers as they are or cut to k each
    if (lane == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3] > MERGE_BUF) {  // (the same for all four)
      if (cnt > k) cut();
      __syncthreads();
      if (lane == 0) s_cnt[wave] = cnt;
      __syncthreads();
    }
    if (wave > 0) return;
    const int e0 = s_cnt[0], e1 = e0 + s_cnt[1], e2 = e1 + s_cnt[2], e3 = e2 + s_cnt[3];
    uint64_t key[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int i = r * 64 + lane;
      const int w = i < e0 ? 0 : (i < e1 ? 1 : (i < e2 ? 2 : 3));
      const int first = w == 0 ? 0 : (w == 1 ? e0 : (w == 2 ? e1 : e2));
      key[r] = i < e3 ? s_buf[w][i - first] : KEY_NONE;
    }
    if (e3 > k) {
      keep_best(key);
    } else {  // k <= 128 of them at most
      wave_sync();
#pragma unroll
      for (int r = 0; r < 2; ++r)
        if (r * 64 + lane < e3) buf[r * 64 + lane] = key[r];
      cnt = e3;
    }
  }
  wave_sync();
  auto put = [&](int r, uint64_t key) {
    int64_t id = -1;
    float d = (metric == RABITQ_L2) ? INFINITY : -INFINITY;
    if (key != KEY_NONE) {
      id = (int64_t)(int32_t)(uint32_t)key;
      d = ord2f((uint32_t)(key >> 32));
      if (metric == RABITQ_IP) d = -d;
    }
    out_ids[q * k + r] = id;
    out_dists[q * k + r] = d;
  };
  if (k <= 64) {
    WaveTopK top;
    top.init_sorted(lane < cnt ? buf[lane] : KEY_NONE, lane);
    if (lane < k) put(lane, top.v);
  } else {
    for (int i = cnt + lane; i < 128; i += 64) buf[i] = KEY_NONE;
    wave_sync();
    wave_bitonic_sort(buf, 128, lane);
    for (int r = lane; r < k; r += 64) put(r, buf[r]);
  }
}

// The same merge for k <= 64 and few lists (or k < 4), one wavefront per query: the candidate lists stream through
// a register-resident sorted list, G lanes per list, four entries per lane in flight.
__global__ __launch_bounds__(256) void merge_wave_kernel(const uint64_t* __restrict__ cand_keys,
                                                        const int32_t* __restrict__ cand_cnt, int64_t nq, int k,
                                                        int cap, int nprobe, int metric,
                                                        int64_t* __restrict__ out_ids, float* __restrict__ out_dists) {
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= nq) return;
  const uint64_t* keys = cand_keys + q * nprobe * (int64_t)cap;
  const int32_t* cnt = cand_cnt + q * nprobe;
  int G = 1;  // lanes per list: the largest power of two with G * nprobe <= 64
  while (2 * G * nprobe <= 64) G <<= 1;
  const int ppc = 64 / G, g = lane % G;
  WaveTopK top;
  top.v = KEY_NONE;
  bool first = true;
  for (int jb = 0; jb < nprobe; jb += ppc) {
    const int j = jb + lane / G;
    const int n = (j < nprobe) ? min(cnt[j], cap) : 0;
    const int nmax = (int)wave_reduce_u32((uint32_t)n, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
    const uint64_t* row = keys + (int64_t)min(j, nprobe - 1) * cap;
    for (int e0 = 0; e0 < nmax; e0 += 4 * G) {
      uint64_t kk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + u * G + g;
        kk[u] = (e < n) ? row[e] : KEY_NONE;  // (lists differ in length: reading past a short one would only add traffic)
      }
      if (first) {
        // the lanes' smallest keys start the sorted list; the other keys are then offered to it
        uint64_t mn = kk[0];
        int mu = 0;
#pragma unroll
        for (int u = 1; u < 4; ++u)
          if (kk[u] < mn) { mn = kk[u]; mu = u; }
        top.init_sorted(mn, lane);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (e0 + u * G < nmax) top.push_tile(u == mu ? KEY_NONE : kk[u], k, lane);
        first = false;
        continue;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (e0 + u * G < nmax) top.push_tile(kk[u], k, lane);
      }
    }
  }
  if (lane < k) {
    const uint64_t key = top.v;
    int64_t id = -1;
    float d = (metric == RABITQ_L2) ? INFINITY : -INFINITY;
    if (key != KEY_NONE) {
      id = (int64_t)(int32_t)(uint32_t)key;
      d = ord2f((uint32_t)(key >> 32));
      if (metric == RABITQ_IP) d = -d;
    }
    out_ids[q * k + lane] = id;
    out_dists[q * k + lane] = d;
  }
}

int launch_merge(const uint64_t* cand_keys, const int32_t* cand_cnt, int64_t nq, int k, int nprobe, int metric,
                 int64_t* out_ids, float* out_dists, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  const int cap = next_pow2(k + TILE);
  // Few lists and k <= 64, or the very smallest k: the first keys of all lists fill the sorted register list at once and few
  // of the others have to be inserted (16 lists, k = 10, 10^4 queries: 13.0 us against 18.0; one query 5.4 against 6.3;
  // k = 1, 512 lists, one query 5.4 against 7.8).  From 64 lists on, or for k > 64, the buffer and its bisection win (64
  // lists, k = 10, 2500 queries: 13.6 against 15.5 us; k = 4, 256 queries: 7.5 against 11.0; figures above).
  // Where there are too few queries to fill the chip, a query is shared by four wavefronts (one query, k = 128, 16 lists:
  // 15.4 us against 17.6 with one; 64 queries, k = 100, 128 lists: 19.0 against 28.9; unpruned lists, one query, k = 35, 512
  // lists: 51 against 145).  1024 queries, k = 65, 16 lists: 18.5 against 24.1, but 2048: 21.6 against 15.9; with k <= 64 the
  // two meet at 512 (64 lists, k = 35: 14.2 against 14.7, 1024: 15.8 against 15.0), and a k below 8 leaves too few
  // keys to share (64 lists, k = 4, 8 queries: 7.5 against 6.9).
  if (k <= 64 && (nprobe < 64 || k < 4))
    hipLaunchKernelGGL(merge_wave_kernel, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, st, cand_keys, cand_cnt, nq, k,
                       cap, nprobe, metric, out_ids, out_dists);
  else if (k >= 8 && nq <= (k <= 64 ? 512 : 1024))
    hipLaunchKernelGGL(merge_kernel<true>, dim3((unsigned)nq), dim3(256), 0, st, cand_keys, cand_cnt, nq, k, cap, nprobe,
                       metric, out_ids, out_dists);
  else
    hipLaunchKernelGGL(merge_kernel<false>, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, st, cand_keys, cand_cnt, nq, k,
                       cap, nprobe, metric, out_ids, out_dists);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

__global__ void fill_f32_kernel(float* p, int64_t n, float v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

int launch_fill_f32(float* p, int64_t n, float v, hipStream_t st) {
  if (n <= 0) return RABITQ_OK;
  const unsigned g = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(g), dim3(256), 0, st, p, n, v);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

}  // namespace rq
