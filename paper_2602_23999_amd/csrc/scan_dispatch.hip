// Host-side launchers of the seeding and scan kernels: argument block, work-item
// offsets, and routing to the translation unit that holds the kernels for W = dim/32.
#include <algorithm>
#include <functional>

#include "rq_device.h"
#include "rq_scan_args.h"
#include "rq_small_batch.h"

namespace rq {

// ---------------------------------------------------------------------------------
// item_off[c] = first work item of cluster c; a work item is qw consecutive pairs of
// one cluster times one segment of its tiles.  (One workgroup.)
// ---------------------------------------------------------------------------------
__global__ void zero_i32_kernel(int32_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

// SPLIT (split search): also item16[c] = first work item of cluster c when an item is 16 pairs times one segment, and
// mask_off[c] = first block of survivor bits of cluster c (a block per group of 16 pairs and tile); not written otherwise.
// ORDERED: entry i is about cluster order[i].  One workgroup whose time is its load latencies: a thread's 8 entries are
// fetched together (8192 lists, split: 69 us when 256 threads walked 32 entries each; see SCAN_PER).
template <int NT, bool SPLIT, bool ORDERED>
__global__ __launch_bounds__(NT) void item_offsets_kernel(const int32_t* __restrict__ pair_off,
                                                                   const int32_t* __restrict__ tile_off,
                                                                   const int32_t* __restrict__ order, int n, int qw,
                                                                   int tseg, int segmax, int32_t* __restrict__ item_off,
                                                                   int32_t* __restrict__ item16,
                                                                   uint32_t* __restrict__ mask_off) {
  constexpr int NV = SPLIT ? 3 : 1;
  __shared__ uint32_t s_wave[NV][NT / 64];
  uint32_t carry[NV] = {0};
  for (int base = 0; base < n; base += NT * SCAN_PER) {
    const int s = base + (int)threadIdx.x * SCAN_PER;
    // (entry i is about cluster i, or about the i-th longest cluster when an order is given; entries past the last
    // are fetched as the last and count nothing)
    uint32_t val[SCAN_PER][NV], sum[NV] = {0}, run[NV];
    int po[SCAN_PER], pe[SCAN_PER], to[SCAN_PER], te[SCAN_PER];
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
      const int r = min(s + e, n - 1), c = ORDERED ? order[r] : r;
      po[e] = pair_off[c]; pe[e] = pair_off[c + 1];
      to[e] = tile_off[c]; te[e] = tile_off[c + 1];
    }
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
      const bool in = s + e < n;
      const uint32_t pairs = in ? (uint32_t)(pe[e] - po[e]) : 0u, tiles = (uint32_t)(te[e] - to[e]);
      const uint32_t nseg = (uint32_t)seg_count((int)tiles, tseg, segmax);
      val[e][0] = (qw == 1 ? pairs : (pairs + qw - 1) / (uint32_t)qw) * nseg;
      if (SPLIT) {
        const uint32_t groups = (pairs + QM - 1) / QM;
        val[e][NV - 2] = groups * nseg;
        val[e][NV - 1] = groups * tiles;
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) sum[v] += val[e][v];
    }
    block_chunk_scan<NT, NV>(sum, run, carry, s_wave);
#pragma unroll
    for (int e = 0; e < SCAN_PER; ++e) {
      if (s + e < n) {
        item_off[s + e] = (int32_t)run[0];
        if (SPLIT) {
          item16[s + e] = (int32_t)run[NV - 2];
          mask_off[s + e] = run[NV - 1];
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) run[v] += val[e][v];
    }
  }
  if (threadIdx.x == 0) {
    item_off[n] = (int32_t)carry[0];
    if (SPLIT) {
      item16[n] = (int32_t)carry[NV - 2];
      mask_off[n] = carry[NV - 1];
    }
  }
}

// One wavefront per cluster writes the descriptors of its work items of qw pairs: 4 of the split search (with their first block
// of survivor bits), 16 of the group scan (mask_off == nullptr).
__global__ __launch_bounds__(64) void item_desc_kernel(const int32_t* __restrict__ pair_off, const int32_t* __restrict__ tile_off,
                                                      const int32_t* __restrict__ item_off, const uint32_t* __restrict__ mask_off,
                                                      const int32_t* __restrict__ order, int qw, int tseg, int segmax, ItemDesc* __restrict__ desc) {
  const int i0 = item_off[blockIdx.x], n = item_off[blockIdx.x + 1] - i0;
  if (n <= 0) return;
  const int c = order != nullptr ? order[blockIdx.x] : (int)blockIdx.x;
  const int t0 = tile_off[c], tiles = tile_off[c + 1] - t0;
  const int p0 = pair_off[c], cnt = pair_off[c + 1] - p0;
  const int nseg = seg_count(tiles, tseg, segmax);
  const int seglen = (tiles + nseg - 1) / nseg;
  const uint32_t m0 = mask_off != nullptr ? mask_off[c] : 0u;
  for (int it = threadIdx.x; it < n; it += 64) {
    const int grp = it / nseg, sidx = it - grp * nseg;
    ItemDesc d;
    d.pbeg = p0 + grp * qw;
    d.np_mg = min(qw, cnt - grp * qw) | ((grp & 3) << 8);
    d.t0 = t0;
    d.ts = t0 + sidx * seglen;
    d.te = min(t0 + tiles, d.ts + seglen);
    d.nseg = nseg;
    d.mblock = m0 + (uint32_t)((grp >> 2) * tiles + sidx * seglen);
    d.pad = 0;
    desc[i0 + it] = d;
  }
}

// One wavefront per entry r of the item table (cluster order[r], or cluster r without an order) writes the descriptors
// of its work items of one pair (prefetching variant of the popcount kernel).
__global__ __launch_bounds__(64) void stream_desc_kernel(ScanArgs a, StreamDesc* __restrict__ desc) {
  const int r = blockIdx.x;
  const int i0 = a.item_off[r], n = a.item_off[r + 1] - i0;
  if (n <= 0) return;
  const int c = a.order ? a.order[r] : r;
  const int t0 = a.tile_off[c], tiles = a.tile_off[c + 1] - t0;
  const int p0 = a.pair_off[c];
  const int nseg = seg_count(tiles, a.tseg, a.segmax);
  const int seglen = (tiles + nseg - 1) / nseg;
  for (int it = threadIdx.x; it < n; it += 64) {
    const int pi = it / nseg, sidx = it - pi * nseg;
    const int pp = a.pair_ids[p0 + pi];
    const int q = pair_query(a, pp);
    StreamDesc d{};
    d.pp = pp;
    d.q = q;
    d.t0 = t0;
    d.ts = t0 + sidx * seglen;
    d.te = min(t0 + tiles, d.ts + seglen);
    d.nseg = nseg;
    d.ppos = p0 + pi;
    d.S = a.sum_qhat[q];
    d.G = a.probe_G[pp];
    d.E = a.probe_E[pp];
    d.delta = a.delta[q];
    d.sumq = a.sum_q[q];
    desc[i0 + it] = d;
  }
}

// segments per cluster, sorted, for the work-item bound of a launch (cached per segment length and limit)
static void update_seg_cache(const rabitq_index* ix, int tseg, int segmax) {
  std::vector<int>& nseg = ix->seg_sorted;
  if (ix->seg_sorted_max == segmax && ix->seg_sorted_tseg == tseg) return;
  nseg.resize(ix->host_tiles.size());
  for (size_t c = 0; c < nseg.size(); ++c) nseg[c] = seg_count(ix->host_tiles[c], tseg, segmax);
  std::sort(nseg.begin(), nseg.end(), std::greater<int>());
  ix->seg_sorted_max = segmax;
  ix->seg_sorted_tseg = tseg;
  ix->seg_total = 0;
  for (int v : nseg) ix->seg_total += v;
}

// Work-item bound.  Cluster c with cnt_c pairs and nseg_c segments has ceil(cnt_c / per_item) * nseg_c work items, at
// most (cnt_c / per_item + 1) * nseg_c.  Every query probes nprobe distinct clusters, so cnt_c <= nq and sum cnt_c =
// nq * nprobe: the sum is largest when the nprobe clusters with the most segments are probed by every query.
static int64_t item_bound(const rabitq_index* ix, int64_t nq, int nprobe, int per_item) {
  const std::vector<int>& nseg = ix->seg_sorted;
  int64_t top = 0;
  for (int i = 0; i < nprobe && i < (int)nseg.size(); ++i) top += nseg[i];
  const int64_t m = ix->seg_total + (nq * top + per_item - 1) / per_item;
  return ((m + 7) / 8) * 8;
}

int64_t split_mask_blocks(rabitq_index* ix, int64_t nq, int nprobe) {
  if (ix->tiles_prefix.empty()) {
    std::vector<int> t(ix->host_tiles.begin(), ix->host_tiles.end());
    std::sort(t.begin(), t.end(), std::greater<int>());
    ix->tiles_prefix.assign(t.size() + 1, 0);
    for (size_t i = 0; i < t.size(); ++i) ix->tiles_prefix[i + 1] = ix->tiles_prefix[i] + t[i];
  }
  const size_t top = std::min<size_t>((size_t)nprobe, ix->tiles_prefix.size() - 1);
  return (nq * ix->tiles_prefix[top] + QM - 1) / QM + ix->n_tiles;
}

// few pairs per list, popcount kernel, neither split nor by groups: the shape the prefetching variant is for
static bool stream_shape(const rabitq_index* ix, int64_t nq, int nprobe, int k) {
  return effective_impl(ix) == 0 && nq * nprobe <= 4 * (int64_t)ix->nlist && !split_wanted(ix, nq, nprobe) &&
         !group_wanted(ix, nq, nprobe, k);
}
static ScanPlan plan_for(const rabitq_index* ix, int64_t nq, int nprobe, int k, bool streaming, bool group = false);
static ScanPlan group_plan(const rabitq_index* ix, int64_t nq, int nprobe, int k) { return plan_for(ix, nq, nprobe, k, false, true); }
// descriptor slots (of sizeof(ItemDesc)) the prefetching variant needs for (nq, nprobe, k)
// work items of one pair: a pair has as many as its list has segments, at most those of the longest list
static int64_t stream_item_bound(const rabitq_index* ix, int64_t nq, int nprobe, const ScanPlan& plan) {
  const int64_t m = nq * nprobe * seg_count(ix->max_tiles, plan.tseg, plan.segmax);
  return ((m + 7) / 8) * 8;
}
static int64_t stream_desc_slots(const rabitq_index* ix, int64_t nq, int nprobe, int k) {
  return stream_item_bound(ix, nq, nprobe, plan_for(ix, nq, nprobe, k, true)) *
         (int64_t)(sizeof(StreamDesc) / sizeof(ItemDesc));
}

int ensure_stream_buffers(rabitq_index* ix, int64_t nq, int nprobe, int k) {
  if (!stream_shape(ix, nq, nprobe, k)) return RABITQ_OK;
  const int64_t slots = stream_desc_slots(ix, nq, nprobe, k);
  if (slots <= ix->item_desc_cap || slots > 0x7fffffff) return RABITQ_OK;
  RQ_HIP(hipDeviceSynchronize());
  if (ix->item_desc) (void)hipFree(ix->item_desc);
  ix->item_desc = nullptr;
  ix->item_desc_cap = 0;
  RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->item_desc), (size_t)slots * sizeof(ItemDesc)));
  ix->item_desc_cap = slots;
  return RABITQ_OK;
}

ScanRoute scan_route(rabitq_index* ix, int64_t nq, int nprobe, int k) {
  if (ix->item_desc == nullptr) return ROUTE_SINGLE;
  if (group_wanted(ix, nq, nprobe, k)) {
    const ScanPlan plan = group_plan(ix, nq, nprobe, k);
    update_seg_cache(ix, plan.tseg, plan.segmax);
    if (item_bound(ix, nq, nprobe, plan.qw) <= ix->item_desc_cap) return ROUTE_GROUP;
  } else if (split_wanted(ix, nq, nprobe) && ix->surv_mask != nullptr) {
    const ScanPlan plan = plan_for(ix, nq, nprobe, k, false);
    update_seg_cache(ix, plan.tseg, plan.segmax);
    if (split_mask_blocks(ix, nq, nprobe) <= ix->surv_mask_blocks && item_bound(ix, nq, nprobe, plan.qw) <= ix->item_desc_cap)
      return ROUTE_SPLIT;
  }
  return ROUTE_SINGLE;
}

int ensure_split_buffers(rabitq_index* ix, int64_t nq, int nprobe, int k) {
  const bool group = group_wanted(ix, nq, nprobe, k);  // (keeps its survivors to itself)
  if (!group && !split_wanted(ix, nq, nprobe)) return RABITQ_OK;
  int64_t need = group ? 0 : split_mask_blocks(ix, nq, nprobe);
  const ScanPlan plan = plan_for(ix, nq, nprobe, k, false, group);
  update_seg_cache(ix, plan.tseg, plan.segmax);
  int64_t items = item_bound(ix, nq, nprobe, plan.qw);
  if (need <= ix->surv_mask_blocks && items <= ix->item_desc_cap) return RABITQ_OK;
  if (need >= ((int64_t)1 << 32) || items > 0x7fffffff) return RABITQ_OK;  // beyond 32-bit offsets: the search is not split
  RQ_HIP(hipDeviceSynchronize());
  if (need > ix->surv_mask_blocks) {
    if (ix->surv_mask) (void)hipFree(ix->surv_mask);
    ix->surv_mask = nullptr;
    ix->surv_mask_blocks = 0;
    RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->surv_mask), (size_t)need * 16 * sizeof(uint64_t)));
    ix->surv_mask_blocks = need;
  }
  if (items > ix->item_desc_cap) {
    if (ix->item_desc) (void)hipFree(ix->item_desc);
    ix->item_desc = nullptr;
    ix->item_desc_cap = 0;
    RQ_HIP(hipMalloc(reinterpret_cast<void**>(&ix->item_desc), (size_t)items * sizeof(ItemDesc)));
    ix->item_desc_cap = items;
  }
  return RABITQ_OK;
}

__global__ __launch_bounds__(1024) void small_batch_lists_kernel(SmallListArgs b) {
  __shared__ uint32_t s_pairs[1024], s_items[1024];
  small_lists_body<1024>(b, s_pairs, s_items);
}

static int field_bits(int B) {  // long-code field width: B rounded up to 2, 4, 8 (0: no long code)
  if (B <= 1) return 0;
  if (B <= 2) return 2;
  if (B <= 4) return 4;
  return 8;
}

static int next_pow2_host(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

static ScanArgs base_args(const rabitq_index* ix) {
  ScanArgs a{};
  a.short_codes = ix->short_codes;
  a.short_factors = ix->short_factors;
  a.long_codes = ix->long_codes;
  a.long_factors = ix->long_factors;
  a.ids = ix->ids;
  a.tile_off = ix->tile_off;
  a.cluster_size = ix->cluster_size;
  a.D = ix->dim;
  a.B = ix->total_bits;
  a.LW = ix->LW;
  a.nlist = ix->nlist;
  a.flip = ix->total_bits == 8 ? 0x80808080u : 0u;
  a.cB = (float)(((1 << ix->total_bits) - 1) * 0.5 - (a.flip ? 128.0 : 0.0));
  a.qerr = effective_impl(ix) == 2 ? 0.f : (float)((ix->dim - 1.0) / (12.0 * (1.0 - 2.0 / 3.14159265358979323846)));
  return a;
}

static int bad_width() {
  set_error("dim/32 must be one of 1,2,3,4,8,16,24,30,32 in this build");
  return RABITQ_EINVAL;
}

static void set_repr(ScanArgs& a, const rabitq_index* ix, const rabitq_query_repr& r, int form) {
  const bool digits = (form & QUERY_DIGITS) != 0;
  a.qhat_fp8 = (form & QUERY_FP8) != 0;
  a.q_stage = digits ? nullptr : r.q_stage;
  a.q_digits = digits ? reinterpret_cast<const uint32_t*>(r.q_stage) : nullptr;
  a.qhat8 = r.qhat8; a.Dp = qhat_stride(ix->dim);
  a.planes = r.planes; a.delta = r.delta; a.sum_qhat = r.sum_qhat; a.sum_q = r.sum_q; a.lut = r.lut;
}

// Queries as a stage entry point hands them in -> as the scans read them (QueryForm): digits, four positions of the refinement order
// per thread, and the group scan's operand.
__global__ __launch_bounds__(256) void digits_kernel(const float* __restrict__ q_stage, const float* __restrict__ delta, int64_t n, int NQ,
                                                    uint32_t* __restrict__ digits) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t q = i / NQ;
  const uint4 d = digit_quad(four_floats(q_stage + 4 * i), digit_factor(delta[q]));
  uint32_t* out = digits + 4 * NQ * q + (i - q * NQ);
  out[0] = d.x; out[NQ] = d.y; out[2 * NQ] = d.z; out[3 * NQ] = d.w;
}
__global__ __launch_bounds__(256) void fp8_operand_kernel(const int8_t* __restrict__ qhat8, int64_t n, int Dp, int8_t* __restrict__ fp8) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t row = i / Dp * Dp;
  const int d = (int)(i - row);
  fp8[row + qhat_fp8_pos(d)] = (int8_t)qhat_fp8(qhat8[row + qhat_mfma_pos(d)], d & 3);
}

// Scans that read the digits with every candidate (the matrix-core kernel, the group scan of wide codes) would make them from q' again
// each time, and the group scan the 16 operands of an item, which is long for wide codes: a stage entry point makes them first,
// in memory that the handle keeps.  (960-d, 5 bits, 1000 queries x 16 lists: 1250 us by groups, 911 with the digits ready and
// 412 with both; the matrix-core kernel 737 and 468.)  Where the memory cannot be had, as while the stream is captured, the scans take
// what was handed in.
static void convert_stage_queries(rabitq_index* ix, const rabitq_query_repr& r, int64_t nq, bool operand, ScanArgs& a, hipStream_t st) {
  const int64_t digits = nq * ix->dim, bytes = operand ? nq * a.Dp : 0, words = digits + bytes / 4;
  if (words > ix->stage_queries_cap) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone || hipDeviceSynchronize() != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    if (ix->stage_queries) (void)hipFree(ix->stage_queries);
    ix->stage_queries = nullptr;
    ix->stage_queries_cap = 0;
    if (hipMalloc(reinterpret_cast<void**>(&ix->stage_queries), (size_t)words * sizeof(uint32_t)) != hipSuccess) {
      (void)hipGetLastError();
      ix->stage_queries = nullptr;
      return;
    }
    ix->stage_queries_cap = words;
  }
  hipLaunchKernelGGL(digits_kernel, dim3((unsigned)((digits / 4 + 255) / 256)), dim3(256), 0, st, r.q_stage, r.delta, digits / 4,
                     ix->dim / 4, ix->stage_queries);
  a.q_digits = ix->stage_queries;
  if (operand) {
    int8_t* fp8 = reinterpret_cast<int8_t*>(ix->stage_queries + digits);
    hipLaunchKernelGGL(fp8_operand_kernel, dim3((unsigned)((bytes + 255) / 256)), dim3(256), 0, st, r.qhat8, bytes, a.Dp, fp8);
    a.qhat8 = fp8;
    a.qhat_fp8 = true;
  }
}

static int need_lut(const rabitq_index* ix, const rabitq_query_repr& r) {
  if (ix->scan_impl == 2 && r.lut == nullptr) {
    set_error("scan_impl 2 needs the lookup tables (rabitq_query_repr.lut)");
    return RABITQ_EINVAL;
  }
  return RABITQ_OK;
}

int launch_clear_counters(int32_t* cand_cnt, int64_t n, hipStream_t st) {
  if (n <= 0) return RABITQ_OK;
  hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, st, cand_cnt, n);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

int launch_seed(const rabitq_index* ix, const rabitq_query_repr& repr, int form, const int32_t* probe_ids, const float* probe_G,
                const float* probe_E, int64_t nq, int k, int nprobe, float* tau, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  if (int rc = need_lut(ix, repr)) return rc;
  ScanArgs a = base_args(ix);
  set_repr(a, ix, repr, form);
  a.probe_ids = probe_ids; a.probe_G = probe_G; a.probe_E = probe_E;
  set_nprobe(a, nprobe); a.k = k; a.tau_out = tau;
  const int W = ix->W, F = field_bits(ix->total_bits);
  const int impl = effective_impl(ix);
  if (!(seed_part0(a, W, F, impl, nq, st) || seed_part1(a, W, F, impl, nq, st) || seed_part2(a, W, F, impl, nq, st)))
    return bad_width();
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

// Long clusters are scanned in segments of about tseg tiles by separate work items; each segment of a split cluster
// contributes at most k keys to the pair's region of cand_stride keys (cand_cnt is advanced atomically).  The segment
// length adapts to the batch: a large batch has more work items than the chip has wavefront slots and keeps long
// segments (32 tiles); a small batch is cut finer, down to 2 tiles, so that about 4096 items exist.
static ScanPlan plan_for(const rabitq_index* ix, int64_t nq, int nprobe, int k, bool streaming, bool group) {
  ScanPlan p;
  p.streaming = streaming;
  p.qw = group || effective_impl(ix) == 1 ? QM : (p.streaming ? 1 : QW);
  const int64_t np_all = nq * nprobe;
  const int64_t est_items = std::min<int64_t>(np_all, (np_all + p.qw - 1) / p.qw + ix->nlist);
  const int64_t avg_tiles = std::max<int64_t>(1, ix->n_tiles / std::max(1, ix->nlist));
  p.tseg = (int)std::min<int64_t>(32, std::max<int64_t>(2, est_items * avg_tiles / 4096));
  // (a wavefront of the group scan of wide codes takes so long for its 16 pairs that nothing is gained by longer segments: 960-d, 5 bits,
  // 512 lists, 768 groups: 635 us in segments of 6 tiles, 467 in those of 2; 2048 groups: 1450 and 917)
  if (group && !group_narrow(ix->W)) p.tseg = 2;
  if (ix->seg_tiles > 0) p.tseg = ix->seg_tiles;
  p.segmax = std::max(1, next_pow2_host(k + TILE) / k);
  if (group && group_narrow(ix->W)) p.segmax = 1;  // (a wavefront owns its pairs' candidate regions)
  return p;
}

// Few pairs per list: every list is read from memory about once, by the prefetching variant of the popcount kernel,
// whose work items are single pairs with a descriptor each (never together with the split search, whose items are
// groups of pairs).  Taken when the handle's descriptor memory is large enough (ensure_stream_buffers, called by the
// entry points that may allocate); otherwise the general kernel does the same work.
ScanPlan scan_plan(const rabitq_index* ix, int64_t nq, int nprobe, int k) {
  const bool streaming = stream_shape(ix, nq, nprobe, k) && ix->item_desc != nullptr &&
                         stream_desc_slots(ix, nq, nprobe, k) <= ix->item_desc_cap;
  return plan_for(ix, nq, nprobe, k, streaming);
}

static SmallListArgs small_list_args(const rabitq_index* ix, const int32_t* probe_ids, int64_t nq, int nprobe, int k,
                                     int32_t* pair_off, int32_t* pair_ids, uint32_t* scratch, int32_t* cand_cnt) {
  const ScanPlan p = scan_plan(ix, nq, nprobe, k);
  SmallListArgs b{};
  b.probe_ids = probe_ids; b.nq = (int)nq; b.nprobe = nprobe; b.nlist = ix->nlist; b.tile_off = ix->tile_off;
  b.qw = p.qw; b.tseg = p.tseg; b.segmax = p.segmax; b.mask = scratch; b.pair_off = pair_off; b.pair_ids = pair_ids;
  b.item_off = ix->tile_off + (ix->nlist + 1); b.cand_cnt = cand_cnt;
  b.desc = nullptr;
  return b;
}

int launch_small_batch_lists(const rabitq_index* ix, const int32_t* probe_ids, int64_t nq, int nprobe, int k,
                             int32_t* pair_off, int32_t* pair_ids, uint32_t* scratch, int32_t* cand_cnt, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  if (nq > SMALL_BATCH_MAX) { set_error("small-batch list builder: more than 64 queries"); return RABITQ_EINVAL; }
  const SmallListArgs b = small_list_args(ix, probe_ids, nq, nprobe, k, pair_off, pair_ids, scratch, cand_cnt);
  hipLaunchKernelGGL(small_batch_lists_kernel, dim3(1), dim3(1024), 0, st, b);
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

int launch_small_select_seed(const rabitq_index* ix, const rabitq_query_repr& repr, const float* scores, int64_t nq, int k,
                             int nprobe, int32_t* probe_ids, float* probe_G, float* probe_E, float* tau, int32_t* pair_off,
                             int32_t* pair_ids, uint32_t* scratch, int32_t* cand_cnt, hipStream_t st) {
  if (nq <= 0) return RABITQ_OK;
  if (nq > SMALL_BATCH_MAX || nprobe > 64 || k > 64 || effective_impl(ix) == 2) {
    set_error("fused selection + seeding: needs at most 64 queries, nprobe <= 64, k <= 64 and a bitwise scan");
    return RABITQ_EINVAL;
  }
  ScanArgs a = base_args(ix);
  set_repr(a, ix, repr, QUERY_DIGITS);  // (qhat8 is not read)
  a.probe_ids = probe_ids; a.probe_G = probe_G; a.probe_E = probe_E;
  set_nprobe(a, nprobe); a.k = k; a.tau_out = tau;
  SmallSelectArgs b{};
  b.scores = scores; b.sq_norm = repr.sq_norm; b.centroid_sq = ix->centroid_sq; b.metric = ix->metric;
  // (with one probed list and 1-bit codes the scan's own top-k selects what a seeded threshold would: no seeding)
  b.do_seed = (ix->prune && !(nprobe == 1 && ix->total_bits == 1)) ? 1 : 0;
  b.probe_ids = probe_ids; b.probe_G = probe_G; b.probe_E = probe_E;
  b.ticket = ix->tile_off + 2 * (ix->nlist + 1);
  b.lists = small_list_args(ix, probe_ids, nq, nprobe, k, pair_off, pair_ids, scratch, cand_cnt);
  if (scan_plan(ix, nq, nprobe, k).streaming) {
    // (the workgroup that builds the lists also writes the descriptors of the prefetching scan's work items)
    b.lists.desc = reinterpret_cast<StreamDesc*>(ix->item_desc);
    b.lists.probe_G = probe_G; b.lists.probe_E = probe_E;
    b.lists.delta = repr.delta; b.lists.sum_q = repr.sum_q; b.lists.sum_qhat = repr.sum_qhat;
  }
  const int W = ix->W, F = field_bits(ix->total_bits);
  if (!(small_part0(a, b, W, F, st) || small_part1(a, b, W, F, st) || small_part2(a, b, W, F, st))) return bad_width();
  RQ_HIP(hipGetLastError());
  return RABITQ_OK;
}

int launch_scan(rabitq_index* ix, const rabitq_query_repr& repr, int form, const float* probe_G, const float* probe_E,
                const int32_t* pair_off, const int32_t* pair_ids, const float* tau, int64_t nq, int k, int nprobe,
                uint64_t* cand_keys, int32_t* cand_cnt, int32_t* dbg_ip, const int64_t* dbg_off, const ScanStreams& ss) {
  if (nq <= 0) return RABITQ_OK;
  const hipStream_t st = ss.main, sst = ss.setup;
  if (int rc = need_lut(ix, repr)) return rc;
  ScanArgs a = base_args(ix);
  set_repr(a, ix, repr, form);
  const int impl = effective_impl(ix);
  // Many pairs per list: groups of 16 pairs, estimates on the matrix cores (group scan or split search), where the handle's
  // buffers are large enough (ensure_split_buffers, called by the entry points that may allocate).
  const ScanRoute route = scan_route(ix, nq, nprobe, k);
  const bool group = route == ROUTE_GROUP, split = route == ROUTE_SPLIT;
  if (form == 0 && ix->total_bits > 1 && (group ? !group_narrow(ix->W) : !split && impl == 1))
    convert_stage_queries(ix, repr, nq, group, a, st);
  const ScanPlan plan = route == ROUTE_SINGLE ? scan_plan(ix, nq, nprobe, k) : plan_for(ix, nq, nprobe, k, false, group);
  const int qw = plan.qw;
  a.probe_G = probe_G; a.probe_E = probe_E; a.pair_off = pair_off; a.pair_ids = pair_ids; a.tau = tau;
  set_nprobe(a, nprobe); a.k = k;
  a.cand_stride = next_pow2_host(k + TILE);
  // LDS pool entries per pair: the popcount kernel may append a whole tile at once
  // (the matrix-core kernel's four wavefronts may together append 4 x 16 refined keys per round, or four whole
  // tiles when there is no long code)
  a.pool = next_pow2_host(k + TILE);
  if (impl == 1 && ix->total_bits == 1) a.pool = next_pow2_host(k + 4 * TILE);

  a.cand_keys = cand_keys; a.cand_cnt = cand_cnt; a.dbg_ip = dbg_ip; a.dbg_off = dbg_off;
  // work-item offsets live in the second half of the tile_off allocation (owned by the handle)
  int32_t* item_off = ix->tile_off + (ix->nlist + 1);
  a.item_off = item_off;
  a.tseg = plan.tseg;
  a.segmax = plan.segmax;
  a.streaming = plan.streaming ? 1 : 0;
  // Few pairs per list: the lists are read from memory about once each and a work item lasts as long as its list is
  // long, so the launch ends when its last long item does.  Handing the items out longest list first leaves the short
  // ones for the end (the popcount kernel's own item table only: the small-batch builder and the split search keep
  // cluster order, where items of one cluster share a cache).
  if (a.streaming && !ss.setup_done && ix->longest_first && ix->cluster_order != nullptr) a.order = ix->cluster_order;
  if (group) a.order = ix->cluster_order + ix->nlist;  // (dealt to the XCDs)
  if (!a.streaming) update_seg_cache(ix, a.tseg, a.segmax);
  const int64_t max_items = a.streaming ? stream_item_bound(ix, nq, nprobe, plan) : item_bound(ix, nq, nprobe, qw);
  ss.split = split || group;
  ss.estimated = split;
  ss.grouped = group;
  ss.streamed = a.streaming != 0;
  int32_t* item16 = ix->tile_off + 2 * (ix->nlist + 1) + TICKET_WORDS;
  uint32_t* mask_off = reinterpret_cast<uint32_t*>(item16 + (ix->nlist + 1));
  if (ss.setup_b) RQ_HIP(hipEventRecord(ss.setup_b, sst));
  // (one launch for the item table and, when the search is split, the two tables of its first half; a small batch's
  // list builder has written the item table already, with the same values)
  if (!ss.setup_done || split || group)
  {
    const bool small = ix->nlist <= SCAN_SMALL * SCAN_PER;
    auto table = split ? (small ? item_offsets_kernel<SCAN_SMALL, true, false> : item_offsets_kernel<SCAN_LARGE, true, false>)
                       : (small ? item_offsets_kernel<SCAN_SMALL, false, false> : item_offsets_kernel<SCAN_LARGE, false, false>);
    if (a.order)  // (streaming and group scan, never the split search)
      table = small ? item_offsets_kernel<SCAN_SMALL, false, true> : item_offsets_kernel<SCAN_LARGE, false, true>;
    hipLaunchKernelGGL(table, dim3(1), dim3(small ? SCAN_SMALL : SCAN_LARGE), 0, sst, pair_off, ix->tile_off, a.order,
                       ix->nlist, qw, a.tseg, a.segmax, item_off, item16, mask_off);
  }
  if (!ss.setup_done && !ss.counters_clear) {
    if (int rc = launch_clear_counters(cand_cnt, nq * nprobe, sst)) return rc;
  }
  if (a.streaming) a.stream_desc = reinterpret_cast<const StreamDesc*>(ix->item_desc);
  if (a.streaming && !ss.desc_done) {
    hipLaunchKernelGGL(stream_desc_kernel, dim3((unsigned)ix->nlist), dim3(64), 0, sst, a,
                       reinterpret_cast<StreamDesc*>(ix->item_desc));
  }
  if (split || group) {
    hipLaunchKernelGGL(item_desc_kernel, dim3((unsigned)ix->nlist), dim3(64), 0, sst, pair_off, ix->tile_off, item_off,
                       group ? nullptr : mask_off, a.order, qw, a.tseg, a.segmax, ix->item_desc);
    a.item_desc = ix->item_desc;
    if (group && !group_narrow(ix->W)) a.pool = group_pool(k);
  }
  if (split) {
    a.item_off16 = item16;
    a.mask_off = mask_off;
    a.surv_mask = ix->surv_mask;
    // (the refinement-only kernel lives on wavefronts in flight: smaller pools, checked every second round of 16 keys)
    a.pool = std::max(64, next_pow2_host(k + 32));
  }
  if (ss.setup_e) RQ_HIP(hipEventRecord(ss.setup_e, sst));
  if (sst != st) {
    RQ_HIP(hipEventRecord(ss.join, sst));
    RQ_HIP(hipStreamWaitEvent(st, ss.join, 0));
  }
  if (ss.scan_b) RQ_HIP(hipEventRecord(ss.scan_b, st));
  if (max_items > 0x7fffffff) {
    set_error("scan: too many work items");
    return RABITQ_EINVAL;
  }
  // (the prefetching variant's grid: the usual number of items, three for every two pairs, when the bound is larger;
  // its workgroups go on to further items if there are more.  So do the group scan's; its items are usually pairs / 16 and half
  // a group per list, some of them more than once for their segments)
  const int64_t usual = group ? (nq * nprobe / QM + ix->nlist) * 5 / 4 + 1024 : nq * nprobe + nq * nprobe / 2 + 1024;
  const unsigned grid = (unsigned)(a.streaming || group ? std::min(max_items, (usual + 7) / 8 * 8) : max_items);
  const bool dbg = dbg_ip != nullptr;
  const int W = ix->W, F = field_bits(ix->total_bits);
  if (split) {
    const int64_t items16 = item_bound(ix, nq, nprobe, QM);  // the same bound with 16 pairs per item
    if (ss.est_b) RQ_HIP(hipEventRecord(ss.est_b, st));
    if (!estimate_mfma(a, W, (unsigned)items16, dbg, st)) return bad_width();
    RQ_HIP(hipGetLastError());
    if (ss.est_e) RQ_HIP(hipEventRecord(ss.est_e, st));
  }
  if (group) {
    if (!scan_group(a, W, F, grid, dbg, st)) return bad_width();
  } else if (!(scan_part0(a, W, F, impl, grid, dbg, st) || scan_part1(a, W, F, impl, grid, dbg, st) ||
        scan_part2(a, W, F, impl, grid, dbg, st)))
    return bad_width();
  RQ_HIP(hipGetLastError());
  if (ss.scan_e) RQ_HIP(hipEventRecord(ss.scan_e, st));
  return RABITQ_OK;
}

}  // namespace rq
