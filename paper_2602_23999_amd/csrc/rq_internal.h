// Internal declarations shared by the translation units of librabitq_hip.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <string>
#include <vector>

#include "rabitq.h"

namespace rq {

constexpr int TILE = RABITQ_TILE;
constexpr int QW = 4;        // queries handled by one wavefront of the popcount scan
constexpr int QM = 16;       // queries handled by one wavefront of the matrix-core scan
inline int qhat_stride(int D) { return (D + 63) / 64 * 64; }

struct Workspace {
  // per query
  float* q_rot = nullptr;
  rabitq_query_repr repr = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  int64_t cap_lut = 0;  // queries the lookup tables were sized for (allocated on first use of scan_impl 2)
  float* tau = nullptr;
  // coarse
  float* scores = nullptr;
  int32_t* probe_ids = nullptr;
  float* probe_G = nullptr;
  float* probe_E = nullptr;
  // lists
  int32_t* pair_off = nullptr;
  int32_t* pair_ids = nullptr;
  uint32_t* list_scratch = nullptr;
  // candidates
  uint64_t* cand_keys = nullptr;
  int32_t* cand_cnt = nullptr;
  // capacities the buffers were sized for
  int64_t cap_nq = 0;
  int64_t cap_pairs = 0;
  int64_t cap_cand = 0;
  int64_t cap_scratch = 0;
};

}  // namespace rq

namespace rq { struct ItemDesc; }

struct rabitq_index {
  int32_t dim = 0, W = 0, nlist = 0, total_bits = 0, metric = 0, F = 0, LW = 0;  // LW = long words per slot
  int64_t n = 0, n_tiles = 0, n_slots = 0;
  int device = 0;
  // device arrays
  float* rotation = nullptr;        // [D][D]
  float* mean_rot = nullptr;        // [D] mean * P of a centred index (nullptr: not centred)
  std::vector<float> host_mean;     // [D] the mean itself (empty: not centred)
  float* centroids_t = nullptr;     // [D][nlist]  (transposed c')
  float* centroid_sq = nullptr;     // [nlist]
  int32_t* tile_off = nullptr;      // [nlist+1] tile offsets | [nlist+1] scan work-item offsets | [TICKET_WORDS] zeroed ticket
                                    // | [nlist+1] work items of 16 pairs | [nlist+1] first survivor block (split search)
  int32_t* cluster_size = nullptr;  // [nlist]
  int32_t* cluster_order = nullptr; // [nlist] clusters by descending tile count, equal counts by ascending id
                                    // | [nlist] the same dealt to the XCDs (xcd_first)
  uint32_t* short_codes = nullptr;
  float* short_factors = nullptr;
  uint32_t* long_codes = nullptr;
  float* long_factors = nullptr;
  int32_t* ids = nullptr;
  std::vector<int32_t> host_tiles;  // tiles per cluster (host copy, sizes the scan grid)
  int32_t max_tiles = 0;            // the longest list's
  // segments per cluster in descending order for the segment limit seg_sorted_max and length seg_sorted_tseg, and their sum (scan grid bound)
  mutable std::vector<int> seg_sorted;
  mutable int seg_sorted_max = -1, seg_sorted_tseg = -1;
  mutable int64_t seg_total = 0;
  // options
  int prune = 1;
  int scan_impl = 3;  // 0 popcount, 1 matrix cores, 2 lookup tables, 3 chosen by code width (see effective_impl),
                      // 4 estimates on the matrix cores + refinement by the popcount kernel (split search)
  // survivor bits of the split search: blocks of 16 words; grown on demand by ensure_split_buffers, kept by the handle
  int last_scan_split = 0;   // the scan of the latest rabitq_search / rabitq_scan was split (rabitq_index_info)
  int last_scan_group = 0;   // ... by the group scan, as one kernel
  int last_scan_stream = 0;  // ... was the prefetching variant of the popcount kernel (one pair per work item)
  int split_min_pairs = 32;  // pairs per list, on average, from which scan_impl 3 / 4 split the search
  int group_min = -1;        // groups of 16 pairs from which they do it as one kernel; -1: chosen by code width (group_min_of)
  uint64_t* surv_mask = nullptr;
  int64_t surv_mask_blocks = 0;
  rq::ItemDesc* item_desc = nullptr;  // descriptors of work items (split search, group scan, streaming scan), grown on demand
  int64_t item_desc_cap = 0;
  uint32_t* stage_queries = nullptr;  // the queries handed to rabitq_scan in the scans' form, grown on demand (launch_scan)
  int64_t stage_queries_cap = 0;      // words
  std::vector<int64_t> tiles_prefix;  // [i] = tiles of the i largest lists (host; filled on first use)
  int overlap = 1;  // list building and scan set-up run beside the seeding on `side`
  int64_t max_batch = 0;  // queries per pass of rabitq_search; 0 = from the workspace budget
  int small_batch = 1;    // batches of at most SMALL_BATCH_MAX queries take the fused low-launch-count kernels
  int longest_first = 1;  // a scan that reads every list about once hands out its work items longest list first
  int seg_tiles = 0;      // tiles per scan work item of a long list; 0 = chosen from the batch (see launch_scan)
  // second stream of a search (default priority) and the events that fork it from and join it to the caller's
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  static constexpr int N_STAGES = 10;
  // begin / end of every stage, on the stream it ran on; bit s of `rec`: stage s was recorded in this search (a
  // small batch runs several stages as one kernel, recorded under the first of them)
  struct EventSet { hipEvent_t b[N_STAGES], e[N_STAGES]; unsigned rec; };
  std::vector<EventSet> prof_sets;  // one per recorded search
  int prof_used = 0, prof_limit = 0;
  unsigned prof_mask = 0x3ffu;  // stages whose events are recorded (bit s = stage s)
  rq::Workspace ws;
};

namespace rq {

// The scan the handle's option selects: "by code width" takes the matrix-core kernel from D = 960 on, where it was
// measured 3.2x faster than the popcount kernel (0.86 against 2.79 ms), and the popcount kernel below (D = 128: 0.28
// against 0.32 ms; at D = 768 the matrix-core kernel wins where the filter works, 4.2 against 5.8 ms, and loses where
// nearly every vector has to be refined, 32 against 22 ms).
// (4 is the popcount kernel everywhere except in launch_scan, which splits the search when it can: see split_search)
inline int effective_impl(const rabitq_index* ix) {
  const int impl = ix->scan_impl == 3 ? (ix->W >= 30 ? 1 : 0) : ix->scan_impl;
  return impl == 4 ? 0 : impl;
}

void set_error(const std::string& s);
int hip_fail(hipError_t e, const char* what);

#define RQ_HIP(call)                                  \
  do {                                                \
    hipError_t e__ = (call);                          \
    if (e__ != hipSuccess) return rq::hip_fail(e__, #call); \
  } while (0)

// order-preserving map float -> uint32 (ascending floats give ascending unsigned ints)
__host__ __device__ inline uint32_t f2ord(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__host__ __device__ inline float ord2f(uint32_t o) {
  uint32_t u = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
  return __builtin_bit_cast(float, u);
}

// ---- launchers (each returns a rabitq_status) ----
// C[M,N] = A[M,K] * B[K,N], row-major fp32.  mode 0: plain.  mode 1 (L2 coarse):
// C = rowv[m] + colv[n] - 2*acc.  mode 2 (IP coarse): C = -acc.  (launch_gemm_nearest, the assignment: colv[n] - 2*acc.)
// mode 4 (rotation of a centred index): C = acc - colv[n].
// tmin: null, or (modes 1 and 2) receives the smallest entry of every 32 columns as f2ord, [M][ceil(N / 32)]
int launch_gemm(const float* A, const float* B, float* C, int64_t M, int N, int K, int mode, const float* rowv,
                const float* colv, uint32_t* tmin, hipStream_t st);
int launch_gemm_nearest(const float* A, const float* B, uint64_t* keys, int64_t M, int N, int K, const float* colv, int* parts,
                        hipStream_t st);
// small batches: Q' = (Q - mean) P, the queries' representation and the coarse scores [nq][nlist] from one launch,
// bit-identical to launch_rotate + launch_query_prep + launch_gemm (mode 1 / 2)
int launch_small_front(const rabitq_index* ix, const float* queries, int64_t nq, float* q_rot, const rabitq_query_repr& o,
                       int form, float* scores, hipStream_t st);
// form: what the members hold (query_form).  The stage entry points hand out and take what the header says (0); a search hands
// its scans what they would otherwise make of it themselves, in the same space: the refinement's digits of q' in
// q_stage, the group scan's operand in qhat8 (rq_device.h).  Same numbers either way.
enum QueryForm { QUERY_DIGITS = 1, QUERY_FP8 = 2 };
struct PrepClear {  // memory that the preparation of a batch sets to zero on the way (none: all zero)
  uint32_t* bitmap = nullptr;
  int64_t n_bitmap = 0;
  int32_t* counters = nullptr;
  int64_t n_counters = 0;
};
PrepClear prep_clear(int64_t nq, int nlist, int nprobe, uint32_t* bitmap, int32_t* counters);
int launch_query_prep(const float* q_rot, int64_t nq, int D, int F, const rabitq_query_repr& out, int form, const PrepClear& clear,
                      hipStream_t st);
// tmin: the smallest score of every 32 lists as f2ord (launch_gemm), or null
bool select_by_minima(int nlist, int nprobe);  // is it worth having
int launch_select_probes(const float* scores, const uint32_t* tmin, const float* sq_norm, const float* centroid_sq, int64_t nq, int nlist,
                         int nprobe, int metric, int32_t* probe_ids, float* probe_G, float* probe_E, hipStream_t st);
int probe_select_variant(int nlist, int nprobe);  // which selection kernel launch_select_probes takes (see stages.hip)
int64_t probe_list_scratch_words(int32_t nlist, int64_t nq);
int launch_clear_list_bitmap(int64_t nq, int nlist, uint32_t* scratch, hipStream_t st);
int launch_build_lists(const int32_t* probe_ids, int64_t nq, int nprobe, int nlist, int32_t* pair_off,
                       int32_t* pair_ids, uint32_t* scratch, hipStream_t st, bool bitmap_is_clear = false);
int launch_seed(const rabitq_index* ix, const rabitq_query_repr& repr, int form, const int32_t* probe_ids, const float* probe_G,
                const float* probe_E, int64_t nq, int k, int nprobe, float* tau, hipStream_t st);
// Streams and events of one scan launch: the set-up kernels (work-item offsets, counter clearing) run on `setup`
// and the scan kernel on `main`; when the two differ, `join` is recorded on `setup` and awaited on `main`.  The
// four profiling events may be null.
struct ScanStreams {
  hipStream_t main = nullptr, setup = nullptr;
  hipEvent_t join = nullptr;
  hipEvent_t setup_b = nullptr, setup_e = nullptr, scan_b = nullptr, scan_e = nullptr;
  hipEvent_t est_b = nullptr, est_e = nullptr;  // around the estimate kernel of a split search
  mutable bool split = false;                  // out: the estimates ran on the matrix cores (group scan or split search)
  mutable bool estimated = false;              // out: ... as a kernel of their own, between est_b and est_e
  mutable bool grouped = false;                // out: ... in the group scan
  mutable bool streamed = false;               // out: the prefetching variant of the popcount kernel ran
  bool counters_clear = false;  // cand_cnt was already zeroed by launch_clear_counters
  bool desc_done = false;       // ... and so were the descriptors of the prefetching scan's work items (launch_small_select_seed)
  bool setup_done = false;      // work-item offsets and counters were already prepared (launch_small_batch_lists)
};
// How a scan launch cuts its work: pairs per work item, tiles per segment of a long list, segments per list at most.
struct ScanPlan { int qw, tseg, segmax; bool streaming; };
ScanPlan scan_plan(const rabitq_index* ix, int64_t nq, int nprobe, int k);
// Batches of at most SMALL_BATCH_MAX queries: pair lists, the scan's work-item offsets and the cleared candidate
// counters from ONE single-workgroup kernel (instead of the seven launches of launch_build_lists + the scan set-up).
// `scratch` holds at least 2 * nlist words.  Same pair_off / pair_ids as launch_build_lists.
constexpr int SMALL_BATCH_MAX = 64;
constexpr int TICKET_WORDS = 4;  // words behind the two offset arrays of rabitq_index::tile_off (zero between launches)
inline int64_t tile_off_words(int nlist) { return 4 * (int64_t)(nlist + 1) + TICKET_WORDS; }
// Split search (scan_impl 4): the first stage runs on the matrix cores for groups of 16 pairs and hands one survivor
// bit per (pair, vector) to the popcount kernel.  Built for every code with a long part (B > 1) of less than 960 dimensions and
// taken, where the group scan below is not, from split_min_pairs pairs per list on average.  split_mask_blocks bounds the
// blocks of survivor bits a search of (nq, nprobe) can need: sum_c ceil(cnt_c / 16) tiles_c <= (nq * tiles of the nprobe
// largest lists) / 16 + all tiles, because every query probes nprobe distinct lists.
inline bool split_built(const rabitq_index* ix) { return ix->total_bits > 1; }
inline bool split_wanted(const rabitq_index* ix, int64_t nq, int nprobe) {
  return (ix->scan_impl == 4 || ix->scan_impl == 3) && split_built(ix) && ix->W < 30 &&
         nq * nprobe >= (int64_t)ix->split_min_pairs * ix->nlist;
}
// ... as one kernel, the group scan (scan_group.hip says why these widths).  For codes of up to 256 dimensions it does not cut
// lists into segments, so the longest list must not outlast the launch: one wavefront works on it, while the chip's about
// 3072 share the rest (1024 lists of 13 tiles and one longer, 8192 groups, a share of 42 tiles each: 348 us with a longest list of
// 32, 433 of 64, 299 split; 20 000 groups, 95 tiles: 583 of 64, 759 of 128, 515 split, 622 split before the digits;
// k > 64, where the split search's pools take room from its wavefronts: 1164 lists of 5 tiles, the longest above 32, 224 and 380).  From D = 960 on it takes the place of the four-wavefront matrix-core kernel from 8 pairs per list on.
// A wavefront has 16 pairs to itself, so a search of few pairs leaves the chip idle: with less than a wavefront for each of its
// 4096 places (16 lists, 424 queries x 8: 120 us split, 244 by groups; 274 lists, 3438 groups: 282 and 342; 1683 lists, 3873
// groups: 320 and 374; 639 lists, 4265 groups: 194 and 152; 227 lists, 11836 groups: 209 and 173; from 512 groups on with the
// shorter work items of D >= 960 and codes of up to 4 bits: 330 us against 401 there) the former kernels keep it.  Longer codes
// of that width have twice the bytes to refine with, which the four-wavefront kernel's fuller rounds of candidates are better at:
// they go by groups from 768 on and for few neighbours (960-d, 5 bits, k = 10: 512 groups 324 us and 404 by groups, 768 groups
// 463 and 467, 1024 groups 652 and 604, the 1000 of hub lists 1095 and 837; k = 32: 1103 and 1190, 3215 and 5433).
// (scan_impl 4 from D = 960 on takes it at any number of groups: there is no split search of that width.)
// Up to 256 dimensions a pair's region holds the smallest power of two from k + 64 on and is cut to k when the 64 keys that a
// round may add do not fit: for k from 33 to 64 after less than 32 new keys, and at 64 after every one, so that the cuts
// outweigh the rest (11407 groups, k = 53: 580 us split, 1040 by groups; 3083, k = 55: 263 and 397; 24008, k = 50: 564 and 576).
// The choice by these two lines is the default; a group_min that is set takes its place.
inline int64_t group_min_of(const rabitq_index* ix, int k) {
  if (ix->group_min >= 0) return ix->group_min;
  if (ix->W < 30) return k > 32 && k <= 64 ? INT64_MAX / QM : 4096;
  if (ix->scan_impl == 4) return 0;
  return ix->total_bits <= 4 ? 512 : (k <= 16 ? 768 : INT64_MAX / QM);
}
inline bool group_wanted(const rabitq_index* ix, int64_t nq, int nprobe, int k) {
  if (!split_built(ix) || (ix->scan_impl != 3 && ix->scan_impl != 4)) return false;
  const int64_t pairs = nq * nprobe;
  if (pairs < QM * group_min_of(ix, k)) return false;
  if (ix->W >= 30) return pairs >= (int64_t)(ix->split_min_pairs < 8 ? ix->split_min_pairs : 8) * ix->nlist;
  if (ix->W > 8 || pairs < (int64_t)ix->split_min_pairs * ix->nlist) return false;
  const int64_t share = (pairs / QM + ix->nlist) * (ix->n_tiles / (ix->nlist > 0 ? ix->nlist : 1) + 1) / 3072;
  return ix->max_tiles <= std::max<int64_t>(share, k > 64 ? 64 : 32);
}
// Which scan a search of this shape gets, given the handle's buffers: SINGLE stands for the kernels of scan_impl 0, 1 and 2.
enum ScanRoute { ROUTE_SINGLE, ROUTE_SPLIT, ROUTE_GROUP };
ScanRoute scan_route(rabitq_index* ix, int64_t nq, int nprobe, int k);
// the form a search's queries take for it
inline int query_form(ScanRoute route) { return QUERY_DIGITS | (route != ROUTE_SINGLE ? QUERY_FP8 : 0); }
int64_t split_mask_blocks(rabitq_index* ix, int64_t nq, int nprobe);
// makes the handle's survivor-bit buffer large enough for (nq, nprobe); may allocate (then it synchronises the device)
int ensure_split_buffers(rabitq_index* ix, int64_t nq, int nprobe, int k);
// makes the handle's descriptor memory large enough for the prefetching scan of (nq, nprobe, k), when that is the shape;
// may allocate (then it synchronises the device)
int ensure_stream_buffers(rabitq_index* ix, int64_t nq, int nprobe, int k);
// The same for nprobe <= 64, k <= 64 and a bitwise scan, preceded in the same kernel by the selection of the probes
// from the coarse scores and the seeding of the thresholds (one workgroup per query; the last one to finish builds the
// lists): everything between the coarse scores and the scan in one launch.
int launch_small_select_seed(const rabitq_index* ix, const rabitq_query_repr& repr, const float* scores, int64_t nq, int k,
                             int nprobe, int32_t* probe_ids, float* probe_G, float* probe_E, float* tau, int32_t* pair_off,
                             int32_t* pair_ids, uint32_t* scratch, int32_t* cand_cnt, hipStream_t st);
int launch_small_batch_lists(const rabitq_index* ix, const int32_t* probe_ids, int64_t nq, int nprobe, int k,
                             int32_t* pair_off, int32_t* pair_ids, uint32_t* scratch, int32_t* cand_cnt, hipStream_t st);
int launch_clear_counters(int32_t* cand_cnt, int64_t n, hipStream_t st);
int launch_scan(rabitq_index* ix, const rabitq_query_repr& repr, int form, const float* probe_G, const float* probe_E,
                const int32_t* pair_off, const int32_t* pair_ids, const float* tau, int64_t nq, int k, int nprobe,
                uint64_t* cand_keys, int32_t* cand_cnt, int32_t* dbg_ip, const int64_t* dbg_off, const ScanStreams& ss);
int launch_merge(const uint64_t* cand_keys, const int32_t* cand_cnt, int64_t nq, int k, int nprobe, int metric,
                 int64_t* out_ids, float* out_dists, hipStream_t st);
int launch_fill_f32(float* p, int64_t n, float v, hipStream_t st);
int build_index_device(rabitq_index* ix, const float* data, const float* rotation_host, int kmeans_iters,
                       int64_t train_size, float eps0, int center, hipStream_t st);
// stores `mean` [D] (host) in the handle together with mean * P on the device
int set_index_mean(rabitq_index* ix, const float* mean, const float* rotation_host, hipStream_t st);
// Q' = (Q - mean) P for the handle's rotation
int launch_rotate(const rabitq_index* ix, const float* q, float* q_rot, int64_t nq, hipStream_t st);

}  // namespace rq
