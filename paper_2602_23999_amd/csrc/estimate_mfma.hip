// First stage of the cluster-local search (Sections 3.3.4, 3.4.1(2)) on the matrix cores, as a kernel of its own:
// 1-bit estimates and the filter for 16 pairs of one cluster per wavefront, one 64-vector tile at a time.  What it
// leaves behind is one bit per (pair, vector): "survives the filter".  The refinement of the survivors, the pools and
// the output are the popcount kernel's, which in this mode reads those bits instead of estimating (scan.hip, MASKED).
// Splitting the stages lets each run at its own occupancy: this kernel needs registers and no LDS, the refinement
// needs LDS and many wavefronts in flight to hide the scattered long-code reads.
//
// Survivor bits.  A block of 128 bytes belongs to (cluster, group of 16 pairs, tile); the blocks of cluster c start at
// mask_off[c] and are ordered [group][tile].  A block is what the 64 lanes of the wavefront hold after the tile: lane
// 16 g + lj writes 16 bits about vectors 4 lj + cb (cb = 0..3) and pairs 4 g + r (r = 0..3) of the group; bit
// 4 cb + r is SET when that vector does NOT survive for that pair.
#include "rq_estimate.h"

namespace rq {

template <int W, bool DBG>
__device__ __forceinline__ void estimate_body(const ScanArgs& a) {
  const int lane = threadIdx.x, lj = lane & 15, g = lane >> 4;

  // XCD-aware order, as in the popcount kernel: each XCD gets a contiguous range of the true item count
  const int n_items = a.item_off16[a.nlist];
  const int per = (n_items + 7) >> 3;
  const int item = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || item >= n_items) return;
  const int c = wave_upper_cluster(a.item_off16, a.nlist, item, lane);
  const int t0 = a.tile_off[c], tc1 = a.tile_off[c + 1];
  const int nseg = seg_count(tc1 - t0, a.tseg, a.segmax);
  const int local = item - a.item_off16[c];
  const int grp = local / nseg, sidx = local - grp * nseg;
  const int seglen = (tc1 - t0 + nseg - 1) / nseg;
  const int ts = t0 + sidx * seglen, te = min(tc1, ts + seglen);
  const int pbeg = a.pair_off[c] + grp * QM;
  const int np = __builtin_amdgcn_readfirstlane(min(QM, a.pair_off[c + 1] - pbeg));
  // first block of this group's tiles
  uint16_t* blocks = reinterpret_cast<uint16_t*>(a.surv_mask + ((int64_t)a.mask_off[c] + (int64_t)grp * (tc1 - t0)) * 16);

  __shared__ __align__(16) int8_t scratch[ESTIMATE_SCRATCH];
  __shared__ float4 table[QM];
  TileEstimator<W, DBG> est;
  if (ts < te) est.fetch(a, ts, lj, g);  // (before the pairs, so that the two waits overlap)
  const int pp = a.pair_ids[pbeg + min(lj, np - 1)];
  float G, dl;
  est.pairs(a, pp, pair_query(a, pp), np, scratch, table, lane, G, dl);
  wave_sync();
  for (int tile = ts; tile < te; ++tile) {
    const uint32_t alive = est.scan(a, min(tile + 1, te - 1), lj, g, [&](int pair, int v, int I) {  // (past the end: a harmless re-read)
      if (pair < np) a.dbg_ip[a.dbg_off[pbeg + pair] + (int64_t)(tile - t0) * TILE + v] = I;
    });
    blocks[(int64_t)(tile - t0) * TILE + lane] = (uint16_t)~alive;
  }
}

// (registers for four wavefronts per SIMD for codes of up to 512 bits, three beyond, where the query operand alone takes 48)
template <int W, bool DBG>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(W > 16 ? 3 : 4))) void estimate_mfma_kernel(ScanArgs a) {
  estimate_body<W, DBG>(a);
}

template <int W>
static void launch_w(const ScanArgs& a, unsigned grid, bool dbg, hipStream_t st) {
  if (dbg)
    hipLaunchKernelGGL((estimate_mfma_kernel<W, true>), dim3(grid), dim3(64), 0, st, a);
  else
    hipLaunchKernelGGL((estimate_mfma_kernel<W, false>), dim3(grid), dim3(64), 0, st, a);
}

// Returns false when the kernel is not built for the code width W (from 960 dimensions on the group scan takes its place).
bool estimate_mfma(const ScanArgs& a, int W, unsigned grid, bool dbg, hipStream_t st) {
  switch (W) {
    case 1: launch_w<1>(a, grid, dbg, st); return true;
    case 2: launch_w<2>(a, grid, dbg, st); return true;
    case 3: launch_w<3>(a, grid, dbg, st); return true;
    case 4: launch_w<4>(a, grid, dbg, st); return true;
    case 8: launch_w<8>(a, grid, dbg, st); return true;
    case 16: launch_w<16>(a, grid, dbg, st); return true;
    case 24: launch_w<24>(a, grid, dbg, st); return true;
    default: return false;
  }
}

}  // namespace rq
