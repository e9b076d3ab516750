// Margin statistics over the rows: what follows the row reduction in mars_margin_stats.
#pragma once

#include "common.h"

namespace mars {

// Distributions of the top-2 statistics over the rows (appendix histogram figure of the paper:
// top-1 logit, logit ratio z2/z1, probability ratio p2/p1, share of negative top-1 logits).
// A histogram over [lo, hi) with `bins` equal cells owns bins + 2 counters: below lo, the cells,
// at or above hi.  The cell is trunc(fl(fl(x - lo) * w)), w = fl32(bins / (hi - lo)), capped.
struct HistSpec {
  float lo[3], hi[3], w[3];
  int bins[3];
};
__device__ __forceinline__ int hist_cell(float x, float lo, float hi, float w, int bins) {
  if (x < lo) return 0;
  if (!(x < hi)) return bins + 1;
  const int k = static_cast<int>(__fmul_rn(__fsub_rn(x, lo), w));
  return min(k, bins - 1) + 1;
}
// counters: [bins0+2 | bins1+2 | bins2+2 | rows, z1 < 0, z1 <= 0, low margin at theta], cleared by the
// row reduction of the same call.  Rows with z1 <= 0 have no ratio (Sec. 3.3) and skip its histogram.
//
// What bounds it is atomics on the same few cache lines.  Where the counters fit into LDS (LOCAL) a work-group takes
// 1024 rows, counts them there and adds what it has counted to the caller's counters, one atomic per non-zero
// cell; otherwise the atomics are spread over many cells and many work-groups.  960 rows, 150
// counters: 6.4 us with 60 work-groups of 16 rows and three device-wide atomics per row, 4.7 now (most of it the launch and the rows' way from
// memory and the way back); 5 200 rows: 75.4 -> 56.3 us per call.
constexpr int kHistThreads = 1024, kHistLocal = 8192;
// Clearing the counters in LDS and going over them at the end is a step per 1024 of them: with many counters for each
// row it costs more than the atomics.  us per call, atomics against LDS: 8 106 counters, 8 rows 6.6 and 7.4, 512 rows 7.9 and 8.6,
// 960 rows 10.1 and 10.6; 152 counters, 8 rows 6.3 and 6.4, 64 rows 7.0 and 6.5; 1 506 counters, 512 rows 8.3 and 7.8.
static inline bool count_in_lds(long rows, long ncounters) { return ncounters <= kHistLocal && ncounters <= 8 * rows; }
constexpr int hist_rows(bool local) { return local ? kHistThreads : kHistThreads / 16; }  // rows of a work-group
template <bool LOCAL>
__global__ __launch_bounds__(kHistThreads) void margin_stats_kernel(const Partial* __restrict__ partials, int rows, int N,
                                                                    int parts, const float* __restrict__ theta, double cind,
                                                                    HistSpec hs, mars_margin_row* __restrict__ rows_out,
                                                                    unsigned int* __restrict__ counters) {
  const int first = blockIdx.x * hist_rows(LOCAL);
  const int n = min(hist_rows(LOCAL), rows - first);
  if (n <= 0) return;
  const int at1 = hs.bins[0] + 2, at2 = at1 + hs.bins[1] + 2, summary = at2 + hs.bins[2] + 2;
  __shared__ unsigned int sh_count[LOCAL ? kHistLocal : 4];
  // LOCAL: everything is counted in LDS; otherwise the summary alone, which would take one atomic per row on four addresses.
  const int nlocal = LOCAL ? summary + 4 : 4;
  unsigned int* const sum = LOCAL ? sh_count + summary : sh_count;
  unsigned int* const cells = LOCAL ? sh_count : counters;
  for (int i = threadIdx.x; i < nlocal; i += kHistThreads) sh_count[i] = 0u;
  __syncthreads();
  const Indicator ind = {MARS_IND_LOGIT_RATIO, cind};
  merge_rows_coop<kHistThreads>(partials + static_cast<size_t>(first) * parts, n, parts, 0.0f, ind,
                                [&](int row) { return theta[(first + row) / N]; },
                                [&](int row, const mars_row_stat& st) {
                                  mars_margin_row m;
                                  m.z1 = st.z1; m.z2 = st.z2;
                                  m.ratio = st.z2 / st.z1;
                                  m.prob_ratio = prob_ratio(st.z1, st.z2, cind);
                                  if (rows_out) rows_out[first + row] = m;
                                  atomicAdd(&cells[hist_cell(m.z1, hs.lo[0], hs.hi[0], hs.w[0], hs.bins[0])], 1u);
                                  if (st.z1 > 0.0f) atomicAdd(&cells[at1 + hist_cell(m.ratio, hs.lo[1], hs.hi[1], hs.w[1], hs.bins[1])], 1u);
                                  atomicAdd(&cells[at2 + hist_cell(m.prob_ratio, hs.lo[2], hs.hi[2], hs.w[2], hs.bins[2])], 1u);
                                  if (st.z1 < 0.0f) atomicAdd(&sum[1], 1u);
                                  if (!(st.z1 > 0.0f)) atomicAdd(&sum[2], 1u);
                                  if (st.relax_ok) atomicAdd(&sum[3], 1u);
                                });
  __syncthreads();
  if (threadIdx.x == 0) sum[0] = static_cast<unsigned int>(n);
  __syncthreads();
  unsigned int* const out = LOCAL ? counters : counters + summary;
  for (int i = threadIdx.x; i < nlocal; i += kHistThreads)
    if (sh_count[i] != 0u) atomicAdd(&out[i], sh_count[i]);
}

}  // namespace mars
