// C ABI of the MARS verification pass (see include/mars.h): argument checks,
// workspace carving and kernel launches.  Nothing here allocates or synchronises.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>

#include "../../include/mars.h"
#include "common.h"
#include "row_reduce.h"
#include "margin.h"
#include "tail.h"
#include "onehot.h"
#include "lmhead.h"

namespace mars {

constexpr int kMaxTargetItems = 768;    // work-groups the row reduction aims for on a large input: three per compute unit
                                        // (four fit; 960 rows of 151 936 run faster as 960 work-groups than as 1 920)
constexpr int kMinTargetItems = 128;    // ... and on a small one
constexpr int kItemElemsLog2 = 16;      // in between: about one work-group per 65 536 elements
constexpr int kMinSplitElems = 8192;    // no split shorter than this
constexpr size_t kAlign = 256;
constexpr int kDefaultSpinLimit = 256;  // polls before a work-group stops waiting for a partner's sum

static size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Splits per row: a function of (rows, V) only, so that the workspace size does not depend on
// the element type.  A large input needs several work-groups per compute unit to keep the memory
// pipeline full.  A small one (a single request) is bound by latency, not by bandwidth: the row
// reduction takes about as long with a few hundred work-groups as with a thousand, while every
// split adds partial results that the per-request kernel behind it has to merge.
static int choose_splits(long rows, int V) {
  long target = (rows * static_cast<long>(V)) >> kItemElemsLog2;
  if (target < kMinTargetItems) target = kMinTargetItems;
  if (target > kMaxTargetItems) target = kMaxTargetItems;
  long want = (target + rows - 1) / rows;
  long cap = V / kMinSplitElems;
  if (cap < 1) cap = 1;
  if (want > cap) want = cap;
  if (want < 1) want = 1;
  return static_cast<int>(want);
}

struct Layout {
  int splits, G;
  size_t partials_off, stats_off, xslots_off, gathered_off, least;
  size_t table_off, low_off, total;
};

// Work-groups per request in the sampling tail: enough to spread a request's row passes over
// the chip when there are few requests, not more than one work-group per compute unit in
// total (they exchange sums, and that is quick only while all of them are resident), and every
// slice at least 4096 vocabulary entries long.  The workspace is laid out for the compute units
// of an MI355X; a GPU with fewer gets fewer work-groups per request at launch (below).
constexpr int kComputeUnits = 256;
static int compute_units() {  // of the current GPU, asked once
  static int cached = 0;
  if (cached <= 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      return kComputeUnits;
    cached = n;
  }
  return cached;
}
static int choose_groups(int B, int V) {
  int G = kComputeUnits / B;
  const int cap = V / 4096;
  if (G > cap) G = cap;
  if (G > kMaxGroupsPerRequest) G = kMaxGroupsPerRequest;
  if (G < 1) G = 1;
  return G;
}

// The chunks of a row of V entries (elt bytes each) reduced in `splits` shares, and the bytes their sums take.
static ChunkSpec row_chunks(int V, size_t elt, int splits) {
  const int nvec = V / static_cast<int>(16 / elt), vps = (nvec + splits - 1) / splits;
  return chunk_spec(splits, vps > 0 ? vps : 1);
}
static size_t table_bytes(long rows, const ChunkSpec& s) {
  return static_cast<size_t>(rows) * s.items * s.slots * kChunkWaves * sizeof(float2);
}

// K = thresholds per request: the row reduction works on the B*N rows once, the per-request
// part on K*B requests (statistics table and exchange words per (threshold, request)).
static Layout layout(int B, int N, int V, int K = 1) {
  Layout L;
  const long rows = static_cast<long>(B) * N;
  L.splits = choose_splits(rows, V);
  L.partials_off = 0;
  // (the merged statistics had a place here; kernels hold them now, and the sizes callers know stay)
  L.stats_off = align_up(static_cast<size_t>(rows) * L.splits * kPartsPerItem * sizeof(Partial));
  L.G = choose_groups(K * B, V);
  L.xslots_off = L.stats_off + align_up(static_cast<size_t>(K) * rows * sizeof(mars_row_stat));
  L.gathered_off = L.xslots_off +
                   align_up(static_cast<size_t>(K) * B * (N + 2) * 2 * L.G * sizeof(unsigned long long));
  L.least = L.gathered_off + align_up(static_cast<size_t>(rows) * sizeof(float2));
  // The sums of the rows' chunks, and what their rounding has left over, half the bytes: where the statistics had their place and the exchange words, which
  // that walk does not need, have theirs, if it is large enough.  (A workspace of the least size has no room for the sums: the draw
  // goes over the row.)
  L.table_off = L.least;
  const size_t wide = table_bytes(rows, row_chunks(V, sizeof(float), L.splits)),
               narrow = table_bytes(rows, row_chunks(V, sizeof(bf16_t), L.splits));
  const size_t table = align_up(wide > narrow ? wide : narrow), low = align_up(table / 2);
  const bool behind = low > L.gathered_off - L.stats_off;
  L.low_off = behind ? L.table_off + table : L.stats_off;
  L.total = L.table_off + table + (behind ? low : 0);
  return L;
}

static bool sizes_ok(int B, int N, int V, int K = 1) {
  if (B < 1 || N < 1 || N > MARS_MAX_NODES || V < MARS_MIN_VOCAB || K < 1 || K > MARS_MAX_THETAS) return false;
  const long rows = static_cast<long>(B) * N * K;
  return rows <= 0x7FFFFFFFL / 64;  // rows * splits must fit the grid and int arithmetic
}

template <typename T, int EPV, bool RAGGED>
static hipError_t launch_row_reduce_t(const void* logits, long rows, int V, int splits, bool sampling, float c,
                                      Partial* partials, const ClearArgs& clr, hipStream_t stream) {
  const int nvec = V / EPV;  // (the most a row can have)
  const int vps = (nvec + splits - 1) / splits;
  const dim3 grid(static_cast<unsigned int>(rows * splits)), block(kRowThreads);
  if (sampling && clr.table)
    hipLaunchKernelGGL((row_reduce_kernel<T, EPV, true, RAGGED, true>), grid, block, 0, stream, static_cast<const T*>(logits), V,
                       splits, vps, c, partials, clr);
  else if (sampling)
    hipLaunchKernelGGL((row_reduce_kernel<T, EPV, true, RAGGED, false>), grid, block, 0, stream, static_cast<const T*>(logits), V,
                       splits, vps, c, partials, clr);
  else
    hipLaunchKernelGGL((row_reduce_kernel<T, EPV, false, RAGGED, false>), grid, block, 0, stream, static_cast<const T*>(logits), V,
                       splits, vps, c, partials, clr);
  return hipGetLastError();
}

// Rows off a 16-byte boundary of at most this many entries are read one element per load.  By vectors one or two of the
// work-group's eight waves do all the work, and a wave with a handful of vectors does not find two batch maxima
// and ranks its elements one by one.  One element per load against vectors, us, bf16: 21 rows of 13 entries with the sum of
// exponentials 3.9 and 5.3; 960 rows of 61 entries 6.3 and 7.8, of 511 7.2 and 7.7, of 1 001 7.4 and 7.8, of 1 501 even.
// Greedy, or fp32: 8 rows of 255 entries 3.6 and 3.9, of 511 3.8-3.9 both, longer ones gain from vectors.
static int single_elements(int dtype, bool sampling) { return dtype == MARS_BF16 && sampling ? 1024 : 512; }
// 16-byte loads; rows that do not all start on a 16-byte boundary take the form that looks for the first one, or, where
// they are short, the one of single elements.
static hipError_t launch_row_reduce(const void* logits, int dtype, long rows, int V, int splits, bool sampling,
                                    float c, Partial* partials, const ClearArgs& clr, hipStream_t stream) {
  const size_t elt = dtype == MARS_BF16 ? 2 : 4;
  const bool even = (reinterpret_cast<uintptr_t>(logits) % 16 == 0) && ((static_cast<size_t>(V) * elt) % 16 == 0);
  if (!even && V <= single_elements(dtype, sampling))
    return dtype == MARS_BF16 ? launch_row_reduce_t<bf16_t, 1, false>(logits, rows, V, splits, sampling, c, partials, clr, stream)
                              : launch_row_reduce_t<float, 1, false>(logits, rows, V, splits, sampling, c, partials, clr, stream);
  if (dtype == MARS_BF16)
    return even ? launch_row_reduce_t<bf16_t, 8, false>(logits, rows, V, splits, sampling, c, partials, clr, stream)
                : launch_row_reduce_t<bf16_t, 8, true>(logits, rows, V, splits, sampling, c, partials, clr, stream);
  return even ? launch_row_reduce_t<float, 4, false>(logits, rows, V, splits, sampling, c, partials, clr, stream)
              : launch_row_reduce_t<float, 4, true>(logits, rows, V, splits, sampling, c, partials, clr, stream);
}

static float log2e_over_t(float temperature) {
  return temperature > 0.0f ? static_cast<float>(1.4426950408889634 / static_cast<double>(temperature)) : 0.0f;
}

// log2(e) / T' for the probability-ratio indicator: T' is the sampling temperature, 1 in greedy mode.
static double indicator_scale(float temperature) {
  return 1.4426950408889634 / (temperature > 0.0f ? static_cast<double>(temperature) : 1.0);
}

static ClearArgs clear_args(char* ws, const Layout& L, int B, int N, int K) {
  ClearArgs clr;
  clr.xslots = reinterpret_cast<unsigned long long*>(ws + L.xslots_off);
  clr.N = N; clr.B = B; clr.xwords = 2 * L.G; clr.copies = K;
  clr.counters = nullptr; clr.ncounters = 0;
  clr.par = nullptr; clr.tok = nullptr; clr.q = nullptr; clr.q_bf16 = 0; clr.gathered = nullptr;
  clr.table = nullptr; clr.table_low = nullptr; clr.slots = 1; clr.batches = 0;
  return clr;
}

// ---------------------------------------------------------------- LM head fused with the row reduction
// Slab height and tile width: see lm_plan.  The hardware hands work-group i to die i mod 8 and a work-group fills a
// compute unit, so the work-groups are dealt out die by die, an equal share to each, and no die is given more
// work-groups than it has compute units (its last ones would start when the others have finished: twice the time).
//
// The forms of the fused kernel and what a unit (bm rows x bn entries) takes in each, us: for a step of 64 hidden elements,
// alone and what is added when all compute units are at work, and for a unit beside its steps, greedy and sampling; and the
// rate at which the weight streams through the chip in this form, TB/s.  Fitted to 2 200 shapes (rows 4-2 048, V 1 000-152 000,
// H 1 024-4 096, both modes, all forms that make sense for the shape).  The figures are good to some 10 %, so the choice is judged by its
// worst shape too: 4 780 shapes (rows 4-2 048, V 1 000-152 000, H 512-5 120, both modes; half with a weight that comes from memory, half with
// the same weight call after call), every form timed in turn.  Against the form through registers the one chosen takes 0.881 times the time (geometric
// mean; the best one 0.872) and is more than 2 % slower on 36 shapes, 8.1 % at worst.  30 of these find their weight in the cache, most with a
// vocabulary of 32 000, which narrow tiles fill the chip with in one round: from memory they win there (60 rows x 4096 55.1 us, 63.3 with tiles
// of 256 entries, 67.6 through registers), from the cache not always (9 rows x 4096 49.3, 43.9, 45.8), and nobody here knows which it is.
// The first four are the kernel that stages through registers, with a tile of 256 (which of them: lm_plan); the others the ring (lmhead.h), which wins
// where there are few units -- a small vocabulary, or up to 256 rows -- since its tiles are narrower and its requests go out earlier,
// where the weight is streamed once, and under sampling on many sizes of more rows: 56 rows x 4096 x 2 250 45 -> 22 us per call, 40 x 4096 x 32 000 74 -> 55, 120 x 4096 x 32 000 73 -> 58, 60 x 4096 x
// 151 936 214 -> 188 (under sampling 254 -> 235).
// The sampling form of 192 rows takes 9.0 us for a unit beside its steps since its stores leave 64 bytes of a row at a time; with the 11.6 of
// before, many rows with few hidden elements went to the ring (1 984 rows x 1024 x 64 000 320 us per call instead of 303, 1 620 x 640 x 62 816 213
// instead of 194).  Without this and the merging (lm_plan) 103 shapes are more than 2 % slower, 18 % at worst.
struct LmForm { int bm, bn, stages; float step, step_full, unit, unit_sampling, rate; };
constexpr LmForm kLmForms[] = {
    {64, 256, 0, 0.48f, 0.28f, 0.0f, 0.0f, 5.4f},
    {128, 256, 0, 0.69f, 0.22f, 0.4f, 5.4f, 4.7f},
    {192, 256, 0, 0.63f, 0.54f, 2.1f, 9.0f, 5.0f},
    {256, 256, 0, 0.80f, 0.68f, 4.4f, 0.0f, 5.0f},  // (greedy: the sampling form does not fit the registers)
    {64, 64, 8, 0.081f, 0.18f, 0.0f, 0.6f, 6.5f},
    {64, 128, 5, 0.15f, 0.30f, 0.0f, 1.2f, 6.4f},
    {64, 256, 3, 0.30f, 0.53f, 0.0f, 1.2f, 6.5f},
    {128, 128, 4, 0.24f, 0.28f, 0.2f, 2.2f, 5.8f},
    {128, 256, 3, 0.48f, 0.37f, 1.2f, 4.8f, 5.9f},
    {256, 128, 3, 0.45f, 0.33f, 1.7f, 5.4f, 4.4f},
};
// A weight of at least this many bytes, read once per call, is read past the caches: 6.9 TB/s instead of 6.2 (the bare stream
// of 1.6 GB and of 1.2 GB).  A smaller one may still lie in the Infinity Cache from the call before.
constexpr size_t kLmOnceBytes = size_t(256) << 20;
struct LmPlan {
  int form, bm, bn, slabs, tiles_n, launch_slabs, parts;
  bool once;  // the weight is read past the caches
  bool wide;  // sizes beyond what a buffer spans
  LmGrid grid;  // of a full launch
};
constexpr int kDies = 8;
// Slabs of a band, at most: work-groups of a die then share weight tiles and hidden states about evenly, and few bands
// leave few columns narrower than a work-group's share, behind which the work-groups of a band are out of step
// with the next one's.  6 656 rows in slabs of 256: 6.26 ms with 5, 6.14 with 7 and 9, 6.08 with 13, 6.10 with 26;
// 2 048 rows x 128 256: 1 620 us with 7 (two bands of 4), 1 576 with 13 (one of 8).
constexpr int kLmBand = 13;
constexpr int kLmFormCount = sizeof(kLmForms) / sizeof(kLmForms[0]);
constexpr double kLmCallUs = 12.0;  // launch and per-request kernel
constexpr double kLmMergeGreedy = 0.01, kLmMergeSampling = 0.02;  // for a partial result of 64 rows
// On a near tie the form through registers: the ring has to be 7 % faster by figures good to some 10 %.  With 0.95 60 instead of 36 of 4 780 shapes
// are more than 2 % slower than through registers, with 0.90 the mean loses 0.7 %.  (What it costs: 960 rows x 1024 x 2 256 27.9 us, 24.6 in the ring.)
constexpr double kLmKnown = 0.93;
struct LmUnits { long slabs, tiles, count, rounds; };
static LmUnits lm_units(const LmForm& m, long rows, int V) {
  LmUnits u;
  u.slabs = (rows + m.bm - 1) / m.bm;
  u.tiles = (static_cast<long>(V) + m.bn - 1) / m.bn;
  u.count = u.slabs * u.tiles;
  u.rounds = (u.count + kComputeUnits - 1) / kComputeUnits;
  return u;
}
// us per call: the units' rounds, or the weight's way from memory, whichever is more (where they are close, more than either).
static double lm_time(const LmForm& m, long rows, int V, int H, bool sampling) {
  const LmUnits u = lm_units(m, rows, V);
  const double rounds = static_cast<double>(u.rounds), fill = static_cast<double>(u.count) / (rounds * kComputeUnits);
  const double work = rounds * ((H / kLmBK) * (m.step + m.step_full * fill) + (sampling ? m.unit_sampling : m.unit));
  const double stream = static_cast<double>(V) * H * 2e-6 / m.rate;
  return std::sqrt(std::sqrt(work * work * work * work + stream * stream * stream * stream)) + kLmCallUs;
}
// us the per-request kernel takes to merge the partial results of a request's rows beyond what kLmCallUs holds: one
// per column of tiles.  (Rows of up to 64 nodes were looked at.)
static double lm_merge_time(const LmForm& m, long rows, int N, int V, bool sampling) {
  const LmUnits u = lm_units(m, rows, V);
  const long width = u.rounds < u.tiles ? u.rounds : u.tiles, columns = (u.tiles + width - 1) / width;
  return (sampling ? kLmMergeSampling : kLmMergeGreedy) * static_cast<double>(columns) * (N < 64 ? N : 64) / 64.0;
}
static LmPlan lm_plan(long rows, int N, int V, int H, bool sampling) {
  LmPlan p;
  p.wide = H > (1 << 22) || V > (1 << 25);
  // Through registers, the slab height that takes the least time: units per work-group x time per unit.  Measured per unit at
  // H = 4096, greedy form: 49-51 us with 64 rows, 61-63 with 128, 80-83 with 192, 100-104 with 256; with two slabs
  // of 64 and a work-group on (nearly) every compute unit the weight's way from memory bounds it, at
  // 78 us (128 rows, one slab: 75); with one slab both heights wait for the weight (60 rows: 215.5 us per call
  // with 64, 218.2 with 128).  The sampling form does not fit the registers with 256.  (Both forms and every H go by these figures.)
  static const double kHeightCost[] = {0.60, 0.75, 1.0, 1.235};
  double least = -1.0;
  for (int f = 0; f < (p.wide ? 1 : sampling ? 3 : 4); ++f) {
    const LmUnits u = lm_units(kLmForms[f], rows, V);
    const bool weight_bound = f == 0 && u.slabs == 2 && u.count >= 192;
    const double time = static_cast<double>(u.rounds) * (weight_bound ? 0.87 : kHeightCost[f]);
    if (least < 0.0 || time < least) { least = time; p.form = f; }
  }
  // Against the ring's forms, by kLmForms; if one of them takes less, the one of them that leaves the least work to it and to the
  // per-request kernel together.  (Tiles half as wide are twice as many partial results: 60 rows x 1024 x 32 000, whose weight
  // stays in the cache, 22.5 us per call with tiles of 128 entries, 20.1 with 256, 20.6 through registers.  The merging counts among the
  // ring's forms alone: counted against the form through registers as well, some shapes went back that take a quarter longer there.)
  const double known = lm_time(kLmForms[p.form], rows, V, H, sampling) * kLmKnown;
  double best = -1.0;
  int ring = -1;
  bool faster = false;
  for (int f = 4; f < kLmFormCount && !p.wide; ++f) {
    // (units of fewer steps than the ring has stages, and many slabs of 64 rows, were not looked at)
    if (kLmForms[f].stages > H / kLmBK || (kLmForms[f].bm == 64 && rows > 4 * 64)) continue;
    const double time = lm_time(kLmForms[f], rows, V, H, sampling);
    const double all = time + lm_merge_time(kLmForms[f], rows, N, V, sampling);
    faster |= time < known;
    if (ring < 0 || all < best) { best = all; ring = f; }
  }
  if (faster) p.form = ring;
  const LmForm& form = kLmForms[p.form];
  p.bm = form.bm; p.bn = form.bn;
  p.tiles_n = static_cast<int>((static_cast<long>(V) + p.bn - 1) / p.bn);
  p.slabs = static_cast<int>((rows + p.bm - 1) / p.bm);
  p.once = p.slabs == 1 && static_cast<size_t>(V) * H * 2 >= kLmOnceBytes;
  // (unit numbers are 32-bit: inputs far beyond the ordinary take several launches)
  const long most = (1L << 30) / p.tiles_n;
  p.launch_slabs = static_cast<int>(p.slabs < most ? p.slabs : most < 1 ? 1 : most);
  LmGrid& g = p.grid;
  g.slabs = p.launch_slabs;
  const int bands = (g.slabs + kLmBand - 1) / kLmBand;
  g.band = (g.slabs + bands - 1) / bands;
  g.tiles_n = p.tiles_n;
  g.units = g.slabs * p.tiles_n;
  g.width = (g.units + kComputeUnits - 1) / kComputeUnits;
  if (g.width > p.tiles_n) g.width = p.tiles_n;
  const int columns = (p.tiles_n + g.width - 1) / g.width;
  g.split = g.slabs == 1 || p.tiles_n % g.width == 0 ? columns : bands == 1 ? columns - 1 : 0;
  g.parts = p.parts = 2 * columns - g.split;
  return p;
}

// The fused kernel over all slabs.
template <bool SAMPLING>
static hipError_t launch_lmhead(const LmPlan& p, const bf16_t* hidden, const bf16_t* weight, int M, int V, int H,
                                Partial* partials, bf16_t* logits_out, float c, LmClear clear, hipStream_t stream) {
  for (int s0 = 0; s0 < p.slabs; s0 += p.launch_slabs) {
    LmGrid g = p.grid;
    g.slabs = p.slabs - s0 < p.launch_slabs ? p.slabs - s0 : p.launch_slabs;
    g.units = g.slabs * g.tiles_n;
    const int groups = (g.units + g.width - 1) / g.width, per_die = (groups + kDies - 1) / kDies;
    const dim3 grid(static_cast<unsigned int>(kDies * per_die)), block(kLmThreads);
    const size_t row0 = static_cast<size_t>(s0) * p.bm;
    const int rows = M - static_cast<int>(row0);
    const bf16_t* h = hidden + row0 * H;
    Partial* out = partials + row0 * p.parts;
    bf16_t* lo = SAMPLING ? logits_out + row0 * V : nullptr;
#define MARS_LM_LAUNCH(...)                                                                                            \
  hipLaunchKernelGGL((lmhead_reduce_kernel<__VA_ARGS__>), grid, block, 0, stream, h, weight, rows, V, H, g, out, lo, c, clear)
#define MARS_LM_RING(BM, BN, STAGES)                                                                                  \
  if (p.once)                                                                                                          \
    hipLaunchKernelGGL((lmhead_ring_kernel<BM, BN, STAGES, SAMPLING, true>), grid, block, 0, stream, h, weight, rows, V, H, g, out, lo, c, clear); \
  else                                                                                                                 \
    hipLaunchKernelGGL((lmhead_ring_kernel<BM, BN, STAGES, SAMPLING, false>), grid, block, 0, stream, h, weight, rows, V, H, g, out, lo, c, clear)
    switch (p.form) {
      case 0:
        if (p.wide) MARS_LM_LAUNCH(64, SAMPLING, true); else MARS_LM_LAUNCH(64, SAMPLING);
        break;
      case 1: MARS_LM_LAUNCH(128, SAMPLING); break;
      case 2: MARS_LM_LAUNCH(192, SAMPLING); break;
      case 3:
        if constexpr (!SAMPLING) MARS_LM_LAUNCH(256, false);
        break;
      case 4: MARS_LM_RING(64, 64, 8); break;
      case 5: MARS_LM_RING(64, 128, 5); break;
      case 6: MARS_LM_RING(64, 256, 3); break;
      case 7: MARS_LM_RING(128, 128, 4); break;
      case 8: MARS_LM_RING(128, 256, 3); break;
      default: MARS_LM_RING(256, 128, 3); break;
    }
#undef MARS_LM_RING
#undef MARS_LM_LAUNCH
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    clear.nwords = 0; clear.nstatus = 0;
  }
  return hipSuccess;
}

struct LmLayout {
  LmPlan plan;
  int G;  // work-groups per request of the sampling walk
  size_t partials_off, stats_off, xslots_off, total;
};
static LmLayout lm_layout(int B, int N, int V, int H, int K, bool sampling) {
  LmLayout L;
  const long rows = static_cast<long>(B) * N;
  L.plan = lm_plan(rows, N, V, H, sampling);
  L.partials_off = 0;
  L.stats_off = align_up(static_cast<size_t>(rows) * L.plan.parts * sizeof(Partial));
  L.G = choose_groups(K * B, V);
  L.xslots_off = L.stats_off + align_up(static_cast<size_t>(K) * rows * sizeof(mars_row_stat));
  L.total = L.xslots_off + align_up(static_cast<size_t>(K) * B * (N + 2) * 2 * L.G * sizeof(unsigned long long));
  return L;
}

// Scratch of mars_verify_static: one copy per GPU, held from the moment the library is loaded on it
// until the process ends.  In host code the array's name is only a handle for the symbol lookup
// below; kernels are given the device address the lookup returns.
static __device__ __align__(256) unsigned char scratch[MARS_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on every GPU seen so far
static std::mutex g_scratch_lock;

// Device address of the current GPU's copy of `scratch` (looked up once per GPU), nullptr on failure.
static void* static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

// Whether all rows begin on 16-byte boundaries.
static bool even_rows(const void* logits, size_t elt, int V) {
  return reinterpret_cast<uintptr_t>(logits) % 16 == 0 && static_cast<size_t>(V) * elt % 16 == 0;
}
static void launch_greedy_tail(const TailArgs& a, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned int>(a.B));
  if (a.N > kWave) hipLaunchKernelGGL(tail_greedy_kernel, grid, dim3(kGreedyThreads), 0, stream, a);
  else if (a.splits > kLaneParts) hipLaunchKernelGGL(tail_greedy_wave_kernel<kGreedyThreads>, grid, dim3(kGreedyThreads), 0, stream, a);
  else hipLaunchKernelGGL(tail_greedy_wave_kernel<kWave>, grid, dim3(kWave), 0, stream, a);
}
static hipError_t launch_onehot_tail(const TailArgs& a, int logits_dtype, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned int>(a.B));
  const bool even = even_rows(a.logits, logits_dtype == MARS_BF16 ? 2 : 4, a.V), row = !a.table;
#define MARS_ONEHOT(T, ROW, NT)                                                                                                \
  if (even) hipLaunchKernelGGL((tail_onehot_kernel<T, false, ROW, NT>), grid, dim3(NT), 0, stream, a);                          \
  else hipLaunchKernelGGL((tail_onehot_kernel<T, true, ROW, NT>), grid, dim3(NT), 0, stream, a)
#define MARS_ONEHOT_ROWS(T)                                                                                                    \
  if (row && a.V <= row_entries(kOneHotThreads)) { MARS_ONEHOT(T, true, kOneHotThreads); }                              \
  else if (row) { MARS_ONEHOT(T, true, 2 * kOneHotThreads); }                                                           \
  else { MARS_ONEHOT(T, false, kOneHotThreads); }
  if (logits_dtype == MARS_BF16) { MARS_ONEHOT_ROWS(bf16_t) }
  else { MARS_ONEHOT_ROWS(float) }
#undef MARS_ONEHOT_ROWS
#undef MARS_ONEHOT
  return hipGetLastError();
}
// The sampling walk: G work-groups per request (a.G), a.B requests.  draft_dtype < 0: one-hot.
static hipError_t launch_sampling_tail(const TailArgs& a, int logits_dtype, int draft_dtype, hipStream_t stream) {
  const int V = a.V;
  if (a.onehot) return launch_onehot_tail(a, logits_dtype, stream);
  const bool dense = draft_dtype >= 0;
  const bool vec = whole_groups(a.logits, logits_dtype == MARS_BF16 ? 2 : 4, dense ? a.dprobs : nullptr, a.N, V);
  // Slices of at most kMaxResident groups of eight per thread stay in registers between passes.  One per thread in the
  // form for rows at every alignment only (rows of up to 4 089 entries): see tail_sampling_body.
  const int slice8 = walk_slice(V, a.G, vec);
  const bool resident = slice8 <= kMaxResident * kSamplingThreads, two = slice8 <= 2 * kSamplingThreads;
  const bool one = !vec && slice8 <= kSamplingThreads;
  const bool qbf = dense && draft_dtype == MARS_BF16;
  const bool lanes = a.N <= kWave;
  const void* kernel;
#define MARS_PICK3(TT, QQ, VV, LL)                                                                            \
  (one        ? reinterpret_cast<const void*>(&tail_sampling_resident_kernel<TT, QQ, VV ? 2 : 1, VV, LL>)       \
   : two      ? reinterpret_cast<const void*>(&tail_sampling_resident_kernel<TT, QQ, 2, VV, LL>)                 \
   : resident ? reinterpret_cast<const void*>(&tail_sampling_resident_kernel<TT, QQ, kMaxResident, VV, LL>)      \
              : reinterpret_cast<const void*>(&tail_sampling_streamed_kernel<TT, QQ, VV, LL>))
#define MARS_PICK2(TT, QQ, VV) (lanes ? MARS_PICK3(TT, QQ, VV, true) : MARS_PICK3(TT, QQ, VV, false))
#define MARS_PICK(TT, QQ) (vec ? MARS_PICK2(TT, QQ, true) : MARS_PICK2(TT, QQ, false))
  if (logits_dtype == MARS_BF16) kernel = qbf ? MARS_PICK(bf16_t, bf16_t) : MARS_PICK(bf16_t, float);
  else kernel = qbf ? MARS_PICK(float, bf16_t) : MARS_PICK(float, float);
#undef MARS_PICK
#undef MARS_PICK2
#undef MARS_PICK3
  TailArgs copy = a;
  copy.slice = slice8;
  void* params[] = {&copy};
  // With G > 1 the work-groups of a request exchange sums.  The grid never exceeds one work-group
  // per compute unit, so on a GPU that is free to run it all of them are resident together and the
  // exchanges take a couple of microseconds; when other work keeps some of them waiting for a
  // compute unit, those that run work out the missing sums themselves (tail.h: exchange_begin) --
  // slower, same bits, and no work-group ever depends on another one being there.
  // (Several work-groups per request: one column of the grid each, so that neither number has to be divided for; they are at
  // most as many as compute units.  One: the requests alone, as many as there are.)
  const unsigned int B = static_cast<unsigned int>(a.B), G = static_cast<unsigned int>(a.G);
  return hipLaunchKernel(kernel, G == 1 ? dim3(B) : dim3(G, B), dim3(resident ? kSamplingThreads : kStreamingThreads), params, 0, stream);
}

// Work-groups per request at launch: what the workspace was laid out for, fewer on a GPU with fewer compute units.
static int launch_groups(int G, int KB) {
  if (static_cast<long>(KB) * G > compute_units()) {
    G = compute_units() / KB;
    if (G < 1) G = 1;
  }
  return G;
}

// How the walk of one-hot draft distributions goes: of trees that a wave can hold with a node per lane (onehot.h), reading the row it draws
// from where that is one page, or the sums of the row's chunks; else by work-groups that go over the row (tail.h).
// The lines were measured with 1-250 requests of 6, 12, 26 and 60 nodes (us per call of tail.h / onehot.h):
//  * A page: bf16 always (33 x 12 nodes x 20 000 entries 17.2 / 16.0, 10 x 60 x 32 000 23.6 / 21.6; the median is 0.95 times the time, the
//    worst of 220 shapes 20 x 60 x 20 001, 1.12). fp32 rows of 20 000 entries and more (80 KB) are read as quickly by three or more work-groups: 4 x 12
//    x 28 000 14.2 / 15.6, 64 x 6 x 24 008 18.9 / 19.5; by two 100 x 6 x 28 000 26.6 / 23.7, 170 x 12 x 24 008 48 / 44; below 20 000 entries 1 x 60 x 16 377 16.1 /
//    14.1, 16 x 26 x 12 000 18.2 / 15.5.
//  * By chunks: where a work-group's slice of the row does not fit its registers.  (What is kept there is read once, and the chunks
//    cost the row reduction and the walk a table.)  64 x 6 x 49 152 (slices of 12 288 entries) 20.0 / 21.6, 85 x 6 x 49 152 (16 384) 24.4 / 22.5; 25 x 6 x
//    120 000 (12 000) 21.8 / 23.5, 32 x 6 x 120 000 (15 000) 24.8 / 23.7; 128 x 6 x 151 936 fp32 96 / 84.  One tree of 60 x 151 936: fp32 3 % slower by
//    chunks, bf16 even over twelve inputs (18.0 / 17.7 on one, 18.9 / 21.2 where rejected tokens held much of their rows).
//  * Rows of bf16 off a 16-byte boundary, which a draw by chunks is longest at: slices of 30 000 entries.  85 x 6 x 74 001 (24 667) 31.0 / 34.4, 64 x 6
//    x 69 231 (17 308) 26.0 / 27.7; 128 x 6 x 65 537 (32 769) 35.6 / 33.3, 64 x 26 x 128 257 (32 065) 87 / 84.  Of 12 288 as the others where four thresholds and
//    more share the row reduction's sums: 5 x 60 x 100 001 with seven 33.1 / 29.0, 12 x 26 x 69 231 32 / 28; with two even.
//  * Few rows with more partial results than a lane merges, which every work-group would merge: by chunks.  One chain of 6 x 151 936 16.2 / 15.1, x 100 001
//    16.4 / 15.7; of 12 even.
enum OneHotForm { kOverTheRow, kByPage, kByChunks };
constexpr int kWidePageF32 = 20000;     // entries
constexpr int kWidePageGroups = 3;
constexpr int kMinRaggedSlice = 30000 / 8;  // groups of eight
constexpr int kSharingThetas = 4;
static OneHotForm onehot_form(const void* logits, int dtype, int B, int N, int V, int K, const Layout& L, const ChunkSpec& chunks, size_t workspace_bytes) {
  if (N > kOneHotNodes) return kOverTheRow;
  const size_t elt = dtype == MARS_BF16 ? 2 : 4;
  if (V <= row_entries(2 * kOneHotThreads))
    return dtype == MARS_BF16 || V < kWidePageF32 || L.G < kWidePageGroups ? kByPage : kOverTheRow;
  if (chunks.slots == 0 || workspace_bytes < L.total) return kOverTheRow;
  const int slice = walk_slice(V, launch_groups(L.G, K * B), whole_groups(logits, elt, nullptr, N, V));
  const bool streamed = slice > kMaxResident * kSamplingThreads;
  const bool quick = dtype == MARS_F32 || even_rows(logits, elt, V) || slice >= kMinRaggedSlice || K >= kSharingThetas;
  return L.splits > kLaneParts || (streamed && quick) ? kByChunks : kOverTheRow;
}

static hipError_t launch_keep(int K, const int32_t* out_len, const int32_t* path, int B, int N, int32_t* keep_rows,
                              int32_t* keep_offsets, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned int>(K)), block(kKeepThreads);
  if (N > 1)
    hipLaunchKernelGGL(compact_keep_kernel<kKeepAhead>, grid, block, 0, stream, out_len, path, B, N, keep_rows, keep_offsets);
  else
    hipLaunchKernelGGL(compact_keep_kernel<0>, grid, block, 0, stream, out_len, path, B, N, keep_rows, keep_offsets);
  return hipGetLastError();
}

static bool lm_sizes_ok(int B, int N, int V, int H, int K) {
  return sizes_ok(B, N, V, K) && H >= kLmBK * kLmDepth && H % (kLmBK * kLmDepth) == 0 && static_cast<long>(B) * N <= (1L << 22);
}

}  // namespace mars

extern "C" {

int mars_version(void) { return 200; }  // 0.2.0: mars_lmhead_verify

const char* mars_status_string(int status) {
  switch (status) {
    case MARS_OK: return "ok";
    case MARS_ERR_ARG: return "invalid argument";
    case MARS_ERR_DTYPE: return "unknown element type";
    case MARS_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case MARS_ERR_HIP: return "HIP call failed";
    case MARS_ERR_SCRATCH: return "sizes need more scratch memory than mars_verify_static holds";
    default: return "unknown status";
  }
}

size_t mars_workspace_bytes(int B, int N, int V) {
  if (!mars::sizes_ok(B, N, V)) return 0;
  return mars::layout(B, N, V).total;
}

int mars_row_reduce(const void* logits, int logits_dtype, float temperature, int B, int N, int V, void* workspace,
                    size_t workspace_bytes, void* hip_stream) {
  using namespace mars;
  if (!logits) return MARS_ERR_ARG;
  if (!sizes_ok(B, N, V)) return MARS_ERR_ARG;
  if (!(temperature >= 0.0f) || std::isinf(temperature)) return MARS_ERR_ARG;
  if (logits_dtype != MARS_F32 && logits_dtype != MARS_BF16) return MARS_ERR_DTYPE;
  const Layout L = layout(B, N, V);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0 || workspace_bytes < L.least)
    return MARS_ERR_WORKSPACE;
  Partial* partials = reinterpret_cast<Partial*>(static_cast<char*>(workspace) + L.partials_off);
  const hipError_t e = launch_row_reduce(logits, logits_dtype, static_cast<long>(B) * N, V, L.splits,
                                         temperature > 0.0f, log2e_over_t(temperature), partials,
                                         clear_args(static_cast<char*>(workspace), L, B, N, 1),
                                         static_cast<hipStream_t>(hip_stream));
  return e == hipSuccess ? MARS_OK : MARS_ERR_HIP;
}

int mars_row_stats(const void* logits, int logits_dtype, const float* theta, float temperature, int B, int N, int V,
                   mars_row_stat* stats, void* workspace, size_t workspace_bytes, void* hip_stream) {
  using namespace mars;
  if (!logits || !theta || !stats) return MARS_ERR_ARG;
  if (!sizes_ok(B, N, V)) return MARS_ERR_ARG;
  if (!(temperature >= 0.0f) || std::isinf(temperature)) return MARS_ERR_ARG;
  if (logits_dtype != MARS_F32 && logits_dtype != MARS_BF16) return MARS_ERR_DTYPE;
  const Layout L = layout(B, N, V);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0 || workspace_bytes < L.least)
    return MARS_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const long rows = static_cast<long>(B) * N;
  Partial* partials = reinterpret_cast<Partial*>(static_cast<char*>(workspace) + L.partials_off);
  const float c = log2e_over_t(temperature);
  if (launch_row_reduce(logits, logits_dtype, rows, V, L.splits, temperature > 0.0f, c, partials,
                        clear_args(static_cast<char*>(workspace), L, B, N, 1), stream) != hipSuccess)
    return MARS_ERR_HIP;
  const int threads = 256, rows_per_group = 16;
  const Indicator ind = {MARS_IND_LOGIT_RATIO, indicator_scale(temperature)};
  hipLaunchKernelGGL(merge_stats_kernel, dim3(static_cast<unsigned int>((rows + rows_per_group - 1) / rows_per_group)),
                     dim3(threads), 0, stream, partials, static_cast<int>(rows), N, L.splits * kPartsPerItem, theta, c,
                     ind, stats);
  return hipGetLastError() == hipSuccess ? MARS_OK : MARS_ERR_HIP;
}

size_t mars_workspace_bytes_ex(int B, int N, int V, int n_theta) {
  if (!mars::sizes_ok(B, N, V, n_theta)) return 0;
  return mars::layout(B, N, V, n_theta).total;
}

int mars_verify(const void* logits, int logits_dtype, const int32_t* draft_tokens, const int32_t* tree_parent,
                const void* draft_probs, int draft_dtype, const float* theta, float temperature,
                const float* uniforms, int B, int N, int V, uint8_t* accept_mask, int32_t* accept_len,
                int32_t* path_idx, int32_t* bonus_token, uint8_t* decision, int32_t* request_status,
                mars_row_stat* stats, mars_req_diag* diag, void* workspace, size_t workspace_bytes,
                void* hip_stream) {
  return mars_verify_ex(logits, logits_dtype, draft_tokens, tree_parent, draft_probs, draft_dtype, theta, temperature,
                        uniforms, B, N, V, accept_mask, accept_len, path_idx, bonus_token, decision, request_status,
                        stats, diag, workspace, workspace_bytes, hip_stream, nullptr);
}

int mars_verify_ex(const void* logits, int logits_dtype, const int32_t* draft_tokens, const int32_t* tree_parent,
                   const void* draft_probs, int draft_dtype, const float* theta, float temperature,
                   const float* uniforms, int B, int N, int V, uint8_t* accept_mask, int32_t* accept_len,
                   int32_t* path_idx, int32_t* bonus_token, uint8_t* decision, int32_t* request_status,
                   mars_row_stat* stats, mars_req_diag* diag, void* workspace, size_t workspace_bytes,
                   void* hip_stream, const mars_verify_options* options) {
  using namespace mars;
  if (!logits || !draft_tokens || !tree_parent || !theta || !accept_mask || !accept_len || !path_idx || !bonus_token)
    return MARS_ERR_ARG;
  int K = 1, indicator = MARS_IND_LOGIT_RATIO, spin_limit = 0, stages = MARS_STAGE_ROWS | MARS_STAGE_REQUESTS;
  int32_t *out_tokens = nullptr, *out_len = nullptr, *keep_rows = nullptr, *keep_offsets = nullptr;
  if (options) {
    K = options->n_theta == 0 ? 1 : options->n_theta;
    indicator = options->indicator;
    spin_limit = options->spin_limit;
    if (spin_limit < 0 || options->stages < 0 || options->stages > 3) return MARS_ERR_ARG;
    if (options->stages != 0) stages = options->stages;
    out_tokens = options->out_tokens; out_len = options->out_len;
    keep_rows = options->keep_rows; keep_offsets = options->keep_offsets;
  }
  if (indicator != MARS_IND_LOGIT_RATIO && indicator != MARS_IND_PROB_RATIO && indicator != MARS_IND_LOGIT_GAP)
    return MARS_ERR_ARG;
  const int given = (out_tokens != nullptr) + (out_len != nullptr) + (keep_rows != nullptr) + (keep_offsets != nullptr);
  if (given != 0 && given != 4) return MARS_ERR_ARG;
  if (!sizes_ok(B, N, V, K)) return MARS_ERR_ARG;
  if (!(temperature >= 0.0f) || std::isinf(temperature)) return MARS_ERR_ARG;
  const bool sampling = temperature > 0.0f;
  if (sampling && !uniforms) return MARS_ERR_ARG;
  if (logits_dtype != MARS_F32 && logits_dtype != MARS_BF16) return MARS_ERR_DTYPE;
  const bool dense = sampling && draft_probs != nullptr;
  if (dense && draft_dtype != MARS_F32 && draft_dtype != MARS_BF16) return MARS_ERR_DTYPE;
  const Layout L = layout(B, N, V, K);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0 || workspace_bytes < L.least)
    return MARS_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const long rows = static_cast<long>(B) * N;
  char* ws = static_cast<char*>(workspace);
  Partial* partials = reinterpret_cast<Partial*>(ws + L.partials_off);
  const float c = log2e_over_t(temperature);

  ClearArgs clr = clear_args(ws, L, B, N, K);
  if (sampling) {  // the sampling walk starts from what the row reduction gathers for it
    clr.par = tree_parent; clr.tok = draft_tokens;
    clr.q = dense ? draft_probs : nullptr;
    clr.q_bf16 = draft_dtype == MARS_BF16 ? 1 : 0;
    clr.gathered = reinterpret_cast<float2*>(ws + L.gathered_off);
  }
  const ChunkSpec chunks = row_chunks(V, logits_dtype == MARS_BF16 ? 2 : 4, L.splits);
  const OneHotForm form =
      sampling && !dense ? onehot_form(logits, logits_dtype, B, N, V, K, L, chunks, workspace_bytes) : kOverTheRow;
  const bool onehot = form != kOverTheRow;
  if (onehot) clr.xwords = 0;  // (one work-group per request: nothing is exchanged)
  if (form == kByChunks) {
    clr.slots = chunks.slots; clr.batches = 1 << chunks.log2_batches;
    clr.table = reinterpret_cast<float2*>(ws + L.table_off);
    clr.table_low = reinterpret_cast<float*>(ws + L.low_off);
  }
  if (sampling && request_status) {  // the sampling tail only raises a request's status
    clr.counters = reinterpret_cast<unsigned int*>(request_status);
    clr.ncounters = static_cast<long>(K) * B;
  }
  if ((stages & MARS_STAGE_ROWS) &&
      launch_row_reduce(logits, logits_dtype, rows, V, L.splits, sampling, c, partials, clr, stream) != hipSuccess)
    return MARS_ERR_HIP;
  if (!(stages & MARS_STAGE_REQUESTS)) return MARS_OK;

  TailArgs a;
  a.logits = logits; a.tok = draft_tokens; a.par = tree_parent;
  a.dprobs = dense ? draft_probs : nullptr;
  a.theta = theta; a.u = uniforms; a.partials = partials;
  a.stats = stats;
  a.gathered = reinterpret_cast<const float2*>(ws + L.gathered_off);
  a.G = sampling ? launch_groups(L.G, K * B) : 1;
  // polls (about a microsecond each) a work-group gives a partner before it works out the partner's sum itself
  a.spin_limit = spin_limit > 0 ? spin_limit : kDefaultSpinLimit;
  a.xslots = clr.xslots;
  a.mask = accept_mask; a.len = accept_len; a.path = path_idx; a.bonus = bonus_token;
  a.dec = decision; a.status = request_status; a.diag = diag;
  a.chunks = chunks; a.table = clr.table; a.table_low = clr.table_low;
  a.onehot = onehot;
  a.B = K * B; a.Bd = B; a.N = N; a.V = V; a.splits = L.splits * kPartsPerItem; a.c = c;
  a.ind.kind = indicator; a.ind.cind = indicator_scale(temperature);
  a.out_tok = out_tokens; a.out_len = out_len;

  // The cache rows that stay: a small kernel behind the walk (one work-group per threshold).
  auto finish = [&]() -> int {
    if (hipGetLastError() != hipSuccess) return MARS_ERR_HIP;
    if (!keep_rows) return MARS_OK;
    return launch_keep(K, out_len, path_idx, B, N, keep_rows, keep_offsets, stream) == hipSuccess ? MARS_OK : MARS_ERR_HIP;
  };

  if (!sampling) {
    launch_greedy_tail(a, stream);
    return finish();
  }
  if (launch_sampling_tail(a, logits_dtype, dense ? draft_dtype : -1, stream) != hipSuccess) return MARS_ERR_HIP;
  return finish();
}

int mars_verify_static(const void* logits, int logits_dtype, const int32_t* draft_tokens, const int32_t* tree_parent,
                       const void* draft_probs, int draft_dtype, const float* theta, float temperature,
                       const float* uniforms, int B, int N, int V, uint8_t* accept_mask, int32_t* accept_len,
                       int32_t* path_idx, int32_t* bonus_token, uint8_t* decision, int32_t* request_status,
                       mars_row_stat* stats, mars_req_diag* diag, void* hip_stream,
                       const mars_verify_options* options) {
  using namespace mars;
  const int K = options && options->n_theta != 0 ? options->n_theta : 1;
  if (!sizes_ok(B, N, V, K)) return MARS_ERR_ARG;
  if (layout(B, N, V, K).least > static_cast<size_t>(MARS_STATIC_SCRATCH_BYTES)) return MARS_ERR_SCRATCH;
  void* ws = static_scratch();
  if (!ws) return MARS_ERR_HIP;
  return mars_verify_ex(logits, logits_dtype, draft_tokens, tree_parent, draft_probs, draft_dtype, theta, temperature,
                        uniforms, B, N, V, accept_mask, accept_len, path_idx, bonus_token, decision, request_status,
                        stats, diag, ws, MARS_STATIC_SCRATCH_BYTES, hip_stream, options);
}

int mars_margin_stats(const void* logits, int logits_dtype, const float* theta, float temperature, int B, int N, int V,
                      const float* range, const int32_t* bins, mars_margin_row* rows_out, uint32_t* counts,
                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  using namespace mars;
  if (!logits || !theta || !range || !bins || !counts) return MARS_ERR_ARG;
  if (!sizes_ok(B, N, V)) return MARS_ERR_ARG;
  if (!(temperature >= 0.0f) || std::isinf(temperature)) return MARS_ERR_ARG;
  if (logits_dtype != MARS_F32 && logits_dtype != MARS_BF16) return MARS_ERR_DTYPE;
  HistSpec hs;
  long ncounters = 4;
  for (int h = 0; h < 3; ++h) {
    const float lo = range[2 * h], hi = range[2 * h + 1];
    if (!(lo < hi) || std::isinf(lo) || std::isinf(hi) || bins[h] < 1 || bins[h] > (1 << 20)) return MARS_ERR_ARG;
    hs.lo[h] = lo; hs.hi[h] = hi; hs.bins[h] = bins[h];
    hs.w[h] = static_cast<float>(static_cast<double>(bins[h]) / (static_cast<double>(hi) - static_cast<double>(lo)));
    ncounters += bins[h] + 2;
  }
  if (ncounters > (1 << 20)) return MARS_ERR_ARG;
  const Layout L = layout(B, N, V);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0 || workspace_bytes < L.least)
    return MARS_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const long rows = static_cast<long>(B) * N;
  char* ws = static_cast<char*>(workspace);
  Partial* partials = reinterpret_cast<Partial*>(ws + L.partials_off);
  // The top-2 alone: the greedy form of the row reduction (no sum-exp); it also clears the counters.
  ClearArgs clr = clear_args(ws, L, B, N, 1);
  clr.counters = counts; clr.ncounters = ncounters;
  if (launch_row_reduce(logits, logits_dtype, rows, V, L.splits, false, 0.0f, partials, clr, stream) != hipSuccess)
    return MARS_ERR_HIP;
  const bool local = count_in_lds(rows, ncounters);
  const dim3 grid(static_cast<unsigned int>((rows + hist_rows(local) - 1) / hist_rows(local))), block(kHistThreads);
  if (local)
    hipLaunchKernelGGL(margin_stats_kernel<true>, grid, block, 0, stream, partials, static_cast<int>(rows), N,
                       L.splits * kPartsPerItem, theta, indicator_scale(temperature), hs, rows_out, counts);
  else
    hipLaunchKernelGGL(margin_stats_kernel<false>, grid, block, 0, stream, partials, static_cast<int>(rows), N,
                       L.splits * kPartsPerItem, theta, indicator_scale(temperature), hs, rows_out, counts);
  return hipGetLastError() == hipSuccess ? MARS_OK : MARS_ERR_HIP;
}

size_t mars_lmhead_workspace_bytes(int B, int N, int V, int H, int n_theta) {
  const int K = n_theta == 0 ? 1 : n_theta;
  if (!mars::lm_sizes_ok(B, N, V, H, K)) return 0;
  const size_t greedy = mars::lm_layout(B, N, V, H, K, false).total, sampling = mars::lm_layout(B, N, V, H, K, true).total;
  return greedy > sampling ? greedy : sampling;
}

int mars_lmhead_verify(const void* hidden, const void* weight, int H, const int32_t* draft_tokens,
                       const int32_t* tree_parent, const float* theta, int B, int N, int V, uint8_t* accept_mask,
                       int32_t* accept_len, int32_t* path_idx, int32_t* bonus_token, uint8_t* decision,
                       int32_t* request_status, mars_row_stat* stats, void* workspace, size_t workspace_bytes,
                       void* hip_stream, const mars_verify_options* options) {
  using namespace mars;
  if (!hidden || !weight || !draft_tokens || !tree_parent || !theta || !accept_mask || !accept_len || !path_idx ||
      !bonus_token)
    return MARS_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(hidden) % 16 != 0 || reinterpret_cast<uintptr_t>(weight) % 16 != 0)
    return MARS_ERR_ARG;
  int K = 1, indicator = MARS_IND_LOGIT_RATIO, lm_stages = MARS_STAGE_ROWS | MARS_STAGE_REQUESTS;
  int32_t *out_tokens = nullptr, *out_len = nullptr, *keep_rows = nullptr, *keep_offsets = nullptr;
  if (options) {
    K = options->n_theta == 0 ? 1 : options->n_theta;
    indicator = options->indicator;
    if (options->spin_limit < 0 || options->stages < 0 || options->stages > 3) return MARS_ERR_ARG;
    if (options->stages != 0) lm_stages = options->stages;
    out_tokens = options->out_tokens; out_len = options->out_len;
    keep_rows = options->keep_rows; keep_offsets = options->keep_offsets;
  }
  if (indicator != MARS_IND_LOGIT_RATIO && indicator != MARS_IND_PROB_RATIO && indicator != MARS_IND_LOGIT_GAP)
    return MARS_ERR_ARG;
  const int given = (out_tokens != nullptr) + (out_len != nullptr) + (keep_rows != nullptr) + (keep_offsets != nullptr);
  if (given != 0 && given != 4) return MARS_ERR_ARG;
  if (!lm_sizes_ok(B, N, V, H, K)) return MARS_ERR_ARG;
  const LmLayout L = lm_layout(B, N, V, H, K, false);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0 || workspace_bytes < L.total)
    return MARS_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const int rows = B * N;
  char* ws = static_cast<char*>(workspace);
  Partial* partials = reinterpret_cast<Partial*>(ws + L.partials_off);
  const LmPlan& p = L.plan;

  if ((lm_stages & MARS_STAGE_ROWS) &&
      launch_lmhead<false>(p, static_cast<const bf16_t*>(hidden), static_cast<const bf16_t*>(weight), rows, V, H, partials,
                           nullptr, 0.0f, LmClear{nullptr, 0, nullptr, 0}, stream) != hipSuccess)
    return MARS_ERR_HIP;
  if (!(lm_stages & MARS_STAGE_REQUESTS)) return MARS_OK;

  TailArgs a;
  a.logits = nullptr; a.tok = draft_tokens; a.par = tree_parent; a.dprobs = nullptr; a.onehot = false;
  a.theta = theta; a.u = nullptr; a.partials = partials;
  a.stats = stats;
  a.G = 1; a.spin_limit = 0; a.xslots = nullptr; a.gathered = nullptr; a.table = nullptr;
  a.mask = accept_mask; a.len = accept_len; a.path = path_idx; a.bonus = bonus_token;
  a.dec = decision; a.status = request_status; a.diag = nullptr;
  a.B = K * B; a.Bd = B; a.N = N; a.V = V; a.splits = p.parts; a.c = 0.0f;
  a.ind.kind = indicator; a.ind.cind = indicator_scale(0.0f);
  a.out_tok = out_tokens; a.out_len = out_len;
  launch_greedy_tail(a, stream);
  if (hipGetLastError() != hipSuccess) return MARS_ERR_HIP;
  if (!keep_rows) return MARS_OK;
  return launch_keep(K, out_len, path_idx, B, N, keep_rows, keep_offsets, stream) == hipSuccess ? MARS_OK : MARS_ERR_HIP;
}

int mars_lmhead_verify_sampling(const void* hidden, const void* weight, int H, const int32_t* draft_tokens,
                                const int32_t* tree_parent, const void* draft_probs, int draft_dtype,
                                const float* theta, float temperature, const float* uniforms, int B, int N, int V,
                                void* logits_out, uint8_t* accept_mask, int32_t* accept_len, int32_t* path_idx,
                                int32_t* bonus_token, uint8_t* decision, int32_t* request_status,
                                mars_row_stat* stats, mars_req_diag* diag, void* workspace, size_t workspace_bytes,
                                void* hip_stream, const mars_verify_options* options) {
  using namespace mars;
  if (!hidden || !weight || !draft_tokens || !tree_parent || !theta || !uniforms || !logits_out || !accept_mask ||
      !accept_len || !path_idx || !bonus_token)
    return MARS_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(hidden) % 16 != 0 || reinterpret_cast<uintptr_t>(weight) % 16 != 0 ||
      reinterpret_cast<uintptr_t>(logits_out) % 16 != 0 || V % 8 != 0)
    return MARS_ERR_ARG;
  if (!(temperature > 0.0f) || std::isinf(temperature)) return MARS_ERR_ARG;
  const bool dense = draft_probs != nullptr;
  if (dense && draft_dtype != MARS_F32 && draft_dtype != MARS_BF16) return MARS_ERR_DTYPE;
  int K = 1, indicator = MARS_IND_LOGIT_RATIO, spin_limit = 0, lm_stages = MARS_STAGE_ROWS | MARS_STAGE_REQUESTS;
  int32_t *out_tokens = nullptr, *out_len = nullptr, *keep_rows = nullptr, *keep_offsets = nullptr;
  if (options) {
    K = options->n_theta == 0 ? 1 : options->n_theta;
    indicator = options->indicator;
    spin_limit = options->spin_limit;
    if (spin_limit < 0 || options->stages < 0 || options->stages > 3) return MARS_ERR_ARG;
    if (options->stages != 0) lm_stages = options->stages;
    out_tokens = options->out_tokens; out_len = options->out_len;
    keep_rows = options->keep_rows; keep_offsets = options->keep_offsets;
  }
  if (indicator != MARS_IND_LOGIT_RATIO && indicator != MARS_IND_PROB_RATIO && indicator != MARS_IND_LOGIT_GAP)
    return MARS_ERR_ARG;
  const int given = (out_tokens != nullptr) + (out_len != nullptr) + (keep_rows != nullptr) + (keep_offsets != nullptr);
  if (given != 0 && given != 4) return MARS_ERR_ARG;
  if (!lm_sizes_ok(B, N, V, H, K)) return MARS_ERR_ARG;
  const LmLayout L = lm_layout(B, N, V, H, K, true);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kAlign != 0 || workspace_bytes < L.total)
    return MARS_ERR_WORKSPACE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const int rows = B * N;
  char* ws = static_cast<char*>(workspace);
  Partial* partials = reinterpret_cast<Partial*>(ws + L.partials_off);
  unsigned long long* xslots = reinterpret_cast<unsigned long long*>(ws + L.xslots_off);
  const LmPlan& p = L.plan;
  const float c = log2e_over_t(temperature);

  if (lm_stages & MARS_STAGE_ROWS) {
    // What the streaming row reduction clears for the walk behind it, the fused kernel does here.
    const LmClear clear = {xslots, static_cast<long>(K) * B * (N + 2) * 2 * L.G, request_status, K * B};
    if (launch_lmhead<true>(p, static_cast<const bf16_t*>(hidden), static_cast<const bf16_t*>(weight), rows, V, H, partials,
                            static_cast<bf16_t*>(logits_out), c, clear, stream) != hipSuccess)
      return MARS_ERR_HIP;
  }
  if (!(lm_stages & MARS_STAGE_REQUESTS)) return MARS_OK;

  TailArgs a;
  a.logits = logits_out; a.tok = draft_tokens; a.par = tree_parent;
  a.dprobs = dense ? draft_probs : nullptr;
  a.theta = theta; a.u = uniforms; a.partials = partials;
  a.gathered = nullptr;  // the walk gathers for itself: no streaming row reduction has run
  // (The sums that the fused kernel leaves, one per column of tiles, are fp32 sums of fp32 sums, for the row statistics; a draw is made from sums in 64 bits, so
  // it goes over the row.)
  a.chunks = {}; a.table = nullptr;
  a.onehot = !dense && N <= kOneHotNodes && V <= row_entries(2 * kOneHotThreads);
  a.stats = stats;
  a.G = launch_groups(L.G, K * B);
  a.spin_limit = spin_limit > 0 ? spin_limit : kDefaultSpinLimit;
  a.xslots = xslots;
  a.mask = accept_mask; a.len = accept_len; a.path = path_idx; a.bonus = bonus_token;
  a.dec = decision; a.status = request_status; a.diag = diag;
  a.B = K * B; a.Bd = B; a.N = N; a.V = V; a.splits = p.parts; a.c = c;
  a.ind.kind = indicator; a.ind.cind = indicator_scale(temperature);
  a.out_tok = out_tokens; a.out_len = out_len;
  if (launch_sampling_tail(a, MARS_BF16, dense ? draft_dtype : -1, stream) != hipSuccess) return MARS_ERR_HIP;
  if (hipGetLastError() != hipSuccess) return MARS_ERR_HIP;
  if (!keep_rows) return MARS_OK;
  return launch_keep(K, out_len, path_idx, B, N, keep_rows, keep_offsets, stream) == hipSuccess ? MARS_OK : MARS_ERR_HIP;
}

}  // extern "C"
