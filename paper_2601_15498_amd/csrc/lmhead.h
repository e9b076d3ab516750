// LM head fused with the row reduction (paper Eq. 2, z = W h, followed by the top-2
// identification of Sec. 3.3): the logits of a tile are formed on the matrix cores, rounded to
// bf16 in registers, reduced to each row's two largest (value desc, index asc) and dropped --
// they are never written to memory.  Output: partial results in the format of the streaming row
// reduction, so that the per-request kernels behind it are the same.
//
// The work is units of a slab of BM hidden-state rows x a tile of 256 vocabulary entries, dealt out evenly (LmCell,
// below).  Per unit a work-group walks the hidden dimension in slabs of 64: both operands are
// staged through LDS (double-buffered, one barrier per slab), four waves in a 2 x 2 arrangement
// each accumulate (BM/2) x 128 logits with v_mfma_f32_32x32x16_bf16.  The weight rows are the
// first MFMA operand and the hidden states the second, so that a lane ends up holding, for one
// hidden-state row, 16 vocabulary entries per accumulator block: the row's top-2 over the wave's
// 128 entries is taken inside the lane, a running pair per row is carried across the tiles of a
// (slab, column) cell, and the two halves of a wave and the two waves that share a row meet at its end.
//
// What bounds it: the matrix cores, the power they draw and the data moved per product.  6 656 rows x 4096 x 151 936: 6.00-6.12 ms =
// 1.35-1.38 PFLOP/s (the library's product alone 1.47; 8192^3: 1.38-1.40), the clock at 1.72 GHz of 2.4 and the matrix
// units busy 3/4 of the time; before (192 rows at most, keys in 32-bit integers, unequal shares) 6.76-6.87 ms.
// 960 rows, sampling form: 1 000 us per call (1 032 in the same run before the stores and what is kept between tiles took their
// present form, below).
//
// Few rows, or few units (a small vocabulary), are not bound by the matrix cores but by the weight's way through the chip, and take
// a second form, the ring (lmhead_ring_kernel): tiles of 64, 128 or 256 entries, so that there are enough units for
// the chip, and operands that go from memory straight to LDS (buffer_load ... lds), STAGES - 1 steps ahead of their use, without
// passing through registers.  With operands one step in LDS and one in registers a step of 64 rows took 0.77 us whatever its tile, a
// trip to memory for every two steps.  A weight that is read once and does not fit the Infinity Cache is read
// with the non-temporal hint: 6.9 TB/s instead of 6.2.  60 rows x 4096 x 151 936: bound by the weight, 1.24 GB in 178-180 us = 6.9
// TB/s (through registers 203-205), and the per-request kernel behind it; 56 x 4096 x 2 250 45 -> 22 us per call.
// Many rows, greedy, mostly stay with the first form: with 256 x 256 two stages of 64 KB are all that fits LDS, and one step of lead
// is too little (960 rows, 192 to a slab: 1 108 us against 940; rows of 64 bytes, four stages: 1 044).  Under sampling the first form
// has at most 192 rows and no epilogue to spare, and where its slabs do not come out even the ring's 128 x 256 and 256 x 128 serve many rows
// too: 512 or 1 024 x 4096 x 151 936, a third of all sizes between 257 and 2 048 rows (which: lm_plan).
#pragma once

#include <type_traits>

#include "common.h"

namespace mars {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kLmThreads = 256;           // 4 waves: 2 (hidden rows) x 2 (vocabulary)
constexpr int kLmBN = 256;                // vocabulary entries per tile
constexpr int kLmBK = 64;                 // hidden-state elements per staged slab
constexpr int kLmStride = kLmBK + 8;      // LDS row stride in elements: 144 bytes, conflict-free 16-byte reads
constexpr int kLmChunks = kLmBK / 8;      // 16-byte chunks per staged row
constexpr int kLmDepth = 2;               // steps between the request of an operand slab and its use
constexpr int kLmMaxBM = 256;             // tallest slab of hidden-state rows (its accumulators are half the register file)

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// Two bf16 patterns (sign and magnitude) as two 16-bit integers in the order of the values: minus the magnitude
// where the sign is set, so that both zeros are one value.
typedef short i16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t lm_ordered_pair(uint32_t w) {
  const i16x2_t m = __builtin_bit_cast(i16x2_t, w) >> 15;
  const i16x2_t mag = __builtin_bit_cast(i16x2_t, (w & 0x7FFF7FFFu) ^ __builtin_bit_cast(uint32_t, m));
  return __builtin_bit_cast(uint32_t, mag - m);
}
// The bf16 value in the upper half of a key, widened.
__device__ __forceinline__ float lm_key_value(int key) {
  const int v = key >> 16;
  return __uint_as_float((v < 0 ? 0x8000u - static_cast<uint32_t>(v) : static_cast<uint32_t>(v)) << 16);
}
// Eight accumulators, read where this stands.  (Read by name, the compiler collects the reads of both forms of the
// epilogue in front of it, 256 registers at once, and spills.  The hardware does not wait for a matrix
// instruction's result here: lm_results_ready() stands between the last of them and the first read.)
template <int FIRST>
__device__ __forceinline__ void lm_acc8(const f32x16_t& block, float (&x)[8]) {
  asm volatile(
      "v_accvgpr_read_b32 %0, %8\n\tv_accvgpr_read_b32 %1, %9\n\tv_accvgpr_read_b32 %2, %10\n\t"
      "v_accvgpr_read_b32 %3, %11\n\tv_accvgpr_read_b32 %4, %12\n\tv_accvgpr_read_b32 %5, %13\n\t"
      "v_accvgpr_read_b32 %6, %14\n\tv_accvgpr_read_b32 %7, %15"
      : "=v"(x[0]), "=v"(x[1]), "=v"(x[2]), "=v"(x[3]), "=v"(x[4]), "=v"(x[5]), "=v"(x[6]), "=v"(x[7])
      : "a"(block[FIRST]), "a"(block[FIRST + 1]), "a"(block[FIRST + 2]), "a"(block[FIRST + 3]), "a"(block[FIRST + 4]),
        "a"(block[FIRST + 5]), "a"(block[FIRST + 6]), "a"(block[FIRST + 7]));
}
// Sixteen of them, rounded to bf16 in pairs.
template <bool BY_ASM>
__device__ __forceinline__ void lm_rounded(const f32x16_t& block, uint32_t (&w)[8]) {
  if constexpr (!BY_ASM) {
#pragma unroll
    for (int p = 0; p < 8; ++p)
      w[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{block[2 * p], block[2 * p + 1]}, bf16x2_t));
    return;
  }
  float x[8];
  lm_acc8<0>(block, x);
#pragma unroll
  for (int p = 0; p < 4; ++p) w[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{x[2 * p], x[2 * p + 1]}, bf16x2_t));
  lm_acc8<8>(block, x);
#pragma unroll
  for (int p = 0; p < 4; ++p) w[4 + p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{x[2 * p], x[2 * p + 1]}, bf16x2_t));
}
__device__ __forceinline__ void lm_results_ready() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // 32 wait states; an instruction of 16 passes asks for 19
  __builtin_amdgcn_sched_barrier(0);
}
// A block of 32 rows x 32 logits on its way out.  Lane l has words 2q, 2q + 1 = entries 8q + 4 (l/32) .. + 3 of row l%32, q = 0 .. 3;
// it leaves with 16 bytes, entries 8k .. 8k + 7, of rows l%16 and l%16 + 16, k = (l/16)%2 + 2 (l/32): 64 bytes of a row per
// store, by exchanges of half-waves and of quarter-waves between registers.  (960 rows x 4096 x 151 936, sampling form, us per call: 8 bytes per
// lane and 16 of a row per store 1 070, 16 and 32 1 059, so 1 054, 16 and 32 with neighbouring lanes on a row 1 063; with the non-temporal hint
// 1 093, all in one run.)
__device__ __forceinline__ void lm_out_lines(const uint32_t (&w)[8], u32x4 (&line)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // first and second word of a pair of entries
    const auto even = __builtin_amdgcn_permlane32_swap(w[i], w[4 + i], false, false);     // chunk 0 | 2: entries 0-3, 4-7
    const auto odd = __builtin_amdgcn_permlane32_swap(w[2 + i], w[6 + i], false, false);  // chunk 1 | 3
    const auto front = __builtin_amdgcn_permlane16_swap(even[0], odd[0], false, false);
    const auto back = __builtin_amdgcn_permlane16_swap(even[1], odd[1], false, false);
    line[0][i] = front[0]; line[1][i] = front[1];
    line[0][2 + i] = back[0]; line[1][2 + i] = back[1];
  }
}
// k1 >= k2, the two largest so far.
__device__ __forceinline__ void lm_top2_step(int& k1, int& k2, int key) {
  k2 = max(min(k1, k2), min(max(k1, k2), key));  // the median of the three
  k1 = max(k1, key);
}

// n rows of an operand, from which a thread stages 16-byte chunks of rows first, first + 32, ...
// As a buffer, reads of rows past the end return zeros, so that the last slab and the last tile need no clamped
// row numbers (sixteen registers of them); a buffer spans less than 2^32 bytes, so a hidden size beyond 2^22 goes
// to a form of its own, with pointers and clamped row numbers.
constexpr int kLmBufferFlags = 0x00020000;  // untyped buffer, 32-bit data format
template <bool BUFFER> struct LmRows;
template <> struct LmRows<true> {
  __amdgpu_buffer_rsrc_t rows;
  unsigned int off, pitch;  // bytes: the thread's first chunk, 32 rows
  __device__ __forceinline__ LmRows(const bf16_t* base, int n, int H, int first, int chunk)
      : rows(__builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, static_cast<int>(static_cast<unsigned int>(n) * H * 2u),
                                               kLmBufferFlags)),
        off((static_cast<unsigned int>(first) * H + chunk) * 2u), pitch(64u * H) {}
  // The offsets of the pieces are formed where they are used, not kept.
  __device__ __forceinline__ void renew() { asm volatile("" : "+v"(off)); }
  __device__ __forceinline__ u32x4 load(int i, int k) const {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, static_cast<int>(off + i * pitch), k * 2, 0));
  }
  // The same 16 bytes of every lane to LDS, lane after lane from byte address `lds` on, past the registers.  (Written by hand:
  // behind the compiler's own form of this load it has every read of LDS wait for all that is in flight.  The wait states:
  // an address word can come from a vector instruction just before.)
  template <bool ONCE>
  __device__ __forceinline__ void to_lds(int i, int k, unsigned int lds) const {
    if (ONCE)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                   :: "s"(lds), "v"(off + i * pitch), "s"(rows), "s"(k * 2) : "memory", "m0");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :: "s"(lds), "v"(off + i * pitch), "s"(rows), "s"(k * 2) : "memory", "m0");
  }
};
template <> struct LmRows<false> {
  const bf16_t* base;
  int last, first, chunk;
  size_t H;
  __device__ __forceinline__ LmRows(const bf16_t* base_, int n, int H_, int first_, int chunk_)
      : base(base_), last(n - 1), first(first_), chunk(chunk_), H(H_) {}
  __device__ __forceinline__ void renew() {}
  __device__ __forceinline__ u32x4 load(int i, int k) const {
    return *reinterpret_cast<const u32x4*>(base + static_cast<size_t>(min(last, first + i * 32)) * H + chunk + k);
  }
  template <bool ONCE> __device__ __forceinline__ void to_lds(int, int, unsigned int) const {}  // (the ring's rows are buffers)
};
// What a work-group does: `width` (slab, tile) units in a row, of an order that runs through bands of a few
// slabs, in a band through columns of `width` tiles, in a column slab by slab.  A (slab, column) cell is then one
// work-group's, or the end of one and the beginning of the next one's: every work-group has the same amount of work
// whatever the numbers (the last one may have less), and those that run side by side on a die share the
// weight tiles of a column and the hidden states of a band's slabs.
// With a single band a column of full width is slabs x width units and begins where a work-group does: only the cells of
// a narrower last column can be shared.  Behind a band whose units are no multiple of `width` any can.
struct LmGrid {
  int slabs, band, tiles_n, width, units, parts;
  int split;  // first column whose cells may belong to two work-groups: from there on two partial results each
};
// Memory the sampling form clears for the walk behind it: exchange words and request status words.
struct LmClear {
  unsigned long long* words;
  long nwords;
  int32_t* status;
  int nstatus;
};
struct LmCell {
  int slab, tile, n;   // tiles tile .. tile + n - 1 of the slab
  int column;
  bool begins, ends;   // the cell's first tile is among them, its last one is
};
__device__ __forceinline__ LmCell lm_cell(int unit, int unit_end, int slabs, int band, int tiles_n, int width) {
  LmCell c;
  const int b = unit / (band * tiles_n);
  const int height = min(band, slabs - b * band);
  const int in_band = unit - b * band * tiles_n;
  c.column = in_band / (height * width);
  const int in_column = in_band - c.column * height * width;
  const int tiles = min(width, tiles_n - c.column * width);
  const int s = in_column / tiles, t = in_column - s * tiles;
  c.slab = b * band + s;
  c.tile = c.column * width + t;
  c.n = min(tiles - t, unit_end - unit);
  c.begins = t == 0;
  c.ends = t + c.n == tiles;
  return c;
}
// Where chunk `chunk` of a row stands among the row's eight places in the ring (and which chunk stands at place `chunk`:
// the same).  Sixteen rows in a row have a chunk on sixteen different groups of four banks.
__device__ __forceinline__ int lm_place(int row, int chunk) { return chunk ^ ((row >> 1) & (kLmChunks - 1)); }
__device__ __forceinline__ unsigned int lm_lds_address(const void* p) {
  return static_cast<unsigned int>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p));
}
// All but the last LEFT loads of this wave have arrived in LDS and all its reads in registers; so have the other waves'.
template <int LEFT>
__device__ __forceinline__ void lm_ring_turn() {
  static_assert(LEFT >= 0 && LEFT < 64, "the counter's range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(LEFT) : "memory");
}
template <int n>
__device__ __forceinline__ void lm_store_lds(const u32x4 (&g)[n], bf16_t* first) {
#pragma unroll
  for (int i = 0; i < n; ++i) *reinterpret_cast<u32x4*>(first + i * 32 * kLmStride) = g[i];
}

// n operand fragments (16 bytes per lane each) of rows 32 apart.
template <int n>
__device__ __forceinline__ void lm_load_frags(u32x4 (&f)[n], const bf16_t* first) {
#pragma unroll
  for (int i = 0; i < n; ++i) f[i] = *reinterpret_cast<const u32x4*>(first + i * 32 * kLmStride);
}

// SAMPLING (Eq. 2 followed by Eq. 3): the rounded logits are also written out, once, from the registers
// they are formed in (the residual passes of the sampling walk read rows of them again), and each row's
// sum of exp2(z*c - ref) is taken on the way, against an integer-valued reference per row that moves up with
// the row's running maximum -- the same (reference, sum) pairs the streaming row reduction leaves.
// parts: partial results per row -- one per column, or two where a cell can belong to two work-groups (the second
// one empty where it does not).  (Two per column throughout made the walk behind 960 rows merge 100 instead of 51: 28.5 us
// there, 32.1 with 100.)
template <int BM, int BN, int STAGES, bool SAMPLING, bool WIDE, bool ONCE>
__device__ __forceinline__ void lmhead_body(const bf16_t* __restrict__ hidden, const bf16_t* __restrict__ weight, int M, int V,
                                            int H, LmGrid grid, Partial* __restrict__ partials,
                                            bf16_t* __restrict__ logits_out, float c, LmClear clear) {
  constexpr bool RING = STAGES > 0;
  constexpr bool BY_ASM = !RING;  // (the ring's forms have the registers)
  constexpr int WM = BM / 2;      // hidden-state rows per wave
  constexpr int WN = BN / 2;      // vocabulary entries per wave
  constexpr int IB = WM / 32;     // 32-row blocks per wave
  constexpr int JB = WN / 32;     // 32-entry vocabulary blocks per wave
  constexpr int A_LOADS = BM * kLmChunks / kLmThreads;   // 16-byte loads per thread and slab, hidden states
  constexpr int W_LOADS = BN * kLmChunks / kLmThreads;   // ... weight rows
  static_assert(BM % 64 == 0 && BM >= 64 && BM <= kLmMaxBM && BN % 64 == 0 && BN >= 64 && BN <= kLmBN, "slab and tile");

  __shared__ __attribute__((aligned(16))) bf16_t sh_a[RING ? 1 : 2][RING ? 1 : BM][kLmStride];
  __shared__ __attribute__((aligned(16))) bf16_t sh_w[RING ? 1 : 2][RING ? 1 : BN][kLmStride];
  __shared__ __attribute__((aligned(1024))) bf16_t sh_ring[RING ? STAGES : 1][RING ? BM + BN : 1][kLmBK];

  // Every lane's two largest and its (reference, sum) of each of its rows, from one tile of a cell to the next.  Through registers
  // (not in the ring, whose forms have them to spare) they stay here between tiles: in registers, twelve to
  // eighteen of them, they were what the kernels spilled, and a spilled value comes back through the counter of the loads and
  // stores under way, so that every tile waited for all of them -- in the sampling form for its own stores of the logits.
  constexpr bool KEPT = !RING;
  __shared__ __attribute__((aligned(16))) unsigned long long sh_best[KEPT ? IB : 1][KEPT ? kLmThreads : 1][2];
  __shared__ __attribute__((aligned(8))) float sh_part[KEPT && SAMPLING ? IB : 1][KEPT && SAMPLING ? kLmThreads : 1][2];
  // The ring: results of the other wave column, on their way to the one that writes them.
  __shared__ unsigned long long sh_key[2][IB][32][2];
  __shared__ float sh_sum[SAMPLING ? 2 : 1][SAMPLING ? IB : 1][32][2];

  // The work-groups are dealt out die by die (block index mod 8 is the die).
  const int per_die = gridDim.x >> 3;
  const int group = (blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
  if (SAMPLING) {
    const long stride = static_cast<long>(gridDim.x) * kLmThreads;
    for (long i = static_cast<long>(blockIdx.x) * kLmThreads + threadIdx.x; i < clear.nwords; i += stride) clear.words[i] = 0ull;
    if (clear.status)
      for (long i = static_cast<long>(blockIdx.x) * kLmThreads + threadIdx.x; i < clear.nstatus; i += stride) clear.status[i] = 0;
  }
  const int unit_begin = group * grid.width, unit_end = min(grid.units, unit_begin + grid.width);
  if (unit_begin >= unit_end) return;
  auto cell_at = [&](int unit) { return lm_cell(unit, unit_end, grid.slabs, grid.band, grid.tiles_n, grid.width); };

  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int wn = wave & 1, wm = wave >> 1;
  const int l32 = lane & 31, half = lane >> 5;
  const int KT = H / kLmBK;

  // What this thread stages per slab of 64: a 16-byte chunk of rows tid/8, tid/8 + 32, ... of the tile -- chunk tid%8, or, in
  // the ring, the one that belongs at place tid%8 of its row (lm_place).
  const int srow = tid / kLmChunks, schunk = (RING ? lm_place(srow, tid % kLmChunks) : tid % kLmChunks) * 8;
  using Rows = LmRows<!WIDE>;
  auto slab_rows = [&](int slab) {
    return Rows(hidden + static_cast<size_t>(slab) * BM * H, min(BM, M - slab * BM), H, srow, schunk);
  };
  auto tile_rows = [&](int tile) {
    return Rows(weight + static_cast<size_t>(tile) * BN * H, min(BN, V - tile * BN), H, srow, schunk);
  };

  unsigned long long best1[IB], best2[IB];  // (KEPT: in LDS; these are not used)
  float sref[IB], ssum[IB];  // SAMPLING: reference (already times c) and sum of this lane's share of its rows
#pragma unroll
  for (int ib = 0; ib < IB; ++ib) { best1[ib] = 0ull; best2[ib] = 0ull; sref[ib] = -1.0e30f; ssum[ib] = 0.0f; }

  // The units are one sequence of steps (unit, slab of 64) whose operand requests do not stop at
  // tile boundaries.  A step's operands are requested kLmDepth steps ahead -- a weight line comes from HBM,
  // microseconds away under load, while a step's multiplications take about one -- into registers that are
  // written to LDS one step ahead of their use, each behind the write that frees it.
  constexpr int D = kLmDepth;
  u32x4 ga[A_LOADS], gw[W_LOADS];
  LmCell l_cell = cell_at(unit_begin);  // the unit the next request is for
  int l_unit = unit_begin, l_at = 0, l_kt = 0;
  // With at most 128 rows (the kernel then streams the weight at the memory rate) every work-group walks the hidden
  // dimension from a starting slab of its own and wraps round -- two slabs of 64 rows as well, which then read the
  // weight each for itself (120 rows x 4096 x 64 000 179 us against 93 in one slab of 128, which such a call takes) -- a sum
  // in another order.  The rows of a tile lie a whole multiple of 128 bytes apart, so work-groups
  // in step would otherwise ask for the same address bits 7..12 all over the chip at the same
  // time; staggered, the weight streams 7 % faster (3 % at 120 rows).  From 180 rows on nothing
  // is gained, and with several slabs it costs 2-5 %: the work-groups of a die would no longer
  // read the same columns of the hidden states at the same time.
  int l_kp = M <= 128 ? (group * 37) % KT : 0;  // the slab of 64 the next request reads
  Rows a_rows = slab_rows(l_cell.slab), w_rows = tile_rows(l_cell.tile);

  // (Requests are unconditional on purpose: with a request under a branch the compiler has to
  // place its s_waitcnt for the case that nothing was issued, which makes every step wait for the
  // loads it has just sent.  Past the last unit its last slabs are simply requested again.
  // The bookkeeping with its branch is kept apart from the loads, which the steps below issue one
  // by one between their matrix instructions.)
  auto request = [&]() {
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) ga[i] = a_rows.load(i, l_kp * kLmBK);
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i) gw[i] = w_rows.load(i, l_kp * kLmBK);
  };
  auto advance = [&]() {
    if (++l_kp == KT) l_kp = 0;
    if (++l_kt == KT) {
      l_kt = 0;
      if (l_unit + 1 < unit_end) {
        ++l_unit;
        if (++l_at == l_cell.n) {
          l_at = 0;
          l_cell = cell_at(l_unit);
          a_rows = slab_rows(l_cell.slab);
        }
        w_rows = tile_rows(l_cell.tile + l_at);
      } else if (RING) {  // past the last unit: nothing is fetched
        a_rows = Rows(hidden, 0, H, srow, schunk);
        w_rows = Rows(weight, 0, H, srow, schunk);
      }
    }
  };

  // The ring: a step's operands go from memory straight to LDS, STAGES - 1 steps ahead of their use, and its fragments
  // from there to registers one step ahead.
  constexpr int kQuarters = kLmBK / 16;
  constexpr unsigned int kStageBytes = static_cast<unsigned int>(RING ? BM + BN : 0) * kLmBK * 2;
  const unsigned int ring_base = lm_lds_address(&sh_ring[0][0][0]);
  unsigned int stage = 0;  // bytes: the stage of the step whose fragments are in registers
  const unsigned int wave_rows = static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(wave)) * 1024u;  // bytes: eight rows of 128
  auto issue = [&](unsigned int to) {
    const unsigned int lds = ring_base + to + wave_rows;
    if constexpr (RING) {
#pragma unroll
      for (int i = 0; i < A_LOADS; ++i) a_rows.template to_lds<false>(i, l_kp * kLmBK, lds + i * 4096);
#pragma unroll
      for (int i = 0; i < W_LOADS; ++i) w_rows.template to_lds<ONCE>(i, l_kp * kLmBK, lds + (A_LOADS + i) * 4096);
    }
  };
  u32x4 rw[RING ? 2 : 1][kQuarters][JB], rh[RING ? 2 : 1][kQuarters][IB];
  int place[kQuarters];  // of this lane's chunk in every quarter, in elements
#pragma unroll
  for (int ks = 0; ks < kQuarters; ++ks) place[ks] = l32 * kLmBK + lm_place(l32, 2 * ks + half) * 8;
  auto read_stage = [&](u32x4(&w)[kQuarters][JB], u32x4(&h)[kQuarters][IB], unsigned int from) {
    const bf16_t* at = &sh_ring[0][0][0] + from / 2;
#pragma unroll
    for (int ks = 0; ks < kQuarters; ++ks) {
#pragma unroll
      for (int r = 0; r < IB; ++r) h[ks][r] = *reinterpret_cast<const u32x4*>(at + (wm * WM + r * 32) * kLmBK + place[ks]);
#pragma unroll
      for (int r = 0; r < JB; ++r) w[ks][r] = *reinterpret_cast<const u32x4*>(at + (BM + wn * WN + r * 32) * kLmBK + place[ks]);
    }
  };
  // operand fragments of the current and the next quarter (lane l: row l%32 of its block,
  // elements 8*(l/32) .. +7 of the 16-deep quarter)
  u32x4 wf[2][JB], hf[2][IB];
  if constexpr (RING) {
#pragma unroll 1
    for (int s = 0; s < STAGES; ++s) {
      issue(s * kStageBytes);
      advance();
    }
    lm_ring_turn<(STAGES - 1) * (A_LOADS + W_LOADS)>();
    read_stage(rw[0], rh[0], 0);
  } else {
    request();
    advance();
    lm_store_lds<A_LOADS>(ga, &sh_a[0][srow][schunk]);
    lm_store_lds<W_LOADS>(gw, &sh_w[0][srow][schunk]);
    request();
    advance();
    __syncthreads();
    lm_load_frags<JB>(wf[0], &sh_w[0][wn * WN + l32][half * 8]);
    lm_load_frags<IB>(hf[0], &sh_a[0][wm * WM + l32][half * 8]);
  }

  LmCell cell = cell_at(unit_begin);  // the unit being multiplied
  int at = 0;
  for (int unit = unit_begin; unit < unit_end; ++unit) {
    const int tile = cell.tile + at, m0 = cell.slab * BM;
    f32x16_t acc[JB][IB];
    // One step; the first of a tile starts its sums from zero (an operand of the instruction, not 256
    // registers to clear).
    auto ring_step = [&](auto first_step, auto parity) {
      constexpr int cur = decltype(parity)::value;
      // Every wave has this step's fragments in registers and its share of the next step in LDS: this step's stage is
      // free for the step STAGES ahead, the next stage can be read.  Requests and reads stand between the multiplications, as in
      // the form below (all in front of them: 960 rows, 128 to a slab, 1 110 us per call against 995).
      lm_ring_turn<(STAGES - 2) * (A_LOADS + W_LOADS)>();
      const unsigned int lds = ring_base + stage + wave_rows;
      const int l_k = l_kp * kLmBK;
      a_rows.renew();
      w_rows.renew();
      stage = stage + kStageBytes == STAGES * kStageBytes ? 0u : stage + kStageBytes;
      const bf16_t* at = &sh_ring[0][0][0] + stage / 2;
      // What goes out in the step, a share of it behind every multiplication: reads of the next step's fragments and
      // requests in turn.
      constexpr int kReads = kQuarters * (IB + JB), kLoads = A_LOADS + W_LOADS, kMfma = kQuarters * IB * JB;
      auto read = [&](int n) __attribute__((always_inline)) {
        const int ks = n / (IB + JB), r = n % (IB + JB);
        if (r < IB) rh[cur ^ 1][ks][r] = *reinterpret_cast<const u32x4*>(at + (wm * WM + r * 32) * kLmBK + place[ks]);
        else rw[cur ^ 1][ks][r - IB] = *reinterpret_cast<const u32x4*>(at + (BM + wn * WN + (r - IB) * 32) * kLmBK + place[ks]);
      };
      auto load = [&](int n) __attribute__((always_inline)) {
        if (n < A_LOADS) a_rows.template to_lds<false>(n, l_k, lds + n * 4096);
        else w_rows.template to_lds<ONCE>(n - A_LOADS, l_k, lds + n * 4096);
      };
#pragma unroll
      for (int m = 0; m < kMfma; ++m) {
        const int ks = m / (IB * JB), jb = m % (IB * JB) / IB, ib = m % IB;
        acc[jb][ib] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, rw[cur][ks][jb]),
                                                              __builtin_bit_cast(bf16x8_t, rh[cur][ks][ib]),
                                                              (decltype(first_step)::value && ks == 0) ? f32x16_t{} : acc[jb][ib],
                                                              0, 0, 0);
#pragma unroll
        for (int n = m * kLoads / kMfma; n < (m + 1) * kLoads / kMfma; ++n) load(n);
#pragma unroll
        for (int n = m * kReads / kMfma; n < (m + 1) * kReads / kMfma; ++n) read(n);
        __builtin_amdgcn_sched_barrier(0);
      }
      advance();
    };
    auto multiply = [&](auto first_step, const int cur) {
      // Four 16-deep multiplication quarters of 4 x IB MFMAs.  A wave is alone on its SIMD, so
      // nothing hides a memory instruction's issue time or an LDS round trip but its own matrix
      // instructions: every memory instruction of the step is slotted between two MFMAs (the
      // code is written in that order and a scheduling barrier behind every MFMA keeps the
      // compiler from regrouping it).  Quarters 0..2: the fragments of the next quarter, the LDS writes
      // of the next step's operands (requested a step ago) and behind each of them the request for the step
      // after next into the registers it frees.  The step's only
      // barrier follows quarter 2 -- by then this stage has been read for the last time (quarter
      // 3's fragments are in registers) and the other one is complete -- so that quarter 3 can
      // already fetch the next step's first fragments.
      constexpr int kRounds = kLmBK / 16;
      constexpr int kMfma = JB * IB;  // MFMAs per quarter
      const int l_k = l_kp * kLmBK;
      a_rows.renew();
      w_rows.renew();
#pragma unroll
      for (int ks = 0; ks < kRounds; ++ks) {
        const bool last = ks + 1 == kRounds;
        // where the fragments of the next quarter come from: this stage, or (quarter 3) the next step's
        const bf16_t* wsrc = last ? &sh_w[cur ^ 1][wn * WN + l32][half * 8]
                                  : &sh_w[cur][wn * WN + l32][(ks + 1) * 16 + half * 8];
        const bf16_t* hsrc = last ? &sh_a[cur ^ 1][wm * WM + l32][half * 8]
                                  : &sh_a[cur][wm * WM + l32][(ks + 1) * 16 + half * 8];
        // this quarter's share of the writes and requests: rows ks, ks+3, ... of either operand; none in quarter 3
        // (behind the barrier)
        const int nA = (last || ks >= A_LOADS) ? 0 : (A_LOADS - ks + kRounds - 2) / (kRounds - 1);
        const int nW = (last || ks >= W_LOADS) ? 0 : (W_LOADS - ks + kRounds - 2) / (kRounds - 1);
        const int nmoves = nA + nW;
#pragma unroll
        for (int i = 0; i < kMfma; ++i) {
          const int jb = i / IB, ib = i % IB;
          acc[jb][ib] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wf[ks & 1][jb]),
                                                                __builtin_bit_cast(bf16x8_t, hf[ks & 1][ib]),
                                                                (decltype(first_step)::value && ks == 0) ? f32x16_t{} : acc[jb][ib],
                                                                0, 0, 0);
          // one fragment of the next quarter behind each of the first MFMAs
#pragma unroll
          for (int r = 0; r < JB + IB; ++r)
            if (min(r, kMfma - 1) == i) {
              if (r < JB) wf[(ks + 1) & 1][r] = *reinterpret_cast<const u32x4*>(wsrc + r * 32 * kLmStride);
              else hf[(ks + 1) & 1][r - JB] = *reinterpret_cast<const u32x4*>(hsrc + (r - JB) * 32 * kLmStride);
            }
          // an LDS write behind some of them and the load into the same registers behind the next, none behind
          // the last two (the barrier after quarter 2 should not have to wait for an LDS instruction just issued)
#pragma unroll
          for (int m = 0; m < nmoves; ++m) {
            const int slot = 1 + m * (kMfma - 3) / nmoves;  // slots 1 .. kMfma - 3
            const int j = m < nA ? ks + m * (kRounds - 1) : ks + (m - nA) * (kRounds - 1);
            if (slot == i) {
              if (m < nA) *reinterpret_cast<u32x4*>(&sh_a[cur ^ 1][srow + j * 32][schunk]) = ga[j];
              else *reinterpret_cast<u32x4*>(&sh_w[cur ^ 1][srow + j * 32][schunk]) = gw[j];
            }
            if (slot + 1 == i) {
              if (m < nA) ga[j] = a_rows.load(j, l_k);
              else gw[j] = w_rows.load(j, l_k);
            }
          }
          __builtin_amdgcn_sched_barrier(0);  // keep this order
        }
        if (ks + 2 == kRounds) __syncthreads();
      }
      advance();
    };
    // (KT is even: a tile starts with stage 0)
    if constexpr (RING) {
      using P0 = std::integral_constant<int, 0>;
      using P1 = std::integral_constant<int, 1>;
      ring_step(std::true_type{}, P0{});
      ring_step(std::false_type{}, P1{});
      for (int kt = 2; kt < KT; kt += 2) {
        ring_step(std::false_type{}, P0{});
        ring_step(std::false_type{}, P1{});
      }
    } else {
      multiply(std::true_type{}, 0);
      multiply(std::false_type{}, 1);
      for (int kt = D; kt < KT; kt += D) {
        multiply(std::false_type{}, 0);
        multiply(std::false_type{}, 1);
      }
    }

    // The tile's logits, in this lane: hidden-state row m0 + wm*WM + ib*32 + l32, vocabulary
    // entries n0 + wn*128 + jb*32 + 8*(r/4) + 4*half + r%4, ascending in o = 16*jb + r.  Rounded to bf16
    // (two at a time, the hardware conversion: nearest even), made order-preserving as 16-bit integers (two
    // at a time), the upper half of a signed 32-bit key with 63 - o below it (larger value first, then the
    // lower entry); a step of the top-2 is a maximum and a median of three.
    const int n0 = tile * BN;
    const int nbase = n0 + wn * WN + 4 * half;
    auto entry_of = [](int o) { return (o >> 4) * 32 + ((o & 15) >> 2) * 8 + (o & 3); };  // relative to nbase
    constexpr int kPast = -2147483647 - 1;
    auto finish_tile = [&](auto ragged_tile) {
    constexpr bool ragged = decltype(ragged_tile)::value;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      if constexpr (KEPT) {  // (a cell's first tile: nothing yet)
        best1[ib] = at == 0 ? 0ull : sh_best[ib][tid][0];
        best2[ib] = at == 0 ? 0ull : sh_best[ib][tid][1];
        if constexpr (SAMPLING) {
          sref[ib] = at == 0 ? -1.0e30f : sh_part[ib][tid][0];
          ssum[ib] = at == 0 ? 0.0f : sh_part[ib][tid][1];
        }
      }
      int k1 = kPast, k2 = kPast;
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) {
        uint32_t w[8];
        lm_rounded<BY_ASM>(acc[jb][ib], w);
        int left = V - nbase;  // (made anew for every block: 64 conditions kept would be 128 scalar registers)
        if (ragged) asm volatile("" : "+v"(left));
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const uint32_t y = lm_ordered_pair(w[p]);
          const int o = 16 * jb + 2 * p;
          int lo = static_cast<int>((y << 16) | static_cast<uint32_t>(63 - o));
          int hi = static_cast<int>((y & 0xFFFF0000u) | static_cast<uint32_t>(62 - o));
          if (ragged) {  // an entry past the vocabulary: below everything, and left out when the keys are looked at
            lo = entry_of(o) < left ? lo : (lo & 63) + kPast;
            hi = entry_of(o + 1) < left ? hi : (hi & 63) + kPast;
          }
          lm_top2_step(k1, k2, lo);
          lm_top2_step(k1, k2, hi);
        }
        // one accumulator block at a time: the operands in flight stay in their registers
        __builtin_amdgcn_sched_barrier(0);
      }
      const int e1 = nbase + entry_of(63 - (k1 & 63)), e2 = nbase + entry_of(63 - (k2 & 63));
      const bool any = !ragged || e1 < V;
      const float top = lm_key_value(k1);
      if (any) top2_insert(best1[ib], best2[ib], make_key(top, e1));
      if (!ragged || e2 < V) top2_insert(best1[ib], best2[ib], make_key(lm_key_value(k2), e2));
      if constexpr (KEPT) { sh_best[ib][tid][0] = best1[ib]; sh_best[ib][tid][1] = best2[ib]; }
      if (SAMPLING) {
        // Second pass over the block row, now that its maximum is known: move the reference if the maximum
        // has risen above it (references are integers, so sums against different ones combine by exact
        // powers of two), add the exponentials of the rounded logits and store these; rows past the end fall outside the buffer.
        // (V is a multiple of 8: four entries are inside the vocabulary or outside it together.)
        const float nref = any ? fmaxf(sref[ib], __builtin_ceilf(top * c)) : sref[ib];
        ssum[ib] *= __builtin_amdgcn_exp2f(sref[ib] - nref);
        sref[ib] = nref;
        // (32 rows are one buffer, of less than 2^32 bytes; a vocabulary beyond 2^25 takes the form with pointers.  The number of
        // rows is made a scalar: a median of three is a vector instruction, and with one word of the buffer in a vector
        // register every store becomes a loop over the lanes' buffers.)
        const int row32 = m0 + __builtin_amdgcn_readfirstlane(wm) * WM + ib * 32;
        const int rows32 = __builtin_amdgcn_readfirstlane(max(0, min(32, M - row32)));
        const __amdgpu_buffer_rsrc_t o_rows = __builtin_amdgcn_make_buffer_rsrc(
            logits_out + static_cast<size_t>(row32) * V, 0, static_cast<int>(static_cast<unsigned int>(rows32) * V * 2u), kLmBufferFlags);
        // (which 16 bytes of the block's rows this lane writes out, lm_out_lines: of rows lane%16 and lane%16 + 16)
        const int ochunk = ((lane >> 4) & 1) + 2 * half;
        const unsigned int first = (static_cast<unsigned int>(lane & 15) * V + n0 + wn * WN + ochunk * 8) * 2;
        bf16_t* out = logits_out + static_cast<size_t>(row32 + l32) * V + nbase;
        float add = 0.0f;
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
          uint32_t w[8];
          lm_rounded<BY_ASM>(acc[jb][ib], w);
          int left = V - nbase;
          if (ragged) asm volatile("" : "+v"(left));
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const uint32_t w0 = w[2 * q4], w1 = w[2 * q4 + 1];
            const int e = jb * 32 + 8 * q4;  // first of the four entries, relative to nbase
            const bool inside = !ragged || e < left;
            if constexpr (WIDE) {
              if (inside && row32 + l32 < M) *reinterpret_cast<uint2*>(out + e) = make_uint2(w0, w1);
            }
            const float x0 = __uint_as_float(w0 << 16), x1 = __uint_as_float(w0 & 0xFFFF0000u);
            const float x2 = __uint_as_float(w1 << 16), x3 = __uint_as_float(w1 & 0xFFFF0000u);
            const float four = (__builtin_amdgcn_exp2f(__builtin_fmaf(x0, c, -nref)) +
                                __builtin_amdgcn_exp2f(__builtin_fmaf(x1, c, -nref))) +
                               (__builtin_amdgcn_exp2f(__builtin_fmaf(x2, c, -nref)) +
                                __builtin_amdgcn_exp2f(__builtin_fmaf(x3, c, -nref)));
            add += inside ? four : 0.0f;
          }
          if constexpr (!WIDE) {
            u32x4 line[2];
            lm_out_lines(w, line);
            const bool inside = !ragged || n0 + wn * WN + jb * 32 + ochunk * 8 < V;
#pragma unroll
            for (int i = 0; i < 2; ++i)
              __builtin_amdgcn_raw_buffer_store_b128(line[i], o_rows,
                                                     inside ? static_cast<int>(first + static_cast<unsigned int>(i) * 32u * V + 64 * jb) : -1, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        ssum[ib] += add;
        if constexpr (KEPT) { sh_part[ib][tid][0] = sref[ib]; sh_part[ib][tid][1] = ssum[ib]; }
      }
    }
    };
    if (BY_ASM) lm_results_ready();
    if (n0 + BN > V) finish_tile(std::true_type{}); else finish_tile(std::false_type{});

    if (++at < cell.n) continue;
    // The cell, or this work-group's part of it, is done.  Lanes l and l + 32 hold the same rows (different
    // vocabulary entries), and so do the two waves side by side (wn = 0, 1): the half-waves combine through a
    // lane exchange, the waves through LDS, and wave column 0 writes the partial result.  (Two barriers at
    // least stand between here and the next use of the LDS words: every step has one.)
    unsigned long long r1[IB], r2[IB];
    float rR[IB];
    double rS[IB];
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      if constexpr (KEPT) {
        best1[ib] = sh_best[ib][tid][0];
        best2[ib] = sh_best[ib][tid][1];
        if constexpr (SAMPLING) { sref[ib] = sh_part[ib][tid][0]; ssum[ib] = sh_part[ib][tid][1]; }
      }
      const unsigned long long o1 = __shfl_xor(best1[ib], 32, kWave), o2 = __shfl_xor(best2[ib], 32, kWave);
      r1[ib] = best1[ib]; r2[ib] = best2[ib];
      top2_insert(r1[ib], r2[ib], o1);
      top2_insert(r1[ib], r2[ib], o2);
      rR[ib] = -3.0e38f; rS[ib] = 0.0;
      if (SAMPLING) {
        const float oR = __shfl_xor(sref[ib], 32, kWave), oS = __shfl_xor(ssum[ib], 32, kWave);
        // (both halves add in the order lower half, upper half: the same bits in either lane)
        const float aR = half == 0 ? sref[ib] : oR, aS = half == 0 ? ssum[ib] : oS;
        const float bR = half == 0 ? oR : sref[ib], bS = half == 0 ? oS : ssum[ib];
        if (aS > 0.0f) absorb_sum(rR[ib], rS[ib], aR, static_cast<double>(aS));
        if (bS > 0.0f) absorb_sum(rR[ib], rS[ib], bR, static_cast<double>(bS));
      }
      if (wn == 1 && half == 0) {
        unsigned long long* key = KEPT ? sh_best[KEPT ? ib : 0][KEPT ? tid : 0] : sh_key[wm][ib][l32];
        key[0] = r1[ib];
        key[1] = r2[ib];
        if constexpr (SAMPLING) {
          float* sum = KEPT ? sh_part[KEPT ? ib : 0][KEPT ? tid : 0] : sh_sum[wm][ib][l32];
          sum[0] = rR[ib];
          sum[1] = static_cast<float>(rS[ib]);
        }
      }
      best1[ib] = 0ull; best2[ib] = 0ull; sref[ib] = -1.0e30f; ssum[ib] = 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
      const int row = m0 + wm * WM + ib * 32 + l32;
      if (wn == 0 && half == 0 && row < M) {
        unsigned long long k1 = r1[ib], k2 = r2[ib];
        const unsigned long long* key = KEPT ? sh_best[KEPT ? ib : 0][KEPT ? tid + kWave : 0] : sh_key[wm][ib][l32];
        top2_insert(k1, k2, key[0]);
        top2_insert(k1, k2, key[1]);
        Partial out;
        out.z1 = neg_inf(); out.id1 = -1; out.z2 = neg_inf(); out.id2 = -1; out.s = 0.0f; out.ref = 0.0f;
        const Partial empty = out;
        if (k1 != 0ull) { out.z1 = key_value(k1); out.id1 = key_index(k1); }
        if (k2 != 0ull) { out.z2 = key_value(k2); out.id2 = key_index(k2); }
        if constexpr (SAMPLING) {
          float R = rR[ib];
          double S = rS[ib];
          const float* sum = KEPT ? sh_part[KEPT ? ib : 0][KEPT ? tid + kWave : 0] : sh_sum[wm][ib][l32];
          if (sum[1] > 0.0f) absorb_sum(R, S, sum[0], static_cast<double>(sum[1]));
          if (S > 0.0) { out.s = static_cast<float>(S); out.ref = R; }
        }
        Partial* to = partials + static_cast<size_t>(row) * grid.parts;
        if (cell.column < grid.split) {
          to[cell.column] = out;
        } else {
          to += 2 * cell.column - grid.split;
          to[cell.begins ? 0 : 1] = out;
          if (cell.begins && cell.ends) to[1] = empty;
        }
      }
    }
    at = 0;
    if (unit + 1 < unit_end) cell = cell_at(unit + 1);
  }
  // (what has been requested past the last step arrives before the LDS is given back)
  if (RING) lm_ring_turn<0>();
}

template <int BM, bool SAMPLING, bool WIDE = false>
__global__ __launch_bounds__(kLmThreads) void lmhead_reduce_kernel(const bf16_t* __restrict__ hidden,
                                                                   const bf16_t* __restrict__ weight, int M, int V,
                                                                   int H, LmGrid grid, Partial* __restrict__ partials,
                                                                   bf16_t* __restrict__ logits_out, float c, LmClear clear) {
  lmhead_body<BM, kLmBN, 0, SAMPLING, WIDE, false>(hidden, weight, M, V, H, grid, partials, logits_out, c, clear);
}
template <int BM, int BN, int STAGES, bool SAMPLING, bool ONCE>
__global__ __launch_bounds__(kLmThreads) void lmhead_ring_kernel(const bf16_t* __restrict__ hidden,
                                                                 const bf16_t* __restrict__ weight, int M, int V, int H,
                                                                 LmGrid grid, Partial* __restrict__ partials,
                                                                 bf16_t* __restrict__ logits_out, float c, LmClear clear) {
  lmhead_body<BM, BN, STAGES, SAMPLING, false, ONCE>(hidden, weight, M, V, H, grid, partials, logits_out, c, clear);
}

}  // namespace mars
