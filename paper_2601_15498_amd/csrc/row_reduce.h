// Row reduction: per (row, split) the two largest logits with their indices under
// (value desc, index asc) and, in sampling mode, the sum of exp2(z*c - ref).
// One streaming read of the logits; this is the HBM-bound kernel of the pass
// (paper Sec. 3.3 top-2 identification, Eq. 3 softmax normaliser).
//
// The per-element work is kept to the minimum the arithmetic units can hide behind the
// memory stream: widen, half a max3 and, when sampling, one fma + exp2 + add.  A lane only
// tracks the maxima of its batches (two 16-byte vectors each): the best and second-best batch
// maximum and the batches they came from, and keeps a raw copy of its best batch in LDS.
// A lane's two largest elements are then known to lie in those two batches, so after the
// stream the few lanes that can hold a candidate look through their LDS copy (and, rarely,
// reload the second batch) and produce exact (value, index) pairs.
//
// Every wave works for itself from the first load to its own result: there is no barrier and
// no cross-wave traffic while the stream runs, so a wave that has finished leaves the memory
// pipeline to the others instead of holding them at a rendezvous.  The waves meet once, at the
// very end, to fold their eight results into the work-group's one.
#pragma once

#include <type_traits>

#include "chunks.h"
#include "common.h"

namespace mars {

constexpr int kRowThreads = 512;  // 8 waves per work-group (512 x 2 measured best of {128..1024} x {1,2,4,8})
constexpr int kUnroll = 2;        // 16-byte loads per lane per batch
// The reference of a wave's sum of exponentials.  What a term's exponent is off by grows with its distance from the
// reference (half a unit of its last place: 5e-8 of the term at 1, 7e-7 at 16), so the largest terms should be near it; and moving it costs some
// forty instructions.  The first batch puts it 2^kHeadLog2 above its maximum, which rows of ordinary logits seldom pass by more than
// 2^kRescaleLog2; a maximum that rises further above the reference, a logit that stands out, moves it there.  (2^6 above: the terms
// of flat rows, 2^10 and more below it, are off by twice as much.)
constexpr float kHeadLog2 = 2.0f;
constexpr float kRescaleLog2 = 2.0f;
constexpr int kLowLog2 = 8;
static_assert(kRowThreads * kUnroll == kChunkVecs && kRowThreads / kWave == kChunkWaves, "a batch, its waves");

// Insert the elements >= cut of one vector into the running key pair (k1 >= k2).  Only a
// vector whose maximum reaches the cut is looked at element by element (normally one or two):
// the insertions are a serial chain run by a wave with one or two live lanes.
// (first: index of the vector's first element in the row.)
template <typename T, int EPV>
__device__ __forceinline__ void scan_vec(const Vec<T, EPV>& v, int first, float cut, unsigned long long& k1,
                                         unsigned long long& k2) {
  float vm = v.get(0);
#pragma unroll
  for (int e = 1; e < EPV; ++e) vm = fmaxf(vm, v.get(e));
  if (vm >= cut) {
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
      const float x = v.get(e);
      if (x >= cut) top2_insert(k1, k2, make_key(x, first + e));
    }
  }
}

// Exact ranking of every element a lane owns (cold path, kept out of line).
// (Results come back by value: a local whose address is handed to an out-of-line function lives in
// scratch memory, and every later access to it becomes a memory round trip.)
struct KeyPair { unsigned long long k1, k2; };
template <typename T, int EPV>
__device__ __noinline__ KeyPair rank_all(const T* __restrict__ vecp, int head, int v_begin, int v_end, int nb, int tid) {
  unsigned long long k1 = 0, k2 = 0;
#pragma unroll 1
  for (int kb = 0; kb < nb; ++kb) {
#pragma unroll 1
    for (int j = 0; j < kUnroll; ++j) {
      const int vec = v_begin + (kb * kUnroll + j) * kRowThreads + tid;
      if (vec < v_end) {
        Vec<T, EPV> v;
        v.load(vecp, static_cast<unsigned int>(vec));
#pragma unroll 1
        for (int e = 0; e < EPV; ++e) top2_insert(k1, k2, make_key(v.get(e), head + vec * EPV + e));
      }
    }
  }
  KeyPair r;
  r.k1 = k1; r.k2 = k2;
  return r;
}

__device__ __forceinline__ unsigned long long lane_value(unsigned long long v, int lane) {
  const unsigned int lo = __builtin_amdgcn_readlane(static_cast<int>(v), lane);
  const unsigned int hi = __builtin_amdgcn_readlane(static_cast<int>(v >> 32), lane);
  return (static_cast<unsigned long long>(hi) << 32) | lo;
}

// What the row reduction does on behalf of the kernel that follows it on the stream: memory it clears,
// and the gather the sampling walk starts from.
struct ClearArgs {
  unsigned long long* xslots;  // exchange words of the sampling tail: [copies*B][N+2][xwords]
  int N, B, xwords, copies;
  unsigned int* counters;      // histogram counters (nullptr / 0 = none)
  long ncounters;
  // Every acceptance test (Eq. 1) needs the logit and the draft probability of a node's token in its
  // parent's row.  Gathered by the per-request kernel that costs a chain of two trips to memory (tree and
  // tokens, then the gather) on its critical path; here, the work-group of the parent's row reads the tree
  // while its first loads are in flight and leaves the pair in `gathered`, at no cost in time.
  // par == nullptr: not wanted (greedy mode, calls without a tree).
  const int32_t* par;
  const int32_t* tok;
  const void* q;               // draft probabilities [B,N,V] or nullptr (one-hot: the pair's second half is 1)
  int q_bf16;
  float2* gathered;            // [B*N]: (logit, draft probability) of node i's token in row par[i]
  // Sums of the shares' chunks (chunks.h) for a draw that has no need of the whole row then: [rows][splits][slots][waves] pairs
  // (sum, reference), and what the rounding of the sums has left over.  nullptr: not wanted.
  float2* table;
  float* table_low;
  int slots, batches;          // chunks of a share, batches of a chunk
};

// RAGGED: rows that do not start on a 16-byte boundary (a vocabulary that is not a multiple of EPV, an array that is not
// aligned).  The stream runs over the row's aligned vectors; the up to 2 (EPV - 1) elements in front of the first
// and behind the last are one element each for the first lanes of the first wave, which takes them in at
// the end.  (This was one element per load for the whole row: 208 rows of 100 001 bf16 entries 20.8 us, now 13.0.)
// CHUNKS: the sums of the shares' chunks are wanted (clr.table).  A form of its own: with that code in it, unused, calls of 15-30 us took 2-4 % more
// (53 chains of 5 x 38 813 bf16 with dense q 20.1 -> 20.7, 3 trees of 5 x 151 936 17.2 -> 17.8).
// (The unaligned bf16 form takes 65 registers then, three work-groups share a compute unit instead of four.  Held to 64 it puts by three values over the
// stream: 208 rows x 100 001 14.2 us instead of 13.4, 1 664 rows 66 instead of 58.)
template <typename T, int EPV, bool SAMPLING, bool RAGGED, bool CHUNKS>
__global__ __launch_bounds__(kRowThreads) void row_reduce_kernel(const T* __restrict__ logits, int V, int splits,
                                                                  int vecs_per_split, float c,
                                                                  Partial* __restrict__ partials, ClearArgs clr) {
  constexpr int U = kUnroll;
  constexpr int BV = kRowThreads * U;  // vectors per batch
  constexpr int NE = U * EPV;          // elements per lane per batch
  constexpr int NW = kRowThreads / kWave;
  const int item = blockIdx.x;
  const int row = item / splits;
  const int split = item - row * splits;
  const T* __restrict__ rowp = logits + static_cast<size_t>(row) * static_cast<size_t>(V);
  // elements in front of the row's first aligned vector, that vector
  const int head = RAGGED ? min(V, static_cast<int>((16u - (reinterpret_cast<uintptr_t>(rowp) & 15u)) % 16u / sizeof(T))) : 0;
  const T* __restrict__ vecp = rowp + head;
  const int nvec = (V - head) / EPV;
  const int v_begin = min(nvec, split * vecs_per_split);
  const int v_end = min(nvec, v_begin + vecs_per_split);
  const int nv = v_end - v_begin;
  const int tid = threadIdx.x;
  const int nb = (nv + BV - 1) / BV;
  const int nfull = nv / BV;  // batches that need no bounds check

  // The first batch is requested before anything else is done: what follows up to the stream proper
  // (clearing memory for the kernel behind this one, the tree of the request, set-up) then runs beside
  // the first trip to memory instead of in front of it.
  Vec<T, EPV> bufA[U], bufB[U];
  // Unconditional loads for a full batch; bounds-checked loads (padding with -inf) for the last one.
  auto load_full = [&](Vec<T, EPV>(&buf)[U], int k) {
    const T* __restrict__ bp = vecp + static_cast<size_t>(v_begin + k * BV) * EPV;  // wave-uniform
#pragma unroll
    for (int j = 0; j < U; ++j) buf[j].load(bp, static_cast<unsigned int>(tid + j * kRowThreads));
    // Keep the scheduler from hoisting uses of the other buffer above these loads: that would
    // turn the wait for the previous batch into a wait before this one is even issued.
    __builtin_amdgcn_sched_barrier(0);
  };
  // A batch that may be cut short, requested ahead all the same: every lane loads, one past the end of the share from
  // the share's last vector, and what such a lane has loaded is replaced when it arrives.
  auto load_edge = [&](Vec<T, EPV>(&buf)[U], int kk) {
    const int base = v_begin + kk * BV + tid;
#pragma unroll
    for (int j = 0; j < U; ++j)
      buf[j].load(vecp, static_cast<unsigned int>(min(base + j * kRowThreads, v_end - 1)));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto trim_edge = [&](Vec<T, EPV>(&buf)[U], int kk) {
    const int base = v_begin + kk * BV + tid;
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (base + j * kRowThreads >= v_end) buf[j].fill_neg_inf();
  };
  // (RAGGED: a share of any length, short ones too.  Their batches one behind the other behind the set-up made a few rows
  // slower than one element per load had been, which streams: 8 rows of 50 257 bf16 entries, greedy, 4.8 us with
  // single elements, 5.1 with vectors, 4.9 now.)
  const bool ahead = RAGGED ? nb > 0 : nfull > 2;
  if (ahead) { if (RAGGED) load_edge(bufA, 0); else load_full(bufA, 0); }
  // The loose elements at the row's ends, one per lane (every wave asks for them, so that no load stands under a
  // condition; the first wave of the first split looks at those in front, of the last one at those behind).
  const int tail = RAGGED ? V - head - nvec * EPV : 0;
  int loose_at = 0;
  float loose = 0.0f;
  if (RAGGED) {
    const int l = tid % kWave;
    loose_at = l < head ? l : l < head + tail ? V - tail + (l - head) : 0;
    loose = widen(rowp[loose_at]);
  }

  // Exchange words of the tail kernel that follows on the stream (xwords per (request, exchange),
  // N + 2 exchanges per request, `copies` sets of B requests): cleared here so that the call
  // needs no separate memset.  Likewise the counters a following kernel accumulates into.
  if (split == 0 && tid < clr.xwords) {
    const int N = clr.N;
    const int b = row / N, i = row - b * N;
    for (int k = 0; k < clr.copies; ++k) {
      unsigned long long* cells =
          clr.xslots + (static_cast<size_t>(k) * clr.B + b) * static_cast<size_t>(N + 2) * clr.xwords;
      cells[static_cast<size_t>(i) * clr.xwords + tid] = 0ull;
      if (i == 0) {
        cells[static_cast<size_t>(N) * clr.xwords + tid] = 0ull;
        cells[static_cast<size_t>(N + 1) * clr.xwords + tid] = 0ull;
      }
    }
  }
  for (long i = static_cast<long>(item) * kRowThreads + tid; i < clr.ncounters;
       i += static_cast<long>(gridDim.x) * kRowThreads)
    clr.counters[i] = 0u;

  // The children of this row's node, at most kGatherPer per thread: tree and tokens are requested now and
  // looked at behind the first loads of the stream.
  constexpr int kGatherPer = (MARS_MAX_NODES + kRowThreads - 1) / kRowThreads;
  const bool gather = clr.par != nullptr && split == 0;
  const int gnode = row % clr.N;
  const size_t greq = static_cast<size_t>(row - gnode);  // first row of the request
  int gpar[kGatherPer], gtok[kGatherPer];
  float2 gval[kGatherPer];
#pragma unroll
  for (int j = 0; j < kGatherPer; ++j) {
    const int i = tid + j * kRowThreads;
    gpar[j] = -2; gtok[j] = -1;
    if (gather && i > gnode && i < clr.N) { gpar[j] = clr.par[greq + i]; gtok[j] = clr.tok[greq + i]; }
  }
  auto gather_issue = [&]() {
#pragma unroll
    for (int j = 0; j < kGatherPer; ++j) {
      gval[j] = make_float2(0.0f, 1.0f);
      if (gpar[j] == gnode && static_cast<unsigned int>(gtok[j]) < static_cast<unsigned int>(V)) {
        gval[j].x = widen(rowp[gtok[j]]);
        if (clr.q) {
          const size_t at = static_cast<size_t>(row) * static_cast<size_t>(V) + gtok[j];
          gval[j].y = clr.q_bf16 ? widen(static_cast<const bf16_t*>(clr.q)[at]) : static_cast<const float*>(clr.q)[at];
        }
      } else {
        gpar[j] = -2;
      }
    }
  };
  auto gather_store = [&]() {
#pragma unroll
    for (int j = 0; j < kGatherPer; ++j)
      if (gpar[j] == gnode) clr.gathered[greq + tid + j * kRowThreads] = gval[j];
  };

  float m1 = neg_inf(), m2 = neg_inf();  // best and second-best batch maximum of this lane
  int b1 = -1, b2 = -1;                  // the (distinct) batches they belong to
  // Sum of exp2(z*c - ref_c) over the lane's elements of the current chunk.  The sums of chunks decide which token is drawn: from the sums
  // of eight terms on they are formed in double, as by a walk that goes over the row.
  std::conditional_t<CHUNKS, double, float> s = 0.0f;
  float ref_c = -1.0e30f;                // wave-uniform, integer-valued reference (already times c)
  float thresh = -3.0e38f;               // rescale when a lane maximum exceeds this (wave-uniform)
  const float inv_c = SAMPLING ? 1.0f / c : 0.0f;
  // Lane j holds the wave's sum over chunk j and its reference, once the stream is past it.
  double chunk_s = 0.0;
  float chunk_ref = 0.0f;
  double done = 0.0;                       // sum of the chunks behind it, against done_ref
  float done_ref = -1.0e30f;
  int chunk = 0, chunk_end = clr.batches;  // the current chunk, the batch behind it

  // Raw copy of every lane's best batch (vector j of lane t at [j][t]: conflict-free 16-byte rows).
  __shared__ Vec<T, EPV> sh_best[U][kRowThreads];
  // Results of the eight waves and the number of waves that have theirs (cleared here; the only barrier
  // of the kernel stands behind every wave's first loads, where nobody has anything to wait for yet).
  __shared__ unsigned long long sh_k[NW][2];
  __shared__ float sh_s[NW], sh_ref[NW];
  __shared__ int sh_done;
  if (tid == 0) sh_done = 0;

  auto load_tail = [&](Vec<T, EPV>(&buf)[U], int k) {
    const int base = v_begin + k * BV + tid;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int vec = base + j * kRowThreads;
      if (vec < v_end) buf[j].load(vecp, static_cast<unsigned int>(vec)); else buf[j].fill_neg_inf();
    }
  };

  auto process = [&](const Vec<T, EPV>(&buf)[U], int k) {
    float x[NE];
#pragma unroll
    for (int j = 0; j < U; ++j)
#pragma unroll
      for (int e = 0; e < EPV; ++e) x[j * EPV + e] = buf[j].get(e);
    // batch maximum: max3 over pairs, two independent chains
    float bm;
    if (NE >= 4) {
      float ma = fmaxf(x[0], x[1]), mb = fmaxf(x[2], x[3]);
#pragma unroll
      for (int i = 4; i + 3 < NE; i += 4) {
        ma = fmaxf(fmaxf(ma, x[i]), x[i + 1]);
        mb = fmaxf(fmaxf(mb, x[i + 2]), x[i + 3]);
      }
      bm = fmaxf(ma, mb);
    } else {
      bm = x[0];
#pragma unroll
      for (int i = 1; i < NE; ++i) bm = fmaxf(bm, x[i]);
    }
    // Best and second-best batch maximum, first occurrence wins ties (later batches have
    // higher vocabulary indices).  A new best demotes the old one.
    const bool gt = bm > m1;
    const bool g2 = bm > m2;
    m2 = gt ? m1 : (g2 ? bm : m2);
    b2 = gt ? b1 : (g2 ? k : b2);
    m1 = gt ? bm : m1;
    b1 = gt ? k : b1;
    if (__any(gt)) {
      if (gt) {
#pragma unroll
        for (int j = 0; j < U; ++j) sh_best[j][tid] = buf[j];
      }
    }
    if (SAMPLING) {
      if (__any(bm > thresh)) {
        // Rare: the wave's maximum rose more than 2^kRescaleLog2 above the reference (or this is
        // the wave's first batch).  Move the reference up before any term of this batch is formed: no
        // exponent ever exceeds kRescaleLog2, and references, which are whole numbers, differ by exact powers of two.
        const float wm = wave_max(bm);
        const float new_ref_c = __builtin_ceilf(wm * c) + (ref_c < -0.5e30f ? kHeadLog2 : 0.0f);
        s *= __builtin_amdgcn_exp2f(ref_c - new_ref_c);
        ref_c = new_ref_c;
        thresh = (ref_c + kRescaleLog2) * inv_c;
      }
      // (in pairs, then fours: as many additions as one behind the other, three roundings instead of eight; CHUNKS: eights, and these in
      // double)
      auto term = [&](int i) { return __builtin_amdgcn_exp2f(__builtin_fmaf(x[i], c, -ref_c)); };
      auto four = [&](int i) { return (term(i) + term(i + 1)) + (term(i + 2) + term(i + 3)); };
      if constexpr (EPV == 1) {
        float t = term(0);
#pragma unroll
        for (int j = 1; j < U; ++j) t += term(j);
        s += t;
      } else if constexpr (CHUNKS) {
#pragma unroll
        for (int i = 0; i < NE; i += 8) s += static_cast<double>(four(i) + four(i + 4));
      } else {
        float bs[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          bs[j] = four(j * EPV);
          if (EPV == 8) bs[j] += four(j * EPV + 4);
        }
        float t = bs[0];
#pragma unroll
        for (int j = 1; j < U; ++j) t += bs[j];
        s += t;
      }
      // The batch's terms are summed here and now.  Left to itself the compiler sinks this block behind
      // the next batch's wait, widening and maxima (the scheduling barriers order instructions, not the
      // passes that move computations towards their uses): a wave then sits out its wait with this work
      // still to do, and thirty-two widened elements are live instead of sixteen -- 76 registers instead
      // of 59, six waves per SIMD instead of eight, three work-groups per compute unit instead of four.
      asm volatile("" : "+v"(s));
    }
  };

  // Behind a chunk's last batch: its sum over the wave, once in two batches or more.  Some sixty instructions; where no draw asks for chunks the headline
  // workload's call takes what it took (68.6 and 68.7 us), where one does the row reduction takes 0.2-0.5 us more (60 rows x 151 936; 6 656 rows of fp32
  // 617 us instead of 588, for a walk of 12 us instead of 68; what the sums are rounded by, stored as well, is 11 of them).
  auto move_done = [&](double more) {  // (the same in all lanes: scalar registers)
    absorb_sum(done_ref, done, ref_c, more);
    done = lane_value(done, 0);
    done_ref = lane_value(done_ref, 0);
  };
  auto end_chunk = [&]() {
    const double ws = wave_sum(static_cast<double>(s));
    const bool mine = tid % kWave == chunk;
    chunk_s = mine ? ws : chunk_s;
    chunk_ref = mine ? ref_c : chunk_ref;
    move_done(ws);
    // A chunk far below the reference, which a logit that stands out has moved up: the next one begins nearer to its terms.
    const int e = __builtin_amdgcn_frexp_exp(ws);
    if (ws > 0.0 && e < -kLowLog2) {
      ref_c += static_cast<float>(e) + 4.0f;
      thresh = (ref_c + kRescaleLog2) * inv_c;
    }
    s = 0.0f;
    ++chunk;
    chunk_end += clr.batches;
  };

  // Double-buffered stream over the full batches: the loads of batch k+1 are in flight while
  // batch k is processed.  Short shares of aligned rows run
  // through a plain loop with bounds-checked loads; keeping that part small keeps the kernel's
  // code small, which matters for the cold code every wave runs once at its end.
  int k = 0;
  if (ahead) {
    __syncthreads();
    gather_issue();
    for (; k + 2 < nfull; k += 2) {
      load_full(bufB, k + 1);
      process(bufA, k);
      load_full(bufA, k + 2);
      process(bufB, k + 1);
      if (CHUNKS && k + 2 == chunk_end) end_chunk();
    }
    // bufA holds batch k; at most two batches follow it (the last full one, the ragged one).  They are
    // requested ahead like the others, so that a wave does not end its stream on one or two
    // trips to memory with nothing else in flight.  (The requests stand under no
    // condition: where no batch follows, the last one is asked for again and not looked at.  Under a
    // condition, even one that is the same for the whole wave, the compiler no longer knows how many loads
    // are in flight and waits for all of them before batch k is processed.  RAGGED, where a share can be a single batch: what
    // is asked for again is the share's last vector alone, by every lane -- 3 000 rows of 4 087 fp32 entries, greedy, 18.4 us
    // with the batch asked for three times, 16.5 so.)
    const bool more1 = k + 1 < nb, more2 = k + 2 < nb;
    load_edge(bufB, RAGGED ? k + 1 : min(k + 1, nb - 1));
    if (RAGGED && k >= nfull) trim_edge(bufA, k);  // (a short share: batch 0 can be the last)
    process(bufA, k);
    load_edge(bufA, RAGGED ? k + 2 : min(k + 2, nb - 1));
    if (more1) { trim_edge(bufB, k + 1); process(bufB, k + 1); }
    if (more2) { trim_edge(bufA, k + 2); process(bufA, k + 2); }
    k = nb;
  } else {
    __syncthreads();
    gather_issue();
  }
#pragma unroll 1
  for (; !RAGGED && k < nb; ++k) {
    load_tail(bufB, k);
    process(bufB, k);
  }
  gather_store();

  // ------------------------------------------------------------------ per-wave epilogue
  const int wave = tid / kWave, lane = tid % kWave;
  float w1 = m1, w2 = m2;
  wave_top2_values(w1, w2);
  // w1 is the wave's maximum; w2, the second largest batch maximum over its lanes, is a lower
  // bound of its runner-up.  Every element >= w2 lies in batch b1 or b2 of a lane whose own
  // maxima reach w2: those lanes look through their batches.
  unsigned long long k1 = 0, k2 = 0;
  if (w2 > neg_inf()) {
    const float cut = w2;
    if (m1 >= cut) {
#pragma unroll 1
      for (int j = 0; j < U; ++j) {
        const int vec = v_begin + (b1 * U + j) * kRowThreads + tid;
        if (vec < v_end) scan_vec<T, EPV>(sh_best[j][tid], head + vec * EPV, cut, k1, k2);
      }
      if (m2 >= cut) {  // rare: both of the lane's batches matter; the second comes from memory
#pragma unroll 1
        for (int j = 0; j < U; ++j) {
          const int vec = v_begin + (b2 * U + j) * kRowThreads + tid;
          if (vec < v_end) {
            Vec<T, EPV> v;
            v.load(vecp, static_cast<unsigned int>(vec));
            scan_vec<T, EPV>(v, head + vec * EPV, cut, k1, k2);
          }
        }
      }
    }
  } else {
    // The wave saw fewer than two finite batch maxima (a tiny or almost entirely masked share):
    // every element it owns, -inf entries included, is ranked exactly.
    const KeyPair r = rank_all<T, EPV>(vecp, head, v_begin, v_end, nb, tid);
    k1 = r.k1; k2 = r.k2;
  }
  if (RAGGED && wave == 0 && (split == 0 || split == splits - 1)) {
    const bool mine = lane < head ? split == 0 : lane < head + tail && split == splits - 1;
    // (an element below w2 cannot be among the two largest: the wave holds two that are not)
    if (mine && !(loose < w2)) top2_insert(k1, k2, make_key(loose, loose_at));
    if (SAMPLING) {
      if (__any(mine && loose > thresh)) {
        const float wm = wave_max(mine ? loose : neg_inf());
        const float new_ref_c = fmaxf(ref_c, __builtin_ceilf(wm * c));
        s *= __builtin_amdgcn_exp2f(ref_c - new_ref_c);
        ref_c = new_ref_c;
      }
      const float t = mine ? __builtin_amdgcn_exp2f(__builtin_fmaf(loose, c, -ref_c)) : 0.0f;
      // (the elements in front belong to the row's first chunk)
      if (CHUNKS && chunk > 0 && split == 0) {
        const double front = wave_sum(lane < head ? static_cast<double>(t) : 0.0);
        if (lane == 0) {
          const float top = fmaxf(chunk_ref, ref_c);
          chunk_s = chunk_s * __builtin_amdgcn_exp2f(chunk_ref - top) + front * __builtin_amdgcn_exp2f(ref_c - top);
          chunk_ref = top;
        }
        move_done(front);
        s += lane < head ? 0.0f : t;
      } else {
        s += t;
      }
    }
  }
  // Wave-level top-2 of the lanes' keys: walk the (few) lanes that hold any.
  unsigned long long K1 = 0, K2 = 0;
  unsigned long long holders = __ballot(k1 != 0ull);
  while (holders != 0ull) {
    const int l = __ffsll(static_cast<long long>(holders)) - 1;
    holders &= holders - 1;
    top2_insert(K1, K2, lane_value(k1, l));
    const unsigned long long second = lane_value(k2, l);
    if (second != 0ull) top2_insert(K1, K2, second);
  }
  float ws = 0.0f;
  if (SAMPLING) {
    const double rest = wave_sum(static_cast<double>(s));
    if (CHUNKS) {
      if (lane == chunk) { chunk_s = rest; chunk_ref = ref_c; }
      if (lane < clr.slots) {  // (a chunk that the row's share does not have: nothing)
        const size_t to = (static_cast<size_t>(item) * clr.slots + lane) * NW + wave;
        const float high = static_cast<float>(chunk_s);
        clr.table[to] = make_float2(high, chunk_ref);
        clr.table_low[to] = static_cast<float>(chunk_s - static_cast<double>(high));
      }
    }
    ws = static_cast<float>(rest);
    if (CHUNKS && chunk > 0) {
      move_done(rest);
      ws = static_cast<float>(done);
      ref_c = done_ref;
    }
  }
  // The wave that is last to have its result folds the eight into the work-group's partial result; the
  // others leave at once.  (LDS operations of one wave are performed in order, so a wave that sees the
  // count complete sees every result behind it.)  The kernel behind this one then reads one partial
  // result per (row, split) instead of eight -- on its critical path, where this merge is not.
  int last = 0;
  if (lane == 0) {
    sh_k[wave][0] = K1; sh_k[wave][1] = K2;
    sh_s[wave] = ws; sh_ref[wave] = ref_c;
    last = __hip_atomic_fetch_add(&sh_done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP) == NW - 1;
  }
  if (!__builtin_amdgcn_readfirstlane(last)) return;
  static_assert(NW == 8, "three butterfly steps merge eight waves");
  unsigned long long B1 = 0, B2 = 0;
  float R = -3.0e38f;
  double S = 0.0;
  if (lane < NW) {
    B1 = sh_k[lane][0]; B2 = sh_k[lane][1];
    if (SAMPLING && sh_s[lane] > 0.0f) { R = sh_ref[lane]; S = static_cast<double>(sh_s[lane]); }
  }
  merge_step<kDppXor1>(B1, B2, R, S);
  merge_step<kDppXor2>(B1, B2, R, S);
  merge_step<kDppHalfMirror>(B1, B2, R, S);
  if (lane == 0) {
    Partial out;
    out.z1 = neg_inf(); out.id1 = -1; out.z2 = neg_inf(); out.id2 = -1; out.s = 0.0f; out.ref = 0.0f;
    if (B1 != 0ull) { out.z1 = key_value(B1); out.id1 = key_index(B1); }
    if (B2 != 0ull) { out.z2 = key_value(B2); out.id2 = key_index(B2); }
    if (SAMPLING && S > 0.0) { out.s = static_cast<float>(S); out.ref = R; }
    partials[item] = out;
  }
}

// Partial results per (row, split).
constexpr int kPartsPerItem = 1;

// Merge the partial results of every row into the statistics table (16 rows per work-group).
__global__ __launch_bounds__(256) void merge_stats_kernel(const Partial* __restrict__ partials, int rows, int N,
                                                          int parts, const float* __restrict__ theta, float c,
                                                          Indicator ind, mars_row_stat* __restrict__ stats) {
  const int first = blockIdx.x * 16;
  const int n = min(16, rows - first);
  if (n <= 0) return;
  merge_rows_coop<256>(partials + static_cast<size_t>(first) * parts, n, parts, c, ind,
                       [&](int row) { return theta[(first + row) / N]; },
                       [&](int row, const mars_row_stat& st) { stats[first + row] = st; });
}

}  // namespace mars
