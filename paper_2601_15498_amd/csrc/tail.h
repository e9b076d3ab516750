// Per-request tail of the verification pass: merge the row partials, take the
// per-node decisions, select the path and produce the correction / bonus token.
// One work-group per request in greedy mode; in sampling mode up to 32 work-groups share a
// request, each owning a slice of the vocabulary.
//
// Greedy mode is Algorithm 1 on a tree: local three-way test per node, reachability
// by pointer jumping, deepest reachable node (lowest index on ties), token = v(1) of
// its row.  Sampling mode is multi-round rejection sampling down the tree (Eq. 1) with
// the runner-up relaxation of Sec. 3.4 as a deterministic accept, residual
// renormalisation after every rejection (Sec. 2.3) and an inverse-CDF draw at the end.
#pragma once

#include "chunks.h"
#include "common.h"

namespace mars {

constexpr int kGreedyThreads = 1024;  // 64 rows merged at a time
constexpr int kSamplingThreads = 512;    // sampling tail whose slices stay in registers
constexpr int kStreamingThreads = 1024;  // sampling tail that streams its slices: more loads in flight per compute unit
constexpr int kMaxTiles = 512;  // CDF tiles kept in LDS for the final draw
constexpr int kMaxGroupsPerRequest = 32;   // work-groups that may share one request

struct TailArgs {
  const void* logits;
  const int32_t* tok;
  const int32_t* par;
  const void* dprobs;  // nullptr = one-hot draft distribution
  const float* theta;
  const float* u;
  const Partial* partials;
  const float2* gathered;   // sampling mode: (logit, draft probability) of every node's token in its parent's row
                            // (left by the row reduction; nullptr: the walk gathers them itself)
  mars_row_stat* stats;     // optional caller's table [B*N]
  uint8_t* mask;
  int32_t* len;
  int32_t* path;
  int32_t* bonus;
  uint8_t* dec;          // optional
  int32_t* status;       // optional
  mars_req_diag* diag;   // optional
  int B, N, V, splits;   // splits = partial results per row
  // Threshold sweep: B = K * Bd requests are verified, request b reading the inputs (logits,
  // tokens, tree, draft distribution, uniforms, row partials) of request b % Bd with its own
  // theta[b]; every output is indexed by b.  Bd == B without a sweep.
  int Bd;
  Indicator ind;         // which low-margin test (Sec. 3.3)
  int32_t* out_tok;      // optional [B,N]: committed sequence V_out (Alg. 1), -1 padded
  int32_t* out_len;      // optional [B]
  float c;               // log2(e) / T, 0 in greedy mode
  // sampling mode: G work-groups share one request and exchange partial sums
  int G;
  int slice;                // groups of eight entries in a work-group's slice (walk_slice)
  int spin_limit;        // polls a work-group gives a partner before it works out the partner's sum itself
  unsigned long long* xslots;  // [B][N+2][G][2] tagged exchange words, cleared by the row reduction
  // one-hot draft distributions: whether the walk of onehot.h is taken; the sums of the rows' chunks (chunks.h), nullptr: it reads the row
  bool onehot;
  ChunkSpec chunks;
  const float2* table;   // [rows][chunks][kChunkWaves] pairs (sum, reference)
  const float* table_low;  // what the sums lack
};

// ---------------------------------------------------------------- shared by both modes
// Outputs of a request that failed validation: nothing accepted, token = v(1) of the root row.
template <int NT>
__device__ void write_rejected_request(const TailArgs& a, int b, int status, int root_top1) {
  const int N = a.N;
  for (int i = threadIdx.x; i < N; i += NT) {
    const size_t r = static_cast<size_t>(b) * N + i;
    a.mask[r] = i == 0 ? 1 : 0;
    a.path[r] = -1;
    if (a.dec) a.dec[r] = 0;
    if (a.out_tok && i > 0) a.out_tok[r] = -1;
  }
  if (threadIdx.x == 0) {
    a.len[b] = 0;
    a.bonus[b] = root_top1;
    if (a.out_tok) { a.out_tok[static_cast<size_t>(b) * N] = root_top1; a.out_len[b] = 1; }
    if (a.status) a.status[b] = status;
    if (a.diag) { mars_req_diag d = {0.0f, 0.0f, 0, 0}; a.diag[b] = d; }
  }
}

// ---------------------------------------------------------------- greedy mode
// The kernel is a chain of latencies, so it makes one trip to memory: the tree and the tokens are
// requested ahead of the partial results, the merged rows go to the caller's table and, for the
// kernel's own use, to LDS, and everything after that -- decisions, reachability, the walk back
// along the accepted path -- reads LDS only.
// Requests of more nodes than a wave has lanes; the others take tail_greedy_wave_kernel.
__global__ __launch_bounds__(kGreedyThreads) void tail_greedy_kernel(TailArgs a) {
  constexpr int NT = kGreedyThreads;
  static_assert(MARS_MAX_NODES <= NT, "a thread holds the parent and the token of one node");
  __shared__ uint8_t sh_code[MARS_MAX_NODES];
  __shared__ uint8_t sh_ok[2][MARS_MAX_NODES];
  __shared__ int16_t sh_anc[2][MARS_MAX_NODES];
  __shared__ int16_t sh_dep[2][MARS_MAX_NODES];
  __shared__ int16_t sh_par[MARS_MAX_NODES];
  __shared__ int32_t sh_tok[MARS_MAX_NODES];
  __shared__ int32_t sh_top1[MARS_MAX_NODES];    // v(1) of the node's row
  __shared__ int32_t sh_relax[MARS_MAX_NODES];   // v(2) of the node's row where its low-margin test holds, else -1
  __shared__ unsigned int sh_best;

  const int b = blockIdx.x;
  const int N = a.N;
  const int i = threadIdx.x;
  const size_t rb = static_cast<size_t>(b) * N;
  const size_t rd = static_cast<size_t>(b % a.Bd) * N;  // where the request's inputs are
  int p = -1, t = 0;
  if (i < N) { p = a.par[rd + i]; t = a.tok[rd + i]; }
  const float theta = a.theta[b];
  // (eight loads in flight per lane: this kernel has the registers, and behind the fused LM head a
  // row has up to a few hundred partial results)
  merge_rows_coop<NT, 8, false>(a.partials + rd * a.splits, N, a.splits, a.c, a.ind, [&](int) { return theta; },
                         [&](int row, const mars_row_stat& st) {
                           if (a.stats) a.stats[rb + row] = st;
                           sh_top1[row] = st.id1;
                           sh_relax[row] = st.relax_ok ? st.id2 : -1;
                         });
  int bad = 0;
  if (i < N) {
    if (i == 0) { if (p != -1) bad |= 1; }
    else {
      if (p < 0 || p >= i) bad |= 1;
      if (t < 0 || t >= a.V) bad |= 2;
    }
    sh_par[i] = static_cast<int16_t>(p);
    sh_tok[i] = t;
  }
  if (i == 0) sh_best = 0;
  if (__syncthreads_or(bad)) {  // (the barrier also publishes what the merge left in LDS)
    const int any_tree = __syncthreads_or(bad & 1);
    write_rejected_request<NT>(a, b, any_tree ? MARS_REQ_BAD_TREE : MARS_REQ_BAD_TOKEN, sh_top1[0]);
    return;
  }

  // Local decision of every node against its parent's row (Alg. 1 if-chain).
  if (i < N) {
    int code = 0, anc = 0, dep = 0;
    if (i > 0) {
      if (t == sh_top1[p]) code = MARS_DEC_EXACT;
      else if (t == sh_relax[p]) code = MARS_DEC_RELAXED;  // (t >= 0: never equal to the -1 of a failed test)
      anc = p; dep = 1;
    }
    sh_code[i] = static_cast<uint8_t>(code);
    sh_ok[0][i] = (i == 0 || code != 0) ? 1 : 0;
    sh_anc[0][i] = static_cast<int16_t>(anc);
    sh_dep[0][i] = static_cast<int16_t>(dep);
  }
  __syncthreads();
  // Pointer jumping: after round k, anc is the 2^k-th ancestor (or the root), dep the number
  // of edges to it and ok the AND of the local decisions along those edges.
  int cur = 0;
  for (int span = 1; span < N; span <<= 1) {
    const int nxt = cur ^ 1;
    if (i < N) {
      const int an = sh_anc[cur][i];
      sh_ok[nxt][i] = sh_ok[cur][i] & sh_ok[cur][an];
      sh_dep[nxt][i] = static_cast<int16_t>(sh_dep[cur][i] + sh_dep[cur][an]);
      sh_anc[nxt][i] = sh_anc[cur][an];
    }
    cur = nxt;
    __syncthreads();
  }
  // Deepest reachable node, lowest index on ties: max of (depth << 16 | (0xFFFF - i)).
  if (i < N) {
    if (sh_ok[cur][i]) atomicMax(&sh_best, (static_cast<unsigned int>(sh_dep[cur][i]) << 16) | (0xFFFFu - i));
    a.mask[rb + i] = i == 0 ? 1 : 0;
    a.path[rb + i] = -1;
    if (a.dec) a.dec[rb + i] = 0;
    if (a.out_tok) a.out_tok[rb + i] = -1;
  }
  __syncthreads();
  if (i == 0) {
    const unsigned int bk = sh_best;
    const int e = 0xFFFF - static_cast<int>(bk & 0xFFFFu);
    const int L = static_cast<int>(bk >> 16);
    int n = e;
    for (int d = L; d >= 1; --d) {
      a.mask[rb + n] = 1;
      a.path[rb + d - 1] = n;
      if (a.dec) a.dec[rb + n] = sh_code[n];
      if (a.out_tok) a.out_tok[rb + d - 1] = sh_tok[n];  // V_out: the accepted drafts ...
      n = sh_par[n];
    }
    a.len[b] = L;
    const int correction = sh_top1[e];  // correction after a rejection, bonus after a leaf
    a.bonus[b] = correction;
    if (a.out_tok) { a.out_tok[rb + L] = correction; a.out_len[b] = L + 1; }  // ... then this token
    if (a.status) a.status[b] = MARS_REQ_OK;
    if (a.diag) { mars_req_diag dg = {0.0f, 0.0f, 0, e}; a.diag[b] = dg; }
  }
}

// The same for requests of at most 64 nodes, a node per lane of one wave: a parent's row, token and decision come by lane
// exchanges, so that behind the trip to memory there is neither LDS traffic nor a barrier, and what a request commits leaves
// in one store per table.  NT: one wave where a lane merges its row alone (kLaneParts partial results at most); else 1024 threads
// merge, and one wave goes on.
// What bounds it is the trip to memory and, where there are many partial results, merging them.  us per call, the kernel above and this
// one: 64 chains of eight drafts x 128 256 with the committed tokens 32.6 -> 30.5, 112 trees of 5 x 32 000 14.1 -> 12.7, 4 trees of 22 x 151 936
// 14.2 -> 12.4, one tree of 60 behind the LM head 187.2 -> 186.2.
template <int NT>
__global__ __launch_bounds__(NT) void tail_greedy_wave_kernel(TailArgs a) {
  constexpr bool MANY = NT > kWave;
  __shared__ int2 sh_top[MANY ? kWave : 1];  // v(1) of the node's row, v(2) where its low-margin test holds, else -1
  const int b = blockIdx.x;
  const int N = a.N;
  const size_t rb = static_cast<size_t>(b) * N;
  const size_t rd = static_cast<size_t>(a.B == a.Bd ? b : b % a.Bd) * N;  // where the request's inputs are
  const int lane = threadIdx.x % kWave;
  const bool live = lane < N;
  const size_t rl = rd + (live ? lane : 0);
  const int par = a.par[rl], tok = a.tok[rl];
  const float theta = a.theta[b];
  int2 top;
  if (!MANY) {
    const mars_row_stat st = lane_row<false>(a.partials + rl * a.splits, a.splits, a.c, a.ind, theta);
    if (live && a.stats) a.stats[rb + lane] = st;
    top = make_int2(st.id1, st.relax_ok ? st.id2 : -1);
  } else {
    // (eight loads in flight per lane: behind the fused LM head a row has up to a few hundred partial results)
    merge_rows_coop<NT, 8, false>(a.partials + rd * a.splits, N, a.splits, a.c, a.ind, [&](int) { return theta; },
                                  [&](int row, const mars_row_stat& st) {
                                    if (a.stats) a.stats[rb + row] = st;
                                    sh_top[row] = make_int2(st.id1, st.relax_ok ? st.id2 : -1);
                                  });
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    top = sh_top[live ? lane : 0];
  }
  const bool bad_tree = live && (lane == 0 ? par != -1 : par < 0 || par >= lane);
  const bool bad_token = live && lane > 0 && (tok < 0 || tok >= a.V);
  if (__any(bad_tree || bad_token)) {
    write_rejected_request<kWave>(a, b, __any(bad_tree) ? MARS_REQ_BAD_TREE : MARS_REQ_BAD_TOKEN, lane_value(top.x, 0));
    return;
  }
  // Local decision of every node against its parent's row (Alg. 1 if-chain).
  const bool node = live && lane > 0;
  const int p = node ? par : 0;
  const int exact = __shfl(top.x, p, kWave), relaxed = __shfl(top.y, p, kWave);
  const int code = !node ? 0 : tok == exact ? MARS_DEC_EXACT : tok == relaxed ? MARS_DEC_RELAXED : 0;
  // Pointer jumping: an ancestor, the edges up to it and the rejections on them, a byte each (63 at most).  At the root all three
  // are 0.
  unsigned int up = node ? static_cast<unsigned int>(p) | 0x100u | (code == 0 ? 0x10000u : 0u) : 0u;
  while (__any((up & 0xFFu) != 0u)) up = (up & 0xFFFF00u) + __shfl(up, static_cast<int>(up & 0xFFu), kWave);
  // Deepest reachable node, lowest index on ties.
  const int depth = static_cast<int>(up >> 8 & 0xFFu);
  const float rank = live && up < 0x10000u ? static_cast<float>(depth * kWave + (kWave - 1 - lane)) : 0.0f;
  const int best = __builtin_amdgcn_readfirstlane(static_cast<int>(wave_max(rank)));  // (the root's is 63)
  const int e = kWave - 1 - best % kWave, L = best / kWave;
  unsigned long long visited = 1ull;
  int path = -1, n = e;
  for (int d = L; d >= 1; --d) {
    visited |= 1ull << n;
    path = lane == d - 1 ? n : path;
    n = lane_value(par, n);
  }
  const bool on_path = ((visited >> lane) & 1ull) != 0ull;
  const int correction = lane_value(top.x, e);  // correction after a rejection, bonus after a leaf
  const int committed = __shfl(tok, lane < L ? path : 0, kWave);
  if (live) {
    a.mask[rb + lane] = on_path ? 1 : 0;
    a.path[rb + lane] = path;
    if (a.dec) a.dec[rb + lane] = static_cast<uint8_t>(on_path ? code : 0);
    if (a.out_tok) a.out_tok[rb + lane] = lane < L ? committed : lane == L ? correction : -1;
  }
  if (lane == 0) {
    a.len[b] = L;
    a.bonus[b] = correction;
    if (a.out_tok) a.out_len[b] = L + 1;
    if (a.status) a.status[b] = MARS_REQ_OK;
    if (a.diag) { mars_req_diag dg = {0.0f, 0.0f, 0, e}; a.diag[b] = dg; }
  }
}

// ---------------------------------------------------------------- sampling mode
// Eight consecutive elements as they lie in memory (one group): requested without being looked at,
// so that nothing waits for them until they are widened.  ALIGNED: on a 16-byte boundary.  Otherwise no more is known,
// and said, than where an element may begin; the hardware takes such an address, and it is the same one load.
typedef u32x4 u32x4_any __attribute__((aligned(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
  u32x4 v;
  template <bool ALIGNED>
  __device__ __forceinline__ void load(const bf16_t* __restrict__ row, int g) {
    const bf16_t* at = row + static_cast<size_t>(g) * 8;
    if (ALIGNED) v = *reinterpret_cast<const u32x4*>(at); else v = *reinterpret_cast<const u32x4_any*>(at);
  }
  __device__ __forceinline__ void widen_to(float (&x)[8]) const {
    x[0] = __uint_as_float(v.x << 16); x[1] = __uint_as_float(v.x & 0xFFFF0000u);
    x[2] = __uint_as_float(v.y << 16); x[3] = __uint_as_float(v.y & 0xFFFF0000u);
    x[4] = __uint_as_float(v.z << 16); x[5] = __uint_as_float(v.z & 0xFFFF0000u);
    x[6] = __uint_as_float(v.w << 16); x[7] = __uint_as_float(v.w & 0xFFFF0000u);
  }
};
template <> struct Raw8<float> {
  f32x4 lo, hi;
  template <bool ALIGNED>
  __device__ __forceinline__ void load(const float* __restrict__ row, int g) {
    const float* at = row + static_cast<size_t>(g) * 8;
    if (ALIGNED) {
      lo = *reinterpret_cast<const f32x4*>(at);
      hi = *reinterpret_cast<const f32x4*>(at + 4);
    } else {
      lo = *reinterpret_cast<const f32x4_any*>(at);
      hi = *reinterpret_cast<const f32x4_any*>(at + 4);
    }
  }
  __device__ __forceinline__ void widen_to(float (&x)[8]) const {
    x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w; x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
  }
};

// The residual chain at the current node: rejection j replaced f by
// max(0, f - q_j) * inv_norm[j] (q_j dense, or one-hot at tok[j]).
// The first kChainRegs entries live in (wave-uniform) registers, so that the per-element
// evaluation touches no memory; longer chains continue in LDS.
constexpr int kChainRegs = 4;
struct Chain {
  const int32_t* tok;      // LDS
  const float* inv_norm;   // LDS; 0 marks "Z was 0, f left unchanged"
  int n;
  int rtok[kChainRegs];
  float rinv[kChainRegs];
};
// Whether the rejection that becomes entry n of a node's chain ends with a barrier even if it exchanges nothing.  Thread 0
// writes the entries in LDS and every wave reads them when it gets there, so two orders need one: behind an entry in LDS,
// whose readers are the tests that follow; and behind the last entry in registers, since a wave may still be testing the previous
// node's last child with that node's entries when another one is here -- no wave gets to this node's first write to
// LDS before all have left the previous node.  (Chains of three rejections and less, the ordinary ones, have no barrier.)
__device__ __host__ __forceinline__ constexpr bool chain_barrier(int n) { return n + 1 >= kChainRegs; }

// f(v) for the current node: softmax term, then the residual chain.
__device__ __forceinline__ float eval_f(float z, float q, int v, float z1, float c, float inv_S, bool dense,
                                        const Chain& ch) {
  float f = __builtin_amdgcn_exp2f((z - z1) * c) * inv_S;
#pragma unroll
  for (int j = 0; j < kChainRegs; ++j) {
    if (j < ch.n) {
      const float qj = dense ? q : (v == ch.rtok[j] ? 1.0f : 0.0f);
      const float g = fmaxf(f - qj, 0.0f);
      f = ch.rinv[j] > 0.0f ? g * ch.rinv[j] : f;
    }
  }
  for (int j = kChainRegs; j < ch.n; ++j) {
    const float qj = dense ? q : (v == ch.tok[j] ? 1.0f : 0.0f);
    const float g = fmaxf(f - qj, 0.0f);
    const float inv = ch.inv_norm[j];
    f = inv > 0.0f ? g * inv : f;
  }
  return f;
}

// The softmax term (Eq. 3) of an entry of a row.
__device__ __forceinline__ float softmax_at(const mars_row_stat& st, float z, float c) {
  return __builtin_amdgcn_exp2f((z - st.z1) * c) * (1.0f / st.sum_exp);
}
// A child tested against the plain softmax of its parent's row (no rejection at that node yet): the
// runner-up of a low-margin row is accepted outright (Alg. 1), anything else with probability
// min(1, f(x)/q(x)) (Eq. 1).  Returns the decision code (0 = rejected) and f(x).
__device__ __forceinline__ int first_try(const mars_row_stat& st, float zx, float qx, int x, float u, float c,
                                         float& fx) {
  fx = 0.0f;
  if (x == st.id2 && st.relax_ok) return MARS_DEC_RELAXED;
  fx = softmax_at(st, zx, c);
  float acc;
  if (fx == 0.0f) acc = 0.0f;
  else if (qx <= 0.0f) acc = 1.0f;
  else acc = fminf(1.0f, fx / qx);
  return u < acc ? MARS_DEC_SAMPLED : 0;
}

// Sum over the work-group.  The caller keeps a barrier between two calls (the exchange that follows
// every call has one), so the staging array needs none in front of the write.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) t += sh[w];
  return t;
}

// Sum of one double per work-group over the G work-groups of a request, in work-group order
// (so every work-group obtains the same bits).  Exchange number `idx` of request b has its own
// 2*G words, cleared by the row reduction of the same call.  A work-group publishes its value as
// two floats (head and tail of the double), each packed with a non-zero tag into one 64-bit
// word, so that a single store both delivers the data and signals arrival; the partners poll
// the words directly.
//
// No work-group depends on another one being there.  A partner whose words have not arrived
// after `spin_limit` polls (it may not have been given a compute unit yet: the GPU is shared with
// other kernels, other streams, other calls of this library) is not waited for any longer: the
// work-group goes over that partner's slice itself, with the partner's own assignment of elements
// to threads and order of additions, so that it obtains the very bits the partner will publish,
// and carries on.  Whatever the placement of the work-groups, every one of them finishes, and
// all agree.  The exchange therefore comes in three steps, and the caller's pass over a slice is
// written once, inside a loop over "whose slice": its own first, then those of the missing partners.
//   exchange_begin  publish `mine`, poll the partners; returns the set of those that did not arrive
//   exchange_fill   the value worked out here for a missing partner
//   exchange_end    the sum, in work-group order
__device__ __forceinline__ unsigned long long pack_tagged(float v) {
  return (1ull << 32) | static_cast<unsigned long long>(__float_as_uint(v));
}
template <int NT>
__device__ __forceinline__ unsigned int exchange_begin(const TailArgs& a, int b, int g, int idx, double mine,
                                                       double* sh_part, unsigned int* sh_missing) {
  const int G = a.G;
  if (G == 1) { sh_part[0] = mine; return 0u; }
  static_assert(2 * kMaxGroupsPerRequest <= kWave, "one wave polls every word of an exchange");
  unsigned long long* cell = a.xslots + (static_cast<size_t>(b) * (a.N + 2) + idx) * (2 * G);
  if (threadIdx.x == 0) {
    const float hi = static_cast<float>(mine);
    const float lo = static_cast<float>(mine - static_cast<double>(hi));
    __hip_atomic_store(&cell[2 * g], pack_tagged(hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&cell[2 * g + 1], pack_tagged(lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *sh_missing = 0u;
  }
  if (threadIdx.x < 2 * G) {
    // One wave polls all 2*G words at once: lane 2i the head of work-group i's value, lane 2i+1 its tail.
    unsigned long long w = 0;
    int spins = 0;
    for (;;) {
      w = __hip_atomic_load(&cell[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((w >> 32) != 0ull) break;
      if (++spins > a.spin_limit) { atomicOr(sh_missing, 1u << (threadIdx.x >> 1)); break; }
      __builtin_amdgcn_s_sleep(1);
    }
    double v = static_cast<double>(__uint_as_float(static_cast<unsigned int>(w)));
    v += __shfl_down(v, 1, kWave);  // even lanes: head + tail
    if ((threadIdx.x & 1) == 0) sh_part[threadIdx.x >> 1] = v;
  }
  __syncthreads();
  // (written again only behind the caller's next barrier; the same in every lane, and said so: what
  // is derived from it -- whose slice comes next, its bounds -- then lives in scalar registers)
  return static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(*sh_missing)));
}
// (a value worked out here goes through the same two floats as one that travelled)
__device__ __forceinline__ void exchange_fill(double* sh_part, int i, double v) {
  if (threadIdx.x == 0) {
    const float hi = static_cast<float>(v);
    const float lo = static_cast<float>(v - static_cast<double>(hi));
    sh_part[i] = static_cast<double>(hi) + static_cast<double>(lo);
  }
}
// (Behind the barrier that ends exchange_begin, or the one the caller keeps behind its last exchange_fill.
// Lane i holds work-group i's value; the same tree of additions in every wave of every work-group.  The
// caller keeps a barrier between this and the next exchange_begin, which writes sh_part again.)
__device__ __forceinline__ double exchange_end(const TailArgs& a, const double* sh_part) {
  if (a.G == 1) return sh_part[0];
  const int lane = threadIdx.x % kWave;
  return wave_sum(lane < a.G ? sh_part[lane] : 0.0);
}

// Everything a pass over a row needs to evaluate the current distribution f.
//
// A row is looked at in groups of eight elements.  VEC: the groups count from the row's start, and every one is
// whole and aligned (V % 8 == 0, arrays on 16-byte boundaries; the host checks both).  Otherwise they count in the
// whole array -- group c holds its elements 8c .. 8c + 7 -- so that on an aligned array every group is still one
// aligned load, and a row begins `shift` elements into its first group and ends somewhere in its last: what lies
// outside the row is masked where a group is used, which only the lanes with those two groups do.  (It was
// eight loads and eight comparisons per group: on 8 trees of 26 nodes over 100 001 bf16 entries the walk took
// 21.4 us, now 18.5.)  The array's own last group may be cut short: it is read element by element.
template <typename T, typename TQ, bool VEC>
struct RowView {
  const T* zrow;
  const TQ* qrow;   // nullptr = one-hot draft distribution
  bool use_q;       // false: this pass does not look at q (no rejection at this node so far), skip its loads
  int V;
  float z1, c, inv_S;
  Chain ch;
  // VEC == false: first group of the row, elements in front of the row in it, the row's last group, and the last
  // group that lies in the array as a whole (below 0 in an array of less than eight elements), counted from the first.
  const T* zgroup;
  const TQ* qgroup;
  int shift, last, whole;
  // Of the request: the group its first row begins in, how many elements into it, how many whole groups lie between
  // it and the array's end, and readable memory for loads from an array of less than eight elements (else nullptr).
  const T* zreq;
  const TQ* qreq;
  int begin;
  long wholes;
  const void* instead;
  // The request whose rows begin at element `at` of arrays of `count` elements.
  __device__ __forceinline__ void request(const T* zarray, const TQ* qarray, size_t at, size_t count, const void* somewhere) {
    if (VEC) {
      zreq = zarray + at;
      qreq = qarray ? qarray + at : nullptr;
    } else {
      const size_t first = at >> 3 << 3;
      begin = static_cast<int>(at & 7);
      wholes = static_cast<long>(count >> 3) - static_cast<long>(at >> 3);
      zreq = zarray + first;
      qreq = qarray ? qarray + first : nullptr;
      instead = count < 8 ? somewhere : nullptr;
    }
  }
  __device__ __forceinline__ void row(int node, bool dense) {
    if (VEC) {
      zrow = zreq + static_cast<size_t>(node) * V;
      qrow = dense ? qreq + static_cast<size_t>(node) * V : nullptr;
    } else {
      const size_t at = static_cast<size_t>(node) * V + begin;
      zrow = zreq + at;
      qrow = dense ? qreq + at : nullptr;
      shift = static_cast<int>(at & 7);
      last = (shift + V - 1) >> 3;
      const long left = wholes - static_cast<long>(at >> 3) - 1;
      whole = static_cast<int>(left < last ? left : last);
      const long first = static_cast<long>(at - shift) + min(whole, 0) * 8;  // (a row in the array's cut-short group)
      zgroup = instead ? static_cast<const T*>(instead) : zreq + first;
      qgroup = instead ? static_cast<const TQ*>(instead) : qreq + first;
    }
  }
  __device__ __forceinline__ int element(int gi, int e) const { return VEC ? gi * 8 + e : gi * 8 + e - shift; }
  __device__ __forceinline__ void load_raw(int gi, Raw8<T>& z) const {
    z.template load<VEC>(VEC ? zrow : zgroup, VEC ? gi : min(gi, max(whole, 0)));
  }
  __device__ __forceinline__ void load_raw_q(int gi, Raw8<TQ>& q) const {
    q.template load<VEC>(VEC ? qrow : qgroup, VEC ? gi : min(gi, max(whole, 0)));
  }
  // What the groups of the draft probabilities are read from.  Where they are not wanted, a load that is made all the
  // same reads group 0 of this: up to 32 bytes of the request's own logits (VEC: whole_groups() asks for that many), or
  // `somewhere`.
  __device__ __forceinline__ const TQ* q_source(bool wanted, const void* somewhere) const {
    return wanted ? (VEC ? qrow : qgroup) : static_cast<const TQ*>(VEC ? static_cast<const void*>(zreq) : somewhere);
  }
  // Requested here, widened where they are needed (see load).
  __device__ __forceinline__ void load(int gi, float (&z)[8], float (&q)[8]) const {
    Raw8<T> rz;
    load_raw(gi, rz);
    rz.widen_to(z);
    if (qrow && use_q) {
      Raw8<TQ> rq;
      load_raw_q(gi, rq);
      rq.widen_to(q);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) q[e] = 0.0f;
    }
  }
  template <typename E>
  __device__ __forceinline__ void reload(const E* row, int gi, float (&x)[8]) const {
#pragma unroll 1
    for (int e = 0; e < 8; ++e) {
      const float y = widen(row[min(max(element(gi, e), 0), V - 1)]);
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = k == e ? y : x[k];
    }
  }
  // The group the array ends in, which load() has not read: element by element.
  __device__ __forceinline__ bool cut_short() const { return !VEC && whole < last; }  // (the same for every lane)
  __device__ __forceinline__ void complete(int gi, float (&z)[8], float (&q)[8]) const {
    if (gi > whole) {
      reload(zrow, gi, z);
      if (qrow && use_q) reload(qrow, gi, q);
    }
  }
  // What of a group lies outside the row: no mass (z = -inf, q = 0).
  __device__ __forceinline__ void mask(int gi, float (&z)[8], float (&q)[8]) const {
    if (VEC || (gi != 0 && gi < last)) return;
    int v0 = element(gi, 0);
    asm volatile("" : "+v"(v0));  // (the masks stay in here: worked out ahead for every group they are 250 scalar registers)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool in = static_cast<unsigned int>(v0 + e) < static_cast<unsigned int>(V);
      z[e] = in ? z[e] : neg_inf();
      q[e] = in ? q[e] : 0.0f;
    }
  }
  // Both, behind the loads of a batch.
  __device__ __forceinline__ void trim(int gi, float (&z)[8], float (&q)[8]) const {
    if (__builtin_expect(cut_short(), 0)) complete(gi, z, q);
    mask(gi, z, q);
  }
  // f of a group's eight elements: as eval_f, the chain entries one after the other (one uniform branch for each
  // entry, not for each entry and element).
  __device__ __forceinline__ void f8(const float (&z)[8], const float (&q)[8], int gi, float (&f)[8]) const {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = __builtin_amdgcn_exp2f((z[e] - z1) * c) * inv_S;
    auto rejected = [&](int tok, float inv) {
      if (!(inv > 0.0f)) return;  // Z was 0: f left unchanged
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = fmaxf(f[e] - (qrow ? q[e] : (element(gi, e) == tok ? 1.0f : 0.0f)), 0.0f) * inv;
    };
#pragma unroll
    for (int j = 0; j < kChainRegs; ++j)
      if (j < ch.n) rejected(ch.rtok[j], ch.rinv[j]);
    for (int j = kChainRegs; j < ch.n; ++j) rejected(ch.tok[j], ch.inv_norm[j]);
  }
};
// Whether the walk takes its VEC form (host): whole rows of groups, arrays on 16-byte boundaries, and requests with 32
// bytes of logits at least -- one row of eight bf16 entries has 16, and where it is the array's last one the load in place of
// draft probabilities that are not wanted (q_source) would run past the array's end.
inline bool whole_groups(const void* logits, size_t elt, const void* dprobs, int N, int V) {
  return V % 8 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0 && reinterpret_cast<uintptr_t>(dprobs) % 16 == 0 &&
         static_cast<size_t>(N) * V * elt >= 32;
}
// Groups a row can touch.
__device__ __host__ __forceinline__ int row_groups(int V, bool vec) { return vec ? V / 8 : static_cast<int>((static_cast<long>(V) + 14) / 8); }

// A streamed pass: n steps, in step s a lane looks at group at(s) (any readable group where it has none).  Two batches
// of BATCH steps take turns, one in flight while the other is worked on, as they come from memory; a step's elements
// are widened when its turn comes.  No load stands under a condition: past the last step that step is asked
// for again and dropped.  (The kernel has 1024 threads, so 128 registers: with the draft probabilities two steps to a
// batch, without them four; half of that where groups have to be masked, for the size of the code.  What
// bounds a pass is the memory latency of a compute unit that streams alone: with one batch at a time, waited for
// and then worked on, seven thresholds on 16 trees of 60 nodes took 118 us per call and 128 chains with dense
// probabilities 73.3; now 98.8 and 70.5.)
template <int BATCH, bool Q, typename T, typename TQ, bool VEC, typename At, typename Body>
__device__ __forceinline__ void stream_steps(const RowView<T, TQ, VEC>& rv, int n, At at, Body body) {
  constexpr int NQ = Q ? BATCH : 1;
  Raw8<T> za[BATCH], zb[BATCH];
  Raw8<TQ> qa[NQ], qb[NQ];
  auto request = [&](Raw8<T>(&z)[BATCH], Raw8<TQ>(&q)[NQ], int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int gi = at(min(s0 + i, n - 1));
      rv.load_raw(gi, z[i]);
      if (Q) rv.load_raw_q(gi, q[i % NQ]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto work = [&](const Raw8<T>(&z)[BATCH], const Raw8<TQ>(&q)[NQ], int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      if (s0 + i >= n) continue;
      float x[8], y[8];
      z[i].widen_to(x);
      if (Q) q[i % NQ].widen_to(y);
      else {
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = 0.0f;
      }
      body(s0 + i, x, y);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  if (n <= 0) return;
  request(za, qa, 0);
  for (int s = 0; s < n; s += 2 * BATCH) {
    request(zb, qb, s + BATCH);
    work(za, qa, s);
    request(za, qa, s + 2 * BATCH);
    work(zb, qb, s + BATCH);
  }
}
template <typename T, typename TQ, bool VEC, typename At, typename Body>
__device__ __forceinline__ void stream_row(const RowView<T, TQ, VEC>& rv, int n, At at, Body body) {
  if (rv.qrow && rv.use_q) stream_steps<VEC ? 2 : 1, true>(rv, n, at, body);
  else stream_steps<VEC ? 4 : 2, false>(rv, n, at, body);
}

// This work-group's share of Z = sum_v max(0, f(v) - q_k(v)) over groups [g_begin, g_end):
// q_k dense, or one-hot at token x.
template <typename T, typename TQ, int NT, bool VEC>
__device__ __forceinline__ double residual_mass_slice(const RowView<T, TQ, VEC>& rv, int g_begin, int g_end, int x) {
  double part = 0.0;
  auto group = [&](int s) { return g_begin + static_cast<int>(threadIdx.x) + s * NT; };
  stream_row(rv, (g_end - g_begin + NT - 1) / NT, [&](int s) { return min(group(s), g_end - 1); },
             [&](int s, float(&z)[8], float(&q)[8]) __attribute__((always_inline)) {
               const int gi = group(s);
               if (gi < g_end) {
                 float f[8], acc = 0.0f;
                 rv.trim(gi, z, q);
                 rv.f8(z, q, gi, f);
#pragma unroll
                 for (int e = 0; e < 8; ++e) {
                   const float qk = rv.qrow ? q[e] : (rv.element(gi, e) == x ? 1.0f : 0.0f);
                   acc += fmaxf(f[e] - qk, 0.0f);
                 }
                 part += static_cast<double>(acc);
               }
             });
  return part;
}

// Prefix sums over the n <= kMaxTiles tile sums in LDS, by one wave: lane l owns the contiguous
// run of `per` tiles starting at l*per; the runs are summed in index order and scanned across the
// lanes.  Every lane ends with the same answers, and the total and the search use the same
// additions (any wave of the work-group may call these and obtains the same bits).
struct TilePrefix {
  double mine;  // sum of the lane's run
  double incl;  // sum of the runs of lanes 0..l
};
__device__ __forceinline__ TilePrefix tile_prefix(const double* sh_tile, int n, int per, int lane) {
  TilePrefix p;
  p.mine = 0.0;
  for (int i = 0; i < per; ++i) {
    const int t = lane * per + i;
    if (t < n) p.mine += sh_tile[t];
  }
  p.incl = wave_prefix_sum(p.mine);
  return p;
}
__device__ __forceinline__ double tile_total(const double* sh_tile, int n, int lane) {
  const int per = (n + kWave - 1) / kWave;
  return lane_value(tile_prefix(sh_tile, n, per, lane).incl, kWave - 1);
}
// The first tile whose inclusive prefix (on top of `before`) exceeds target, and the prefix in
// front of it; when rounding leaves none, the last tile with mass (tile 0 if there is none).
__device__ __forceinline__ void tile_find(const double* sh_tile, int n, int lane, double before, double target,
                                          int& tile, double& cum) {
  const int per = (n + kWave - 1) / kWave;
  const TilePrefix p = tile_prefix(sh_tile, n, per, lane);
  const double excl = before + (p.incl - p.mine);
  int my_last = -1;
  for (int i = 0; i < per; ++i) {
    const int t = lane * per + i;
    if (t < n && sh_tile[t] > 0.0) my_last = t;
  }
  const unsigned long long has = __ballot(my_last >= 0);
  const int last_tile = has != 0ull ? lane_value(my_last, 63 - __clzll(static_cast<long long>(has))) : 0;
  const unsigned long long hit = __ballot(before + p.incl > target);
  int found = -1;
  double front = 0.0;
  if (hit != 0ull) {
    const int hl = __ffsll(static_cast<long long>(hit)) - 1;
    if (lane == hl) {
      double run = excl;
      for (int i = 0; i < per && found < 0; ++i) {
        const int t = lane * per + i;
        if (t < n) {
          if (run + sh_tile[t] > target) { found = t; front = run; } else run += sh_tile[t];
        }
      }
    }
    found = lane_value(found, hl);
    front = lane_value(front, hl);
  }
  if (found < 0) {  // rounding: the last tile with mass, with the prefix in front of it
    found = last_tile;
    const int ol = found / per;
    double run = excl;
    for (int i = 0; i < per; ++i) {
      const int t = lane * per + i;
      if (t < found) run += sh_tile[t];
    }
    front = lane_value(run, ol);
  }
  tile = found;
  cum = front;
}

// A slice that is resident in a partner's registers, gone over from memory here because the partner has
// not arrived (see exchange_begin).  A rarely taken path: one group of eight at a time, so that it adds next
// to nothing to the registers of the walk around it; groups go to threads, and sums are formed, as in the
// owner's resident form.  (The streamed form of the tail needs no such twin: its own pass reads memory.)
template <typename T, typename TQ, int NT, bool VEC>
__device__ __forceinline__ double resident_mass_from_memory(const RowView<T, TQ, VEC>& rv, int gb, int ge, int x) {
  double part = 0.0;
#pragma unroll 1
  for (int gi = gb + static_cast<int>(threadIdx.x); gi < ge; gi += NT) {
    float z[8], q[8];
    rv.load(gi, z, q);
    rv.trim(gi, z, q);
    float f[8], acc = 0.0f;
    rv.f8(z, q, gi, f);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float qk = rv.qrow ? q[e] : (rv.element(gi, e) == x ? 1.0f : 0.0f);
      acc += fmaxf(f[e] - qk, 0.0f);
    }
    part += static_cast<double>(acc);
  }
  return part;
}
// Tile sums (a tile = a step of 64 groups, the steps dealt out to the waves in turn); returns their number.
template <typename T, typename TQ, int NT, int kRes, bool VEC>
__device__ __forceinline__ int resident_tiles_from_memory(const RowView<T, TQ, VEC>& rv, int gb, int ge, double* out) {
  constexpr int NW = NT / kWave;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int nst = (ge - gb + kWave - 1) / kWave;
#pragma unroll 1
  for (int i = 0; i < kRes; ++i) {
    const int s = i * NW + wave;
    if (s < nst) {  // wave-uniform
      const int gi = gb + i * NT + tid;
      float gs = 0.0f;
      if (gi < ge) {
        float z[8], q[8], f[8];
        rv.load(gi, z, q);
        rv.trim(gi, z, q);
        rv.f8(z, q, gi, f);
        gs = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
      }
      const double t = wave_sum(static_cast<double>(gs));
      if (lane == 0) out[s] = t;
    }
  }
  return nst;
}

// A work-group's slice of the vocabulary, in groups of eight elements (a multiple of 64 groups, so that the slices are made of
// whole wave steps).  (Worked out on the host: an integer division is 25 instructions.)
inline int walk_slice(int V, int G, bool vec) { return ((row_groups(V, vec) + G - 1) / G + kWave - 1) / kWave * kWave; }

constexpr float kClosedFormMinNorm = 0.1f; // one-hot residual: Z = 1 - f(x) is used when at least this
constexpr int kMaxResident = 3;            // groups of eight elements a thread can keep in registers

// Where the results go, read from the kernel's arguments again at every stage that writes some (LATE): ten addresses kept in scalar
// registers from the first write to the last were half of what a resident walk moved to vector lanes and back (81 -> 35
// registers).  One tree of 60 nodes x 151 936 19.19 -> 18.94 us per call, 16 trees with dense q 68.01 -> 67.65, 8 trees x
// 100 001 26.67 -> 26.10.  The streamed walk keeps them: 128 dense chains 69.04, read again 69.21.
// (The arguments are one TailArgs at the start of the kernel's argument segment.)
typedef const __attribute__((address_space(4))) TailArgs* LateArgs;
template <bool LATE>
__device__ __forceinline__ auto out_args(const TailArgs& a) {
  if constexpr (LATE) {
    unsigned long long at = reinterpret_cast<unsigned long long>(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(at));
    return reinterpret_cast<LateArgs>(at);
  } else {
    return &a;
  }
}

// RES: every slice is at most RES groups per thread and stays in registers (decided by the host from G and V), 0: it is
// streamed.  Two of them where they are enough -- few requests, or a small vocabulary -- carry two thirds of the
// loads, exponentials, registers and code of three, and the walk is bound by what a wave has to issue and to fetch: 8
// trees over 100 001 entries 28.0 -> 26.5 us per call, 3 over 3 001 with dense probabilities 21.2 -> 19.4, one tree of 60 nodes
// over 151 936 3 % at most.  One where one is enough and rows begin anywhere, which with two had become slower than
// loads of single elements in three, the masks being the more code: one row of 255 fp32 entries 11.6 us per call with single
// elements, 12.9 with two groups, 12.0 with one; 21 rows of 255 15.9, 16.5, 15.0; 960 rows of 13 19.5, 21.3, 19.0.
// VEC: every group of eight elements is whole and aligned (RowView).
// LANES: a tree of at most 64 nodes, a node per lane of every wave: the tests of all nodes against the plain softmax, and after every rejection those of
// the siblings that are left, are made at once, a node's children are one ballot, and there is no barrier before the first sum over the
// vocabulary.  (Larger trees keep theirs in LDS.)  us per call, dense q, in LDS and in lanes: 18 chains of 18 x 3 804 16.2 -> 14.4, 3 of 45 x 2 427 15.9 ->
// 13.6, 45 of 21 x 34 171 28.1 -> 26.2, 27 trees of 21 x 6 026 with seven thresholds 22.5 -> 20.8, 16 of 60 x 151 936 65.8 -> 65.2 and with seven thresholds
// 89.1 -> 87.8; geometric mean over 58 drawn calls 1.043.
// What a wave issues between two trips to memory is what the walk takes: a row with one partial result not merged, a rejected
// first child not tested again, leaves without a look for children, no barrier behind a node's first three rejections where they exchange nothing
// (chain_barrier), and in the draw the prefixes of the tile sums taken once, the last element with mass looked for only where it is
// wanted: 2 us a call, one tree of 60 nodes over 151 936 entries 20.0 -> 18.0, 21 chains of 13 over 32 000 25.7 -> 23.7 (on 16 trees with
// dense q, which are bound by the logits, no more than two runs differ by).
template <typename T, typename TQ, int RES, bool VEC, bool LANES>
__device__ __forceinline__ void tail_sampling_body(const TailArgs& a) {
  constexpr bool RESIDENT = RES > 0;
  constexpr int kResident = RESIDENT ? RES : 1;
  constexpr int NT = RESIDENT ? kSamplingThreads : kStreamingThreads;
  constexpr int NW = NT / kWave;
  __shared__ int16_t sh_par[MARS_MAX_NODES];     // parent of every node
  __shared__ int32_t sh_tok[MARS_MAX_NODES];     // draft token of every node
  __shared__ float sh_zx[MARS_MAX_NODES];        // logit of the node's token in its parent's row
  __shared__ float sh_qx[MARS_MAX_NODES];        // draft probability of the node's token (1 if one-hot)
  __shared__ int32_t sh_ctok[MARS_MAX_NODES];    // residual chain: rejected tokens
  __shared__ float sh_cinv[MARS_MAX_NODES];      // residual chain: 1/Z
  __shared__ mars_row_stat sh_st[MARS_MAX_NODES];  // merged row statistics of the request
  __shared__ double sh_red[NW];
  __shared__ double sh_part[kMaxGroupsPerRequest];
  __shared__ double sh_tile[kMaxTiles];
  __shared__ float sh_u[MARS_MAX_NODES + 1];     // the request's uniforms
  __shared__ double sh_tile2[kMaxTiles];         // tile sums of a partner's slice, when they have to be worked out here
  __shared__ unsigned int sh_missing;            // partners of the current exchange that have not arrived
  __shared__ int sh_bad;                         // validation bits of the request
  __shared__ int32_t sh_first[MARS_MAX_NODES];   // lowest-numbered child of every node (kNoChild: a leaf)
  __shared__ uint8_t sh_code0[MARS_MAX_NODES];   // decision of every node if it is the first child tested
  constexpr int32_t kNoChild = 0x7FFFFFFF;

  const int G = a.G;
  const int b = G == 1 ? blockIdx.x : blockIdx.y, g = G == 1 ? 0 : blockIdx.x;  // (the grid: see launch_sampling_tail)
  const int N = a.N, V = a.V;
  const size_t rb = static_cast<size_t>(b) * N;
  const int bd = a.B == a.Bd ? b : b % a.Bd;  // the request whose inputs this (possibly swept) request reads
  const size_t rd = static_cast<size_t>(bd) * N;
  const int tid = threadIdx.x;
  const int wave = tid / kWave, lane = tid % kWave;
  const T* __restrict__ zall = static_cast<const T*>(a.logits) + rd * static_cast<size_t>(V);
  const TQ* __restrict__ qall = a.dprobs ? static_cast<const TQ*>(a.dprobs) + rd * static_cast<size_t>(V) : nullptr;
  const bool dense = qall != nullptr;

  // Prologue, one node per thread.  It is one trip to memory: tree, tokens, the row's partial results,
  // uniforms, and the logit and draft probability of every node's token in its parent's row (which every
  // acceptance test needs, and which the row reduction of this call has gathered) all go out together.
  // Every work-group of the request does this for itself; they produce identical bits, and only the first
  // writes the caller's outputs.
  const int nwords = (N + kWave - 1) / kWave;
  const int ngroups = row_groups(V, VEC);
  const int slice = a.slice;
  const int g_begin = min(ngroups, g * slice), g_end = min(ngroups, g_begin + slice);
  // LANES, of node `lane`: parent (-2: no draft), token, uniform, draft probability, f(x) in the parent's row, decision; its own row's
  // statistics.
  // (In vector registers, also what is one number or one bit per node: scalar ones are what these kernels run out of.)
  int l_par = -2, l_tok = 0, l_code = 0, l_second = 0;  // (l_second: it is the runner-up of a low-margin row)
  float l_u = 0.0f, l_qx = 1.0f, l_f = 0.0f, u_draw = 0.0f;
  mars_row_stat l_st = {};
  if constexpr (LANES) {
    const bool live = lane < N;
    const size_t rl = rd + (live ? lane : 0);
    const float* __restrict__ ureq = a.u + static_cast<size_t>(bd) * (N + 1);
    const int par = a.par[rl];
    l_tok = a.tok[rl];
    l_u = ureq[live ? lane : 0];
    u_draw = ureq[N];
    const float theta = a.theta[b];
    float zx = 0.0f;
    if (a.gathered) {
      const float2 zq = a.gathered[rl];
      zx = zq.x; l_qx = zq.y;
    }
    if (a.splits <= kLaneParts) {
      l_st = lane_row<true>(a.partials + rl * a.splits, a.splits, a.c, a.ind, theta);
    } else {
      merge_rows_coop<NT, RESIDENT ? 8 : 4>(a.partials + rd * a.splits, N, a.splits, a.c, a.ind, [&](int) { return theta; },
                                            [&](int row, const mars_row_stat& st) { sh_st[row] = st; });
      __syncthreads();
      l_st = sh_st[live ? lane : 0];
    }
    if (g == 0 && wave == 0 && live && a.stats) a.stats[rb + lane] = l_st;
    const bool bad_tree = live && (lane == 0 ? par != -1 : par < 0 || par >= lane);
    const bool bad_token = live && lane > 0 && (l_tok < 0 || l_tok >= V);
    if (__any(bad_tree || bad_token)) {
      if (g == 0)
        write_rejected_request<NT>(a, b, __any(bad_tree) ? MARS_REQ_BAD_TREE : MARS_REQ_BAD_TOKEN, lane_value(l_st.id1, 0));
      return;
    }
    const bool node = live && lane > 0;
    const int p = node ? par : 0;
    if (node && !a.gathered) {  // behind the fused LM head nobody has gathered: a second trip to memory
      const size_t at = static_cast<size_t>(p) * V + l_tok;
      zx = widen(zall[at]);
      if (dense) l_qx = widen(qall[at]);
    }
    if (!node) l_qx = 1.0f;
    l_par = node ? par : -2;
    mars_row_stat above = {};  // of the parent's row
    above.z1 = __shfl(l_st.z1, p, kWave);
    above.sum_exp = __shfl(l_st.sum_exp, p, kWave);
    above.id2 = __shfl(l_st.relax_ok ? l_st.id2 : -1, p, kWave);
    above.relax_ok = 1;
    float fx;
    l_code = first_try(above, zx, l_qx, l_tok, l_u, a.c, fx);
    l_f = softmax_at(above, zx, a.c);
    l_second = l_tok == above.id2 ? 1 : 0;
    asm volatile("" : "+v"(u_draw));
  } else {
    constexpr int kPerThread = (MARS_MAX_NODES + NT - 1) / NT;
    const float theta = a.theta[b];
    const bool few = a.splits <= kFewParts;  // one thread merges a row (else sixteen lanes do)
    const float* __restrict__ ureq = a.u + static_cast<size_t>(bd) * (N + 1);
    int pr[kPerThread], tk[kPerThread];
    float zx[kPerThread], qx[kPerThread], uv[kPerThread];  // (zx, qx: gathered by the row reduction of this call)
    Partial pq[kPerThread][kFewParts];
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int i = tid + t * NT;
      pr[t] = -1; tk[t] = 0; uv[t] = 0.0f; zx[t] = 0.0f; qx[t] = 1.0f;
      if (t * NT < N && i < N) {
        pr[t] = a.par[rd + i];
        tk[t] = a.tok[rd + i];
        // (the streamed form is short of registers here: its partial results are requested further down)
        if (RESIDENT && few) load_partials_of_row(a.partials + (rd + i) * a.splits, a.splits, pq[t]);
        uv[t] = ureq[i];
        if (a.gathered) {
          const float2 zq = a.gathered[rd + i];
          zx[t] = zq.x; qx[t] = zq.y;
        }
      }
    }
    const float u_draw = tid == 0 ? ureq[N] : 0.0f;  // the uniform of the final draw
    const auto to = out_args<RESIDENT>(a);
    // (behind the requests: the barrier has nobody wait for them)
    if (tid == 0) sh_bad = 0;
    for (int i = tid; i < N; i += NT) sh_first[i] = kNoChild;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int i = tid + t * NT;
      if (t * NT < N && i < N) {
        const size_t r = rb + i;
        const int p = pr[t];
        const int x = tk[t];
        int bad = 0;
        if (i == 0) { if (p != -1) bad = 1; }
        else {
          if (p < 0 || p >= i) bad |= 1;
          if (x < 0 || x >= V) bad |= 2;
        }
        if (i == 0 || bad != 0) {  // (nothing was gathered for these)
          zx[t] = 0.0f; qx[t] = 1.0f;
        } else if (!a.gathered) {  // behind the fused LM head nobody has gathered: a second trip to memory
          const size_t at = static_cast<size_t>(p) * V + x;
          zx[t] = widen(zall[at]);
          if (dense) qx[t] = widen(qall[at]);
        }
        sh_par[i] = static_cast<int16_t>(p);
        sh_tok[i] = x;
        if (bad) atomicOr(&sh_bad, bad);
        else if (i > 0) atomicMin(&sh_first[p], i);
        if (g == 0) {
          to->mask[r] = i == 0 ? 1 : 0;
          to->path[r] = -1;
          if (to->dec) to->dec[r] = 0;
        }
      }
    }
    auto emit = [&](int row, const mars_row_stat& st) {
      sh_st[row] = st;
      if (g == 0) {
        if (to->stats) to->stats[rb + row] = st;
      }
    };
    if (few) {
#pragma unroll
      for (int t = 0; t < kPerThread; ++t) {
        const int i = tid + t * NT;
        if (t * NT < N && i < N) {
          if (!RESIDENT) load_partials_of_row(a.partials + (rd + i) * a.splits, a.splits, pq[t]);
          const mars_row_stat st = merge_row_few(pq[t], a.splits, a.c, a.ind, theta);
          sh_st[i] = st;
          if (g == 0) {
            if (to->stats) to->stats[rb + i] = st;
          }
        }
      }
    } else {
      merge_rows_coop<NT, RESIDENT ? 8 : 4>(a.partials + rd * a.splits, N, a.splits, a.c, a.ind, [&](int) { return theta; }, emit);
    }
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int i = tid + t * NT;
      if (t * NT < N && i < N) { sh_zx[i] = zx[t]; sh_qx[i] = qx[t]; sh_u[i] = uv[t]; }
    }
    if (tid == 0) sh_u[N] = u_draw;
    __syncthreads();
    if (sh_bad != 0) {
      if (g == 0) write_rejected_request<NT>(a, b, (sh_bad & 1) ? MARS_REQ_BAD_TREE : MARS_REQ_BAD_TOKEN, sh_st[0].id1);
      return;
    }
    // What the walk decides at a node it reaches is, for the node's first child, a function of the inputs
    // alone: taken here for all nodes at once, so that the walk follows accepted first children at the
    // price of two LDS reads each.
#pragma unroll
    for (int t = 0; t < kPerThread; ++t) {
      const int i = tid + t * NT;
      if (t * NT < N && i < N) {
        int code0 = 0;
        if (i > 0) {
          float fx;
          code0 = first_try(sh_st[pr[t]], zx[t], qx[t], tk[t], uv[t], a.c, fx);
        }
        sh_code0[i] = static_cast<uint8_t>(code0);
      }
    }
    __syncthreads();
  }

  // A slice of at most RES groups per thread stays in registers between the passes over
  // one node: f is then loaded and exponentiated once per visited node, every further
  // rejection at that node only updates it in place, and the final draw reads it where it is.
  // Thread t holds groups g_begin + i*NT + t; "step" s = i*NW + wave is 64 consecutive groups.
  constexpr bool resident = RESIDENT;
  const int nsteps = (g_end - g_begin + kWave - 1) / kWave;
  const float c = a.c;
  const auto walk_to = out_args<RESIDENT>(a);
  int cnode = 0, plen = 0, passes = 0, nexch = 0;
  float last_norm = 0.0f;
  bool pending_norm = false;  // the last rejection's normaliser is still to come out of the final pass
  RowView<T, TQ, VEC> rv;
  rv.V = V; rv.c = c;
  rv.request(static_cast<const T*>(a.logits), static_cast<const TQ*>(a.dprobs), rd * static_cast<size_t>(V),
             static_cast<size_t>(a.Bd) * N * static_cast<size_t>(V), a.partials);
  rv.ch.tok = sh_ctok; rv.ch.inv_norm = sh_cinv; rv.ch.n = 0;
  float fc[kResident][8], qv[kResident][8];  // resident slice: current f and the draft probabilities
  bool have = false;                          // fc holds the current f of this node's slice
  bool raw = false;                           // fc / qv hold the node's raw slice (logits, draft probabilities)
  int applied = 0;                            // chain entries already worked into fc

  // The loads of the resident slice, issued when a pass first needs it.  (Issuing them on arrival at every
  // node, in case a rejection follows, was tried: the next node's loads then have to wait for the registers
  // of the previous node's, and every accepted draft costs a trip to memory -- 86 instead of 80 us per pass.)
  // (With whole groups the loads are kept as they come until the slice is needed -- `widen_resident` -- so that
  // a request made ahead of time is not waited for where it is made.)
  Raw8<T> rz[kResident];
  Raw8<TQ> rq[kResident];
  bool rq_loaded = false;
  auto load_resident = [&]() {
    rq_loaded = rv.qrow && rv.use_q;
    // No load stands under a condition, per lane or per call: a lane past the end of its slice reads the
    // row's last group and throws it away, and when the draft probabilities are not wanted every lane reads
    // 32 bytes in their place: the first ones of the logits or of the partial results.  With a branch between two loads the compiler can no
    // longer count what is in flight and makes each wait for the one before (three trips to memory instead
    // of one); with a branch around them it copies what they return into the registers of the other path
    // right away, and waits for it there.
    const TQ* __restrict__ qsrc = rv.q_source(rq_loaded, a.partials + rd * a.splits);
#pragma unroll
    for (int i = 0; i < kResident; ++i) {
      int gi = min(g_begin + i * NT + tid, ngroups - 1);
      if (!VEC) gi = min(gi, max(rv.whole, 0));
      rz[i].template load<VEC>(VEC ? rv.zrow : rv.zgroup, gi);
      rq[i].template load<VEC>(qsrc, rq_loaded ? gi : 0);
    }
    raw = true;
    have = false;
  };
  auto widen_resident = [&]() {
#pragma unroll
    for (int i = 0; i < kResident; ++i) {
      const int gi = g_begin + i * NT + tid;
      if (gi < g_end) {
        rz[i].widen_to(fc[i]);
        if (rq_loaded) rq[i].widen_to(qv[i]);
      } else {  // nothing there: f = 0 and q = 0 contribute nothing
#pragma unroll
        for (int e = 0; e < 8; ++e) { fc[i][e] = neg_inf(); qv[i][e] = 0.0f; }
      }
      if (!rq_loaded) {
#pragma unroll
        for (int e = 0; e < 8; ++e) qv[i][e] = 0.0f;
      }
    }
    if (!VEC) {
      if (__builtin_expect(rv.cut_short(), 0)) {
#pragma unroll
        for (int i = 0; i < kResident; ++i) {
          const int gi = g_begin + i * NT + tid;
          if (gi < g_end) rv.complete(gi, fc[i], qv[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < kResident; ++i) {
        const int gi = g_begin + i * NT + tid;
        if (gi < g_end) rv.mask(gi, fc[i], qv[i]);
      }
    }
  };
  // Bring the resident slice up to date with the chain (turning the raw slice into f on first use).
  auto refresh_resident = [&]() {
    if (!have) {
      if (!raw) load_resident();
      widen_resident();
#pragma unroll
      for (int i = 0; i < kResident; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          fc[i][e] = __builtin_amdgcn_exp2f((fc[i][e] - rv.z1) * c) * rv.inv_S;  // softmax term (Eq. 3)
      raw = false;
      have = true;
      applied = 0;
    }
    for (int j = applied; j < rv.ch.n; ++j) {
      int tj = sh_ctok[j];
      float inv = sh_cinv[j];
#pragma unroll
      for (int r = 0; r < kChainRegs; ++r)
        if (r == j) { tj = rv.ch.rtok[r]; inv = rv.ch.rinv[r]; }
      if (inv > 0.0f) {
#pragma unroll
        for (int i = 0; i < kResident; ++i) {
          const int gi = g_begin + i * NT + tid;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float qj = dense ? qv[i][e] : (rv.element(gi, e) == tj ? 1.0f : 0.0f);
            fc[i][e] = fmaxf(fc[i][e] - qj, 0.0f) * inv;
          }
        }
      }
    }
    applied = rv.ch.n;
  };

  // Token x, f(x) = fx, is rejected at the current node; `more`: the node has further children.
  auto reject = [&](int x, float fx, bool more) __attribute__((always_inline)) {
    // Rejected: f <- max(0, f - q_k) / Z with Z = sum_v max(0, f(v) - q_k(v)).
    //  * With a one-hot q_k only the entry x changes and Z = 1 - f(x); that form is used while
    //    it is well conditioned.
    //  * After the node's last child nothing is tested against f any more: the division is
    //    left out (factor 1) and Z comes out of the final pass as the total of what is left.
    //  * Otherwise Z is summed over the row, every work-group of the request taking a slice.
    float inv;
    // (a barrier behind an exchange, whose staging arrays are used again, and where the chain asks for one)
    bool sync = chain_barrier(rv.ch.n);
    if (!dense && 1.0f - fx >= kClosedFormMinNorm) {
      last_norm = 1.0f - fx;
      inv = 1.0f / last_norm;
    } else if (!more) {
      pending_norm = true;
      inv = 1.0f;
    } else {
      sync = true;
      // This work-group's slice first, then (rarely) those of partners that have not arrived.  The
      // streamed form reads memory either way and runs one loop over "whose slice"; the resident form has
      // its own slice in registers and a lean pass over memory for the others, kept out of the way
      // behind the exchange (both forms are short of registers in different places).
      if (resident) {
        refresh_resident();
        double part = 0.0;
#pragma unroll
        for (int i = 0; i < kResident; ++i) {
          const int gi = g_begin + i * NT + tid;
          float acc = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float qk = dense ? qv[i][e] : (rv.element(gi, e) == x ? 1.0f : 0.0f);
            acc += fmaxf(fc[i][e] - qk, 0.0f);
          }
          part += static_cast<double>(acc);
        }
        part = block_sum<NT>(part, sh_red);
        unsigned int missing = exchange_begin<NT>(a, b, g, nexch++, part, sh_part, &sh_missing);
        while (missing != 0u) {
          const int who = __ffs(static_cast<int>(missing)) - 1;
          missing &= missing - 1u;
          const int gb = min(ngroups, who * slice), ge = min(ngroups, gb + slice);
          const double theirs = block_sum<NT>(resident_mass_from_memory<T, TQ, NT, VEC>(rv, gb, ge, x), sh_red);
          exchange_fill(sh_part, who, theirs);
          __syncthreads();  // (sh_red is free again)
        }
      } else {
        int who = g;
        unsigned int missing = 0u;
        for (;;) {
          const int gb = min(ngroups, who * slice), ge = min(ngroups, gb + slice);
          const double part = block_sum<NT>(residual_mass_slice<T, TQ, NT, VEC>(rv, gb, ge, x), sh_red);
          if (who == g) {
            missing = exchange_begin<NT>(a, b, g, nexch++, part, sh_part, &sh_missing);
          } else {
            exchange_fill(sh_part, who, part);
            __syncthreads();  // (sh_red is free again)
          }
          if (missing == 0u) break;
          who = __ffs(static_cast<int>(missing)) - 1;
          missing &= missing - 1u;
        }
      }
      const double Z = exchange_end(a, sh_part);
      last_norm = static_cast<float>(Z);
      inv = Z > 0.0 ? static_cast<float>(1.0 / Z) : 0.0f;  // 0: f is left as it is
    }
    if (tid == 0) { sh_ctok[rv.ch.n] = x; sh_cinv[rv.ch.n] = inv; }
#pragma unroll
    for (int j = 0; j < kChainRegs; ++j)
      if (j == rv.ch.n) { rv.ch.rtok[j] = x; rv.ch.rinv[j] = inv; }
    rv.ch.n += 1;
    passes += 1;
    if (sync) __syncthreads();
  };
  // Arrived at a node where the walk stops (leaf) or rejects its first child.
  auto arrive = [&](float z1, float sum_exp, bool leaf) __attribute__((always_inline)) {
    rv.row(cnode, dense);
    rv.z1 = z1; rv.inv_S = 1.0f / sum_exp;
    rv.use_q = dense && !leaf;  // a rejection pass subtracts q; nothing is rejected at a leaf
    rv.ch.n = 0;
    pending_norm = false;
    have = false;
    raw = false;
    applied = 0;
    // The walk stops here or rejects here: at a leaf the final draw reads this row, and a node whose first
    // child is rejected sees a pass over it either now (further children) or in the final draw, unless a later
    // child is accepted off a closed-form normaliser (one-hot draft: the request is then wasted, nothing
    // waits for it).  The row's slice is requested at once, so that its trip to memory runs beside the tests
    // that follow instead of behind them.  (Only here: a node that is merely passed through never asks for its row.)
    if (RESIDENT) load_resident();
  };

  int l_path = -1, l_on = lane == 0 ? 1 : 0;  // LANES: the path's node `lane`, whether node `lane` is on it
  if constexpr (LANES) {
    for (;;) {
      const unsigned long long kids = __ballot(l_par == cnode);
      const bool leaf = kids == 0ull;
      int k = leaf ? 0 : __ffsll(static_cast<long long>(kids)) - 1;
      bool accepted = !leaf && lane_value(l_code, k) != 0;
      if (!accepted) {
        arrive(lane_value(l_st.z1, cnode), lane_value(l_st.sum_exp, cnode), leaf);
        if (leaf) break;
        unsigned long long bits = kids;
        for (;;) {
          bits &= bits - 1ull;
          const int x = lane_value(l_tok, k);
          reject(x, lane_value(l_f, k), bits != 0ull);
          if (bits == 0ull) break;
          // f(x) and the tests of the children that are left, as eval_f and the loop below take them
          int jl = 0;
          float inv = 0.0f;
#pragma unroll
          for (int j = 0; j < kChainRegs; ++j)
            if (j + 1 == rv.ch.n) { inv = rv.ch.rinv[j]; jl = 1; }
          if (jl == 0) inv = sh_cinv[rv.ch.n - 1];
          const float left = fmaxf(l_f - (dense ? l_qx : l_tok == x ? 1.0f : 0.0f), 0.0f) * inv;
          l_f = l_par == cnode && inv > 0.0f ? left : l_f;
          k = __ffsll(static_cast<long long>(bits)) - 1;
          float acc;
          if (l_f == 0.0f) acc = 0.0f;
          else if (l_qx <= 0.0f) acc = 1.0f;
          else acc = fminf(1.0f, l_f / l_qx);
          const int code = l_second != 0 ? MARS_DEC_RELAXED : l_u < acc ? MARS_DEC_SAMPLED : 0;
          accepted = lane_value(code, k) != 0;
          if (accepted) {
            l_code = lane == k ? code : l_code;
            break;
          }
        }
        if (!accepted) break;
      }
      l_on = lane == k ? 1 : l_on;
      l_path = lane == plen ? k : l_path;
      cnode = k;
      plen += 1;
    }
    if (g == 0 && wave == 0) {  // (the committed tokens' padding and the token drawn last: below)
      const int committed = __shfl(l_tok, lane < plen ? l_path : 0, kWave);
      if (lane < N) {
        walk_to->mask[rb + lane] = static_cast<uint8_t>(l_on);
        walk_to->path[rb + lane] = l_path;
        if (walk_to->dec) walk_to->dec[rb + lane] = static_cast<uint8_t>(l_on != 0 && lane > 0 ? l_code : 0);
        if (walk_to->out_tok && lane < plen) walk_to->out_tok[rb + lane] = committed;
      }
    }
  } else
  for (;;) {
    const int k1 = __builtin_amdgcn_readfirstlane(sh_first[cnode]);
    const bool leaf = k1 >= N;
    {
      const int code0 = !leaf ? __builtin_amdgcn_readfirstlane(static_cast<int>(sh_code0[k1])) : 0;
      if (code0 != 0) {  // the first child is accepted: nothing else at this node matters
        if (tid == 0 && g == 0) {
          walk_to->mask[rb + k1] = 1;
          walk_to->path[rb + plen] = k1;
          if (walk_to->dec) walk_to->dec[rb + k1] = static_cast<uint8_t>(code0);
          if (walk_to->out_tok) walk_to->out_tok[rb + plen] = sh_tok[k1];
        }
        cnode = k1;
        plen += 1;
        continue;
      }
    }
    const mars_row_stat st = sh_st[cnode];
    arrive(st.z1, st.sum_exp, leaf);
    // The children of cnode as bit masks over the nodes (increasing node index = increasing bit), 64
    // nodes to a word.  Every wave forms the words for itself from the parents in LDS: no wave waits for
    // another one on the way down the tree.
    auto kids_word = [&](int wd) {
      const int i = wd * kWave + lane;
      return __ballot(i < N && i > cnode && sh_par[i] == cnode);
    };
    int accepted = -1;
    if (leaf) break;
    // The first child is rejected: sh_code0 says so.
    int k = k1, wd = k1 / kWave;
    unsigned long long bits = kids_word(wd) & (~1ull << (k1 % kWave));  // the children behind it
    for (;;) {
      bool more = bits != 0ull;          // does cnode have further children after k?
      for (int w2 = wd + 1; w2 < nwords && !more; ++w2) more = kids_word(w2) != 0ull;
      const int x = sh_tok[k];
      // Every thread takes the decision for itself from the same LDS-resident inputs (same
      // instructions, same bits): no broadcast and no barrier per tested child.
      int code = 0;
      float fx = 0.0f;
      if (rv.ch.n == 0) {
        fx = softmax_at(st, sh_zx[k], c);
      } else if (x == st.id2 && st.relax_ok) {
        code = MARS_DEC_RELAXED;  // runner-up in a low-margin row: accepted outright
      } else {
        const float qx = sh_qx[k];
        fx = eval_f(sh_zx[k], qx, x, st.z1, c, rv.inv_S, dense, rv.ch);
        // Eq. 1: accept with probability min(1, f(x)/q(x))
        float acc;
        if (fx == 0.0f) acc = 0.0f;
        else if (qx <= 0.0f) acc = 1.0f;
        else acc = fminf(1.0f, fx / qx);
        if (sh_u[k] < acc) code = MARS_DEC_SAMPLED;
      }
      if (code) {
        if (tid == 0 && g == 0) {
          walk_to->mask[rb + k] = 1;
          walk_to->path[rb + plen] = k;
          if (walk_to->dec) walk_to->dec[rb + k] = static_cast<uint8_t>(code);
          if (walk_to->out_tok) walk_to->out_tok[rb + plen] = x;
        }
        accepted = k;
        break;
      }
      reject(x, fx, more);
      while (bits == 0ull && wd + 1 < nwords) bits = kids_word(++wd);
      if (bits == 0ull) break;
      k = wd * kWave + __ffsll(static_cast<long long>(bits)) - 1;
      bits &= bits - 1;
    }
    if (accepted < 0) break;
    cnode = accepted;
    plen += 1;
  }

  // ---------------------------------------------------------------- inverse-CDF draw from f at cnode
  const auto draw_to = out_args<RESIDENT>(a);
  const int last_top1 = LANES ? lane_value(l_st.id1, cnode) : sh_st[cnode].id1;
  const float u_last = LANES ? u_draw : sh_u[N];
  // Without a rejection at this node f is the plain softmax: the draft distribution is not read.
  // (A resident slice that was loaded for a rejection already holds it.)
  rv.use_q = dense && rv.ch.n > 0;
  // Tiles of the slice, in vocabulary order.  Resident slice: a tile is one step (64 groups).
  // Otherwise wave w owns a contiguous run of steps and a tile is `rep` consecutive steps of it.
  const int steps_per_wave = (nsteps + NW - 1) / NW;
  const int rep = max(1, (steps_per_wave * NW + kMaxTiles - 1) / kMaxTiles);
  const int tiles_per_wave = (steps_per_wave + rep - 1) / rep;
  const int ntiles = resident ? nsteps : tiles_per_wave * NW;

  auto step_group = [&](int w, int sw) {  // streamed slice: group of this lane in step sw of wave w, -1 = none
    const int gi = g_begin + (w * steps_per_wave + sw) * kWave + lane;
    return (sw < steps_per_wave && gi < g_end) ? gi : -1;
  };
  auto group_sum = [&](const float (&z)[8], const float (&q)[8], int gi, float (&f)[8]) {
    rv.f8(z, q, gi, f);
    return ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
  };

  double total = 0.0, before = 0.0;
  int owner = 0;
  TilePrefix own = {0.0, 0.0};  // resident slice (at most one tile per lane): the tile sums and their prefixes
  static_assert(!RESIDENT || kResident * NW <= kWave, "one tile per lane");
  for (int attempt = 0; attempt < 2; ++attempt) {
    // This work-group's slice first (tile sums into sh_tile, which the search below reads), then (rarely)
    // those of partners that have not arrived (into sh_tile2); the two forms as above.
    if (resident) {
      refresh_resident();
#pragma unroll
      for (int i = 0; i < kResident; ++i) {
        const int s = i * NW + wave;
        if (s < nsteps) {  // wave-uniform
          const float gs = ((fc[i][0] + fc[i][1]) + (fc[i][2] + fc[i][3])) +
                           ((fc[i][4] + fc[i][5]) + (fc[i][6] + fc[i][7]));
          const double t = wave_sum(static_cast<double>(gs));
          if (lane == 0) sh_tile[s] = t;
        }
      }
      __syncthreads();
      // slice total = sum of its tiles, the last of the prefixes that the search below uses
      own.mine = lane < nsteps ? sh_tile[lane] : 0.0;
      own.incl = wave_prefix_sum(own.mine);
      unsigned int missing = exchange_begin<NT>(a, b, g, N + attempt, lane_value(own.incl, kWave - 1), sh_part, &sh_missing);
      while (missing != 0u) {
        const int who = __ffs(static_cast<int>(missing)) - 1;
        missing &= missing - 1u;
        const int gb = min(ngroups, who * slice), ge = min(ngroups, gb + slice);
        const int nt = resident_tiles_from_memory<T, TQ, NT, kResident, VEC>(rv, gb, ge, sh_tile2);
        __syncthreads();
        exchange_fill(sh_part, who, tile_total(sh_tile2, nt, lane));
        __syncthreads();  // (sh_tile2 may be filled again)
      }
    } else {
      int who = g;
      unsigned int missing = 0u;
      for (;;) {
        const int gb = min(ngroups, who * slice), ge = min(ngroups, gb + slice);
        double* tiles = who == g ? sh_tile : sh_tile2;
        // tile sums of a streamed slice
        const int spw = (((ge - gb + kWave - 1) / kWave) + NW - 1) / NW;  // steps per wave of this slice
        const int rp = max(1, (spw * NW + kMaxTiles - 1) / kMaxTiles);
        const int tpw = (spw + rp - 1) / rp;
        auto group_at = [&](int sw) { return gb + (wave * spw + sw) * kWave + lane; };  // this lane's in step sw of its wave
        double acc = 0.0;
        int tile_steps = 0, next_tile = wave * tpw;
        stream_row(rv, spw, [&](int sw) { const int gi = group_at(sw); return gi < ge ? gi : ngroups - 1; },
                   [&](int sw, float(&z)[8], float(&q)[8]) __attribute__((always_inline)) {
                     const int gi = group_at(sw);
                     if (gi < ge) {
                       float f[8];
                       rv.trim(gi, z, q);
                       acc += static_cast<double>(group_sum(z, q, gi, f));
                     }
                     if (++tile_steps == rp || sw + 1 == spw) {
                       const double t = wave_sum(acc);
                       if (lane == 0) tiles[next_tile] = t;
                       ++next_tile;
                       tile_steps = 0;
                       acc = 0.0;
                     }
                   });
        __syncthreads();
        const double slice_total = tile_total(tiles, tpw * NW, lane);
        if (who == g) {
          missing = exchange_begin<NT>(a, b, g, N + attempt, slice_total, sh_part, &sh_missing);
        } else {
          exchange_fill(sh_part, who, slice_total);
          __syncthreads();  // (sh_tile2 may be filled again)
        }
        if (missing == 0u) break;
        who = __ffs(static_cast<int>(missing)) - 1;
        missing &= missing - 1u;
      }
    }
    // Which work-group's slice holds the target?  The last one with mass if rounding leaves none.  Lane i
    // holds the total of work-group i and the prefix up to it; the grand total is the last prefix.
    if (G == 1) {
      total = sh_part[0];
    } else {
      const double pg = lane < G ? sh_part[lane] : 0.0;
      const double pincl = wave_prefix_sum(pg);
      total = lane_value(pincl, kWave - 1);
      const double target = static_cast<double>(u_last) * total;
      const unsigned long long hit = __ballot(lane < G && pincl > target);
      if (hit != 0ull) {
        owner = __ffsll(static_cast<long long>(hit)) - 1;
      } else {
        const unsigned long long mass = __ballot(lane < G && pg > 0.0);
        owner = mass != 0ull ? 63 - __clzll(static_cast<long long>(mass)) : 0;
      }
      before = lane_value(pincl - pg, owner);
    }
    if (!(pending_norm && total <= 0.0)) break;
    // The postponed normaliser turned out to be 0: that rejection leaves f as it was
    // (cannot happen in exact arithmetic).  Drop it from the chain and draw again.
    if (tid == 0) sh_cinv[rv.ch.n - 1] = 0.0f;
#pragma unroll
    for (int j = 0; j < kChainRegs; ++j)
      if (j == rv.ch.n - 1) rv.ch.rinv[j] = 0.0f;
    pending_norm = false;
    last_norm = 0.0f;
    have = false;
    raw = false;
    applied = 0;
    __syncthreads();
  }
  if (pending_norm) last_norm = static_cast<float>(total);
  const double target = static_cast<double>(u_last) * total;
  if (g == 0 && tid == 0) draw_to->len[b] = plen;
  // (The request's status was set to MARS_REQ_OK by the row reduction of this call.)
  // V_out (Alg. 1): the accepted drafts were written as they were accepted; the first work-group
  // pads behind the slot of the final token, which the work-group that draws it fills in.  (No
  // address is written by two work-groups.)
  if (g == 0 && draw_to->out_tok) {
    for (int j = plen + 1 + tid; j < N; j += NT) draw_to->out_tok[rb + j] = -1;
    if (tid == 0) draw_to->out_len[b] = plen + 1;
  }
  if (g != owner) return;

  // The owning work-group locates the tile (every wave does, from the same LDS values).
  int tile = -1;
  double cum = before;
  if (total > 0.0) {
    if (resident) {  // as tile_find, a tile per lane
      const double front = before + (own.incl - own.mine);
      const unsigned long long hit = __ballot(lane < nsteps && before + own.incl > target);
      if (hit != 0ull) {
        tile = __ffsll(static_cast<long long>(hit)) - 1;
      } else {
        const unsigned long long has = __ballot(own.mine > 0.0);
        tile = has != 0ull ? 63 - __clzll(static_cast<long long>(has)) : 0;
      }
      cum = lane_value(front, tile);
    } else {
      tile_find(sh_tile, ntiles, lane, before, target, tile, cum);
    }
  }
  // One wave finishes: the one holding the tile in registers, or wave 0 re-reading it.
  const int finder = (resident && tile >= 0) ? tile % NW : 0;
  if (wave != finder) return;

  int pick = -1;
  float pick_f = 0.0f;
  if (total > 0.0) {
    const int tw = resident ? 0 : tile / tiles_per_wave, ts = resident ? 0 : (tile % tiles_per_wave) * rep;
    const int nrep = resident ? 1 : rep;
    int last_pos_v = -1;
    float last_pos_f = 0.0f;
    for (int r = 0; r < nrep && pick < 0; ++r) {
      int gi;
      float f[8];
      float gs = 0.0f;
      if (resident) {
        const int ii = tile / NW;
        gi = g_begin + ii * NT + tid;
        if (gi >= g_end) gi = -1;
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = 0.0f;
#pragma unroll
        for (int i = 0; i < kResident; ++i)
          if (i == ii) {
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = fc[i][e];
          }
        gs = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
      } else {
        gi = step_group(tw, ts + r);
        if (gi >= 0) {
          float z[8], q[8];
          rv.load(gi, z, q);
          rv.trim(gi, z, q);
          gs = group_sum(z, q, gi, f);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) f[e] = 0.0f;
        }
      }
      const double gincl = wave_prefix_sum(static_cast<double>(gs));
      const unsigned long long hit = __ballot(cum + gincl > target);
      // the last element with mass, in case rounding leaves no step above the target
      auto remember_last = [&]() {
        int my_last = -1;
#pragma unroll
        for (int e = 0; e < 8; ++e) if (f[e] > 0.0f) my_last = e;
        const unsigned long long has = __ballot(my_last >= 0);
        if (has != 0ull) {
          const int hl = 63 - __clzll(static_cast<long long>(has));
          const int le = lane_value(my_last, hl);
          float fv = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) if (e == my_last) fv = f[e];
          last_pos_f = lane_value(fv, hl);
          last_pos_v = rv.element(lane_value(gi, hl), le);
        }
      };
      if (hit != 0ull) {
        const int hl = __ffsll(static_cast<long long>(hit)) - 1;
        double run = cum + lane_value(gincl - static_cast<double>(gs), hl);
        int pe = -1;
        float pf = 0.0f;
        if (lane == hl) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            if (pe < 0) {
              run += static_cast<double>(f[e]);
              if (run > target) { pe = e; pf = f[e]; }
            }
          }
        }
        pe = lane_value(pe, hl);
        if (pe >= 0) {
          pick_f = lane_value(pf, hl);
          pick = rv.element(lane_value(gi, hl), pe);
        } else {  // rounding left no step above the target inside the lane: last element with mass
          remember_last();
          pick = last_pos_v; pick_f = last_pos_f;
          break;
        }
      } else {
        remember_last();
        cum += lane_value(gincl, kWave - 1);
      }
    }
    if (pick < 0) { pick = last_pos_v; pick_f = last_pos_f; }
  }
  if (pick < 0) { pick = last_top1; pick_f = 0.0f; }  // degenerate: no mass anywhere
  if (lane == 0) {
    draw_to->bonus[b] = pick;
    if (draw_to->out_tok) draw_to->out_tok[rb + plen] = pick;
    if (draw_to->diag) {
      mars_req_diag dg;
      dg.bonus_prob = total > 0.0 ? static_cast<float>(static_cast<double>(pick_f) / total) : 0.0f;
      dg.last_residual_norm = last_norm;
      dg.residual_passes = passes;
      dg.last_node = cnode;
      draw_to->diag[b] = dg;
    }
  }
}

template <typename T, typename TQ, int RES, bool VEC, bool LANES>
__global__ __launch_bounds__(kSamplingThreads) void tail_sampling_resident_kernel(TailArgs a) {
  tail_sampling_body<T, TQ, RES, VEC, LANES>(a);
}
template <typename T, typename TQ, bool VEC, bool LANES>
__global__ __launch_bounds__(kStreamingThreads) void tail_sampling_streamed_kernel(TailArgs a) {
  tail_sampling_body<T, TQ, 0, VEC, LANES>(a);
}

// ---------------------------------------------------------------- cache rows that stay
// After the walk: the rows of the root and of the accepted nodes of every request, as flat row
// numbers bd*N + node, request by request in path order ("standard rollback" of Sec. 3.4 keeps
// exactly these), with the exclusive prefix sums of their counts.  One work-group per set of Bd
// requests (per threshold of a sweep); unused entries of keep_rows are -1.
//
// The kernel is one trip to memory: the first AHEAD path entries of a request go out with its length, before
// anybody knows how many of them count (read one after the other behind the length they cost a trip each: 64
// chains of eight drafts took 33.9 us per call, now 33.0; two of six 13.8, now 12.4).  Where nothing is accepted they cost 0.1-0.2 us
// in vain; requests of a single node have no path to read: AHEAD = 0 (300 of them 13.2 us per call with eight, 12.8).
constexpr int kKeepThreads = 256;
constexpr int kKeepAhead = 8;
template <int AHEAD>
__global__ __launch_bounds__(kKeepThreads) void compact_keep_kernel(const int32_t* __restrict__ out_len,
                                                                    const int32_t* __restrict__ path, int Bd, int N,
                                                                    int32_t* __restrict__ keep_rows,
                                                                    int32_t* __restrict__ keep_offsets) {
  constexpr int NT = kKeepThreads;
  __shared__ int sh_wave[NT / kWave];
  __shared__ int sh_carry;
  const int k = blockIdx.x;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int32_t* len = out_len + static_cast<size_t>(k) * Bd;
  const int32_t* pth = path + static_cast<size_t>(k) * Bd * N;
  int32_t* rows = keep_rows + static_cast<size_t>(k) * Bd * N;
  int32_t* offs = keep_offsets + static_cast<size_t>(k) * (Bd + 1);
  if (tid == 0) sh_carry = 0;
  __syncthreads();
  for (int b0 = 0; b0 < Bd; b0 += NT) {
    const int b = b0 + tid;
    const int mine = b < Bd ? len[b] : 0;
    int ahead[AHEAD ? AHEAD : 1];
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) ahead[j] = pth[static_cast<size_t>(min(b, Bd - 1)) * N + min(j, N - 1)];
    // inclusive scan inside the wave, then across the waves of the work-group
    int incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int o = __shfl_up(incl, d, kWave);
      if (lane >= d) incl += o;
    }
    if (lane == kWave - 1) sh_wave[wave] = incl;
    __syncthreads();
    int before = sh_carry;
    for (int w = 0; w < wave; ++w) before += sh_wave[w];
    const int start = before + incl - mine;
    if (b < Bd) {
      offs[b] = start;
      rows[start] = b * N;  // the root's row
#pragma unroll
      for (int j = 0; j < AHEAD; ++j)
        if (j + 1 < mine) rows[start + j + 1] = b * N + ahead[j];
      for (int j = AHEAD + 1; j < mine; ++j) rows[start + j] = b * N + pth[static_cast<size_t>(b) * N + j - 1];
    }
    __syncthreads();
    if (tid == NT - 1) sh_carry = before + incl;
    __syncthreads();
  }
  const int total = sh_carry;
  if (tid == 0) offs[Bd] = total;
  for (int i = total + tid; i < Bd * N; i += NT) rows[i] = -1;
}

}  // namespace mars
