// The sampling walk where the draft model's distribution is not kept: every draft token is a one-hot q (Eq. 1 accepts it
// with probability f(x), a rejection takes x out of f and divides by what is left).  One work-group per request, trees
// of at most 64 nodes.
//
// Nothing here goes over a row: a rejection changes one entry, so what the walk needs of a row is its largest two and its sum
// (which the row reduction leaves), the logits of the draft tokens (gathered on the way), and for the token drawn last
// the sums of the row's chunks (chunks.h) and the one chunk that the draw falls into, 16 384 entries as a rule.
//
// Every wave holds the whole tree, a node per lane, and does everything but the last step for itself, without LDS traffic
// between waves and without a barrier: the tests of all nodes are made at once (a node's test depends on the inputs and on its
// earlier siblings alone), and the walk is a few scalar instructions per accepted draft.
//
// What bounds it: three trips to memory one behind the other (the tree, the sums, the chunk: 1.4, 0.5 and 0.8 us) and the issue of
// single waves in between, 9-12 us in all; it was a pass over the row's entries by every request's work-groups for the draw, and an exchange
// of their sums.  That pass is quick while a request has so many work-groups that each keeps its slice in registers, so these calls stay with it
// (mars.hip: onehot_form).  us, that walk and this one: 256 trees of 26 x 151 936 fp32 (a work-group per request read 600 KB) 59 -> 14-17 for the
// kernel alone, 648 -> 633 for the call; 64 chains of 6 x 151 936 bf16 38 -> 34, 128 of 7 66 -> 58.  With the tests, the walk and the draw in LDS and
// behind barriers, as in tail_sampling_body, the same method took 25 us on the first.
#pragma once

#include "chunks.h"
#include "tail.h"

namespace mars {

constexpr int kOneHotNodes = kWave;
constexpr int kOneHotThreads = 512;
constexpr int kPageEntries = 32;   // the draw looks at a row, or at a chunk, in pages of this many entries per thread (48: no gain)
// The sum of a chunk less a token's own term is a difference of fp32 sums.  If the token holds more than this share of what is left of the row, the
// part of the chunk that it was summed with is summed again without it.
constexpr double kTakenShare = 0.25;

// ROW: a vocabulary of one page (of 512 threads up to 16 368 entries, of 1 024 up to 32 752).  The row itself is read where the walk stops,
// one trip instead of those to the sums and to a chunk, rejected tokens are left out where the terms are formed, and the row reduction
// leaves no sums of chunks.  us per call, the walk that goes over the row by all of a request's work-groups / by chunks / this one: 30 trees of 32 x 3 458
// bf16 19.5 / 23.3 / 19.7, one of 19 x 3 645 13.8 / 16.2 / 11.9, 6 of 63 x 6 940 19.1 / 16.9 / 13.8, 52 of 15 x 4 742 fp32 20.4 / 20.2 / 16.2, 23 of
// 37 x 32 000 bf16 25.0 / 25.2 / 22.3, 4 of 34 x 32 000 19.6 / 16.8 / 14.9; 33 of 12 x 32 000 20.2 / 21.0 / 21.2, and in fp32 10 chains of 13 x 32 000 16.7
// / 17.7 / 16.9.
constexpr int row_entries(int threads) { return threads * kPageEntries - 16; }  // (loose elements are a vector in front and one behind)
template <typename T, bool RAGGED, bool ROW, int NT>
__global__ __launch_bounds__(NT, NT > 512 ? 4 : RAGGED || ROW ? 2 : 4) void tail_onehot_kernel(TailArgs a) {
  constexpr int NW = NT / kWave;
  constexpr int EPV = 16 / sizeof(T), PV = kPageEntries / EPV;  // entries of a vector, vectors per thread and page
  constexpr int TILES = (PV * NW + kWave - 1) / kWave;  // of a page, per lane
  static_assert(TILES <= 2, "one tile per lane, or two");
  __shared__ mars_row_stat sh_st[kOneHotNodes];               // many partial results per row: the merged statistics
  __shared__ unsigned long long sh_kids[NW][kOneHotNodes];    // children of every node, a copy per wave
  __shared__ double sh_tile[2][PV * NW];                      // sums of a page's tiles: 64 vectors each
  __shared__ double sh_piece[2][NW];                          // sums of a piece that is summed again, one per wave

  const int b = blockIdx.x;
  const int N = a.N, V = a.V;
  const size_t rb = static_cast<size_t>(b) * N;
  const int bd = a.B == a.Bd ? b : b % a.Bd;  // the request whose inputs this (possibly swept) request reads
  const size_t rd = static_cast<size_t>(bd) * N;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const T* __restrict__ zall = static_cast<const T*>(a.logits) + rd * static_cast<size_t>(V);
  const float c = a.c;

  // ---------------------------------------------------------------- the tree, a node per lane: one trip to memory
  const bool live = lane < N;
  const size_t rl = rd + (live ? lane : 0);
  const int par = a.par[rl], tok = a.tok[rl];
  const float u = a.u[static_cast<size_t>(bd) * (N + 1) + (live ? lane : N)];
  const float u_draw = a.u[static_cast<size_t>(bd) * (N + 1) + N];
  const float theta = a.theta[b];
  float zx = 0.0f;
  if (!ROW || a.gathered) zx = a.gathered[rl].x;
  mars_row_stat st;
  if (a.splits <= kLaneParts) {
    st = lane_row<true>(a.partials + rl * a.splits, a.splits, c, a.ind, theta);
  } else {
    merge_rows_coop<NT, 4>(a.partials + rd * a.splits, N, a.splits, c, a.ind, [&](int) { return theta; },
                           [&](int row, const mars_row_stat& s) { sh_st[row] = s; });
    __syncthreads();
    st = sh_st[live ? lane : 0];
  }
  if (wave == 0 && live && a.stats) a.stats[rb + lane] = st;
  const bool bad_tree = live && (lane == 0 ? par != -1 : par < 0 || par >= lane);
  const bool bad_token = live && lane > 0 && (tok < 0 || tok >= V);
  if (__any(bad_tree || bad_token)) {
    write_rejected_request<NT>(a, b, __any(bad_tree) ? MARS_REQ_BAD_TREE : MARS_REQ_BAD_TOKEN, lane_value(st.id1, 0));
    return;
  }
  const bool node = live && lane > 0;  // (the root is no draft)
  if (ROW && !a.gathered && node) zx = widen(zall[static_cast<size_t>(par) * V + tok]);  // behind the fused LM head: a second trip
  const int p = node ? par : 0;
  // (LDS operations of a wave are performed in order; the fences keep the compiler's order)
  sh_kids[wave][lane] = 0ull;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (node) atomicOr(&sh_kids[wave][p], 1ull << lane);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const unsigned long long kids = sh_kids[wave][lane], family = sh_kids[wave][p];
  const unsigned long long older = node ? family & ((1ull << lane) - 1ull) : 0ull;  // its earlier siblings
  // f(x) in the parent's row before any rejection (Eq. 3), and whether x is the runner-up of a low-margin row
  const float f0 = __builtin_amdgcn_exp2f((zx - __shfl(st.z1, p, kWave)) * c) * __shfl(1.0f / st.sum_exp, p, kWave);
  const int second = __shfl(st.relax_ok ? st.id2 : -1, p, kWave);
  const bool runner_up = node && tok == second;

  // ---------------------------------------------------------------- decisions, walk, and the sums of the row it stops at
  float norm = -1.0f;  // Z of this node's rejection where it had to be summed (0: f was left as it was)
  float f;             // f(x) when the node is tested
  int code = 0, cnode = 0, plen = 0, passes = 0, path = -1;
  float last_norm = 0.0f;
  unsigned long long visited = 1ull;
  const T* __restrict__ rowp = zall;
  int head = 0, nvec = 0, tail = 0;
  float R = 0.0f, z1 = 0.0f;
  unsigned long long gone = 0ull;  // nodes whose tokens are out of f at cnode
  double total = 0.0, mass = 0.0;  // (mass: lane l's of chunk l)
  Vec<T, EPV> raw[PV];             // a page of the row as it lies in memory, the terms of its entries, of its vectors
  float e[PV][EPV], g[PV];
  double tile_first = 0.0, tile_sum = 0.0, tile_incl = 0.0;  // lane l: of the first of its tiles, of its tiles, of all up to them
  float2 part[kChunkWaves];        // what the lane's chunk was summed in: the eight waves'
  float low[kChunkWaves];          // and what the rounding of these has left over
  const ChunkSpec spec = a.chunks;
  const int nchunks = spec.items * spec.slots;
  int turn = 0;
  auto vector_of = [&](int v) { return RAGGED && v < head ? -1 : (v - head) / EPV; };
  // Chunk of an entry, the piece of it that the entry was summed with: a wave's vectors.
  struct Place { int chunk, piece; };
  Place at = {0, 0};                // of this node's token, if it is out of f
  unsigned long long redone = 0ull;  // nodes whose tokens' pieces have been summed again
  auto place_of = [&](int v) {
    int vec = vector_of(v);
    asm volatile("" : "+v"(vec));  // (worked out where it is wanted, not ahead for every lane)
    Place to = {0, 0};  // (loose elements: the first wave's)
    if (RAGGED && vec >= nvec) {
      const int first = min(nvec, (spec.items - 1) * spec.vps);
      to.chunk = (spec.items - 1) * spec.slots + chunk_last(spec, nvec - first);
    } else if (!RAGGED || vec >= 0) {
      to.chunk = chunk_of(spec, nvec, vec);
      to.piece = (vec - chunk_range(spec, nvec, to.chunk).begin) / kWave % kChunkWaves;
    }
    return to;
  };
  // (far below z1 the rounding of z*c - R would show: the exponent's integer part is taken exactly)
  auto precise = [&](float x) {
    const float n = __builtin_rintf(x * c);
    return __builtin_ldexpf(__builtin_amdgcn_exp2f(__builtin_fmaf(x, c, -n)), static_cast<int>(fmaxf(n - R, -1000.0f)));
  };
  auto scaled = [&](double s, float ref) {
    return s > 0.0 ? ldexp(s, static_cast<int>(fmaxf(ref - R, -1000.0f))) : 0.0;
  };
  auto sum_of = [](float high, float left) { return static_cast<double>(high) + static_cast<double>(left); };
  // (ROW: against the row's largest logit, whose term is 1 then; else against 2^R, as the sums)
  auto term_of = [&](float x) {
    return __builtin_amdgcn_exp2f(ROW ? (x - z1) * c : __builtin_fmaf(x, c, -R));
  };
  // The page from vector `page` on of vectors [range.begin, range.end) and, as a vector in front of the row's first and one behind its
  // last, the loose elements.
  // `beside` is done while the page is on its way.
  auto read_page = [&](int page, const ChunkRange& range, bool front, bool back, auto beside) __attribute__((always_inline)) {
    const T* __restrict__ vecp = rowp + head;
    const int begin = front ? -1 : range.begin, end = back ? nvec + 1 : range.end;
    if (range.end > range.begin) {
#pragma unroll
      for (int m = 0; m < PV; ++m)
        raw[m].load(vecp, static_cast<unsigned int>(min(max(page + m * NT + tid, range.begin), range.end - 1)));
    } else {
#pragma unroll
      for (int m = 0; m < PV; ++m) raw[m].fill_neg_inf();
    }
    __builtin_amdgcn_sched_barrier(0);
    beside();
#pragma unroll
    for (int m = 0; m < PV; ++m) {
      const int vec = page + m * NT + tid;
      const bool in = vec >= range.begin && vec < range.end;
#pragma unroll
      for (int n = 0; n < EPV; ++n) e[m][n] = 0.0f;
      if (page + m * NT + wave * kWave >= range.end) continue;
#pragma unroll
      for (int n = 0; n < EPV; ++n) {
        const float t = term_of(raw[m].get(n));
        e[m][n] = in ? t : 0.0f;
      }
    }
    if (front || back) {
#pragma unroll
      for (int n = 0; n < EPV; ++n) {
        const int vf = head - EPV + n, vb = head + nvec * EPV + n;
        const float ef = vf >= 0 ? term_of(widen(rowp[max(vf, 0)])) : 0.0f;
        const float eb = vb < V ? term_of(widen(rowp[min(vb, V - 1)])) : 0.0f;
#pragma unroll
        for (int m = 0; m < PV; ++m) {
          const int vec = page + m * NT + tid;
          if (front && vec == begin) e[m][n] = ef;
          if (back && vec == end - 1) e[m][n] = eb;
        }
      }
    }
    for (unsigned long long m = gone; m != 0ull; m &= m - 1ull) {
      const int x = lane_value(tok, __ffsll(static_cast<long long>(m)) - 1), vec = vector_of(x), at = vec - page;
      if (at < 0 || at >= PV * NT || tid != at % NT) continue;
      const int flat = at / NT * EPV + (x - head - vec * EPV);
#pragma unroll
      for (int i = 0; i < PV; ++i)
#pragma unroll
        for (int n = 0; n < EPV; ++n) e[i][n] = i * EPV + n == flat ? 0.0f : e[i][n];
    }
#pragma unroll
    for (int m = 0; m < PV; ++m) {
      g[m] = (e[m][0] + e[m][1]) + (e[m][2] + e[m][3]);
      if (EPV == 8) g[m] += (e[m][EPV - 4] + e[m][EPV - 3]) + (e[m][EPV - 2] + e[m][EPV - 1]);
      double t = 0.0;
      if (page + m * NT + wave * kWave < end) t = wave_sum(static_cast<double>(g[m]));
      if (lane == 0) sh_tile[turn][m * NW + wave] = t;
    }
    __syncthreads();
    tile_first = lane < PV * NW ? sh_tile[turn][lane * TILES] : 0.0;
    tile_sum = TILES == 2 ? tile_first + sh_tile[turn][lane * TILES + 1] : tile_first;
    tile_incl = wave_prefix_sum(tile_sum);
    turn ^= 1;
  };
  for (;;) {
    // The tests of all nodes, in rounds: in round r a node takes its r-th sibling's rejection into its f.  With a one-hot q
    // that is a division by Z = 1 - f(x), where that is not a small difference.
    f = f0;
    bool blocked = false;
    for (unsigned long long m = older; __any(m != 0ull);) {
      const int j = m != 0ull ? __ffsll(static_cast<long long>(m)) - 1 : lane;
      const float fj = __shfl(f, j, kWave), nj = __shfl(norm, j, kWave);
      const int tj = __shfl(tok, j, kWave);
      const float z = nj >= 0.0f ? nj : 1.0f - fj;
      if (m != 0ull) {
        blocked |= nj < 0.0f && !(z >= kClosedFormMinNorm);
        const float g = (tok == tj ? 0.0f : f) * (1.0f / z);
        f = z > 0.0f ? g : f;
      }
      m &= m - 1ull;
    }
    code = !node ? 0 : runner_up ? MARS_DEC_RELAXED : u < fminf(1.0f, f) ? MARS_DEC_SAMPLED : 0;
    const float z_own = norm >= 0.0f ? norm : 1.0f - f;
    const unsigned long long taken = __ballot(code != 0 && !blocked), unknown = __ballot(blocked);
    // The walk: the first child that is accepted.
    cnode = 0; plen = 0; passes = 0; path = -1; last_norm = 0.0f; visited = 1ull;
    unsigned long long here;
    auto kids_of = [&](int n) {
      return (static_cast<unsigned long long>(static_cast<unsigned int>(lane_value(static_cast<int>(kids >> 32), n))) << 32) |
             static_cast<unsigned int>(lane_value(static_cast<int>(kids), n));
    };
    auto last_of = [](unsigned long long m) { return 63 - __clzll(static_cast<long long>(m)); };
    for (;;) {
      here = kids_of(cnode);
      const unsigned long long yes = here & taken;
      if (yes == 0ull) break;
      const int k = __ffsll(static_cast<long long>(yes)) - 1;
      const unsigned long long rejected = here & ((1ull << k) - 1ull);
      passes += __popcll(rejected);
      if (rejected != 0ull) last_norm = lane_value(z_own, last_of(rejected));
      path = lane == plen ? k : path;
      visited |= 1ull << k;
      plen += 1;
      cnode = k;
    }
    // All its children are rejected, or one whose Z has to be summed: then the later ones wait for it.
    const unsigned long long wait = here & unknown;
    const bool draw = wait == 0ull;
    const unsigned long long out = draw ? here : here & ((wait & (0ull - wait)) - 1ull);
    const int last = out != 0ull ? last_of(out) : 0;
    passes += __popcll(out);
    gone = out & __ballot(norm != 0.0f);
    const float z_last = lane_value(z_own, last), norm_last = lane_value(norm, last);
    const bool summed = out != 0ull && norm_last < 0.0f && !(z_last >= kClosedFormMinNorm);  // Z comes out of the sums below
    if (out != 0ull && !summed) last_norm = z_last;

    // The sums of the row's chunks against 2^R, lane l's of chunk l.
    rowp = zall + static_cast<size_t>(cnode) * V;
    head = RAGGED ? min(V, static_cast<int>((16u - (reinterpret_cast<uintptr_t>(rowp) & 15u)) % 16u / sizeof(T))) : 0;
    nvec = (V - head) / EPV;
    tail = RAGGED ? V - head - nvec * EPV : 0;
    z1 = lane_value(st.z1, cnode);
    R = __builtin_ceilf(z1 * c);  // (an integer, as the references of the sums)
    if constexpr (ROW) {
      read_page(head > 0 ? -1 : 0, {0, nvec}, head > 0, tail > 0, [] {});
      total = lane_value(tile_incl, kWave - 1);
      if (!summed) break;
      if (!(total > 0.0)) {  // nothing is left without it: f stays as it was
        norm = lane == last ? 0.0f : norm;
        continue;
      }
      double z = total / static_cast<double>(lane_value(st.sum_exp, cnode));
      for (unsigned long long m = gone & ~(1ull << last); m != 0ull; m &= m - 1ull)
        z /= static_cast<double>(lane_value(z_own, __ffsll(static_cast<long long>(m)) - 1));
      if (!draw) {
        norm = lane == last ? static_cast<float>(z) : norm;
        continue;
      }
      last_norm = static_cast<float>(z);
      break;
    }
    const size_t first = (rd + cnode) * nchunks * kChunkWaves;
    const float2* __restrict__ table = a.table + first;
    const float* __restrict__ table_low = a.table_low + first;
    const int mine_at = min(lane, nchunks - 1) * kChunkWaves;
    const float4* __restrict__ t = reinterpret_cast<const float4*>(table + mine_at);
    const float4* __restrict__ tl = reinterpret_cast<const float4*>(table_low + mine_at);
#pragma unroll
    for (int w = 0; w < kChunkWaves; w += 2) {
      const float4 q = t[w / 2];
      part[w] = make_float2(q.x, q.y);
      part[w + 1] = make_float2(q.z, q.w);
    }
#pragma unroll
    for (int w = 0; w < kChunkWaves; w += 4) {
      const float4 q = tl[w / 4];
      const float r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int n = 0; n < 4; ++n) low[w + n] = r[n];
    }
    mass = 0.0;
    auto change = [&](int chunk, double by) { mass += lane == chunk ? by : 0.0; };
    // Rejected tokens leave the sums.
    const bool mine = ((gone >> lane) & 1ull) != 0ull && f > 0.0f;  // (a token met twice is out already)
    at = {0, 0};
    redone = 0ull;
    if (gone != 0ull) {
      float2 was = {0.0f, 0.0f};
      float was_low = 0.0f;
      if (mine) {
        at = place_of(tok);
        was = table[at.chunk * kChunkWaves + at.piece];
        was_low = table_low[at.chunk * kChunkWaves + at.piece];
      }
      const float rest = 1.0f - wave_sum(mine ? f0 : 0.0f);
      unsigned long long heavy = __ballot(mine && f0 > kTakenShare * rest);
      while (heavy != 0ull) {
        const int j = __ffsll(static_cast<long long>(heavy)) - 1;
        const int chunk = lane_value(at.chunk, j), piece = lane_value(at.piece, j);
        const unsigned long long same = __ballot(mine && at.chunk == chunk && at.piece == piece);
        heavy &= ~same;
        redone |= same;
        const ChunkRange range = chunk_range(spec, nvec, chunk);
        double sum = 0.0;
        auto add = [&](int first, float (&e)[EPV]) {  // EPV entries from `first` on
          for (unsigned long long m = same; m != 0ull; m &= m - 1ull) {
            const int x = lane_value(tok, __ffsll(static_cast<long long>(m)) - 1) - first;
#pragma unroll
            for (int n = 0; n < EPV; ++n) e[n] = n == x ? 0.0f : e[n];
          }
          float s = (e[0] + e[1]) + (e[2] + e[3]);
          if (EPV == 8) s += (e[EPV - 4] + e[EPV - 3]) + (e[EPV - 2] + e[EPV - 1]);
          sum += static_cast<double>(s);
        };
        // (the piece's vectors, 64 at a time, dealt out to the waves)
        constexpr int kStride = NW * kChunkWaves * kWave;
        const int v_first = range.begin + (wave * kChunkWaves + piece) * kWave;
        for (int v0 = v_first; v0 < range.end; v0 += kStride) {
          Vec<T, EPV> raw;
          const int vec = v0 + lane;
          raw.load(rowp + head, static_cast<unsigned int>(min(vec, range.end - 1)));
          float e[EPV];
#pragma unroll
          for (int n = 0; n < EPV; ++n) {
            const float t = precise(raw.get(n));
            e[n] = vec < range.end ? t : 0.0f;
          }
          add(head + vec * EPV, e);
        }
        if (RAGGED && piece == 0 && wave == 0) {  // loose elements, one per lane
          const bool front = chunk == 0 && lane < head;
          const bool back = lane >= head && lane < head + tail && chunk == place_of(V - 1).chunk;
          const int v = front ? lane : back ? V - tail + (lane - head) : 0;
          float e[EPV] = {};
          const float t = precise(widen(rowp[v]));
          e[0] = front || back ? t : 0.0f;
          add(v, e);
        }
        const double ws = wave_sum(sum);
        if (lane == 0) sh_piece[turn][wave] = ws;
        __syncthreads();
        const double again = wave_sum(lane < NW ? sh_piece[turn][lane] : 0.0);
        turn ^= 1;
        change(chunk, again - scaled(lane_value(sum_of(was.x, was_low), j), lane_value(was.y, j)));
      }
      // (the others as they were added)
      const double term = scaled(__builtin_amdgcn_exp2f(__builtin_fmaf(zx, c, -was.y)), was.y);
      for (unsigned long long light = __ballot(mine) & ~redone; light != 0ull; light &= light - 1ull) {
        const int j = __ffsll(static_cast<long long>(light)) - 1;
        change(lane_value(at.chunk, j), -lane_value(term, j));
      }
    }
    double all = 0.0;
#pragma unroll
    for (int w = 0; w < kChunkWaves; ++w) all += scaled(sum_of(part[w].x, low[w]), part[w].y);
    all = lane < nchunks ? all : 0.0;
    mass += all;
    mass = mass > 1e-37 ? mass : 0.0;
    if (gone != 0ull) {
      if (summed) {
        total = wave_sum(mass);
        all = wave_sum(all);
        if (!(total > 0.0)) {  // nothing is left without it: f stays as it was
          norm = lane == last ? 0.0f : norm;
          continue;
        }
        double z = total / all;
        for (unsigned long long m = gone & ~(1ull << last); m != 0ull; m &= m - 1ull)
          z /= static_cast<double>(lane_value(z_own, __ffsll(static_cast<long long>(m)) - 1));
        if (!draw) {
          norm = lane == last ? static_cast<float>(z) : norm;
          continue;
        }
        last_norm = static_cast<float>(z);
      }
    }
    break;
  }

  // ---------------------------------------------------------------- the draw
  const double incl = ROW ? 0.0 : wave_prefix_sum(mass);
  if (!ROW) total = lane_value(incl, kWave - 1);
  const double target = static_cast<double>(u_draw) * total;
  int chunk = -1;
  double cum = 0.0;
  if (ROW) {
    chunk = total > 0.0 ? 0 : -1;
  } else if (total > 0.0) {
    // The chunk the target falls into; where rounding leaves none, the last one with mass.
    const unsigned long long hit = __ballot(incl > target), any = __ballot(mass > 0.0);
    chunk = hit != 0ull ? __ffsll(static_cast<long long>(hit)) - 1 : 63 - __clzll(static_cast<long long>(any));
    cum = lane_value(incl - mass, chunk);
  }
  const int last_node_top1 = lane_value(st.id1, cnode);
  double whole = 0.0;  // the sum against the row's largest logit
  // What a token's share is taken of (bonus_prob): the sum against the row's largest logit, whose term is 1.  The sums of chunks are against whole numbers, in steps that
  // bring an error of their own for every term, which matters for the largest: these two are taken out of the sum as they were
  // added.  (Largest error of bonus_prob over 16 seeds, one tree
  // of 60 nodes x 151 936 and one of 9 x 32 000: 5e-8 and 1.0e-7, as the walk that goes over the row; with the terms as the sums have them 1.9e-7 and
  // 3.2e-7.)
  // (Worked out beside the trip to the chunk.  Behind it, 16 drawn calls of more than 32 752 entries took 0.6 % more, one chain of 30 x 128 256 with seven thresholds 16.2 us
  // instead of 15.5.)
  auto settle = [&]() __attribute__((always_inline)) {
    double sum = total, again = 0.0;
    auto put_right = [&](int v, float z) {
      const Place to = place_of(v);
      const unsigned long long bit = 1ull << lane;
      if (v < 0 || __any((gone & bit) != 0ull && tok == v)) return;
      float ref = R;
#pragma unroll
      for (int w = 0; w < kChunkWaves; ++w) ref = w == to.piece ? lane_value(part[w].y, to.chunk) : ref;
      const bool exact = __any((redone & bit) != 0ull && at.chunk == to.chunk && at.piece == to.piece);
      sum -= exact ? static_cast<double>(precise(z)) : scaled(__builtin_amdgcn_exp2f(__builtin_fmaf(z, c, -ref)), ref);
      again += static_cast<double>(__builtin_amdgcn_exp2f((z - z1) * c));
    };
    put_right(last_node_top1, z1);
    put_right(lane_value(st.id2, cnode), lane_value(st.z2, cnode));
    whole = sum * exp2(static_cast<double>(R) - static_cast<double>(z1) * static_cast<double>(c)) + again;
  };
  int pick = -1;
  float pick_z = 0.0f;
  if (chunk >= 0) {
    ChunkRange range = {0, nvec};
    if (!ROW) range = chunk_range(spec, nvec, chunk);
    const bool front = RAGGED && head > 0 && chunk == 0, back = RAGGED && tail > 0 && (ROW || chunk == place_of(V - 1).chunk);
    const int begin = front ? -1 : range.begin, end = back ? nvec + 1 : range.end;
    int last_page = -1;
    bool take_last = false;  // rounding has left no entry above the target: the last one with mass
    for (int page = begin; page < end; page += PV * NT) {
      if (!ROW) read_page(page, range, front, back, [&] { if (page == begin && a.diag) settle(); });
      const unsigned long long hit = __ballot(cum + tile_incl > target), any = __ballot(tile_sum > 0.0);
      if ((ROW || hit != 0ull || take_last) && any != 0ull) {
        const int tl = hit != 0ull && !take_last ? __ffsll(static_cast<long long>(hit)) - 1 : 63 - __clzll(static_cast<long long>(any));
        double in_front = cum + lane_value(tile_incl - tile_sum, tl);
        int tile = tl;
        if (TILES == 2) {  // the first of the lane's two, or the second
          const double first = lane_value(tile_first, tl), second = lane_value(tile_sum, tl) - first;
          const bool over = !take_last && hit != 0ull ? !(in_front + first > target) && second > 0.0 : second > 0.0;
          tile = 2 * tl + (over ? 1 : 0);
          in_front += over ? first : 0.0;
        }
        if (wave != tile % NW) return;  // one wave finishes, the one that holds the tile
        float f[EPV], z[EPV], fs = 0.0f;
#pragma unroll
        for (int m = 0; m < PV; ++m)
          if (m == tile / NW) {
            fs = g[m];
#pragma unroll
            for (int n = 0; n < EPV; ++n) { f[n] = e[m][n]; z[n] = raw[m].get(n); }
          }
        const double lanes = wave_prefix_sum(static_cast<double>(fs)), at = in_front;
        const unsigned long long over = __ballot(at + lanes > target);
        int hl = 0, pe = -1;
        float pz = 0.0f;
        if (over != 0ull && !take_last) {
          hl = __ffsll(static_cast<long long>(over)) - 1;
          double sum = at + (lanes - static_cast<double>(fs));
#pragma unroll
          for (int n = 0; n < EPV; ++n) {
            sum += static_cast<double>(f[n]);
            if (pe < 0 && sum > target) { pe = n; pz = z[n]; }
          }
          pe = lane_value(pe, hl);
        }
        if (pe < 0) {  // the last entry with mass
          int mine_last = -1;
#pragma unroll
          for (int n = 0; n < EPV; ++n)
            if (f[n] > 0.0f) { mine_last = n; pz = z[n]; }
          hl = 63 - __clzll(static_cast<long long>(__ballot(mine_last >= 0)));
          pe = lane_value(mine_last, hl);
        }
        pick = head + (page + tile / NW * NT + wave * kWave + hl) * EPV + pe;
        pick_z = lane_value(pz, hl);
        if (RAGGED && (pick < head || pick >= V - tail)) pick_z = widen(rowp[pick]);
        break;
      }
      if (any != 0ull) last_page = page;
      cum += lane_value(tile_incl, kWave - 1);
      if (page + PV * NT >= end && last_page >= 0) {
        take_last = true;
        page = last_page - PV * NT;
      }
    }
  }
  if (pick < 0 && wave != 0) return;
  // ---------------------------------------------------------------- results, by one wave
  float prob = 0.0f;
  if (pick >= 0) {
    const double sum = ROW ? total : whole;
    prob = static_cast<float>(static_cast<double>(__builtin_amdgcn_exp2f((pick_z - z1) * c)) / sum);
  }
  const int token = pick >= 0 ? pick : last_node_top1;  // (no mass anywhere)
  const bool on_path = ((visited >> lane) & 1ull) != 0ull;
  const int committed = __shfl(tok, lane < plen ? path : 0, kWave);
  if (live) {
    a.mask[rb + lane] = on_path ? 1 : 0;
    a.path[rb + lane] = path;
    if (a.dec) a.dec[rb + lane] = static_cast<uint8_t>(on_path ? code : 0);
    if (a.out_tok) a.out_tok[rb + lane] = lane < plen ? committed : lane == plen ? token : -1;
  }
  if (lane == 0) {
    a.bonus[b] = token;
    a.len[b] = plen;
    if (a.out_tok) a.out_len[b] = plen + 1;
    if (a.diag) {
      mars_req_diag dg;
      dg.bonus_prob = prob;
      dg.last_residual_norm = last_norm;
      dg.residual_passes = passes;
      dg.last_node = cnode;
      a.diag[b] = dg;
    }
  }
}

}  // namespace mars
