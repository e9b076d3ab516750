// Chunks of a row: runs of entries whose sums of exponentials the row reduction leaves, so that the final draw of a walk
// that needs nothing but the softmax of the row (Eq. 3, less the tokens that were rejected) reads the sums and one or two
// chunks instead of the whole row.
//
// A row is `items` shares of `vps` 16-byte vectors.  A share is streamed in batches of kChunkVecs vectors; `batches` of them
// are a chunk, the last chunk takes what is left: the batches behind the stream's main loop, and the share's ragged end.  (A row's loose elements, in front of its first aligned vector and
// behind its last, belong to its first and its last chunk.)
#pragma once

#include <hip/hip_runtime.h>

namespace mars {

constexpr int kChunkVecs = 1024;   // vectors of a batch
constexpr int kChunkWaves = 8;     // sums of a chunk: one per wave of the row reduction
constexpr int kMaxSlots = 10;      // chunks of a share, at most
constexpr int kMaxChunks = 64;     // ... of a row, if the row reduction leaves their sums

// (What the two functions below divide by comes as factors: an integer division is 25 instructions.)
struct ChunkSpec {
  int items, vps;
  int slots, log2_batches;   // chunks of a share (1: it is one), batches of a chunk
  unsigned int per_slot;     // 2^16 / slots, rounded up
  float per_vps;             // 1 / vps
};

// The batch behind the row reduction's main loop, of a share of nfull whole ones.
__device__ __host__ __forceinline__ constexpr int chunk_stream_end(int nfull) { return nfull > 2 ? (nfull - 1) & ~1 : 0; }
// The last chunk of a share of nv vectors.
__device__ __host__ __forceinline__ int chunk_last(const ChunkSpec& s, int nv) {
  return s.slots == 1 ? 0 : chunk_stream_end(nv / kChunkVecs) >> s.log2_batches;
}
// Chunk `i` of a row of nvec vectors: vectors [begin, end).
struct ChunkRange { int begin, end; };
__device__ __host__ __forceinline__ ChunkRange chunk_range(const ChunkSpec& s, int nvec, int i) {
  const int item = static_cast<int>(static_cast<unsigned int>(i) * s.per_slot >> 16), j = i - item * s.slots;
  const long first = static_cast<long>(item) * s.vps;
  const int v_begin = first < nvec ? static_cast<int>(first) : nvec, v_end = nvec - v_begin < s.vps ? nvec : v_begin + s.vps;
  const int last = chunk_last(s, v_end - v_begin), size = kChunkVecs << s.log2_batches;
  if (j > last) return {v_end, v_end};
  return {v_begin + j * size, j == last ? v_end : v_begin + (j + 1) * size};
}
// The chunk that holds vector `vec` of the row.
__device__ __host__ __forceinline__ int chunk_of(const ChunkSpec& s, int nvec, int vec) {
  int item = static_cast<int>(static_cast<float>(vec) * s.per_vps);  // (off by one at most)
  const long at = static_cast<long>(vec) - static_cast<long>(item) * s.vps;
  item += at < 0 ? -1 : at >= s.vps ? 1 : 0;
  const int v_begin = item * s.vps, v_end = nvec - v_begin < s.vps ? nvec : v_begin + s.vps;
  const int last = chunk_last(s, v_end - v_begin), j = (vec - v_begin) / kChunkVecs >> s.log2_batches;
  return item * s.slots + (j < last ? j : last);
}
// `items` shares of at most vps vectors in `slots` chunks each.
inline ChunkSpec chunk_spec(int items, int vps, int slots, int log2_batches) {
  return {items, vps, slots, log2_batches, slots > 0 ? (0xFFFFu + slots) / slots : 0u, 1.0f / static_cast<float>(vps)};
}
// The same, the chunks those of the row reduction (slots == 0: more than a draw can look through).
inline ChunkSpec chunk_spec(int items, int vps) {
  const int end = chunk_stream_end(vps / kChunkVecs);
  int k = 1;
  while ((end >> k) + 1 > kMaxSlots) ++k;
  while (end >> k != 0 && static_cast<long>(items) * ((end >> k) + 1) > kMaxChunks) ++k;
  const int slots = (end >> k) + 1;
  return chunk_spec(items, vps, static_cast<long>(items) * slots > kMaxChunks ? 0 : slots, k);
}

}  // namespace mars
