// The chunks of a row (csrc/chunks.h) on the CPU: for shares of all kinds of lengths they cover the row's vectors once, in order,
// end where the row reduction's loop ends them, and every vector is found in its own.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#pragma clang force_cuda_host_device begin
#include "../paper_2601_15498_amd/csrc/chunks.h"
#pragma clang force_cuda_host_device end

using namespace mars;

static long failed = 0, rows = 0;
static void fail(const char* what, const ChunkSpec& s, int nvec, int i) {
  if (failed++ < 10) std::printf("%s: %d vectors, %d shares of %d, %d chunks of 2^%d batches: chunk %d\n", what, nvec, s.items, s.vps, s.slots, s.log2_batches, i);
}

// The row reduction's stream over one share: the vectors it has behind it whenever it ends a chunk, and at the end.
static std::vector<int> chunk_ends(int nv, int batches) {
  std::vector<int> ends;
  const int nfull = nv / kChunkVecs;
  int end = batches;
  for (int k = 0; k + 2 < nfull; k += 2)
    if (k + 2 == end) { ends.push_back(end * kChunkVecs); end += batches; }
  ends.push_back(nv);
  return ends;
}

static void check(const ChunkSpec& s, int nvec) {
  ++rows;
  int at = 0;
  for (int item = 0; item < s.items; ++item) {
    const int begin = item * static_cast<long>(s.vps) < nvec ? item * s.vps : nvec, end = nvec - begin < s.vps ? nvec : begin + s.vps;
    const std::vector<int> ends = chunk_ends(end - begin, 1 << s.log2_batches);
    if (static_cast<int>(ends.size()) > s.slots) fail("too many", s, nvec, item * s.slots);
    for (int j = 0; j < s.slots; ++j) {
      const int i = item * s.slots + j;
      const ChunkRange r = chunk_range(s, nvec, i);
      if (r.begin != at || r.end < r.begin) fail("gap", s, nvec, i);
      if (r.end != begin + (j < static_cast<int>(ends.size()) ? ends[j] : ends.back())) fail("end", s, nvec, i);
      at = r.end;
      for (int v : {r.begin, r.begin + 1, (r.begin + r.end) / 2, r.end - 1})
        if (v >= r.begin && v < r.end && chunk_of(s, nvec, v) != i) fail("not found", s, nvec, i);
    }
  }
  if (at != nvec) fail("not covered", s, nvec, -1);
}

int main() {
  // rows of the row reduction: any number of shares, lengths around whole batches; a row has the most vectors or one less
  for (int items : {1, 2, 3, 5, 7, 18, 40, 64})
    for (int batches = 0; batches < 90; batches += batches < 24 ? 1 : 7)
      for (int more : {-1, 0, 1, 511, 1023}) {
        const int nvec = items * batches * kChunkVecs + more;
        if (nvec < 1) continue;
        const ChunkSpec s = chunk_spec(items, (nvec + items - 1) / items);
        if (s.slots < 1 || s.items * s.slots > kMaxChunks || s.slots > kMaxSlots) { fail("count", s, nvec, -1); continue; }
        check(s, nvec);
        if (nvec > 1) check(s, nvec - 1);
      }
  if (chunk_spec(65, 100).slots != 0) fail("accepted", chunk_spec(65, 100), 6500, -1);
  // far along a long row
  check(chunk_spec(64, (1 << 28) / 64 + 5, 10, 15), 1 << 28);
  std::printf("%ld rows, %ld failed\n", rows, failed);
  return failed != 0;
}
