// The order of the accesses to the sampling walk's residual chain in LDS (csrc/tail.h: entries kChainRegs and up), run on
// the CPU.  Every wave walks by itself; what orders one wave's access against another's is a barrier between them.  Thread 0
// writes entry n when the node's child n is rejected; every wave reads the entries in front of n when it tests child n, when
// it sums a row and when it draws.  All ways through up to three nodes are gone through with the barriers that
// chain_barrier() asks for: a write and a read of one entry without a barrier between them, in either order, is a fault.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

static inline __host__ float __uint_as_float(unsigned int x) { return __builtin_bit_cast(float, x); }

#pragma clang force_cuda_host_device begin
#include "../include/mars.h"
#include "../paper_2601_15498_amd/csrc/common.h"
#include "../paper_2601_15498_amd/csrc/row_reduce.h"
#include "../paper_2601_15498_amd/csrc/tail.h"
#pragma clang force_cuda_host_device end

// No kernel is launched here: nothing to register.
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* none; return &none; }
void __hipRegisterFunction(...) {}
void __hipRegisterVar(...) {}
void __hipUnregisterFatBinary(void**) {}
}

constexpr int kMost = 12;  // rejections at a node

struct Node {
  int rejections;
  int exchanges;  // how many of them sum the row, the first ones (dense draft probabilities: all, or all but the node's last child's)
};

// Barriers so far, and how many there were at an entry's last write and last read.
template <typename Rule>
struct Chain {
  Rule rule;
  long barriers = 0, faults = 0;
  std::vector<long> written, read;
  explicit Chain(Rule r) : rule(r), written(kMost + 1, -1), read(kMost + 1, -1) {}
  void reads(int n) {
    for (int j = mars::kChainRegs; j < n; ++j) {
      faults += written[j] == barriers;
      read[j] = barriers;
    }
  }
  void node(const Node& at) {
    for (int n = 0; n < at.rejections; ++n) {
      if (n > 0) reads(n);  // the test of child n (the first one is tested without a chain)
      if (n < at.exchanges) {
        reads(n);           // the row's sum, and the barriers of its exchange
        ++barriers;
      }
      if (n >= mars::kChainRegs) {
        faults += read[n] == barriers;
        written[n] = barriers;
      }
      if (n < at.exchanges || rule(n)) ++barriers;
    }
    reads(at.rejections);  // the test of the child that is accepted, or the draw
  }
};

template <typename Rule>
static long faults(Rule rule, long* ways) {
  long found = 0;
  std::vector<Node> nodes;
  for (int r = 0; r <= kMost; ++r)
    for (int e : {0, r - 1, r})
      if (e >= 0) nodes.push_back({r, e});
  for (const Node& a : nodes)
    for (const Node& b : nodes)
      for (const Node& c : nodes) {
        Chain<Rule> chain(rule);
        chain.node(a);
        chain.node(b);
        chain.node(c);
        found += chain.faults;
        ++*ways;
      }
  return found;
}

int main() {
  long ways = 0, other = 0;
  const long found = faults([](int n) { return mars::chain_barrier(n); }, &ways);
  // A barrier only behind the entries that live in LDS: nothing keeps the write of a node's first one behind the previous
  // node's reads, and it has to show here.
  const long missing = faults([](int n) { return n >= mars::kChainRegs; }, &other);
  std::printf("%ld ways, %ld out of order, %s\n", ways, found, missing ? "a missing barrier shows" : "a missing barrier does not show");
  return found != 0 || missing == 0;
}
