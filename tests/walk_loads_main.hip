// The sampling walk's view of a row (csrc/tail.h: RowView), run on the CPU: every load it makes of every group of
// every row, from arrays at every alignment that end where their allocation ends, under AddressSanitizer and with the
// alignment of every access checked.  What is loaded and trimmed is compared with the array, element by element.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include <sanitizer/asan_interface.h>

// (the headers have this for the device alone)
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

using namespace mars;

static float z_value(size_t i) { return static_cast<float>(static_cast<int>(i * 7 % 251) - 100); }
static float q_value(size_t i) { return static_cast<float>(i * 5 % 241 + 1) / 256.0f; }
static void put(float& x, float v) { x = v; }
static void put(bf16_t& x, float v) { x = static_cast<bf16_t>(__builtin_bit_cast(unsigned int, v) >> 16); }

// An array of n elements, k behind the beginning of an allocation and at its very end.
template <typename T>
struct Array {
  T* base;
  size_t n, k;
  Array(size_t n_, size_t k_, float (*value)(size_t)) : base(static_cast<T*>(std::malloc((n_ + k_) * sizeof(T)))), n(n_), k(k_) {
    for (size_t i = 0; i < n; ++i) put(base[k + i], value(i));
    ASAN_POISON_MEMORY_REGION(base, k * sizeof(T));  // (in steps of eight bytes)
  }
  ~Array() {
    ASAN_UNPOISON_MEMORY_REGION(base, k * sizeof(T));
    std::free(base);
  }
  T* data() const { return base + k; }
};

static long failed = 0, cases = 0, loads = 0;
static volatile float sink;  // what is read and not looked at

template <typename T, typename TQ, bool VEC>
static void check(const T* z, const TQ* q, int B, int N, int V, const void* spare) {
  RowView<T, TQ, VEC> rv;
  rv.V = V;
  rv.ch.n = 0;
  const int groups = row_groups(V, VEC);
  std::vector<int> seen(V);
  for (int b = 0; b < B; ++b) {
    rv.request(z, q, static_cast<size_t>(b) * N * V, static_cast<size_t>(B) * N * V, spare);
    for (int node = 0; node < N; ++node)
      for (int use = 0; use < 2; ++use) {
        rv.use_q = use != 0;
        rv.row(node, q != nullptr);
        const bool dense = q != nullptr && rv.use_q;
        Raw8<TQ> r;
        r.template load<VEC>(rv.q_source(false, spare), 0);
        float unused[8];
        r.widen_to(unused);
        for (float u : unused) sink = u;
        std::fill(seen.begin(), seen.end(), 0);
        for (int gi = 0; gi < groups; ++gi) {
          float x[8], y[8];
          rv.load(gi, x, y);
          rv.trim(gi, x, y);
          ++loads;
          for (int e = 0; e < 8; ++e) {
            const int v = rv.element(gi, e);
            const bool in = v >= 0 && v < V;
            const size_t at = (static_cast<size_t>(b) * N + node) * V + v;
            if (in) ++seen[v];
            if (x[e] != (in ? z_value(at) : -INFINITY) || y[e] != (in && dense ? q_value(at) : 0.0f)) {
              if (failed++ < 10) std::printf("B %d N %d V %d request %d node %d group %d element %d: %g %g\n", B, N, V, b, node, gi, e, x[e], y[e]);
            }
          }
        }
        for (int v = 0; v < V; ++v)
          if (seen[v] != 1 && failed++ < 10) std::printf("B %d N %d V %d node %d: entry %d seen %d times\n", B, N, V, node, v, seen[v]);
      }
  }
}

template <typename T, typename TQ>
static void run(int B, int N, int V, bool dense, int k) {
  const size_t n = static_cast<size_t>(B) * N * V;
  Array<T> z(n, k, z_value);
  Array<TQ> q(dense ? n : 1, k == 0 ? 0 : 8 - k, q_value);
  alignas(16) static char spare[32];
  const T* zp = z.data();
  const TQ* qp = dense ? q.data() : nullptr;
  ++cases;
  if (whole_groups(zp, sizeof(T), qp, N, V))
    check<T, TQ, true>(zp, qp, B, N, V, spare);
  else
    check<T, TQ, false>(zp, qp, B, N, V, spare);
}

int main() {
  const int sizes[][3] = {{1, 1, 2}, {1, 1, 7}, {1, 1, 8}, {1, 2, 8}, {2, 1, 9}, {3, 1, 5}, {1, 3, 16}, {2, 3, 24}, {2, 5, 13},
                          {3, 4, 61}, {2, 3, 63}, {1, 3, 65}, {2, 2, 520}, {2, 2, 1001}};
  for (const auto& s : sizes)
    for (int dense = 0; dense < 2; ++dense)
      for (int k = 0; k < 8; ++k) {
        run<bf16_t, float>(s[0], s[1], s[2], dense != 0, k);
        run<bf16_t, bf16_t>(s[0], s[1], s[2], dense != 0, k);
        run<float, float>(s[0], s[1], s[2], dense != 0, k);
        run<float, bf16_t>(s[0], s[1], s[2], dense != 0, k);
      }
  std::printf("%ld cases, %ld loads, %ld failed\n", cases, loads, failed);
  return failed != 0;
}
