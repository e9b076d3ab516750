// How the LM head's work is dealt out, run on the CPU: mars_lmhead_verify and mars_lmhead_verify_sampling are called as
// they are (every HIP call below stands in for the runtime and launches nothing), and what each launch's work-groups
// would do is gone through with the kernel's own cell arithmetic (csrc/lmhead.h: lm_cell).  Every tile of every slab has
// to belong to exactly one work-group and every partial result of every row to be written exactly once.
// Arguments: "B N V H sampling bands launches shared form" per case, the last four what the case must show ("-" = anything): bands
// of slabs, launches, whether a cell is shared between two work-groups, and the form of the kernel that runs: rows x entries of a
// unit, "ring" behind it where the operands go straight to LDS, and "-once" where the weight is read past the caches.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

static inline __host__ float __uint_as_float(unsigned int x) { return __builtin_bit_cast(float, x); }

#pragma clang force_cuda_host_device begin
#include "../paper_2601_15498_amd/csrc/mars.hip"
#pragma clang force_cuda_host_device end

struct Launch {
  const void* kernel;
  dim3 grid;
  int M, V, H;
  mars::LmGrid g;
  const char *hidden, *partials, *logits;
  long cleared;
};
static std::vector<Launch> launches;
static std::map<const void*, int> heights;  // the fused kernel's forms
static std::map<const void*, std::string> names;
static dim3 call_grid;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* none; return &none; }
void __hipRegisterFunction(...) {}
void __hipRegisterVar(...) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3, size_t, hipStream_t) { call_grid = grid; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = call_grid; *block = dim3(1); *shared = 0; *stream = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3, void** args, size_t, hipStream_t) {
  if (heights.count(kernel)) {
    Launch l;
    l.kernel = kernel; l.grid = grid;
    l.hidden = *static_cast<const char**>(args[0]);
    l.M = *static_cast<int*>(args[2]); l.V = *static_cast<int*>(args[3]); l.H = *static_cast<int*>(args[4]);
    l.g = *static_cast<mars::LmGrid*>(args[5]);
    l.partials = *static_cast<const char**>(args[6]);
    l.logits = *static_cast<const char**>(args[7]);
    l.cleared = static_cast<mars::LmClear*>(args[9])->nwords;
    launches.push_back(l);
  }
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
}

template <int BM, bool S, bool W = false>
static void form() {
  const void* kernel = reinterpret_cast<const void*>(&mars::lmhead_reduce_kernel<BM, S, W>);
  heights[kernel] = BM;
  names[kernel] = std::to_string(BM) + "x256" + (W ? "-wide" : "");
}

template <int BM, int BN, int STAGES, bool S, bool ONCE>
static void ring_form() {
  const void* kernel = reinterpret_cast<const void*>(&mars::lmhead_ring_kernel<BM, BN, STAGES, S, ONCE>);
  heights[kernel] = BM;
  names[kernel] = std::to_string(BM) + "x" + std::to_string(BN) + "ring" + (ONCE ? "-once" : "");
}
template <int BM, int BN, int STAGES>
static void ring() {
  ring_form<BM, BN, STAGES, false, false>(); ring_form<BM, BN, STAGES, false, true>();
  ring_form<BM, BN, STAGES, true, false>(); ring_form<BM, BN, STAGES, true, true>();
}

static int fail(const char* what, int B, int N, int V, int H, int sampling) {
  std::printf("%s: B %d N %d V %d H %d sampling %d\n", what, B, N, V, H, sampling);
  return 1;
}

static int check(int B, int N, int V, int H, int sampling, const std::string& bands, const std::string& many, const std::string& shared,
                 const std::string& form) {
  using namespace mars;
  launches.clear();
  char* const base = reinterpret_cast<char*>(1ul << 40);  // (nothing is read or written)
  char *hidden = base, *workspace = 2 * (1ul << 40) + static_cast<char*>(nullptr), *logits = 3 * (1ul << 40) + static_cast<char*>(nullptr);
  int32_t* other = reinterpret_cast<int32_t*>(4 * (1ul << 40));
  float* f = reinterpret_cast<float*>(other);
  const size_t bytes = mars_lmhead_workspace_bytes(B, N, V, H, 1);
  const int rc = sampling ? mars_lmhead_verify_sampling(hidden, base, H, other, other, nullptr, 0, f, 1.0f, f, B, N, V, logits,
                                                        reinterpret_cast<uint8_t*>(other), other, other, other, nullptr, nullptr,
                                                        nullptr, nullptr, workspace, bytes, nullptr, nullptr)
                          : mars_lmhead_verify(hidden, base, H, other, other, f, B, N, V, reinterpret_cast<uint8_t*>(other), other,
                                               other, other, nullptr, nullptr, nullptr, workspace, bytes, nullptr, nullptr);
  if (bytes == 0 || rc != MARS_OK || launches.empty()) return fail("not launched", B, N, V, H, sampling);
  const long rows = static_cast<long>(B) * N;
  long next_row = 0;
  bool any_shared = false;
  for (const Launch& l : launches) {
    const LmGrid& g = l.g;
    const int bm = heights[l.kernel], per_die = static_cast<int>(l.grid.x) / 8;
    if (l.grid.x % 8 != 0 || (per_die > 32 && g.slabs <= 256)) return fail("more work-groups on a die than compute units", B, N, V, H, sampling);
    if (l.hidden != hidden + next_row * H * 2 || l.partials != workspace + next_row * g.parts * static_cast<long>(sizeof(Partial)) ||
        (sampling && l.logits != logits + next_row * V * 2) || l.M != rows - next_row)
      return fail("a launch does not begin where the one before ends", B, N, V, H, sampling);
    if ((l.cleared != 0) != (sampling && next_row == 0)) return fail("words cleared other than once", B, N, V, H, sampling);
    if (static_cast<long>(g.slabs) * g.tiles_n != g.units) return fail("units", B, N, V, H, sampling);
    const int columns = (g.tiles_n + g.width - 1) / g.width;
    if (g.parts > (g.slabs <= g.band ? columns + 1 : 2 * columns)) return fail("empty partial results", B, N, V, H, sampling);
    if (static_cast<size_t>(rows) * g.parts * sizeof(Partial) > bytes) return fail("workspace", B, N, V, H, sampling);
    std::vector<unsigned char> written(static_cast<size_t>(g.slabs) * g.parts);
    std::vector<int> tiles(static_cast<size_t>(g.slabs) * columns);
    for (int block = 0; block < static_cast<int>(l.grid.x); ++block) {
      const int group = (block & 7) * per_die + (block >> 3);
      const long begin = static_cast<long>(group) * g.width;
      if (begin >= g.units) continue;
      const int end = static_cast<int>(begin + g.width < g.units ? begin + g.width : g.units);
      for (int unit = static_cast<int>(begin); unit < end;) {
        const LmCell c = lm_cell(unit, end, g.slabs, g.band, g.tiles_n, g.width);
        const int width = c.column + 1 < columns ? g.width : g.tiles_n - c.column * g.width;
        const int at = c.tile - c.column * g.width;
        if (c.n < 1 || c.slab < 0 || c.slab >= g.slabs || c.column < 0 || c.column >= columns || at < 0 || at + c.n > width ||
            c.begins != (at == 0) || c.ends != (at + c.n == width))
          return fail("a cell out of range", B, N, V, H, sampling);
        // (two pieces of one cell do not overlap: one is its beginning, the other its end, and the lengths add up)
        tiles[static_cast<size_t>(c.slab) * columns + c.column] += c.n;
        unsigned char* w = &written[static_cast<size_t>(c.slab) * g.parts];
        if (c.column < g.split) {
          if (!c.begins || !c.ends) return fail("a shared cell without a place for both", B, N, V, H, sampling);
          ++w[c.column];
        } else {
          w += 2 * c.column - g.split;
          ++w[c.begins ? 0 : 1];
          if (c.begins && c.ends) ++w[1];
          any_shared |= !(c.begins && c.ends);
        }
        unit += c.n;
      }
    }
    for (int s = 0; s < g.slabs; ++s)
      for (int c = 0; c < columns; ++c)
        if (tiles[static_cast<size_t>(s) * columns + c] != (c + 1 < columns ? g.width : g.tiles_n - c * g.width))
          return fail("tiles left out or done twice", B, N, V, H, sampling);
    for (unsigned char w : written)
      if (w != 1) return fail("a partial result not written exactly once", B, N, V, H, sampling);
    next_row += static_cast<long>(g.slabs) * bm;
  }
  if (next_row < rows) return fail("rows left out", B, N, V, H, sampling);
  const LmGrid& g = launches[0].g;
  const int nbands = (g.slabs + g.band - 1) / g.band;
  if ((bands != "-" && std::to_string(nbands) != bands) || (many != "-" && std::to_string(launches.size()) != many) ||
      (shared != "-" && (shared == "1") != any_shared)) {
    std::printf("%d bands, %zu launches, %sshared cells\n", nbands, launches.size(), any_shared ? "" : "no ");
    return fail("not the plan the case stands for", B, N, V, H, sampling);
  }
  const std::string& runs = names[launches[0].kernel];
  if (form != "-" && form != runs) return fail(("another form than " + form + " (" + runs + ")").c_str(), B, N, V, H, sampling);
  return 0;
}

int main(int argc, char** argv) {
  form<64, false>(); form<64, false, true>(); form<128, false>(); form<192, false>(); form<256, false>();
  form<64, true>(); form<64, true, true>(); form<128, true>(); form<192, true>();
  ring<64, 64, 8>(); ring<64, 128, 5>(); ring<64, 256, 3>(); ring<128, 128, 4>(); ring<128, 256, 3>(); ring<256, 128, 3>();
  int failed = 0, cases = 0;
  for (int i = 1; i + 8 < argc; i += 9, ++cases)
    failed += check(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]), std::atoi(argv[i + 3]), std::atoi(argv[i + 4]),
                    argv[i + 5], argv[i + 6], argv[i + 7], argv[i + 8]);
  std::printf("%d cases, %d failed\n", cases, failed);
  return failed != 0;
}
