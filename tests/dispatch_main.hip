// Which kernels a call takes, run on the CPU: mars_verify_ex is called as it is (every HIP call below stands in for the runtime and
// launches nothing) and the kernels that it would launch are written down.
// Arguments: "B N V dtype offset K draft workspace kernels" per case: dtype bf16 | f32 of the logits, which begin `offset` entries behind a 16-byte
// boundary; K thresholds; draft onehot | f32; workspace full | least; what the names of the row reduction and the per-request kernel,
// "row_reduce_kernel<...> tail_...<...>", have to begin with, in the order of the launches, "|" between them ("-": anything).
#include <hip/hip_runtime.h>

#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

static inline __host__ float __uint_as_float(unsigned int x) { return __builtin_bit_cast(float, x); }

#pragma clang force_cuda_host_device begin
#include "../paper_2601_15498_amd/csrc/mars.hip"
#pragma clang force_cuda_host_device end

static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> all;
  return all;
}
static std::vector<std::string> launched;
static dim3 call_grid;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* none; return &none; }
void __hipRegisterFunction(void**, const void* kernel, const char*, const char* name, unsigned int, void*, void*, void*, void*, int*) {
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  std::string s = plain ? plain : name;
  std::free(plain);
  s = s.substr(0, s.find('('));
  if (s.rfind("void ", 0) == 0) s = s.substr(5);
  if (s.rfind("mars::", 0) == 0) s = s.substr(6);
  for (size_t at; (at = s.find("unsigned short")) != std::string::npos;) s.replace(at, 14, "bf16");
  names()[kernel] = s;
}
void __hipRegisterVar(...) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3, size_t, hipStream_t) { call_grid = grid; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = call_grid; *block = dim3(1); *shared = 0; *stream = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t, hipStream_t) {
  launched.push_back(names().count(kernel) ? names()[kernel] : "?");
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
}

static int check(char** a) {
  const int B = std::atoi(a[0]), N = std::atoi(a[1]), V = std::atoi(a[2]), K = std::atoi(a[5]);
  const bool f32 = std::string(a[3]) == "f32", dense = std::string(a[6]) != "onehot", full = std::string(a[7]) == "full";
  launched.clear();
  char* const base = reinterpret_cast<char*>(1ul << 40);  // (nothing is read or written)
  const char* logits = base + std::atoi(a[4]) * (f32 ? 4 : 2);
  int32_t* i = reinterpret_cast<int32_t*>(base);
  float* f = reinterpret_cast<float*>(base);
  const mars::Layout L = mars::layout(B, N, V, K);
  if (L.total != mars_workspace_bytes_ex(B, N, V, K)) { std::printf("workspace: %s x %s x %s\n", a[0], a[1], a[2]); return 1; }
  mars_verify_options o = {};
  o.n_theta = K;
  const int rc = mars_verify_ex(logits, f32 ? MARS_F32 : MARS_BF16, i, i, dense ? base : nullptr, MARS_F32, f, 1.0f, f, B, N, V,
                                reinterpret_cast<uint8_t*>(base), i, i, i, nullptr, nullptr, nullptr, nullptr, base, full ? L.total : L.least, nullptr, &o);
  std::string all;
  for (const std::string& s : launched) all += (all.empty() ? "" : "|") + s;
  bool ok = rc == MARS_OK && launched.size() == 2;
  const std::string want = a[8];
  const size_t bar = want.find('|');
  if (ok && want != "-")
    ok = launched[0].rfind(want.substr(0, bar), 0) == 0 && (bar == std::string::npos || launched[1].rfind(want.substr(bar + 1), 0) == 0);
  if (!ok || std::getenv("MARS_SAY")) std::printf("%s x %s x %s %s +%s, %s thresholds, %s, %s: %d %s\n", a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], rc, all.c_str());
  return !ok;
}

int main(int argc, char** argv) {
  int failed = 0, cases = 0;
  for (int i = 1; i + 8 < argc; i += 9, ++cases) failed += check(argv + i);
  std::printf("%d cases, %d failed\n", cases, failed);
  return failed != 0;
}
