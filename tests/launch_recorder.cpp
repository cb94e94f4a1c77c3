// Runs library calls on a machine without a GPU and prints what they would launch.  The HIP entry points that libaura_fuse.so uses are
// defined here, in the program, so the library finds these instead of the runtime's.  One call per line of standard input:
//   call N B n_views H Hf D dtype K P flags norm_eps temperature fail
// (call: single, scores, fuse, selected, of B objects of equal shares, or densify, from B sources; fail: the kernel whose launch shall fail, or -).  Per call one line:
//   status kernel(grid x, grid y, block) ... with S and E where the events of aura_time_next_fusion are recorded.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../include/aura_fuse.h"

namespace {
struct Dim3 {
  unsigned x, y, z;
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> n;
  return n;
}
Dim3 g_grid, g_block;
std::string g_fail, g_log;
int g_error = 0;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module = nullptr; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[host] = name; }
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t, void*) {
  g_grid = grid;
  g_block = block;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = g_grid;
  *block = g_block;
  *shared = 0;
  *stream = nullptr;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*) {
  const std::string name = names().count(f) ? names()[f] : "?";
  g_error = !g_fail.empty() && name.find(g_fail) != std::string::npos ? 719 : 0;
  g_log += " " + name + "(" + std::to_string(grid.x) + "," + std::to_string(grid.y) + "," + std::to_string(block.x) + ")";
  return g_error;
}
int hipGetLastError() {
  const int e = g_error;
  g_error = 0;
  return e;
}
int hipEventRecord(void* event, void*) {
  g_log += event == reinterpret_cast<void*>(1) ? " S" : " E";
  return 0;
}
int hipGetDevice(int* d) { return *d = 0; }
int hipDeviceGetAttribute(int* value, int, int) {
  *value = 256;
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return 0;
}
}

int main(int argc, char** argv) {
  if (argc > 1 && !strcmp(argv[1], "names")) {
    for (const auto& n : names()) puts(n.second.c_str());
    return 0;
  }
  char call[16], fail[64];
  long long N;
  int B, V, H, Hf, D, dtype, K, P;
  unsigned flags;
  float eps, T;
  while (scanf("%15s %lld %d %d %d %d %d %d %d %d %u %f %f %63s", call, &N, &B, &V, &H, &Hf, &D, &dtype, &K, &P, &flags, &eps, &T, fail) == 14) {
    // (nothing here is read or written by the host: any aligned address does)
    char* const at = reinterpret_cast<char*>(uintptr_t(1) << 40);
    float* const f = reinterpret_cast<float*>(at);
    int32_t* const i = reinterpret_cast<int32_t*>(at);
    uint8_t* const m = reinterpret_cast<uint8_t*>(at);
    aura_views_t views{V, H, H, Hf, Hf, D, dtype, f, f, at};
    aura_params_t par{0.01f, 1e-6f, T, eps, flags};
    std::vector<int64_t> pts(B + 1);
    std::vector<int32_t> vs(B + 1);
    for (int b = 0; b <= B; ++b) {
      pts[b] = N * b / B;
      vs[b] = V * b / B;
    }
    const int64_t* po = B > 1 ? pts.data() : nullptr;
    const int32_t* vo = B > 1 ? vs.data() : nullptr;
    g_fail = strcmp(fail, "-") ? fail : "";
    g_log.clear();
    g_error = 0;
    aura_time_next_fusion(reinterpret_cast<void*>(1), reinterpret_cast<void*>(2));
    const size_t ws = ~size_t(0);
    int s;
    if (!strcmp(call, "single"))
      s = aura_fuse_score_integrate(&views, &par, f, N, po, vo, B, f, AURA_F32, K, f, P, 0, nullptr, 1.0f, nullptr, nullptr, 0, i, m, V, f, f,
                                    i, f, nullptr, at, ws, nullptr);
    else if (!strcmp(call, "scores"))
      s = aura_fuse_scores(&views, &par, f, N, po, vo, B, f, AURA_F32, K, f, P, f, i, m, V, f, f, i, at, ws, nullptr);
    else if (!strcmp(call, "fuse"))
      s = aura_fuse_features(&views, &par, f, N, po, vo, B, f, i, at, ws, nullptr);
    else if (!strcmp(call, "densify"))   // (8 of B sources)
      s = aura_knn_densify(f, N, D, f, B, f, K, 8, f, P, &par, f, f, i, i, at, ws, nullptr);
    else
      s = aura_fuse_selected(&views, &par, f, N, po, vo, B, m, V, f, i, at, ws, nullptr);
    printf("%d%s\n", s, g_log.c_str());
  }
  return 0;
}
