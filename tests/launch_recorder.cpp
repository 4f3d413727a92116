// The HIP runtime calls of libkvcrush.so, replaced for a process without a GPU: launches are written
// down (kernel, grid, block, dynamic LDS, and of a score kernel's parameters S, n_bh, n_pieces and turn) instead of run.  Loaded with RTLD_GLOBAL before the library,
// so that the library's references find these definitions first.
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <map>
#include <string>

struct Dim3 {
  uint32_t x, y, z;
};
static std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> names;
  return names;
}
static std::string log_text;
static char symbol_memory[256];

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetDevice(int* dev) {
  *dev = 0;
  return 0;
}
int hipGetSymbolAddress(void** ptr, const void*) {
  *ptr = (void*)(((uintptr_t)symbol_memory + 255) & ~(uintptr_t)255);
  return 0;
}
// As the runtime does: a launch of 2^32 threads or more along a dimension, an empty one, or one with too
// many workgroups along y or z is refused.
int hipLaunchKernel(const void* host, Dim3 grid, Dim3 block, void** args, size_t lds, void*) {
  const bool refused = !grid.x || !grid.y || !grid.z || (uint64_t)grid.x * block.x > 0xFFFFFFFFull || grid.y > 65535 || grid.z > 65535;
  char line[256];
  const int n = snprintf(line, sizeof line, " %u %u %u %u %zu %d", grid.x, grid.y, grid.z, block.x, lds, refused ? 1 : 0);
  if (kernels()[host].find("ScoreParams") != std::string::npos) {
    const int32_t* p = (const int32_t*)((const char*)args[0] + 88);  // B, Hq, Hkv, S, G, reduce_groups, heads_per_wg, n_blocks, ...
    snprintf(line + n, sizeof line - n, " %d %d %d %d\n", p[3], p[8], p[9], p[10]);
  } else {
    snprintf(line + n, sizeof line - n, "\n");
  }
  log_text += kernels()[host] + line;
  return refused ? 9 : 0;
}
const char* recorded(void) { return log_text.c_str(); }
void forget(void) { log_text.clear(); }
}
