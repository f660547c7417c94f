// A HIP runtime without a device, for tests of the library's host code: memory is host memory that is never touched by a kernel, launches are
// noted down and do nothing.  Loaded ahead of the library (RTLD_GLOBAL), so that its calls come here.
#include <stddef.h>
#include <string.h>
#include <sys/mman.h>

#include <map>
#include <string>

namespace {

struct Dim3 {
  unsigned x, y, z;
};
constexpr int kSuccess = 0, kOutOfMemory = 2;
std::map<const void*, std::string>& names() {                  // (the library registers its kernels before main)
  static std::map<const void*, std::string> m;
  return m;
}
std::map<void*, size_t> g_blocks;
std::string g_log;
size_t g_capacity = ~(size_t)0, g_used = 0, g_most = 0;
int g_last_error = kSuccess, g_capturing = 0;
Dim3 g_grid, g_block;
size_t g_lds;
void* g_stream;
char g_symbol[64];

}  // namespace

extern "C" {

// ---- for the test
void stub_capacity(size_t bytes) { g_capacity = bytes; }
size_t stub_used() { return g_used; }
size_t stub_most() { const size_t m = g_most; g_most = g_used; return m; }   // since the last call
void stub_capturing(int yes) { g_capturing = yes; }
int stub_last_error() { return g_last_error; }
const char* stub_log() { return g_log.c_str(); }               // "kernel grid.x\n" of every launch
void stub_clear_log() { g_log.clear(); }

// ---- the runtime
int hipMalloc(void** p, size_t n) {
  if (n > g_capacity - g_used || g_capacity < g_used) {
    *p = nullptr;
    return g_last_error = kOutOfMemory;
  }
  void* at = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (at == MAP_FAILED) return g_last_error = kOutOfMemory;
  g_blocks[at] = n;
  g_used += n;
  if (g_used > g_most) g_most = g_used;
  *p = at;
  return kSuccess;
}
int hipFree(void* p) {
  if (!p) return kSuccess;
  auto it = g_blocks.find(p);
  if (it == g_blocks.end()) return g_last_error = 1;
  munmap(p, it->second ? it->second : 1);
  g_used -= it->second;
  g_blocks.erase(it);
  return kSuccess;
}
int hipGetLastError() {
  const int e = g_last_error;
  g_last_error = kSuccess;
  return e;
}
int hipGetDevice(int* d) { *d = 0; return kSuccess; }
int hipDeviceGetAttribute(int* v, int attribute, int) {
  *v = attribute == 63 ? 256 : 160 * 1024;                     // hipDeviceAttributeMultiprocessorCount, else the LDS of a workgroup
  return kSuccess;
}
int hipDeviceSynchronize() { return kSuccess; }
int hipStreamSynchronize(void*) { return kSuccess; }
int hipStreamIsCapturing(void*, int* status) { *status = g_capturing; return kSuccess; }
int hipEventCreate(void** e) { *e = nullptr; return kSuccess; }
int hipEventDestroy(void*) { return kSuccess; }
int hipEventRecord(void*, void*) { return kSuccess; }
int hipEventSynchronize(void*) { return kSuccess; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0.f; return kSuccess; }
int hipFuncSetAttribute(const void*, int, int) { return kSuccess; }
int hipMemcpy(void* to, const void* from, size_t n, int) { memcpy(to, from, n); return kSuccess; }
int hipMemset(void* p, int v, size_t n) { memset(p, v, n); return kSuccess; }
int hipGetSymbolAddress(void** p, const void*) { *p = g_symbol; return kSuccess; }
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void**, size_t, void*) {
  g_log += names()[f] + " " + std::to_string(grid.x) + "\n";
  return kSuccess;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  g_grid = grid; g_block = block; g_lds = lds; g_stream = stream;
  return kSuccess;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = g_grid; *block = g_block; *lds = g_lds; *stream = g_stream;
  return kSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, Dim3*, Dim3*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"
