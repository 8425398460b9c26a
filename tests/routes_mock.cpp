// Stand-in for the HIP runtime calls of libidp_dg.so (preloaded into a process
// that only loads the library): device memory is host memory, kernels do not
// run, and every launch is written to stdout with its (mangled) name and
// grid, so that a test sees which kernels an entry point launches.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

struct dim3 { unsigned x, y, z; };
static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
static dim3 g_grid, g_block;
static size_t g_shm;
static void* g_stream;

extern "C" {
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "mock error"; }
int hipMalloc(void** p, size_t n) { *p = calloc(1, n + 1); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
int hipFree(void* p) { free(p); return 0; }
int hipHostFree(void* p) { return hipFree(p); }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { return hipMemset(d, v, n); }
int hipStreamSynchronize(void*) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void*, void*) { puts("event"); return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char a[4096]; *p = a; return 0; }
unsigned __hipPushCallConfiguration(dim3 g, dim3 b, size_t shm, void* s) {
  g_grid = g; g_block = b; g_shm = shm; g_stream = s;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shm, void** s) {
  *g = g_grid; *b = g_block; *shm = g_shm; *s = g_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, void*) {
  printf("%s %u\n", names()[f].c_str(), g.x);
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}
