// The HIP calls that libqd makes, on a machine without a GPU: device and pinned memory come from the heap
// and are counted, copies are made at once, kernels are recorded and not run. Loaded ahead of the HIP
// runtime by the tests of the library's host side: what it allocates, launches and does when an
// allocation fails.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

struct Dim3 { uint32_t x, y, z; };
struct Launch { const char* name; Dim3 grid, block; size_t lds; };

static std::mutex mu;
static std::map<void*, size_t> live[2];               // 0: device, 1: pinned
static size_t held[2], peak[2];
static long long made[2], limit[2] = {-1, -1};        // allocations made; bytes that may be held (-1: any)
static int capturing = 0, last_error = 0;
static long long waits = 0;
static std::map<const void*, std::string> names;
static std::vector<Launch> launched;
static thread_local struct { Dim3 grid, block; size_t lds; void* stream; } config;

static int take(int kind, void** p, size_t n) {
  std::lock_guard<std::mutex> lock(mu);
  if (limit[kind] >= 0 && held[kind] + n > size_t(limit[kind])) return last_error = 2;   // out of memory
  *p = std::malloc(n ? n : 1);
  live[kind][*p] = n;
  held[kind] += n;
  if (held[kind] > peak[kind]) peak[kind] = held[kind];
  ++made[kind];
  return 0;
}

static int give(int kind, void* p) {
  std::lock_guard<std::mutex> lock(mu);
  if (!p) return 0;
  auto it = live[kind].find(p);
  if (it == live[kind].end()) return last_error = 1;
  held[kind] -= it->second;
  live[kind].erase(it);
  std::free(p);
  return 0;
}

extern "C" {
// what the tests ask and set
long long host_held(int kind) { return (long long)held[kind]; }
long long host_peak(int kind) { return (long long)peak[kind]; }
long long host_made(int kind) { return made[kind]; }
long long host_waits() { return waits; }
void host_limit(int kind, long long bytes) { limit[kind] = bytes; }
void host_capture(int on) { capturing = on; }
void host_reset() {
  launched.clear();
  for (int k = 0; k < 2; ++k) {
    peak[k] = held[k];
    made[k] = 0;
  }
  waits = 0;
}
int host_launches() { return int(launched.size()); }
const char* host_launch(int i, uint32_t* grid, uint32_t* block, uint64_t* lds) {
  *grid = launched[size_t(i)].grid.x;
  *block = launched[size_t(i)].block.x;
  *lds = launched[size_t(i)].lds;
  return launched[size_t(i)].name;
}

// the runtime
int hipGetDevice(int* d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipMalloc(void** p, size_t n) { return take(0, p, n); }
int hipFree(void* p) { return give(0, p); }
int hipHostMalloc(void** p, size_t n, unsigned) { return take(1, p, n); }
int hipHostFree(void* p) { return give(1, p); }
int hipMemcpy(void* d, const void* s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { std::memcpy(d, s, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { std::memset(d, v, n); return 0; }
int hipStreamSynchronize(void*) { ++waits; return 0; }
int hipStreamIsCapturing(void*, int* s) {   // -1: the null stream beside another thread's capture
  *s = capturing;
  return capturing < 0 ? last_error = 906 : 0;
}
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "refused by the test"; }
int hipEventCreate(void** e) { *e = std::malloc(1); return 0; }
int hipEventDestroy(void* e) { std::free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.0f; return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  config = {grid, block, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
  std::lock_guard<std::mutex> lock(mu);
  launched.push_back(Launch{names[f].c_str(), grid, block, lds});
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}
