// hip_host_stub.cpp -- the HIP calls that libfaco_hip.so makes, on host memory
// and without a device: loaded ahead of the library (RTLD_GLOBAL) they take the
// runtime's place, so that a CPU test can read what the library's host code
// does: the launches it makes (grid, block, LDS), the copies it enqueues, the
// host memory it allocates.  Kernels do not run.  Every copy of a DevState to
// the host reports the initial search as ended.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

// the device header's structures (their layout only)
#define __device__
#define __host__
#define __forceinline__ inline
struct int2 { int x, y; };
struct alignas(16) int4 { int x, y, z, w; };
#include "../paper_2203_02228_amd/csrc/faco_device.hpp"

struct Dim3 { uint32_t x, y, z; };
struct Launch { uint32_t grid[3], block[3]; uint64_t lds; };

static std::vector<Launch> g_launch;
static int64_t g_copies, g_news, g_events;
static int g_capturing, g_blocks_per_cu = 8;
static struct { Dim3 g, b; size_t lds; void *s; } g_cfg;
static unsigned char g_scratch[1 << 20];

void *operator new(size_t n) {
  ++g_news;
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept {
  ++g_news;
  return std::malloc(n ? n : 1);
}
void *operator new[](size_t n) { return operator new(n); }
void *operator new[](size_t n, const std::nothrow_t &t) noexcept { return operator new(n, t); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
void operator delete[](void *p) noexcept { std::free(p); }

extern "C" {

void stub_reset() {
  g_launch.clear();
  g_launch.reserve(4096);
  g_copies = g_news = g_events = 0;
}
int stub_launch_count() { return (int)g_launch.size(); }
void stub_launch(int i, uint64_t *out) {
  const Launch &L = g_launch[(size_t)i];
  for (int k = 0; k < 3; ++k) {
    out[k] = L.grid[k];
    out[3 + k] = L.block[k];
  }
  out[6] = L.lds;
}
int64_t stub_copies() { return g_copies; }
int64_t stub_news() { return g_news; }
int64_t stub_events() { return g_events; }
void stub_set_capturing(int on) { g_capturing = on; }
void stub_set_blocks_per_cu(int n) { g_blocks_per_cu = n; }

int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void *s) {
  g_cfg = {g, b, lds, s};
  return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **s) {
  *g = g_cfg.g;
  *b = g_cfg.b;
  *lds = g_cfg.lds;
  *s = g_cfg.s;
  return 0;
}
int hipLaunchKernel(const void *, Dim3 g, Dim3 b, void **, size_t lds, void *) {
  g_launch.push_back({{g.x, g.y, g.z}, {b.x, b.y, b.z}, lds});
  return 0;
}
int hipMalloc(void **p, size_t n) {
  *p = std::calloc(1, n);
  return *p ? 0 : 2;
}
int hipFree(void *p) {
  std::free(p);
  return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *) {
  if (n <= (1u << 20)) std::memset(p, v, n);
  return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *) {
  ++g_copies;
  std::memcpy(d, s, n);
  if (kind == 2 && n == sizeof(faco::DevState)) ((faco::DevState *)d)->init_done = 1;
  return 0;
}
// 900: hipErrorStreamCaptureUnsupported
int hipStreamSynchronize(void *) { return g_capturing ? 900 : 0; }
int hipStreamIsCapturing(void *, int *status) {
  *status = g_capturing ? 1 : 0;
  return 0;
}
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) {
  *s = g_scratch;
  return 0;
}
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) {
  *g = g_scratch;
  return 0;
}
int hipGraphInstantiate(void **x, void *, void **, char *, size_t) {
  *x = g_scratch;
  return 0;
}
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipEventCreate(void **e) {
  ++g_events;
  *e = g_scratch;
  return 0;
}
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) {
  *ms = 1.0f;
  return 0;
}
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *d) {
  *d = 0;
  return 0;
}
int hipDeviceGetAttribute(int *v, int, int) {
  *v = 256;  // compute units
  return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = g_blocks_per_cu;
  return 0;
}
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int e) { return e == 900 ? "stream is capturing" : "error"; }
int hipGetSymbolAddress(void **p, const void *) {
  *p = g_scratch;
  return 0;
}

}  // extern "C"
