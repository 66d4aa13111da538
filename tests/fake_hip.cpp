// Stand-in for the HIP runtime on a machine without a GPU: device memory is host
// memory up to a limit, launches do nothing.  Loaded before libshk.so, it lets the
// CPU tests see what the library allocates, keeps and frees.
#include <chrono>
#include <condition_variable>
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>

namespace {
std::mutex mu;
constexpr size_t HEAD = 64;   // a block's size stands before it
size_t live = 0, limit = ~size_t(0);
int last = 0;
constexpr int OOM = 2;
// a gate that hipFree waits at: 0 open, 1 armed, 2 a caller waits
std::condition_variable cv;
int gate = 0;

int alloc(void** p, size_t bytes) {
  std::lock_guard<std::mutex> g(mu);
  if (bytes > limit - (live < limit ? live : limit)) return last = OOM;
  char* q = static_cast<char*>(std::calloc(bytes + HEAD, 1));
  std::memcpy(q, &bytes, sizeof bytes);
  *p = q + HEAD;
  live += bytes;
  return 0;
}
int release(void* p) {
  std::unique_lock<std::mutex> g(mu);
  if (!p) return 0;
  if (gate == 1) {
    gate = 2;
    cv.notify_all();
    cv.wait_for(g, std::chrono::seconds(10), [] { return gate == 0; });
    gate = 0;
  }
  char* q = static_cast<char*>(p) - HEAD;
  size_t bytes;
  std::memcpy(&bytes, q, sizeof bytes);
  live -= bytes;
  std::free(q);
  return 0;
}
int no_new = 0;
}  // namespace

// the library's host allocations
void* operator new(size_t n) {
  if (no_new) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
size_t fake_live() { std::lock_guard<std::mutex> g(mu); return live; }
void fake_limit(size_t bytes) { std::lock_guard<std::mutex> g(mu); limit = bytes; }
void fake_no_new(int on) { no_new = on; }   // from now on they fail
void fake_gate_arm() { std::lock_guard<std::mutex> g(mu); gate = 1; }
int fake_gate_entered() {   // waits until a hipFree stands at the gate
  std::unique_lock<std::mutex> g(mu);
  return cv.wait_for(g, std::chrono::seconds(10), [] { return gate == 2; });
}
int fake_gate_open() {      // 1 if it still stood there
  std::lock_guard<std::mutex> g(mu);
  const int held = gate == 2;
  gate = 0;
  cv.notify_all();
  return held;
}

int hipMalloc(void** p, size_t n) { return alloc(p, n); }
int hipMallocAsync(void** p, size_t n, void*) { return alloc(p, n); }
int hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(n, 1); return 0; }
int hipHostFree(void* p) { std::free(p); return 0; }
int hipFree(void* p) { return release(p); }
int hipFreeAsync(void* p, void*) { return release(p); }
int hipMemcpy(void* d, const void* s, size_t n, int) { std::memmove(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { std::memmove(d, s, n); return 0; }
int hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { std::memset(d, v, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { const int e = last; last = 0; return e; }
const char* hipGetErrorString(int) { return "fake"; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { *s = nullptr; return 0; }
int hipStreamDestroy(void*) { return 0; }
int hipEventCreate(void** e) { *e = nullptr; return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = nullptr; return 1; }
int hipStreamBeginCapture(void*, int) { return 1; }
int hipStreamEndCapture(void*, void**) { return 1; }
int hipGraphInstantiate(void**, void*, void**, char*, size_t) { return 1; }
int hipGraphLaunch(void*, void*) { return 1; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }

struct Dim { unsigned x, y, z; };
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { return 0; }
int __hipPushCallConfiguration(Dim, Dim, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* s, void** st) {
  *g = *b = Dim{1, 1, 1};
  *s = 0;
  *st = nullptr;
  return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* h = nullptr; return &h; }
void __hipRegisterFunction() {}
void __hipRegisterVar() {}
void __hipUnregisterFatBinary(void**) {}
}
