// launches.cpp -- the HIP stand-in of hip_stub.cpp as part of a shared library
// with libgap's host code, for tests that drive the C ABI from Python and look
// at what the host does: which kernels it launches with which grids, what it
// allocates, and host copies that do not wait for work queued on a
// non-blocking stream.  Test infrastructure: no kernel runs, but the two that
// only move words (k_gather, k_raise) are carried out here.
#include <hip/hip_runtime_api.h>

#define __hipRegisterFunction stub_register_function
#define hipLaunchKernel stub_launch_kernel
#define hipExtLaunchKernel stub_ext_launch_kernel
#define hipMalloc stub_malloc
#define hipMemcpy stub_memcpy
#define hipMemsetAsync stub_memset_async
#define hipStreamSynchronize stub_stream_synchronize
// (declared first: the stand-in's own definitions get the other names)
extern "C" {
hipError_t stub_launch_kernel(const void*, dim3, dim3, void**, size_t, hipStream_t);
hipError_t stub_malloc(void**, size_t);
hipError_t stub_memcpy(void*, const void*, size_t, hipMemcpyKind);
hipError_t stub_memset_async(void*, int, size_t, hipStream_t);
hipError_t stub_stream_synchronize(hipStream_t);
}
#include "hip_stub.cpp"
#undef __hipRegisterFunction
#undef hipLaunchKernel
#undef hipExtLaunchKernel
#undef hipMalloc
#undef hipMemcpy
#undef hipMemsetAsync
#undef hipStreamSynchronize

#include <new>

// host allocations of at least g_fail_at bytes fail (the stand-in and the
// recorder make none of more than about 600)
static size_t g_fail_at = ~(size_t)0;
void* operator new(size_t n) {
  void* p = n >= g_fail_at ? nullptr : malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

namespace {

struct Launch { std::string name; unsigned grid; };
struct Fill { uintptr_t lo, hi; };
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;   // (kernels are registered before this file's globals)
  return m;
}
std::deque<Launch> g_launches;
std::map<hipStream_t, std::deque<Fill>> g_fills;   // enqueued on non-blocking streams, not waited for
std::deque<std::string> g_races;
std::map<hipStream_t, long long> g_queued;          // launches since the stream was last waited for
long long g_allocs = 0;
long long* g_status = nullptr;                      // the library's status words: {error, chunks + 1 of both stores}

void record(const void* f, dim3 g, void** a) {
  const std::string& n = names()[f];
  g_launches.push_back({n, g.x * g.y * g.z});
  if (n.find("k_gather") != std::string::npos) {
    const char* status = *(char**)a[0];
    const char* src = *(char**)a[1];
    const long long words = *(long long*)a[2];
    char* out = *(char**)a[3];
    memcpy(out, status, 24);
    memcpy(out + 64, src, 4 * words);
  }
  if (n.find("k_raise") != std::string::npos) **(int**)a[0] |= *(int*)a[1];
}

// a host copy runs ahead of what non-blocking streams still hold
void check_race(const void* p, size_t n, const char* what) {
  const uintptr_t lo = (uintptr_t)p, hi = lo + n;
  for (auto& s : g_fills)
    for (const Fill& f : s.second)
      if (lo < f.hi && f.lo < hi) {
        char buf[128];
        snprintf(buf, sizeof buf, "%s of %zu bytes does not wait for the fill of its memory", what, n);
        g_races.push_back(buf);
        return;
      }
}

}  // namespace

extern "C" {

void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned int l, void* a, void* b,
                           void* c, void* d, int* e) {
  names()[host] = name;
  stub_register_function(m, host, dev, name, l, a, b, c, d, e);
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t sh, hipStream_t s) {
  record(f, g, a);
  ++g_queued[s];
  return stub_launch_kernel(f, g, b, a, sh, s);
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t sh, hipStream_t s, hipEvent_t start,
                              hipEvent_t stop, int fl) {
  record(f, g, a);
  ++g_queued[s];
  return stub_ext_launch_kernel(f, g, b, a, sh, s, start, stop, fl);
}
hipError_t hipMalloc(void** p, size_t n) {
  ++g_allocs;
  return stub_malloc(p, n);
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyHostToDevice) check_race(d, n, "copy to the device");
  if (k == hipMemcpyDeviceToHost) check_race(s, n, "copy to the host");
  if (k == hipMemcpyDeviceToHost && n == 24) g_status = (long long*)s;
  return stub_memcpy(d, s, n, k);
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t s) {
  if (s && (S(s)->flags & hipStreamNonBlocking)) g_fills[s].push_back({(uintptr_t)p, (uintptr_t)p + n});
  return stub_memset_async(p, v, n, s);
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  g_fills.erase(s);
  g_queued.erase(s);
  return stub_stream_synchronize(s);
}

// ---- what the tests ask
void* rec_stream(void) {
  hipStream_t s = nullptr;
  hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  return s;
}
void rec_fail_at(long long n) { g_fail_at = n < 0 ? ~(size_t)0 : (size_t)n; }
void rec_clear(void) { g_launches.clear(); }
long long rec_count(void) { return (long long)g_launches.size(); }
const char* rec_name(long long i) { return g_launches[(size_t)i].name.c_str(); }
long long rec_grid(long long i) { return g_launches[(size_t)i].grid; }
long long rec_queued(void) {
  long long n = 0;
  for (auto& q : g_queued) n += q.second;
  return n;
}
long long rec_allocs(void) { return g_allocs; }
long long rec_races(void) { return (long long)g_races.size(); }
const char* rec_race(long long i) { return g_races[(size_t)i].c_str(); }
// the chunks the last re-sort left, as the next synchronising call reads them
void rec_set_chunks(long long lep, long long pho) {
  g_status[1] = lep + 1;
  g_status[2] = pho + 1;
}

}  // extern "C"
