// The HIP runtime calls that libmfgmg.so makes, on host memory: what the
// library's device set-up does with failed calls can then be tested without a
// GPU.  Kernels are never run; a copy from the device delivers
// ones, so that the host's part of the set-up (eigenvalue estimates, coarse
// factorisation, pressure mass) sees well-posed numbers.  Loaded with
// RTLD_GLOBAL before the library, these definitions are found first.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>

namespace {
int64_t mallocs = 0, fail_malloc = 0, copies = 0, fail_copy = 0, uploaded = 0, held = 0;
int64_t news = 0, fail_new = 0;
constexpr int kOutOfMemory = 2, kInvalid = 1;

int copy(void* dst, const void* src, size_t n, int kind) {
  if (kind == 2) {   // device to host
    const double one = 1.0;
    for (size_t i = 0; i + sizeof(one) <= n; i += sizeof(one)) std::memcpy(static_cast<char*>(dst) + i, &one, sizeof(one));
  } else {
    std::memcpy(dst, src, n);
  }
  return 0;
}
}  // namespace

extern "C" {
// the n-th call from now fails (0: none): hipMalloc, synchronous hipMemcpy,
// operator new of the library's host code (from the n-th on)
void stub_fail_malloc(int64_t n) { mallocs = 0, fail_malloc = n; }
void stub_fail_copy(int64_t n) { copies = 0, fail_copy = n; }
void stub_fail_new(int64_t n) { news = 0, fail_new = n; }
int64_t stub_mallocs() { return mallocs; }
int64_t stub_copies() { return copies; }
int64_t stub_uploaded() { return uploaded; }   // bytes, synchronous copies
int64_t stub_news() { return news; }
int64_t stub_held() { return held; }   // device allocations not freed

int hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (++mallocs == fail_malloc) return kOutOfMemory;
  *p = std::calloc(n ? n : 1, 1);
  held += *p != nullptr;
  return *p ? 0 : kOutOfMemory;
}
int hipFree(void* p) {
  held -= p != nullptr;
  std::free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(n ? n : 1, 1);
  return *p ? 0 : kOutOfMemory;
}
int hipHostFree(void* p) {
  std::free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int kind) {
  uploaded += kind == 1 ? int64_t(n) : 0;
  return ++copies == fail_copy ? kInvalid : copy(d, s, n, kind);
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*) { return copy(d, s, n, kind); }
int hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) { return hipMemset(d, v, n); }
int hipMemcpyToSymbol(const void*, const void*, size_t, size_t, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  *p = nullptr;
  return kInvalid;
}
int hipLaunchKernel(const void*, ...) {
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int e) { return e ? "failed" : "no error"; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) {
  *s = nullptr;
  return 0;
}
int hipStreamDestroy(void*) { return 0; }
int hipStreamBeginCapture(void*, int) { return kInvalid; }
int hipStreamEndCapture(void*, void**) { return kInvalid; }
int hipGraphInstantiate(void**, void*, void*, char*, size_t) { return kInvalid; }
int hipGraphLaunch(void*, void*) { return kInvalid; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int __hipPushCallConfiguration(...) { return 0; }
int __hipPopCallConfiguration(...) { return 0; }
void* __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipRegisterFunction(...) {}
void __hipRegisterVar(...) {}
void __hipUnregisterFatBinary(void*) {}
}

void* operator new(size_t n) {
  ++news;
  if (fail_new && news >= fail_new) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
