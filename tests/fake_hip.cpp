// A stand-in for the HIP runtime and hipFFT on a host without a device: memory is host memory, kernels
// and transforms do nothing, and one chosen call of them fails.  Loaded before libtfs.so, its symbols
// take the place of the real ones (tests/test_launch_errors.py).
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>

namespace {
long calls = 0, fail_at = -1;
int last = 0, plans = 0;
size_t refuse_new = 0;
struct Dim3 { uint32_t x, y, z; };

int call(int error) {
  if (calls++ != fail_at) return 0;
  return error;
}
}  // namespace

extern "C" {
// fail the k-th call from now on (k < 0: none)
void fake_fail_at(long k) { calls = 0; fail_at = k; last = 0; }
long fake_calls() { return calls; }
int fake_plans() { return plans; }
// host allocations of `bytes` or more throw (0: none)
void fake_refuse_new(size_t bytes) { refuse_new = bytes; }

int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*) {
  const int e = call(719);
  if (e) last = e;
  return e;
}
int hipGetLastError() { const int e = last; last = 0; return e; }
const char* hipGetErrorString(int) { return "stand-in failure"; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  const int e = call(719);
  if (e) return last = e;
  std::memcpy(d, s, n);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return 0; }
int hipMalloc(void** p, size_t n) { *p = std::calloc(n ? n : 1, 1); return *p ? 0 : 2; }
int hipFree(void* p) { std::free(p); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 0; return 1; }     // the library's defaults
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { static double scratch[1 << 17]; *p = scratch; return 0; }
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) {
  *g = *b = Dim3{1, 1, 1};
  *s = 0;
  *st = nullptr;
  return 0;
}
int hipfftPlanMany(void** h, int, int*, int*, int, int, int*, int, int, int, int) { *h = &last; ++plans; return 0; }
int hipfftDestroy(void*) { --plans; return 0; }
int hipfftSetStream(void*, void*) { return 0; }
int hipfftExecD2Z(void*, double*, void*) { return call(6); }
int hipfftExecZ2D(void*, void*, double*) { return call(6); }
}

void* operator new(size_t n) {
  if (refuse_new && n >= refuse_new) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
