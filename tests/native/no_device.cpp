// The HIP host calls that libg10.so makes, without a device: "device" memory is host memory, kernels do not run, and
// allocations fail from the n-th on where the test asks for it.  Beside them the array form of operator new that
// the library uses, counted.  Loaded ahead of the library (RTLD_GLOBAL) by tests/test_no_memory.py.
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <new>
#include <set>

typedef int Err;                                  // hipError_t: 0 success, 2 out of memory
struct Dim3 { uint32_t x, y, z; };

static std::set<void*>& blocks() { static std::set<void*>* s = new std::set<void*>(); return *s; }
static std::set<void*>& arrays() { static std::set<void*>* s = new std::set<void*>(); return *s; }
static long made = 0, fail_at = -1;

static Err take(void** out, size_t n) {
  if (made++ >= fail_at && fail_at >= 0) { *out = nullptr; return 2; }
  *out = calloc(1, n ? n : 1);
  blocks().insert(*out);
  return 0;
}
static Err give(void* p) { blocks().erase(p); free(p); return 0; }

extern "C" {
void test_fail_at(long n) { made = 0; fail_at = n; }
long test_made() { return made; }
long test_blocks() { return (long)blocks().size(); }
long test_arrays() { return (long)arrays().size(); }

Err hipGetDevice(int* d) { *d = 0; return 0; }
Err hipGetLastError() { return 0; }
const char* hipGetErrorString(Err) { return ""; }
Err hipMalloc(void** p, size_t n) { return take(p, n); }
Err hipFree(void* p) { return give(p); }
Err hipHostMalloc(void** p, size_t n, unsigned) { return take(p, n); }
Err hipHostFree(void* p) { return give(p); }
Err hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { memcpy(d, s, n); return 0; }
Err hipMemsetAsync(void* d, int v, size_t n, void*) { memset(d, v, n); return 0; }
Err hipStreamSynchronize(void*) { return 0; }
Err hipStreamCreateWithFlags(void** s, unsigned) { *s = (void*)1; return 0; }
Err hipStreamDestroy(void*) { return 0; }
Err hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
Err hipEventCreate(void** e) { *e = (void*)1; return 0; }
Err hipEventDestroy(void*) { return 0; }
Err hipEventRecord(void*, void*) { return 0; }
Err hipEventElapsedTime(float* ms, void*, void*) { *ms = 0; return 0; }
Err hipFuncSetAttribute(const void*, int, int) { return 0; }
Err hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*) { return 0; }
Err hipExtLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*, void*, void*, int) { return 0; }
}

void* operator new[](size_t n, const std::nothrow_t&) noexcept {
  void* p = malloc(n ? n : 1);
  if (p) arrays().insert(p);
  return p;
}
void operator delete[](void* p) noexcept { arrays().erase(p); free(p); }
void operator delete[](void* p, size_t) noexcept { arrays().erase(p); free(p); }
