// device_cus() of the library's host code, with a HIP runtime of two calls that
// counts, and operator new that counts: prints the compute units it gives for
// devices 0, 3, 3, 0 and 70, the attribute queries and the allocations.
#include <cstdio>
#include <cstdlib>
#include <new>

#include <hip/hip_runtime_api.h>

#include "internal.hpp"

static int g_dev = 0, g_queries = 0;
static long g_allocs = 0;

extern "C" hipError_t hipGetDevice(int* dev) {
  *dev = g_dev;
  return hipSuccess;
}
extern "C" hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int dev) {
  ++g_queries;
  *v = 100 + dev;
  return hipSuccess;
}
void* operator new(size_t n) {
  ++g_allocs;
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
  int got[5], i = 0;
  g_allocs = 0;
  for (int d : {0, 3, 3, 0, 70}) {
    g_dev = d;
    got[i++] = bitsmoe::device_cus();
  }
  const long allocs = g_allocs;
  std::printf("%d %d %d %d %d %d %ld\n", got[0], got[1], got[2], got[3], got[4], g_queries, allocs);
}
