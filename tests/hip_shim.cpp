// Stands between libdc.so and the HIP runtime in the tests of failing calls
// (loaded with RTLD_GLOBAL before either): memory that runs out after a number
// of allocations, and launches that never happen.
#include <dlfcn.h>

#include <atomic>
#include <cstddef>

namespace {

constexpr int OUT_OF_MEMORY = 2;  // hipErrorOutOfMemory
struct Dim3 {
  unsigned x, y, z;
};
std::atomic<long> allow{-1};    // allocations until they fail (-1: never)
std::atomic<int> last{0};       // the error that the failing allocation leaves behind
std::atomic<long> launches{0};  // seen so far
std::atomic<long> drop_from{-1};  // launches from this one on are dropped (-1: none)

template <class F>
F real(const char* name) {
  static void* const lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
  return reinterpret_cast<F>(dlsym(lib, name));
}

}  // namespace

extern "C" {

void shim_allow(long n) { allow = n; }
void shim_drop_from(long n) { drop_from = n; }
long shim_launches() { return launches; }

int hipMalloc(void** p, size_t n) {
  static const auto f = real<int (*)(void**, size_t)>("hipMalloc");
  if (allow == 0) {
    last = OUT_OF_MEMORY;
    return OUT_OF_MEMORY;
  }
  if (allow > 0) --allow;
  return f(p, n);
}

int hipGetLastError() {
  static const auto f = real<int (*)()>("hipGetLastError");
  const int e = last.exchange(0);
  return e ? e : f();
}

int hipLaunchKernel(const void* fn, Dim3 grid, Dim3 block, void** args, size_t lds, void* stream) {
  static const auto f =
      real<int (*)(const void*, Dim3, Dim3, void**, size_t, void*)>("hipLaunchKernel");
  const long i = launches++;
  if (drop_from >= 0 && i >= drop_from) return 0;
  return f(fn, grid, block, args, lds, stream);
}
}
