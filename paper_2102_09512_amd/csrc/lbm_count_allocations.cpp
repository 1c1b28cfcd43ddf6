// Linked into the debug library liblbm_counted.so with --wrap=hipMalloc: counts
// the library's device allocations (hipMalloc is the only call that it makes
// them by), so a test can hold an entry point to none.
#include <atomic>
#include <cstddef>

namespace {
std::atomic<long long> count{0};
}

extern "C" {

int __real_hipMalloc(void** p, size_t bytes);

int __wrap_hipMalloc(void** p, size_t bytes) {
  ++count;
  return __real_hipMalloc(p, bytes);
}

long long lbm_debug_allocations() { return count; }
}
