// Device memory of a stated size, for tests: hipMalloc, hipFree and
// hipMemGetInfo with a count of the bytes held and a limit above which an
// allocation is refused.  Loaded before the HIP runtime, so that the library
// under test binds to these.
#include <dlfcn.h>

#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>

namespace {
std::mutex mu;
std::map<void*, size_t> held;
size_t used = 0, peak = 0, limit = SIZE_MAX;
template <class F>
F real(const char* name) {
  return reinterpret_cast<F>(dlsym(RTLD_NEXT, name) ? dlsym(RTLD_NEXT, name)
                                                    : dlsym(dlopen("libamdhip64.so", RTLD_NOW | RTLD_NOLOAD), name));
}
constexpr int kOutOfMemory = 2;  // hipErrorOutOfMemory
}  // namespace

extern "C" {

int hipMalloc(void** p, size_t bytes) {
  std::lock_guard<std::mutex> lock(mu);
  if (used + bytes > limit) return kOutOfMemory;
  const int e = real<int (*)(void**, size_t)>("hipMalloc")(p, bytes);
  if (e == 0 && *p) {
    held[*p] = bytes;
    used += bytes;
    if (used > peak) peak = used;
  }
  return e;
}

int hipFree(void* p) {
  std::lock_guard<std::mutex> lock(mu);
  const auto it = held.find(p);
  if (it != held.end()) {
    used -= it->second;
    held.erase(it);
  }
  return real<int (*)(void*)>("hipFree")(p);
}

int hipMemGetInfo(size_t* free_b, size_t* total_b) {
  std::lock_guard<std::mutex> lock(mu);
  if (limit == SIZE_MAX) return real<int (*)(size_t*, size_t*)>("hipMemGetInfo")(free_b, total_b);
  *free_b = limit > used ? limit - used : 0;
  *total_b = limit;
  return 0;
}

uint64_t limited_used() { return used; }
uint64_t limited_peak() { return peak; }
void limited_set(uint64_t bytes) {
  limit = bytes ? bytes : SIZE_MAX;
  peak = used;
}
}
