// Test asset: stands in front of the HIP runtime's allocation calls (loaded before the library, with its symbols global) and
// makes device memory end at a budget, so that running out of it is an ordinary, repeatable error.
#include <dlfcn.h>

#include <cstddef>
#include <mutex>
#include <unordered_map>

namespace {
std::mutex mu;
std::unordered_map<void*, size_t> live;
size_t live_bytes = 0, budget = 0;   // budget 0: no end
int host_fails = 0;
constexpr int kSuccess = 0, kOutOfMemory = 2;

template <class F>
F real(const char* name)
{
    static void* hip = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);   // the library under test has it loaded
    return (F)dlsym(hip, name);
}
}  // namespace

extern "C" {
int hipMalloc(void** p, size_t bytes)
{
    std::lock_guard<std::mutex> lock(mu);
    if (budget && live_bytes + bytes > budget) return kOutOfMemory;
    const int rc = real<int (*)(void**, size_t)>("hipMalloc")(p, bytes);
    if (rc == kSuccess) {
        live[*p] = bytes;
        live_bytes += bytes;
    }
    return rc;
}

int hipFree(void* p)
{
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = live.find(p);
        if (it != live.end()) {
            live_bytes -= it->second;
            live.erase(it);
        }
    }
    return real<int (*)(void*)>("hipFree")(p);
}

int hipMemGetInfo(size_t* free_b, size_t* total_b)
{
    const int rc = real<int (*)(size_t*, size_t*)>("hipMemGetInfo")(free_b, total_b);
    std::lock_guard<std::mutex> lock(mu);
    if (rc == kSuccess && budget) *free_b = budget > live_bytes ? budget - live_bytes : 0;
    return rc;
}

int hipHostMalloc(void** p, size_t bytes, unsigned flags)
{
    return host_fails ? kOutOfMemory : real<int (*)(void**, size_t, unsigned)>("hipHostMalloc")(p, bytes, flags);
}

void shim_budget(size_t bytes)
{
    std::lock_guard<std::mutex> lock(mu);
    budget = bytes;
}
size_t shim_live()
{
    std::lock_guard<std::mutex> lock(mu);
    return live_bytes;
}
void shim_host_fails(int yes) { host_fails = yes; }
}
