// Test asset: stands in front of the HIP runtime's launch call (loaded before the library, with its symbols global) and notes the
// name and the grid of every kernel that is launched.
#include <dlfcn.h>

#include <cstring>
#include <mutex>
#include <string>
#include <unordered_map>

namespace {
std::mutex mu;
std::unordered_map<const void*, std::string> names;
std::string seen;

template <class F>
F real(const char* name)
{
    static void* hip = dlopen("libamdhip64.so.7", RTLD_LAZY);
    return (F)dlsym(hip, name);
}
struct Dim3 {
    unsigned x, y, z;
};
}  // namespace

extern "C" {
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid, void* block, void* grid,
                           int* warp)
{
    {
        std::lock_guard<std::mutex> lock(mu);
        names[host] = name;
    }
    real<decltype(&__hipRegisterFunction)>("__hipRegisterFunction")(modules, host, device, name, limit, tid, bid, block, grid, warp);
}

int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t lds, void* stream)
{
    {
        std::lock_guard<std::mutex> lock(mu);
        seen += names[f] + " " + std::to_string(grid.x) + "," + std::to_string(grid.y) + "," + std::to_string(grid.z) + "\n";
    }
    return real<int (*)(const void*, Dim3, Dim3, void**, size_t, void*)>("hipLaunchKernel")(f, grid, block, args, lds, stream);
}

// The launches since the last call, one a line; their number of bytes, or what a longer buffer would take.
size_t shim_launches(char* out, size_t room)
{
    std::lock_guard<std::mutex> lock(mu);
    const size_t n = seen.size();
    if (n <= room) {
        std::memcpy(out, seen.data(), n);
        seen.clear();
    }
    return n;
}
}
