// csrc/pool.cpp over a device of 64 MiB whose allocations only count bytes.
#include <cstdlib>
#include <map>

#include "../paper_2112_10913_amd/csrc/api_internal.h"

namespace {

std::map<void*, size_t> g_device, g_pinned;
size_t g_used = 0, g_capacity = (size_t)64 << 20;
int g_calls = 0;

}  // namespace

extern "C" {

hipError_t hipGetDevice(int* dev)
{
    *dev = 0;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes)
{
    ++g_calls;
    const size_t held = (bytes + 4095) / 4096 * 4096;      // whole pages
    if (g_used + held > g_capacity) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    g_device[*p] = held;
    g_used += held;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    const auto it = g_device.find(p);
    if (it == g_device.end()) return hipErrorInvalidValue;
    g_used -= it->second;
    g_device.erase(it);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned)
{
    *p = std::malloc(1);
    g_pinned[*p] = bytes;
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    g_pinned.erase(p);
    std::free(p);
    return hipSuccess;
}

// for the test
void replay_capacity(size_t bytes) { g_capacity = bytes; }
size_t replay_used() { return g_used; }
int replay_calls() { return g_calls; }
int replay_pinned() { return (int)g_pinned.size(); }
void* replay_pool_malloc(size_t bytes)
{
    void* p;
    return citron::pool_malloc(&p, bytes) == hipSuccess ? p : nullptr;
}
void replay_pool_free(void* p) { citron::pool_free(p); }
void* replay_device_malloc(size_t bytes)
{
    void* p;
    return citron::device_malloc(&p, bytes) == hipSuccess ? p : nullptr;
}
void replay_device_free(void* p) { (void)hipFree(p); }
void* replay_host_malloc(size_t bytes)
{
    void* p;
    return citron::pool_host_malloc(&p, bytes) == hipSuccess ? p : nullptr;
}
void replay_host_free(void* p, size_t bytes) { citron::pool_host_free(p, bytes); }
void replay_release() { citron::pool_release(); }

}  // extern "C"
