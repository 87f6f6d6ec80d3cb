// Reuse of device and pinned host blocks between graph handles.
//
// A graph that comes in, is counted and goes makes and drops about thirty
// device blocks and a pinned one; hipMalloc, hipFree (which waits for the
// device) and hipHostMalloc were 5.5 of the 18.2 ms of load + order + counts
// of a 2^20-vertex graph and more than half of the 0.44 ms of a 2^8-vertex
// one.  Freed blocks are kept, at most kPoolBytes per device and
// kPoolHostBlocks pinned ones, the oldest given back first, all of them when
// an allocation fails, here or through device_malloc, which the library's
// other device memory comes from, or when the program asks (pool_release).  A
// block is only handed to pool_free once the work that
// used it has completed, so its next owner may use it on any stream.
#include "api_internal.h"

#include <list>
#include <unordered_map>

namespace citron {

namespace {

constexpr size_t kPoolBytes = (size_t)1 << 30;        // cached per device
constexpr size_t kPoolMaxBlock = (size_t)1 << 28;     // larger blocks are not cached
constexpr size_t kPoolHostBlocks = 64;

struct Block {
    void* p;
    int dev;
    size_t size;
};

struct Pool {
    std::mutex mu;
    std::list<Block> idle;                            // oldest first
    std::unordered_map<void*, Block> live;
    std::unordered_map<int, size_t> idle_bytes;
    std::list<std::pair<void*, size_t>> host;
};

// never destroyed: handles may outlive static destructors, and the runtime
// frees a process's memory by itself
Pool& pool()
{
    static Pool* p = new Pool();
    return *p;
}

// Sizes in eighths of a power of two, so that graphs of about one size share
// blocks at the price of at most an eighth.  A block that is not kept has
// nothing to share and is as large as asked.
size_t size_class(size_t bytes)
{
    if (bytes > kPoolMaxBlock) return bytes;
    size_t step = 64;
    while (step * 16 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

void drop_oldest(Pool& P, int dev)
{
    for (auto it = P.idle.begin(); it != P.idle.end(); ++it)
        if (it->dev == dev) {
            (void)hipFree(it->p);
            P.idle_bytes[dev] -= it->size;
            P.idle.erase(it);
            return;
        }
}

// hipMalloc on the current device dev; if that fails, once more without the
// device's idle blocks.
hipError_t malloc_or_drop(Pool& P, int dev, void** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess && P.idle_bytes[dev] > 0) {
        (void)hipGetLastError();
        while (P.idle_bytes[dev] > 0) drop_oldest(P, dev);
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) *p = nullptr;
    return e;
}

}  // namespace

hipError_t device_malloc(void** p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    return malloc_or_drop(P, dev, p, bytes ? bytes : 1);
}

void pool_release()
{
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    for (const Block& b : P.idle) (void)hipFree(b.p);
    P.idle.clear();
    P.idle_bytes.clear();
    for (const auto& h : P.host) (void)hipHostFree(h.first);
    P.host.clear();
}

hipError_t pool_malloc(void** p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t size = size_class(bytes ? bytes : 1);
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    for (auto it = P.idle.rbegin(); it != P.idle.rend(); ++it)
        if (it->dev == dev && it->size == size) {
            *p = it->p;
            P.live[*p] = *it;
            P.idle_bytes[dev] -= size;
            P.idle.erase(std::next(it).base());
            return hipSuccess;
        }
    e = malloc_or_drop(P, dev, p, size);
    if (e != hipSuccess) return e;
    P.live[*p] = Block{*p, dev, size};
    return hipSuccess;
}

void pool_free(void* p)
{
    if (!p) return;
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    const auto it = P.live.find(p);
    if (it == P.live.end()) return;
    const Block b = it->second;
    P.live.erase(it);
    if (b.size > kPoolMaxBlock) {
        (void)hipFree(p);
        return;
    }
    P.idle.push_back(b);
    P.idle_bytes[b.dev] += b.size;
    while (P.idle_bytes[b.dev] > kPoolBytes) drop_oldest(P, b.dev);
}

hipError_t pool_host_malloc(void** p, size_t bytes)
{
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    for (auto it = P.host.begin(); it != P.host.end(); ++it)
        if (it->second == bytes) {
            *p = it->first;
            P.host.erase(it);
            return hipSuccess;
        }
    return hipHostMalloc(p, bytes, hipHostMallocDefault);
}

void pool_host_free(void* p, size_t bytes)
{
    if (!p) return;
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    if (P.host.size() >= kPoolHostBlocks) {
        (void)hipHostFree(p);
        return;
    }
    P.host.emplace_back(p, bytes);
}

}  // namespace citron
