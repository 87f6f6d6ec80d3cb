// Reuse of device and pinned host blocks between graph handles.
//
// A graph that comes in, is counted and goes makes and drops about thirty
// device blocks and a pinned one; hipMalloc, hipFree (which waits for the
// device) and hipHostMalloc were 5.5 of the 18.2 ms of load + order + counts
// of a 2^20-vertex graph and more than half of the 0.44 ms of a 2^8-vertex
// one.  Freed blocks are kept, at most kPoolBytes per device and
// kPoolHostBlocks pinned ones, the oldest given back first, all of them when
// an allocation fails, here or through device_malloc, which the library's
// other device memory comes from, or when the program asks (pool_release).
// A block is only handed to pool_free once the work that
// used it has completed, so its next owner may use it on any stream.
#include "api_internal.h"

#include <deque>
#include <list>
#include <map>
#include <new>
#include <unordered_map>

namespace citron {

namespace {

constexpr size_t kPoolBytes = (size_t)1 << 30;        // cached per device
constexpr size_t kPoolMaxBlock = (size_t)1 << 28;     // larger blocks are not cached
constexpr size_t kPoolHostBlocks = 64;
constexpr size_t kPage = 4096;                        // what a block takes at least

struct Block {
    void* p;
    int dev;
    size_t size;
};
typedef std::list<Block> Blocks;

// Idle blocks of one device: by age, and of each size by age again, so that
// neither a search nor giving the oldest back looks at the others.
struct Idle {
    Blocks all;                                       // oldest first
    std::map<size_t, std::deque<Blocks::iterator>> by_size;
    size_t bytes = 0;
};

struct Pool {
    std::mutex mu;
    std::unordered_map<void*, Block> live;
    std::unordered_map<int, Idle> idle;
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
// blocks at the price of at most an eighth; a page at least, which the device
// gives a smaller block too.  A block that is not kept has nothing to share
// and is as large as asked.
size_t size_class(size_t bytes)
{
    if (bytes > kPoolMaxBlock) return bytes;
    if (bytes <= kPage) return kPage;
    size_t step = kPage / 16;
    while (step * 16 < bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

void drop_oldest(Idle& I)
{
    const Block b = I.all.front();
    const auto it = I.by_size.find(b.size);           // its oldest is the oldest of all
    it->second.pop_front();
    if (it->second.empty()) I.by_size.erase(it);
    I.all.pop_front();
    I.bytes -= b.size;
    (void)hipFree(b.p);
}

// hipMalloc on the current device dev; if that fails, once more without the
// device's idle blocks.
hipError_t malloc_or_drop(Pool& P, int dev, void** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    const auto it = P.idle.find(dev);
    if (e != hipSuccess && it != P.idle.end() && !it->second.all.empty()) {
        (void)hipGetLastError();
        while (!it->second.all.empty()) drop_oldest(it->second);
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
    for (auto& dev : P.idle)
        while (!dev.second.all.empty()) drop_oldest(dev.second);
    for (const auto& h : P.host) (void)hipHostFree(h.first);
    P.host.clear();
}

// (no exception leaves these functions: without host memory for the books, a
// block is not handed out, or not kept)
hipError_t pool_malloc(void** p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t size = size_class(bytes);
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    try {
        Idle& I = P.idle[dev];
        const auto it = I.by_size.find(size);
        if (it != I.by_size.end()) {
            const Blocks::iterator newest = it->second.back();
            P.live[newest->p] = *newest;
            *p = newest->p;
            it->second.pop_back();
            if (it->second.empty()) I.by_size.erase(it);
            I.all.erase(newest);
            I.bytes -= size;
            return hipSuccess;
        }
        e = malloc_or_drop(P, dev, p, size);
        if (e == hipSuccess) P.live[*p] = Block{*p, dev, size};
        return e;
    } catch (const std::bad_alloc&) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
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
    bool listed = false;
    try {
        Idle& I = P.idle[b.dev];
        I.all.push_back(b);
        listed = true;
        I.by_size[b.size].push_back(std::prev(I.all.end()));
        I.bytes += b.size;
        while (I.bytes > kPoolBytes) drop_oldest(I);
    } catch (const std::bad_alloc&) {
        if (listed) {
            Idle& I = P.idle[b.dev];
            I.all.pop_back();
            const auto c = I.by_size.find(b.size);
            if (c != I.by_size.end() && c->second.empty()) I.by_size.erase(c);
        }
        (void)hipFree(p);
    }
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
    try {
        if (P.host.size() < kPoolHostBlocks) {
            P.host.emplace_back(p, bytes);
            return;
        }
    } catch (const std::bad_alloc&) {
    }
    (void)hipHostFree(p);
}

}  // namespace citron
