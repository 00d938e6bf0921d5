#include "pcsr_pool.h"

#include <algorithm>
#include <map>
#include <mutex>
#include <unordered_map>

namespace pcsr {
namespace {

struct Block {
    size_t bytes;
    int device;
};
struct Idle {
    void *p;
    uint64_t since; // allocation count when it was freed
};
struct Cache {
    std::multimap<size_t, Idle> idle; // by size
    size_t bytes = 0;
};

struct Pool {
    std::mutex mu;
    std::unordered_map<void *, Block> live;
    std::map<int, Cache> caches;
    uint64_t clock = 0;
};

Pool &pool()
{
    static Pool *p = new Pool; // never destroyed: handles may outlive static destruction
    return *p;
}

size_t rounded(size_t bytes)
{
    const size_t unit = bytes >= (size_t(1) << 20) ? size_t(1) << 20 : 4096;
    return (std::max<size_t>(bytes, 1) + unit - 1) / unit * unit;
}

void drop(Cache &c, std::multimap<size_t, Idle>::iterator it)
{
    (void)hipFree(it->second.p);
    c.bytes -= it->first;
    c.idle.erase(it);
}

} // namespace

hipError_t pool_alloc(void **out, size_t bytes)
{
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const size_t need = rounded(bytes);
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    ++P.clock;
    Cache &c = P.caches[dev];
    // a block up to a quarter (or 1 MB) larger than asked for
    auto it = c.idle.lower_bound(need);
    if (it != c.idle.end() && it->first <= need + std::max(need / 4, size_t(1) << 20)) {
        *out = it->second.p;
        P.live[*out] = {it->first, dev};
        c.bytes -= it->first;
        c.idle.erase(it);
        return hipSuccess;
    }
    e = hipMalloc(out, need);
    if (e == hipErrorOutOfMemory && !c.idle.empty()) {
        (void)hipGetLastError();
        while (!c.idle.empty()) drop(c, c.idle.begin());
        e = hipMalloc(out, need);
    }
    if (e != hipSuccess) {
        *out = nullptr;
        return e;
    }
    P.live[*out] = {need, dev};
    return hipSuccess;
}

void pool_free(void *p)
{
    if (!p) return;
    Pool &P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) {
        (void)hipFree(p);
        return;
    }
    Cache &c = P.caches[it->second.device];
    const size_t bytes = it->second.bytes;
    P.live.erase(it);
    if (bytes > kPoolBytes) {
        (void)hipFree(p);
        return;
    }
    c.idle.insert({bytes, {p, P.clock}});
    c.bytes += bytes;
    for (auto i = c.idle.begin(); i != c.idle.end();) {
        auto at = i++;
        if (P.clock - at->second.since > kPoolIdleAllocs) drop(c, at);
    }
    while (c.bytes > kPoolBytes) {
        auto oldest = c.idle.begin();
        for (auto i = c.idle.begin(); i != c.idle.end(); ++i)
            if (i->second.since < oldest->second.since) oldest = i;
        drop(c, oldest);
    }
}

bool pool_quiesce(int device)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (dev != device && hipSetDevice(device) != hipSuccess) return false;
    const hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) (void)hipGetLastError();
    if (dev != device) (void)hipSetDevice(dev);
    return e == hipSuccess;
}

void pool_release(void *p)
{
    if (!p) return;
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> lock(P.mu);
        P.live.erase(p);
    }
    (void)hipFree(p);
}

} // namespace pcsr
