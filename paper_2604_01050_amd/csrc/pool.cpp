// Cached device and pinned host blocks (pool.h).
#include "pool.h"

#include <list>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

namespace sbqa {
namespace {

struct Cache {
    std::list<Block> blocks;   // oldest first
    size_t bytes = 0;
};

std::mutex g_pool_mu;
// never destroyed: the HIP runtime may be gone when static objects are
std::map<std::pair<int, bool>, Cache> &caches() {
    static auto *m = new std::map<std::pair<int, bool>, Cache>();
    return *m;
}

// Size classes: 64 KiB steps up to 2 MiB, then 32nds of a power of two (6% more at
// most); blocks that are not cached anyway (pool_put) to 64 KiB.
size_t size_class(size_t bytes, size_t limit) {
    size_t step = (size_t)64 << 10;
    if (bytes <= limit / 2)
        while (bytes > 32 * step) step *= 2;
    return bytes == 0 ? step : (bytes + step - 1) / step * step;
}

constexpr size_t limit_of(bool host) { return host ? POOL_HOST_BYTES : POOL_DEVICE_BYTES; }

// (a device block on its own device, whichever the calling thread has current)
hipError_t raw_get(int device, bool host, size_t bytes, void **p) {
    if (host) return hipHostMalloc(p, bytes, hipHostMallocCoherent);
    int cur = device;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != device) e = hipSetDevice(device);
    if (e == hipSuccess) e = hipMalloc(p, bytes);
    if (cur != device) (void)hipSetDevice(cur);
    return e;
}

void raw_free(bool host, const std::vector<Block> &bs) {
    for (const Block &b : bs) {
        if (host) (void)hipHostFree(b.p);
        else (void)hipFree(b.p);
    }
}

}  // namespace

hipError_t pool_get(int device, bool host, size_t bytes, Block *b) {
    const size_t want = size_class(bytes, limit_of(host));
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        Cache &c = caches()[{device, host}];
        for (auto it = c.blocks.begin(); it != c.blocks.end(); ++it)
            if (it->bytes == want) {
                *b = *it;
                c.bytes -= want;
                c.blocks.erase(it);
                return hipSuccess;
            }
    }
    void *p = nullptr;
    hipError_t e = raw_get(device, host, want, &p);
    if (e != hipSuccess) {
        // out of memory: give everything cached back and try once more
        std::vector<Block> all;
        {
            std::lock_guard<std::mutex> lk(g_pool_mu);
            Cache &c = caches()[{device, host}];
            all.assign(c.blocks.begin(), c.blocks.end());
            c.blocks.clear();
            c.bytes = 0;
        }
        if (all.empty()) return e;
        (void)hipGetLastError();
        raw_free(host, all);
        e = raw_get(device, host, want, &p);
        if (e != hipSuccess) return e;
    }
    b->p = p;
    b->bytes = want;
    return hipSuccess;
}

void pool_put(int device, bool host, Block b) {
    if (!b.p) return;
    const size_t limit = limit_of(host);
    std::vector<Block> out;
    if (b.bytes > limit / 2) {
        out.push_back(b);
    } else {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        Cache &c = caches()[{device, host}];
        c.blocks.push_back(b);
        c.bytes += b.bytes;
        while (c.bytes > limit) {
            out.push_back(c.blocks.front());
            c.bytes -= c.blocks.front().bytes;
            c.blocks.pop_front();
        }
    }
    raw_free(host, out);
}

void pool_trim() {
    std::vector<Block> dev, host;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        for (auto &kv : caches()) {
            std::vector<Block> &to = kv.first.second ? host : dev;
            to.insert(to.end(), kv.second.blocks.begin(), kv.second.blocks.end());
            kv.second = Cache();
        }
    }
    raw_free(false, dev);
    raw_free(true, host);
}

}  // namespace sbqa
