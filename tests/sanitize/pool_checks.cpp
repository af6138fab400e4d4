// Checks of the block pool (pool.h) without a GPU, its HIP calls replaced by
// ones that keep count: sizes, the bounds of what is kept, the device of a block,
// memory given back when an allocation fails, several threads. Prints
// "pool checks passed".
#include "../../paper_2604_01050_amd/csrc/pool.h"

#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

namespace {

struct Raw {
    int device;
    size_t bytes;
    bool host;
};
std::mutex mu;
std::map<void *, Raw> live;
std::map<int, size_t> held;   // bytes per device
size_t held_host = 0, capacity = (size_t)1 << 60;
thread_local int current = 0;

#define CHECK(cond)                                                                     \
    do {                                                                                \
        if (!(cond)) {                                                                  \
            std::printf("CHECK failed, line %d: %s\n", __LINE__, #cond);                \
            std::exit(1);                                                               \
        }                                                                               \
    } while (0)

}  // namespace

hipError_t hipMalloc(void **p, size_t bytes) {
    std::lock_guard<std::mutex> lk(mu);
    if (held[current] + bytes > capacity) return hipErrorOutOfMemory;
    *p = std::malloc(1);   // (an address of its own)
    live[*p] = Raw{current, bytes, false};
    held[current] += bytes;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
    std::lock_guard<std::mutex> lk(mu);
    *p = std::malloc(1);
    live[*p] = Raw{-1, bytes, true};
    held_host += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> lk(mu);
    CHECK(live.count(p) && !live[p].host);
    held[live[p].device] -= live[p].bytes;
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::lock_guard<std::mutex> lk(mu);
    CHECK(live.count(p) && live[p].host);
    held_host -= live[p].bytes;
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int *device) { return *device = current, hipSuccess; }
hipError_t hipSetDevice(int device) { return current = device, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }

using namespace sbqa;

static void check_sizes() {
    for (size_t bytes = 1; bytes < ((size_t)40 << 30); bytes += bytes / 7 + 1) {
        Block b;
        CHECK(pool_get(0, false, bytes, &b) == hipSuccess && b.bytes >= bytes && live[b.p].bytes == b.bytes);
        CHECK(b.bytes - bytes <= std::max<size_t>((size_t)64 << 10, bytes / 16));
        if (bytes > POOL_DEVICE_BYTES / 2) CHECK(b.bytes - bytes < (size_t)64 << 10);   // not kept: not rounded up
        pool_put(0, false, b);
        CHECK(held[0] <= POOL_DEVICE_BYTES);
        if (bytes > POOL_DEVICE_BYTES / 2) CHECK(!live.count(b.p));
    }
}

// Blocks lie on the device that was asked for, whichever the thread has current,
// which stays as it was.
static void check_devices() {
    for (int device = 0; device < 3; ++device)
        for (int cur = 0; cur < 3; ++cur) {
            current = cur;
            Block b[3];
            for (Block &x : b) CHECK(pool_get(device, false, 70000, &x) == hipSuccess && live[x.p].device == device);
            CHECK(current == cur);
            for (const Block &x : b) pool_put(device, false, x);
        }
    current = 0;
}

// An allocation that fails takes what is cached on its device and tries again.
static void check_full_device() {
    pool_trim();
    std::vector<Block> bs(40);
    for (Block &b : bs) CHECK(pool_get(1, false, (size_t)4 << 20, &b) == hipSuccess);
    for (const Block &b : bs) pool_put(1, false, b);
    CHECK(held[1] == (size_t)160 << 20);
    capacity = (size_t)200 << 20;
    Block big;
    CHECK(pool_get(1, false, (size_t)190 << 20, &big) == hipSuccess && held[1] == (size_t)190 << 20);
    Block more;
    CHECK(pool_get(1, false, (size_t)20 << 20, &more) == hipErrorOutOfMemory && !more.p);
    capacity = (size_t)1 << 60;
    pool_put(1, false, big);
}

// What is cached is bounded, of the host's blocks too, and goes back when asked.
static void check_bounds() {
    for (bool host : {false, true}) {
        std::vector<Block> bs(600);
        for (Block &b : bs) CHECK(pool_get(0, host, (size_t)1 << 20, &b) == hipSuccess);
        for (const Block &b : bs) pool_put(0, host, b);
        CHECK((host ? held_host : held[0]) <= (host ? POOL_HOST_BYTES : POOL_DEVICE_BYTES));
    }
    CHECK(held[0] && held_host);
    pool_trim();
    CHECK(!held[0] && !held[1] && !held[2] && !held_host && live.empty());
}

// A block is with one holder at a time, whatever the threads do.
static void check_threads() {
    std::vector<std::thread> ts;
    for (int t = 0; t < 4; ++t)
        ts.emplace_back([t] {
            std::mt19937 g(t);
            std::vector<std::pair<Block, bool>> mine;
            for (int n = 0; n < 3000; ++n) {
                const bool host = g() % 4 == 0;
                if (g() % 2 || mine.empty()) {
                    Block b;
                    CHECK(pool_get(0, host, (size_t)1 << (10 + g() % 12), &b) == hipSuccess);
                    *static_cast<char *>(b.p) = (char)t;   // (a race here is a block with two holders)
                    mine.push_back({b, host});
                } else {
                    const size_t k = g() % mine.size();
                    CHECK(*static_cast<char *>(mine[k].first.p) == (char)t);
                    pool_put(0, mine[k].second, mine[k].first);
                    mine.erase(mine.begin() + (long)k);
                }
                if (n % 700 == 0) pool_trim();
            }
            for (auto &m : mine) pool_put(0, m.second, m.first);
        });
    for (std::thread &t : ts) t.join();
    pool_trim();
    CHECK(live.empty());
}

int main() {
    check_sizes();
    check_devices();
    check_full_device();
    check_bounds();
    check_threads();
    std::printf("pool checks passed\n");
    return 0;
}
