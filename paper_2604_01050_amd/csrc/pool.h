// Device and pinned host blocks kept for reuse. A context takes about twenty
// buffers and gives them back when it is destroyed; taken from the runtime
// each time they cost 2 to 50 us per device block (freeing one also waits for
// the whole device, so that retiring a served instance stalled the others) and
// 0.05 to 0.8 ms per pinned block. Blocks given back are cached per device, up
// to POOL_DEVICE_BYTES and POOL_HOST_BYTES, the oldest returned to the runtime
// beyond that, all of a device's when one of its allocations fails, all there are
// at sbqa_release_cached. Any thread may call.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace sbqa {

constexpr size_t POOL_DEVICE_BYTES = (size_t)256 << 20;   // cached per device
constexpr size_t POOL_HOST_BYTES = (size_t)64 << 20;

struct Block {
    void *p = nullptr;
    size_t bytes = 0;   // size class, >= the size asked for
};

// A block of at least `bytes` on `device`, or of pinned coherent host memory;
// contents undefined.
hipError_t pool_get(int device, bool host, size_t bytes, Block *b);

// Gives a block back. Every use of it, on any stream, has completed.
void pool_put(int device, bool host, Block b);

// Returns every cached block, of all devices and the host's, to the runtime.
void pool_trim();

// A block for the length of a scope. The scope's end must lie behind a
// synchronisation with every use.
class PoolBlock {
  public:
    PoolBlock(int device, bool host) : device_(device), host_(host) {}
    ~PoolBlock() { pool_put(device_, host_, b_); }
    PoolBlock(const PoolBlock &) = delete;
    PoolBlock &operator=(const PoolBlock &) = delete;
    hipError_t get(size_t bytes) { return pool_get(device_, host_, bytes, &b_); }
    template <class T> T *as() const { return static_cast<T *>(b_.p); }

  private:
    int device_;
    bool host_;
    Block b_;
};

}  // namespace sbqa
