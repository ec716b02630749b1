// Device and pinned memory of calls that bring none.
//
// The device's default memory pool gives every block back to the driver when
// the stream is next waited for, so each call paid for mapping and unmapping
// it: 70-420 us per call for 40 MB to 1 GB in a process with little memory,
// several milliseconds in one holding tens of GB.  Blocks up to POOL_BLOCK_MAX
// come from a pool of the library's own (one per device, created at first use)
// that keeps at most POOL_KEEP_BYTES of freed memory and gives the rest back;
// 35 us per call whatever the size.  Larger blocks, and allocations inside a
// stream capture (which become graph nodes), use the default pool.  The runtime
// orders reuse between streams and threads.  Before an allocation of the
// library fails, the pool's idle memory is given back and it is tried again;
// lz_release_memory() gives it back to other allocators of the process.
#include <chrono>
#include <cstring>
#include <mutex>
#include <thread>

#include "../../include/lanczos_topk.h"
#include "lz_internal.h"

namespace lz {
namespace {

constexpr size_t POOL_KEEP_BYTES = (size_t)2 << 30;
constexpr size_t POOL_BLOCK_MAX = (size_t)1 << 30;
constexpr int POOL_MAX_DEVICES = 64;

std::mutex pool_mu;
hipMemPool_t pools[POOL_MAX_DEVICES] = {};
bool tried[POOL_MAX_DEVICES] = {};

// The device a stream belongs to, -1 if it cannot be told.  The default streams
// are the current device's (hipGetStreamDeviceId takes no such handle but null:
// it follows the others).
int stream_device(hipStream_t s) {
    if (s != nullptr && s != hipStreamLegacy && s != hipStreamPerThread) return hipGetStreamDeviceId(s);
    int dev = -1;
    return hipGetDevice(&dev) == hipSuccess ? dev : -1;
}

// Pool of a device; null if it has none.
hipMemPool_t workspace_pool(int dev) {
    if (dev < 0 || dev >= POOL_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lk(pool_mu);
    if (!tried[dev]) {
        tried[dev] = true;
        hipMemPoolProps props;
        std::memset(&props, 0, sizeof(props));
        props.allocType = hipMemAllocationTypePinned;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        hipMemPool_t pool = nullptr;
        uint64_t keep = POOL_KEEP_BYTES;
        if (hipMemPoolCreate(&pool, &props) != hipSuccess) {
            (void)hipGetLastError();
        } else if (hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipMemPoolDestroy(pool);
        } else {
            pools[dev] = pool;
        }
    }
    return pools[dev];
}

// Gives the idle memory of a pool back to the driver; false if it had none.
bool trim(hipMemPool_t pool) {
    uint64_t before = 0, after = 0;
    if (hipMemPoolGetAttribute(pool, hipMemPoolAttrReservedMemCurrent, &before) == hipSuccess &&
        hipMemPoolTrimTo(pool, 0) == hipSuccess &&
        hipMemPoolGetAttribute(pool, hipMemPoolAttrReservedMemCurrent, &after) == hipSuccess)
        return after < before;
    (void)hipGetLastError();
    return false;
}

// Runs alloc again after a failure, first giving the idle memory of the
// device's pool back.  The runtime drops its last references to a block on a
// thread of its own: the driver had it 0.6 ms after the trim, so the
// allocation is tried for 20 times that.
template <class Alloc> hipError_t retry(int dev, Alloc&& alloc) {
    bool freed = false;
    if (dev >= 0 && dev < POOL_MAX_DEVICES) {
        std::lock_guard<std::mutex> lk(pool_mu);
        freed = pools[dev] && trim(pools[dev]);
    }
    hipError_t e = alloc();
    for (int i = 0; freed && e != hipSuccess && i < 12; ++i) {
        (void)hipGetLastError();
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
        e = alloc();
    }
    return e;
}

// Pinned state buffers not in use, linked through their first word.
std::mutex host_mu;
void* host_free = nullptr;

}  // namespace

State* HostState::get() {
    if (st_) return st_;
    {
        std::lock_guard<std::mutex> lk(host_mu);
        if (host_free) {
            st_ = (State*)host_free;
            host_free = *(void**)st_;
        }
    }
    if (!st_ && hipHostMalloc((void**)&st_, sizeof(State), hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        st_ = nullptr;
    }
    return st_;
}

HostState::~HostState() {
    if (!st_) return;
    std::lock_guard<std::mutex> lk(host_mu);
    *(void**)st_ = host_free;
    host_free = st_;
}

// An allocation that failed for good: reported by its status alone, not by the
// next launch's error check too.
static hipError_t settle(hipError_t e) {
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

// Stream-ordered allocation on s; freed with hipFreeAsync.
hipError_t workspace_alloc(void** p, size_t bytes, hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)
        return settle(hipMallocAsync(p, bytes, s));
    const int dev = stream_device(s);
    const hipMemPool_t pool = bytes <= POOL_BLOCK_MAX ? workspace_pool(dev) : nullptr;
    if ((pool ? hipMallocFromPoolAsync(p, bytes, pool, s) : hipMallocAsync(p, bytes, s)) == hipSuccess)
        return hipSuccess;
    (void)hipGetLastError();
    // Blocks that the stream has yet to free are idle once it has been waited for.
    (void)hipStreamSynchronize(s);
    return settle(retry(dev, [&] { return hipMallocAsync(p, bytes, s); }));
}

// hipMalloc on the current device.
hipError_t device_alloc(void** p, size_t bytes) {
    const hipError_t e = settle(hipMalloc(p, bytes));
    int dev = -1;
    if (e == hipSuccess || hipGetDevice(&dev) != hipSuccess) return e;
    return settle(retry(dev, [&] { return hipMalloc(p, bytes); }));
}

}  // namespace lz

extern "C" int lz_release_memory(void) {
    int rc = LZ_OK;
    std::lock_guard<std::mutex> lk(lz::pool_mu);
    for (hipMemPool_t pool : lz::pools)
        if (pool && hipMemPoolTrimTo(pool, 0) != hipSuccess) {
            (void)hipGetLastError();
            rc = LZ_ERR_HIP;
        }
    return rc;
}
