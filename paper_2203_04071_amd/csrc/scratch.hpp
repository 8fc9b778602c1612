// Device memory of the library: the allocations of handles, and the pool that scratch memory of calls comes from.  Host code only.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

namespace adapt_api {

// Debugging aid: with ADAPT_POISON_ALLOC set in the environment every device allocation of the library is filled with
// 0xA5 bytes before use, so that code which relies on fresh memory being zero shows up in the tests.
bool poison_on();
hipError_t dbg_poison(void *p, size_t bytes, hipStream_t s);

// Scratch memory of calls comes from a pool of the library's own, one per device, that keeps up to SCRATCH_KEEP bytes between
// calls: the device's default pool gives everything back at every synchronisation, and a program that waits for each result
// then pays for mapping the memory again (waiting after every call: 12-bit 3 x 3 layer 291 -> 218 us, retraining step 299 -> 250 us;
// with tables of 268 MB made for the call, 2000 rows 1024 -> 1024, 8 bits: 588 -> 202 us, 412 us by the whole-table kernel).
// What no call uses is given back when the last multiplier table on the device is destroyed, and when an allocation of the
// library finds no memory (and by the runtime at every hipFree of the process: the next call maps its scratch anew, 199 MB in 130 us).  A call that is being recorded allocates through the default pool, as a node of the graph.
constexpr uint64_t SCRATCH_KEEP = 1ull << 30;
constexpr int SCRATCH_DEVICES = 64;
struct ScratchPool {
    std::atomic<hipMemPool_t> pool{nullptr};
    std::atomic<int> tables{0};     // multiplier tables on this device
};
inline ScratchPool g_scratch[SCRATCH_DEVICES];
inline std::mutex g_scratch_lock;

inline ScratchPool *scratch_of(int dev) { return dev >= 0 && dev < SCRATCH_DEVICES ? &g_scratch[dev] : nullptr; }
inline ScratchPool *scratch_here() {
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess) return scratch_of(dev);
    (void)hipGetLastError();
    return nullptr;
}

// the current device's pool; nullptr where it cannot be made (the next call tries again)
inline hipMemPool_t scratch_pool(ScratchPool *sp) {
    if (!sp) return nullptr;
    hipMemPool_t pool = sp->pool.load(std::memory_order_acquire);
    if (pool) return pool;
    std::lock_guard<std::mutex> lock(g_scratch_lock);
    if ((pool = sp->pool.load(std::memory_order_relaxed))) return pool;
    hipMemPoolProps props{};
    props.allocType = hipMemAllocationTypePinned;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = (int)(sp - g_scratch);
    uint64_t keep = SCRATCH_KEEP;
    bool ok = hipMemPoolCreate(&pool, &props) == hipSuccess;
    if (ok && hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) {
        (void)hipMemPoolDestroy(pool);
        ok = false;
    }
    if (!ok) {
        (void)hipGetLastError();
        return nullptr;
    }
    sp->pool.store(pool, std::memory_order_release);
    return pool;
}

inline void trim_scratch(ScratchPool *sp) {
    const hipMemPool_t pool = sp ? sp->pool.load(std::memory_order_acquire) : nullptr;
    if (pool && hipMemPoolTrimTo(pool, 0) != hipSuccess) (void)hipGetLastError();
}

// a multiplier table (of either kind) was made on a device, is gone
inline void scratch_table_made(int dev) {
    if (ScratchPool *sp = scratch_of(dev)) sp->tables.fetch_add(1, std::memory_order_relaxed);
}
inline void scratch_table_gone(int dev) {
    ScratchPool *sp = scratch_of(dev);
    if (sp && sp->tables.fetch_sub(1, std::memory_order_acq_rel) == 1) trim_scratch(sp);
}

// whether calls on this stream are being recorded, or may be (the question has no answer)
inline bool is_capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

inline hipError_t dbg_malloc_async(void **p, size_t bytes, hipStream_t s) {
    ScratchPool *const sp = is_capturing(s) ? nullptr : scratch_here();
    const hipMemPool_t pool = scratch_pool(sp);
    hipError_t e = pool ? hipMallocFromPoolAsync(p, bytes, pool, s) : hipMallocAsync(p, bytes, s);
    if (e != hipSuccess && pool) {      // (what the pool keeps may be what is missing, and the default pool may hold memory too)
        (void)hipGetLastError();
        trim_scratch(sp);
        e = hipMallocAsync(p, bytes, s);
    }
    if (e == hipSuccess && poison_on()) e = dbg_poison(*p, bytes, s);
    return e;
}
inline hipError_t dbg_malloc(void **p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        trim_scratch(scratch_here());
        e = hipMalloc(p, bytes);
    }
    if (e == hipSuccess && poison_on()) {
        e = dbg_poison(*p, bytes, nullptr);
        if (e == hipSuccess) e = hipDeviceSynchronize();
    }
    return e;
}

}  // namespace adapt_api
