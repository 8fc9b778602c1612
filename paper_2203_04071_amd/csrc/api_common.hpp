// Shared by the translation units of the C ABI: error reporting, device allocations, the table handle.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/adapt_mi355.h"
#include "byte_form.hpp"
#include "elementwise.hpp"
#include "scratch.hpp"

namespace adapt_api {

extern thread_local char g_err[512];        // defined in api_core.hip

inline int fail(int code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr)                                                                                  \
    do {                                                                                               \
        hipError_t e_ = (expr);                                                                        \
        if (e_ != hipSuccess)                                                                          \
            return fail(e_ == hipErrorOutOfMemory ? ADAPT_ERR_OUT_OF_MEMORY : ADAPT_ERR_HIP, "%s: %s", \
                        #expr, hipGetErrorString(e_));                                                 \
    } while (0)

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline unsigned ew_grid(size_t work_items) {
    size_t g = (work_items + adapt::EW_THREADS - 1) / adapt::EW_THREADS;
    if (g < 1) g = 1;
    if (g > 256 * 16) g = 256 * 16;   // grid-stride loops: 16 blocks per compute unit is plenty
    return (unsigned)g;
}

// workgroups of the kernels that end in atomics (absmax_kernel, histogram_abs_kernel): at most RED_BLOCKS, at least 4 elements a thread
inline unsigned red_grid(size_t n) {
    const size_t g = (n + adapt::RED_THREADS * 4 - 1) / (adapt::RED_THREADS * 4);
    return (unsigned)(g < 1 ? 1 : (g > adapt::RED_BLOCKS ? adapt::RED_BLOCKS : g));
}

// Scratch memory of one call: the partial sums of a product whose inner dimension is split, and the activation copy.  Plain
// entry points take it from the stream-ordered allocator and give it back in stream order; a packed-weights handle keeps one
// grow-only buffer, so that its calls allocate nothing once they have run at their largest size (they can then be
// recorded into a HIP graph).  How much partial sums need depends on the plan and does not grow with the size, so that part of
// the buffer is reserved for every product of up to part_rows rows.
struct Workspace {
    void *mem = nullptr;        // partial sums, the copy behind them (one allocation: a handle's first call waits for it)
    size_t part_bytes = 0, copy_bytes = 0;
    long long part_rows = 0;
    void *copy() const { return mem ? static_cast<char *>(mem) + part_bytes : nullptr; }
    bool holds(size_t copy, long long rows, size_t part = 0) const { return mem && copy_bytes >= copy && part_rows >= rows && part_bytes >= part; }
};

// copy_bytes at *copy and part_bytes at *part for a product of `rows` rows; reserve(): the bytes of partial sums that products of up to
// `rows` rows need.  Given back by ws_put(*copy).
template <typename Reserve>
inline int ws_get(Workspace *cache, size_t copy_bytes, size_t part_bytes, long long rows, Reserve &&reserve, hipStream_t s, void **copy, int32_t **part) {
    if (!cache) {
        HIP_TRY(dbg_malloc_async(copy, copy_bytes + part_bytes, s));
        *part = part_bytes ? reinterpret_cast<int32_t *>(static_cast<char *>(*copy) + copy_bytes) : nullptr;
        return ADAPT_OK;
    }
    if (!cache->holds(copy_bytes, rows, part_bytes)) {
        Workspace w = *cache;
        if (rows > w.part_rows || part_bytes > w.part_bytes) {      // (what the call itself needs in any case)
            size_t bytes = reserve();
            bytes = ((part_bytes > bytes ? part_bytes : bytes) + 255) / 256 * 256;
            w.part_bytes = bytes > w.part_bytes ? bytes : w.part_bytes;
            w.part_rows = rows > w.part_rows ? rows : w.part_rows;
        }
        w.copy_bytes = copy_bytes > w.copy_bytes ? copy_bytes : w.copy_bytes;
        if (!w.mem || w.part_bytes > cache->part_bytes || w.copy_bytes > cache->copy_bytes) {
            if (w.mem) HIP_TRY(hipFree(w.mem));     // waits for the device: no earlier call still uses it
            *cache = Workspace{};
            w.mem = nullptr;
            HIP_TRY(dbg_malloc(&w.mem, w.part_bytes + w.copy_bytes));
        }
        *cache = w;
    }
    *copy = cache->copy();
    *part = part_bytes ? static_cast<int32_t *>(cache->mem) : nullptr;
    return ADAPT_OK;
}

inline int ws_put(Workspace *cache, void *p, hipStream_t s, int rc) {
    if (cache || !p) return rc;
    hipError_t fe = hipFreeAsync(p, s);
    if (rc == ADAPT_OK && fe != hipSuccess) rc = fail(ADAPT_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(fe));
    return rc;
}

// compute units of the current device (asked once per device; 256 when there is no device to ask)
inline int device_cus() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int cu = cached[dev].load(std::memory_order_relaxed);
    if (cu > 0) return cu;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0) return 256;
    cached[dev].store(cu, std::memory_order_relaxed);
    return cu;
}

inline adapt::FastDiv fast_div(uint32_t d) {
    int l = 0;
    while ((1ull << l) < d) ++l;
    adapt::FastDiv f;
    f.k = 31 + l;
    f.M = (uint32_t)((1ull << f.k) / d + 1);
    f.d = d;
    return f;
}

}  // namespace adapt_api

struct adapt_lut {
    int bits;
    int storage;            // 0: one signed 16-bit image; 1: low (unsigned) + high (signed) images
    int32_t min_entry, max_entry;
    int device;
    int rs;                 // entries per image row = 2^b + 2
    int img_bytes;          // per image, multiple of 16
    uint16_t *img_dev[2];   // [0] = only / low half, [1] = high half
    uint16_t *lut16_dev[2]; // same halves, plain [a & mask][w & mask] order (source of the derived line tables)
    adapt_api::ByteForm byte;   // for the byte kernel, if the table has such a form:
    uint16_t *img8_dev;         // its error bytes [w + H][a + H], in the allocation of lut16_dev[0], else nullptr
};
