// "Columns" kernel: products on operands of 9 to 12 bits whose table is an exact product plus an error of 16 bits.
//
// Such a table, T[a][w] = a w + c + e[a][w] with e an int16 (adapt_lut16_create looks for the form), does not fit LDS (b = 12:
// 32 MB), but what ONE inner index needs of it does: the columns e[.][w_kn] of its weights, 8 KB each at 12 bits.  A workgroup
// therefore owns 4 output channels and 4096 NR output pixels, and walks the inner dimension in stages of 2^(13 - b) indices:
// it copies the columns of a stage into LDS, the four channels of an entry side by side (8 bytes), and every lookup of a
// pixel is then one 8-byte LDS read for four channels.  Every column is read from memory once per row tile, whole and
// coalesced, where lut_big.hpp gathers single entries from memory.
//     acc[m][n] = sum_k e[a_mk][w_nk]  +  sum_k a_mk w_nk  +  K c
// : the exact products of two consecutive inner indices are one v_dot2_i32_i16 per output, and so is every addition of a
// looked-up entry (with 1 on the half that counts).  Sums wrap in 32 bits, so the split is exact.
//
// Activation copy: words of two consecutive channels of a tap (signed codes), [image][row][channel pair][residue of the column
// modulo the horizontal stride][column / stride], as in lut_byte.hpp: a run of four output pixels of a row is four consecutive
// words for every stride.  Rows are virtual (an image row counts as Wo rounded up to runs of four).
//
// What bounds it (one MI355X; 3 x 3, 64 -> 64 channels, 32 images of 32 x 32, whole layer 196 us at 12 bits and 121 us at 9, against
// 1700 and 1160 us of the gathering kernel): no unit by itself.  LDS is busy for 39 % of the time (7 clocks a read of 64 lanes,
// half of them bank conflicts: 64 random entries), the vector ALU for 48 %.  Timed when the layer took 207 us (it mapped its scratch
// memory anew): taking the columns' loads and stores out saved 70 us at 12 bits, the exact product or the additions 12 us
// each.  8192 pixels per workgroup, because a column is loaded and stored once per row tile (4096: 290 us at 12 bits) and larger
// ones would need more slices, whose sums cost as much (8 slices instead of 4: 254 us).
//
// Split inner dimension: ksplit workgroups share a tile; all but the last to arrive leave their sums in memory, the last one
// adds them to its own and finishes (the scheme of lut_byte.hpp).
#pragma once
#include "lut_big.hpp"

namespace adapt {

constexpr int COLS_THREADS = 1024;
constexpr int COLS_NT = 4;                  // channels of a tile
constexpr int COLS_BUF = 65536;             // LDS of a stage: 2^(13 - b) tables of 2^b entries of 8 bytes
constexpr int COLS_MIN_BITS = 9, COLS_MAX_BITS = 12;

typedef short s16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

struct ColsParams {
    const uint32_t *xt;         // activation copy
    const int16_t *e;           // columns [w & mask] of the error, one more of zeros; order inside a column: cols_order()
    const uint4 *words;         // [n_tile][pair][2]: weight pairs of the four channels, column numbers of the four channels
    int32_t *out;
    int32_t *partial;           // ksplit > 1: [tile][slice][pixel of a thread][1024] x 16 B
    uint32_t *arrived;          // ksplit > 1: one counter per tile, zero before the launch
    int Mv, N, n_tiles, m_tiles, ksplit;
    int pairs, cp, kw, stages;  // channel pairs of all taps, of one tap; filter width; stages (pairs rounded up)
    int Wo, Wv;
    int img_stride, oy_stride, ch_stride, ky_stride;    // words of xt
    int dw, sw, wsub;
    int corr;                   // K c
    int linear, out_plane;      // output [M][N] instead of NCHW
    FastDiv d_HoWv, d_Wv, d_cp, d_kw, d_sw;
    int deq, act;
    float scale;
    const float *scales, *bias;
};

// entry at position i of a stored column: groups of four are entries 2 u, 2 u + 1 and the same in the upper half, so that
// the 8 bytes a lane loads become two 16-byte LDS stores at consecutive addresses of consecutive lanes
__host__ __device__ __forceinline__ int cols_order(int i, int bits) { return ((i >> 2) << 1) + (i & 1) + (((i >> 1) & 1) << (bits - 1)); }

// smallest and largest T[a][w] - a w of a table in the order of lut_big.hpp; range[0] = min, range[1] = max (few workgroups:
// each ends in two atomics on the same words)
static __global__ __launch_bounds__(256) void cols_range_kernel(const int32_t *__restrict__ t, int bits, int32_t *range) {
    const size_t n = (size_t)1 << bits, total = n * n, stride = (size_t)gridDim.x * 256;
    const int h = 1 << (bits - 1);
    int lo = 0x7fffffff, hi = -0x7fffffff - 1;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
        const int w = (int)(i >> bits) - h, a = (int)(i & (n - 1)) - h;
        const int e = (int)((uint32_t)t[i] - (uint32_t)(a * w));
        lo = min(lo, e);
        hi = max(hi, e);
    }
    for (int d = 32; d > 0; d >>= 1) {
        lo = min(lo, __shfl_xor(lo, d));
        hi = max(hi, __shfl_xor(hi, d));
    }
    __shared__ int part[2][4];
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = lo;
        part[1][threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicMin(range, min(min(part[0][0], part[0][1]), min(part[0][2], part[0][3])));
        atomicMax(range + 1, max(max(part[1][0], part[1][1]), max(part[1][2], part[1][3])));
    }
}
static __global__ void cols_range_init_kernel(int32_t *range) {
    range[0] = 0x7fffffff;
    range[1] = -0x7fffffff - 1;
}

// e[w & mask][.] = T - a w - c in stored order, and the column of zeros
static __global__ __launch_bounds__(256) void cols_pack_table_kernel(const int32_t *__restrict__ t, int16_t *__restrict__ e, int bits, int c) {
    const size_t n = (size_t)1 << bits, total = n * (n + 1), stride = (size_t)gridDim.x * 256;
    const int h = 1 << (bits - 1), mask = (int)n - 1;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
        const int col = (int)(i >> bits), at = cols_order((int)(i & (n - 1)), bits);
        const int w = ((col & mask) ^ h) - h, a = (at ^ h) - h;
        e[i] = (size_t)col < n ? (int16_t)(int)((uint32_t)t[((size_t)(w + h) << bits) + (size_t)(a + h)] - (uint32_t)(a * w) - (uint32_t)c) : (int16_t)0;
    }
}

// weights [N][Cin][taps] -> ColsParams::words (zero weights and the column of zeros beyond the last pair and the odd channel);
// clears the arrival counters
static __global__ __launch_bounds__(256) void cols_pack_words_kernel(const int16_t *__restrict__ w, uint32_t *__restrict__ words, uint32_t *arrived,
                                                                     int n_arrived, int N, int Cin, int taps, int cp, int pairs, int padded, int n_tiles,
                                                                     int bits) {
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < n_arrived) arrived[i] = 0u;
    if (i >= n_tiles * padded * COLS_NT) return;
    const int ch = i & 3, np = i >> 2, nt = np / padded, p = np - nt * padded;
    const int tap = p / cp, c = p - tap * cp, n = nt * COLS_NT + ch;
    const int h = 1 << (bits - 1), mask = 2 * h - 1;
    uint32_t wv[2], col[2];
    for (int j = 0; j < 2; ++j) {
        const bool real = p < pairs && 2 * c + j < Cin;
        const int v = real && n < N ? ((w[((size_t)n * Cin + 2 * c + j) * taps + tap] & mask) ^ h) - h : 0;
        wv[j] = (uint32_t)v & 0xffffu;
        col[j] = real ? (uint32_t)v & (uint32_t)mask : (uint32_t)mask + 1u;
    }
    uint32_t *const o = words + (size_t)np * 8;
    o[ch] = wv[0] | wv[1] << 16;
    o[4 + ch] = col[0] | col[1] << 16;
}

// activation sources: int16 codes (wrapped into the operand width), or fp32 quantised on the fly (quantize_i16_kernel)
struct ColsI16 {
    const int16_t *x;
    int h, mask;
    __device__ __forceinline__ uint32_t code(size_t i) const { return (uint32_t)((((int)x[i] & mask) ^ h) - h) & 0xffffu; }
};
struct ColsF32 {
    const float *x;
    float scale, Q;
    __device__ __forceinline__ uint32_t code(size_t i) const {
        float r = rintf(x[i] / scale);
        if (r != r) r = 0.0f;
        if (r > Q) r = Q;
        if (r < -Q) r = -Q;
        return (uint32_t)(int)r & 0xffffu;
    }
};

// NCHW -> [N][H + 2 ph][cp][sw][wsub] words, zero borders
template <typename Src>
__global__ __launch_bounds__(256) void cols_copy_kernel(const Src x, uint32_t *__restrict__ xt, int C, int H, int W, int ph, int pw, FastDiv dwsub,
                                                        FastDiv dsw, FastDiv dcp, FastDiv dhp, uint32_t total) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= total) return;
    const uint32_t r0 = dwsub.div(i), xs = i - r0 * dwsub.d;
    const uint32_t r1 = dsw.div(r0), xr = r0 - r1 * dsw.d;
    const uint32_t r2 = dcp.div(r1), c = (r1 - r2 * dcp.d) * 2u;
    const uint32_t n = dhp.div(r2), yp = r2 - n * dhp.d;
    const int y = (int)yp - ph, xx = (int)(xs * dsw.d + xr) - pw;
    uint32_t v = 0;
    if (y >= 0 && y < H && xx >= 0 && xx < W) {
        const size_t HW = (size_t)H * W, at = ((size_t)n * C + c) * HW + (size_t)y * W + xx;
        v = x.code(at);
        if ((int)c + 1 < C) v |= x.code(at + HW) << 16;
    }
    xt[i] = v;
}

// [M][K] -> [K / 2][Mp] words (rows beyond M are never stored by their reader and stay as they are): tiles of 64 rows x 32
// pairs go through LDS so that reads and writes coalesce
template <typename Src>
__global__ __launch_bounds__(256) void cols_rows_kernel(const Src a, uint32_t *__restrict__ xt, int M, int K, int cp, int Mp) {
    __shared__ uint32_t tile[32][65];
    const int m0 = blockIdx.x * 64, c0 = blockIdx.y * 32, tid = threadIdx.x;
    for (int pass = 0; pass < 8; ++pass) {
        const int ml = pass * 8 + tid / 32, c = tid % 32, m = m0 + ml, k = (c0 + c) * 2;
        uint32_t v = 0;
        if (m < M && k < K) {
            v = a.code((size_t)m * K + k);
            if (k + 1 < K) v |= a.code((size_t)m * K + k + 1) << 16;
        }
        tile[c][ml] = v;
    }
    __syncthreads();
    for (int pass = 0; pass < 8; ++pass) {
        const int c = pass * 4 + tid / 64, ml = tid % 64;
        if (m0 + ml < M && c0 + c < cp) xt[(size_t)(c0 + c) * Mp + m0 + ml] = tile[c][ml];
    }
}

// (v & mask) | base in one instruction (the compiler makes two, with the mask as a literal)
__device__ __forceinline__ uint32_t cols_and_or(uint32_t v, uint32_t mask, uint32_t base) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(mask), "s"(base));
    return r;
}

// BITS: operand width.  NR: runs of four pixels per thread.
template <int BITS, int NR>
__global__ __launch_bounds__(COLS_THREADS) void lut_cols_kernel(const ColsParams p) {
    constexpr int KP = 1 << (12 - BITS);            // channel pairs of a stage
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    constexpr int UNITS = 1 << (BITS - 2);          // 8-byte groups of a column
    __shared__ __attribute__((aligned(COLS_BUF))) unsigned char tbl[2 * COLS_BUF];
    __shared__ uint32_t shared_word;
    const int tid = threadIdx.x;
    // units (channel tile, slice) x row tiles.  Workgroups that read the same columns - one unit, all row tiles - go to one XCD
    // (consecutive workgroups go to consecutive XCDs) and run side by side, where the number of units allows it
    const int units = p.n_tiles * p.ksplit;
    int unit, mt;
    if ((units & 7) == 0) {
        const int local = blockIdx.x >> 3, u8 = local / p.m_tiles;
        mt = local - u8 * p.m_tiles;
        unit = u8 * 8 + (int)(blockIdx.x & 7u);
    } else {
        unit = blockIdx.x / (unsigned)p.m_tiles;
        mt = blockIdx.x - unit * p.m_tiles;
    }
    const int nt = unit % p.n_tiles, ks = unit / p.n_tiles;
    const int s_begin = (int)((long long)ks * p.stages / p.ksplit), s_end = (int)((long long)(ks + 1) * p.stages / p.ksplit);
    const uint4 *const words = p.words + (size_t)nt * p.stages * KP * 2;

    const int run0 = mt * (COLS_THREADS * NR) + tid;            // run j of this thread: run0 + j * 1024
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool live = (mt * (COLS_THREADS * NR) + wave * 64) * 4 < p.Mv;          // some pixel of this wave exists
    uint32_t base[NR];
    const FastDiv dr = p.d_HoWv, dc = p.d_Wv;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const int r0 = (run0 + j * COLS_THREADS) * 4;
        const uint32_t r = r0 < p.Mv ? (uint32_t)r0 : 0u;
        const uint32_t img = dr.div(r), pix = r - img * dr.d, a = dc.div(pix), b = pix - a * dc.d;
        base[j] = img * (uint32_t)p.img_stride + a * (uint32_t)p.oy_stride + b;
    }

    int acc[NR * 4][COLS_NT];
#pragma unroll
    for (int i = 0; i < NR * 4; ++i)
#pragma unroll
        for (int c = 0; c < COLS_NT; ++c) acc[i][c] = 0;

    // The words of a pair come through vector loads, one pair (column numbers: one stage) ahead: scalar loads would share their
    // counter with the LDS reads, and every first read of a pair would wait for them
    uint32_t vzero = 0;
    asm("" : "+v"(vzero));
    auto pair_words = [&](int at, int half) { return *reinterpret_cast<const uint4 *>(reinterpret_cast<const unsigned char *>(words + (size_t)at * 2 + half) + vzero); };
    // columns of a stage: 2 units of 8 bytes per thread and channel (the table of a unit is the same for the whole wave)
    constexpr int NCW = KP > 1 ? 2 : 1;
    u32x2_t ld[2][COLS_NT];
    uint4 cw[NCW];
    auto load_numbers = [&](int stage) {
#pragma unroll
        for (int u = 0; u < NCW; ++u) cw[u] = pair_words(stage * KP + ((u * COLS_THREADS + wave * 64) >> (BITS - 1)), 1);
    };
    auto load_cols = [&]() {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int U = u * COLS_THREADS + wave * 64, kk = U >> (BITS - 2);
            const int pos = (U & (UNITS - 1)) + (tid & 63);
            const uint4 q = cw[NCW > 1 ? u : 0];
            const uint32_t col[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int c = 0; c < COLS_NT; ++c) {
                const uint32_t number = (uint32_t)__builtin_amdgcn_readfirstlane((int)col[c]) >> (16 * (kk & 1)) & 0xffffu;
                ld[u][c] = *reinterpret_cast<const u32x2_t *>(p.e + ((size_t)number << BITS) + pos * 4);
            }
        }
    };
    auto store_cols = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int U = u * COLS_THREADS + tid, kk = U >> (BITS - 2), pos = U & (UNITS - 1);
            unsigned char *const to = tbl + buf * COLS_BUF + (kk << (BITS + 3)) + pos * 16;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint4 v;
                v.x = __builtin_amdgcn_perm(ld[u][1][h], ld[u][0][h], 0x05040100u);
                v.y = __builtin_amdgcn_perm(ld[u][3][h], ld[u][2][h], 0x05040100u);
                v.z = __builtin_amdgcn_perm(ld[u][1][h], ld[u][0][h], 0x07060302u);
                v.w = __builtin_amdgcn_perm(ld[u][3][h], ld[u][2][h], 0x07060302u);
                *reinterpret_cast<uint4 *>(to + h * (4 << BITS)) = v;
            }
        }
    };

    // words of pair c of tap (ky, kx), walked in order
    int pair = s_begin * KP;
    int c, kx, ky;
    {
        const int tap = (int)p.d_cp.div((uint32_t)pair);
        c = pair - tap * p.cp;
        ky = (int)p.d_kw.div((uint32_t)tap);
        kx = tap - ky * p.kw;
    }
    auto load_words = [&](u32x4_a4 (&w)[NR]) {
        const uint32_t xo = (uint32_t)(kx * p.dw), xs = p.d_sw.div(xo), xr = xo - xs * p.d_sw.d;
        const uint32_t off = (uint32_t)(c * p.ch_stride + ky * p.ky_stride) + xr * (uint32_t)p.wsub + xs;
#pragma unroll
        for (int j = 0; j < NR; ++j) w[j] = *reinterpret_cast<const u32x4_a4 *>(p.xt + base[j] + off);
        if (++c == p.cp) {
            c = 0;
            if (++kx == p.kw) { kx = 0; ++ky; }
        }
    };
    const s16x2_t one_lo = {1, 0}, one_hi = {0, 1};
    typedef const __attribute__((address_space(3))) u32x2_t *lds_entry_t;
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const uint32_t lds_tbl = (uint32_t)(uintptr_t)(lds_ptr_t)tbl;
    uint32_t mask8 = MASK << 3;
    asm("" : "+v"(mask8));             // (in a vector register: see cols_and_or)
    auto gather = [&](uint32_t t, const u32x4_a4 (&w)[NR], const uint4 wp) {
        const uint32_t wx[4] = {wp.x, wp.y, wp.z, wp.w};
        u32x2_t d[NR * 4][2];
#pragma unroll
        for (int i = 0; i < NR * 4; ++i) {
            const uint32_t a = w[i >> 2][i & 3];
            d[i][0] = *(lds_entry_t)(uintptr_t)cols_and_or(a << 3, mask8, t);
            d[i][1] = *(lds_entry_t)(uintptr_t)(cols_and_or(a >> 13, mask8, t) + (8u << BITS));
        }
        __builtin_amdgcn_sched_barrier(0);      // (all reads are on their way before the first is waited for)
#pragma unroll
        for (int i = 0; i < NR * 4; ++i) {
            const s16x2_t av = __builtin_bit_cast(s16x2_t, (uint32_t)w[i >> 2][i & 3]);
            const uint32_t e0[2] = {d[i][0].x, d[i][0].y}, e1[2] = {d[i][1].x, d[i][1].y};
#pragma unroll
            for (int n = 0; n < COLS_NT; ++n) {
                acc[i][n] = __builtin_amdgcn_sdot2(av, __builtin_bit_cast(s16x2_t, wx[n]), acc[i][n], false);
                acc[i][n] = __builtin_amdgcn_sdot2(__builtin_bit_cast(s16x2_t, e0[n >> 1]), n & 1 ? one_hi : one_lo, acc[i][n], false);
                acc[i][n] = __builtin_amdgcn_sdot2(__builtin_bit_cast(s16x2_t, e1[n >> 1]), n & 1 ? one_hi : one_lo, acc[i][n], false);
            }
        }
    };

    load_numbers(s_begin);
    load_cols();
    store_cols(0);
    if (s_begin + 1 < s_end) load_numbers(s_begin + 1);
    const int p_end = min(p.pairs, s_end * KP);
    u32x4_a4 w[NR];
    uint4 wp{};
    if (live && pair < p_end) {
        load_words(w);
        wp = pair_words(pair, 0);
    }
    __syncthreads();
    for (int s = s_begin; s < s_end; ++s) {
        const int buf = (s - s_begin) & 1;
        if (s + 1 < s_end) {
            load_cols();
            load_numbers(min(s + 2, s_end - 1));
        }
        if (live) {
#pragma unroll 1
            for (int j = 0; j < KP && pair < p_end; ++j, ++pair) {
                u32x4_a4 cur[NR];
#pragma unroll
                for (int i = 0; i < NR; ++i) cur[i] = w[i];
                const uint4 wp_cur = wp;
                if (pair + 1 < p_end) {         // one pair ahead
                    load_words(w);
                    wp = pair_words(pair + 1, 0);
                }
                gather(lds_tbl + (uint32_t)(buf * COLS_BUF + (j << (BITS + 4))), cur, wp_cur);
            }
        }
        if (s + 1 < s_end) store_cols(buf ^ 1);
        __syncthreads();
    }

    // slices: see the head of this file.  Device-scope (write-through) stores and loads, one counter per tile
    if (p.ksplit > 1) {
        const int tile = nt * p.m_tiles + mt;
        unsigned long long *const slices = reinterpret_cast<unsigned long long *>(p.partial) + (size_t)tile * p.ksplit * (NR * 4 * COLS_THREADS * 2);
        if (live) {
            unsigned long long *const mine = slices + (size_t)ks * (NR * 4 * COLS_THREADS * 2);
#pragma unroll
            for (int i = 0; i < NR * 4; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    __hip_atomic_store(mine + (size_t)(i * 2 + h) * COLS_THREADS + tid,
                                       (unsigned long long)(uint32_t)acc[i][2 * h] | (unsigned long long)(uint32_t)acc[i][2 * h + 1] << 32,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        __syncthreads();
        if (tid == 0) shared_word = __hip_atomic_fetch_add(p.arrived + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (shared_word != (uint32_t)(p.ksplit - 1)) return;
        if (live) {
            for (int o = 0; o < p.ksplit; ++o) {
                if (o == ks) continue;
                const unsigned long long *const theirs = slices + (size_t)o * (NR * 4 * COLS_THREADS * 2);
#pragma unroll
                for (int i = 0; i < NR * 4; ++i)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const unsigned long long v = __hip_atomic_load(theirs + (size_t)(i * 2 + h) * COLS_THREADS + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        acc[i][2 * h] += (int)(uint32_t)v;
                        acc[i][2 * h + 1] += (int)(uint32_t)(v >> 32);
                    }
            }
        }
    }

    const int n0 = nt * COLS_NT, nch = min(COLS_NT, p.N - n0);
    uint32_t v[NR * 4][COLS_NT];
#pragma unroll
    for (int i = 0; i < NR * 4; ++i)
#pragma unroll
        for (int n = 0; n < COLS_NT; ++n) v[i][n] = (uint32_t)acc[i][n] + (uint32_t)p.corr;
    if (p.deq) {
        float sc[COLS_NT], bi[COLS_NT];
#pragma unroll
        for (int n = 0; n < COLS_NT; ++n) {
            const int ch = min(n0 + n, p.N - 1);
            sc[n] = p.scales ? p.scales[ch] : p.scale;
            bi[n] = p.bias ? p.bias[ch] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < NR * 4; ++i)
#pragma unroll
            for (int n = 0; n < COLS_NT; ++n) {
                float y = (float)(int32_t)v[i][n] * sc[n];
                if (p.bias) y = y + bi[n];
                if (p.act == 1) y = y > 0.0f ? y : 0.0f;
                v[i][n] = __float_as_uint(y);
            }
        if (p.act == 2) {       // through LDS, so that the code of tanh is there once (each thread keeps to its own words)
            __syncthreads();
            float *const mine = reinterpret_cast<float *>(tbl) + tid;
#pragma unroll
            for (int i = 0; i < NR * 4; ++i)
#pragma unroll
                for (int n = 0; n < COLS_NT; ++n) mine[(i * COLS_NT + n) * COLS_THREADS] = __uint_as_float(v[i][n]);
#pragma unroll 1
            for (int i = 0; i < NR * 4 * COLS_NT; ++i) mine[i * COLS_THREADS] = tanh_spec(mine[i * COLS_THREADS]);
#pragma unroll
            for (int i = 0; i < NR * 4; ++i)
#pragma unroll
                for (int n = 0; n < COLS_NT; ++n) v[i][n] = __float_as_uint(mine[(i * COLS_NT + n) * COLS_THREADS]);
        }
    }
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        const int r0 = (run0 + j * COLS_THREADS) * 4;
        if (r0 >= p.Mv) continue;
        const uint32_t img = dr.div((uint32_t)r0), pix = (uint32_t)r0 - img * dr.d, a = dc.div(pix), b = pix - a * dc.d;
        const int nv = min(4, p.Wo - (int)b);
        const size_t plane = p.linear ? 1 : (size_t)p.out_plane;
        const size_t at = p.linear ? (size_t)b * p.N + n0 : ((size_t)img * p.N + n0) * plane + (size_t)a * p.Wo + b;
        const size_t px = p.linear ? (size_t)p.N : 1;
        int32_t *const o = p.out + at;
        const bool al = (reinterpret_cast<uintptr_t>(p.out) & 15u) == 0 && nv == 4 && nch == 4;
        if (al && !p.linear && ((at | plane) & 3) == 0) {
#pragma unroll
            for (int n = 0; n < COLS_NT; ++n) *reinterpret_cast<uint4 *>(o + n * plane) = make_uint4(v[4 * j][n], v[4 * j + 1][n], v[4 * j + 2][n], v[4 * j + 3][n]);
        } else if (al && p.linear && (p.N & 3) == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<uint4 *>(o + i * px) = make_uint4(v[4 * j + i][0], v[4 * j + i][1], v[4 * j + i][2], v[4 * j + i][3]);
        } else {
#pragma unroll
            for (int n = 0; n < COLS_NT; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n < nch && i < nv) o[n * plane + i * px] = (int32_t)v[4 * j + i][n];
        }
    }
}

}  // namespace adapt
