// "Byte" kernel: the derived-table product (see lut_lines.hpp) for tables that are an exact product plus an error of one
// byte.
//
// Byte form of a table: T[a][w] = (a & am) * (w & wm) + c + e[a][w] with -128 <= e <= 127, where am and wm clear up to
// three low bits (all ones: the plain product).  A multiplier that is the exact product plus an error spanning at most 255
// has this form, and so has one that drops low operand bits (plus such an error); adapt_lut_create looks for it.  Then
//     acc[m][n] = sum_k e[a_mk][w_nk]  +  sum_k (a_mk & am)(w_nk & wm)  +  K c
// : every term is still looked up, but an entry is one byte, so one 16-byte LDS read serves 16 output channels instead of
// 8 and a table streamed from L2 serves twice the channels; the middle sum is an ordinary int8 matrix product, which costs
// one matrix instruction per 16 reads.  Sums wrap in 32 bits, so the split is exact.
//
// Derived tables D[a][slot][ch] = e[a][w] in 256-byte lines: line a of a step's table holds, for the step's 16 inner
// indices ("slots"), the bytes of the 16 output channels of the tile.
//
// Mapping.  Workgroup = 16 waves, 256 R output pixels and one tile of 16 channels; a wave = 16 row slots (R pixels each)
// x 4 k-subs: lane l serves row slot l % 16 and k-sub q = l / 16.  In a step each k-sub takes one group of four slots
// (one activation word per pixel): 4 R reads of 16 bytes per lane.  v_mfma_i32_16x16x64_i8 computes D[i][j] += sum_k A[i][k]
// B[k][j] with lane l holding column j = l % 16 of B for the 16 k of block l / 16.  With B = the 16 bytes a lane has just
// read and A[ch][.] = 1 on byte ch of every block, D[ch][j] collects the entries of channel ch over the four k-subs of row
// slot j: one instruction widens, adds and reduces 64 x 16 entries.  Lane l ends with channels 4 (l / 16) .. + 3 of row
// slot l % 16, for each of its R pixels: exactly what an epilogue wants (runs of pixels per channel, four channels of a
// pixel as one word of the next layer's copy), no exchange between lanes.
//
// No bank conflicts by construction: the 16 lanes of a k-sub read 16 different slots in every instruction (row slot r
// takes group q ^ (r % 4) and, in read t, byte (t + r / 4) % 4 of it).
//
// The exact product needs, as B, the activations of four steps (64 inner indices): a lane holds the words of group
// q ^ (r % 4) of the four steps; two exchanges between lanes (v_permlane16_swap: l <-> l ^ 16, v_permlane32_swap: l <->
// l ^ 32) and selects by the bits of r % 4 leave k-sub q with the four groups of step q, in order.  The A operand is the
// packed weights of the four steps ([step][channel][slot] bytes).  Matrix and vector instructions of a SIMD do not overlap
// here (16.6 clocks for the one, 4 for the other, 10.8 for a lane exchange, all of them adding up), so this costs a fifth of
// the loop wherever the fill of LDS does not hide it; interleaving it with the reads changed nothing.
//
// LDS: tables of up to 32 KB (7 bits and fewer, or 8 bits behind a ReLU) in four buffers, of 64 KB in two; line address =
// buffer | activation byte << 8 | slot << 4, built by one v_perm_b32.  Tables are copied by LDS-direct loads, three steps
// ahead where there are four buffers: with two, nothing is on its way between the end of one copy and the start of the next,
// and every step pays the latency of L2 again (32 KB tables, two pixels per row slot: 1580 clocks a step with two buffers, 1450
// with four).
//
// Inner dimension.  Channels come in groups of four per filter tap; byte_slot() numbers the groups of all taps without
// gaps (only the last step is padded), and a table in LDS holds the byte offset of every group inside a window: strides,
// dilations, channel counts and taps need no further case.  Activation copy: [image][row][channel group][residue of the
// column modulo the horizontal stride][column / stride] words, so that consecutive output pixels are consecutive words
// for every stride.
//
// Rows are virtual: an image row of Wo pixels counts as Wv = Wo rounded up to runs of V = min(R, 4) pixels; what lies
// beyond is computed and not stored.
//
// What bounds it (one MI355X): with 64 KB tables the path that fills LDS (46 B per clock and compute unit, plus the latency of
// L2 once per step), with smaller ones or many pixels per table the matrix and vector instructions (20.6 clocks a read and
// SIMD), which equal what the LDS delivers (5.1 clocks a read).  One-byte entries halve all of it per lookup.  Measured against
// the two-digit form (lut_quad.hpp): 3 x 3, 64 -> 64 channels, 32 images of 32 x 32, 8 bits: 41 -> 31 us; 128 -> 256 channels, 64
// images of 16 x 16: 78 us = 62 T lookups/s; against the 128-byte-line kernel on odd sizes (100 -> 200 channels, stride 2,
// 27 -> 14 pixels wide, 50 images): 271 -> 81 us.  A launch costs 6500 clocks before its first step (first table) and 1400 to 3500
// behind the last.
//
// Split inner dimension: ksplit workgroups share a tile.  All but the last to arrive (a counter per tile) leave their sums
// in memory, the last one adds them to its own and finishes; its slice is a little longer, so that the others have stored
// by then.  The exchange goes through device-scope (sc1) stores, loads and one atomic: no cache write-back, no second launch,
// and nobody waits for anybody.
#pragma once
#include <type_traits>

#include "epilogue.hpp"

namespace adapt {

constexpr int BYTE_THREADS = 1024;
constexpr int BYTE_LINE = 256;              // bytes of a line: 16 slots x 16 channels
constexpr int BYTE_BUF = 65536;
constexpr int BYTE_STEP = 16;               // inner indices per step
constexpr int BYTE_TILE = 16;               // output channels per tile
constexpr int BYTE_ROW_SLOTS = 256;         // per workgroup
constexpr int BYTE_MAX_STEPS = 2040;        // steps of a product (room for the group offsets of a slice in LDS)
constexpr int BYTE_PF_DIST = 2;             // the L2 prefetch runs this many steps ahead of the table being copied
constexpr int BYTE_MAX_TILES = 1024;        // output tiles of a launch that splits the inner dimension (arrival counters)

typedef uint32_t b32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t b32x2_t __attribute__((ext_vector_type(2)));
typedef int bi32x4_t __attribute__((ext_vector_type(4)));

struct ByteParams {
    const int8_t *xt;           // activation copy (signed codes), smaller than 2^32 bytes
    const uint4 *dt;            // derived tables [phase][n_tile][step][line][slot] x 16 B
    const int8_t *wx;           // weights of the exact product [phase][n_tile][step][channel][slot]
    int32_t *out;
    int32_t *partial;           // ksplit > 1: [tile][slice][pixel of a slot][1024 lanes] x 16 B
    uint32_t *arrived;          // ksplit > 1: one counter per tile, zero between launches
    int Mv;                     // virtual rows
    int N, n_tiles, m_tiles, phases;
    int cg, taps, kw, steps;    // channel groups per tap, taps, filter width, steps of the whole inner dimension
    int ksplit, even;           // slices of the inner dimension: slice i ends at step (i + 1) even / ksplit, the last one at the end
    int bits, copy_lines;       // copy_lines: 2^bits, or half of it where all activations are >= 0
    int Wo, Wv;                 // output width (per phase), the same rounded up to runs
    uint32_t img_stride, oy_stride;     // bytes of xt per image / output row
    uint32_t ch_stride, ky_stride;      // bytes of xt per channel group / filter row
    int dw, wsub;               // horizontal dilation; columns per residue class of a copied row
    uint32_t amask;             // am in every byte
    int corr;                   // c x real lookups of an output
    FastDiv d_HoWv, d_Wv, d_ntiles, d_mtiles, d_phases, d_ksplit, d_taps, d_rest, d_kw, d_sw;
    uint32_t xt_off[4];         // per phase: bytes into xt,
    int oy0[4], ox0[4];         // position of its first output pixel; pixel (a, b) of a phase is (oy0 + a step, ox0 + b step)
    int out_step;
    int linear;                 // output [M][N] instead of [img][N][rows][out_w]
    int out_plane, out_w;
    int deq, act;               // as in LinesParams
    float scale;
    const float *scales, *bias, *resid;
    int no_out;
    ChainOut chain;
    const int32_t *zsum;        // transposed convolution with border terms (see LinesParams)
    FastDiv cv_s;
    int cv_Ho, cv_Wo, cv_H, cv_W, cv_kh, cv_kw, cv_pad, cv_Ly, cv_Lx;
};

// Flat channel group f of the inner dimension -> (tap, channel group of that tap).  Whole steps first, the taps of one
// block of 16 channels one after the other (a workgroup then re-reads the same activation lines, shifted, in consecutive
// steps); then the cg % 4 groups that are left of every tap, packed.
template <typename D1, typename D2>
__host__ __device__ __forceinline__ void byte_slot(int f, int taps, int cg, const D1 &div_taps, const D2 &div_rest, int *tap, int *c) {
    const int full = cg >> 2, rest = cg & 3, whole = full * taps * 4;
    if (f < whole) {
        const int s = f >> 2, blk = div_taps(s);
        *tap = s - blk * taps;
        *c = blk * 4 + (f & 3);
    } else {
        const int g = f - whole, t = rest ? div_rest(g) : taps;
        *tap = t;
        *c = full * 4 + (g - t * rest);
    }
}

// A operand that adds: lane l holds row i = l % 16, 1 on byte i of its block
__device__ __forceinline__ bi32x4_t byte_ones(int lane) {
    const int i = lane & 15, v = 1 << (8 * (i & 3));
    bi32x4_t a = {0, 0, 0, 0};
    if ((i >> 2) == 0) a.x = v;
    else if ((i >> 2) == 1) a.y = v;
    else if ((i >> 2) == 2) a.z = v;
    else a.w = v;
    return a;
}

// address = permute(activation word, column word, selector); read the 16 bytes there (OFF: constant part of the address)
template <int OFF>
__device__ __forceinline__ void byte_fetch(b32x4_t &v, uint32_t word, uint32_t colw, uint32_t sel) {
    uint32_t tmp;
    asm volatile("v_perm_b32 %[t], %[wd], %[cw], %[sl]\n\t"
                 "ds_read_b128 %[v], %[t] offset:%[of]"
                 : [v] "+v"(v), [t] "=&v"(tmp)
                 : [wd] "v"(word), [cw] "v"(colw), [sl] "v"(sel), [of] "n"(OFF));
}

template <int WAITN>
__device__ __forceinline__ void byte_add(bi32x4_t &d, b32x4_t &v, const bi32x4_t &a) {
    asm volatile("s_waitcnt lgkmcnt(%[wn])\n\t"
                 "v_mfma_i32_16x16x64_i8 %[d], %[a], %[v], %[d]"
                 : [d] "+v"(d)
                 : [v] "v"(v), [a] "v"(a), [wn] "n"(WAITN));
}

// Run i of row slot rs: image, row and first column of its V pixels; false if it lies past the end (the position is then
// that of run 0, a valid one)
template <int R>
__device__ __forceinline__ bool byte_run_pos(const ByteParams &p, int mt, int rs, int i, int &img, int &a, int &b) {
    constexpr int V = R < 4 ? R : 4, NRUN = R / V;
    const int r0 = ((mt * BYTE_ROW_SLOTS + rs) * NRUN + i) * V;
    const bool live = r0 < p.Mv;
    const FastDiv dr = p.d_HoWv, dc = p.d_Wv;
    const uint32_t r = live ? (uint32_t)r0 : 0u;
    img = (int)dr.div(r);
    const uint32_t pix = r - (uint32_t)img * dr.d;
    a = (int)dc.div(pix);
    b = (int)(pix - (uint32_t)a * dc.d);
    return live;
}

// The sums of a tile whose inner dimension is split: true in the workgroup that finishes the tile, which then holds the sum
// of all slices.  The workgroup of the last slice looks first: if all others have arrived it keeps its sums to itself.
// Everyone else stores its sums and counts itself in (and is the last one if the count says so).
template <int R, int NACC>
__device__ __forceinline__ bool byte_join_slices(const ByteParams &p, bi32x4_t (&acc)[NACC], uint32_t *shared_word, int tid, int tile, int ks, bool live) {
    const uint32_t others = (uint32_t)(p.ksplit - 1);
    const uint32_t voff = (uint32_t)tid * 16u;
    int32_t *const slices = p.partial + (size_t)tile * p.ksplit * (R * BYTE_THREADS * 4);
    bool alone = false;
    if (ks == p.ksplit - 1) {           // (the long slice; a look costs 1 us, which the others save)
        if (tid == 0) shared_word[0] = __hip_atomic_load(p.arrived + tile, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        alone = shared_word[0] == others;
    }
    if (!alone) {
        int32_t *const mine = slices + (size_t)ks * (R * BYTE_THREADS * 4);
        if (live) {
#pragma unroll
            for (int i = 0; i < R; ++i)
                asm volatile("global_store_dwordx4 %[o], %[v], %[sa] sc1" : : [o] "v"(voff), [v] "v"(acc[i]), [sa] "s"(mine + i * (BYTE_THREADS * 4)) : "memory");
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        __syncthreads();
        if (tid == 0) shared_word[0] = __hip_atomic_fetch_add(p.arrived + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (shared_word[0] != others) return false;
    }
    if (tid == 0) __hip_atomic_store(p.arrived + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!live) return true;
    constexpr int B = 8 / R;                          // slices whose loads are in flight together
    for (int o = 0; o < p.ksplit; o += B) {
        bi32x4_t t[B][R];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int from = o + j < p.ksplit ? o + j : ks;         // (past the end: any valid address)
            const int32_t *const theirs = slices + (size_t)from * (R * BYTE_THREADS * 4);
#pragma unroll
            for (int i = 0; i < R; ++i)
                asm volatile("global_load_dwordx4 %[v], %[o], %[sa] sc1" : [v] "=v"(t[j][i]) : [o] "v"(voff), [sa] "s"(theirs + i * (BYTE_THREADS * 4)) : "memory");
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const bool add = o + j < p.ksplit && o + j != ks;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                asm volatile("" : "+v"(t[j][i]));
                if (add) acc[i] += t[j][i];
            }
        }
    }
    return true;
}

// What becomes of the finished sums of a lane: channels cb .. cb + 3 of its R pixels.
// LEVEL 0: rescaling, bias, residual, ReLU.  1: also border terms of a transposed convolution and the next layer's copy.
// 2: also tanh (16 or 32 inlined copies of it: an instantiation of its own).  3: the same in the kernel for tables whose
// exact product drops low bits of the activations.
template <int R, int LEVEL, int NACC>
__device__ __forceinline__ void byte_epilogue(const ByteParams &p, const bi32x4_t (&acc)[NACC], const float (&sc)[4], const float (&bi)[4], int mt, int rs,
                                              int ph, int cb) {
    constexpr int V = R < 4 ? R : 4, NRUN = R / V;
    const int nch = min(4, p.N - cb);
    const int oy0 = pick4(p.oy0, ph), ox0 = pick4(p.ox0, ph);
    const int px = p.linear ? p.N : p.out_step;             // elements between consecutive pixels of a run,
    const size_t plane = p.linear ? 1 : (size_t)p.out_plane;       // and between channels
#pragma unroll
    for (int run = 0; run < NRUN; ++run) {
        int img, a, b;
        if (!byte_run_pos<R>(p, mt, rs, run, img, a, b)) continue;
        const int oy = oy0 + a * p.out_step, ox = ox0 + b * p.out_step;
        const int nv = min(V, p.Wo - b);            // pixels of the run that exist
        const bool whole = nv == V && nch == 4;
        const size_t at = p.linear ? (size_t)b * p.N + cb : ((size_t)img * p.N + cb) * plane + (size_t)oy * p.out_w + ox;
        // runs of a channel are one access where they are contiguous and aligned; in a linear layer the four channels are
        const bool vec = whole && px == 1 && ((at | plane) & (V - 1)) == 0;
        const bool vec_ch = whole && p.linear && (p.N & 3) == 0;
        uint32_t v[4][V];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < V; ++i) v[r][i] = (uint32_t)acc[run * V + i][r] + (uint32_t)p.corr;
        if (LEVEL >= 1 && p.zsum && (oy < p.cv_Ly || oy >= p.cv_Ho - p.cv_Ly || ox < p.cv_Lx || ox + (V - 1) * p.out_step >= p.cv_Wo - p.cv_Lx)) {
            for (int r = 0; r < nch; ++r) {
                uint32_t extra[V];
                convt_border_terms<V>(p, cb + r, oy, ox, extra);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    v[0][i] -= r == 0 ? extra[i] : 0u;
                    v[1][i] -= r == 1 ? extra[i] : 0u;
                    v[2][i] -= r == 2 ? extra[i] : 0u;
                    v[3][i] -= r == 3 ? extra[i] : 0u;
                }
            }
        }
        if (p.deq) {
            float y[4][V];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < V; ++i) y[r][i] = (float)(int32_t)v[r][i] * sc[r];
            if (p.bias) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < V; ++i) y[r][i] = y[r][i] + bi[r];
            }
            if (p.resid) {
                const float *const q = p.resid + at;
                float t[4][V];
                if (vec && V == 4 && (reinterpret_cast<uintptr_t>(p.resid) & 15u) == 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float4 f = *reinterpret_cast<const float4 *>(q + r * plane);
                        t[r][0] = f.x; t[r][1] = f.y; t[r][V - 2] = f.z; t[r][V - 1] = f.w;
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int i = 0; i < V; ++i) t[r][i] = r < nch && i < nv ? q[r * plane + (size_t)(i * px)] : 0.0f;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < V; ++i) y[r][i] = y[r][i] + t[r][i];
            }
            if (p.act == 1) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < V; ++i) y[r][i] = y[r][i] > 0.0f ? y[r][i] : 0.0f;
            } else if (LEVEL >= 2 && p.act == 2) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < V; ++i) y[r][i] = tanh_spec(y[r][i]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < V; ++i) v[r][i] = __float_as_uint(y[r][i]);
            if (LEVEL >= 1 && p.chain.buf) {
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    uint32_t code = 0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) code |= r < nch ? p.chain.code(y[r][i]) << (8 * r) : 0u;
                    if (i < nv) p.chain.put4(img, cb, oy, ox + i * p.out_step, code);
                }
                if (p.no_out) continue;
            }
        }
        int32_t *const o = p.out + at;
        const bool al = (reinterpret_cast<uintptr_t>(p.out) & (V * 4 - 1)) == 0;
        if (vec && al) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (V == 4) *reinterpret_cast<uint4 *>(o + r * plane) = make_uint4(v[r][0], v[r][1], v[r][V - 2], v[r][V - 1]);
                else *reinterpret_cast<uint2 *>(o + r * plane) = make_uint2(v[r][0], v[r][1]);
            }
        } else if (vec_ch && (reinterpret_cast<uintptr_t>(p.out) & 15u) == 0) {
#pragma unroll
            for (int i = 0; i < V; ++i) *reinterpret_cast<uint4 *>(o + (size_t)(i * px)) = make_uint4(v[0][i], v[1][i], v[2][i], v[3][i]);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < V; ++i)
                    if (r < nch && i < nv) o[r * plane + (size_t)(i * px)] = (int32_t)v[r][i];
        }
    }
}

// DOPS: table copy operations per wave and step = copied lines * 256 B / (16 waves * 1 KB): 4 / 2 / 1 for 256 / 128 / <= 64
// lines (fewer: one operation with fewer lanes).  R: pixels per row slot.  LEVEL: see byte_epilogue.
template <int DOPS, int R, int LEVEL>
__global__ __launch_bounds__(BYTE_THREADS) void lut_byte_kernel(const ByteParams p) {
    static_assert(R == 8 || R == 4 || R == 2, "pixels per row slot");
    constexpr int V = R < 4 ? R : 4;        // pixels per run: one load
    constexpr int NRUN = R / V;
    constexpr int NL = NRUN;                // activation loads per lane and step
    constexpr int NP = DOPS >= 2 ? 1 : 0;   // L2 prefetch loads per step (tables of one copy operation are not prefetched)
    // Tables of up to 32 KB: four buffers, a table is copied three steps ahead.  64 KB: two buffers, one step ahead.
    constexpr bool DEEP = DOPS <= 2;
    constexpr int AHEAD = DEEP ? 3 : 1;
    constexpr int NACC = R < 4 ? 4 : R;     // accumulators: with two pixels, two each (reads t and t + 1 do not depend on each other)
    // 160 KB; the alignment puts the buffers at multiples of 64 KB, which the address arithmetic needs
    __shared__ __attribute__((aligned(BYTE_BUF))) uint4 tbl[2 * (BYTE_BUF / 16)];
    __shared__ uint32_t goff[(BYTE_MAX_STEPS + 8) * 4];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;                // k-sub
    const int rl = lane & 15;               // row slot inside the wave
    const int rs = wave * 16 + rl;          // row slot inside the workgroup
    const int g = q ^ (rl & 3);             // this lane's channel group inside every step
    // Workgroup order: channel tile fastest; consecutive workgroups go to consecutive XCDs, so with 8 tiles (or a multiple)
    // a tile's tables stay in one L2, with 4 / 2 / 1 tiles every 2nd / 4th / 8th workgroup of a tile shares an XCD
    // (xcd_span).  The phases of a transposed convolution vary fastest among the workgroups of one XCD, so that the pixels
    // they interleave meet in its L2.
    const int wg = (int)p.d_ntiles.div(blockIdx.x);
    const int nt = blockIdx.x - wg * p.n_tiles;
    int xcd_span = (p.n_tiles < 8 && 8 % p.n_tiles == 0) ? 8 / p.n_tiles : 1;
    const int pf_span = xcd_span;
    if ((p.m_tiles * p.ksplit) % xcd_span) xcd_span = 1;
    const int wx_ = wg & (xcd_span - 1), wy = wg / xcd_span;
    const int wz = (int)p.d_phases.div((uint32_t)wy);
    const int ph = wy - wz * p.phases;
    const int rest = wz * xcd_span + wx_;
    const int ks = (int)p.d_mtiles.div((uint32_t)rest);
    const int mt = rest - ks * p.m_tiles;
    const int8_t *const xt = p.xt + pick4(p.xt_off, ph);
    const uint32_t table_bytes = (uint32_t)BYTE_LINE << p.bits;             // distance between the tables of two steps
    const uint32_t copy_bytes = (uint32_t)p.copy_lines * BYTE_LINE;
    const uint32_t line_mask = (uint32_t)(p.copy_lines - 1) * 0x01010101u;  // activation byte -> line
    const int s_begin = (int)p.d_ksplit.div((uint32_t)(ks * p.even));
    const int nsteps = (ks + 1 < p.ksplit ? (int)p.d_ksplit.div((uint32_t)((ks + 1) * p.even)) : p.steps) - s_begin;
    const bool live = (mt * BYTE_ROW_SLOTS + wave * 16) * R < p.Mv;         // some row of this wave exists
    const size_t first_table = (size_t)(ph * p.n_tiles + nt) * p.steps + s_begin;
    const unsigned char *const dt = reinterpret_cast<const unsigned char *>(p.dt) + first_table * table_bytes;
    const int8_t *const wx = p.wx + first_table * (BYTE_TILE * BYTE_STEP);
    typedef __attribute__((address_space(3))) void *lds_ptr_t;
    const uint32_t lds_tbl = (uint32_t)(uintptr_t)(lds_ptr_t)tbl;

    // table copy: operation o of wave w moves the 1 KB chunk (o * 16 + w); tables below 16 KB use part of the lanes
    const int lanes_act = DOPS > 1 ? 64 : min(64, (int)(copy_bytes >> 8));
    const uint64_t dma_mask = ~0ull >> (64 - lanes_act);
    const uint32_t dma_voff = (uint32_t)lane * 16u;
    // (8-bit tables: workgroup number `rest` of a tile and phase starts two chunks further on than its predecessor, so that
    // the workgroups that stream one table do not all ask L2 for the same lines at the same moment)
    const uint32_t dma_rot = DOPS == 4 ? (uint32_t)rest * 2u : 0u;
    // L2 prefetch: a table is new to the L2 that serves it, so each of up to 32 workgroups that stream it at about the same
    // time touches its share of the 128-byte lines BYTE_PF_DIST steps ahead of the copy, one plain load per wave (the
    // result is never used).
    const int pf_peers = max(1, min(32 / p.phases, (int)(gridDim.x / (unsigned)(p.n_tiles * p.phases * p.ksplit)) / pf_span));
    const int pf_share = 1 << (31 - __builtin_clz((unsigned)pf_peers));
    const int pf_lines = (int)(copy_bytes >> 7);
    const int pf_per_wg = (pf_lines + pf_share - 1) / pf_share;
    const int pf_per_wave = (pf_per_wg + 15) >> 4;
    const uint32_t pf_voff =
        128u * (uint32_t)min(((rest / pf_span) & (pf_share - 1)) * pf_per_wg + wave * pf_per_wave + min(lane, pf_per_wave - 1), pf_lines - 1);
    uint32_t pf_sink = 0;
    auto prefetch = [&](int step) {
        if constexpr (NP == 0) return;
        const int at = step < nsteps ? step : nsteps - 1;
        asm volatile("global_load_dword %[d], %[vo], %[sa]" : [d] "+v"(pf_sink) : [vo] "v"(pf_voff), [sa] "s"(dt + (size_t)(unsigned)at * table_bytes));
    };

    // Past the end of the slice there is nothing to copy.  DEEP: as many small loads are issued instead, so that the counted
    // waits stay the same (nothing waits for them in particular).  Two buffers: the wave waits for everything it has in
    // flight, which is little more than the activations it needs next.  (One asm statement: the branch stays inside it.)
    // (first_c: the first table, which always exists - no load then targets pf_sink while the compiler still computes addresses)
    auto dma = [&](int step, int buf, auto first_c, uint32_t &sink) {
        constexpr bool FIRST = decltype(first_c)::value;
        const unsigned char *src[DOPS];
        uint32_t to[DOPS];
#pragma unroll
        for (int o = 0; o < DOPS; ++o) {
            const uint32_t chunk = DOPS == 4 ? ((uint32_t)(o * 16 + wave) + dma_rot) & 63u : (uint32_t)(o * 16 + wave);
            const uint32_t at = DOPS > 1 ? chunk * 1024u : (uint32_t)(wave * lanes_act) * 16u;
            src[o] = dt + (size_t)(unsigned)step * table_bytes + at;
            to[o] = lds_tbl + (uint32_t)buf * (DEEP ? BYTE_BUF / 2 : BYTE_BUF) + at;
        }
        uint64_t save;
        const uint32_t po = pf_voff;        // (named here: asm operands inside the branches below do not capture)
        const int ns = nsteps;
#define BYTE_COPY_BEGIN "s_cmp_lt_i32 %[st], %[ns]\n\ts_cbranch_scc0 .Lbyte_none%=\n\ts_mov_b64 %[sv], exec\n\ts_mov_b64 exec, %[mk]\n\t"
#define BYTE_COPY_OP(i) "s_mov_b32 m0, %[t" #i "]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[vo], %[a" #i "]\n\t"
#define BYTE_NO_COPY "global_load_dword %[sk], %[po], %[tb]\n\t"
#define BYTE_COPY_END(ops) "s_mov_b64 exec, %[sv]\n\ts_branch .Lbyte_done%=\n.Lbyte_none%=:\n\t" ops ".Lbyte_done%=:"
        if constexpr (FIRST) {
#pragma unroll
            for (int o = 0; o < DOPS; ++o)
                asm volatile("s_mov_b64 %[sv], exec\n\ts_mov_b64 exec, %[mk]\n\t" BYTE_COPY_OP(0) "s_mov_b64 exec, %[sv]"
                             : [sv] "=&s"(save)
                             : [vo] "v"(dma_voff), [mk] "s"(dma_mask), [a0] "s"(src[o]), [t0] "s"(to[o])
                             : "memory");
        } else if constexpr (DOPS == 4)
            asm volatile(BYTE_COPY_BEGIN BYTE_COPY_OP(0) BYTE_COPY_OP(1) BYTE_COPY_OP(2) BYTE_COPY_OP(3) BYTE_COPY_END("s_waitcnt vmcnt(0)\n")
                         : [sv] "=&s"(save), [sk] "+v"(sink)
                         : [vo] "v"(dma_voff), [po] "v"(po), [tb] "s"(dt), [mk] "s"(dma_mask), [st] "s"(step), [ns] "s"(ns), [a0] "s"(src[0]), [t0] "s"(to[0]), [a1] "s"(src[1]),
                           [t1] "s"(to[1]), [a2] "s"(src[2]), [t2] "s"(to[2]), [a3] "s"(src[3]), [t3] "s"(to[3])
                         : "memory", "scc");
        else if constexpr (DOPS == 2)
            asm volatile(BYTE_COPY_BEGIN BYTE_COPY_OP(0) BYTE_COPY_OP(1) BYTE_COPY_END(BYTE_NO_COPY BYTE_NO_COPY)
                         : [sv] "=&s"(save), [sk] "+v"(sink)
                         : [vo] "v"(dma_voff), [po] "v"(po), [tb] "s"(dt), [mk] "s"(dma_mask), [st] "s"(step), [ns] "s"(ns), [a0] "s"(src[0]), [t0] "s"(to[0]), [a1] "s"(src[1]),
                           [t1] "s"(to[1])
                         : "memory", "scc");
        else
            asm volatile(BYTE_COPY_BEGIN BYTE_COPY_OP(0) BYTE_COPY_END(BYTE_NO_COPY)
                         : [sv] "=&s"(save), [sk] "+v"(sink)
                         : [vo] "v"(dma_voff), [po] "v"(po), [tb] "s"(dt), [mk] "s"(dma_mask), [st] "s"(step), [ns] "s"(ns), [a0] "s"(src[0]), [t0] "s"(to[0])
                         : "memory", "scc");
#undef BYTE_COPY_BEGIN
#undef BYTE_COPY_OP
#undef BYTE_COPY_END
#undef BYTE_NO_COPY
    };

    // byte offset of flat channel group f inside a window
    const int groups = p.taps * p.cg;
    auto group_off = [&](int f) -> uint32_t {
        if (f >= groups) f = 0;             // (padding of the last step, or past a slice: any valid address)
        int tap, c;
        byte_slot(f, p.taps, p.cg, [&](int v) { return (int)p.d_taps.div((uint32_t)v); }, [&](int v) { return (int)p.d_rest.div((uint32_t)v); }, &tap, &c);
        const int ky = (int)p.d_kw.div((uint32_t)tap), kx = tap - ky * p.kw;
        const uint32_t xo = (uint32_t)(kx * p.dw), xs = p.d_sw.div(xo), xr = xo - xs * p.d_sw.d;
        return (uint32_t)c * p.ch_stride + (uint32_t)ky * p.ky_stride + 4u * (xr * (uint32_t)p.wsub + xs);
    };
    dma(0, 0, std::true_type{}, pf_sink);
    for (int i = tid; i < nsteps * 4 + 8; i += BYTE_THREADS) goff[i] = group_off(s_begin * 4 + i);

    // runs of V consecutive pixels of one output row
    uint32_t base[NRUN];
#pragma unroll
    for (int i = 0; i < NRUN; ++i) {
        int img, a, b;
        byte_run_pos<R>(p, mt, rs, i, img, a, b);
        base[i] = (uint32_t)img * p.img_stride + (uint32_t)a * p.oy_stride + (uint32_t)b * 4u;
    }
    typedef typename std::conditional<V == 4, b32x4_t, b32x2_t>::type run_t;
    auto load_acts = [&](run_t (&w)[NRUN], uint32_t off) {
        const int8_t *const from = xt;
#pragma unroll
        for (int i = 0; i < NRUN; ++i) {
            const uint32_t at = base[i] + off;
            if constexpr (V == 4) asm volatile("global_load_dwordx4 %[v], %[b], %[xr]" : [v] "+v"(w[i]) : [b] "v"(at), [xr] "s"(from));
            else asm volatile("global_load_dwordx2 %[v], %[b], %[xr]" : [v] "+v"(w[i]) : [b] "v"(at), [xr] "s"(from));
        }
    };

    bi32x4_t acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = bi32x4_t{0, 0, 0, 0};
    run_t W[4][NRUN];                       // activation words of the four steps of a group
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < NRUN; ++i) W[k][i] = run_t{};
    b32x4_t rv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) rv[i] = b32x4_t{0, 0, 0, 0};
    bi32x4_t wa = {0, 0, 0, 0};             // A operand of the exact product of the group

    // Address pieces.  Column word for read t in buffer u: byte 0 = slot * 16, byte 2 = buffer.  Selector: result byte 0 =
    // column byte 0, byte 1 = activation byte e, byte 2 = column byte 2, byte 3 = 0 (bytes of the first source of
    // v_perm_b32 are numbered 4..7, those of the second 0..3, 0x0c gives zero).
    // (DEEP: buffers 2 u and 2 u + 1 share a column word, the odd one is a constant offset of 32 KB away)
    uint32_t colw[2][4], sel[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const uint32_t e = (uint32_t)((t + (rl >> 2)) & 3);
        sel[t] = 0x0c020000u | ((4u + e) << 8);
#pragma unroll
        for (int u = 0; u < 2; ++u) colw[u][t] = ((4u * (uint32_t)g + e) << 4) | ((lds_tbl >> 16) + (uint32_t)u) << 16;
    }
    const bi32x4_t ones = byte_ones(lane);
    const uint32_t wx_voff = (uint32_t)(q * (BYTE_TILE * BYTE_STEP) + rl * BYTE_STEP);
    const bool bit0 = rl & 1, bit1 = rl & 2;

    // behind a wait: what the loads have written is not read, moved or copied any earlier
    auto settle = [&]() {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < NRUN; ++i) asm volatile("" : "+v"(W[k][i]));
        asm volatile("" : "+v"(wa));
    };
    // the exact product of the four steps whose words are in W, for pixel i of the slot (see the head of this file)
    auto exact = [&](int i) {
        auto s01 = __builtin_amdgcn_permlane16_swap(W[0][i / V][i % V], W[1][i / V][i % V], false, false);
        auto s23 = __builtin_amdgcn_permlane16_swap(W[2][i / V][i % V], W[3][i / V][i % V], false, false);
        const uint32_t x0 = bit0 ? s01[1] : s01[0], x1 = bit0 ? s01[0] : s01[1];
        const uint32_t y0 = bit0 ? s23[1] : s23[0], y1 = bit0 ? s23[0] : s23[1];
        auto e0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);       // groups with low bit 0
        auto e1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);       // low bit 1
        bi32x4_t b;
        b.x = (int)(bit1 ? e0[1] : e0[0]);
        b.y = (int)(bit1 ? e1[1] : e1[0]);
        b.z = (int)(bit1 ? e0[0] : e0[1]);
        b.w = (int)(bit1 ? e1[0] : e1[1]);
        if constexpr (LEVEL == 3) {
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] &= (int)p.amask;
        }
        asm volatile("s_nop 1\n\tv_mfma_i32_16x16x64_i8 %[d], %[a], %[b], %[d]" : [d] "+v"(acc[i]) : [a] "v"(wa), [b] "v"(b));
    };

    // one step's reads: read t of the R pixels, t = 0..3, four in flight
    auto run_step = [&](auto bc, const run_t (&w)[NRUN]) {
        constexpr int buf = decltype(bc)::value, u = DEEP ? buf >> 1 : buf, off = DEEP && (buf & 1) ? BYTE_BUF / 2 : 0;
        constexpr int NR = 4 * R;
        uint32_t word[R];
#pragma unroll
        for (int i = 0; i < R; ++i) word[i] = DEEP ? w[i / V][i % V] & line_mask : w[i / V][i % V];
#pragma unroll
        for (int n = 0; n < 4; ++n) byte_fetch<off>(rv[n], word[n % R], colw[u][n / R], sel[n / R]);
#pragma unroll
        for (int n = 0; n < NR - 4; ++n) {
            byte_add<3>(acc[n % NACC], rv[n & 3], ones);
            byte_fetch<off>(rv[n & 3], word[(n + 4) % R], colw[u][(n + 4) / R], sel[(n + 4) / R]);
        }
        byte_add<3>(acc[(NR - 4) % NACC], rv[0], ones);
        byte_add<2>(acc[(NR - 3) % NACC], rv[1], ones);
        byte_add<1>(acc[(NR - 2) % NACC], rv[2], ones);
        byte_add<0>(acc[(NR - 1) % NACC], rv[3], ones);
    };

    // Step k of a group, step s of the slice.  A wave's memory operations retire in order, which is what the counted waits
    // rely on.  Per step it issues
    //   DEEP:      NL activation loads of the next step, (k = 0) the group's weights, DOPS copy operations of the table three
    //              steps ahead, the prefetch.  Waiting for a step's activations then means that the next table has landed too
    //              and leaves the two after it in flight; the step ends with a barrier alone.
    //   two bufs:  DOPS copy operations of the next table, NL loads, (k = 0) the weights, the prefetch.  The step ends when
    //              this wave's part of the copy has landed; the newer loads stay in flight across the barrier.
    // In the last step of a group the exact product comes first: the next loads go where its words are.
    uint32_t gv = 0;                        // group offset of the next step
    uint32_t gaddr = (uint32_t)(uintptr_t)(lds_ptr_t)goff + (uint32_t)g * 4u + 32u;         // that of the step after it
    auto step = [&](auto kc, int s) {
        constexpr int k = decltype(kc)::value;
        constexpr int nx = NL + NP + (k == 0 ? 1 : 0);      // operations of a step besides the copies
        constexpr int newer = NP + (k == 1 ? 1 : 0) + (DEEP ? DOPS : 0);    // of the previous step, issued after its activation loads
        if constexpr (!DEEP) dma(s + 1, (k + 1) & 1, std::false_type{}, pf_sink);
        if constexpr (k == 3) {
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"(newer + (DEEP ? 0 : DOPS)) : "memory");
            settle();
#pragma unroll
            for (int i = 0; i < R; ++i) exact(i);
        }
        load_acts(W[(k + 1) & 3], gv);
        if constexpr (k == 0) {
            const int8_t *const from = wx + (size_t)(unsigned)s * (BYTE_TILE * BYTE_STEP);
            asm volatile("global_load_dwordx4 %[v], %[o], %[sa]" : [v] "+v"(wa) : [o] "v"(wx_voff), [sa] "s"(from));
        }
        asm volatile("ds_read_b32 %[d], %[a]" : [d] "+v"(gv) : [a] "v"(gaddr));
        gaddr += 16u;
        if constexpr (DEEP) dma(s + AHEAD, (k + AHEAD) & 3, std::false_type{}, pf_sink);
        prefetch(s + AHEAD + BYTE_PF_DIST);
        if constexpr (k != 3) {
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"(newer + DOPS + nx) : "memory");
#pragma unroll
            for (int i = 0; i < NRUN; ++i) asm volatile("" : "+v"(W[k][i]));
        }
        run_step(std::integral_constant<int, DEEP ? k : (k & 1)>{}, W[k]);
        if constexpr (DEEP) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : [g] "+v"(gv) : : "memory");
        else asm volatile("s_waitcnt vmcnt(%[nx]) lgkmcnt(0)\n\ts_barrier" : [g] "+v"(gv) : [nx] "n"(nx) : "memory");
    };
    using std::integral_constant;

    // prologue: offsets, table and activations of the first step; DEEP: the next two tables are on their way
    load_acts(W[0], group_off(s_begin * 4 + g));
    if constexpr (DEEP) {
        dma(1, 1, std::false_type{}, pf_sink);
        dma(2, 2, std::false_type{}, pf_sink);
    }
#pragma unroll
    for (int d = 0; d < BYTE_PF_DIST; ++d) prefetch(AHEAD + d);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"((DEEP ? 2 * DOPS : 0) + NP * BYTE_PF_DIST) : "memory");
    gv = goff[4 + g];
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(gv) : : "memory");

    if (live) {
        int s = 0;
        for (; s + 4 <= nsteps; s += 4) {
            step(integral_constant<int, 0>{}, s);
            step(integral_constant<int, 1>{}, s + 1);
            step(integral_constant<int, 2>{}, s + 2);
            step(integral_constant<int, 3>{}, s + 3);
        }
        const int left = nsteps - s;
        if (left > 0) {
            step(integral_constant<int, 0>{}, s);
            if (left > 1) {
                step(integral_constant<int, 1>{}, s + 1);
                if (left > 2) step(integral_constant<int, 2>{}, s + 2);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");                  // retire what is still in flight
        if (left > 0) {                     // the last, incomplete group: no weights for the steps it does not have
            settle();
            if (q >= left) wa = bi32x4_t{0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < R; ++i) exact(i);
        }
        // the last matrix instructions have to leave the pipe before a vector instruction reads their registers (every
        // accumulator passes through an asm statement behind the waiting one, so that no read can be scheduled ahead of it)
        asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");
#pragma unroll
        for (int i = 0; i < NACC; ++i) asm volatile("" : "+v"(acc[i]));
    } else {                                // no row of this wave exists: it copies its part of the tables
        uint32_t sink = 0;
        for (int s = 0; s < nsteps; ++s) {
            dma(s + AHEAD, DEEP ? (s + AHEAD) & 3 : (s + 1) & 1, std::false_type{}, sink);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(DEEP ? 2 * DOPS : 0) : "memory");
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        asm volatile("" : : "v"(sink));
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");      // (for the prefetch loads of either branch)
    asm volatile("" : : "v"(pf_sink));

    if constexpr (NACC > R) {
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i] += acc[i + R];
    }

    // From here on the launch parameters are read again from the kernel arguments: kept in scalar registers across the loop,
    // they would not fit.
    const __attribute__((address_space(4))) ByteParams *args = (const __attribute__((address_space(4))) ByteParams *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const ByteParams &pe = *(const ByteParams *)args;
    // (requested before the slices are joined: the values travel meanwhile)
    const int cb = nt * BYTE_TILE + 4 * q;
    float sc[4] = {pe.scale, pe.scale, pe.scale, pe.scale}, bi[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (pe.scales) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[r] = pe.scales[min(cb + r, pe.N - 1)];
    }
    if (pe.bias) {
#pragma unroll
        for (int r = 0; r < 4; ++r) bi[r] = pe.bias[min(cb + r, pe.N - 1)];
    }
    if (pe.ksplit > 1 && !byte_join_slices<R>(pe, acc, goff, tid, (ph * pe.m_tiles + mt) * pe.n_tiles + nt, ks, live)) return;
    if (cb < pe.N) byte_epilogue<R, LEVEL>(pe, acc, sc, bi, mt, rs, ph, cb);
}

// ------------------------------------------------------------------------------------------------ packing

struct BytePack {
    const uint16_t *lut16;      // [a & mask][w & mask]
    const int8_t *w;
    uint4 *dt;
    int8_t *wx;
    int bits, N, Cin, taps, cg, n_tiles, steps;
    int tables, per_wg;         // phases * n_tiles * steps; tables per workgroup
    int wmode;                  // 0: [N][Cin][taps]; 1: [Cin][N][kh][kw], transposed convolution with stride st (phases as in pack_line_tables_convt_kernel)
    int kh, kw, st;
    int c, am, wm;              // see the head of this file (am, wm as signed masks)
    uint32_t *arrived;          // counters to clear, or nullptr
};

// A workgroup (blockIdx.y = band of BYTE_PACK_LINES table lines, blockIdx.x = group of p.per_wg tables) keeps the bytes
// e[a][.] of its band in LDS and looks them up there; per table its 256 threads fetch the 16 x 16 weights, then thread
// (slot, line residue) makes every 16th line, so that a wave stores whole kilobytes.  An entry is one LDS byte and a merge.
// Measured against gathering 16-bit entries from memory with one workgroup per table: 144 tables of 64 KB 30 -> 15 us, 3087
// tables 140 -> 65 us (3.1 TB/s).
constexpr int BYTE_PACK_LINES = 64;
static __global__ __launch_bounds__(256) void pack_byte_tables_kernel(const BytePack p) {
    __shared__ uint8_t band[BYTE_PACK_LINES * (256 + 4)];       // rows of lines + 4 bytes (consecutive rows start in different banks)
    __shared__ __align__(16) uint16_t index[2][16 * 16];        // [slot][channel]: column of the band
    const int tid = threadIdx.x;
    const int lines = 1 << p.bits, mask = lines - 1, half = lines >> 1, row = lines + 4;
    const int first = blockIdx.y * BYTE_PACK_LINES, here = min(BYTE_PACK_LINES, lines - first);
    const int t0 = (int)blockIdx.x * p.per_wg, t1 = min(t0 + p.per_wg, p.tables);
    if (p.arrived && blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = tid; i < BYTE_MAX_TILES; i += 256) p.arrived[i] = 0u;
    for (int i = tid; i < here * lines; i += 256) {
        const int r = i >> p.bits, u = i & mask, l = first + r;
        const int a = (l < half ? l : l - lines) & p.am, w = (u < half ? u : u - lines) & p.wm;
        band[r * row + u] = (uint8_t)((int)(int16_t)p.lut16[(size_t)l * lines + u] - a * w - p.c);
    }
    if (tid < here) band[tid * row + lines] = 0;                // column of weights that do not exist
    for (int tb = t0; tb < t1; ++tb) {
        const int tn = tb / p.steps, step = tb - tn * p.steps, nt = tn % p.n_tiles, phase = tn / p.n_tiles;
        uint16_t *const idx = index[(tb - t0) & 1];
        {
            const int slot = tid & 15, ch = tid >> 4;
            int tap, c;
            const int rest = p.cg & 3;
            byte_slot(step * 4 + (slot >> 2), p.taps, p.cg, [&](int v) { return v / p.taps; }, [&](int v) { return v / rest; }, &tap, &c);
            const int n = nt * BYTE_TILE + ch, ci = c * 4 + (slot & 3);
            int u = lines;
            if (n < p.N && ci < p.Cin && tap < p.taps) {
                size_t wi;
                if (p.wmode == 0) {
                    wi = ((size_t)n * p.Cin + ci) * p.taps + tap;
                } else {
                    const int Tx = p.kw / p.st, Ty = p.kh / p.st, mw = tap / Tx, nw = tap - mw * Tx;
                    const int ry = phase / p.st, rx = phase - ry * p.st;
                    const int ky = ry + p.st * (Ty - 1 - mw), kx = rx + p.st * (Tx - 1 - nw);
                    wi = (((size_t)ci * p.N + n) * p.kh + ky) * p.kw + kx;
                }
                u = (int)p.w[wi] & mask;
            }
            idx[slot * 16 + ch] = (uint16_t)u;
            if (blockIdx.y == 0) p.wx[(size_t)tb * (BYTE_TILE * BYTE_STEP) + ch * BYTE_STEP + slot] = (int8_t)(u == lines ? 0 : (u < half ? u : u - lines) & p.wm);
        }
        __syncthreads();            // (two buffers: a wave is at most one table ahead of the slowest)
        const int slot = tid & 15;
        const uint4 q0 = *reinterpret_cast<const uint4 *>(idx + slot * 16), q1 = *reinterpret_cast<const uint4 *>(idx + slot * 16 + 8);
        const uint32_t q[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
        uint4 *const dst = p.dt + ((size_t)tb * lines + first) * 16 + slot;
        for (int l = tid >> 4; l < here; l += 16) {
            const uint8_t *const from = band + l * row;
            uint32_t d[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
                d[g] = (uint32_t)from[q[2 * g] & 0xffffu] | (uint32_t)from[q[2 * g] >> 16] << 8 | (uint32_t)from[q[2 * g + 1] & 0xffffu] << 16 |
                       (uint32_t)from[q[2 * g + 1] >> 16] << 24;
            dst[(size_t)l * 16] = make_uint4(d[0], d[1], d[2], d[3]);
        }
    }
}

// ------------------------------------------------------------------------------------------------ activation copies

// NCHW -> [N][H + 2 ph][cg][sw][wsub] words of four channels (signed codes), zero borders and padded channels: column xp of
// a padded row is word (xp % sw) * wsub + xp / sw of its channel group.  U words per thread, all their operands requested
// before the first is converted.  Tensors below 2^31 elements.
template <typename Src, int U>
__global__ __launch_bounds__(256) void byte_copy_kernel(const Src x, int8_t *__restrict__ xt, int C, int H, int W, int ph, int pw, FastDiv dwsub,
                                                        FastDiv dsw, FastDiv dcg, FastDiv dhp, uint32_t total) {
    const uint32_t threads = gridDim.x * 256u, t = blockIdx.x * 256u + threadIdx.x;
    const uint32_t HW = (uint32_t)H * (uint32_t)W;
    typename Src::raw_t raw[U][4];
    bool live[U], have[U][4];
    uint32_t dst[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = t + (uint32_t)u * threads;
        live[u] = i < total;
        const uint32_t ii = live[u] ? i : 0u;
        const uint32_t r0 = dwsub.div(ii), xs = ii - r0 * dwsub.d;
        const uint32_t r1 = dsw.div(r0), xr = r0 - r1 * dsw.d;
        const uint32_t r2 = dcg.div(r1), c4 = r1 - r2 * dcg.d;
        const uint32_t n = dhp.div(r2), yp = r2 - n * dhp.d;
        const int y = (int)yp - ph, xx = (int)(xs * dsw.d + xr) - pw;
        const bool inside = live[u] && y >= 0 && y < H && xx >= 0 && xx < W;
        const uint32_t src = ((n * (uint32_t)C + c4 * 4u) * (uint32_t)H + (uint32_t)(inside ? y : 0)) * (uint32_t)W + (uint32_t)(inside ? xx : 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            have[u][c] = inside && (int)(c4 * 4u) + c < C;
            raw[u][c] = x.load(have[u][c] ? src + (uint32_t)c * HW : 0u);
        }
        dst[u] = ii * 4u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint32_t v = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) v |= (have[u][c] ? x.code8(raw[u][c]) : 0u) << (8 * c);
        if (live[u]) *reinterpret_cast<uint32_t *>(xt + dst[u]) = v;
    }
}

// [M][K] -> [cg][Mp] words of four inner indices (signed codes), zero beyond K (rows beyond M are never stored by their
// reader and stay as they are): a tile of 64 rows x 64 inner indices goes through LDS so that reads and writes coalesce.
template <typename Src>
__global__ __launch_bounds__(256) void byte_rows_kernel(const Src a, int8_t *__restrict__ at, int M, int K, int cg, int Mp) {
    __shared__ uint32_t tile[16][65];
    const int m0 = blockIdx.x * 64, c0 = blockIdx.y * 16;
    const int tid = threadIdx.x;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int ml = pass * 16 + tid / 16, c = tid % 16;
        const int m = m0 + ml, k = (c0 + c) * 4;
        uint32_t v = 0;
        if (m < M) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (k + i < K) v |= a.code8(a.x[(size_t)m * K + k + i]) << (8 * i);
        }
        tile[c][ml] = v;
    }
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int c = pass * 4 + tid / 64, ml = tid % 64;
        const int m = m0 + ml;
        if (m < M && c0 + c < cg) *reinterpret_cast<uint32_t *>(at + ((size_t)(c0 + c) * Mp + m) * 4) = tile[c][ml];
    }
}

}  // namespace adapt
