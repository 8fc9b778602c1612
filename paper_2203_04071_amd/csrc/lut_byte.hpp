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
// (one activation word per pixel): 4 R reads of 16 bytes per lane.  The matrix instruction computes D[i][j] += sum_k A[i][k]
// B[k][j] with lane l holding column j = l % 16 of B for the k of block l / 16.  With B = the bytes a lane has read
// and A[ch][.] = 1 on byte ch of every 16, D[ch][j] collects the entries of channel ch over the four k-subs of row
// slot j: one instruction widens, adds and reduces.  Of four neighbouring bytes of a row of that A at most one is not zero, so the
// sparse instruction (v_smfmac_i32_16x16x128_i8) takes two reads for the time of one (16.2 clocks of a SIMD either way).  Lane l ends
// with channels 4 (l / 16) .. + 3 of row slot l % 16, for each of its R pixels: exactly what an epilogue wants (runs of pixels per
// channel, four channels of a pixel as one word of the next layer's copy), no exchange between lanes.
//
// No bank conflicts by construction.  A 16-byte read is served in four passes of 16 lanes; lanes 0-3, 12-15, 20-23 and 24-27 share one
// (4-11, 16-19, 28-31 the next, and the same 32 lanes on; which is what the times of 13 mappings say).  In read t row
// slot r takes byte (t + r) % 4 of its word and group q, with bit 1 of it flipped for r >= 8: 16 different slots in every pass,
// 4.15 clocks a read (q alone: 8).
//
// The exact product needs, as B, the activations of a step in an order that is the same in every row slot.  Row slots 8 to 15 hold
// their groups two lanes of a column further, so one exchange between lanes for two steps (v_permlane32_swap: l <-> l ^ 32) and two
// selects by r >= 8 give a lane two groups of one of the two steps (v_mfma_i32_16x16x32_i8).  The A operand is the packed weights
// of the two steps ([step][channel][groups 0, 2, 1, 3] bytes).  It runs between the reads of the step after, a pixel every other
// pair.  (Before: groups q ^ (r % 4), two exchanges and four selects per word pair, all pixels in one go ahead of a step's reads:
// 4200 of the 18000 clocks of four steps with R = 8, with LDS idle; 128 -> 256 channels, 64 images of 16 x 16, 7 bits.)
//
// LDS: tables of up to 32 KB (7 bits and fewer, or 8 bits behind a ReLU) in four buffers, of 64 KB in two; line address =
// buffer | activation byte << 8 | slot << 4, built by one v_perm_b32.  Tables are copied by LDS-direct loads, three steps
// ahead where there are four buffers: with two, nothing is on its way between the end of one copy and the start of the next,
// and every step pays the latency of L2 again.  (Plain loads that touch a table two steps ahead of its copy gained nothing and cost
// 2 to 4 % once the copies were spread over the step.)
//
// Waves take turns by priority: a wave drops one level after every quarter of a step's reads, so that all 16 reach the barrier at about
// the same time; oldest first, as the hardware does it, four waves were left alone with the last third of a step (3250 -> 2850 clocks).
//
// Tables whose entries do not change with the low bits of an activation (multipliers that drop them) have a line for every code that is left;
// the copies hold the codes without those bits (8 bits, two of them dropped: 16 instead of 64 KB a step).
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
// What bounds it (one MI355X): LDS.  A step of R = 8 is 512 reads of a compute unit = 2125 clocks, and its table's way into LDS 256
// (32 KB); measured 2850 to 3300 (odd and even steps; 4700 before reads, exact product and copies were interleaved and paired).  With
// 64 KB tables and R <= 4 the path that fills LDS (46 B per clock and compute unit) is as long.  Measured against the two-digit form
// (lut_quad.hpp): 3 x 3, 64 -> 64 channels, 32 images of 32 x 32, 8 bits: 41 -> 30 us; against the
// 128-byte-line kernel on odd sizes (100 -> 200 channels, stride 2, 27 -> 14 pixels wide, 50 images): 271 -> 64 us, 52 with a table that
// drops two bits of the activation.  A launch costs 4500 clocks before its first step (first table).
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
constexpr int BYTE_GOFF = (BYTE_MAX_STEPS + 8) * 4;         // words of that room; border terms lie at its end, where they fit
constexpr int BYTE_MAX_TILES = 1024;        // output tiles of a launch that splits the inner dimension (arrival counters)

typedef uint32_t b32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t b32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t b32x8_t __attribute__((ext_vector_type(8)));
typedef int bi32x4_t __attribute__((ext_vector_type(4)));
typedef int bi32x2_t __attribute__((ext_vector_type(2)));

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
    int units;                  // > 0: workgroups by units, see the kernel
    int ksplit, even;           // slices of the inner dimension: slice i ends at step (i + 1) even / ksplit, the last one at the end
    int bits, copy_lines;       // 2^bits lines of a table; copy_lines: all of them, or half where all activations are >= 0
    int shift;                  // low bits that the copied codes do without
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
    int edge_rows, edge_cols;   // classes of border positions whose terms fit LDS (see byte_edge_class), or 0
};

// Rows (columns) of a transposed convolution's output by the window taps that have no input there.  Position q of a phase, of T taps
// and H input rows (H >= T - 1), meets tap m if 0 <= q - m < H: class 1 + q below T - 1, T + q - H from H on, 0 (none missing) between;
// 2 T - 1 classes.
__host__ __device__ __forceinline__ int byte_edge_class(int q, int T, int H) { return q < T - 1 ? 1 + q : (q >= H ? T + q - H : 0); }
__host__ __device__ __forceinline__ bool byte_edge_missing(int cls, int m, int T) { return cls > 0 && (cls < T ? m > cls - 1 : m <= cls - T); }

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

// Place of a slot among the 16 bytes of a step and channel in the weights of the exact product: groups 0, 2, 1, 3
__host__ __device__ __forceinline__ int byte_wx_pos(int slot) { return ((slot >> 2 & 1) * 2 + (slot >> 3)) * 4 + (slot & 3); }

// A operand that adds, sparse form: of every four bytes of a row two are held, `index` names their places.  Row i = l % 16 has 1 on byte
// i of both reads of its lanes: in the group of four that holds byte i a 1 at its place, zeros elsewhere (places p and 3 are named; for p = 3
// it is the second that carries the 1).
__device__ __forceinline__ bi32x4_t byte_ones(int lane) {
    const int i = lane & 15, v = 1 << (16 * (i >> 2 & 1) + ((i & 3) == 3 ? 8 : 0));
    return (i >> 3) == 0 ? bi32x4_t{v, 0, v, 0} : bi32x4_t{0, v, 0, v};
}
__device__ __forceinline__ uint32_t byte_ones_index(int lane) { return 0x11111111u * (((lane & 3) == 3 ? 0u : (uint32_t)(lane & 3)) | 12u); }

// address = permute(activation word, column word, selector); read the 16 bytes there (OFF: constant part of the address)
template <int OFF>
__device__ __forceinline__ void byte_fetch(b32x4_t &v, uint32_t word, uint32_t colw, uint32_t sel) {
    uint32_t tmp;
    asm volatile("v_perm_b32 %[t], %[wd], %[cw], %[sl]\n\t"
                 "ds_read_b128 %[v], %[t] offset:%[of]"
                 : [v] "=v"(v), [t] "=&v"(tmp)
                 : [wd] "v"(word), [cw] "v"(colw), [sl] "v"(sel), [of] "n"(OFF));
}

// d += the entries of two reads, once at most WAITN younger reads are in flight
template <int WAITN>
__device__ __forceinline__ void byte_add(bi32x4_t &d, b32x4_t &first, b32x4_t &second, const bi32x4_t &a, uint32_t index) {
    asm volatile("s_waitcnt lgkmcnt(%[wn])" : [f] "+v"(first), [s] "+v"(second) : [wn] "n"(WAITN));
    const b32x8_t both = __builtin_shufflevector(first, second, 0, 1, 2, 3, 4, 5, 6, 7);
    asm volatile("v_smfmac_i32_16x16x128_i8 %[d], %[a], %[v], %[i]" : [d] "+v"(d) : [v] "v"(both), [a] "v"(a), [i] "v"(index));
}

__device__ __forceinline__ void byte_exact(bi32x4_t &d, const bi32x2_t &a, const bi32x2_t &b) {
    asm volatile("s_nop 1\n\tv_mfma_i32_16x16x32_i8 %[d], %[a], %[b], %[d]" : [d] "+v"(d) : [a] "v"(a), [b] "v"(b));
}

__device__ __forceinline__ void byte_lds_word(uint32_t &v, uint32_t addr) { asm volatile("ds_read_b32 %[d], %[a]" : [d] "+v"(v) : [a] "v"(addr)); }

__device__ __forceinline__ void byte_load_weights(bi32x2_t &v, uint32_t off, const int8_t *from) {
    asm volatile("global_load_dwordx2 %[v], %[o], %[sa]" : [v] "+v"(v) : [o] "v"(off), [sa] "s"(from));
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
// LEVEL 0: rescaling, bias, residual, ReLU.  1: also the next layer's copy.  2: also border terms of a transposed convolution (an
// instantiation of its own: its code costs the ordinary chained layers 0.2 us a launch).  3: also tanh (16 or 32 inlined copies of it).
// 4: the same in the kernel for tables whose exact product drops low bits of the activations.
// edge: the border terms of the tile's channels by class of the position, four words of 16 bytes each, in LDS (or nullptr).
// NARROW: the lane holds R / 4 pixels of the slot, from pixel `first` on (channels 0 .. 3 of the tile), instead of all.
template <int R, int LEVEL, bool NARROW, int NACC>
__device__ __forceinline__ void byte_epilogue(const ByteParams &p, const bi32x4_t (&acc)[NACC], const float (&sc)[4], const float (&bi)[4], int mt, int rs,
                                              int ph, int cb, const uint4 *edge, int first) {
    constexpr int V = NARROW ? R / 4 : (R < 4 ? R : 4), NRUN = NARROW ? 1 : R / V;
    const int nch = min(4, p.N - cb);
    const int oy0 = pick4(p.oy0, ph), ox0 = pick4(p.ox0, ph);
    const int px = p.linear ? p.N : p.out_step;             // elements between consecutive pixels of a run,
    const size_t plane = p.linear ? 1 : (size_t)p.out_plane;       // and between channels
#pragma unroll
    for (int run = 0; run < NRUN; ++run) {
        int img, a, b;
        if (!byte_run_pos<R>(p, mt, rs, NARROW ? first >> 2 : run, img, a, b)) continue;
        if (NARROW) b += first & 3;
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
        if (LEVEL >= 2 && p.zsum && (oy < p.cv_Ly || oy >= p.cv_Ho - p.cv_Ly || ox < p.cv_Lx || ox + (V - 1) * p.out_step >= p.cv_Wo - p.cv_Lx)) {
            if (edge) {         // (class 0 holds zeros)
                const int Ty = (p.edge_rows + 1) >> 1, Tx = (p.edge_cols + 1) >> 1;
                const int cy = byte_edge_class((int)p.cv_s.div((uint32_t)(oy + p.cv_pad)), Ty, p.cv_H) * p.edge_cols;
                const int qx = (int)p.cv_s.div((uint32_t)(ox + p.cv_pad));
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    // (pixels beyond the row are not stored: any class)
                    const uint4 e = edge[(cy + min(byte_edge_class(qx + i, Tx, p.cv_W), p.edge_cols - 1)) * 4 + ((cb >> 2) & 3)];
                    v[0][i] -= e.x; v[1][i] -= e.y; v[2][i] -= e.z; v[3][i] -= e.w;
                }
            } else for (int r = 0; r < nch; ++r) {
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
                        t[r][0] = f.x; t[r][V > 1 ? 1 : 0] = f.y; t[r][V > 2 ? V - 2 : 0] = f.z; t[r][V - 1] = f.w;
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
            } else if (LEVEL >= 3 && p.act == 2) {
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
                if (V == 4) *reinterpret_cast<uint4 *>(o + r * plane) = make_uint4(v[r][0], v[r][V > 1 ? 1 : 0], v[r][V > 2 ? V - 2 : 0], v[r][V - 1]);
                else if (V == 2) *reinterpret_cast<uint2 *>(o + r * plane) = make_uint2(v[r][0], v[r][V - 1]);
                else o[r * plane] = (int32_t)v[r][0];
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
// AT_ONCE: a step's memory operations ahead of its reads (see below)
template <int DOPS, int R, int LEVEL, bool AT_ONCE = false>
__global__ __launch_bounds__(BYTE_THREADS) void lut_byte_kernel(const ByteParams p) {
    static_assert(R == 8 || R == 4 || R == 2, "pixels per row slot");
    constexpr int V = R < 4 ? R : 4;        // pixels per run: one load
    constexpr int NRUN = R / V;
    constexpr int NL = NRUN;                // activation loads per lane and step
    constexpr int NPAIR = 2 * R;            // pairs of reads per lane and step
    // Tables of up to 32 KB: four buffers, a table is copied three steps ahead.  64 KB: two buffers, one step ahead.
    constexpr bool DEEP = DOPS <= 2;
    constexpr int AHEAD = DEEP ? 3 : 1;
    constexpr int NACC = R < 4 ? 4 : R;     // accumulators: with two pixels, two each (reads t and t + 1 do not depend on each other)
    // 160 KB; the alignment puts the buffers at multiples of 64 KB, which the address arithmetic needs
    __shared__ __attribute__((aligned(BYTE_BUF))) uint4 tbl[2 * (BYTE_BUF / 16)];
    __shared__ __attribute__((aligned(16))) uint32_t goff[BYTE_GOFF];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;                // k-sub
    const int rl = lane & 15;               // row slot inside the wave
    const int rs = wave * 16 + rl;          // row slot inside the workgroup
    const int g = q ^ ((rl & 8) >> 2);      // this lane's channel group inside every step
    // Workgroup order: channel tile fastest; consecutive workgroups go to consecutive XCDs, so with 8 tiles (or a multiple)
    // a tile's tables stay in one L2, with 4 / 2 / 1 tiles every 2nd / 4th / 8th workgroup of a tile shares an XCD
    // (xcd_span).  The phases of a transposed convolution vary fastest among the workgroups of one XCD, so that the pixels
    // they interleave meet in its L2.
    // By units: a unit is the row tiles that read the same tables (a slice of a channel tile); unit u runs on XCD u % 8, its
    // row tiles one behind the other.  Elsewhere (13 tiles, say) every XCD fetches most tables: 1111 rows, K = 777, N = 999, 8 bits:
    // 75 -> 50 us; 100 -> 200 channels, stride 2, 27 -> 14 pixels wide, 50 images: 79 -> 64 us.
    const int wg = (int)p.d_ntiles.div(blockIdx.x);
    int nt = blockIdx.x - wg * p.n_tiles;
    int xcd_span = (p.n_tiles < 8 && 8 % p.n_tiles == 0) ? 8 / p.n_tiles : 1;
    if ((p.m_tiles * p.ksplit) % xcd_span) xcd_span = 1;
    const int wx_ = wg & (xcd_span - 1), wy = wg / xcd_span;
    const int wz = (int)p.d_phases.div((uint32_t)wy);
    int ph = wy - wz * p.phases;
    const int rest = wz * xcd_span + wx_;
    int ks = (int)p.d_mtiles.div((uint32_t)rest), mt = rest - ks * p.m_tiles;
    if (p.units > 0) {
        const int local = (int)(blockIdx.x >> 3), ul = (int)p.d_mtiles.div((uint32_t)local), unit = ul * 8 + (int)(blockIdx.x & 7);
        if (unit >= p.units) return;
        mt = local - ul * p.m_tiles;
        ks = (int)p.d_ntiles.div((uint32_t)unit);
        nt = unit - ks * p.n_tiles;
        ph = 0;
    }
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
    // (8-bit tables: every row tile starts two chunks further on than its predecessor, so that the workgroups that stream one table do not all
    // ask L2 for the same lines at the same moment)
    const uint32_t dma_rot = DOPS == 4 ? (uint32_t)mt * 2u : 0u;
    uint32_t pf_sink = 0;                   // (what loads that only keep a count bring back)

    // One of the DOPS operations that copy a step's table.  Past the end of the slice there is nothing to copy.  DEEP: a small load
    // is issued instead, so that the counted waits stay the same (nothing waits for it in particular); with two buffers no wait
    // counts what is not there.  (One asm statement: the branch stays inside it.)
    // (first_c: the first table, which always exists - no load then targets pf_sink while the compiler still computes addresses)
    auto dma = [&](int o, int step, int buf, auto first_c, uint32_t &sink) {
        constexpr bool FIRST = decltype(first_c)::value;
        const uint32_t chunk = DOPS == 4 ? ((uint32_t)(o * 16 + wave) + dma_rot) & 63u : (uint32_t)(o * 16 + wave);
        const uint32_t at = DOPS > 1 ? chunk * 1024u : (uint32_t)(wave * lanes_act) * 16u;
        const unsigned char *const src = dt + (size_t)(unsigned)step * table_bytes + at;
        const uint32_t to = lds_tbl + (uint32_t)buf * (DEEP ? BYTE_BUF / 2 : BYTE_BUF) + at;
        uint64_t save;
        const int ns = nsteps;              // (named here: asm operands inside the branches below do not capture)
#define BYTE_COPY_OP "s_mov_b64 %[sv], exec\n\ts_mov_b64 exec, %[mk]\n\ts_mov_b32 m0, %[to]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[vo], %[sa]\n\ts_mov_b64 exec, %[sv]\n\t"
        if constexpr (FIRST)
            asm volatile(BYTE_COPY_OP : [sv] "=&s"(save) : [vo] "v"(dma_voff), [mk] "s"(dma_mask), [sa] "s"(src), [to] "s"(to) : "memory");
        else if constexpr (DEEP)
            asm volatile("s_cmp_lt_i32 %[st], %[ns]\n\ts_cbranch_scc0 .Lbyte_none%=\n\t" BYTE_COPY_OP
                         "s_branch .Lbyte_done%=\n.Lbyte_none%=:\n\tglobal_load_dword %[sk], %[vo], %[tb]\n.Lbyte_done%=:"
                         : [sv] "=&s"(save), [sk] "+v"(sink)
                         : [vo] "v"(dma_voff), [tb] "s"(dt), [mk] "s"(dma_mask), [st] "s"(step), [ns] "s"(ns), [sa] "s"(src), [to] "s"(to)
                         : "memory", "scc");
        else
            asm volatile("s_cmp_lt_i32 %[st], %[ns]\n\ts_cbranch_scc0 .Lbyte_done%=\n\t" BYTE_COPY_OP ".Lbyte_done%=:"
                         : [sv] "=&s"(save)
                         : [vo] "v"(dma_voff), [mk] "s"(dma_mask), [st] "s"(step), [ns] "s"(ns), [sa] "s"(src), [to] "s"(to)
                         : "memory", "scc");
#undef BYTE_COPY_OP
    };
    auto dma_all = [&](int step, int buf, auto first_c, uint32_t &sink) {
#pragma unroll
        for (int o = 0; o < DOPS; ++o) dma(o, step, buf, first_c, sink);
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
    dma_all(0, 0, std::true_type{}, pf_sink);
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
    auto load_acts = [&](int i, run_t (&w)[NRUN], uint32_t off) {
        const int8_t *const from = xt;
        const uint32_t at = base[i] + off;
        if constexpr (V == 4) asm volatile("global_load_dwordx4 %[v], %[b], %[xr]" : [v] "+v"(w[i]) : [b] "v"(at), [xr] "s"(from));
        else asm volatile("global_load_dwordx2 %[v], %[b], %[xr]" : [v] "+v"(w[i]) : [b] "v"(at), [xr] "s"(from));
    };

    bi32x4_t acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = bi32x4_t{0, 0, 0, 0};
    run_t W[4][NRUN];                       // activation words of the four steps of a group
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int i = 0; i < NRUN; ++i) W[k][i] = run_t{};
    b32x4_t rv[2][2];
    bi32x2_t wa[2] = {{0, 0}, {0, 0}};      // A operands of the exact products of steps 0 and 1, 2 and 3 of a group

    // Address pieces.  Column word for read t in buffer u: byte 0 = slot * 16, byte 2 = buffer.  Selector: result byte 0 =
    // column byte 0, byte 1 = activation byte e, byte 2 = column byte 2, byte 3 = 0 (bytes of the first source of
    // v_perm_b32 are numbered 4..7, those of the second 0..3, 0x0c gives zero).
    // (DEEP: buffers 2 u and 2 u + 1 share a column word, the odd one is a constant offset of 32 KB away.  The words are those of the
    // step at hand: flipped in place, two sets of them would not fit the registers.)
    uint32_t colw[4], sel[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const uint32_t e = (uint32_t)((t + rl) & 3);
        sel[t] = 0x0c020000u | ((4u + e) << 8);
        colw[t] = ((4u * (uint32_t)g + e) << 4) | (lds_tbl >> 16) << 16;
    }
    const bi32x4_t ones = byte_ones(lane);
    const uint32_t ones_index = byte_ones_index(lane);
    const uint32_t wx_voff = (uint32_t)((q >> 1) * (BYTE_TILE * BYTE_STEP) + rl * BYTE_STEP + (q & 1) * 8);
    const bool bit3 = rl & 8;

    // The exact product of two steps, of whose words the lane holds first and second, into accumulator j (see the head of this file).
    auto exact = [&](uint32_t first, uint32_t second, const bi32x2_t &weights, int j) {
        auto s = __builtin_amdgcn_permlane32_swap(first, second, false, false);
        bi32x2_t b;
        b.x = (int)(bit3 ? s[1] : s[0]);
        b.y = (int)(bit3 ? s[0] : s[1]);
        if constexpr (LEVEL == 4) {
            b.x = (int)((uint32_t)b.x << p.shift) & (int)p.amask;       // (what crosses into the next byte falls to bits that am clears)
            b.y = (int)((uint32_t)b.y << p.shift) & (int)p.amask;
        }
        byte_exact(acc[j], weights, b);
    };

    // one step's reads, in pairs: reads 0 and 1 of the R pixels, then reads 2 and 3; two pairs in flight; between(m): what is issued
    // behind pair m
    auto run_step = [&](auto bc, const run_t (&w)[NRUN], auto &&between) {
        constexpr int buf = decltype(bc)::value, off = DEEP && (buf & 1) ? BYTE_BUF / 2 : 0;
        uint32_t word[R];
#pragma unroll
        for (int i = 0; i < R; ++i) word[i] = DEEP ? w[i / V][i % V] & line_mask : w[i / V][i % V];
        auto fetch = [&](int m) {
#pragma unroll
            for (int t = 0; t < 2; ++t) byte_fetch<off>(rv[m & 1][t], word[m % R], colw[m / R * 2 + t], sel[m / R * 2 + t]);
        };
        fetch(0);
        fetch(1);
#pragma unroll
        for (int m = 0; m < NPAIR - 2; ++m) {
            byte_add<2>(acc[m % NACC], rv[m & 1][0], rv[m & 1][1], ones, ones_index);
            fetch(m + 2);
            between(m);
        }
        byte_add<2>(acc[(NPAIR - 2) % NACC], rv[0][0], rv[0][1], ones, ones_index);
        between(NPAIR - 2);
        byte_add<0>(acc[(NPAIR - 1) % NACC], rv[1][0], rv[1][1], ones, ones_index);
        between(NPAIR - 1);
    };

    // Step k of a group, step s of the slice.  A wave's memory operations retire in order, which is what the counted waits
    // rely on.  Per step it issues
    //   DEEP:      NL activation loads of the next step, (k even) the weights of this step and the next, DOPS copy operations of the
    //              table three steps ahead.  Waiting for a step's activations then means that the next table has landed
    //              too and leaves the two after it in flight; the step ends with a barrier alone.
    //   two bufs:  DOPS copy operations of the next table, NL loads, (k even) the weights.  The step ends when this wave's
    //              part of the copy has landed; the newer loads stay in flight across the barrier.
    // All of it is spread over the step's reads: issued in one go ahead of them, it kept the last waves from their reads for
    // half of the step (32 KB tables, 8 pixels per row slot: 2200 of 4000 clocks).  The exact product of two steps goes between the
    // reads of the step behind them.
    // AT_ONCE (two pixels per row slot, tables of 16 KB and less, one row tile, so that every table is read once): what is issued late in a step is waited
    // for a step and a third later, and with steps this short a stream of tables from memory had too little in flight.  Issued ahead of
    // the wait for the step's own words it has two steps.  Linear layers of 6 bits: 3000 x 3000, 128 and 256 rows 124 and 136 -> 110 and 118 us; 4096 x 4096,
    // 256 rows 207 -> 200.  With several row tiles or tables of 32 KB enough is in flight, and spread is the faster one
    // (128 images of 8 x 8, 64 -> 64 channels: 17.6 us, 18.4 at once).
    uint32_t gv = 0;                        // group offset of the next step
    uint32_t gaddr = (uint32_t)(uintptr_t)(lds_ptr_t)goff + (uint32_t)g * 4u + 32u;         // that of the step after it
    auto step = [&](auto kc, int s) {
        constexpr int k = decltype(kc)::value;
        constexpr int NW = k % 2 == 0 ? 1 : 0;              // loads of weights
        constexpr int EV = NL + NW + DOPS;                  // operations of a step,
        constexpr int FIRST_LOAD = DEEP ? 0 : DOPS;         // of which these come first: the loads, or the copies
        auto issue = [&](int j) {
            const int l = j - FIRST_LOAD;
            if (l >= 0 && l < NL) {
                load_acts(l, W[(k + 1) & 3], gv);
                if (l == NL - 1) {
                    byte_lds_word(gv, gaddr);
                    gaddr += 16u;
                }
            } else if (NW && l == NL) {
                byte_load_weights(wa[k / 2], wx_voff, wx + (size_t)(unsigned)s * (BYTE_TILE * BYTE_STEP));
            } else {
                dma(DEEP ? j - NL - NW : j, s + AHEAD, DEEP ? (k + AHEAD) & 3 : (k + 1) & 1, std::false_type{}, pf_sink);
            }
        };
        if constexpr (AT_ONCE) {
#pragma unroll
            for (int j = 0; j < EV; ++j) issue(j);
        }
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"(DEEP ? DOPS + (AT_ONCE ? EV : 0) : 0) : "memory");
#pragma unroll
        for (int i = 0; i < NRUN; ++i) asm volatile("" : "+v"(W[k][i]));
        if constexpr (k % 2 == 0) asm volatile("" : "+v"(wa[k == 0 ? 1 : 0]));
        asm volatile("s_setprio 3");
        run_step(std::integral_constant<int, DEEP ? k : (k & 1)>{}, W[k], [&](int m) {
            if (m == NPAIR / 4 - 1) asm volatile("s_setprio 2");
            if (m == NPAIR / 2 - 1) asm volatile("s_setprio 1");
            if (m == NPAIR * 3 / 4 - 1) asm volatile("s_setprio 0");
#pragma unroll
            for (int j = 0; j < EV; ++j)
                if (!AT_ONCE && m == j * (DEEP ? NPAIR - 1 : NPAIR * 3 / 4) / EV) issue(j);
            // (into accumulators that the pairs around do not use)
            if constexpr (k % 2 == 0) {
                constexpr int from = k == 0 ? 2 : 0;
                const int j = (m + NACC / 2) % NACC, i = j % R;
                if (m % 2 == (m >= R ? 1 : 0)) exact(W[from][i / V][i % V], W[from + 1][i / V][i % V], wa[from / 2], j);
            }
        });
        if constexpr (!DEEP || k % 2 == 1) {
#pragma unroll
            for (int t = 0; t < 4; ++t) asm volatile("v_xor_b32 %0, 0x10000, %0" : "+v"(colw[t]));
        }
        if constexpr (DEEP) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : [g] "+v"(gv) : : "memory");
        else asm volatile("s_waitcnt vmcnt(%[nx]) lgkmcnt(0)\n\ts_barrier" : [g] "+v"(gv) : [nx] "n"(NL + NW) : "memory");
    };
    using std::integral_constant;

    // Border terms of the tile's 16 channels by class of the position: what the taps without an input there have added.  Read one by one
    // in the epilogue, a lane's terms were up to 32 loads behind each other: 28000 - 44000 clocks of a workgroup with short
    // rows.  (Their loads travel beside the first table's copy.)
    if (LEVEL >= 2 && p.edge_cols) {
        const int ec = p.edge_cols, Ty = (p.edge_rows + 1) >> 1, Tx = (ec + 1) >> 1, st = (int)p.cv_s.d;
        const int ry = (int)((uint32_t)(pick4(p.oy0, ph) + p.cv_pad) - p.cv_s.div((uint32_t)(pick4(p.oy0, ph) + p.cv_pad)) * p.cv_s.d);
        const int rx = (int)((uint32_t)(pick4(p.ox0, ph) + p.cv_pad) - p.cv_s.div((uint32_t)(pick4(p.ox0, ph) + p.cv_pad)) * p.cv_s.d);
        for (int i = tid; i < p.edge_rows * ec * BYTE_TILE; i += BYTE_THREADS) {
            const int cls = i / BYTE_TILE, cy = cls / ec, cx = cls - cy * ec;
            const int32_t *const z = p.zsum + (size_t)min(nt * BYTE_TILE + i % BYTE_TILE, p.N - 1) * p.cv_kh * p.cv_kw;
            uint32_t sum = 0;
            for (int m = 0; m < Ty; ++m)
                for (int n = 0; n < Tx; ++n)
                    if (byte_edge_missing(cy, m, Ty) || byte_edge_missing(cx, n, Tx)) sum += (uint32_t)z[(ry + st * m) * p.cv_kw + rx + st * n];
            goff[BYTE_GOFF - p.edge_rows * ec * BYTE_TILE + i] = sum;
        }
    }

    // prologue: offsets, table and activations of the first step; DEEP: the next two tables are on their way
    {
        const uint32_t off = group_off(s_begin * 4 + g);
#pragma unroll
        for (int i = 0; i < NRUN; ++i) load_acts(i, W[0], off);
    }
    if constexpr (DEEP) {
        dma_all(1, 1, std::false_type{}, pf_sink);
        dma_all(2, 2, std::false_type{}, pf_sink);
    }
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(DEEP ? 2 * DOPS : 0) : "memory");
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
        // the exact product of the last one or two steps (of one: no weights for the step that does not exist)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < NRUN; ++i) asm volatile("" : "+v"(W[k][i]));
        asm volatile("" : "+v"(wa[0]));
        asm volatile("" : "+v"(wa[1]));
        const bool early = left == 1 || left == 2;
        bi32x2_t weights = early ? wa[0] : wa[1];
        if ((left & 1) && q >= 2) weights = bi32x2_t{0, 0};
#pragma unroll
        for (int i = 0; i < R; ++i)
            exact(early ? W[0][i / V][i % V] : W[2][i / V][i % V], early ? W[1][i / V][i % V] : W[3][i / V][i % V], weights, i);
        // the last matrix instructions have to leave the pipe before a vector instruction reads their registers (every
        // accumulator passes through an asm statement behind the waiting one, so that no read can be scheduled ahead of it)
        asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");
#pragma unroll
        for (int i = 0; i < NACC; ++i) asm volatile("" : "+v"(acc[i]));
    } else {                                // no row of this wave exists: it copies its part of the tables
        uint32_t sink = 0;
        for (int s = 0; s < nsteps; ++s) {
            dma_all(s + AHEAD, DEEP ? (s + AHEAD) & 3 : (s + 1) & 1, std::false_type{}, sink);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(DEEP ? 2 * DOPS : 0) : "memory");
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        asm volatile("" : : "v"(sink));
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");      // (for the counted loads of either branch)
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
    const uint4 *const edge = LEVEL >= 2 && pe.edge_cols ? reinterpret_cast<const uint4 *>(goff + BYTE_GOFF - pe.edge_rows * pe.edge_cols * BYTE_TILE) : nullptr;
    // At most four channels in the tile: a quarter of the lanes hold all of it.  With tanh (60 instructions a value) every lane takes a
    // quarter of its column's pixels instead, through the LDS of the tables: 3 channels of 64 x 64, 33000 -> 8000 clocks.
    if constexpr (LEVEL == 3 && R >= 4) {
        if (pe.N - nt * BYTE_TILE <= 4) {
            constexpr int P = R / 4;
            if (!live) return;
            uint4 *const col = tbl + rs * R;
            if (q == 0) {
#pragma unroll
                for (int i = 0; i < R; ++i) col[i] = make_uint4((uint32_t)acc[i].x, (uint32_t)acc[i].y, (uint32_t)acc[i].z, (uint32_t)acc[i].w);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");        // (written and read by the same wave)
            bi32x4_t mine[P];
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const uint4 t = col[q * P + i];
                mine[i] = bi32x4_t{(int)t.x, (int)t.y, (int)t.z, (int)t.w};
            }
            float sc0[4] = {pe.scale, pe.scale, pe.scale, pe.scale}, bi0[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (pe.scales) sc0[r] = pe.scales[min(nt * BYTE_TILE + r, pe.N - 1)];
                if (pe.bias) bi0[r] = pe.bias[min(nt * BYTE_TILE + r, pe.N - 1)];
            }
            byte_epilogue<R, LEVEL, true>(pe, mine, sc0, bi0, mt, rs, ph, nt * BYTE_TILE, edge, q * P);
            return;
        }
    }
    if (cb < pe.N) byte_epilogue<R, LEVEL, false>(pe, acc, sc, bi, mt, rs, ph, cb, edge, 0);
}

// ------------------------------------------------------------------------------------------------ packing

struct BytePack {
    const uint16_t *lut16;      // [a & mask][w & mask]
    const int8_t *w;
    uint4 *dt;
    int8_t *wx;
    int bits, shift, N, Cin, taps, cg, n_tiles, steps;      // operand bits; tables have 2^(bits - shift) lines
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
    const int cols = 1 << p.bits, mask = cols - 1, half = cols >> 1, row = cols + 4, lines = cols >> p.shift;
    const int first = blockIdx.y * BYTE_PACK_LINES, here = min(BYTE_PACK_LINES, lines - first);
    const int t0 = (int)blockIdx.x * p.per_wg, t1 = min(t0 + p.per_wg, p.tables);
    if (p.arrived && blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = tid; i < BYTE_MAX_TILES; i += 256) p.arrived[i] = 0u;
    for (int i = tid; i < here * cols; i += 256) {
        const int r = i >> p.bits, u = i & mask, l = (first + r) << p.shift;
        const int a = (l < half ? l : l - cols) & p.am, w = (u < half ? u : u - cols) & p.wm;
        band[r * row + u] = (uint8_t)((int)(int16_t)p.lut16[(size_t)l * cols + u] - a * w - p.c);
    }
    if (tid < here) band[tid * row + cols] = 0;                // column of weights that do not exist
    for (int tb = t0; tb < t1; ++tb) {
        const int tn = tb / p.steps, step = tb - tn * p.steps, nt = tn % p.n_tiles, phase = tn / p.n_tiles;
        uint16_t *const idx = index[(tb - t0) & 1];
        {
            const int slot = tid & 15, ch = tid >> 4;
            int tap, c;
            const int rest = p.cg & 3;
            byte_slot(step * 4 + (slot >> 2), p.taps, p.cg, [&](int v) { return v / p.taps; }, [&](int v) { return v / rest; }, &tap, &c);
            const int n = nt * BYTE_TILE + ch, ci = c * 4 + (slot & 3);
            int u = cols;
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
            if (blockIdx.y == 0) p.wx[(size_t)tb * (BYTE_TILE * BYTE_STEP) + ch * BYTE_STEP + byte_wx_pos(slot)] = (int8_t)(u == cols ? 0 : (u < half ? u : u - cols) & p.wm);
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
