// Backward pass of an approximate linear layer under the straight-through estimator (Sec. III-A, "Retraining"):
// the quantiser passes a gradient where its clamp did not act, the multiplier table is differentiated as the exact
// product.  Both gradients are dense fp32 contractions with one fake-quantised operand,
//
//     dx[m][k] = inside(x[m][k]) * sum_n dy[m][n] * w^[n][k]          w^ = s_w * q(w)
//     dw[n][k] = inside(w[n][k]) * sum_m dy[m][n] * x^[m][k]          x^ = s_x * q(x)
//
// so this is the one part of the library that belongs on the matrix pipe as a plain product: v_mfma_f32_32x32x2_f32,
// operands staged through LDS, the fake quantisation applied while a tile is staged and the clip mask in the epilogue
// (no quantised copy of x or w is ever written to memory).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "elementwise.hpp"

namespace adapt {

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int STE_TR = 32;          // contraction indices per staged chunk
constexpr int STE_THREADS = 256;    // four waves, 2 x 2 over the workgroup's output tile (x KS, see the kernel)

// geometry of a convolution whose unfolded input takes part in a product (see the end of this file)
struct SteConvGeo {
    int N, C, H, W, O, kh, kw, sh, sw, ph, pw, dh, dw, Ho, Wo;
    FastDiv dkw, dWo, dHoWo, dC, dCp, dW, dHW, dsh, dsw;     // the divisors of the index decodes below (Cp: C rounded up to 4)
};

// n / f.d: multiply-and-shift for 32-bit indices (exact below 2^31), a plain division otherwise
template <typename Idx>
__device__ __forceinline__ Idx ste_div(Idx n, const FastDiv &f) {
    if constexpr (sizeof(Idx) == 4) return (Idx)f.div((uint32_t)n);
    else return n / (Idx)f.d;
}

// c[i][j] = inside(o[i][j]) * sum_r A(i, r) * fq(b[r][j])
struct SteParams {
    const float *a;     // A_T: element (i, r) at a[r * lda + i]; else at a[i * lda + r]
    const float *b;     // [R][J], fake-quantised with scale sb while it is staged
    const float *o;     // [I][J], decides the clip mask with scale so; nullptr: no mask
    float *c;           // [I][J]
    int I, J, R, lda;
    float sb, so, Q;
    int cps;            // chunks of STE_TR contraction indices per grid z: z > 0 writes its partial sums to c + z * I * J
    int im2col;         // b is the channel-last copy of an image tensor (already fake-quantised) and stands for its unfolded
    SteConvGeo g;       //   matrix: b[r][j] = x(n, oy s - p + ky d, ..., c) with r = (n, oy, ox), j = (ky, kx, c), zero outside the image
};

__device__ __forceinline__ float ste_fake_quant(float x, float s, float Q) {
    float r = rintf(x / s);         // IEEE divide, round half to even: the forward quantiser's decision
    if (r != r) r = 0.0f;
    if (r > Q) r = Q;
    if (r < -Q) r = -Q;
    return r * s;
}

// the same code times a factor of its own
__device__ __forceinline__ float ste_fake_quant(float x, float s, float Q, float factor) {
    float r = rintf(x / s);
    if (r != r) r = 0.0f;
    if (r > Q) r = Q;
    if (r < -Q) r = -Q;
    return r * factor;
}

__device__ __forceinline__ bool ste_inside(float x, float s, float Q) { return fabsf(rintf(x / s)) <= Q; }     // NaN: false

// Four consecutive elements of a row-major matrix (col a multiple of 4).  FULL: the whole tile lies inside the matrix
// and rows are 16-byte aligned, one load.  Otherwise: zero outside the matrix, read without a branch from clamped
// addresses (rows, cols >= 1), so that the loads of a chunk stay in flight together.
template <bool FULL>
__device__ __forceinline__ float4 ste_load4(const float *__restrict__ base, int row, int col, int rows, int cols, int ld) {
    if (FULL) return *reinterpret_cast<const float4 *>(base + (size_t)row * (size_t)ld + (size_t)col);
    const float *q = base + (size_t)min(row, rows - 1) * (size_t)ld;
    const bool in_row = row < rows;
    float4 v;
    v.x = q[min(col + 0, cols - 1)];
    v.y = q[min(col + 1, cols - 1)];
    v.z = q[min(col + 2, cols - 1)];
    v.w = q[min(col + 3, cols - 1)];
    v.x = (in_row && col + 0 < cols) ? v.x : 0.0f;
    v.y = (in_row && col + 1 < cols) ? v.y : 0.0f;
    v.z = (in_row && col + 2 < cols) ? v.z : 0.0f;
    v.w = (in_row && col + 3 < cols) ? v.w : 0.0f;
    return v;
}

// Four consecutive elements of a row of the unfolded input of a convolution (row = (n, oy, ox), col = (ky, kx, c), a multiple of
// 4) from the fake-quantised, channel-last copy xq [N][H][W][Cp] (ste_channels_last_kernel): one 16-byte load, no unfolded
// copy exists.  Elements outside the image are to be zero: `inside` says so, and is applied when the value is stored (applied here,
// every load would be waited for before the matrix instructions of the chunk).  Rows beyond the matrix are read from its last row (the other operand is
// zero there), columns beyond it from its last ones (never stored).
__device__ __forceinline__ float4 ste_load4_unfolded(const float *__restrict__ xq, int row, int col, int rows, int cols, const SteConvGeo &g, uint32_t &inside) {
    const uint32_t m = (uint32_t)min(row, rows - 1);
    const uint32_t n = g.dHoWo.div(m), pix = m - n * (uint32_t)(g.Ho * g.Wo);
    const int oy = (int)g.dWo.div(pix), ox = (int)pix - oy * g.Wo;
    const uint32_t k = (uint32_t)min(col, cols - 4);
    const uint32_t tap = g.dCp.div(k), c = k - tap * g.dCp.d;
    const int ky = (int)g.dkw.div(tap), kx = (int)tap - ky * g.kw;
    const int iy = oy * g.sh - g.ph + ky * g.dh, ix = ox * g.sw - g.pw + kx * g.dw;
    const bool ok = iy >= 0 && iy < g.H && ix >= 0 && ix < g.W;
    const size_t at = ok ? (((size_t)n * g.H + iy) * g.W + ix) * g.dCp.d + c : 0;
    inside = ok ? ~0u : 0u;
    return *reinterpret_cast<const float4 *>(xq + at);
}

// TILE x TILE outputs per workgroup (128: four 32 x 32 blocks per wave; 64: one), FULL as above.  Chunks of 32
// contraction indices alternate between two LDS buffers: while the matrix pipe works on one, the next chunk's global
// loads are in flight and are fake-quantised into the other; one barrier per chunk.
// KS = 2: eight waves; waves w and w + 4 share an output quarter and take alternate pairs of contraction indices, their
// sums are added through LDS at the end (a fixed order).  For launches with about one workgroup per compute unit:
// two waves per SIMD, so that one wave's staging arithmetic runs under the other's matrix instructions.
// UNFOLD: b is a copy of an image tensor that stands for its unfolded matrix (p.im2col; a template parameter so that the plain
// products carry no trace of it: a run-time branch around the loads cost them 10 - 30 %).
template <bool A_T, int TILE, bool FULL, int KS, bool UNFOLD = false>
__global__ __launch_bounds__(STE_THREADS * KS) void ste_gemm_kernel(SteParams p) {
    constexpr int THREADS = STE_THREADS * KS;
    constexpr int LDB = TILE + 4;                   // LDS row length in floats: 16-byte rows, shifted by 4 banks per row
    constexpr int LDA = A_T ? TILE + 4 : TILE + 1;  // written element by element when the tile arrives transposed
    constexpr int PASSES = TILE * STE_TR / 4 / THREADS;     // staging passes of THREADS x 4 floats over a 32 x TILE chunk
    constexpr int TPR = TILE / 4;                   // threads per staged row
    constexpr int RPP = THREADS / TPR;              // rows per pass
    constexpr int IPP = THREADS / 8;                // rows of a transposed tile per pass
    constexpr int WT = TILE / 2, NB = WT / 32;
    __shared__ __align__(16) float As[2][STE_TR][LDA];      // [r][i]
    __shared__ __align__(16) float Bs[2][STE_TR][LDB];      // [r][j]
    const int tid = threadIdx.x, lane = tid & 63, wave = (tid >> 6) & 3, kh = tid >> 8;
    const int i0 = blockIdx.y * TILE, j0 = blockIdx.x * TILE;
    const int wi = (wave & 1) * WT, wj = (wave >> 1) * WT;

    f32x16_t acc[NB][NB];
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[bi][bj][v] = 0.0f;

    float4 ra[PASSES], rb[PASSES];
    uint32_t in_image[UNFOLD ? PASSES : 1];
    auto fetch = [&](int r0) {
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const int r = tid / TPR + RPP * pass, c4 = (tid % TPR) * 4;
            if constexpr (UNFOLD) rb[pass] = ste_load4_unfolded(p.b, r0 + r, j0 + c4, p.R, p.J, p.g, in_image[pass]);
            else rb[pass] = ste_load4<FULL>(p.b, r0 + r, j0 + c4, p.R, p.J, p.J);
            if (A_T) {
                ra[pass] = ste_load4<FULL>(p.a, r0 + r, i0 + c4, p.R, p.I, p.lda);
            } else {
                const int i = (tid >> 3) + IPP * pass, r4 = (tid & 7) * 4;
                ra[pass] = ste_load4<FULL>(p.a, i0 + i, r0 + r4, p.I, p.R, p.lda);
            }
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const int r = tid / TPR + RPP * pass, c4 = (tid % TPR) * 4;
            float4 q = rb[pass];
            if constexpr (UNFOLD) {
                q.x = __uint_as_float(__float_as_uint(q.x) & in_image[pass]);
                q.y = __uint_as_float(__float_as_uint(q.y) & in_image[pass]);
                q.z = __uint_as_float(__float_as_uint(q.z) & in_image[pass]);
                q.w = __uint_as_float(__float_as_uint(q.w) & in_image[pass]);
            } else {
                q.x = ste_fake_quant(rb[pass].x, p.sb, p.Q);
                q.y = ste_fake_quant(rb[pass].y, p.sb, p.Q);
                q.z = ste_fake_quant(rb[pass].z, p.sb, p.Q);
                q.w = ste_fake_quant(rb[pass].w, p.sb, p.Q);
            }
            *reinterpret_cast<float4 *>(&Bs[buf][r][c4]) = q;
            if (A_T) {
                *reinterpret_cast<float4 *>(&As[buf][r][c4]) = ra[pass];
            } else {                                        // the tile arrives with r contiguous: transposed on the way in
                const int i = (tid >> 3) + IPP * pass, r4 = (tid & 7) * 4;
                As[buf][r4 + 0][i] = ra[pass].x;
                As[buf][r4 + 1][i] = ra[pass].y;
                As[buf][r4 + 2][i] = ra[pass].z;
                As[buf][r4 + 3][i] = ra[pass].w;
            }
        }
    };

    // this workgroup's share of the contraction (only the products over an unfolded input are ever split over grid z)
    const int ch0 = UNFOLD ? blockIdx.z * p.cps : 0;
    const int chunks = UNFOLD ? max(0, min((p.R + STE_TR - 1) / STE_TR, ch0 + p.cps) - ch0) : (p.R + STE_TR - 1) / STE_TR;
    float *const cout = UNFOLD ? p.c + (size_t)blockIdx.z * (size_t)p.I * (size_t)p.J : p.c;
    if (chunks > 0) { fetch(ch0 * STE_TR); stash(0); }
    __syncthreads();
    for (int ch = 0; ch < chunks; ++ch) {
        const int cur = ch & 1;
        const bool more = ch + 1 < chunks;
        if (more) fetch((ch0 + ch + 1) * STE_TR);
        // one instruction: lane l supplies A(i = l % 32, k = l / 32) and B(k = l / 32, j = l % 32)
        const int kr = lane >> 5, c = lane & 31;
        // all operands of the chunk are requested before its first matrix instruction: one LDS latency per chunk
        float av[STE_TR / 2 / KS][NB], bv[STE_TR / 2 / KS][NB];
#pragma unroll
        for (int k2 = 0; k2 < STE_TR / 2 / KS; ++k2)
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                av[k2][q] = As[cur][2 * (KS * k2 + kh) + kr][wi + 32 * q + c];
                bv[k2][q] = Bs[cur][2 * (KS * k2 + kh) + kr][wj + 32 * q + c];
            }
        __builtin_amdgcn_sched_barrier(0);          // (the scheduler would otherwise sink each read to its use)
#pragma unroll
        for (int k2 = 0; k2 < STE_TR / 2 / KS; ++k2)
#pragma unroll
            for (int bi = 0; bi < NB; ++bi)
#pragma unroll
                for (int bj = 0; bj < NB; ++bj)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[k2][bi], bv[k2][bj], acc[bi][bj], 0, 0, 0);
        if (more) stash(cur ^ 1);           // the other buffer: every wave left it before the previous barrier
        __syncthreads();
    }

    if (KS == 2) {          // (the loop ended with a barrier: the staging buffers are free, but this has its own)
        __shared__ float red[KS == 2 ? 4 * NB * NB * 16 * 64 : 1];
        if (kh == 1) {
#pragma unroll
            for (int bi = 0; bi < NB; ++bi)
#pragma unroll
                for (int bj = 0; bj < NB; ++bj)
#pragma unroll
                    for (int v = 0; v < 16; ++v) red[((wave * NB * NB + bi * NB + bj) * 16 + v) * 64 + lane] = acc[bi][bj][v];
        }
        __syncthreads();
        if (kh == 1) return;
#pragma unroll
        for (int bi = 0; bi < NB; ++bi)
#pragma unroll
            for (int bj = 0; bj < NB; ++bj)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[bi][bj][v] += red[((wave * NB * NB + bi * NB + bj) * 16 + v) * 64 + lane];
    }

    // register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of a 32 x 32 block
#pragma unroll
    for (int bi = 0; bi < NB; ++bi) {
#pragma unroll
        for (int bj = 0; bj < NB; ++bj) {
            const int j = j0 + wj + 32 * bj + (lane & 31);
            float ov[16];                   // the mask's operand first, all 16 requests together (c and o never overlap)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = i0 + wi + 32 * bi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                ov[v] = (p.o && (FULL || (i < p.I && j < p.J))) ? p.o[(size_t)i * (size_t)p.J + (size_t)j] : 0.0f;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = i0 + wi + 32 * bi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (FULL || (i < p.I && j < p.J))
                    cout[(size_t)i * (size_t)p.J + (size_t)j] = (!p.o || ste_inside(ov[v], p.so, p.Q)) ? acc[bi][bj][v] : 0.0f;
            }
        }
    }
}

// c[i] = inside(o[i]) * (part[0][i] + part[1][i] + ... + part[S-1][i]), in that order: the partial sums of a product whose
// contraction was split over grid z.  Eight parts are requested together (one at a time, 57 parts of 36864 took 15.5 us, the
// latency of memory 57 times over; now 5.4 us).
// taps > 0: the parts are rows of (tap, channel), taps x Cp columns, and c, o the weight tensor [row][C][all_taps], of which these
// are taps tap0 .. tap0 + taps - 1.  scale: of the sums.
__global__ __launch_bounds__(256) void ste_reduce_masked_kernel(const float *__restrict__ part, int S, size_t n, const float *__restrict__ o,
                                                                float so, float Q, float *__restrict__ c, int taps, int C, int Cp, int tap0, int all_taps, float scale) {
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
        float s = part[i];
        int z = 1;
        for (; z + 8 <= S; z += 8) {
            float t[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) t[q] = part[(size_t)(z + q) * n + i];
#pragma unroll
            for (int q = 0; q < 8; ++q) s += t[q];
        }
        for (; z < S; ++z) s += part[(size_t)z * n + i];
        size_t at = i;
        if (taps > 0) {
            const size_t row = i / ((size_t)taps * Cp), rem = i - row * (size_t)taps * Cp;
            const int tap = (int)(rem / Cp), ch = (int)(rem - (size_t)tap * Cp);
            if (ch >= C) continue;
            at = (row * C + ch) * (size_t)all_taps + tap0 + tap;
        }
        c[at] = (!o || ste_inside(o[at], so, Q)) ? s * scale : 0.0f;
    }
}

// part[z][o] = sum over the images n = z, z + Z, ... and all pixels of dy[n][o][pix] from the NCHW tensor (grid: O x Z
// workgroups; every thread a strided share in ascending order, then a fixed tree); ste_reduce_masked_kernel adds the Z parts
__global__ __launch_bounds__(256) void ste_bias_grad_nchw_kernel(const float *__restrict__ dy, float *__restrict__ db, int N, int O, int P) {
    __shared__ float part[256];
    const int o = blockIdx.x;
    float s = 0.0f;
    for (int n = blockIdx.y; n < N; n += gridDim.y) {
        const float *q = dy + ((size_t)n * O + o) * (size_t)P;
        for (int e = threadIdx.x; e < P; e += 256) s += q[e];
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) db[(size_t)blockIdx.y * O + o] = part[0];
}

// db[n] = sum_m dy[m][n]: 32 columns per workgroup, 32 threads per column take every 32nd row with four running sums
// each; fixed order, so the result does not depend on the launch
constexpr int STE_COLSUM_THREADS = 1024;
__global__ __launch_bounds__(STE_COLSUM_THREADS) void ste_colsum_kernel(const float *__restrict__ dy, float *__restrict__ db, int M, int N) {
    __shared__ float part[32][33];
    const int c = threadIdx.x & 31, ph = threadIdx.x >> 5;
    const int n = blockIdx.x * 32 + c;
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
    if (n < N) {
        const float *q = dy + n;
        int m = ph;
        for (; m + 96 < M; m += 128) {
            s0 += q[(size_t)m * (size_t)N];
            s1 += q[(size_t)(m + 32) * (size_t)N];
            s2 += q[(size_t)(m + 64) * (size_t)N];
            s3 += q[(size_t)(m + 96) * (size_t)N];
        }
        for (; m < M; m += 32) s0 += q[(size_t)m * (size_t)N];
    }
    part[ph][c] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (ph == 0 && n < N) {
        float t = part[0][c];
#pragma unroll
        for (int q = 1; q < 32; ++q) t += part[q][c];
        db[n] = t;
    }
}

// ---- convolution (groups = 1): the same two products over the unfolded input --------------------------------------
// y[m][o] = sum_k col(x^)[m][k] * w^[o][k] with m = (n, oy, ox), k = (c, ky, kx) (Sec. III-B: the convolution as a matrix
// product over the unfolded input), so dw = mask(w) . dy_rows^T . col(x^) and dx gathers dy . w^ over the taps that reach a
// pixel (a fixed order) under mask(x).  col(x) is never written: the product reads it from a fake-quantised channel-last copy
// of x (ste_load4_unfolded).  Stride 1: dx is one product whose operand is read from dy itself (ste_dx_kernel); other strides:
// dcol = dy_rows . fq(w), then ste_col2im_kernel.

// src [N][C][P] -> dst [N][P][ld] (zeros in channels C .. ld - 1), fake-quantised with (s, Q) if s > 0.  64 channels x 32
// pixels go through LDS so that reads and writes coalesce (without it: 8.4 MB in 14 us, now 5 us).
__global__ __launch_bounds__(256) void ste_channels_last_kernel(const float *__restrict__ src, float *__restrict__ dst, int N, int C, int P, int ld, float s, float Q) {
    __shared__ float tile[64][33];
    const int c0 = blockIdx.y * 64, tid = threadIdx.x, blocks = (int)((P + 31LL) / 32);
    // (planes beyond the grid: a launch is limited to 2^32 threads)
    for (int n = blockIdx.z, b = blockIdx.x; n < N; b += gridDim.x) {
        if (b >= blocks) {
            b = (int)blockIdx.x - (int)gridDim.x;
            n += gridDim.z;
            continue;
        }
        const int p0 = b * 32;
        const int pl = tid & 31, cl = tid >> 5;
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = c0 + cl + 8 * q;
            const bool ok = c < C && p0 + pl < P;
            const float t = src[ok ? ((size_t)n * C + c) * (size_t)P + (size_t)(p0 + pl) : 0];
            v[q] = ok ? t : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) tile[cl + 8 * q][pl] = s > 0.0f ? ste_fake_quant(v[q], s, Q) : v[q];
        __syncthreads();
        const int wc = tid & 63, wp = tid >> 6;
        if (c0 + wc < ld) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int pp = wp + 4 * q;
                if (p0 + pp < P) dst[((size_t)n * P + (size_t)(p0 + pp)) * (size_t)ld + (size_t)(c0 + wc)] = tile[wc][pp];
            }
        }
        __syncthreads();
    }
}

// w [O][C][T] -> wp [O][T][C] (T = kh kw taps): with the channel last in dcol's columns, the lanes of the gather kernel
// below, which run along channels, read consecutive floats
__global__ __launch_bounds__(256) void ste_taps_first_kernel(const float *__restrict__ w, float *__restrict__ wp, int O, int C, int T) {
    const size_t total = (size_t)O * C * T, stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
        const size_t o = i / ((size_t)C * T), rem = i - o * (size_t)C * T, t = rem / C, c = rem - t * C;
        wp[i] = w[(o * C + c) * T + t];
    }
}

// w [O][C][T] -> wq [T][O][Cp], fake-quantised, zeros in the padded channels: the other operand of ste_dx_kernel
__global__ __launch_bounds__(256) void ste_weights_by_tap_kernel(const float *__restrict__ w, float *__restrict__ wq, int O, int C, int Cp, int T, float s, float Q) {
    const size_t total = (size_t)T * O * Cp, stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
        const size_t t = i / ((size_t)O * Cp), rem = i - t * (size_t)O * Cp, o = rem / Cp, c = rem - o * Cp;
        wq[i] = c < (size_t)C ? ste_fake_quant(w[(o * C + c) * T + t], s, Q) : 0.0f;
    }
}

struct SteDxParams {
    const float *dy, *wq, *x;   // [N][O][Ho Wo], [tap][O][Cp], [N][C][H W]
    float *dx;
    int pixels, Cp;             // N H W
    float so, Q;
    SteConvGeo g;
};

// dx of a convolution with stride 1: dx[n][c][iy][ix] = inside(x) * sum over taps (ky, kx ascending) of sum over o of
// w^[o][c][tap] dy[n][o][iy + ph - ky dh][ix + pw - kx dw].  A workgroup owns 64 channels x 64 pixels; chunks of 32 output
// channels of a tap go through two LDS buffers (lanes along pixels: 256-byte loads from dy), a wave multiplies a 32 x 32 block.
// The sum of a tap is finished before it is added, the order of the dcol form: same rounding, same results.  Against that
// form (product 43 us, 75 MB written and read again by a gather of 39 us, 64 -> 64 channels, 3 x 3, 32 images of 32 x 32, fp32):
// 40 us.  Bounded by the matrix pipe (fp32: 2.4 GFLOP, 15 us) and the latency of a chunk.
__global__ __launch_bounds__(STE_THREADS, 2) void ste_dx_kernel(const SteDxParams p) {
    constexpr int LD = 96;                                  // rows 2 k and 2 k + 1 of a read lie in different halves of the banks
    __shared__ __align__(16) float As[2][STE_TR][LD];       // [o][c]
    __shared__ __align__(16) float Bs[2][STE_TR][LD];       // [o][pixel]
    const SteConvGeo &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    const int wi = (wave & 1) * 32, wj = (wave >> 1) * 32;
    const int P = g.Ho * g.Wo, HW = g.H * g.W, taps = g.kh * g.kw;
    auto decode = [&](int j, int &n, int &pin) {
        n = (int)g.dHW.div((uint32_t)j);
        pin = j - n * HW;
    };
    // staging: this thread's pixel, and rows wave + 4 i of a chunk
    int sn, spin;
    decode(min(j0 + lane, p.pixels - 1), sn, spin);
    const int sy = (int)g.dW.div((uint32_t)spin), sx = spin - sy * g.W;
    const float *const dyn = p.dy + (size_t)sn * g.O * (size_t)P;
    const int ac = min(i0 + (tid & 15) * 4, p.Cp - 4);
    const int cpt = (g.O + STE_TR - 1) / STE_TR, chunks = taps * cpt;
    int ky = 0, kx = 0, tap = 0, part = 0;                  // of the chunk that is fetched next
    // What is fetched stays untouched until it is stored: zeros (outside the image, beyond the last channel) are put in by then.
    // (Selected right behind its load, every value was waited for before the matrix instructions of the chunk: 59 -> 40 us.)
    float rb[2][8];
    f32x4_t ra[2][2];
    uint32_t inside[2];
    int from_o[2];
    auto fetch = [&](float (&b)[8], f32x4_t (&a)[2], uint32_t &in, int &first_o) {
        const int oy = sy + g.ph - ky * g.dh, ox = sx + g.pw - kx * g.dw, o0 = part * STE_TR;
        const bool ok = oy >= 0 && oy < g.Ho && ox >= 0 && ox < g.Wo;
        const float *const from = dyn + (ok ? oy * g.Wo + ox : 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int o = o0 + wave + 4 * i;                // (the same in the whole wave)
            b[i] = from[(size_t)min(o, g.O - 1) * (size_t)P];
        }
        in = ok ? ~0u : 0u;
        first_o = o0;
        const float *const wt = p.wq + (size_t)tap * g.O * (size_t)p.Cp;
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const f32x4_t *>(wt + (size_t)min(o0 + (tid >> 4) + 16 * i, g.O - 1) * (size_t)p.Cp + ac);
        if (++part == cpt) {
            part = 0;
            ++tap;
            if (++kx == g.kw) {
                kx = 0;
                ++ky;
            }
        }
    };
    auto stash = [&](int buf, const float (&b)[8], const f32x4_t (&a)[2], uint32_t in, int first_o) {
#pragma unroll
        for (int i = 0; i < 8; ++i) Bs[buf][wave + 4 * i][lane] = __uint_as_float(__float_as_uint(b[i]) & (first_o + wave + 4 * i < g.O ? in : 0u));
#pragma unroll
        for (int i = 0; i < 2; ++i) *reinterpret_cast<f32x4_t *>(&As[buf][(tid >> 4) + 16 * i][(tid & 15) * 4]) = a[i];
    };
    f32x16_t acc, tot;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = tot[v] = 0.0f;
    int left = cpt;                 // chunks of this tap that are still to be multiplied
    // chunk ch lies in LDS buffer S = ch % 2 and was fetched into register set S; set 1 - S holds the next one (requested a chunk
    // ago), set S takes the one after it
    auto chunk = [&](int ch, auto set_c) {
        constexpr int S = decltype(set_c)::value;
        if (ch + 2 < chunks) fetch(rb[S], ra[S], inside[S], from_o[S]);
        const int kr = lane >> 5, c = lane & 31;
        float av[STE_TR / 2], bv[STE_TR / 2];
#pragma unroll
        for (int k2 = 0; k2 < STE_TR / 2; ++k2) {
            av[k2] = As[S][2 * k2 + kr][wi + c];
            bv[k2] = Bs[S][2 * k2 + kr][wj + c];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k2 = 0; k2 < STE_TR / 2; ++k2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[k2], bv[k2], acc, 0, 0, 0);
        if (ch + 1 < chunks) stash(1 - S, rb[1 - S], ra[1 - S], inside[1 - S], from_o[1 - S]);
        if (--left == 0) {
            left = cpt;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                tot[v] += acc[v];
                acc[v] = 0.0f;
            }
        }
        __syncthreads();
    };
    fetch(rb[0], ra[0], inside[0], from_o[0]);
    if (chunks > 1) fetch(rb[1], ra[1], inside[1], from_o[1]);
    stash(0, rb[0], ra[0], inside[0], from_o[0]);
    __syncthreads();
    for (int ch = 0; ch < chunks; ch += 2) {
        chunk(ch, std::integral_constant<int, 0>{});
        if (ch + 1 < chunks) chunk(ch + 1, std::integral_constant<int, 1>{});
    }
    const int j = j0 + wj + (lane & 31);
    if (j >= p.pixels) return;
    int n, pin;
    decode(j, n, pin);
    float xv[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = i0 + wi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        xv[v] = c < g.C ? p.x[((size_t)n * g.C + c) * (size_t)HW + (size_t)pin] : 0.0f;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = i0 + wi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (c < g.C) p.dx[((size_t)n * g.C + c) * (size_t)HW + (size_t)pin] = ste_inside(xv[v], p.so, p.Q) ? tot[v] : 0.0f;
    }
}

// ---- the same two products on 16-bit matrix instructions ----------------------------------------------------------
// Operands of up to 9 bits: a code is a bf16 number, so one operand of either product needs no more than that, and the gradient is
// the sum of three bf16 numbers (24 bits).  Every product of a piece and a code is exact in fp32, sums are fp32: nothing is
// rounded that the fp32 form does not round (there a fake-quantised value is rounded; here the sum is scaled once).  Each
// piece has an accumulator of its own: that of the first, which carries the sum, is rounded once for 16 products, and the others
// hold their piece times 2^8 and 2^16, about the size of the first.  (Unscaled, the third piece of a gradient below 2^-110 is
// subnormal and has fewer than eight bits: 2-norm of the error 5e-6 at 1e-35.)  Three bf16
// instructions replace eight fp32 ones of twice their length.  A code carries the power of two of its scale, so that products have
// the range they have in fp32 (but for the last binade: a scaled piece may be twice its number); what is left of the scale, in [1, 2), multiplies the sum.
// Error against 64 bits (2-norm of the difference over that of the result), fp32 form -> this one: weight gradient 1.8e-7 -> 1.4e-7, input
// gradient 1.2e-7 -> 7.3e-8 (64 -> 64 channels, 3 x 3, 8 images of 32 x 32); 13 other layers likewise or better.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// v = p[0] + 2^-8 p[1] + 2^-16 p[2], of whose words the upper halves count.  Exact for every v, subnormal ones included, and none of the
// three is larger than 2^(exponent of v + 1) (2^-123 where v is subnormal).  An infinity is the first piece alone; a NaN is one in the second piece, whatever is left of it in
// the first.
__device__ __forceinline__ void ste_split(float v, uint32_t (&p)[3]) {
    p[0] = __float_as_uint(v) & 0xffff0000u;
    const float r = fabsf(v) == __builtin_inff() ? 0.0f : (v - __uint_as_float(p[0])) * 0x1p8f;
    p[1] = __float_as_uint(r) & 0xffff0000u;
    p[2] = __float_as_uint((r - __uint_as_float(p[1])) * 0x1p8f);
}

// the value of three sums of such pieces
__device__ __forceinline__ float ste_join(float first, float second, float third) { return __builtin_fmaf(__builtin_fmaf(third, 0x1p-8f, second), 0x1p-8f, first); }

// upper halves of a and b as one word, a's in the lower half
__device__ __forceinline__ uint32_t ste_halves(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// the code of x with scale s, times pow2, as upper half of a word (exact)
__device__ __forceinline__ uint32_t ste_code16(float x, float s, float Q, float pow2) { return __float_as_uint(ste_fake_quant(x, s, Q, pow2)); }

// src [N][C][P] -> dst [N][P][ld] bf16 (zeros in channels C .. ld - 1): codes with (s, Q) times pow2 if s > 0, else three planes of pieces,
// `plane` elements apart.  The walk of ste_channels_last_kernel; a thread writes two channels at once (ld is a multiple of 4).
// rows: the values as they are too, [N][P][C], or nullptr (a launch of its own for them cost a layer with strides 2 us).
__global__ __launch_bounds__(256) void ste_channels_last16_kernel(const float *__restrict__ src, uint16_t *__restrict__ dst, int N, int C, int P, int ld, float s, float Q,
                                                                  float pow2, size_t plane, float *__restrict__ rows) {
    __shared__ float tile[64][33];
    const int c0 = blockIdx.y * 64, tid = threadIdx.x, blocks = (int)((P + 31LL) / 32);
    for (int n = blockIdx.z, b = blockIdx.x; n < N; b += gridDim.x) {
        if (b >= blocks) {
            b = (int)blockIdx.x - (int)gridDim.x;
            n += gridDim.z;
            continue;
        }
        const int p0 = b * 32;
        const int pl = tid & 31, cl = tid >> 5;
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = c0 + cl + 8 * q;
            const bool ok = c < C && p0 + pl < P;
            const float t = src[ok ? ((size_t)n * C + c) * (size_t)P + (size_t)(p0 + pl) : 0];
            v[q] = ok ? t : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) tile[cl + 8 * q][pl] = v[q];
        __syncthreads();
        const int wc = (tid & 31) * 2, wp = tid >> 5;
        if (c0 + wc < ld) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int pp = wp + 8 * q;
                if (p0 + pp < P) {
                    const float x0 = tile[wc][pp], x1 = tile[wc + 1][pp];
                    uint32_t *const to = reinterpret_cast<uint32_t *>(dst + ((size_t)n * P + (size_t)(p0 + pp)) * (size_t)ld + (size_t)(c0 + wc));
                    if (s > 0.0f) {
                        *to = ste_halves(ste_code16(x0, s, Q, pow2), ste_code16(x1, s, Q, pow2));
                    } else {
                        uint32_t a[3], d[3];
                        ste_split(x0, a);
                        ste_split(x1, d);
#pragma unroll
                        for (int i = 0; i < 3; ++i) to[i * (plane / 2)] = ste_halves(a[i], d[i]);
                    }
                }
            }
        }
        if (rows && c0 + (tid & 63) < C) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int pp = (tid >> 6) + 4 * q;
                if (p0 + pp < P) rows[((size_t)n * P + (size_t)(p0 + pp)) * (size_t)C + (size_t)(c0 + (tid & 63))] = tile[tid & 63][pp];
            }
        }
        __syncthreads();
    }
}

struct SteDwParams {
    const uint16_t *a;          // [piece][R][lda] bf16, pieces `plane` elements apart
    const uint16_t *b;          // channel-last copy of the image tensor, codes as bf16 [N][H][W][Cp]
    float *c;                   // [z][I][J] partial sums
    size_t plane;
    int I, J, R, lda, cps;
    SteConvGeo g;
};

// Partial sums of dy^T . col(x) (see ste_gemm_kernel with an unfolded operand): 64 x 64 outputs per workgroup, a 32 x 32 block per wave,
// chunks of 32 contraction indices through two LDS buffers, transposed on the way in (a thread packs two rows of four columns: rows of
// 18 words keep writes two-way and reads free of bank conflicts).
__global__ __launch_bounds__(STE_THREADS) void ste_dw16_kernel(const SteDwParams p) {
    constexpr int LD = 18;                                  // words of a row of 32 bf16
    __shared__ __align__(16) uint32_t As[2][3][64][LD];     // [piece][i][r]
    __shared__ __align__(16) uint32_t Bs[2][64][LD];        // [j][r]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    const int wi = (wave & 1) * 32, wj = (wave >> 1) * 32;
    const int pair = tid >> 4, c4 = (tid & 15) * 4;
    const SteConvGeo &g = p.g;
    // this thread's columns: of dy (clamped: what lies beyond is never stored), and the tap and channels of x
    const int ac = min(i0 + c4, p.lda - 4);
    const uint32_t k = (uint32_t)min(j0 + c4, p.J - 4), tap = g.dCp.div(k), ch = k - tap * g.dCp.d;
    const int ky = (int)g.dkw.div(tap), kx = (int)tap - ky * g.kw;
    const int offy = ky * g.dh - g.ph, offx = kx * g.dw - g.pw;
    uint2 ra[3][2], rb[2];
    uint32_t live[2], in[2];
    auto fetch = [&](int r0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = r0 + 2 * pair + h;
            const uint32_t m = (uint32_t)min(row, p.R - 1);
            live[h] = row < p.R ? ~0u : 0u;
#pragma unroll
            for (int q = 0; q < 3; ++q) ra[q][h] = *reinterpret_cast<const uint2 *>(p.a + q * p.plane + (size_t)m * (size_t)p.lda + (size_t)ac);
            const uint32_t n = g.dHoWo.div(m), pix = m - n * (uint32_t)(g.Ho * g.Wo);
            const int oy = (int)g.dWo.div(pix), ox = (int)pix - oy * g.Wo, iy = oy * g.sh + offy, ix = ox * g.sw + offx;
            const bool ok = iy >= 0 && iy < g.H && ix >= 0 && ix < g.W;
            in[h] = ok ? ~0u : 0u;
            rb[h] = *reinterpret_cast<const uint2 *>(p.b + (ok ? (((size_t)n * g.H + iy) * g.W + ix) * g.dCp.d + ch : 0));
        }
    };
    // rows r and r + 1 of four columns -> the word of both of each column
    auto put = [&](uint32_t (*to)[LD], const uint2 &e, const uint2 &o, uint32_t me, uint32_t mo) {
        const uint32_t e0 = e.x & me, e1 = e.y & me, o0 = o.x & mo, o1 = o.y & mo;
        to[c4 + 0][pair] = __builtin_amdgcn_perm(o0, e0, 0x05040100u);
        to[c4 + 1][pair] = __builtin_amdgcn_perm(o0, e0, 0x07060302u);
        to[c4 + 2][pair] = __builtin_amdgcn_perm(o1, e1, 0x05040100u);
        to[c4 + 3][pair] = __builtin_amdgcn_perm(o1, e1, 0x07060302u);
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < 3; ++q) put(As[buf][q], ra[q][0], ra[q][1], live[0], live[1]);
        put(Bs[buf], rb[0], rb[1], in[0], in[1]);
    };
    auto operand = [&](const uint32_t *row) {               // 8 bf16 of a row (8-byte aligned)
        const uint2 lo = *reinterpret_cast<const uint2 *>(row), hi = *reinterpret_cast<const uint2 *>(row + 2);
        return __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
    };
    f32x16_t acc[3];                // one for each piece
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = acc[2][v] = 0.0f;
    const int ch0 = blockIdx.z * p.cps, chunks = max(0, min((p.R + STE_TR - 1) / STE_TR, ch0 + p.cps) - ch0);
    if (chunks > 0) {
        fetch(ch0 * STE_TR);
        stash(0);
    }
    __syncthreads();
    for (int c = 0; c < chunks; ++c) {
        const int cur = c & 1;
        const bool more = c + 1 < chunks;
        if (more) fetch((ch0 + c + 1) * STE_TR);
        bf16x8_t a[2][3], b[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int at = 8 * ks + 4 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 3; ++q) a[ks][q] = operand(&As[cur][q][wi + (lane & 31)][at]);
            b[ks] = operand(&Bs[cur][wj + (lane & 31)][at]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks][q], b[ks], acc[q], 0, 0, 0);
        if (more) stash(cur ^ 1);
        __syncthreads();
    }
    float *const cout = p.c + (size_t)blockIdx.z * (size_t)p.I * (size_t)p.J;
    const int j = j0 + wj + (lane & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int i = i0 + wi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (i < p.I && j < p.J) cout[(size_t)i * (size_t)p.J + (size_t)j] = ste_join(acc[0][v], acc[1][v], acc[2][v]);
    }
}

// w [O][C][T] -> wq [T][Op / 8][Cq][8] bf16 codes times pow2, zeros beyond O and C (Op: O rounded up to 32, Cq: C to 64)
__global__ __launch_bounds__(256) void ste_weights16_kernel(const float *__restrict__ w, uint4 *__restrict__ wq, int O, int C, int Op, int Cq, int T, float s, float Q, float pow2) {
    const size_t total = (size_t)T * (Op / 8) * Cq, stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += stride) {
        const size_t t = i / ((size_t)(Op / 8) * Cq), rem = i - t * (size_t)(Op / 8) * Cq, og = rem / Cq, c = rem - og * Cq;
        uint32_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const size_t o = og * 8 + q;
            v[q] = o < (size_t)O && c < (size_t)C ? ste_code16(w[(o * C + c) * T + t], s, Q, pow2) : 0u;
        }
        wq[i] = make_uint4(ste_halves(v[0], v[1]), ste_halves(v[2], v[3]), ste_halves(v[4], v[5]), ste_halves(v[6], v[7]));
    }
}

struct SteDx16Params {
    const float *dy, *x;
    const uint4 *wq;
    float *dx;
    int pixels, og, Cq;         // N H W; groups of 8 output channels per tap, channels, as wq has them
    float so, Q, scale;
    SteConvGeo g;
};

// ste_dx_kernel on bf16 instructions: the gradient of a chunk is split while it is staged ([piece][pixel][o], so that a lane's eight
// output channels are one 16-byte read), the weights go from memory to registers as the instruction wants them.
__global__ __launch_bounds__(STE_THREADS, 2) void ste_dx16_kernel(const SteDx16Params p) {
    constexpr int LD = 20;                                  // words of a row of 32 bf16: 16-byte rows, 4 banks apart
    __shared__ __align__(16) uint32_t Bs[2][3][64][LD];     // [piece][pixel][o]
    const SteConvGeo &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    const int wi = (wave & 1) * 32, wj = (wave >> 1) * 32;
    const int P = g.Ho * g.Wo, HW = g.H * g.W;
    auto decode = [&](int j, int &n, int &pin) {
        n = (int)g.dHW.div((uint32_t)j);
        pin = j - n * HW;
    };
    int sn, spin;
    decode(min(j0 + lane, p.pixels - 1), sn, spin);
    const int sy = (int)g.dW.div((uint32_t)spin), sx = spin - sy * g.W;
    const float *const dyn = p.dy + (size_t)sn * g.O * (size_t)P;
    const int cpt = p.og / 4, chunks = g.kh * g.kw * cpt;
    int ky = 0, kx = 0, part = 0, group = 0;                // of the chunk that is fetched next
    float rb[2][8];
    uint4 ra[2][2];
    uint32_t inside[2];
    int from_o[2];
    auto fetch = [&](float (&b)[8], uint4 (&a)[2], uint32_t &in, int &first_o) {
        const int oy = sy + g.ph - ky * g.dh, ox = sx + g.pw - kx * g.dw, o0 = part * STE_TR + 8 * wave;
        const bool ok = oy >= 0 && oy < g.Ho && ox >= 0 && ox < g.Wo;
        const float *const from = dyn + (ok ? oy * g.Wo + ox : 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) b[i] = from[(size_t)min(o0 + i, g.O - 1) * (size_t)P];
        in = ok ? ~0u : 0u;
        first_o = o0;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) a[ks] = p.wq[((size_t)group + 2 * ks + (lane >> 5)) * (size_t)p.Cq + (size_t)(i0 + wi + (lane & 31))];
        group += 4;
        if (++part == cpt) {
            part = 0;
            if (++kx == g.kw) {
                kx = 0;
                ++ky;
            }
        }
    };
    auto stash = [&](int buf, const float (&b)[8], uint32_t in, int first_o) {
        uint32_t s[8][3];
#pragma unroll
        for (int i = 0; i < 8; ++i) ste_split(__uint_as_float(__float_as_uint(b[i]) & (first_o + i < g.O ? in : 0u)), s[i]);
#pragma unroll
        for (int q = 0; q < 3; ++q)
            *reinterpret_cast<uint4 *>(&Bs[buf][q][lane][4 * wave]) =
                make_uint4(ste_halves(s[0][q], s[1][q]), ste_halves(s[2][q], s[3][q]), ste_halves(s[4][q], s[5][q]), ste_halves(s[6][q], s[7][q]));
    };
    f32x16_t acc[3], tot;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = acc[2][v] = tot[v] = 0.0f;
    int left = cpt;                 // chunks of this tap that are still to be multiplied
    auto chunk = [&](int ch, auto set_c) {                  // see ste_dx_kernel
        constexpr int S = decltype(set_c)::value;
        const uint4 a0 = ra[S][0], a1 = ra[S][1];
        if (ch + 2 < chunks) fetch(rb[S], ra[S], inside[S], from_o[S]);
        bf16x8_t b[2][3];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int q = 0; q < 3; ++q) b[ks][q] = *reinterpret_cast<const bf16x8_t *>(&Bs[S][q][wj + (lane & 31)][8 * ks + 4 * (lane >> 5)]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ks ? a1 : a0), b[ks][q], acc[q], 0, 0, 0);
        if (ch + 1 < chunks) stash(1 - S, rb[1 - S], inside[1 - S], from_o[1 - S]);
        if (--left == 0) {
            left = cpt;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                tot[v] += acc[0][v];            // (the others are small: rounded less than the first at any length)
                acc[0][v] = 0.0f;
            }
        }
        __syncthreads();
    };
    fetch(rb[0], ra[0], inside[0], from_o[0]);
    if (chunks > 1) fetch(rb[1], ra[1], inside[1], from_o[1]);
    stash(0, rb[0], inside[0], from_o[0]);
    __syncthreads();
    for (int ch = 0; ch < chunks; ch += 2) {
        chunk(ch, std::integral_constant<int, 0>{});
        if (ch + 1 < chunks) chunk(ch + 1, std::integral_constant<int, 1>{});
    }
    const int j = j0 + wj + (lane & 31);
    if (j >= p.pixels) return;
    int n, pin;
    decode(j, n, pin);
    float xv[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = i0 + wi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        xv[v] = c < g.C ? p.x[((size_t)n * g.C + c) * (size_t)HW + (size_t)pin] : 0.0f;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = i0 + wi + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (c < g.C) p.dx[((size_t)n * g.C + c) * (size_t)HW + (size_t)pin] = ste_inside(xv[v], p.so, p.Q) ? ste_join(tot[v], acc[1][v], acc[2][v]) * p.scale : 0.0f;
    }
}

// dx[n][c][iy][ix] = inside(x) * sum over the taps (ky, kx ascending) that land on (iy, ix) of dcol[(n, oy, ox)][(ky, kx, c)]
template <typename Idx>
__global__ __launch_bounds__(256) void ste_col2im_kernel(const float *__restrict__ dcol, const float *__restrict__ x, float *__restrict__ dx,
                                                         SteConvGeo g, float s_x, float Q, size_t total) {
    const Idx stride = (Idx)gridDim.x * 256;
    const size_t K = (size_t)g.C * g.kh * g.kw;
    for (Idx i = (Idx)blockIdx.x * 256 + threadIdx.x; i < (Idx)total; i += stride) {
        // neighbouring lanes take neighbouring channels of one pixel: their reads of dcol are consecutive floats of one
        // row; the one store and the one read of x per lane are the strided side
        const Idx pixel = ste_div<Idx>(i, g.dC);
        const int c = (int)(i - pixel * (Idx)g.C);
        const Idx n = ste_div<Idx>(pixel, g.dHW);
        const int pin = (int)(pixel - n * (Idx)(g.H * g.W));
        const int iy = (int)g.dW.div((uint32_t)pin), ix = pin - iy * g.W;
        const size_t at = (((size_t)n * g.C + c) * g.H + iy) * g.W + ix;
        float s = 0.0f;
        for (int ky = 0; ky < g.kh; ++ky) {
            const int ty = iy + g.ph - ky * g.dh;
            if (ty < 0) continue;
            const int oy = (int)g.dsh.div((uint32_t)ty);
            if (oy * g.sh != ty || oy >= g.Ho) continue;
            for (int kx = 0; kx < g.kw; ++kx) {
                const int tx = ix + g.pw - kx * g.dw;
                if (tx < 0) continue;
                const int ox = (int)g.dsw.div((uint32_t)tx);
                if (ox * g.sw != tx || ox >= g.Wo) continue;
                s += dcol[(((size_t)n * g.Ho + oy) * g.Wo + ox) * K + (size_t)(ky * g.kw + kx) * g.C + c];
            }
        }
        dx[at] = ste_inside(x[at], s_x, Q) ? s : 0.0f;
    }
}

}  // namespace adapt
