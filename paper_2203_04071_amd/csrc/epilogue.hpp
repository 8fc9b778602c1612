// What the derived-table kernels share at both ends: the activation sources of the copies they read, and what becomes of a
// finished sum (rescaling, border terms of a transposed convolution, the next layer's input copy).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elementwise.hpp"

namespace adapt {

// A layer's output written a second time as the NEXT convolution's input copy: quantised with that layer's activation
// scale (the quantiser of Sec. III-A), as table line indices, at the element's place in the zero-padded x-major or
// channel-last copy (see pad_channels_last_kernel) whose borders and padded channels were zeroed beforehand.  The next
// layer then needs no copy kernel of its own.  buf == nullptr: nothing to do.
// Copies for layers that move their window by more than one pixel hold the columns of a row in residue classes modulo the
// horizontal stride (col_pos, see byte_copy_kernel); Wp is the length of a row as stored.
struct ChainOut {
    int8_t *buf;
    int xmajor, Hp, Wp, Cp, ph, pw;
    float scale, Q;
    uint32_t mask;
    int shift;              // low bits of the codes that the reader's tables do not tell apart (they are left out)
    uint32_t wsub;          // columns per residue class (read only if dsw.d > 1)
    FastDiv dsw;            // division by the horizontal stride of the layer that reads the copy; d <= 1: columns in order
    __device__ __forceinline__ uint32_t col_pos(uint32_t col) const {
        if (dsw.d <= 1) return col;
        const uint32_t q = dsw.div(col);
        return (col - q * dsw.d) * wsub + q;
    }
    // element (image, channel c, row oy, column ox) of the producing layer's fp32 output y
    __device__ __forceinline__ void put(int img, int c, int oy, int ox, float y) const {
        const uint32_t q = (uint32_t)((int)(int8_t)code(y) >> shift);
        // (a copy is smaller than 2^32 bytes: 32-bit offsets)
        const uint32_t row = (uint32_t)img * (uint32_t)Hp + (uint32_t)(oy + ph), col = col_pos((uint32_t)(ox + pw));
        const uint32_t a = xmajor ? ((row * (uint32_t)(Cp >> 2) + (uint32_t)(c >> 2)) * (uint32_t)Wp + col) * 4u + (uint32_t)(c & 3)
                                  : (row * (uint32_t)Wp + col) * (uint32_t)Cp + (uint32_t)c;
        buf[a] = (int8_t)q;
    }
    // the same for channels c .. c + 3 (c a multiple of 4, Cp a multiple of 4) of one pixel: they are one aligned word
    // of either copy
    __device__ __forceinline__ uint32_t code(float y) const { return (uint32_t)quant1(y, scale, Q) & mask; }
    __device__ __forceinline__ void put4(int img, int c, int oy, int ox, uint32_t codes) const {
        if (shift)          // (four signed bytes at once; the same in the whole launch)
            codes = ((codes >> shift) & ((0xffu >> shift) * 0x01010101u)) | ((codes >> 7) & 0x01010101u) * ((0xff00u >> shift) & 0xffu);
        const uint32_t row = (uint32_t)img * (uint32_t)Hp + (uint32_t)(oy + ph), col = col_pos((uint32_t)(ox + pw));
        const uint32_t a = xmajor ? ((row * (uint32_t)(Cp >> 2) + (uint32_t)(c >> 2)) * (uint32_t)Wp + col) * 4u
                                  : (row * (uint32_t)Wp + col) * (uint32_t)Cp + (uint32_t)c;
        *reinterpret_cast<uint32_t *>(buf + a) = codes;
    }
};

// What the window taps WITHOUT an input pixel added to the V output pixels (oy, ox + i * stride), i = 0 .. V - 1, of channel
// co of a transposed convolution (see LinesParams::zsum); zero away from the border.  The V pixels belong to one phase: they
// share the row's taps and the column residue, so every zero sum is loaded once.
template <int V, typename P>
__device__ __forceinline__ void convt_border_terms(const P &p, int co, int oy, int ox, uint32_t (&extra)[V]) {
    const int st = (int)p.cv_s.d;
    const int qy = (int)p.cv_s.div((uint32_t)(oy + p.cv_pad)), ry = oy + p.cv_pad - qy * st;
    const int qx = (int)p.cv_s.div((uint32_t)(ox + p.cv_pad)), rx = ox + p.cv_pad - qx * st;
    const int32_t *z = p.zsum + (size_t)co * p.cv_kh * p.cv_kw;
#pragma unroll
    for (int i = 0; i < V; ++i) extra[i] = 0;
    for (int m = 0; m * st + ry < p.cv_kh; ++m) {
        const bool yin = qy - m >= 0 && qy - m < p.cv_H;
        for (int nn = 0; nn * st + rx < p.cv_kw; ++nn) {
            const int x0 = qx - nn;             // input column of pixel 0; pixel i has x0 + i
            if (yin && x0 >= 0 && x0 + V - 1 < p.cv_W) continue;
            const uint32_t zz = (uint32_t)z[(ry + st * m) * p.cv_kw + (rx + st * nn)];
#pragma unroll
            for (int i = 0; i < V; ++i)
                if (!(yin && (unsigned)(x0 + i) < (unsigned)p.cv_W)) extra[i] += zz;
        }
    }
}

// What is stored for the finished sum v of output channel n (see LinesParams::deq); off: element offset of the output
// position (for the residual input).  EXTRA: the instantiation also knows tanh; the plain one does not (eight inlined copies
// of that code in an epilogue cost the ordinary layers about a microsecond per launch)
template <bool EXTRA = false, typename P>
__device__ __forceinline__ uint32_t finish_sum(const P &p, uint32_t v, int n, size_t off) {
    if (!p.deq) return v;
    float y = (float)(int32_t)v * (p.scales ? p.scales[n] : p.scale);
    if (p.bias) y = y + p.bias[n];
    if (p.resid) y = y + p.resid[off];
    if (p.act == 1) y = y > 0.0f ? y : 0.0f;
    else if (EXTRA && p.act == 2) y = tanh_spec(y);
    return __float_as_uint(y);
}

// per-phase launch parameters without indexing the by-value argument block dynamically
template <typename T>
__device__ __forceinline__ T pick4(const T *v, int i) {
    return i == 0 ? v[0] : (i == 1 ? v[1] : (i == 2 ? v[2] : v[3]));
}

// Activation sources of the copy kernels: already quantised int8, or fp32 quantised on the fly with the quantiser of
// quantize_kernel (Sec. III-A), so that a layer needs no separate quantisation pass.  The copies hold table line
// indices (the kernels that extract a bit field do not care, the quad kernel relies on it).
// byte(): the operand as a table line index, i.e. its two's-complement bits below 2^b (mask = 2^b - 1)
// load() / code(): the two halves of byte(), for kernels that request several operands before they convert the first
// code8(): the operand itself as a signed byte (wrapped into b bits), without its low `shift` bits: what the copies of the byte kernel hold
struct SrcI8 {
    typedef int8_t raw_t;
    const int8_t *x;
    uint32_t mask;
    int shift = 0;
    __device__ __forceinline__ uint32_t byte(size_t i) const { return (uint32_t)(uint8_t)x[i] & mask; }
    __device__ __forceinline__ raw_t load(uint32_t i) const { return x[i]; }
    __device__ __forceinline__ uint32_t code(raw_t v) const { return (uint32_t)(uint8_t)v & mask; }
    __device__ __forceinline__ uint32_t code8(raw_t v) const {
        const uint32_t h = (mask + 1u) >> 1;
        return (uint32_t)((int)((((uint32_t)(uint8_t)v & mask) ^ h) - h) >> shift) & 0xffu;
    }
};
struct SrcF32 {
    typedef float raw_t;
    const float *x;
    float scale, Q;
    uint32_t mask;
    int shift = 0;
    __device__ __forceinline__ uint32_t byte(size_t i) const { return (uint32_t)quant1(x[i], scale, Q) & mask; }
    __device__ __forceinline__ raw_t load(uint32_t i) const { return x[i]; }
    __device__ __forceinline__ uint32_t code(raw_t v) const { return (uint32_t)quant1(v, scale, Q) & mask; }
    __device__ __forceinline__ uint32_t code8(raw_t v) const { return (uint32_t)(quant1(v, scale, Q) >> shift) & 0xffu; }
};

}  // namespace adapt
