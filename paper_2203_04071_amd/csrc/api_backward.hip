// C ABI, part 4: the backward pass of Sec. III-A's retraining (straight-through estimator) and the optimiser step.
#include "api_common.hpp"
#include "ste_backward.hpp"

using namespace adapt_api;

namespace {

// Shape of the gradient products' launch: 128 x 128 outputs per workgroup where that still occupies three quarters of
// the compute units, else 64 x 64; eight waves per workgroup instead of four (KS = 2) where there are fewer than two
// workgroups per compute unit.  Env ADAPT_STE_TILE = 64 / 128 and ADAPT_STE_KS = 1 / 2 force one (for measurements).
// `full`: whole tiles, 16-byte rows.
int ste_env(const char *name) {
    const char *e = getenv(name);
    return e ? atoi(e) : 0;
}
// Floats of partial sums a split product may need: it is split only below 256 tiles of 64 x 64, into at most
// 512 / tiles + 1 parts.  (An unsplit one over an unfolded input passes through there as well: see SteConvPlan.)
constexpr size_t STE_PARTIAL_FLOATS = (size_t)(512 + 256) * 64 * 64;

// partials != nullptr: a product over an unfolded input (im2col); with few output tiles and a long contraction it is split
// over grid z into partial sums, which ste_reduce_masked_kernel adds in a fixed order (its columns are taps tap0 .. of a filter of
// all_taps).
void launch_ste_gemm(const adapt::SteParams &p_in, bool a_t, bool aligned, hipStream_t s, float *partials = nullptr, int tap0 = 0, int all_taps = 0) {
    static const int env_tile = ste_env("ADAPT_STE_TILE"), env_ks = ste_env("ADAPT_STE_KS");
    adapt::SteParams p = p_in;
    const int cus = device_cus();
    const long long t128 = (((long long)p.I + 127) / 128) * (((long long)p.J + 127) / 128);
    int tile = 4 * t128 >= 3 * cus ? 128 : 64;
    // whole 64-tiles where 128-tiles would be ragged: the unguarded 16-byte loads are worth more than the larger tile
    const bool whole_ok = aligned && p.R % adapt::STE_TR == 0 && p.lda % 4 == 0 && p.R > 0;
    if (tile == 128 && whole_ok && (p.I % 128 || p.J % 128) && p.I % 64 == 0 && p.J % 64 == 0) tile = 64;
    if (env_tile == 64 || env_tile == 128) tile = env_tile;
    dim3 grid((unsigned)((p.J + tile - 1) / tile), (unsigned)((p.I + tile - 1) / tile), 1);
    const int chunks = (p.R + adapt::STE_TR - 1) / adapt::STE_TR;
    const long long tiles = (long long)grid.x * grid.y;
    p.cps = chunks > 0 ? chunks : 1;
    int parts = 1;
    if (partials && p.im2col && tile == 64 && tiles < cus && chunks >= 8) {       // (the kernels split only in their unfolded-input form)
        int want = (int)((2 * cus + tiles - 1) / tiles);
        if (want > chunks / 4) want = chunks / 4;                   // at least four chunks per part
        if (want >= 2) {
            p.cps = (chunks + want - 1) / want;
            parts = (chunks + p.cps - 1) / p.cps;
        }
    }
    if (p.im2col) { grid.z = (unsigned)parts; p.c = partials; p.o = nullptr; }
    int ks = tiles * parts < 2 * cus ? 2 : 1;
    if (env_ks == 1 || env_ks == 2) ks = env_ks;
    const bool full = aligned && p.I % tile == 0 && p.J % tile == 0 && p.R % adapt::STE_TR == 0 && p.lda % 4 == 0 && p.R > 0;
#define STE_LAUNCH4(AT, T, F, U) \
    do { if (ks == 2) adapt::ste_gemm_kernel<AT, T, F, 2, U><<<grid, adapt::STE_THREADS * 2, 0, s>>>(p); \
         else adapt::ste_gemm_kernel<AT, T, F, 1, U><<<grid, adapt::STE_THREADS, 0, s>>>(p); } while (0)
#define STE_LAUNCH2(AT, T, U) do { if (full) STE_LAUNCH4(AT, T, true, U); else STE_LAUNCH4(AT, T, false, U); } while (0)
    if (a_t && p.im2col) { if (tile == 128) STE_LAUNCH2(true, 128, true); else STE_LAUNCH2(true, 64, true); }
    else if (a_t) { if (tile == 128) STE_LAUNCH2(true, 128, false); else STE_LAUNCH2(true, 64, false); }
    else { if (tile == 128) STE_LAUNCH2(false, 128, false); else STE_LAUNCH2(false, 64, false); }
#undef STE_LAUNCH2
#undef STE_LAUNCH4
    if (p.im2col) {             // (one part too: the columns are in another order than the weight tensor)
        const size_t n = (size_t)p.I * (size_t)p.J;
        const size_t blocks = (n + 255) / 256;
        adapt::ste_reduce_masked_kernel<<<(unsigned)(blocks < 4096 ? blocks : 4096), 256, 0, s>>>(partials, parts, n, p_in.o, p_in.so, p_in.Q,
                                                                                                  p_in.c, p.g.kh * p.g.kw, p.g.C, (int)p.g.dCp.d, tap0, all_taps, 1.0f);
    }
}

// Weight gradient of a convolution on bf16 instructions (ste_dw16_kernel): partial sums as launch_ste_gemm makes them, 64 x 64 outputs
// per workgroup and two workgroups per compute unit where the contraction of R rows is long enough.
dim3 ste_dw16_grid(int I, int J, int R, int *chunks_per_slice) {
    const int cus = device_cus(), chunks = (R + adapt::STE_TR - 1) / adapt::STE_TR;
    dim3 grid((unsigned)((J + 63) / 64), (unsigned)((I + 63) / 64), 1);
    const long long tiles = (long long)grid.x * grid.y;
    *chunks_per_slice = chunks;
    if (tiles < cus && chunks >= 8) {
        int want = (int)((2 * cus + tiles - 1) / tiles);
        if (want > chunks / 4) want = chunks / 4;
        if (want >= 2) {
            *chunks_per_slice = (chunks + want - 1) / want;
            grid.z = (unsigned)((chunks + *chunks_per_slice - 1) / *chunks_per_slice);
        }
    }
    return grid;
}
// o, so: mask; scale: of the sums
void launch_ste_dw16(const adapt::SteDwParams &p_in, const float *o, float so, float Q, float scale, float *dw, hipStream_t s, float *partials, int tap0, int all_taps) {
    adapt::SteDwParams p = p_in;
    const dim3 grid = ste_dw16_grid(p.I, p.J, p.R, &p.cps);
    p.c = partials;
    adapt::ste_dw16_kernel<<<grid, adapt::STE_THREADS, 0, s>>>(p);
    const size_t n = (size_t)p.I * (size_t)p.J, blocks = (n + 255) / 256;
    adapt::ste_reduce_masked_kernel<<<(unsigned)(blocks < 4096 ? blocks : 4096), 256, 0, s>>>(partials, (int)grid.z, n, o, so, Q, dw, p.g.kh * p.g.kw, p.g.C,
                                                                                              (int)p.g.dCp.d, tap0, all_taps, scale);
}

// s = pow2 * rest with rest in [1, 2)
void split_scale(float s, float *pow2, float *rest) {
    int e;
    *rest = 2.0f * frexpf(s, &e);
    *pow2 = ldexpf(1.0f, e - 1);
}

}  // namespace

extern "C" {

int adapt_ste_linear_backward_f32(const float *dy_dev, const float *x_dev, const float *w_dev, int M, int K, int N, float s_x,
                                  float s_w, int bits, float *dx_dev, float *dw_dev, float *db_dev, void *stream) {
    const char *who = "adapt_ste_linear_backward_f32";
    if (M < 0 || K < 0 || N < 0) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: negative size", who);
    if (bits < 2 || bits > 16) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: bits=%d not in [2,16]", who, bits);
    if (!(s_x > 0.0f) || !(s_w > 0.0f) || s_x > 3.0e38f || s_w > 3.0e38f)
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: scales must be finite and > 0", who);
    const bool want_dx = dx_dev && M > 0 && K > 0, want_dw = dw_dev && N > 0 && K > 0, want_db = db_dev && N > 0;
    if ((want_dx || want_dw || want_db) && M > 0 && N > 0 && !dy_dev) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL dy_dev", who);
    if ((want_dx || want_dw) && ((M > 0 && !x_dev) || (N > 0 && !w_dev))) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL x_dev / w_dev", who);
    for (const void *q : {(const void *)dy_dev, (const void *)x_dev, (const void *)w_dev, (const void *)dx_dev, (const void *)dw_dev, (const void *)db_dev})
        if (reinterpret_cast<uintptr_t>(q) & 3u) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: pointer not aligned to 4 bytes", who);
    if ((dx_dev && (dx_dev == x_dev || dx_dev == dy_dev || dx_dev == w_dev)) || (dw_dev && (dw_dev == w_dev || dw_dev == dy_dev || dw_dev == x_dev)))
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: a gradient must not alias an input", who);
    if (((long long)M + 63) / 64 > 65535 || ((long long)N + 63) / 64 > 65535)
        return fail(ADAPT_ERR_UNSUPPORTED, "%s: M and N are limited to %d", who, 65535 * 64);
    hipStream_t s = (hipStream_t)stream;
    const float Q = (float)((1 << (bits - 1)) - 1);
    if (want_dx) {          // dx [M][K] = inside(x) * dy [M][N] . fq(w) [N][K]
        adapt::SteParams p{};
        p.a = dy_dev; p.b = w_dev; p.o = x_dev; p.c = dx_dev;
        p.I = M; p.J = K; p.R = N; p.lda = N;
        p.sb = s_w; p.so = s_x; p.Q = Q;
        launch_ste_gemm(p, false, aligned16(dy_dev) && aligned16(w_dev), s);
        HIP_TRY(hipGetLastError());
    }
    if (want_dw) {          // dw [N][K] = inside(w) * dy^T [N][M] . fq(x) [M][K]
        adapt::SteParams p{};
        p.a = dy_dev; p.b = x_dev; p.o = w_dev; p.c = dw_dev;
        p.I = N; p.J = K; p.R = M; p.lda = N;
        p.sb = s_x; p.so = s_w; p.Q = Q;
        launch_ste_gemm(p, true, aligned16(dy_dev) && aligned16(x_dev), s);
        HIP_TRY(hipGetLastError());
    }
    if (want_db) {
        adapt::ste_colsum_kernel<<<(unsigned)((N + 31) / 32), adapt::STE_COLSUM_THREADS, 0, s>>>(dy_dev, db_dev, M, N);
        HIP_TRY(hipGetLastError());
    }
    return ADAPT_OK;
}

}  // extern "C"

namespace {
constexpr long long MAX_COLS = 0x3fffff00;         // of one product: 31-bit columns, and four threads per column in a launch of less than 2^32

struct SteConvPlan {
    adapt::SteConvGeo g;
    long long M, K;
    bool direct;                // stride 1: the input gradient is one product (ste_dx_kernel, ste_dx16_kernel)
    int dw_rows;                // filter rows per product of the weight gradient: all, unless there are more than MAX_COLS columns (tap, channel rounded up to 4)
    size_t rows_bytes, col_bytes, wp_bytes, xq_bytes, part_bytes, total;    // of the forms on fp32 instructions: what a call needs in any case
    // Weight gradient on bf16 instructions: its copies and sums, which nothing needs once it is finished, lie over everything but the rows
    // that a strided layer's input gradient reads (kept_bytes).  all: with room for them; only layers with more output than input channels need more.
    int lda;
    size_t kept_bytes, pieces_bytes, codes_bytes, sums_bytes, all;
};
int ste_conv_plan(SteConvPlan *pl, int N, int Cin, int H, int W, int Cout, int kh, int kw, int stride_h, int stride_w, int pad_h, int pad_w,
                  int dil_h, int dil_w, bool want_dx, bool want_dw, const char *who) {
    if (N < 0 || Cin < 1 || H < 1 || W < 1 || Cout < 1 || kh < 1 || kw < 1 || stride_h < 1 || stride_w < 1 || pad_h < 0 || pad_w < 0 ||
        dil_h < 1 || dil_w < 1)
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: bad dimension", who);
    const long long Ho = ((long long)H + 2LL * pad_h - (long long)dil_h * (kh - 1) - 1) / stride_h + 1;
    const long long Wo = ((long long)W + 2LL * pad_w - (long long)dil_w * (kw - 1) - 1) / stride_w + 1;
    if ((long long)H + 2LL * pad_h < (long long)dil_h * (kh - 1) + 1 || (long long)W + 2LL * pad_w < (long long)dil_w * (kw - 1) + 1)
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: the filter does not fit the padded image", who);
    pl->M = (long long)N * Ho * Wo;
    pl->K = (long long)Cin * kh * kw;
    if (pl->M > 65535LL * 64 || pl->K > 0x7fffffffLL || Ho > 0x7fffffffLL || Wo > 0x7fffffffLL || (long long)N * Cin * H * W > (1LL << 40))
        return fail(ADAPT_ERR_UNSUPPORTED, "%s: tensor too large (N Ho Wo is limited to %d)", who, 65535 * 64);
    if ((long long)H * W > 0x7fffffffLL || Ho * Wo > 0x7fffffffLL)
        return fail(ADAPT_ERR_UNSUPPORTED, "%s: an image plane is limited to 2^31 - 1 pixels", who);
    adapt::SteConvGeo &g = pl->g;
    g = adapt::SteConvGeo{};
    g.N = N; g.C = Cin; g.H = H; g.W = W; g.O = Cout; g.kh = kh; g.kw = kw; g.sh = stride_h; g.sw = stride_w; g.ph = pad_h; g.pw = pad_w;
    g.dh = dil_h; g.dw = dil_w; g.Ho = (int)Ho; g.Wo = (int)Wo;
    const long long Cp = ((long long)Cin + 3) / 4 * 4;
    g.dkw = fast_div((uint32_t)kw); g.dWo = fast_div((uint32_t)Wo); g.dCp = fast_div((uint32_t)Cp);
    g.dHoWo = fast_div((uint32_t)(Ho * Wo)); g.dC = fast_div((uint32_t)Cin); g.dW = fast_div((uint32_t)W); g.dHW = fast_div((uint32_t)(H * W));
    g.dsh = fast_div((uint32_t)stride_h); g.dsw = fast_div((uint32_t)stride_w);
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    pl->rows_bytes = up((size_t)pl->M * Cout * sizeof(float));
    const long long row_cols = (long long)kw * Cp;
    if (want_dw && row_cols > 0x7fffff00LL)
        return fail(ADAPT_ERR_UNSUPPORTED, "%s: a filter row is limited to 2^31 - 256 weights (channels rounded up to 4)", who);
    pl->dw_rows = (int)(kh * row_cols <= MAX_COLS ? kh : (row_cols < MAX_COLS ? MAX_COLS / row_cols : 1));
    pl->direct = stride_h == 1 && stride_w == 1 && (long long)N * H * W < 0x7fffff00LL && kh * row_cols <= MAX_COLS;
    pl->col_bytes = want_dx && !pl->direct ? up((size_t)pl->M * (size_t)pl->K * sizeof(float)) : 0;
    const size_t cols = (size_t)kh * kw * (size_t)Cp;
    pl->xq_bytes = want_dw ? up((size_t)N * H * W * (size_t)Cp * sizeof(float)) : 0;
    const size_t dw_cols = (size_t)pl->dw_rows * (size_t)row_cols;
    pl->part_bytes = up((want_dw && Cout * dw_cols > STE_PARTIAL_FLOATS ? Cout * dw_cols : STE_PARTIAL_FLOATS) * sizeof(float));
    pl->wp_bytes = want_dx ? up((size_t)Cout * cols * sizeof(float)) : 0;
    pl->total = pl->all = pl->rows_bytes + pl->col_bytes + pl->wp_bytes + pl->xq_bytes + pl->part_bytes;
    if (want_dw && pl->M > 0) {
        int cps;
        pl->lda = (int)(((long long)Cout + 3) / 4 * 4);
        pl->kept_bytes = want_dx && !pl->direct ? pl->rows_bytes : 0;
        pl->pieces_bytes = up((size_t)pl->M * pl->lda * 6);
        pl->codes_bytes = up((size_t)N * H * W * (size_t)Cp * 2);
        pl->sums_bytes = up((size_t)ste_dw16_grid(Cout, (int)dw_cols, (int)pl->M, &cps).z * Cout * dw_cols * sizeof(float));
        const size_t need = pl->kept_bytes + pl->pieces_bytes + pl->codes_bytes + pl->sums_bytes;
        pl->all = need > pl->all ? need : pl->all;
    }
    return ADAPT_OK;
}
}  // namespace

extern "C" {

int adapt_ste_conv2d_backward_workspace(int N, int Cin, int H, int W, int Cout, int kh, int kw, int stride_h, int stride_w, int pad_h,
                                        int pad_w, int dil_h, int dil_w, int want_dx, int want_dw, size_t *bytes) {
    const char *who = "adapt_ste_conv2d_backward_workspace";
    if (!bytes) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL pointer", who);
    SteConvPlan pl;
    int rc = ste_conv_plan(&pl, N, Cin, H, W, Cout, kh, kw, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, want_dx != 0, want_dw != 0, who);
    if (rc) return rc;
    *bytes = pl.all;
    return ADAPT_OK;
}

int adapt_ste_conv2d_backward_f32(const float *dy_dev, const float *x_dev, const float *w_dev, int N, int Cin, int H, int W, int Cout,
                                  int kh, int kw, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w, float s_x,
                                  float s_w, int bits, float *dx_dev, float *dw_dev, float *db_dev, void *workspace_dev,
                                  size_t workspace_bytes, void *stream) {
    const char *who = "adapt_ste_conv2d_backward_f32";
    if (bits < 2 || bits > 16) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: bits=%d not in [2,16]", who, bits);
    if (!(s_x > 0.0f) || !(s_w > 0.0f) || s_x > 3.0e38f || s_w > 3.0e38f)
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: scales must be finite and > 0", who);
    SteConvPlan pl;
    int rc = ste_conv_plan(&pl, N, Cin, H, W, Cout, kh, kw, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, dx_dev != nullptr,
                           dw_dev != nullptr, who);
    if (rc) return rc;
    if (pl.M > 0 && (!dy_dev || !x_dev || !w_dev)) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL pointer", who);
    for (const void *q : {(const void *)dy_dev, (const void *)x_dev, (const void *)w_dev, (const void *)dx_dev, (const void *)dw_dev,
                          (const void *)db_dev})
        if (reinterpret_cast<uintptr_t>(q) & 3u) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: pointer not aligned to 4 bytes", who);
    if ((dx_dev && (dx_dev == x_dev || dx_dev == dy_dev || dx_dev == w_dev)) || (dw_dev && (dw_dev == w_dev || dw_dev == dy_dev || dw_dev == x_dev)))
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: a gradient must not alias an input", who);
    if (!dx_dev && !dw_dev && !db_dev) return ADAPT_OK;
    hipStream_t s = (hipStream_t)stream;
    const adapt::SteConvGeo &g = pl.g;
    const float Q = (float)((1 << (bits - 1)) - 1);
    const size_t w_elems = (size_t)Cout * (size_t)pl.K, x_elems = (size_t)N * Cin * H * W;
    if (pl.M == 0) {        // no samples: the weight and bias gradients are zero, there is no input gradient
        if (dw_dev) adapt::fill_u32_kernel<<<ew_grid(w_elems), 256, 0, s>>>(reinterpret_cast<uint32_t *>(dw_dev), 0u, w_elems);
        if (db_dev) adapt::fill_u32_kernel<<<ew_grid((size_t)Cout), 256, 0, s>>>(reinterpret_cast<uint32_t *>(db_dev), 0u, (size_t)Cout);
        HIP_TRY(hipGetLastError());
        return ADAPT_OK;
    }
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 255u) || workspace_bytes < pl.total)
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: workspace of %zu bytes, aligned to 256, needed (adapt_ste_conv2d_backward_workspace)", who,
                    pl.total);
    char *ws = static_cast<char *>(workspace_dev);
    float *rows = reinterpret_cast<float *>(ws);
    float *dcol = reinterpret_cast<float *>(ws + pl.rows_bytes);
    float *wp = reinterpret_cast<float *>(ws + pl.rows_bytes + pl.col_bytes);           // the weights in the order that the input gradient reads
    float *xq = reinterpret_cast<float *>(ws + pl.rows_bytes + pl.col_bytes + pl.wp_bytes);
    float *partials = reinterpret_cast<float *>(ws + pl.total - pl.part_bytes);         // used by one kernel pair at a time (stream order)
    const int M = (int)pl.M, K = (int)pl.K, P = g.Ho * g.Wo, HW = H * W, Cp = (int)g.dCp.d;
    const size_t col_n = (size_t)M * K;     // elements of dcol
    auto channels_last = [&](const float *src, float *dst, int C, int pixels, int ld, float scale) {
        const long long blocks = (pixels + 31LL) / 32;
        const dim3 grid((unsigned)(blocks < (1 << 22) ? blocks : (1 << 22)), (unsigned)((ld + 63) / 64), (unsigned)(N < 65535 ? N : 65535));
        adapt::ste_channels_last_kernel<<<grid, 256, 0, s>>>(src, dst, N, C, pixels, ld, scale, Q);
    };
    // Codes of up to 9 bits are bf16 numbers: both products on bf16 instructions (a scale whose power of two is not a normal number, or
    // leaves none to the codes, takes the fp32 form).  64 -> 64 channels, 3 x 3, 32 images of 32 x 32: weight gradient 43 -> 28 us,
    // input gradient 42 -> 28 us, with errors against 64 bits of 0.4 to 0.9 of the fp32 form (2-norms of 4e-8 to 2e-7 over 14 layers).
    const bool codes16 = bits <= 9;
    // Weight gradient of at most 64 columns (taps x channels): one pass over the copies, which are 6 bytes an element of dY instead of 4.  What is read
    // and written of dY (10 bytes, 14 with the rows of a strided layer) beyond the last-level cache costs more than the instructions gain: 1 -> 250
    // channels, 1 x 1, fp32 form / this one: 210 MB 116 / 121 us, 280 MB 211 / 242, 1.6 GB 720 / 863; 8 -> 112: 183 MB 129 / 119, 257 MB 237 / 252.
    const bool beyond_cache = (long long)pl.dw_rows * kw * Cp <= 64 && (size_t)M * Cout * (dx_dev && !pl.direct ? 14 : 10) > ((size_t)192 << 20);
    const bool dw16 = dw_dev && !beyond_cache && codes16 && s_x > 1e-30f && s_x < 1e30f && workspace_bytes >= pl.kept_bytes + pl.pieces_bytes + pl.codes_bytes + pl.sums_bytes;
    // Input gradient: the 16-bit form pays for its start (its weights come padded, its gradient is split while it is staged) and gains with
    // every chunk of 32 output channels of a tap.  Speed against the fp32 form, up to one workgroup per compute unit: 1 chunk 0.85 - 0.92,
    // 4 chunks 0.92 - 0.98, 6 chunks 0.99 - 1.02, 18 chunks 1.10 - 1.14; up to two: 2 chunks 0.95 - 1.00, 3 chunks 0.96 - 1.05, 9 chunks
    // 1.19 - 1.34; more: 1 chunk 0.93 - 1.07, 2 chunks 0.97 - 1.15, 9 chunks 1.21 - 1.44.
    const long long dx_chunks = (long long)kh * kw * ((Cout + 31) / 32), dx_wgs = ((long long)N * HW + 63) / 64 * ((Cin + 63) / 64);
    const bool dx16 = codes16 && s_w > 1e-30f && s_w < 1e30f && dx_chunks >= (dx_wgs > 2 * device_cus() ? 2 : (dx_wgs > device_cus() ? 3 : 6));
    if (dw16) {
        const int lda = pl.lda;
        const size_t plane = (size_t)M * lda;
        char *const copies = ws + pl.kept_bytes;
        uint16_t *const pieces = reinterpret_cast<uint16_t *>(copies), *const codes = reinterpret_cast<uint16_t *>(copies + pl.pieces_bytes);
        float *const sums = reinterpret_cast<float *>(copies + pl.pieces_bytes + pl.codes_bytes);
        float pow2, rest;
        split_scale(s_x, &pow2, &rest);
        auto copy16 = [&](const float *src, uint16_t *dst, int C, int pixels, int ld, float scale, float factor, float *as_rows) {
            const long long blocks = (pixels + 31LL) / 32;
            const dim3 grid((unsigned)(blocks < (1 << 22) ? blocks : (1 << 22)), (unsigned)((ld + 63) / 64), (unsigned)(N < 65535 ? N : 65535));
            adapt::ste_channels_last16_kernel<<<grid, 256, 0, s>>>(src, dst, N, C, pixels, ld, scale, Q, factor, plane, as_rows);
        };
        copy16(dy_dev, pieces, Cout, P, lda, 0.0f, 1.0f, pl.kept_bytes ? rows : nullptr);
        HIP_TRY(hipGetLastError());
        copy16(x_dev, codes, Cin, HW, Cp, s_x, pow2, nullptr);
        HIP_TRY(hipGetLastError());
        adapt::SteDwParams p{};
        p.a = pieces; p.b = codes; p.plane = plane; p.I = Cout; p.R = M; p.lda = lda; p.g = g;
        for (int ky = 0; ky < kh; ky += pl.dw_rows) {
            p.g.kh = kh - ky < pl.dw_rows ? kh - ky : pl.dw_rows;
            p.g.ph = g.ph - ky * g.dh;
            p.J = p.g.kh * kw * Cp;
            launch_ste_dw16(p, w_dev, s_w, Q, rest, dw_dev, s, sums, ky * kw, kh * kw);
            HIP_TRY(hipGetLastError());
        }
    } else if (dw_dev || (dx_dev && !pl.direct)) {
        channels_last(dy_dev, rows, Cout, P, Cout, 0.0f);
        HIP_TRY(hipGetLastError());
    }
    if (dw_dev && !dw16) {  // dw [Cout][K] = inside(w) * rows^T [Cout][M] . fq(col(x)) [M][K], col(x) read from the copy xq
        channels_last(x_dev, xq, Cin, HW, Cp, s_x);
        HIP_TRY(hipGetLastError());
        adapt::SteParams p{};
        p.a = rows; p.b = xq; p.o = w_dev; p.c = dw_dev;
        p.I = Cout; p.R = M; p.lda = Cout;
        p.sb = s_x; p.so = s_w; p.Q = Q;
        p.im2col = 1; p.g = g;
        for (int ky = 0; ky < kh; ky += pl.dw_rows) {
            p.g.kh = kh - ky < pl.dw_rows ? kh - ky : pl.dw_rows;
            p.g.ph = g.ph - ky * g.dh;
            p.J = p.g.kh * kw * Cp;
            launch_ste_gemm(p, true, true, s, partials, ky * kw, kh * kw);          // (both operands lie in the workspace)
            HIP_TRY(hipGetLastError());
        }
    }
    // weights for the input gradient: fp32 [taps][Cout][Cp], or bf16 with Cout rounded up to 32 and the channels to 64, where the
    // workspace holds that (and the padding of narrow layers is not gigabytes, for filters of millions of taps)
    const size_t Op = ((size_t)Cout + 31) / 32 * 32, Cq = ((size_t)Cin + 63) / 64 * 64, wq_bytes = (size_t)kh * kw * Op * Cq * 2;
    if (dx_dev && pl.direct && dx16 && wq_bytes <= pl.total && (wq_bytes <= pl.wp_bytes * 4 || wq_bytes <= ((size_t)64 << 20))) {
        float pow2, rest;
        split_scale(s_w, &pow2, &rest);
        uint4 *const wq = reinterpret_cast<uint4 *>(ws);        // (the weight gradient is done with what it had there)
        adapt::ste_weights16_kernel<<<ew_grid((size_t)kh * kw * (Op / 8) * Cq), 256, 0, s>>>(w_dev, wq, Cout, Cin, (int)Op, (int)Cq, kh * kw, s_w, Q, pow2);
        HIP_TRY(hipGetLastError());
        adapt::SteDx16Params p{};
        p.dy = dy_dev; p.x = x_dev; p.wq = wq; p.dx = dx_dev;
        p.pixels = N * HW; p.og = (int)(Op / 8); p.Cq = (int)Cq; p.so = s_x; p.Q = Q; p.scale = rest; p.g = g;
        adapt::ste_dx16_kernel<<<dim3((unsigned)((p.pixels + 63) / 64), (unsigned)((Cin + 63) / 64)), adapt::STE_THREADS, 0, s>>>(p);
        HIP_TRY(hipGetLastError());
    } else if (dx_dev && pl.direct) {
        const size_t wq_n = (size_t)kh * kw * Cout * Cp;
        adapt::ste_weights_by_tap_kernel<<<ew_grid(wq_n), 256, 0, s>>>(w_dev, wp, Cout, Cin, Cp, kh * kw, s_w, Q);
        HIP_TRY(hipGetLastError());
        adapt::SteDxParams p{};
        p.dy = dy_dev; p.wq = wp; p.x = x_dev; p.dx = dx_dev;
        p.pixels = N * HW; p.Cp = Cp; p.so = s_x; p.Q = Q; p.g = g;
        adapt::ste_dx_kernel<<<dim3((unsigned)((p.pixels + 63) / 64), (unsigned)((Cin + 63) / 64)), adapt::STE_THREADS, 0, s>>>(p);
        HIP_TRY(hipGetLastError());
    } else if (dx_dev) {    // dcol [M][K] = rows [M][Cout] . fq(w) [Cout][K]; dx = inside(x) * the taps of dcol gathered onto the image
        adapt::SteParams p{};
        adapt::ste_taps_first_kernel<<<ew_grid(w_elems), 256, 0, s>>>(w_dev, wp, Cout, Cin, kh * kw);
        HIP_TRY(hipGetLastError());
        p.a = rows; p.b = wp; p.o = nullptr; p.c = dcol;
        p.I = M; p.J = K; p.R = Cout; p.lda = Cout;
        p.sb = s_w; p.so = 1.0f; p.Q = Q;
        launch_ste_gemm(p, false, true, s);
        HIP_TRY(hipGetLastError());
        if (x_elems < 0x7fffffffull && col_n < 0x7fffffffull)
            adapt::ste_col2im_kernel<uint32_t><<<ew_grid(x_elems), 256, 0, s>>>(dcol, x_dev, dx_dev, g, s_x, Q, x_elems);
        else adapt::ste_col2im_kernel<size_t><<<ew_grid(x_elems), 256, 0, s>>>(dcol, x_dev, dx_dev, g, s_x, Q, x_elems);
        HIP_TRY(hipGetLastError());
    }
    if (db_dev) {
        const int Z = N < 16 ? N : 16;
        if ((size_t)Z * Cout <= STE_PARTIAL_FLOATS && Z > 1) {
            adapt::ste_bias_grad_nchw_kernel<<<dim3((unsigned)Cout, (unsigned)Z), 256, 0, s>>>(dy_dev, partials, N, Cout, P);
            adapt::ste_reduce_masked_kernel<<<(unsigned)((Cout + 255) / 256), 256, 0, s>>>(partials, Z, (size_t)Cout, nullptr, 1.0f, Q, db_dev, 0, 0, 0, 0, 0, 1.0f);
        } else {
            adapt::ste_bias_grad_nchw_kernel<<<dim3((unsigned)Cout, 1), 256, 0, s>>>(dy_dev, db_dev, N, Cout, P);
        }
        HIP_TRY(hipGetLastError());
    }
    return ADAPT_OK;
}

int adapt_relu_backward_f32(const float *dy_dev, const float *y_dev, float *dx_dev, size_t n, void *stream) {
    if ((!dy_dev || !y_dev || !dx_dev) && n) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_relu_backward_f32: NULL pointer");
    if (!n) return ADAPT_OK;
    adapt::relu_backward_kernel<<<ew_grid(n), adapt::EW_THREADS, 0, (hipStream_t)stream>>>(dy_dev, y_dev, dx_dev, n);
    HIP_TRY(hipGetLastError());
    return ADAPT_OK;
}

int adapt_sgd_step_f32(float *w_dev, const float *g_dev, size_t n, float lr, void *stream) {
    if ((!w_dev || !g_dev) && n) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_sgd_step_f32: NULL pointer");
    if (w_dev == g_dev && n) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_sgd_step_f32: w_dev and g_dev must differ");
    if (!n) return ADAPT_OK;
    adapt::sgd_kernel<<<ew_grid(n), adapt::EW_THREADS, 0, (hipStream_t)stream>>>(w_dev, g_dev, n, lr);
    HIP_TRY(hipGetLastError());
    return ADAPT_OK;
}

}  // extern "C"
