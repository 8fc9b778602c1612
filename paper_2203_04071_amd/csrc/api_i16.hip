// C ABI, part 3: operands wider than 8 bits (tables in device memory) and multipliers given as functions.
#include "api_common.hpp"
#include "cols_plan.hpp"
#include "lut_cols.hpp"

using namespace adapt_api;

struct adapt_lut16 {
    int bits;               // 2..12
    int device;
    int32_t *t_dev;         // [w + H][a + H], 2^b x 2^b int32
    int16_t *e_dev;         // columns of the error where the table has the form of lut_cols.hpp, else nullptr
    int e_c;                // the c of that form
};

// looks whether a table has the form of lut_cols.hpp and makes its columns (without memory for them: products gather from t_dev)
static hipError_t make_columns(adapt_lut16 *l) {
    if (l->bits < adapt::COLS_MIN_BITS || l->bits > adapt::COLS_MAX_BITS) return hipSuccess;
    const size_t n = (size_t)1 << l->bits, bytes = n * (n + 1) * sizeof(int16_t);
    int16_t *e_dev = nullptr;
    if (dbg_malloc((void **)&e_dev, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return hipSuccess;
    }
    int32_t *const range_dev = reinterpret_cast<int32_t *>(e_dev);      // (until the columns are written)
    int32_t range[2] = {0, 0};
    adapt::cols_range_init_kernel<<<1, 1, 0, nullptr>>>(range_dev);
    adapt::cols_range_kernel<<<512, 256, 0, nullptr>>>(l->t_dev, l->bits, range_dev);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpy(range, range_dev, sizeof(range), hipMemcpyDeviceToHost);
    const bool fits = e == hipSuccess && (long long)range[1] - range[0] <= 65535;
    if (fits) {
        l->e_c = (int)((uint32_t)range[0] + 32768u);
        adapt::cols_pack_table_kernel<<<ew_grid(n * (n + 1)), 256, 0, nullptr>>>(l->t_dev, e_dev, l->bits, l->e_c);
        e = hipGetLastError();
    }
    if (fits && e == hipSuccess) l->e_dev = e_dev;
    else (void)hipFree(e_dev);
    return e;
}

extern "C" {

/* ------------------------------------------------------------------ operands wider than 8 bits, function multipliers */

int adapt_lut16_create(adapt_lut16 **out, int bits, const int32_t *table_host) {
    if (!out) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_lut16_create: out is NULL");
    *out = nullptr;
    if (!table_host) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_lut16_create: table_host is NULL");
    if (bits < 2 || bits > 12) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_lut16_create: bits=%d not in [2,12]", bits);
    const size_t bytes = ((size_t)1 << (2 * bits)) * sizeof(int32_t);
    adapt_lut16 *l = new (std::nothrow) adapt_lut16();
    if (!l) return fail(ADAPT_ERR_OUT_OF_MEMORY, "adapt_lut16_create: host allocation failed");
    l->bits = bits; l->t_dev = nullptr; l->e_dev = nullptr; l->e_c = 0; l->device = 0;
    int32_t *tmp = nullptr;
    (void)hipGetDevice(&l->device);
    hipError_t e = dbg_malloc((void **)&l->t_dev, bytes);
    if (e == hipSuccess) e = dbg_malloc((void **)&tmp, bytes);
    if (e == hipSuccess) e = hipMemcpy(tmp, table_host, bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        adapt::big_transpose_kernel<<<ew_grid(bytes / 4), 256, 0, nullptr>>>(tmp, l->t_dev, bits);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = make_columns(l);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (tmp) (void)hipFree(tmp);
    if (e != hipSuccess) {
        if (l->t_dev) (void)hipFree(l->t_dev);
        if (l->e_dev) (void)hipFree(l->e_dev);
        delete l;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? ADAPT_ERR_OUT_OF_MEMORY : ADAPT_ERR_HIP, "adapt_lut16_create: %s", hipGetErrorString(e));
    }
    scratch_table_made(l->device);
    *out = l;
    return ADAPT_OK;
}

static int func_args(const char *who, int kind, int param, int bits, int max_bits) {
    if (kind < 0 || kind > 2) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: kind=%d not in [0,2]", who, kind);
    if (bits < 2 || bits > max_bits) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: bits=%d not in [2,%d]", who, bits, max_bits);
    if (param < 0 || param >= bits) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: param=%d not in [0,bits)", who, param);
    return ADAPT_OK;
}

int adapt_lut16_create_from_func(adapt_lut16 **out, int kind, int param, int bits) {
    if (!out) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_lut16_create_from_func: out is NULL");
    *out = nullptr;
    int rc = func_args("adapt_lut16_create_from_func", kind, param, bits, 12);
    if (rc) return rc;
    const size_t entries = (size_t)1 << (2 * bits);
    adapt_lut16 *l = new (std::nothrow) adapt_lut16();
    if (!l) return fail(ADAPT_ERR_OUT_OF_MEMORY, "adapt_lut16_create_from_func: host allocation failed");
    l->bits = bits; l->t_dev = nullptr; l->e_dev = nullptr; l->e_c = 0; l->device = 0;
    (void)hipGetDevice(&l->device);
    hipError_t e = dbg_malloc((void **)&l->t_dev, entries * sizeof(int32_t));
    if (e == hipSuccess) {
        adapt::big_table_from_func_kernel<<<ew_grid(entries), 256, 0, nullptr>>>(l->t_dev, bits, kind, param);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = make_columns(l);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        if (l->t_dev) (void)hipFree(l->t_dev);
        if (l->e_dev) (void)hipFree(l->e_dev);
        delete l;
        (void)hipGetLastError();
        return fail(e == hipErrorOutOfMemory ? ADAPT_ERR_OUT_OF_MEMORY : ADAPT_ERR_HIP, "adapt_lut16_create_from_func: %s",
                    hipGetErrorString(e));
    }
    scratch_table_made(l->device);
    *out = l;
    return ADAPT_OK;
}

int adapt_lut16_destroy(adapt_lut16 *lut) {
    if (!lut) return ADAPT_OK;
    const int device = lut->device;
    if (lut->t_dev) (void)hipFree(lut->t_dev);
    if (lut->e_dev) (void)hipFree(lut->e_dev);
    delete lut;
    scratch_table_gone(device);
    return ADAPT_OK;
}

int adapt_lut16_bits(const adapt_lut16 *lut) {
    if (!lut) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_lut16_bits: lut is NULL");
    return lut->bits;
}

int adapt_quantize_i16_f32(const float *x_dev, int16_t *q_dev, size_t n, float scale, int bits, void *stream) {
    if ((!x_dev || !q_dev) && n) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_quantize_i16_f32: NULL pointer");
    if (bits < 2 || bits > 16) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_quantize_i16_f32: bits=%d not in [2,16]", bits);
    if (!(scale > 0.0f)) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_quantize_i16_f32: scale must be > 0");
    if (n == 0) return ADAPT_OK;
    adapt::quantize_i16_kernel<<<ew_grid(n), 256, 0, (hipStream_t)stream>>>(x_dev, q_dev, n, scale, (float)((1 << (bits - 1)) - 1));
    HIP_TRY(hipGetLastError());
    return ADAPT_OK;
}

}  // extern "C"

namespace {

// whole-layer form: fp32 activations (n_in of them) and the finishing pass of the product kernel
struct BigLayer {
    const float *xf = nullptr;
    size_t n_in = 0;
    float s_x = 1.0f, Q = 0.0f;
    float s_out = 1.0f;
    const float *s_out_vec = nullptr, *bias = nullptr;
    int act = 0;
};

template <int BITS>
void launch_cols_bits(const adapt::ColsParams &p, unsigned grid, int NR, hipStream_t s) {
    if (NR == 2) adapt::lut_cols_kernel<BITS, 2><<<grid, adapt::COLS_THREADS, 0, s>>>(p);
    else adapt::lut_cols_kernel<BITS, 1><<<grid, adapt::COLS_THREADS, 0, s>>>(p);
}

// residue classes of the columns of the activation copy: the horizontal stride, where the window moves at all
int cols_classes(const adapt::BigParams &g) { return g.conv && g.Wo == 1 ? 1 : g.sw; }

// Plan of a product on the columns kernel (g as in run_big); NR == 0 where offsets would not fit 32 bits.  Every product of a
// table with columns goes there: whole layers take 30 to 200 us against 45 to 1730 us of the gathering kernel, from 64 pixels
// and 5 -> 9 channels (37 against 45 us) to 32 images of 32 x 32 pixels and 64 -> 64 channels, 3 x 3 (12 bits: 196 against 1730
// us, 9 bits: 121 against 1160 us).
ColsPlan cols_plan_of(const adapt_lut16 *lut, const adapt::BigParams &g) {
    ColsPlanIn in;
    const int images = g.conv ? g.M / g.HoWo : 1, Wo = g.conv ? g.Wo : g.M;
    in.runs = (long long)(g.conv ? images * (g.HoWo / g.Wo) : 1) * ((Wo + 3) / 4);
    in.n_tiles = (g.N + adapt::COLS_NT - 1) / adapt::COLS_NT;
    in.pairs = (long long)g.taps * ((g.Cin + 1) / 2);
    in.bits = lut->bits; in.cu = device_cus();
    ColsPlan pl = plan_cols(in);
#ifdef ADAPT_TUNING_KNOBS
    if (const char *e = getenv("ADAPT_COLS_PLAN")) {        // "NR,ksplit" (NR 0: the gathering kernel): tuning experiments only
        int NR = 0, ks = 0;
        if (sscanf(e, "%d,%d", &NR, &ks) == 2 && ks >= 1) {
            pl.NR = NR; pl.ksplit = ks;
            if (pl.ksplit > cols_stages(in)) pl.ksplit = (int)cols_stages(in);
        }
    }
#endif
    // 32-bit offsets into the copy and its virtual rows
    const long long Hp = g.H + 2LL * g.ph, Wp = g.W + 2LL * g.pw, sw = cols_classes(g);
    const long long copy = g.conv ? (long long)images * Hp * ((g.Cin + 1) / 2) * ((Wp + sw - 1) / sw * sw) : (long long)((g.Cin + 1) / 2) * ((g.M + 3) / 4 * 4);
    const long long packed = in.n_tiles * (in.pairs + 8) * adapt::COLS_NT;
    if (copy >= 0x1fffff00LL || in.runs * 4 + 8192 >= 0x7fffffffLL || packed >= 0x10000000LL) pl.NR = 0;
    return pl;
}

// the columns kernel (lut_cols.hpp); x: int16 codes, or layer->xf.  no_room: its scratch memory could not be had
int run_cols(const adapt_lut16 *lut, const ColsPlan &pl, const int16_t *x, const int16_t *w, int32_t *out, const adapt::BigParams &g, hipStream_t s,
             const BigLayer *layer, bool *no_room) {
    const int cp = (g.Cin + 1) / 2, KP = 1 << (12 - lut->bits), h = 1 << (lut->bits - 1);
    const int images = g.conv ? g.M / g.HoWo : 1, Ho = g.conv ? g.HoWo / g.Wo : 1, Wo = g.conv ? g.Wo : g.M;
    const int Hp = g.H + 2 * g.ph, Wp = g.W + 2 * g.pw, sw = cols_classes(g), wsub = (Wp + sw - 1) / sw, Mp = (g.M + 3) / 4 * 4;
    adapt::ColsParams p{};
    p.pairs = g.taps * cp; p.cp = cp; p.kw = g.kw; p.stages = (p.pairs + KP - 1) / KP;
    p.N = g.N; p.n_tiles = (g.N + adapt::COLS_NT - 1) / adapt::COLS_NT;
    p.Wo = Wo; p.Wv = (Wo + 3) / 4 * 4; p.Mv = images * Ho * p.Wv;
    const int per_wg = adapt::COLS_THREADS * pl.NR;         // runs
    p.m_tiles = (p.Mv / 4 + per_wg - 1) / per_wg; p.ksplit = pl.ksplit;
    const size_t tiles = (size_t)p.m_tiles * p.n_tiles;
    if (tiles * p.ksplit > 0x7fffffffull) return fail(ADAPT_ERR_UNSUPPORTED, "too many workgroups");
    const size_t copy_words = g.conv ? (size_t)images * Hp * cp * sw * wsub : (size_t)cp * Mp;
    const size_t copy_bytes = (copy_words * 4 + 64 + 255) / 256 * 256, words_bytes = ((size_t)p.n_tiles * p.stages * KP * 32 + 255) / 256 * 256;
    const size_t n_arrived = p.ksplit > 1 ? tiles : 0;
    const size_t part_bytes = p.ksplit > 1 ? tiles * p.ksplit * pl.NR * 4 * adapt::COLS_THREADS * 16 : 0;
    unsigned char *mem = nullptr;
    const hipError_t me = dbg_malloc_async((void **)&mem, copy_bytes + words_bytes + part_bytes + n_arrived * 4, s);
    if (me == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        *no_room = true;
        return ADAPT_OK;
    }
    HIP_TRY(me);
    uint32_t *const xt = reinterpret_cast<uint32_t *>(mem), *const words = reinterpret_cast<uint32_t *>(mem + copy_bytes);
    p.xt = xt; p.words = reinterpret_cast<const uint4 *>(words); p.e = lut->e_dev; p.out = out;
    p.partial = reinterpret_cast<int32_t *>(mem + copy_bytes + words_bytes);
    p.arrived = reinterpret_cast<uint32_t *>(mem + copy_bytes + words_bytes + part_bytes);
    if (g.conv) {
        p.ch_stride = sw * wsub; p.img_stride = Hp * cp * p.ch_stride; p.oy_stride = g.sh * cp * p.ch_stride; p.ky_stride = g.dh * cp * p.ch_stride;
        p.dw = g.dw; p.sw = sw; p.wsub = wsub;
    } else {
        p.ch_stride = Mp; p.dw = 1; p.sw = 1; p.wsub = Mp; p.linear = 1;
    }
    p.out_plane = g.HoWo;
    p.corr = (int)((uint32_t)g.taps * (uint32_t)g.Cin * (uint32_t)lut->e_c);
    p.d_HoWv = fast_div((uint32_t)(Ho * p.Wv)); p.d_Wv = fast_div((uint32_t)p.Wv);
    p.d_cp = fast_div((uint32_t)cp); p.d_kw = fast_div((uint32_t)g.kw); p.d_sw = fast_div((uint32_t)p.sw);
    p.deq = layer ? 1 : 0; p.act = layer ? layer->act : 0; p.scale = layer ? layer->s_out : 1.0f;
    p.scales = layer ? layer->s_out_vec : nullptr; p.bias = layer ? layer->bias : nullptr;
    const size_t pack_n = (size_t)p.n_tiles * p.stages * KP * adapt::COLS_NT, pack_threads = pack_n > n_arrived ? pack_n : n_arrived;
    adapt::cols_pack_words_kernel<<<(unsigned)((pack_threads + 255) / 256), 256, 0, s>>>(w, words, p.arrived, (int)n_arrived, g.N, g.Cin, g.taps, cp, p.pairs,
                                                                                     p.stages * KP, p.n_tiles, lut->bits);
    const adapt::ColsI16 si{x, h, 2 * h - 1};
    const adapt::ColsF32 sf{layer ? layer->xf : nullptr, layer ? layer->s_x : 1.0f, layer ? layer->Q : 0.0f};
    if (g.conv) {
        const unsigned blocks = (unsigned)((copy_words + 255) / 256);
        const adapt::FastDiv a = fast_div((uint32_t)wsub), b = fast_div((uint32_t)sw), c = fast_div((uint32_t)cp), d = fast_div((uint32_t)Hp);
        if (layer) adapt::cols_copy_kernel<<<blocks, 256, 0, s>>>(sf, xt, g.Cin, g.H, g.W, g.ph, g.pw, a, b, c, d, (uint32_t)copy_words);
        else adapt::cols_copy_kernel<<<blocks, 256, 0, s>>>(si, xt, g.Cin, g.H, g.W, g.ph, g.pw, a, b, c, d, (uint32_t)copy_words);
    } else {
        const dim3 grid((unsigned)((g.M + 63) / 64), (unsigned)((cp + 31) / 32));
        if (layer) adapt::cols_rows_kernel<<<grid, 256, 0, s>>>(sf, xt, g.M, g.Cin, cp, Mp);
        else adapt::cols_rows_kernel<<<grid, 256, 0, s>>>(si, xt, g.M, g.Cin, cp, Mp);
    }
    const unsigned grid = (unsigned)(tiles * p.ksplit);
    if (lut->bits == 12) launch_cols_bits<12>(p, grid, pl.NR, s);
    else if (lut->bits == 11) launch_cols_bits<11>(p, grid, pl.NR, s);
    else if (lut->bits == 10) launch_cols_bits<10>(p, grid, pl.NR, s);
    else launch_cols_bits<9>(p, grid, pl.NR, s);
    int rc = ADAPT_OK;
    hipError_t le = hipGetLastError();
    if (le != hipSuccess) rc = fail(ADAPT_ERR_HIP, "columns kernel launch: %s", hipGetErrorString(le));
    hipError_t fe = hipFreeAsync(mem, s);
    if (rc == ADAPT_OK && fe != hipSuccess) rc = fail(ADAPT_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(fe));
    return rc;
}

int run_big(const adapt_lut16 *lut, int kind, int param, const int16_t *x, const int16_t *w, int32_t *out, adapt::BigParams p, hipStream_t s,
            const BigLayer *layer);

// fp32 activations as int16 codes in a stream-ordered temporary, for the kernels that read those
int run_big_quantised(const adapt_lut16 *lut, int kind, int param, const int16_t *w, int32_t *out, const adapt::BigParams &p, hipStream_t s, BigLayer layer) {
    int16_t *q = nullptr;
    HIP_TRY(dbg_malloc_async((void **)&q, layer.n_in * sizeof(int16_t), s));
    adapt::quantize_i16_kernel<<<ew_grid(layer.n_in), 256, 0, s>>>(layer.xf, q, layer.n_in, layer.s_x, layer.Q);
    hipError_t qe = hipGetLastError();
    int rc = qe == hipSuccess ? ADAPT_OK : fail(ADAPT_ERR_HIP, "quantise launch: %s", hipGetErrorString(qe));
    layer.xf = nullptr;
    if (rc == ADAPT_OK) rc = run_big(lut, kind, param, q, w, out, p, s, &layer);
    hipError_t fe = hipFreeAsync(q, s);
    if (rc == ADAPT_OK && fe != hipSuccess) rc = fail(ADAPT_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(fe));
    return rc;
}

// table form: lut != nullptr; function form: lut == nullptr and (kind, param)
int run_big(const adapt_lut16 *lut, int kind, int param, const int16_t *x, const int16_t *w, int32_t *out, adapt::BigParams p, hipStream_t s,
            const BigLayer *layer) {
    if (p.M == 0 || p.N == 0) return ADAPT_OK;
    const bool have_x = x || (layer && layer->xf);
    if (lut && lut->e_dev && have_x && p.taps * (long long)p.Cin > 0) {
        const ColsPlan pl = cols_plan_of(lut, p);
        if (pl.NR > 0) {
            bool no_room = false;
            const int rc = run_cols(lut, pl, x, w, out, p, s, layer && layer->xf ? layer : nullptr, &no_room);
            if (!no_room) return rc;
        }
    }
    if (layer && layer->xf) return run_big_quantised(lut, kind, param, w, out, p, s, *layer);
    p.deq = layer ? 1 : 0; p.act = layer ? layer->act : 0; p.scale = layer ? layer->s_out : 1.0f;
    p.scales = layer ? layer->s_out_vec : nullptr; p.bias = layer ? layer->bias : nullptr;
    const long long K = (long long)p.taps * p.Cin;
    const int NT = lut ? adapt::BIG_NT_TABLE : adapt::BIG_NT_FUNC, threads = lut ? adapt::BIG_THREADS_TABLE : adapt::BIG_THREADS_FUNC;
    p.Npad = (p.N + NT - 1) / NT * NT;
    if (K * p.Npad > 0x7fffffffLL) return fail(ADAPT_ERR_UNSUPPORTED, "weights with more than 2^31-1 packed words");
    const long long wgs = (long long)((p.M + threads - 1) / threads) * (p.Npad / NT);
    if (wgs > 0x7fffffffLL) return fail(ADAPT_ERR_UNSUPPORTED, "too many workgroups");
    int32_t *words = nullptr;
    HIP_TRY(dbg_malloc_async((void **)&words, (size_t)(K > 0 ? K : 1) * p.Npad * sizeof(int32_t), s));
    int rc = ADAPT_OK;
    if (K > 0) {
        const size_t n = (size_t)K * p.Npad;
        adapt::big_pack_weights_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(w, words, (int)K, p.N, p.Npad, p.Cin, p.taps,
                                                                                 lut ? lut->bits : 0);
        hipError_t pe = hipGetLastError();
        if (pe != hipSuccess) rc = fail(ADAPT_ERR_HIP, "big_pack_weights launch: %s", hipGetErrorString(pe));
    }
    p.x = x; p.words = words; p.out = out;
    const dim3 grid((unsigned)wgs);
    if (rc == ADAPT_OK) {
        constexpr int FN = adapt::BIG_NT_FUNC, FT = adapt::BIG_THREADS_FUNC;
        if (lut) {
            adapt::MulTable mt{lut->t_dev, 1 << (lut->bits - 1), (1 << lut->bits) - 1};
            adapt::big_rows_kernel<adapt::MulTable, adapt::BIG_NT_TABLE, adapt::BIG_THREADS_TABLE, true><<<grid, threads, 0, s>>>(p, mt);
        } else if (kind == adapt::FUNC_EXACT) {
            adapt::big_rows_kernel<adapt::MulFunc<adapt::FUNC_EXACT>, FN, FT, false><<<grid, threads, 0, s>>>(p, adapt::MulFunc<adapt::FUNC_EXACT>{param});
        } else if (kind == adapt::FUNC_TRUNC) {
            adapt::big_rows_kernel<adapt::MulFunc<adapt::FUNC_TRUNC>, FN, FT, false><<<grid, threads, 0, s>>>(p, adapt::MulFunc<adapt::FUNC_TRUNC>{param});
        } else {
            adapt::big_rows_kernel<adapt::MulFunc<adapt::FUNC_MITCHELL>, FN, FT, false><<<grid, threads, 0, s>>>(p, adapt::MulFunc<adapt::FUNC_MITCHELL>{param});
        }
        hipError_t le = hipGetLastError();
        if (le != hipSuccess) rc = fail(ADAPT_ERR_HIP, "big_rows launch: %s", hipGetErrorString(le));
    }
    hipError_t fe = hipFreeAsync(words, s);
    if (rc == ADAPT_OK && fe != hipSuccess) rc = fail(ADAPT_ERR_HIP, "hipFreeAsync: %s", hipGetErrorString(fe));
    return rc;
}

int big_linear(const char *who, const adapt_lut16 *lut, int kind, int param, const int16_t *a, const int16_t *w, int32_t *acc, int M,
               int K, int N, void *stream, const BigLayer *layer = nullptr) {
    if (M < 0 || K < 0 || N < 0) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: negative dimension", who);
    if (M == 0 || N == 0) return ADAPT_OK;
    if (!acc || (K > 0 && ((!a && !(layer && layer->xf)) || !w))) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL pointer", who);
    if ((long long)M * N > 0x7fffffffLL || (long long)M * K > 0x7fffffffLL || (long long)N * K > 0x7fffffffLL)
        return fail(ADAPT_ERR_UNSUPPORTED, "%s: tensor with more than 2^31-1 elements", who);
    adapt::BigParams p{};
    p.M = M; p.N = N; p.conv = 0; p.Cin = K; p.taps = 1; p.kw = 1;
    p.H = p.W = p.Wo = p.HoWo = 1; p.sh = p.sw = p.dh = p.dw = 1; p.ph = p.pw = 0;
    p.kstride = 1; p.img_stride = K;
    return run_big(lut, kind, param, a, w, acc, p, (hipStream_t)stream, layer);
}

int big_conv2d(const char *who, const adapt_lut16 *lut, int kind, int param, const int16_t *x, const int16_t *w, int32_t *acc, int N,
               int Cin, int H, int W, int Cout, int kh, int kw, int sh, int sw, int ph, int pw, int dh, int dw, void *stream,
               const BigLayer *layer = nullptr) {
    if (N < 0 || Cin < 1 || H < 1 || W < 1 || Cout < 1 || kh < 1 || kw < 1 || sh < 1 || sw < 1 || ph < 0 || pw < 0 || dh < 1 || dw < 1)
        return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: bad dimension", who);
    const long long eh = (long long)H + 2LL * ph - (long long)dh * (kh - 1) - 1, ew = (long long)W + 2LL * pw - (long long)dw * (kw - 1) - 1;
    if (eh < 0 || ew < 0) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: filter larger than padded input", who);
    const long long Ho = eh / sh + 1, Wo = ew / sw + 1;
    if (N == 0) return ADAPT_OK;
    if ((!x && !(layer && layer->xf)) || !w || !acc) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL pointer", who);
    if ((long long)N * Cout * Ho * Wo > 0x7fffffffLL || (long long)N * Cin * H * W > 0x7fffffffLL ||
        (long long)Cout * Cin * kh * kw > 0x7fffffffLL)
        return fail(ADAPT_ERR_UNSUPPORTED, "%s: tensor with more than 2^31-1 elements", who);
    adapt::BigParams p{};
    p.M = (int)(N * Ho * Wo); p.N = Cout; p.conv = 1; p.Cin = Cin; p.taps = kh * kw; p.kw = kw;
    p.H = H; p.W = W; p.Wo = (int)Wo; p.HoWo = (int)(Ho * Wo);
    p.sh = sh; p.sw = sw; p.ph = ph; p.pw = pw; p.dh = dh; p.dw = dw;
    p.kstride = H * W; p.img_stride = Cin * H * W;
    return run_big(lut, kind, param, x, w, acc, p, (hipStream_t)stream, layer);
}

}  // namespace

extern "C" {

int adapt_approx_linear_i16(const adapt_lut16 *lut, const int16_t *a_dev, const int16_t *w_dev, int32_t *acc_dev, int M, int K, int N,
                            void *stream) {
    if (!lut) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_approx_linear_i16: lut is NULL");
    return big_linear("adapt_approx_linear_i16", lut, 0, 0, a_dev, w_dev, acc_dev, M, K, N, stream);
}

int adapt_approx_linear_func_i16(int kind, int param, int bits, const int16_t *a_dev, const int16_t *w_dev, int32_t *acc_dev, int M,
                                 int K, int N, void *stream) {
    int rc = func_args("adapt_approx_linear_func_i16", kind, param, bits, 16);
    if (rc) return rc;
    return big_linear("adapt_approx_linear_func_i16", nullptr, kind, param, a_dev, w_dev, acc_dev, M, K, N, stream);
}

int adapt_approx_conv2d_i16(const adapt_lut16 *lut, const int16_t *x_dev, const int16_t *w_dev, int32_t *acc_dev, int N, int Cin, int H,
                            int W, int Cout, int kh, int kw, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                            void *stream) {
    if (!lut) return fail(ADAPT_ERR_INVALID_ARGUMENT, "adapt_approx_conv2d_i16: lut is NULL");
    return big_conv2d("adapt_approx_conv2d_i16", lut, 0, 0, x_dev, w_dev, acc_dev, N, Cin, H, W, Cout, kh, kw, stride_h, stride_w, pad_h,
                      pad_w, dil_h, dil_w, stream);
}

int adapt_approx_conv2d_func_i16(int kind, int param, int bits, const int16_t *x_dev, const int16_t *w_dev, int32_t *acc_dev, int N,
                                 int Cin, int H, int W, int Cout, int kh, int kw, int stride_h, int stride_w, int pad_h, int pad_w,
                                 int dil_h, int dil_w, void *stream) {
    int rc = func_args("adapt_approx_conv2d_func_i16", kind, param, bits, 16);
    if (rc) return rc;
    return big_conv2d("adapt_approx_conv2d_func_i16", nullptr, kind, param, x_dev, w_dev, acc_dev, N, Cin, H, W, Cout, kh, kw, stride_h,
                      stride_w, pad_h, pad_w, dil_h, dil_w, stream);
}


/* ------------------------------------------------------------------ whole layers on operands of up to 16 bits */

}  // extern "C"

namespace {

// lut != NULL: table form (its bits); else the function (kind, param) at `bits`.  The product takes the
// fp32 activations and the finishing pass with it.
template <class Product>
int i16_layer(const char *who, const adapt_lut16 *lut, int kind, int param, int bits, const float *x_dev, size_t n_in, float s_x, float s_out,
              const float *s_out_vec_dev, const float *bias_dev, int act, Product product) {
    if (lut) bits = lut->bits;
    else if (int rc = func_args(who, kind, param, bits, 16)) return rc;
    if (act < 0 || act > 2) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: act=%d not in {0, 1, 2}", who, act);
    if (!(s_x > 0.0f)) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: s_x must be > 0", who);
    BigLayer layer;
    layer.s_out = s_out; layer.s_out_vec = s_out_vec_dev; layer.bias = bias_dev; layer.act = act;
    if (n_in == 0) return product(layer);       // (no inner dimension: the sums are 0, the finishing pass still runs)
    if (!x_dev) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: NULL pointer", who);
    layer.xf = x_dev; layer.n_in = n_in; layer.s_x = s_x; layer.Q = (float)((1 << (bits - 1)) - 1);
    return product(layer);
}

}  // namespace

extern "C" {

int adapt_linear_layer_i16_f32(const adapt_lut16 *lut, int kind, int param, int bits, const float *x_dev, const int16_t *w_dev, float *y_dev,
                               int M, int K, int N, float s_x, float s_out, const float *s_out_vec_dev, const float *bias_dev, int act,
                               void *stream) {
    const char *who = "adapt_linear_layer_i16_f32";
    if (M < 0 || K < 0 || N < 0) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: negative dimension", who);
    return i16_layer(who, lut, kind, param, bits, x_dev, (size_t)M * K, s_x, s_out, s_out_vec_dev, bias_dev, act,
                     [&](const BigLayer &layer) {
                         return big_linear(who, lut, kind, param, nullptr, w_dev, reinterpret_cast<int32_t *>(y_dev), M, K, N, stream, &layer);
                     });
}

int adapt_conv2d_layer_i16_f32(const adapt_lut16 *lut, int kind, int param, int bits, const float *x_dev, const int16_t *w_dev, float *y_dev,
                               int N, int Cin, int H, int W, int Cout, int kh, int kw, int stride_h, int stride_w, int pad_h, int pad_w,
                               int dil_h, int dil_w, float s_x, float s_out, const float *s_out_vec_dev, const float *bias_dev, int act,
                               void *stream) {
    const char *who = "adapt_conv2d_layer_i16_f32";
    if (N < 0 || Cin < 1 || H < 1 || W < 1) return fail(ADAPT_ERR_INVALID_ARGUMENT, "%s: bad dimension", who);
    return i16_layer(who, lut, kind, param, bits, x_dev, (size_t)N * Cin * H * W, s_x, s_out, s_out_vec_dev, bias_dev, act,
                     [&](const BigLayer &layer) {
                         if (N == 0) return (int)ADAPT_OK;
                         return big_conv2d(who, lut, kind, param, nullptr, w_dev, reinterpret_cast<int32_t *>(y_dev), N, Cin, H, W, Cout, kh, kw,
                                           stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, stream, &layer);
                     });
}

}  // extern "C"
