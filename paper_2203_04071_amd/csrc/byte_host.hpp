// Host side of the byte kernel (lut_byte.hpp): shapes, packing, activation copies and launches.  Included by api_layers.hip
// behind LayerIO and struct adapt_weights.
#pragma once

namespace {

// derived tables of one set of weights in the byte form
struct ByteTables {
    uint4 *dt = nullptr;
    int8_t *wx = nullptr;           // weights of the exact product
    uint32_t *arrived = nullptr;    // arrival counters of split products
};

struct ByteShape {
    int N, Cin, kh, kw;             // filter of one phase
    int phases, st;                 // transposed convolution: st * st phases
    int cg, steps, n_tiles;
    int lbits;                      // 2^lbits lines of a table (operand bits less those that change no entry)
    size_t dt_bytes, wx_bytes;      // all phases together
};

ByteShape byte_shape(int bits, int shift, int N, int Cin, int kh, int kw, int st = 1) {
    ByteShape q;
    q.lbits = bits - shift;
    q.N = N; q.Cin = Cin; q.kh = kh / st; q.kw = kw / st; q.st = st; q.phases = st * st;
    q.cg = (Cin + 3) / 4;
    q.steps = (int)(((long long)q.kh * q.kw * q.cg + 3) / 4);
    q.n_tiles = (N + adapt::BYTE_TILE - 1) / adapt::BYTE_TILE;
    const size_t tables = (size_t)q.phases * q.n_tiles * q.steps;
    q.dt_bytes = tables * ((size_t)adapt::BYTE_LINE << q.lbits);
    q.wx_bytes = tables * adapt::BYTE_TILE * adapt::BYTE_STEP + 1024;       // (a group of four steps may read past the last one)
    return q;
}

int pack_byte(const adapt_lut *lut, const int8_t *w, const ByteShape &q, const ByteTables &t, bool convt, hipStream_t s) {
    adapt::BytePack p;
    p.lut16 = lut->lut16_dev[0]; p.w = w; p.dt = t.dt; p.wx = t.wx; p.arrived = t.arrived;
    p.bits = lut->bits; p.shift = lut->byte.shift; p.N = q.N; p.Cin = q.Cin; p.taps = q.kh * q.kw; p.cg = q.cg; p.n_tiles = q.n_tiles; p.steps = q.steps;
    p.wmode = convt ? 1 : 0; p.kh = q.kh * q.st; p.kw = q.kw * q.st; p.st = q.st;
    p.c = lut->byte.c; p.am = lut->byte.am; p.wm = lut->byte.wm;
    // about eight workgroups per compute unit: enough to hide the latencies, and each stages its band for several tables
    const int bands = ((1 << q.lbits) + adapt::BYTE_PACK_LINES - 1) / adapt::BYTE_PACK_LINES;
    p.tables = q.phases * q.n_tiles * q.steps;
    p.per_wg = (int)((long long)p.tables * bands / (8 * device_cus()));
    p.per_wg = p.per_wg < 1 ? 1 : (p.per_wg > 64 ? 64 : p.per_wg);
    adapt::pack_byte_tables_kernel<<<dim3((unsigned)((p.tables + p.per_wg - 1) / p.per_wg), (unsigned)bands), 256, 0, s>>>(p);
    HIP_TRY(hipGetLastError());
    return ADAPT_OK;
}

bool byte_packable(const ByteShape &q, size_t limit) {
    return q.dt_bytes <= limit && (size_t)q.phases * q.n_tiles * q.steps < 0x7fffffffull && q.steps <= adapt::BYTE_MAX_STEPS;
}

// one-shot use: tables in a stream-ordered temporary
template <typename F>
int with_temp_byte_tables(const adapt_lut *lut, const int8_t *w, const ByteShape &q, bool convt, hipStream_t s, F &&body) {
    const size_t dtb = (q.dt_bytes + 255) / 256 * 256, wxb = (q.wx_bytes + 255) / 256 * 256;
    unsigned char *mem = nullptr;
    HIP_TRY(dbg_malloc_async((void **)&mem, dtb + wxb + adapt::BYTE_MAX_TILES * sizeof(uint32_t), s));
    ByteTables t;
    t.dt = reinterpret_cast<uint4 *>(mem); t.wx = reinterpret_cast<int8_t *>(mem + dtb); t.arrived = reinterpret_cast<uint32_t *>(mem + dtb + wxb);
    int rc = pack_byte(lut, w, q, t, convt, s);
    if (rc == ADAPT_OK) rc = body(t);
    (void)hipFreeAsync(mem, s);
    return rc;
}

// activation side of one product
struct ByteCall {
    int images, Ho, Wo;             // output of one phase (linear: 1, 1, M)
    uint32_t img_stride, oy_stride, ch_stride, ky_stride;       // bytes of the copy
    int dw = 1, sw = 1, wsub;
    bool linear = false;
    std::vector<uint32_t> xt_off{0};                    // per phase
    std::vector<int> oy0{0}, ox0{0};
    int out_step = 1, out_plane = 1, out_w = 0;
    bool nonneg = false;
    const int32_t *zsum = nullptr;
    int cv_Ho = 0, cv_Wo = 0, cv_H = 0, cv_W = 0, cv_kh = 0, cv_kw = 0, cv_s = 1, cv_pad = 0, cv_Ly = 0, cv_Lx = 0;
};

BytePlanIn byte_plan_in(const ByteShape &q, int images, int Ho, int Wo, bool nonneg, int cu = 0) {
    BytePlanIn in;
    in.rows4 = (long long)images * Ho * ((Wo + 3) / 4 * 4); in.rows2 = (long long)images * Ho * ((Wo + 1) / 2 * 2);
    in.tiles = q.n_tiles * q.phases; in.steps = q.steps; in.copy_lines = (1 << q.lbits) >> (nonneg ? 1 : 0); in.cu = cu > 0 ? cu : device_cus();
    return in;
}

BytePlan byte_plan_of(const ByteShape &q, int images, int Ho, int Wo, bool nonneg, int cu = 0) {
    BytePlan pl = plan_byte(byte_plan_in(q, images, Ho, Wo, nonneg, cu));
#ifdef ADAPT_TUNING_KNOBS
    if (const char *e = getenv("ADAPT_BYTE_PLAN")) {        // "R,ksplit": tuning experiments only (not compiled into the product)
        int R = 0, ks = 0;
        if (sscanf(e, "%d,%d", &R, &ks) == 2 && ks >= 1 && ks <= q.steps) {
            pl.R = R; pl.ksplit = ks; pl.even = byte_even_steps(q.steps, ks);
        }
    }
#endif
    return pl;
}

// whether the byte kernel is the better one for M rows of a linear layer; pack: the tables are to be made for this call;
// storage: of the table (1: the whole-table kernel runs twice); *plan: the byte kernel's, where it is
bool byte_pays(const ByteShape &q, int bits, int storage, int M, bool pack, int cu, BytePlan *plan) {
#ifdef ADAPT_TUNING_KNOBS
    if (const char *e = getenv("ADAPT_BYTE_PAYS")) {
        *plan = byte_plan_of(q, 1, 1, M, false, cu);
        return atoi(e) != 0;
    }
#endif
    const long long rows = rows_clocks(bits, M, q.N, q.Cin, cu > 0 ? cu : device_cus()) * (storage + 1);
    if (!byte_beats_rows(byte_call_clocks_floor(q.steps, 1 << q.lbits, q.dt_bytes, pack), rows)) return false;
    *plan = byte_plan_of(q, 1, 1, M, false, cu);
    return byte_beats_rows(byte_call_clocks(*plan, q.dt_bytes, pack), rows);
}
// No linear layer of up to M rows on these (packed) tables runs on the byte kernel: what is cheapest for one row (more rows make every
// plan dearer and rule some out) against the most that any of them takes on the other kernel
bool byte_never_pays(const ByteShape &q, int bits, int storage, int M) {
    const long long one_row = byte_call_clocks(byte_plan_of(q, 1, 1, 1, false), q.dt_bytes, false);
    return !byte_beats_rows(one_row, rows_clocks_up_to(bits, M, q.N, q.Cin, device_cus()) * (storage + 1));
}
bool byte_call_pays(const adapt_lut *lut, const ByteShape &q, int M, bool pack, BytePlan *plan) {
    return byte_pays(q, lut->bits, lut->storage, M, pack, 0, plan);
}

// room for the sums that the slices of a split product leave behind: `bytes` for this one, reserve() for all that are no larger
struct BytePartials {
    const ByteShape &q;
    long long rows;
    size_t bytes;
    BytePartials(const ByteShape &shape, const BytePlan &pl, int images, int Ho, int Wo) : q(shape) {
        const BytePlanIn in = byte_plan_in(q, images, Ho, Wo, false);
        rows = in.rows4;
        bytes = byte_partial_bytes(pl.R, pl.ksplit, pl.R >= 4 ? in.rows4 : in.rows2, launch_tiles());
    }
    long long launch_tiles() const { return (long long)q.n_tiles * (q.phases < 4 ? q.phases : 4); }
    // (whether all activations are known to be >= 0 changes the plan, and is only known call by call)
    size_t reserve() const {
        const BytePlanIn all = byte_plan_in(q, 1, 1, 1, false), half = byte_plan_in(q, 1, 1, 1, true);
        const size_t a = byte_partial_reserve(all, rows, launch_tiles()), h = byte_partial_reserve(half, rows, launch_tiles());
        return a > h ? a : h;
    }
};

// virtual rows are counted in 31 bits (image rows of one pixel count as four)
bool byte_rows_ok(long long image_rows, long long Wo) { return image_rows * ((Wo + 3) / 4 * 4) + 4096 <= 0x7fffffffLL; }

int run_byte(const adapt_lut *lut, const ByteTables &t, const ByteShape &q, const BytePlan &pl, const ByteCall &c, const int8_t *xt, int32_t *partial,
             int32_t *out, hipStream_t s, const LayerIO *io) {
    const int lbits = q.lbits, R = pl.R, V = R < 4 ? R : 4;
    adapt::ByteParams p;
    p.xt = xt; p.out = out; p.partial = partial; p.arrived = t.arrived;
    p.Wo = c.Wo; p.Wv = (c.Wo + V - 1) / V * V;
    const long long Mv = (long long)c.images * c.Ho * p.Wv;
    if (!byte_rows_ok((long long)c.images * c.Ho, c.Wo)) return fail(ADAPT_ERR_UNSUPPORTED, "byte path: more than 2^31 rows");
    p.Mv = (int)Mv;
    p.N = q.N; p.n_tiles = q.n_tiles; p.m_tiles = (int)((Mv + 256 * R - 1) / (256 * R));
    p.cg = q.cg; p.taps = q.kh * q.kw; p.kw = q.kw; p.steps = q.steps; p.ksplit = pl.ksplit; p.even = pl.even;
    p.bits = lbits; p.shift = lut->byte.shift; p.copy_lines = (1 << lbits) >> (c.nonneg ? 1 : 0);
    p.img_stride = c.img_stride; p.oy_stride = c.oy_stride; p.ch_stride = c.ch_stride; p.ky_stride = c.ky_stride; p.dw = c.dw; p.wsub = c.wsub;
    p.amask = (uint32_t)(lut->byte.am & 0xff) * 0x01010101u;
    p.corr = (int)(uint32_t)((long long)q.kh * q.kw * q.Cin * lut->byte.c);
    p.d_HoWv = fast_div((uint32_t)(c.Ho * p.Wv)); p.d_Wv = fast_div((uint32_t)p.Wv);
    p.d_ntiles = fast_div((uint32_t)q.n_tiles); p.d_mtiles = fast_div((uint32_t)p.m_tiles); p.d_ksplit = fast_div((uint32_t)p.ksplit);
    p.d_taps = fast_div((uint32_t)p.taps); p.d_rest = fast_div((uint32_t)((q.cg & 3) ? q.cg & 3 : 1)); p.d_kw = fast_div((uint32_t)q.kw);
    p.d_sw = fast_div((uint32_t)c.sw);
    p.out_step = c.out_step; p.linear = c.linear ? 1 : 0; p.out_plane = c.out_plane; p.out_w = c.out_w;
    const bool deq = io && io->deq;
    p.deq = deq ? 1 : 0; p.act = deq ? io->act : 0; p.scale = deq ? io->s_out : 1.0f;
    p.scales = deq ? io->s_out_vec : nullptr; p.bias = deq ? io->bias : nullptr; p.resid = deq ? io->resid : nullptr;
    p.chain = deq ? io->chain : adapt::ChainOut{};
    p.no_out = out ? 0 : 1;
    if (!out && !p.chain.buf) return fail(ADAPT_ERR_INVALID_ARGUMENT, "byte path: no output");
    p.zsum = c.zsum; p.cv_s = fast_div((uint32_t)c.cv_s);
    p.cv_Ho = c.cv_Ho; p.cv_Wo = c.cv_Wo; p.cv_H = c.cv_H; p.cv_W = c.cv_W; p.cv_kh = c.cv_kh; p.cv_kw = c.cv_kw; p.cv_pad = c.cv_pad;
    p.cv_Ly = c.cv_Ly; p.cv_Lx = c.cv_Lx;
    p.edge_rows = p.edge_cols = 0;
    if (p.zsum && c.cv_H >= q.kh - 1 && c.cv_W >= q.kw - 1) {       // border terms by class: where they fit behind the group offsets
        const long long rows = 2 * q.kh - 1, cols = 2 * q.kw - 1;
        if (rows * cols * adapt::BYTE_TILE + 4LL * q.steps + 8 <= adapt::BYTE_GOFF) { p.edge_rows = (int)rows; p.edge_cols = (int)cols; }
    }
    const int level = lut->byte.am != -1 ? 4 : p.act == 2 ? 3 : (p.zsum ? 2 : (p.chain.buf ? 1 : 0));
    if (p.ksplit > 1 && !partial) return fail(ADAPT_ERR_HIP, "byte path: no room for partial sums");
    const int n_phases = (int)c.xt_off.size();
    const size_t tables = (size_t)q.n_tiles * q.steps;          // of one phase
    for (int first = 0; first < n_phases; first += 4) {         // up to four phases per launch
        p.phases = n_phases - first < 4 ? n_phases - first : 4;
        p.d_phases = fast_div((uint32_t)p.phases);
        p.dt = t.dt + first * tables * (((size_t)adapt::BYTE_LINE << lbits) / 16);
        p.wx = t.wx + first * tables * (adapt::BYTE_TILE * adapt::BYTE_STEP);
        for (int i = 0; i < 4; ++i) {
            const int f = first + (i < p.phases ? i : 0);
            p.xt_off[i] = c.xt_off[f]; p.oy0[i] = c.oy0[f]; p.ox0[i] = c.ox0[f];
        }
        long long grid = (long long)p.m_tiles * q.n_tiles * p.phases * p.ksplit;
        p.units = byte_by_units(q.n_tiles, p.m_tiles, p.phases, p.ksplit, device_cus()) ? q.n_tiles * p.ksplit : 0;
        if (grid > 0x7fffffffLL) return fail(ADAPT_ERR_UNSUPPORTED, "byte path: grid too large");
        if (p.ksplit > 1 && grid / p.ksplit > adapt::BYTE_MAX_TILES) return fail(ADAPT_ERR_HIP, "byte path: more tiles than arrival counters");
        if (p.units) grid = (long long)(p.units + 7) / 8 * 8 * p.m_tiles;
        HIP_TRY(launch_byte(p, (unsigned)grid, R, level, s));
    }
    return ADAPT_OK;
}

// Copies are addressed by unsigned 32-bit byte offsets.  (They hold at most twice what the callers' limit of 2^31 bytes is taken from:
// the channels rounded up to four, not eight, and less than a stride's worth of columns more per row.)
constexpr long long BYTE_MAX_COPY = 0xfffffe00LL;

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

// int8 or fp32 activations -> the copy of byte_copy_kernel
int launch_byte_copy(const LayerIO *io, const int8_t *x, int bits, int shift, int8_t *xt, int N, int C, int H, int W, int ph, int pw, int sw, int wsub,
                     hipStream_t s) {
    const int cg = (C + 3) / 4;
    const size_t total = (size_t)N * (H + 2 * ph) * cg * sw * wsub;
    constexpr int U = 2;
    const unsigned blocks = (unsigned)(((total + U - 1) / U + 255) / 256);
    const adapt::FastDiv dws = fast_div((uint32_t)wsub), dsw = fast_div((uint32_t)sw), dcg = fast_div((uint32_t)cg), dhp = fast_div((uint32_t)(H + 2 * ph));
    const uint32_t mask = (1u << bits) - 1u;
    if (io && io->xf)
        adapt::byte_copy_kernel<adapt::SrcF32, U><<<blocks, 256, 0, s>>>(adapt::SrcF32{io->xf, io->s_x, io->Q, mask, shift}, xt, C, H, W, ph, pw, dws, dsw, dcg, dhp, (uint32_t)total);
    else
        adapt::byte_copy_kernel<adapt::SrcI8, U><<<blocks, 256, 0, s>>>(adapt::SrcI8{x, mask, shift}, xt, C, H, W, ph, pw, dws, dsw, dcg, dhp, (uint32_t)total);
    HIP_TRY(hipGetLastError());
    return ADAPT_OK;
}

// Residue classes of the columns of a convolution's copy: the horizontal stride, where it matters.  (With one output column the window
// never moves; classes of a stride beyond the image would be mostly empty, up to billions of words per row.)
int byte_col_classes(int sw, long long Wo) { return Wo > 1 ? sw : 1; }

// bytes of a convolution's copy (padded image Hp x Wp, sw residue classes), 0 if it does not fit 32-bit offsets
size_t byte_copy_bytes(int N, int Cin, int Hp, int Wp, int sw) {
    const long long n = (long long)N * Hp * ((Cin + 3) / 4) * ((Wp + sw - 1) / sw * sw) * 4;
    return n <= BYTE_MAX_COPY ? align256((size_t)n + 64) : 0;
}

// activation copy of a linear layer
size_t byte_linear_copy_bytes(const ByteShape &q, int M) { return align256((size_t)q.cg * ((M + 3) / 4 * 4) * 4 + 64); }

// linear layer: x [M][K] int8 (a) or fp32 (io->xf); pl: byte_plan_of its shape
int byte_linear(const adapt_lut *lut, const ByteTables &t, const ByteShape &q, const int8_t *a, int32_t *out, int M, hipStream_t s, Workspace *ws,
                const LayerIO *io, const BytePlan &pl) {
    const int Mp = (M + 3) / 4 * 4;
    const size_t copy_bytes = byte_linear_copy_bytes(q, M);
    if ((long long)q.cg * Mp * 4 > BYTE_MAX_COPY) return fail(ADAPT_ERR_UNSUPPORTED, "byte path: tensor with more than 2^31-1 elements");
    const BytePartials sums(q, pl, 1, 1, M);
    unsigned char *mem = nullptr;
    int32_t *partial = nullptr;
    int rc = ws_get(ws, copy_bytes, sums.bytes, sums.rows, [&] { return sums.reserve(); }, s, (void **)&mem, &partial);
    if (rc) return rc;
    int8_t *xt = reinterpret_cast<int8_t *>(mem);
    const dim3 grid((unsigned)((M + 63) / 64), (unsigned)((q.cg + 15) / 16));
    const uint32_t mask = (1u << lut->bits) - 1u;
    if (io && io->xf) adapt::byte_rows_kernel<<<grid, 256, 0, s>>>(adapt::SrcF32{io->xf, io->s_x, io->Q, mask, lut->byte.shift}, xt, M, q.Cin, q.cg, Mp);
    else adapt::byte_rows_kernel<<<grid, 256, 0, s>>>(adapt::SrcI8{a, mask, lut->byte.shift}, xt, M, q.Cin, q.cg, Mp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return ws_put(ws, mem, s, fail(ADAPT_ERR_HIP, "activation copy: %s", hipGetErrorString(e)));
    ByteCall c;
    c.images = 1; c.Ho = 1; c.Wo = M; c.linear = true;
    c.img_stride = 0; c.oy_stride = 0; c.ch_stride = 4u * (uint32_t)Mp; c.ky_stride = 0; c.wsub = Mp;
    rc = run_byte(lut, t, q, pl, c, xt, partial, out, s, io);
    return ws_put(ws, mem, s, rc);
}

// what lies in a prepared handle's workspace, or a fresh copy of x in it
template <typename Copy>
int byte_input(size_t copy_bytes, const BytePartials &sums, Workspace *ws, bool input_ready, hipStream_t s, unsigned char **mem, int32_t **partial, Copy &&copy) {
    if (input_ready) {
        if (!ws || !ws->holds(copy_bytes, sums.rows, sums.bytes))
            return fail(ADAPT_ERR_INVALID_ARGUMENT, "chained layer: the input buffer was not prepared for this geometry");
        *mem = static_cast<unsigned char *>(ws->copy());
        *partial = static_cast<int32_t *>(ws->mem);
        return ADAPT_OK;
    }
    int rc = ws_get(ws, copy_bytes, sums.bytes, sums.rows, [&] { return sums.reserve(); }, s, (void **)mem, partial);
    if (rc) return rc;
    if ((rc = copy(reinterpret_cast<int8_t *>(*mem)))) return ws_put(ws, *mem, s, rc);
    return ADAPT_OK;
}

int byte_conv2d(const adapt_lut *lut, const ByteTables &t, const ByteShape &q, const int8_t *x, int32_t *out, int N, int H, int W, int Ho, int Wo, int sh,
                int sw, int ph, int pw, int dh, int dw, hipStream_t s, Workspace *ws, const LayerIO *io = nullptr, const adapt_weights *wh = nullptr,
                bool input_ready = false) {
    const int csw = byte_col_classes(sw, Wo), Hp = H + 2 * ph, Wp = W + 2 * pw, wsub = (Wp + csw - 1) / csw;
    const size_t copy_bytes = byte_copy_bytes(N, q.Cin, Hp, Wp, csw);
    if (!copy_bytes) return fail(ADAPT_ERR_UNSUPPORTED, "byte path: tensor with more than 2^31-1 elements");
    ByteCall c;
    c.nonneg = input_ready && wh && wh->chain_in.nonneg;
    const BytePlan pl = byte_plan_of(q, N, Ho, Wo, c.nonneg);
    if (!input_ready && wh && wh->chain_in.valid) {     // an ordinary call with another geometry ends the prepared state
        const auto &ci = wh->chain_in;
        if (ci.N != N || ci.H != H || ci.W != W || ci.sh != sh || ci.sw != sw || ci.ph != ph || ci.pw != pw || ci.dh != dh || ci.dw != dw)
            wh->chain_in.valid = false;
        wh->chain_in.nonneg = false;        // (and any other leaves its own copy there)
    }
    const BytePartials sums(q, pl, N, Ho, Wo);
    unsigned char *mem = nullptr;
    int32_t *partial = nullptr;
    int rc = byte_input(copy_bytes, sums, ws, input_ready, s, &mem, &partial, [&](int8_t *xt) {
        return launch_byte_copy(io, x, lut->bits, lut->byte.shift, xt, N, q.Cin, H, W, ph, pw, csw, wsub, s);
    });
    if (rc) return rc;
    const uint32_t row = 4u * (uint32_t)csw * (uint32_t)wsub;      // bytes of one channel group of one padded row
    c.images = N; c.Ho = Ho; c.Wo = Wo;
    const uint32_t line = (uint32_t)q.cg * row;                     // and of a whole padded row
    c.ch_stride = row; c.img_stride = (uint32_t)Hp * line; c.oy_stride = (uint32_t)sh * line; c.ky_stride = (uint32_t)dh * line;
    c.dw = dw; c.sw = csw; c.wsub = wsub;
    c.out_plane = Ho * Wo; c.out_w = Wo;
    rc = run_byte(lut, t, q, pl, c, reinterpret_cast<int8_t *>(mem), partial, out, s, io);
    return ws_put(ws, mem, s, rc);
}

// geometries of the phase form (convt_phases_ok); q: byte_shape with the stride
int byte_conv_transpose2d(const adapt_lut *lut, const ByteTables &t, const ByteShape &q, const int32_t *zsum, const int8_t *x, int32_t *out, int N, int H,
                          int W, int pad, hipStream_t s, Workspace *ws, const LayerIO *io = nullptr, const adapt_weights *wh = nullptr,
                          bool input_ready = false) {
    const int st = q.st, Ty = q.kh, Tx = q.kw, kh = Ty * st, kw = Tx * st;
    const int Hp = H + 2 * (Ty - 1), Wp = W + 2 * (Tx - 1);
    const int Ho = (H - 1) * st - 2 * pad + kh, Wo = (W - 1) * st - 2 * pad + kw;
    const size_t copy_bytes = byte_copy_bytes(N, q.Cin, Hp, Wp, 1);
    if (!copy_bytes) return fail(ADAPT_ERR_UNSUPPORTED, "byte path: tensor with more than 2^31-1 elements");
    ByteCall c;
    c.images = N; c.Ho = Ho / st; c.Wo = Wo / st;
    c.nonneg = input_ready && wh && wh->chain_in.nonneg;
    const BytePlan pl = byte_plan_of(q, N, c.Ho, c.Wo, c.nonneg);
    if (!input_ready && wh) wh->chain_in.valid = false;     // (an ordinary call overwrites a prepared copy)
    const BytePartials sums(q, pl, N, c.Ho, c.Wo);
    unsigned char *mem = nullptr;
    int32_t *partial = nullptr;
    int rc = byte_input(copy_bytes, sums, ws, input_ready, s, &mem, &partial, [&](int8_t *xt) {
        return launch_byte_copy(io, x, lut->bits, lut->byte.shift, xt, N, q.Cin, H, W, Ty - 1, Tx - 1, 1, Wp, s);
    });
    if (rc) return rc;
    const uint32_t row = 4u * (uint32_t)Wp, line = (uint32_t)q.cg * row;
    c.ch_stride = row; c.img_stride = (uint32_t)Hp * line; c.oy_stride = c.ky_stride = line; c.wsub = Wp;
    c.out_step = st; c.out_plane = Ho * Wo; c.out_w = Wo;
    c.xt_off.clear(); c.oy0.clear(); c.ox0.clear();
    for (int ry = 0; ry < st; ++ry)
        for (int rx = 0; rx < st; ++rx) {
            // first window of the phase: see lines_conv_transpose2d
            const int qy0 = pad > ry ? (pad - ry + st - 1) / st : 0, qx0 = pad > rx ? (pad - rx + st - 1) / st : 0;
            c.xt_off.push_back((uint32_t)qy0 * c.oy_stride + (uint32_t)qx0 * 4u);
            c.oy0.push_back(st * qy0 + ry - pad);
            c.ox0.push_back(st * qx0 + rx - pad);
        }
    const int Ly = kh - st - pad > 0 ? kh - st - pad : 0, Lx = kw - st - pad > 0 ? kw - st - pad : 0;
    if (Ly > 0 || Lx > 0) c.zsum = zsum;
    c.cv_Ho = Ho; c.cv_Wo = Wo; c.cv_H = H; c.cv_W = W; c.cv_kh = kh; c.cv_kw = kw; c.cv_s = st; c.cv_pad = pad; c.cv_Ly = Ly; c.cv_Lx = Lx;
    rc = run_byte(lut, t, q, pl, c, reinterpret_cast<int8_t *>(mem), partial, out, s, io);
    return ws_put(ws, mem, s, rc);
}

}  // namespace
