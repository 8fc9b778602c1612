// How a product on the byte kernel (lut_byte.hpp) is spread over the chip: pixels per row slot and slices of the inner
// dimension.  Host code only (no device calls).
#pragma once
#include <stddef.h>

namespace adapt_api {

struct BytePlanIn {
    long long rows4, rows2;     // virtual rows with image rows rounded up to runs of 4 / of 2 pixels (all images, one phase)
    int tiles;                  // tiles of 16 output channels x phases
    int steps;                  // steps of 16 inner indices
    int copy_lines;             // table lines a step copies (2^bits, or half of it)
    int cu;
};

struct BytePlan {
    int R;                      // pixels per row slot (a workgroup owns 256 R)
    int ksplit, even;           // slices of the inner dimension: slice i ends at step (i + 1) even / ksplit, the last one at the end
    long long clocks;           // estimate for the launch
};

// The last slice is longer than the others by about the time they take to leave their sums (see lut_byte.hpp)
inline int byte_even_steps(int steps, int ksplit) {
    const int slice = steps / ksplit;
    return ksplit > 1 ? steps - (slice >= 12 ? 3 : (slice >= 6 ? 2 : (slice >= 3 ? 1 : 0))) : steps;
}
inline int byte_last_slice(int steps, int ksplit) { return steps - (int)((long long)(ksplit - 1) * byte_even_steps(steps, ksplit) / ksplit); }

// Estimated clocks of a launch, fitted to measured ones (3 x 3, 64 -> 64 channels, 32 images of 32 x 32, and 64 x 64 pixels of
// one image; one MI355X).  Per step of a workgroup 432 R for the reads and the matrix instructions behind them, and the part
// of the copies (table and activations, 54 B per clock) that these do not hide: R = 8 / 4 / 2 with 256 lines 3810 / 2420 /
// 1950 measured, with 128 lines 3770 / 2140 / 1450, with 64 lines 3470 / 1900 / 1140.  (The loop has become faster since: 2930 / 2480 / 2060,
// 2790 / 1780 / 1170, 2800 / 1270 / 950 on a part of the chip, less when all of it runs.  Of 19 layers under all plans, the plans chosen
// by these numbers are the best or within 4 % of it but for one, those chosen by the new ones lose up to 20 %.)
inline long long byte_step_clocks(int R, int copy_lines) {
    const double fill = (copy_lines * 256.0 + R * 4096.0) / 54.0;
    return 432LL * R + (long long)(fill * (R == 8 ? 0.225 : (R == 4 ? 0.45 : 0.72)));
}

// Whether the workgroups of a launch go to the XCDs by units (see lut_byte_kernel): where every XCD then gets as few workgroups as it would
// get otherwise, where the row tiles of a channel tile do not share an XCD anyway, and where the tables that an XCD need not fetch weigh more than the
// activations of all row tiles that it then does.  Speed by units against channel tile fastest, mean (extremes), 8 bits:
//     up to 7 row tiles: 3 - 8 channel tiles 1.02 (0.97 - 1.20), 13 - 15 1.14 (0.99 - 1.53), 33 and 50 1.14 (0.98 - 1.58)
//     8 - 13 row tiles: 9 - 12 channel tiles 1.00 (0.95 - 1.17), 13 - 15 1.06 (0.97 - 1.24), 33 and 50 1.45 (1.36 - 1.57)
//     14 - 16: 9 - 12 0.96 (0.87 - 1.10), 13 - 15 0.98 (0.94 - 1.04), 33 and 50 1.14 (1.01 - 1.27)
//     17 - 32: 3 0.89 (0.82 - 0.96), 13 - 15 0.97 (0.89 - 1.05), 20 and 22 0.97 (0.89 - 1.06), 33 and 50 1.12 (1.00 - 1.29)
// (7 bits likewise, with half of the gains)
inline bool byte_by_units(int n_tiles, int m_tiles, int phases, int ksplit, int cu) {
    if (phases != 1 || m_tiles == 1 || n_tiles % 8 == 0 || 8 % n_tiles == 0 || cu % 8 != 0) return false;
    if (n_tiles <= 32 && m_tiles > (n_tiles < 13 ? 7 : 13)) return false;
    const long long units = (long long)n_tiles * ksplit, per_xcd = (units + 7) / 8 * m_tiles, wgs = units * m_tiles;
    return (per_xcd + cu / 8 - 1) / (cu / 8) <= (wgs + cu - 1) / cu && per_xcd * 8 <= 0x7fffffffLL;
}

inline long long byte_plan_clocks(const BytePlanIn &in, int R, int ksplit) {
    const long long rows = R >= 4 ? in.rows4 : in.rows2;
    const long long wgs = (rows + 256 * R - 1) / (256 * R) * in.tiles * ksplit;
    const long long rounds = (wgs + in.cu - 1) / in.cu;
    // start (first table, group offsets) and end of a workgroup: 8000 + 350 R
    long long c = rounds * (byte_last_slice(in.steps, ksplit) * byte_step_clocks(R, in.copy_lines) + 8000 + 350 * R);
    // slices: the workgroup that finishes a tile looks for the others (4000) and reads 16 R KB from each (550 R, less if few of
    // the rows exist)
    if (ksplit > 1) c += 4000 + (ksplit - 1) * (550LL * R * (rows < 256 * R ? rows : 256 * R) / (256 * R) + 150);
    return c;
}

inline BytePlan plan_byte(const BytePlanIn &in) {
    BytePlan best{0, 1, in.steps, 0};
    const int Rs[3] = {8, 4, 2};
    for (int R : Rs) {
        const long long rows = R >= 4 ? in.rows4 : in.rows2;
        const long long tiles = (rows + 256 * R - 1) / (256 * R) * in.tiles;
        for (int ks = 1; ks <= 32 && ks <= in.steps; ++ks) {
            if (ks > 1 && (tiles * ks > 2LL * in.cu || tiles > 1024)) break;
            const long long c = byte_plan_clocks(in, R, ks);
            if (best.R == 0 || c < best.clocks) best = BytePlan{R, ks, byte_even_steps(in.steps, ks), c};
        }
    }
    return best;
}

// Bytes of the sums that the slices of a split product leave behind: 16 R KB per workgroup (launch_tiles: channel tiles x phases
// of one launch).
inline size_t byte_partial_bytes(int R, int ksplit, long long rows, long long launch_tiles) {
    return ksplit > 1 ? (size_t)((rows + 256 * R - 1) / (256 * R) * launch_tiles * ksplit) * R * 16384 : 0;
}

// The most that any product of up to `rows4` virtual rows needs of them, whatever its plan.  A plan splits the inner dimension
// where there are few tiles, so fewer rows often need more (8 bits, K = 777, N = 999: 4.7 MB for 6000 rows, 36 MB for
// 4000): a buffer that has to last for all smaller products is sized by this bound, which only grows with the rows.  For every R and
// number of row tiles t: the slices that the estimate chooses there.  One row tile: the fewer rows, the cheaper a slice, so those of
// one row; with 8 or 4 pixels per row slot only from half a tile on (below, half as many pixels make one tile too, and are cheaper).
// in: tiles, steps, copy_lines and cu count.
inline size_t byte_partial_reserve(BytePlanIn in, long long rows4, long long launch_tiles) {
    size_t most = 0;
    for (int R = 2; R <= 8; R *= 2)
        for (long long t = 1; t * in.tiles <= in.cu && t * in.tiles <= 1024; ++t) {
            if (rows4 <= (t > 1 ? (t - 1) * 256 * R : (R > 2 ? 128 * R : 0))) break;
            in.rows4 = in.rows2 = t > 1 ? t * 256 * R : 1;
            int slices = 1;
            long long least = 0;
            for (int ks = 1; ks <= 32 && ks <= in.steps && t * in.tiles * ks <= 2LL * in.cu; ++ks) {
                const long long c = byte_plan_clocks(in, R, ks);
                if (ks == 1 || c < least) { least = c; slices = ks; }
            }
            const size_t bytes = byte_partial_bytes(R, slices, in.rows4, launch_tiles);
            most = bytes > most ? bytes : most;
        }
    return most;
}

// A product on the whole-table kernel (lut_rows.hpp), as run_rows lays it out
struct RowsShape {
    int NT, MT;                 // channels and rows per workgroup
};
inline RowsShape rows_shape(long long M, long long N, long long K, int groups, int cu) {
    // prefer 16 outputs per lane; shrink the tile until the grid covers the chip
    RowsShape r{16, 1024};
    auto wgs = [&] { return (M + r.MT - 1) / r.MT * ((N + r.NT - 1) / r.NT) * groups; };
    while (r.MT > 64 && (r.MT / 2 >= M || (wgs() < cu && K / (1024 / (r.MT / 2)) >= 16))) r.MT /= 2;
    if ((wgs() < cu && N > 8) || (groups > 1 && N <= 8)) r.NT = 8;
    return r;
}

// Estimated clocks of a linear layer on it (one MI355X, 2.2 GHz): 16 waves of ceil(K / slices) NT reads of LDS at 4.3 clocks each where
// activations come as whole words, 8 where they come byte by byte (K no multiple of 4), behind the copy of the
// table into LDS at 10 B per clock.  Measured 777 x 999 x 1024 rows, 8 bits: 190 us (196 estimated); 4096 x 4096 x 4000 rows, 8, 7 and 6 bits: 11.3, 8.1 and
// 5.3 ms (8.2: the clocks of a read are about 6, 4.5 and 3.2 where many rows share a table; see byte_beats_rows for what the choice loses).
inline long long rows_clocks_in(const RowsShape &r, int bits, long long M, long long N, long long K, int cu) {
    const long long slices = 1024 / r.MT, kc = (K + slices - 1) / slices, wgs = (M + r.MT - 1) / r.MT * ((N + r.NT - 1) / r.NT);
    const long long table = ((1LL << bits) * ((1LL << bits) + 2)) * 2, red = slices > 1 ? 4096LL * r.NT : 0;
    const int per_cu = (table > red ? table : red) <= 80 * 1024 ? 2 : 1;
    const long long rounds = wgs <= cu ? 1 : (wgs + cu * per_cu - 1) / (cu * per_cu) * per_cu;
    return rounds * ((long long)(16 * kc * r.NT * (K % 4 == 0 && kc % 4 == 0 ? 4.3 : 8.0)) + table / 10) + 4000;
}

inline long long rows_clocks(int bits, long long M, long long N, long long K, int cu) { return rows_clocks_in(rows_shape(M, N, K, 1, cu), bits, M, N, K, cu); }

// A bound above that estimate for every number of rows up to M: in a given tile shape more rows only take longer, so the longest of
// the shapes that any of them can get (64 rows per workgroup, or less than twice its rows; 16 channels only where the grid then covers
// the chip)
inline long long rows_clocks_up_to(int bits, long long M, long long N, long long K, int cu) {
    long long most = 0;
    for (int MT = 64; MT <= 1024 && (MT == 64 || MT / 2 < M); MT *= 2)
        for (int NT = 8; NT <= 16; NT *= 2) {
            if (NT == 16 && N > 8 && (M + MT - 1) / MT * ((N + 15) / 16) < cu) continue;
            const long long c = rows_clocks_in(RowsShape{NT, MT}, bits, M, N, K, cu);
            most = c > most ? c : most;
        }
    return most;
}

// Estimated clocks of a whole call on the byte kernel: the launch, or the stream of its tables where that takes longer (2300 B
// per clock, and up to 40000 clocks more where they come from HBM: 202 MB 39 us in the caches and 75 us behind other
// work), and the activation copy; pack: with tables made for this call
// (1400 B per clock behind one more allocation and launch).
inline long long byte_call_clocks(const BytePlan &pl, size_t table_bytes, bool pack) {
    const long long stream = (long long)(table_bytes / 2300), first = (long long)((table_bytes < 200000000 ? table_bytes : 200000000) / 5000);
    return (pl.clocks > stream ? pl.clocks : stream) + first + 11000 + (pack ? 30000 + (long long)(table_bytes / 1400) : 0);
}

// A bound below that estimate, whatever the plan, without a search for one (64 rows, K = 256, N = 128: 0.01 instead of 0.65 us on the
// host, of a call of 20 us).
inline long long byte_call_clocks_floor(int steps, int copy_lines, size_t table_bytes, bool pack) {
    const int slice = steps < 32 ? 1 : steps / 32;
    return byte_call_clocks(BytePlan{2, 1, 0, slice * byte_step_clocks(2, copy_lines) + 8000 + 2 * 350}, table_bytes, pack);
}

// Where tables of the byte form exist (or are to be made), the byte kernel is taken if its estimate times 1.2 is below that of
// the whole-table kernel.  Both estimates were fitted to earlier forms of the kernels, which have become faster by different factors since.
// Measured both ways on the present ones (330 packed layers of 1 to 4095 rows, K from 16 and N from 8 to 4096, 6 to 8 bits): 2.7 % slower in the mean
// than with the better kernel each time.  14 of them lose more than 20 % and 3 us, most on the whole-table kernel with slices that are no whole
// words, whose loop takes up to twice the 8 clocks assumed; e.g. (whole table / byte kernel) 8 bits, 195 rows, K = 2529, N = 391: 147 / 53 us, taken: whole
// table.  8 bits, K = 777, N = 999: 256 rows 58 / 39 us (whole table), 1024 rows 190 / 50 (byte); K = N = 4096: 256 rows 715 / 733 (whole table), 1024 rows
// 2842 / 749 (byte).  Tables made for the call: 8 bits, K = N = 1024, 1024 rows 197 / 153 (whole table).
inline bool byte_beats_rows(long long byte_clk, long long rows_clk) { return byte_clk + byte_clk / 5 < rows_clk; }

}  // namespace adapt_api
