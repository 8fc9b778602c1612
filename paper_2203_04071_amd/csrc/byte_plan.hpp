// How a product on the byte kernel (lut_byte.hpp) is spread over the chip: pixels per row slot and slices of the inner
// dimension.  Host code only (no device calls).
#pragma once

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
// 1950 measured, with 128 lines 3770 / 2140 / 1450, with 64 lines 3470 / 1900 / 1140.
inline long long byte_step_clocks(int R, int copy_lines) {
    const double fill = (copy_lines * 256.0 + R * 4096.0) / 54.0;
    return 432LL * R + (long long)(fill * (R == 8 ? 0.225 : (R == 4 ? 0.45 : 0.72)));
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

}  // namespace adapt_api
