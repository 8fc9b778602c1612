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
    int ksplit, gps;            // slices of the inner dimension, steps per slice
    long long clocks;           // estimate for the launch
};

// Clocks of one step of a workgroup: the LDS reads (64 R wave-reads of 1 KB at about 200 B per clock) and, hardly
// overlapped with them, what is brought into the compute unit (the table, R activation words per lane).
inline long long byte_step_clocks(int R, int copy_lines) {
    return 330LL * R + (long long)(copy_lines * 256 + R * 4096) / 50 + 150;
}

inline long long byte_plan_clocks(const BytePlanIn &in, int R, int ksplit, int gps) {
    const long long rows = R >= 4 ? in.rows4 : in.rows2;
    const long long wgs = (rows + 256 * R - 1) / (256 * R) * in.tiles * ksplit;
    const long long rounds = (wgs + in.cu - 1) / in.cu;
    long long c = rounds * (gps * byte_step_clocks(R, in.copy_lines) + 4000);
    // slices: every workgroup stores 16 R KB of sums, the last one of a tile reads the others'
    if (ksplit > 1) c += 3000 + R * 700LL * ksplit;
    return c;
}

inline BytePlan plan_byte(const BytePlanIn &in) {
    BytePlan best{0, 1, in.steps, 0};
    const int Rs[3] = {8, 4, 2};
    for (int R : Rs) {
        const long long rows = R >= 4 ? in.rows4 : in.rows2;
        const long long tiles = (rows + 256 * R - 1) / (256 * R) * in.tiles;
        for (int ks = 1; ks <= 32 && ks <= in.steps; ++ks) {
            const int gps = (in.steps + ks - 1) / ks;
            if (ks > 1 && ((in.steps + gps - 1) / gps != ks || tiles * ks > 2LL * in.cu || tiles > 1024)) continue;
            const long long c = byte_plan_clocks(in, R, ks, gps);
            if (best.R == 0 || c < best.clocks) best = BytePlan{R, ks, gps, c};
        }
    }
    return best;
}

}  // namespace adapt_api
