// How a product on the columns kernel (lut_cols.hpp) is spread over the chip.  Host code only (no device calls).
#pragma once

namespace adapt_api {

struct ColsPlanIn {
    long long runs;             // runs of four output pixels (image rows rounded up)
    long long n_tiles, pairs;   // tiles of four channels, pairs of inner indices
    int bits, cu;
};

struct ColsPlan {
    int NR;                     // runs per thread (a workgroup owns 4096 NR pixels)
    int ksplit;                 // slices of the inner dimension
    long long clocks;           // estimate for the launch
};

inline long long cols_stages(const ColsPlanIn &in) { return (in.pairs + (1 << (12 - in.bits)) - 1) >> (12 - in.bits); }

// Estimated clocks of a launch, fitted to measured ones (3 x 3, 64 -> 64 channels, one MI355X, whole layers, 40 us of them
// outside this kernel): a stage costs 2300 for its columns (12 bits, 64 pixels: 18 / 36 stages 60 / 80 us) and 85 per pair and
// 256 pixels (32 images of 32 x 32, two runs per thread: 207 us at 12 bits, 131 us at 9); a slice that is joined 1000 per run
// of a thread (one image of 32 x 32 at 10 bits: 16 / 32 slices 42 / 84 us).
inline long long cols_plan_clocks(const ColsPlanIn &in, int NR, int ksplit) {
    const long long tiles = (in.runs + 1024 * NR - 1) / (1024 * NR) * in.n_tiles;
    const long long mine = (cols_stages(in) + ksplit - 1) / ksplit, rounds = (tiles * ksplit + in.cu - 1) / in.cu;
    const long long waves = in.runs < 1024 * NR ? (in.runs + 63) / 64 : 16 * NR;        // runs / 64 that a workgroup has to do
    return rounds * (mine * (2300 + (waves * 85 << (12 - in.bits))) + 6000) + (ksplit > 1 ? 4000 + ksplit * 1000LL * NR : 0);
}

inline ColsPlan plan_cols(const ColsPlanIn &in) {
    ColsPlan best{0, 1, 0};
    const long long stages = cols_stages(in);
    for (int NR = 1; NR <= 2; ++NR)
        for (int ks = 1; ks <= 64 && ks <= stages; ++ks) {
            const long long tiles = (in.runs + 1024 * NR - 1) / (1024 * NR) * in.n_tiles;
            if (ks > 1 && (tiles * ks > 2LL * in.cu)) break;
            const long long c = cols_plan_clocks(in, NR, ks);
            if (best.NR == 0 || c < best.clocks) best = ColsPlan{NR, ks, c};
        }
    return best;
}

}  // namespace adapt_api
