// Which multiplier tables the byte kernel (lut_byte.hpp) serves.  Host code only.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace adapt_api {

// T[a][w] = (a & am) * (w & wm) + c + an error of one byte (found == false: there is no such form)
struct ByteForm {
    bool found = false;
    int c = 0, am = -1, wm = -1;
    int shift = 0;              // low bits of an activation that change no entry at all (no more than am clears): 2^shift rows are the same
};

// table: [a + H][w + H], entries of 16 bits.  The exact product of the operands, or of the operands without their low ta / tw
// bits (multipliers that drop them), has to leave an error that spans at most 255.  The first pair that does is taken.
inline ByteForm find_byte_form(int bits, const int32_t *table) {
    const int n = 1 << bits, H = n >> 1;
    for (int sum = 0; sum <= 6; ++sum)
        for (int ta = sum < 3 ? sum : 3; ta >= 0; --ta) {
            const int tw = sum - ta;
            if (tw > 3) break;
            const int am = -(1 << ta), wm = -(1 << tw);
            int lo = table[0] - (-H & am) * (-H & wm), hi = lo;
            for (int a = -H; a < H && hi - lo <= 255; ++a)
                for (int w = -H; w < H; ++w) {
                    const int e = table[(size_t)(a + H) * n + (w + H)] - (a & am) * (w & wm);
                    lo = e < lo ? e : lo;
                    hi = e > hi ? e : hi;
                }
            if (hi - lo > 255) continue;
            ByteForm f;
            f.found = true;
            f.c = lo + 128; f.am = am; f.wm = wm;
            for (int t = ta < bits - 2 ? ta : bits - 2; t > 0 && f.shift == 0; --t) {       // (four different rows at least)
                bool same = true;
                for (int a = 0; a < n && same; ++a)
                    for (int w = 0; w < n && same; ++w) same = table[(size_t)a * n + w] == table[(size_t)(a & -(1 << t)) * n + w];
                if (same) f.shift = t;
            }
            return f;
        }
    return ByteForm{};
}

}  // namespace adapt_api
