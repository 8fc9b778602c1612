"""Which tables have a byte form (host code, compiled for the CPU under the undefined-behaviour sanitizer)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_04071_amd", "csrc")

PROGRAM = r'''
#include <cstdio>
#include <vector>
#include "byte_form.hpp"
using namespace adapt_api;

// product of the operands without their low ta / tw bits, plus lo in every entry but the first, hi there
static std::vector<int32_t> table(int bits, int ta, int tw, int lo, int hi) {
    const int n = 1 << bits, H = n / 2;
    std::vector<int32_t> t((size_t)n * n);
    for (int a = -H; a < H; ++a)
        for (int w = -H; w < H; ++w) t[(size_t)(a + H) * n + (w + H)] = (a & -(1 << ta)) * (w & -(1 << tw)) + lo;
    t.front() += hi - lo;       // (its operands have no low bits: no mask takes part of this away)
    return t;
}

int main() {
    int bad = 0;
    for (int bits = 2; bits <= 8; ++bits)
        for (int lo = -200; lo <= 200; lo += 100) {
            const ByteForm f = find_byte_form(bits, table(bits, 0, 0, lo, lo + 255).data());
            bad += !f.found || f.c != lo + 128 || f.am != -1 || f.wm != -1;
        }
    for (int ta = 0; ta <= 3; ++ta)
        for (int tw = 0; tw <= 3; ++tw) {
            const ByteForm f = find_byte_form(8, table(8, ta, tw, -100, 155).data());
            bad += !f.found || f.am != -(1 << ta) || f.wm != -(1 << tw) || f.c != 28;
            bad += find_byte_form(8, table(8, ta, tw, -100, 156).data()).found;         // one more than a byte holds
        }
    bad += find_byte_form(8, table(8, 4, 4, 0, 0).data()).found;
    const std::vector<int32_t> ends = {-32768, 32767, 32767, -32768, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 32767};
    bad += find_byte_form(2, ends.data()).found;
    std::printf("%d\n", bad);
    return bad;
}
'''


def test_byte_form(tmp_path):
    src, exe = tmp_path / "form.cpp", tmp_path / "form"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True,
                   timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
