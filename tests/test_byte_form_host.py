"""Which tables have a byte form (host code, compiled for the CPU under the undefined-behaviour sanitizer)."""
import os
import subprocess

import numpy as np
import pytest

from test_gpu_byte import BARE, table as gpu_table

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
    // activations that share a line: as many low bits as the product drops and as change no entry, four lines at least
    for (int bits = 2; bits <= 8; ++bits)
        for (int ta = 1; ta <= 3; ++ta)
            for (int low = 0; low <= ta; ++low) {       // the error takes part of the dropped bits, all but `low` of them
                if (ta >= bits) continue;
                const int n = 1 << bits, H = n / 2;
                std::vector<int32_t> t((size_t)n * n);
                for (int a = 0; a < n; ++a)
                    for (int w = 0; w < n; ++w)
                        t[(size_t)a * n + w] = ((a - H) & -(1 << ta)) * (w - H) + ((a >> ta) == 0 ? (w == 0 ? 127 : (w == H ? -128 : 0)) : ((a & -(1 << low) & ((1 << ta) - 1)) ? 1 : 0));
                const int want = low < bits - 2 ? low : bits - 2;
                ByteForm f = find_byte_form(bits, t.data());
                bad += !f.found || f.am != -(1 << ta) || f.shift != want;
                if (want == 0) continue;
                t[(size_t)n * n - 1] += 1;              // one entry of its own: nothing is shared
                f = find_byte_form(bits, t.data());
                bad += !f.found || f.am != -(1 << ta) || f.shift != 0;
            }
    std::printf("%d\n", bad);
    return bad;
}
'''

SHARED = r'''
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "byte_form.hpp"

int main(int argc, char **argv) {
    const int bits = std::atoi(argv[1]);
    std::vector<int32_t> t((size_t)1 << (2 * bits));
    if (argc != 2 || std::fread(t.data(), 4, t.size(), stdin) != t.size()) return 1;
    const adapt_api::ByteForm f = adapt_api::find_byte_form(bits, t.data());
    std::printf("%d %d\n", (int)f.found, f.shift);
    return 0;
}
'''


def test_byte_form(tmp_path):
    src, exe = tmp_path / "form.cpp", tmp_path / "form"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True,
                   timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.fixture(scope="module")
def shared_lines(tmp_path_factory):
    """(found, shift) of a table, by the library's own search."""
    d = tmp_path_factory.mktemp("form")
    src, exe = d / "shared.cpp", d / "shared"
    src.write_text(SHARED)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True,
                   timeout=120)
    return lambda bits, t: tuple(int(v) for v in subprocess.run([str(exe), str(bits)], input=np.ascontiguousarray(t, np.int32).tobytes(), check=True,
                                                                capture_output=True, timeout=60).stdout.split())


@pytest.mark.parametrize("bits,kind", BARE)
def test_tables_of_the_gpu_tests_share_lines(shared_lines, bits, kind):
    """What the GPU tests of shared lines are named for: that many low bits of an activation are left out of its line."""
    for seed in range(20):
        t = gpu_table(kind, bits, np.random.default_rng(seed))
        assert shared_lines(bits, t) == (1, int(kind[-1]) if kind.startswith("share") else 2)
