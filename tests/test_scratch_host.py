"""Room for partial sums (host code only: the plan headers, compiled for the CPU).  Smaller products are split more, so what
one product needs is no measure for what a smaller one needs; what a handle reserves has to be."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_04071_amd", "csrc")

PROGRAM = r'''
#include <cstdio>
#include <cstdlib>
#include "byte_plan.hpp"
#include "lines_plan.hpp"
using namespace adapt_api;

static int bad(const char *what, long long a, long long b, long long c, long long d) {
    std::printf("%s: %lld %lld %lld %lld\n", what, a, b, c, d);
    return 1;
}

int main() {
    int shrinks = 0;        // how often a larger product needs less: what makes the reservation necessary
    const int cu = 256;
    const struct { int n_tiles, phases, steps; } byte_shapes[] = {{63, 1, 49}, {32, 1, 32}, {4, 1, 36}, {2, 1, 18}, {1, 1, 9}, {13, 1, 57}, {16, 1, 144},
                                                                 {4, 1, 256}, {1, 4, 16}, {16, 4, 128}, {1, 9, 20}, {1, 64, 3}, {256, 1, 256}, {1, 1, 2040}};
    for (const auto &q : byte_shapes)
        for (int lines = 4; lines <= 256; lines *= 4) {
            const long long launch = (long long)q.n_tiles * (q.phases < 4 ? q.phases : 4);
            BytePlanIn in{0, 0, q.n_tiles * q.phases, q.steps, lines, cu};
            size_t held = 0, before = 0;
            for (long long rows = 1; rows < 300000; rows += rows < 9000 ? 7 : 997) {
                in.rows4 = (rows + 3) / 4 * 4;
                const size_t room = byte_partial_reserve(in, in.rows4, launch);
                if (room < held) return bad("byte: the room shrinks", q.n_tiles, q.steps, lines, rows);
                held = room;
                // image rows of any width: between rows4 / 4 * 2 and rows4 rows in runs of two
                BytePlanIn one = in;
                one.rows4 = 4; one.rows2 = 2;
                const long long one_row = plan_byte(one).clocks;
                for (long long rows2 : {(rows + 1) / 2 * 2, in.rows4, in.rows4 / 2}) {
                    in.rows2 = rows2;
                    const BytePlan pl = plan_byte(in);
                    if (rows2 >= 2 && pl.clocks < one_row) return bad("byte: cheaper than one row", q.n_tiles, q.steps, lines, rows);
                    const size_t need = byte_partial_bytes(pl.R, pl.ksplit, pl.R >= 4 ? in.rows4 : in.rows2, launch);
                    for (bool pack : {false, true})         // (the choice of the kernel may stop at the bound)
                        if (byte_call_clocks_floor(in.steps, lines, rows * 64, pack) > byte_call_clocks(pl, rows * 64, pack))
                            return bad("byte: the floor is above the estimate", q.n_tiles, q.steps, lines, rows);
                    if (need > room) return bad("byte: more than the room", q.n_tiles, q.steps, lines, rows);
                    shrinks += need < before;
                    before = need;
                }
            }
        }
    const struct { int n_tiles, phases, cc, taps, quad_steps; } line_shapes[] = {{8, 1, 8, 9, 36}, {8, 1, 8, 9, 0}, {2, 1, 2, 9, 9}, {25, 1, 13, 9, 0}, {125, 1, 100, 1, 0},
                                                                                 {4, 4, 16, 4, 32}, {1, 4, 4, 1, 0}, {256, 1, 64, 1, 0}, {1, 1, 512, 1, 256}};
    for (const auto &q : line_shapes)
        for (int Wo : {1, 7, 8, 32})
            for (int sw = 1; sw <= 2; ++sw) {
                size_t held = 0;
                for (int lines = 1; lines < 40000; lines += lines < 600 ? 1 : 131) {
                    const int M = lines * Wo;
                    const size_t out = (size_t)M * q.phases * q.n_tiles * 8;        // (the last tile full: the most outputs)
                    const LinesPlan pl = plan_lines(PlanIn{M, q.n_tiles * q.phases, q.cc, q.taps, Wo, sw, q.quad_steps, 8, cu});
                    const size_t room = lines_partial_reserve(cu, out);
                    if (room < held) return bad("lines: the room shrinks", q.n_tiles, q.taps, Wo, M);
                    if (lines_partial_bytes(pl, out) > room) return bad("lines: more than the room", q.n_tiles, q.taps, Wo, M);
                    held = room;
                }
            }
    // the whole-table kernel's estimate for all smaller row counts, and what it says about them
    for (int bits = 2; bits <= 8; bits += 2)
        for (int K : {1, 16, 100, 256, 534, 777, 1024, 4096})
            for (int N : {1, 8, 9, 64, 128, 300, 912, 2048, 4096}) {
                long long most = 0;
                for (int M = 1; M < 4096; M += M < 700 ? 1 : 11) {
                    const long long c = rows_clocks(bits, M, N, K, cu), bound = rows_clocks_up_to(bits, M, N, K, cu);
                    most = c > most ? c : most;
                    if (most > bound) return bad("rows: the bound is below an estimate", bits, K, N, M);
                }
            }
    std::printf("ok %d\n", shrinks);
    return shrinks > 0 ? 0 : 1;
}
'''


def test_room_for_partial_sums_covers_every_smaller_product(tmp_path):
    src = tmp_path / "room.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "room"
    subprocess.run(["g++", "-O1", "-std=c++17", "-include", "initializer_list", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


# The allocation functions against a device with 1000 MB: what the library's pool keeps, and what the default pool holds, is
# in nobody else's way.
MEMORY = r'''
#define __HIP_PLATFORM_AMD__
#include "scratch.hpp"
#include <cstdio>
#include <map>
using namespace adapt_api;

static const size_t MB = (size_t)1 << 20, CAPACITY = 1000 * MB;
static size_t used, kept[2];                    // by allocations; by pools without a user (0: the library's, 1: the default one)
static int pools_made, fail_pools, trims, device;
static bool capturing;
static uint64_t threshold;
static std::map<void *, std::pair<size_t, int>> live;
static char *next_address = (char *)0x1000;

static hipError_t take(void **p, size_t bytes, int pool) {
    const size_t reuse = pool >= 0 ? (kept[pool] < bytes ? kept[pool] : bytes) : 0;
    if (used + kept[0] + kept[1] - reuse + bytes > CAPACITY) return hipErrorOutOfMemory;
    if (pool >= 0) kept[pool] -= reuse;
    used += bytes;
    *p = next_address += 256;
    live[*p] = {bytes, pool};
    return hipSuccess;
}
static void give(void *p) {
    const auto it = live.find(p);
    used -= it->second.first;
    if (it->second.second >= 0) kept[it->second.second] += it->second.first;
    live.erase(it);
}
extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) { return take(p, bytes, -1); }
hipError_t hipMallocAsync(void **p, size_t bytes, hipStream_t) {
    kept[1] = 0;                                // (the default pool gives back at the next synchronisation)
    return take(p, bytes, 1);
}
hipError_t hipMallocFromPoolAsync(void **p, size_t bytes, hipMemPool_t, hipStream_t) { return take(p, bytes, 0); }
hipError_t hipMemPoolCreate(hipMemPool_t *pool, const hipMemPoolProps *) {
    if (fail_pools-- > 0) return hipErrorOutOfMemory;
    *pool = (hipMemPool_t)(size_t)++pools_made;
    return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *v) { threshold = *(uint64_t *)v; return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { ++trims; kept[0] = 0; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) {
    *st = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
}
namespace adapt_api {
bool poison_on() { return false; }
hipError_t dbg_poison(void *, size_t, hipStream_t) { return hipSuccess; }
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
    void *a = nullptr, *b = nullptr, *c = nullptr;
@BODY@
    return 0;
}
'''


def run_memory(tmp_path, body):
    src, exe = tmp_path / "memory.cpp", tmp_path / "memory"
    src.write_text(MEMORY.replace("@BODY@", body))
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-w", "-I", CSRC, "-I", "/opt/rocm/include", str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_scratch_that_is_kept_refuses_nothing(tmp_path):
    run_memory(tmp_path, r'''
    // a handle's allocation finds the memory that the pool keeps
    CHECK(dbg_malloc_async(&a, 250 * MB, nullptr) == hipSuccess);
    give(a);
    CHECK(kept[0] == 250 * MB);
    CHECK(dbg_malloc(&b, 900 * MB) == hipSuccess && trims == 1);
    // too much is still too much
    CHECK(dbg_malloc(&c, 200 * MB) == hipErrorOutOfMemory);
    CHECK(dbg_malloc_async(&c, 200 * MB, nullptr) == hipErrorOutOfMemory);
    give(b);
    // scratch that the library's pool cannot have comes from the default pool
    CHECK(dbg_malloc_async(&a, 200 * MB, nullptr) == hipSuccess);
    give(a);
    kept[1] = 700 * MB;
    CHECK(dbg_malloc_async(&a, 600 * MB, nullptr) == hipSuccess && live[a].second == 1);
    give(a);
    // recorded calls allocate through the default pool
    capturing = true;
    CHECK(dbg_malloc_async(&a, MB, nullptr) == hipSuccess && live[a].second == 1);
''')


def test_a_pool_that_could_not_be_made_is_tried_again(tmp_path):
    run_memory(tmp_path, r'''
    fail_pools = 1;
    CHECK(dbg_malloc_async(&a, MB, nullptr) == hipSuccess && live[a].second == 1 && pools_made == 0);
    CHECK(dbg_malloc_async(&b, MB, nullptr) == hipSuccess && live[b].second == 0 && pools_made == 1);
    CHECK(dbg_malloc_async(&c, MB, nullptr) == hipSuccess && pools_made == 1);
''')


def test_scratch_is_kept_until_the_last_table_of_its_device_is_gone(tmp_path):
    run_memory(tmp_path, r'''
    scratch_table_made(0);
    scratch_table_made(0);
    scratch_table_made(1);
    CHECK(dbg_malloc_async(&a, 100 * MB, nullptr) == hipSuccess);
    give(a);
    scratch_table_gone(1);          // another device's, which has no pool
    scratch_table_gone(0);
    CHECK(trims == 0 && kept[0] == 100 * MB);
    scratch_table_gone(0);
    CHECK(trims == 1 && kept[0] == 0);
    scratch_table_made(0);
    CHECK(dbg_malloc_async(&a, 100 * MB, nullptr) == hipSuccess);
    give(a);
    scratch_table_gone(0);
    CHECK(trims == 2);
''')


def test_scratch_of_a_retraining_step_stays_mapped(tmp_path):
    run_memory(tmp_path, r'''
    // a 1024 x 1024 linear layer on plain weights, 8 bits: its tables and weights, partial sums, the activation copy of 8192 rows
    CHECK(dbg_malloc_async(&a, MB, nullptr) == hipSuccess);
    CHECK(threshold >= 1024ull * 1024 * (256 + 1) + 67 * MB + 8192ull * 1024);
''')
