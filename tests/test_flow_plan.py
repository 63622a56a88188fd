"""How the whole-slice codec kernels cut their work (csrc/gvq_flow_plan.h), checked on the CPU: the header is plain C++."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_03617_amd", "csrc")


def _run(tmp_path, body):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <vector>\n#include "gvq_flow_plan.h"\n' + body)
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wno-parentheses", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout[-4000:]
    return out.stdout


def test_no_work_group_gets_much_more_than_its_share(tmp_path):
    """Slices of the busiest work-group against an even share, over numbers of slices, of bases, and rows a tile has room for.
    Rows come in units (a sixteenth of the most a tile holds at worst), a basis ends with a tile that may be short, and a run
    may cost an eighth: the bound is the sum of the three."""
    _run(tmp_path, r"""
int main()
{
    unsigned seed = 1;
    auto rnd = [&]() { return seed = seed * 1664525u + 1013904223u, (seed >> 8); };
    for (int n = 0; n < 4000; ++n) {
        const int unit = 16 << rnd() % 3, most = unit * (1 + rnd() % 10), slots = rnd() % 2 ? 512 : 256;
        const int bases = rnd() % 2 ? 1 : 2 + rnd() % 200;
        const long slices = bases + (long)(slots * (double)most * (0.01 + rnd() % 1000 / 60.0));
        std::vector<int64_t> offs(bases + 1);
        for (int b = 0; b <= bases; ++b) offs[b] = slices * b / bases;
        const int rows = flow_tile_rows(offs.data(), bases, most, unit, slots);
        if (rows < 1 || rows > most || rows % 16) { printf("rows %d of %d\n", rows, most); return 1; }
        const int64_t tiles = flow_tiles(offs.data(), bases, rows);
        const int r = bases > 1 ? flow_run(tiles, slots, rnd() % 2 ? 8 : 4) : 1;
        const int64_t runs = (tiles + r - 1) / r, got = (runs + slots - 1) / slots * r;   // tiles of the busiest
        // the tiles that most rows a tile would give are the least there can be
        const int64_t least = (flow_tiles(offs.data(), bases, most) + slots - 1) / slots;
        if (8 * got > 9 * least) { printf("%ld slices in %d bases, %d rows of %d, run %d: %ld tiles, %ld will do\n", slices, bases, rows, most, r, (long)got, (long)least); return 1; }
        // one basis: no more rows than an even share needs, rounded up to the unit
        if (bases == 1 && rows > unit && (long)(rows - unit) * slots * least >= slices) { printf("%ld slices: %d rows\n", slices, rows); return 1; }
    }
    return 0;
}
""")


def test_short_ranges_reach_the_whole_chip(tmp_path):
    _run(tmp_path, r"""
int main()
{
    // 41667 slices, room for 640 rows a tile: 512 work-groups get one tile each, not 66
    const int64_t offs[2] = {0, 41667};
    const int rows = flow_tile_rows(offs, 1, 640, 64, 512);
    return rows == 128 ? 0 : (printf("%d\n", rows), 1);
}
""")


def test_division_by_multiplication(tmp_path):
    _run(tmp_path, r"""
int main()
{
    for (unsigned n = 1; n < 4096; ++n)
        for (unsigned i = 0; i < 4096; ++i)
            if ((unsigned)(((unsigned long long)(2u * i) * flow_divisor((int)n)) >> 32) != i / n) { printf("%u / %u\n", i, n); return 1; }
    return 0;
}
""")


def test_every_plan_has_an_instance_and_every_instance_a_plan(tmp_path):
    """A plan without an instance would send its shapes to the LDS-tiled kernels without a word (an odd slice length then
    goes number by number); an instance without a plan would be compiled for nothing."""
    _run(tmp_path, r"""
#include <set>
#include <tuple>
int main()
{
    typedef std::tuple<int, int, int, int> key;   // waves, exact, tiles per wave or steps of comps, steps or element tiles
    std::set<key> compress, decompress;
    for (int d = 2; d <= 1024; ++d)
        for (int k = 1; k <= d && k <= 128; ++k) {
            const FlowPlan c = flow_compress_plan(d, k), e = flow_decompress_plan(d, k);
            auto none = [](auto, auto, auto, auto) {};
            // what the kernels are stated to take
            if (!c.waves != (d < 4 || d > 512) || !e.waves != (d > 640 && k > 96 || d > 896 && k > 64)) { printf("no plan: %d %d\n", d, k); return 1; }
            if (c.waves) {
                if (!flow_compress_instance(c, none)) { printf("no compress instance: %d %d\n", d, k); return 1; }
                if (16 * c.ntw * c.wn < k || 32 * c.steps < d || c.rows < 16 || c.rows % 16 || c.lds(c.rows) * c.per_cu > 160 * 1024
                    || c.rows * ((d + 3) / 4) > 64 * c.waves * flow_words(c.waves)) { printf("compress plan: %d %d\n", d, k); return 1; }
                compress.insert(key(c.waves, c.exact, c.ntw, c.steps));
            }
            if (!e.waves) continue;
            if (!flow_decompress_instance(e, none)) { printf("no decompress instance: %d %d\n", d, k); return 1; }
            if (32 * e.kst < k || 16 * e.etw * e.wn < d || e.rows < 16 || e.rows % 16 || e.lds(e.rows) * e.per_cu > 160 * 1024
                || e.rows * ((k + 3) / 4) > 64 * e.waves * 4) { printf("decompress plan: %d %d\n", d, k); return 1; }
            decompress.insert(key(e.waves, e.exact, e.kst, e.etw));
        }
    for (int waves = 4; waves <= 8; waves *= 2)
        for (int exact = 0; exact < 2; ++exact)
            for (int t = 1; t <= 8; ++t)
                for (int s = 1; s <= 16; ++s) {
                    FlowPlan p;
                    p.waves = waves; p.exact = exact; p.ntw = p.kst = t; p.steps = p.etw = s;
                    auto same = [&](auto a, auto b, auto c, auto d) {
                        if (a != t || b != s || c != exact || d != waves) { printf("wrong instance\n"); exit(1); }
                    };
                    if (flow_compress_instance(p, same) != (compress.count(key(waves, exact, t, s)) == 1)
                        || flow_decompress_instance(p, same) != (decompress.count(key(waves, exact, t, s)) == 1)) {
                        printf("instance without a plan: %d waves, exact %d, %d, %d\n", waves, exact, t, s);
                        return 1;
                    }
                }
    return 0;
}
""")


def _shape_lists():
    import importlib.util
    spec = importlib.util.spec_from_file_location("flow_shapes", os.path.join(os.path.dirname(os.path.abspath(__file__)), "test_gpu_flow.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod.INSTANCES, mod.INSTANCE_ELEMENTS


def test_the_gpu_tests_run_every_instance_and_several_tiles_each(tmp_path):
    pytest.importorskip("torch")
    shapes, elements = _shape_lists()
    _run(tmp_path, "static const int shapes[][2] = {" + ", ".join("{%d, %d}" % s for s in shapes) + "};\n"
         + "static const int64_t elements = %d;" % elements + r"""
#include <set>
#include <tuple>
typedef std::tuple<int, int, int, int, int> key;
static void reached(int d, int k, bool bf16, std::set<key>& to, double* least)
{
    const FlowShape s = {d, k, 1, bf16, (elements + d - 1) / d, 256};
    const FlowPlan c = flow_compress_plan(d, k), e = flow_decompress_plan(d, k);
    if (flow_takes_compress(s)) { to.insert(key(0, c.waves, c.exact, c.ntw, c.steps)); if (least && flow_tiles_each(s, c) < *least) *least = flow_tiles_each(s, c); }
    if (flow_takes_decompress(s)) { to.insert(key(1, e.waves, e.exact, e.kst, e.etw)); if (least && flow_tiles_each(s, e) < *least) *least = flow_tiles_each(s, e); }
}
int main()
{
    for (int bf16 = 0; bf16 < 2; ++bf16) {
        std::set<key> all, run;
        double least = 1e9;
        for (int d = 2; d <= 1024; ++d)
            for (int k = 1; k <= d && k <= 128; ++k) reached(d, k, bf16, all, nullptr);
        for (auto& s : shapes) reached(s[0], s[1], bf16, run, &least);
        if (run != all || least < 2.0) { printf("%zu of %zu instances, %.2f tiles per work-group\n", run.size(), all.size(), least); return 1; }
    }
    return 0;
}
""")


def test_which_shapes_come_here(tmp_path):
    """Both sides of every rule, and that a shape which comes here can be run here."""
    _run(tmp_path, r"""
static int bad = 0;
static void want(const char* what, bool got, bool wanted) { if (got != wanted) { printf("%s\n", what); bad = 1; } }
int main()
{
    auto c = [](int d, int k, double elements, int bases = 1, bool bf16 = false) { return flow_takes_compress({d, k, bases, bf16, (int64_t)(elements / d), 256}); };
    auto e = [](int d, int k, double elements, int bases = 1, bool bf16 = false) { return flow_takes_decompress({d, k, bases, bf16, (int64_t)(elements / d), 256}); };
    for (int d = 2; d <= 1024; d += 7)
        for (int k = 1; k <= d && k <= 140; k = k < 8 ? k + 1 : k + 5)
            for (double n : {3e4, 5e5, 3e6, 2.4e7, 1.4e8})
                for (int bases : {1, 24})
                    for (bool bf16 : {false, true}) {
                        auto none = [](auto, auto, auto, auto) {};
                        if (c(d, k, n, bases, bf16) && !flow_compress_instance(flow_compress_plan(d, k), none)) return 1;
                        if (e(d, k, n, bases, bf16) && !flow_decompress_instance(flow_decompress_plan(d, k), none)) return 1;
                    }
    want("whole words", c(100, 25, 6.1e7) && e(100, 25, 6.1e7), true);
    want("short odd slices, hardly any of them", c(13, 3, 5e5) || e(13, 3, 5e5), false);
    want("more of them", c(13, 3, 2e7) && e(13, 3, 2e7), true);
    want("long odd slices, any number", c(201, 50, 3e4) && e(201, 50, 3e4) && c(511, 16, 1e8) && e(1001, 16, 1e8), true);
    want("idle waves", c(400, 16, 2.4e7) || e(400, 16, 2.4e7) || c(200, 16, 1e8, 1, true) || e(160, 16, 1e8, 1, true), false);
    want("idle waves, small", c(400, 16, 5e5) && e(400, 16, 5e5), true);
    want("eight waves", c(400, 100, 1e8), false);
    want("long slices with several bases or bf16", c(400, 60, 1e8, 24) || c(400, 60, 1e8, 1, true), false);
    want("the same, one basis", c(400, 60, 1e8), true);
    want("long slices to bf16", e(400, 60, 1e8, 1, true), false);
    want("the same, comps of no whole words", e(400, 62, 1e8, 1, true) && e(400, 75, 1e8, 1, true), true);
    want("multiples of 256", e(256, 50, 1e8) || e(768, 96, 1e8, 24), false);
    return bad;
}
""")


def test_resident_shapes_with_ragged_comps(tmp_path):
    """Which of them the whole-slice kernels take for compress: measured times of both on either side of every line."""
    _run(tmp_path, r"""
struct Case { int d, k; bool bf16; double million; int per_basis; bool here; };   // elements per basis, 0: one basis
int main()
{
    const Case cases[] = {
        {16, 5, false, 16.1, 0, true}, {16, 5, false, 12, 0, false}, {16, 5, false, 48, 6000, true}, {16, 5, false, 60, 3000, false},
        {16, 11, true, 16.1, 6000, true}, {16, 11, true, 8, 0, false}, {16, 11, true, 60, 3000, false}, {16, 4, false, 60, 0, false},
        {16, 2, true, 8.1, 0, true}, {16, 2, true, 4, 0, false}, {16, 5, true, 60, 3000, true}, {16, 5, true, 60, 1000, false},
        {32, 11, false, 32.1, 0, true}, {32, 11, false, 16, 0, false}, {32, 11, false, 60, 15000, true}, {32, 11, false, 48, 10000, false},
        {32, 11, true, 8, 0, true}, {32, 11, true, 8, 1000000, false}, {32, 11, true, 24, 6000, true}, {32, 3, true, 60, 3000, false},
        {32, 30, false, 32.1, 3000, true}, {32, 30, true, 8, 0, true}, {32, 22, false, 100, 3000, false}, {32, 22, true, 48, 6000, true},
        {64, 19, false, 32.1, 0, true}, {64, 17, false, 60, 0, false}, {64, 17, true, 60, 0, false}, {64, 21, true, 48, 0, true},
        {64, 21, true, 32, 0, false}, {64, 29, true, 32.1, 15000, true}, {64, 29, true, 60, 3000, false}, {64, 29, false, 60, 10000, false},
        {64, 30, true, 60, 0, false}, {128, 13, false, 60, 0, false}};
    for (const Case& c : cases)
        for (int cus : {256, 128}) {   // half the chip: half the size
            const int64_t M = (int64_t)(c.million * 1e6) * cus / 256;
            const int bases = c.per_basis ? (int)(M / c.per_basis) : 1;
            if (flow_takes_compress(FlowShape{c.d, c.k, bases, c.bf16, M / c.d, cus}) != c.here) { printf("d %d k %d %g M\n", c.d, c.k, c.million); return 1; }
        }
    return 0;
}
""")
