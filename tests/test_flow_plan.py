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
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
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
