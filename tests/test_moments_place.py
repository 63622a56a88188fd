"""Where a thread of the int8 moments kernel finds and leaves its numbers (csrc/gvq_moments_place.h), checked on the CPU: the
header is plain C++."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_03617_amd", "csrc")


def test_every_read_is_in_its_block_or_out_of_every_block(tmp_path):
    """All slice lengths the kernel takes, both storages, all panels and threads: an element's 16 reads lie where the element does;
    a column past the slice's end starts past the block's end by its own offset, before the rows' distances are added."""
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(r"""
#include <cstdio>
#include "gvq_moments_place.h"
int main()
{
    for (int d = 65; d <= 1024; ++d)
        for (int bytes = 2; bytes <= 4; bytes += 2) {
            const int np = int_panels(d), pw = 16 * int_tiles(d);
            const unsigned block = 64u * d * bytes;
            if (np * pw < d || (np > 1 ? pw > 96 : pw > 128)) { printf("panels of %d\n", d); return 1; }
            for (int pa = 0; pa < np; ++pa)
                for (int pb = pa; pb < np; ++pb)
                    for (int c = 0; c < (pa == pb ? pw : 2 * pw); ++c)
                        for (int q = 0; q < 4; ++q) {
                            const int e = c >= pw ? pb * pw + c - pw : pa * pw + c;
                            const unsigned p = int_place(int_from(e, q, d, bytes), c, q);
                            if (int_place_column(p) != c || int_place_quarter(p) != q
                                || int_place_lds(p) != (c / 16) * 1024u + q * 256u + (c % 16) * 16u) { printf("item %d %d\n", c, q); return 1; }
                            const unsigned first = int_place_from(p);
                            if (e >= d ? first < block : first != (16u * q * d + e) * bytes || first + 15u * d * bytes + bytes > block) {
                                printf("d = %d, %d bytes: element %d from byte %u of %u\n", d, bytes, e, first, block);
                                return 1;
                            }
                        }
        }
    return 0;
}
""")
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout[-2000:]
