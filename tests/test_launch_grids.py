"""Grids of the launches whose workgroups can pass what one grid dimension holds
(2^32 - 1 threads): grid_of of csrc/lpv_grid.h, compiled for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2407_02068_amd", "csrc")

SIZES = (1, 7, 8, 4800, 2**20 - 1, 2**20, 2**20 + 1, 2**22, 2**23, 2**24 - 8, 2**24, 2**24 + 1,
         # the most workgroups the argument checks let through: the delta curve's 4096
         # block-rows x 65002 vectors and 1024 score workgroups a row, the kept 16 x 16
         # blocks of a 65536 x 65536 weight, and 2^31 rows in tiles of 64 x 1024 runs of 64
         # outputs
         4096 * (65002 + 1024), 2**24, 2**25 * 2**10)


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_grid_of(tmp_path):
    src = tmp_path / "g.cpp"
    src.write_text('#include <stdio.h>\n#include "lpv_grid.h"\nint main() {\n' + "".join(
        '    { lpv::Grid2 g = lpv::grid_of(%dll); printf("%%u %%u\\n", g.x, g.y); }\n' % n
        for n in SIZES) + "}\n")
    exe = str(tmp_path / "g")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True)
    lines = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    assert len(lines) == len(SIZES)
    for n, line in zip(SIZES, lines):
        x, y = map(int, line.split())
        assert x * y >= n > x * (y - 1)          # every piece, no empty row
        assert x * 1024 < 2**32 and y <= 65535   # within the runtime's limits
        assert y == 1 or x % 8 == 0              # the XCD of a workgroup is its number mod 8
        assert y > 1 or x == n
