"""The launch shape of a run as host arithmetic, compiled by itself: for every trajectory count up to the
largest the ABI takes, 2^64 - 1, a block of 1 to 16 waves, a grid of at least one block, and a lane for every
trajectory of a run that is spread."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2410_13683_amd", "csrc")
PROGRAM = r"""
#include "launch_shape.hpp"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv)
{
    for (int i = 1; i + 2 < argc; i += 3) {
        int grid = std::atoi(argv[i + 1]), block = std::atoi(argv[i + 2]);
        fpt::spread_run(std::strtoull(argv[i], nullptr, 10), 256, grid, block);
        std::printf("%d %d\n", grid, block);
    }
}
"""
COUNTS = [1, 63, 64, 65, 64 * 255, 64 * 256, 64 * 256 + 1, 64 * 256 * 15 + 1, 64 * 256 * 16 - 64, 64 * 256 * 16,
          64 * 256 * 16 + 1, 10 ** 9, 2 ** 63, 2 ** 64 - 64, 2 ** 64 - 63, 2 ** 64 - 1]


@pytest.mark.parametrize("full", [(256, 1024), (512, 512), (256, 512), (1, 64)])
def test_shape_holds_every_count(tmp_path, full):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "shape.cpp", tmp_path / "shape"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    args = [str(v) for n in COUNTS for v in (n, *full)]
    out = subprocess.run([str(exe), *args], check=True, capture_output=True, text=True).stdout.split()
    for n, grid, block in zip(COUNTS, map(int, out[::2]), map(int, out[1::2])):
        lanes = full[0] * full[1]
        assert block % 64 == 0 and 64 <= block <= full[1] and 1 <= grid <= full[0], (n, grid, block)
        if n > lanes - 64:
            assert (grid, block) == full
        else:
            assert n <= grid * block < n + 64 * 256 + block
