"""Sizes that a launch and the buffer it writes have to share, on the CPU:
csrc/fvv_unet_sizes.h is host arithmetic, compiled here by itself."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_00558_amd", "csrc")

BIAS_SRC = r"""
#include "fvv_unet_sizes.h"
#include <cstdio>
int main()
{
    /* (rows of channels of a layer's input, channels of a block) of the convolutions that write bias partials */
    const int shapes[][2] = {{32, 32}, {64, 32}, {64, 64}, {128, 32}, {128, 64}, {256, 32}, {256, 64}};
    long n = 0, bad = 0;
    for (auto &sh : shapes)
        for (size_t floats : {(size_t)512, (size_t)768, (size_t)4096, (size_t)100000, (size_t)2048 * 128})
            for (int grid = 8; grid <= 1 << 20; grid = grid < 4096 ? grid + 8 : grid * 2) {
                const int mg = sh[0] / sh[1], g = unet_bias_grid(grid, mg, sh[0], floats);
                const bool fits = (size_t)(g / mg) * sh[0] <= floats;
                const bool whole = g >= 8 && g % 8 == 0 && g <= grid;
                /* no smaller than the buffer asks for */
                const bool most = g == grid || ((size_t)(g / mg) + 8 / mg) * sh[0] > floats;
                ++n;
                bad += !(fits && whole && most);
            }
    printf("%ld %ld\n", n, bad);
    return bad != 0;
}
"""


def run(tmp_path, src):
    c = tmp_path / "s.cpp"
    c.write_text(src)
    exe = tmp_path / "s"
    try:
        subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(c), "-o", str(exe)], check=True,
                       capture_output=True, text=True)
    except OSError as e:
        pytest.skip(f"no C++ compiler: {e}")
    return subprocess.run([str(exe)], capture_output=True, text=True).stdout.split()


def test_bias_partials_fit_their_buffer(tmp_path):
    """Whatever the device's resident blocks, a launch writes no more rows of
    bias partials than its buffer holds, decided before the launch."""
    n, bad = map(int, run(tmp_path, BIAS_SRC))
    assert n > 1000 and bad == 0
