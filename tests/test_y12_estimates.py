"""The estimates that decide the 12-bit coding's rounding (csrc/fvv_y12.h), on
the CPU: the header compiled as C++ with the hardware reciprocal replaced by the
quotient moved by as much as the hardware's may be off (2^-23, either way) and
the conversion instruction by its definition, under a sanitizer that ends the
program at any other conversion out of an integer's range and at an overflow.
Every millimetre value and code, for planes from a float32 step apart to 60
orders of magnitude: where the estimate calls itself sure it is the Eq. 2
sequence's value."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_00558_amd", "csrc")

STUB = r"""
#pragma once
#include <algorithm>
#include <cmath>
#define __host__
#define __device__
#define __forceinline__ inline
using std::fabs; using std::floor; using std::max; using std::min;
extern double rcp_off;
inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x * (1.0 + rcp_off); }
inline double __builtin_amdgcn_fract(double x) { return x - std::floor(x); }
inline int cvt_i32(double v) { return v != v ? 0 : v >= 2147483647.0 ? 2147483647 : v <= -2147483648.0 ? -2147483647 - 1 : (int)v; }
#define asm(...) (i = cvt_i32(v))   /* the one instruction: v_cvt_i32_f64 i, v */
"""

MAIN = r"""
#include "fvv_y12.h"
#include <cstdio>
double rcp_off = 0.0;
int main()
{
    const float planes[][2] = {{0.5f, 10.f}, {1.f, 8.f}, {0.001f, 65.f}, {2.f, 2.0000002f}, {1.f, 1.0005f}, {1.f, 1.00001f},
                               {1e-30f, 1e30f}, {1e-38f, 3e38f}, {60.f, 65.f}, {1e-4f, 1.1e-4f}, {1e6f, 2e6f}};
    long bad = 0, unsure = 0, n = 0;
    for (auto &pl : planes)
        for (double off : {0.0, 0x1p-23, -0x1p-23}) {
            rcp_off = off;
            const y12_planes p = y12_make_planes(pl[0], pl[1]);
            for (uint32_t mm = 0; mm < 65536; ++mm, ++n) {
                bool sure = true;
                const uint32_t c = y12_quantise_est(mm, p, sure);
                if (!sure) ++unsure;
                else if (c != y12_quantise(mm, p)) ++bad;
            }
            for (uint32_t code = 0; code < 4096; ++code, ++n) {
                bool sure = true;
                const uint32_t mm = y12_dequantise_est(code, p, sure);
                if (!sure) ++unsure;
                else if (mm != y12_dequantise(code, p)) ++bad;
            }
        }
    printf("%ld %ld %ld\n", n, bad, unsure);
    return 0;
}
"""


def test_estimates_decide_as_the_divisions(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    src, exe = tmp_path / "y.cpp", tmp_path / "y"
    src.write_text(MAIN)
    try:
        subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-fsanitize=float-cast-overflow",
                        "-fsanitize=signed-integer-overflow", "-fno-sanitize-recover=all", "-I", str(tmp_path), "-I", CSRC,
                        str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    except OSError as e:
        pytest.skip(f"no C++ compiler: {e}")
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-500:]
    n, bad, unsure = map(int, res.stdout.split())
    assert n == 11 * 3 * (65536 + 4096) and bad == 0
    print(unsure, "of", n, "left to the divisions")
