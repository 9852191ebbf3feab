"""The kernels' reciprocal of a projected depth: the hardware estimate y0 (within
one ulp of 1/b) and one Newton step y0 + y0 (1 - b y0) in fused multiply-adds,
nothing else.  On the CPU: exact from every float within one ulp of 1/b, for
every significand of three binades, but for one start: b all ones and y0 the
neighbour below 1/b.  That it is not the device's estimate is checked on the
device, over every binade of the depths the kernels accept (0.01 m to 2^126)."""
import subprocess

import pytest

SRC = r"""
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
static float u2f(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static uint32_t f2u(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
int main(void) {
    unsigned long long n = 0, bad = 0, one = 0;
    for (int e = -8; e <= 8; e += 8)
        for (uint32_t m = 0; m < (1u << 23); ++m) {
            const float b = u2f(((uint32_t)(127 + e) << 23) | m);
            volatile float unit = 1.0f;
            const float want = unit / b;
            const long double exact = 1.0L / (long double)b;
            const long double ulp = ldexpl(1.0L, ilogbl(exact) - 23);
            for (int d = -2; d <= 2; ++d) {
                const float y0 = u2f(f2u(want) + (uint32_t)d);
                if (fabsl((long double)y0 - exact) > ulp) continue;   /* the estimate's bound */
                ++n;
                if (f2u(fmaf(fmaf(-b, y0, 1.0f), y0, y0)) == f2u(want)) continue;
                if (m == 0x7FFFFFu && (long double)y0 < exact) ++one; else ++bad;
            }
        }
    printf("%llu %llu %llu\n", n, bad, one);
    return 0;
}
"""


def test_step_is_exact_from_every_start_but_one(tmp_path):
    c, exe = tmp_path / "r.c", tmp_path / "r"
    c.write_text(SRC)
    try:
        subprocess.run(["gcc", "-O2", "-ffp-contract=off", "-fno-fast-math", str(c), "-o", str(exe), "-lm"],
                       check=True, capture_output=True)
    except (OSError, subprocess.CalledProcessError) as e:
        pytest.skip(f"no C compiler: {e}")
    n, bad, one = map(int, subprocess.run([str(exe)], capture_output=True, text=True).stdout.split())
    assert n >= 3 * (1 << 23) and bad == 0
    assert one == 3   # once per binade: the device must not start there


@pytest.mark.gpu
@pytest.mark.parametrize("lo,hi", [(-7, 30), (31, 70), (71, 125)])
def test_step_is_exact_on_the_device(lo, hi):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2007_00558_amd as m
    m.lib()
    print(f"[gpu] reciprocal check over the binades {lo}..{hi}", flush=True)
    assert m.check_reciprocal(0, lo, hi) == 0
