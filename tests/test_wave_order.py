"""Kernels in which a wave's lanes read LDS that its other lanes wrote, without
a barrier, order the accesses with one sequence (release, wave barrier,
acquire): a release alone does not hold back the loads after it.  Checked on the
sources, since a compiler that happens to keep the order hides its absence."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ORDER = re.compile(r'__device__ __forceinline__ void wave_order\(\)\s*\{\s*'
                   r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*'
                   r'__builtin_amdgcn_wave_barrier\(\);\s*'
                   r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);\s*\}')


def test_wavefront_fences_come_in_order():
    users = 0
    for path in glob.glob(os.path.join(ROOT, "paper_2007_00558_amd", "csrc", "*.hip")):
        with open(path) as f:
            src = f.read()
        rest, n = ORDER.subn("", src)
        assert '"wavefront"' not in rest, path
        users += n * len(re.findall(r"\bwave_order\(\);", rest))
    assert users >= 4
