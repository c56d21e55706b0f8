"""LDS bytes handed between the lanes of one wave: the compiler barrier at the
hand-off has to be a memory operation.  s_waitcnt and wave_barrier are not one
to the compiler, so every wave_barrier in the kernel sources must stand between
a release and an acquire fence."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_20725_amd", "csrc")


def test_every_wave_barrier_is_fenced():
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = open(path).read()
        fenced = re.findall(r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*'
                            r'__builtin_amdgcn_wave_barrier\(\);\s*'
                            r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);', text)
        bare = len(re.findall(r"__builtin_amdgcn_wave_barrier\(", text)) - len(fenced)
        assert bare == 0, "%s: %d wave_barrier calls without fences" % (os.path.basename(path), bare)
        found += len(fenced)
    assert found > 0
