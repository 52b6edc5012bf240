"""Lanes of a wave that hand data to each other through LDS do it behind wave_lds_exchange(): a bare wave
barrier orders no memory, and whether the compiler then keeps the store before another lane's load
would rest on what it can prove about the two addresses."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0901_3163_amd", "csrc")
FENCED = re.compile(r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*'
                    r'__builtin_amdgcn_wave_barrier\(\);\s*'
                    r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);')


def test_no_wave_barrier_without_fences():
    seen = 0
    for p in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = open(p).read()
        seen += len(FENCED.findall(text))
        assert "__builtin_amdgcn_wave_barrier" not in FENCED.sub("", text), os.path.basename(p)
    assert seen == 1  # the helper
