"""CPU checks of rules that the kernel sources keep and no test of values can see."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_03060_amd", "csrc")


def _sources():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))):
        yield os.path.basename(path), open(path).read()


def test_roots_and_reciprocals_are_the_full_ones():
    """No hardware approximation (v_sqrt, v_rcp, v_rsq) in place of a root or a division."""
    for name, text in _sources():
        assert not re.search(r"__builtin_amdgcn_(sqrt|rsq|rcp)", text), name


def test_wave_barriers_order_memory():
    """A wave barrier orders the waves' scheduling, not their LDS accesses: a fence stands on either side."""
    for name, text in _sources():
        lines = text.splitlines()
        for i, line in enumerate(lines):
            if "__builtin_amdgcn_wave_barrier" in line:
                assert "__builtin_amdgcn_fence(__ATOMIC_RELEASE, \"wavefront\")" in lines[i - 1], (name, i + 1)
                assert "__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, \"wavefront\")" in lines[i + 1], (name, i + 1)
