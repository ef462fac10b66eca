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
