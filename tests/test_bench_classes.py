"""CPU checks of the benchmark's launch classes against the kernels of the present sources: names as the
profiler prints them, and the sources whose change makes a class's recorded counters stale.
"""
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2309_03060_amd", "csrc")
sys.path.insert(0, ROOT)
import bench  # noqa: E402

MODE = "void cola::(anonymous namespace)::k_mode<cola::(anonymous namespace)::"


@pytest.mark.parametrize("name,cls", [
    (MODE + "ModeF32, 1, 4, false, false, 1, false>(cola::PassArgs, unsigned int, unsigned int, unsigned int)",
     "contract_cols_f32"),
    (MODE + "ModeF64, 2, 3, true, true, 0, false>(cola::PassArgs, unsigned int, unsigned int, unsigned int)",
     "contract_rows_f64"),
    ("void cola::k_slab23<cola::SlabF64, false>(cola::SlabArgs)", "slab23_f64"),
    ("void cola::(anonymous namespace)::k_fused_cg<1, true>(cola::FusedCgArgs)", "k_fused_cg"),
])
def test_kernel_class(name, cls):
    assert bench.kernel_class(name) == cls


@pytest.mark.parametrize("kind", sorted(bench.KERNEL_SOURCES))
def test_digests_cover_the_headers_of_their_sources(kind):
    """Every header of the package that a class's kernels include belongs to its digest, and the mode
    products that launch_contract dispatches to are part of its class."""
    files = bench.KERNEL_SOURCES[kind]
    for f in files:
        for h in re.findall(r'#include "(\w+\.h)"', open(os.path.join(CSRC, f)).read()):
            if os.path.exists(os.path.join(CSRC, h)) and h not in ("op.h", "trace.h"):
                assert h in files, (kind, f, h)
    if kind == "contract":
        assert "modepass.hip" in files
