"""The registers that the launch rules count on, read from the built library: a compute unit's SIMD has 512 vector registers a
lane, in steps of 8, so a kernel of at most 64 runs eight wavefronts on it, one of at most 80 six."""
import os
import re

import pytest

import paper_2109_00170_amd as alcs
from kernel_metadata import LLVM, kernels

pytestmark = pytest.mark.skipif(not (os.path.exists(os.path.join(LLVM, "llvm-readelf")) and os.path.exists(alcs.library_path())),
                                reason="needs the built library and llvm-readelf")

UNITS = ("alcs::", "alcs::fused::", "alcs::bf16io::")


@pytest.mark.parametrize("unit", UNITS)
def test_aligned_resident_kernels_fit_eight_wavefronts(unit):
    # one group per wavefront, groups of at most 4 channels, or 16 with one pixel per lane (launches of several rounds put two
    # workgroups of 16 wavefronts on a compute unit then)
    names = [n for n in kernels() if re.fullmatch(re.escape(unit) + r"k_pw_resident<([124], [124]|16, 1), (true|false), 0, 1>", n)]
    assert len(names) == 13
    for n in names:
        assert kernels()[n].vgprs <= 64 and kernels()[n].scratch == 0, (n, kernels()[n])


@pytest.mark.parametrize("unit", UNITS[:2])
def test_aligned_chunked_kernels(unit):
    names = [n for n in kernels() if n.startswith(unit + "k_pw_chunked<") and n.endswith(", 0>")]
    assert len(names) == 35
    for n in names:
        k = kernels()[n]
        assert k.vgpr_spills == 0 and k.scratch == 0, (n, k)
        if re.search(r"<[12], 1, ", n):  # V = 1, 2, one pixel a lane: what layers of more than 639 channels run
            assert k.vgprs <= 80, (n, k)
