"""What the compiler makes of the fp32 projections (no GPU needed: hipcc cross-compiles to gfx950 assembly).

Their inner loops are latency bound: the rows of a k-step have to be requested together.  Left alone the compiler has put
a wait for everything in flight behind each row's load, and has turned the lane sums into an array indexed by selects.
"""
import os
import re
import subprocess

import pytest

from paper_2410_01699_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "gemm_f32.s")
    subprocess.run(["hipcc", *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, "sjd_gemm.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    return {tuple(int(x) for x in m.group(1, 2, 3)): m.group(4) for m in re.finditer(
        r"\n_Z15gemm_f32_kernelILi(\d+)ELi(\d+)ELb([01])EE[^\n]*:(.*?)\n\.Lfunc_end", text, re.S)}


def test_variants(kernels):
    assert {k[0] for k in kernels} == {8, 16, 32} and len(kernels) == 12


# The first k-step is peeled off: the weights, then the rows 16 at a time, twice, are at most four waits for all that is in
# flight.  (One behind each row's load made 9, 22 and 33 of them in the store variants.)  The lane sums choose rows - 1 times between
# two values and their opposites, for each of one or two features; rotation, gate and normalisation add a few.
def test_rows_are_requested_together(kernels):
    for (rows, epi, norm), code in kernels.items():
        drains, selects = len(re.findall(r"s_waitcnt vmcnt\(0\)", code)), code.count("v_cndmask")
        assert norm or drains <= 6, (rows, epi, drains)          # (normalised rows come from LDS)
        assert selects <= 4 * rows + 40, (rows, epi, norm, selects)
