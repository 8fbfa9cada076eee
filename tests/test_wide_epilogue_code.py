"""What the compiler makes of the wide projections' second kernel (no GPU needed: hipcc cross-compiles to gfx950 assembly)."""
import os
import re
import subprocess

from paper_2410_01699_amd import build


# Workgroups have up to 1024 threads: with at most 64 registers two of them share a CU.  The variant for many slices holds 64
# registers of slices alone.
def test_registers(tmp_path):
    out = str(tmp_path / "wide.s")
    subprocess.run(["hipcc", *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, "sjd_gemm_wide.hip"), "-o", out],
                   check=True, capture_output=True)
    regs = {tuple(int(x) for x in m.group(1, 2, 3)): int(m[4]) for m in re.finditer(
        r"\.name:\s+_Z25gemm_wide_epilogue_kernelILi(\d+)ELi(\d+)ELi(\d+)EE\S*\n(?:(?!\.name:).)*?\.vgpr_count:\s+(\d+)", open(out).read(), re.S)}
    assert {k[2] for k in regs} == {4, 16} and len(regs) == 10
    for (epi, pro, slices), count in regs.items():
        assert slices > 4 or count <= 64, (epi, pro, count)
