"""What the compiler makes of the window attention (no GPU needed: hipcc cross-compiles to gfx950 assembly).

Each kernel comes twice, with non-temporal loads of keys and values (NT) and with plain ones.  Of two loads that differ only in that
hint the compiler makes one, and drops the hint, as soon as it meets both behind one condition.
"""
import os
import re
import subprocess

from paper_2410_01699_amd import build


def test_loads_of_the_cache(tmp_path):
    out = str(tmp_path / "attention.s")
    subprocess.run(["hipcc", *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, "sjd_attention.hip"), "-o", out],
                   check=True, capture_output=True)
    found = 0
    for m in re.finditer(r"\n_Z17attn_split_kernelILi(\d+)ELi(\d)ELi(\d)ELb([01])EE[^\n]*:(.*?)\n\.Lfunc_end", open(out).read(), re.S):
        hd, mt, waves, nt, code = int(m[1]), int(m[2]), int(m[3]), m[4] == "1", m[5]
        loads = re.findall(r"global_load_dwordx4 [^\n]*", code)
        hinted = [x for x in loads if x.rstrip().endswith(" nt")]
        # a block: 2 halves x hd / 32 k-steps of K and hd / 16 tiles of V, two planes each, for the first block and for the next
        block = 2 * (2 * hd // 32 + hd // 16)
        assert len(hinted) == (2 * block if nt else 0), (hd, mt, waves, nt)
        assert len(loads) >= 2 * block
        found += 1
    assert found == 16
