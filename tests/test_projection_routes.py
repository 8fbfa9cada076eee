"""Which kernel a bf16 projection runs on (no GPU needed: the rules are host code behind sjd_gemm_plan)."""
import pytest

from paper_2410_01699_amd import binding as B


# A sliced launch has one counter per column of workgroups, 1024 of them; a projection with more columns goes elsewhere.
@pytest.mark.parametrize("M,N,K", [(40, 65552, 512), (64, 65552, 4096), (16, 131152, 262304), (32, 131152, 262304)])
def test_sliced_columns_have_counters(M, N, K):
    kernel, tn, g, ks = B.sjd_gemm_plan(M, N, K, resid=True)
    assert kernel != "sliced"


@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 64, 65, 128])
def test_what_a_plan_promises(M):
    for tiles in list(range(1, 300)) + list(range(300, 5000, 37)):
        for K in (32, 64, 512, 1536, 4096, 11008, 1 << 21):
            for resid in (False, True):
                kernel, tn, g, ks = B.sjd_gemm_plan(M, tiles * 16, K, resid)
                assert tiles % tn == 0 and tn * g <= 8
                if kernel == "sliced":
                    assert resid and tn == 1 and -(-tiles // g) <= 1024 and 2 <= ks <= 8 and K // 32 // ks >= 8
                elif kernel != "wide":
                    assert ks == 1 and (kernel == "span" or M <= 32)
                else:
                    assert M > 32
