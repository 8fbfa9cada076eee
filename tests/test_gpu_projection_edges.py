"""Projections at the edges of how their launches are cut (GPU only).

The check and its tolerance are those of test_gpu_forward.test_gemm_against_fp64: sampled outputs, one by one, against
fp64 dot products, 2e-5 * sqrt(K / 128).
"""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_forward as forward  # noqa: E402
from test_gpu_forward import B          # noqa: E402,F401  (fixture)

pytestmark = pytest.mark.gpu


# shapes whose features do not fill the last workgroup, at the row counts of several variants.  Rules on sizes send (64, 4272, 3104) and
# (40, 1040, 4096) to slices, (112, 6528, 1056) to whole spans, the others to the wide kernel.
@pytest.mark.parametrize("M,N,K", [(64, 4272, 3104), (128, 4272, 3104), (40, 1040, 4096), (112, 6528, 1056),
                                   (64, 12336, 416), (64, 16416, 288)])
def test_wide_column_groups(B, M, N, K):        # noqa: F811
    forward.test_gemm_against_fp64(B, 2, M, N, K)


# the wide kernel's second kernel takes a column group (8 or 12 n tiles, or 16) per workgroup: a last group of 3 tiles with seven
# and eight K-slices, the last one short; two of 8 and of 16 tiles whose grids are rounded up; 12 tiles of which the last group has 9
@pytest.mark.parametrize("M,N,K,plan", [(128, 4272, 3104, (1, 2, 7)), (64, 4272, 8576, (1, 2, 8)), (112, 12848, 640, (1, 2, 2)),
                                        (64, 29504, 512, (2, 2, 2)), (64, 32784, 512, (3, 1, 2)), (128, 32784, 288, (3, 1, 1))])
def test_wide_column_groups_run_there(B, M, N, K, plan):        # noqa: F811
    assert B.sjd_gemm_plan(M, N, K, resid=True) == ("wide", *plan)
    forward.test_gemm_against_fp64(B, 2, M, N, K)


# Precision of a whole output against 64 bits: the 7B QKV and gate/up projections above 96 rows, which split K over the waves of a
# workgroup.  Eight chains of 16 k-steps (QKV) are 2.02e-7 (2-norm) away, four of 32 (gate/up) 2.80e-7, whatever the rows and the seed;
# fewer are longer chains of fp32 sums: 3.24e-7 for three, 3.97e-7 for two.
@pytest.mark.parametrize("M", [97, 128])
@pytest.mark.parametrize("N", [12288, 22016])
def test_sliced_projection_precision(B, M, N):        # noqa: F811
    K = 4096
    g = torch.Generator(device="cuda").manual_seed(N + M)
    A = torch.randn((M, K), generator=g, device="cuda")
    A = ((A.view(torch.int32) + 0x7F) & -256).view(torch.float32)           # 16 significant bits, as the kernel takes them
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    B.sjd_gemm_test(2, A, W.view(torch.int16), M, N, K, C)
    ref = A.double() @ W.double().T
    rel = float((C.double() - ref).norm() / ref.norm())
    forward._say(f"{M} x {N} x {K}: {rel:.3e} from 64 bits")
    assert rel < 3.0e-7
