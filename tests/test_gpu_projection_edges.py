"""Projections at the edges of how their launches are cut (GPU only).

The check and its tolerance are those of test_gpu_forward.test_gemm_against_fp64: sampled outputs, one by one, against
fp64 dot products, 2e-5 * sqrt(K / 128).
"""
import pytest

import test_gpu_forward as forward
from test_gpu_forward import B          # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# the wide kernel's second kernel takes a column group (8 or 12 n tiles, or 16) per workgroup: a last group of 3 tiles
# whose grid is rounded up to 40 groups, more than four K-slices with a short last one, groups of 12 and of 16
@pytest.mark.parametrize("M,N,K", [(64, 4272, 3104), (128, 4272, 3104), (40, 1040, 4096), (112, 6528, 1056),
                                   (64, 12336, 416), (64, 16416, 288)])
def test_wide_column_groups(B, M, N, K):        # noqa: F811
    forward.test_gemm_against_fp64(B, 2, M, N, K)
