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


# A second round of workgroups that own their features is mostly empty: such projections run on the skinny and the wide kernel (two-tile
# groups at 17 to 32 rows excepted).  (27648, 5120), (18432, 6144), (32768, 6144), (28672, 4096), (44032, 8192): gate/up and QKV of wide
# decoders, 342 to 918 workgroups.
@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 48, 64, 65, 96, 128])
def test_spans_are_one_round(M):
    wide = [(27648, 5120), (18432, 6144), (32768, 6144), (28672, 4096), (44032, 8192), (36864, 7168)]
    for N, K in wide:
        kernel, tn, g, ks = B.sjd_gemm_plan(M, N, K)
        assert kernel == ("wide" if M > 32 else "span" if M > 16 and (N, K) == (32768, 6144) else "skinny")
    for tiles in range(1, 5000, 7):
        for K in (512, 4096, 8192):
            kernel, tn, g, ks = B.sjd_gemm_plan(M, tiles * 16, K)
            assert kernel != "span" or -(-tiles // tn // g) <= 256 or (16 < M <= 32 and tn == 2)
    # four tiles a workgroup above 96 rows: four waves only (gate/up of d = 3072, QKV of d = 5120, 16384 logits of d = 4096)
    for N, K in ((16384, 3072), (15360, 5120), (16384, 4096)):
        assert (B.sjd_gemm_plan(M, N, K)[0] == "span") == (32 < M <= 96 or (M <= 32 and N == 16384)), (M, N, K)
    assert B.sjd_gemm_plan(M, 16384, 2048)[0] == "span"
    # long reductions above 64 rows
    assert B.sjd_gemm_plan(M, 24576, 8192)[0] == ("wide" if M > 64 else "span")
    # what fills the chip in one round stays: 7B QKV and gate/up above 32 rows, gate/up at any row count
    assert B.sjd_gemm_plan(M, 22016, 4096)[0] == "span" and (B.sjd_gemm_plan(M, 12288, 4096)[0] == "span") == (M > 32)


# Few tiles (O and down of narrow decoders) are cut in K where that is faster: not the short reductions up to 32 rows, and in two slices
# (129 to 255 tiles) only while a slice's share of the activations is small.
@pytest.mark.parametrize("N,K,rows", [(512, 2048, (33, 128)), (1024, 2048, (33, 128)), (512, 2304, (1, 128)), (1536, 4096, (1, 128)),
                                      (2048, 8192, (1, 128)), (1536, 1536, (33, 128)), (3072, 3072, (33, 64)), (2560, 6912, (1, 48)),
                                      (3072, 8192, (1, 48)), (3584, 18944, (1, 48)), (4096, 4096, (33, 64)), (4096, 11008, (1, 32))])
def test_where_slices_pay(N, K, rows):
    for M in range(1, 129):
        kernel = B.sjd_gemm_plan(M, N, K, resid=True)[0]
        assert (kernel == "sliced") == (rows[0] <= M <= rows[1]), (M, kernel)
