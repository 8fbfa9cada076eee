"""The span projection kernel, whole and cut into K-slices, at the edges of how its launches are cut, and the wide kernel beside it
(GPU only).

The check and its tolerance are those of test_gpu_forward.test_gemm_against_fp64: sampled outputs, one by one, against
fp64 dot products, 2e-5 * sqrt(K / 128).  Whole outputs are also held to 3e-7 of 64 bits in the 2-norm: chains of 32
k-steps of fp32 sums are 2.8e-7 away, of 64 k-steps 4e-7.
"""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_forward as forward  # noqa: E402
from test_gpu_forward import B          # noqa: E402,F401  (fixture)

pytestmark = pytest.mark.gpu


def check(B, M, N, K, *plan):
    """against fp64, on the kernel that is meant (its name, tiles per packed group, groups per workgroup, K-slices); the test
    entry routes like O and down"""
    assert B.sjd_gemm_plan(M, N, K, resid=True)[:len(plan)] == plan
    forward.test_gemm_against_fp64(B, 2, M, N, K)


# tiles per packed group, groups per workgroup; reductions of one-tile groups are short here or have many tiles, else they are sliced
SHAPES = [
    (1536, 480, 1, 1),      # 15 k-steps: two for every wave but the last
    (4272, 480, 1, 2),      # 267 groups, one in the last workgroup
    (12176, 416, 1, 3),     # 761 groups, two in the last workgroup
    (6528, 1056, 2, 1),     # 33 k-steps: an odd walk, the last wave's shorter
    (16384, 96, 2, 2),      # 3 k-steps: waves without any
    (22048, 160, 2, 3),     # 689 groups, two in the last workgroup
    (12288, 288, 3, 1),     # 9 k-steps: two each, one for the fifth wave, none behind it
    (24576, 64, 3, 2),
]


@pytest.mark.parametrize("N,K,tn,g", SHAPES)
@pytest.mark.parametrize("M", [33, 48, 49, 64, 65, 96, 97, 128])
def test_spans_above_32_rows(B, M, N, K, tn, g):        # noqa: F811
    check(B, M, N, K, "span", tn, g)


# one-tile groups with a longer reduction: 40 and 33 k-steps
@pytest.mark.parametrize("N,K,g", [(3840, 1280, 1), (4272, 1056, 2)])
@pytest.mark.parametrize("M", [65, 96, 97, 128])
def test_spans_of_one_tile_groups(B, M, N, K, g):        # noqa: F811
    check(B, M, N, K, "span", 1, g)


# (up to 32 rows: two-tile and three-tile groups, 256 workgroups or fewer; 342 at 17 to 32)
@pytest.mark.parametrize("N,K,tn,g", [(22016, 4096, 2, 3), (22048, 160, 2, 3), (16384, 1536, 2, 2), (24576, 64, 3, 2), (32768, 96, 2, 3)])
@pytest.mark.parametrize("M", [1, 16, 17, 32])
def test_spans_up_to_32_rows(B, M, N, K, tn, g):        # noqa: F811
    check(B, M, N, K, *(("span", tn, g) if N < 32768 or M > 16 else ("skinny", tn)))


# walks of 8 to 15 k-steps a wave, which start at different k-steps: 8 each, 10 each, 12 with 11 in the last, 15 with 11
@pytest.mark.parametrize("M", [16, 32, 64, 128])
@pytest.mark.parametrize("K", [2048, 2560, 3040, 3712])
def test_short_walks_start_apart(B, M, K):        # noqa: F811
    check(B, M, 16384, K, *(("span", 2, 2) if M <= 96 or K < 3072 else ("wide", 2)))


# K cut into slices (one-tile groups): g tiles by ks slices.  8 x 8 up to 32 rows, also with five tiles in the last column and a
# short last slice; 4 x 4 at 33 .. 64; 2 x 4 (96 tiles), also with one tile in the last column, up to 32 rows with 72 k-steps and more;
# 2 x 8 (16 tiles; 8, 9 and 72 k-steps in all slices together); 2 x 2, of 16 k-steps and (160 tiles) of 216
@pytest.mark.parametrize("N,K,g,ks,Ms", [(4096, 11008, 8, 8, (1, 16, 17, 32)), (4176, 8384, 8, 8, (5, 16, 32)), (4096, 4096, 4, 4, (33, 48, 49, 64)),
                                         (1536, 4096, 2, 4, (1, 16, 17, 33, 48, 64, 65, 96, 128)), (1536, 1536, 2, 4, (33, 64, 96, 128)),
                                         (1040, 2112, 2, 4, (40, 100)), (1040, 2336, 2, 4, (16, 31)), (256, 2048, 2, 8, (33, 128)),
                                         (256, 2080, 2, 8, (64,)), (256, 2304, 2, 8, (16, 31)), (256, 512, 2, 2, (33, 80)),
                                         (2560, 6912, 2, 2, (16, 32, 48))])
def test_sliced_spans(B, N, K, g, ks, Ms):        # noqa: F811
    for M in Ms:
        check(B, M, N, K, "sliced", 1, g, ks)


# the wide kernel where nothing else goes: 8 K-slices with a short last one over a ragged column, two-tile groups; few tiles
# in two long slices' place; more than 256 workgroups of spans, one-tile and two-tile groups
@pytest.mark.parametrize("M,N,K,tn", [(64, 4112, 8416, 1), (128, 4112, 4224, 1), (64, 8160, 4096, 2), (96, 8160, 4096, 2), (49, 2560, 6912, 1),
                                      (128, 2560, 6912, 1), (80, 12336, 416, 1), (33, 32768, 96, 2), (128, 32768, 96, 2)])
def test_wide_ragged(B, M, N, K, tn):        # noqa: F811
    check(B, M, N, K, "wide", tn)


# 4097 one-tile groups: more columns of workgroups than a sliced launch has counters for
def test_more_columns_than_counters(B):        # noqa: F811
    check(B, 40, 65552, 512, "wide")


# Whoever arrives last adds the slices, always in the same order: a forward, whose O and down have the epilogue that adds to the residual
# stream, has the same bits every time.  2 x 4 and, at 7B widths, 8 x 8 (down, 16 rows) and 4 x 4 (O, 64 rows).
@pytest.mark.parametrize("L", [16, 64])
@pytest.mark.parametrize("d,heads,ffn", [(1536, 24, 4096), (4096, 32, 11008)])
def test_sliced_sums_have_one_order(B, d, heads, ffn, L):        # noqa: F811
    from paper_2410_01699_amd import synth
    routes = {B.sjd_gemm_plan(L, d, d, True), B.sjd_gemm_plan(L, d, ffn, True)}
    assert ("sliced", 1, 2, 4) in routes if d == 1536 else ("sliced", 1, 8, 8) in routes if L == 16 else ("sliced", 1, 4, 4) in routes
    shape = synth.ModelShape(2, d, heads, ffn, 512, 256, 512, 256, synth.DTYPE_BF16)
    m = B.sjd_init_model(B.config_from_shape(shape), synth.make_weights(shape, seed=5, threads=16))
    kv = B.sjd_kv_create(m)
    try:
        q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        B.sjd_prefill(m, kv, synth.random_tokens(70, 0, 256, seed=1), None, B.sjd_sampler(8, 1.0), B.sjd_init(0, 0, -1), q)
        toks = forward._dev(synth.random_tokens(L, 256, 512, seed=2))
        outs = [torch.empty((L, shape.v_s), dtype=torch.float32, device="cuda") for _ in range(40)]
        for o in outs:
            B.sjd_forward_logits(m, kv, toks, L, o)
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all() and all(torch.equal(outs[0], o) for o in outs[1:])
    finally:
        B.sjd_kv_free(kv)
        B.sjd_free_model(m)


@pytest.mark.parametrize("kernel,M,N,K", [("sliced", 16, 4096, 11008), ("sliced", 32, 4096, 11008), ("sliced", 64, 4096, 4096),
                                          ("sliced", 16, 1536, 4096), ("sliced", 128, 1536, 4096), ("span", 16, 22016, 4096),
                                          ("span", 32, 22016, 4096), ("span", 64, 22016, 4096), ("span", 96, 22016, 4096),
                                          ("span", 64, 12288, 4096), ("span", 64, 4608, 1536), ("span", 128, 8192, 1536)])
def test_span_precision(B, kernel, M, N, K):        # noqa: F811
    assert B.sjd_gemm_plan(M, N, K, resid=True)[0] == kernel
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


# The tuning aid's "model's choice" for O and down is the sliced kernel where the model runs it (7B down at 32 rows 21 us, skinny
# kernel 30).  At more rows it has room for as many slices as a handle.
def test_model_choice_of_the_tuning_aid(B):        # noqa: F811
    def us(wk, u):
        return min(B.sjd_gemm_bench(32, 4096, 11008, 1, wk, u, -20) for _ in range(3))

    model, sliced, skinny = us(-1, 0), us(208, 8), us(0, 0)
    forward._say(f"model's choice {model:.1f} us, sliced {sliced:.1f}, skinny {skinny:.1f}")
    assert abs(model - sliced) < abs(model - skinny)
    for M, N, K in ((64, 1536, 4096), (128, 4096, 11008), (128, 1536, 1536)):
        assert B.sjd_gemm_bench(M, N, K, 1, -1, 0, -3) > 0
    for wk, u in ((-1, 2), (-2, 0)):
        with pytest.raises(B.SjdError):
            B.sjd_gemm_bench(16, 4096, 4096, 1, wk, u, -3)
