"""sjd_forward_logits writes the L rows it is asked for and none behind them (GPU only).

The kernels compute whole operand tiles (16, 32, 64, 96 or 128 rows; fp32 models 8, 16 or 32), so the caller's buffer
here has a row for each of them, filled with a value that no logit takes.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2410_01699_amd import synth  # noqa: E402

MARK = -12345.0

# bf16: one and two tiles of the skinny kernel, the span kernel above 32 rows at the row counts of its variants, with and without a
# remainder; 16384 codes: the span kernel at any row count.  fp32: rows in one, two and more blocks of 8
CASES = ([(synth.DTYPE_BF16, 1024, L) for L in (1, 5, 16, 17, 33, 65, 97, 127, 128)] +
         [(synth.DTYPE_BF16, 16384, L) for L in (3, 17, 31, 32, 33)] +
         [(synth.DTYPE_F32, 1024, L) for L in (1, 5, 8, 9, 17, 32)])


@pytest.mark.parametrize("dtype,codes,L", CASES)
def test_rows_behind_the_window_stay(dtype, codes, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_01699_amd import binding as B
    shape = synth.ModelShape(1, 256, 4, 512, 1024 + codes, 1024, 1024 + codes, 200, dtype)
    m = B.sjd_init_model(B.config_from_shape(shape), synth.make_weights(shape, seed=3))
    kv = B.sjd_kv_create(m)
    try:
        q = torch.empty(codes, dtype=torch.float32, device="cuda")
        B.sjd_prefill(m, kv, synth.random_tokens(20, 0, 1024, seed=1), None, B.sjd_sampler(8, 1.0), B.sjd_init(0, 0, -1), q)
        toks = torch.from_numpy(synth.random_tokens(L, 1024, 1024 + codes, seed=2)).cuda()
        rows = torch.full((B.SJD_MAX_ROWS, codes), MARK, dtype=torch.float32, device="cuda")
        B.sjd_forward_logits(m, kv, toks, L, rows)
        torch.cuda.synchronize()
        assert bool((rows[:L] != MARK).all()) and bool((rows[L:] == MARK).all())
    finally:
        B.sjd_kv_free(kv)
        B.sjd_free_model(m)
