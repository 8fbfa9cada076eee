"""Prompts of ids followed by embedding rows (GPU only): a chunk of a prompt may hold both.

The check and its tolerances are those of test_gpu_forward._check_forward: logits of windows behind the prompt against
the fp64 oracle.
"""
import numpy as np
import pytest

from paper_2410_01699_amd import synth

import test_gpu_forward as forward
from test_gpu_forward import B          # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# chunks are 128 rows (bf16) and 32 rows (fp32): the change from ids to rows at a chunk's first row, last row, inside
# it, and a last chunk of one row
CASES = [(synth.DTYPE_BF16, 1, 120), (synth.DTYPE_BF16, 3, 126), (synth.DTYPE_BF16, 127, 1), (synth.DTYPE_BF16, 128, 5),
         (synth.DTYPE_BF16, 100, 100), (synth.DTYPE_BF16, 2, 3), (synth.DTYPE_F32, 5, 40), (synth.DTYPE_F32, 31, 2)]


@pytest.mark.parametrize("dtype,n_ids,n_embeds", CASES)
def test_mixed_prompt(B, dtype, n_ids, n_embeds):        # noqa: F811
    bf16 = dtype == synth.DTYPE_BF16
    shape = synth.ModelShape(2, 256, 4, 512, 2048, 1024, 2048, 280, dtype)
    blob = synth.make_weights(shape, seed=7)
    rng = np.random.default_rng(11)
    emb = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits((rng.standard_normal((n_embeds, 256)) * 0.02).astype(np.float32)))
    prompt = synth.random_tokens(n_ids, 0, 1024, seed=1)
    toks = synth.random_tokens(24, 1024, 2048, seed=2)
    worst = forward._check_forward(B, shape, blob, prompt, [(toks[:16], 5), (toks[16:24], 8)],
                                   forward.TOL_BF16 if bf16 else forward.TOL_F32, emb.reshape(n_embeds, 256))
    forward._say(f"{n_ids} ids + {n_embeds} rows: worst {worst:.3e}")
