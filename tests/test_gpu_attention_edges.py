"""Window attention over caches so long that a wave walks several blocks of keys (GPU only).

The check and its tolerance are those of test_gpu_forward._check_forward: logits against the fp64 oracle.  Weights of
0.1 make the scores O(1) (std about 2), so that a block that is left out or read twice shows.
"""
import pytest

from paper_2410_01699_amd import synth

import test_gpu_forward as forward
from test_gpu_forward import B          # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# 4190 positions are 131 blocks of 32 in at most 16 splits of 4 waves: waves with three blocks, two, one (the last
# split) and none; windows of 1, 16 (one query tile), 32 (two) and 64 (two groups of two), for every head size
@pytest.mark.parametrize("hd", [32, 64, 128])
def test_long_cache(B, hd):        # noqa: F811
    shape = synth.ModelShape(1, 2 * hd, 2, 4 * hd, 512, 256, 512, 4400, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9, std=0.1)
    prompt = synth.random_tokens(4126, 0, 256, seed=1)
    toks = synth.random_tokens(160, 256, 512, seed=2)
    windows = [(toks[:64], 64), (toks[64:80], 5), (toks[80:112], 17), (toks[112:113], 1)]
    worst = forward._check_forward(B, shape, blob, prompt, windows, forward.TOL_BF16)
    forward._say(f"heads of {hd}: worst {worst:.3e}")
