"""Forwards of fp32 models at the edges of the projections that normalise, rotate and gate by themselves (GPU only).

Rows come in blocks of 8 where the weights are at most 2^20 values, else in variants of 8, 16 and 32; in blocks of 8 a
projection normalises its own input where (up to 8) rows x features fit 4096 values.  Logits against the fp64 oracle, with the bar of test_gpu_forward for fp32 models.
"""
import pytest

torch = pytest.importorskip("torch")
from paper_2410_01699_amd import synth  # noqa: E402

import test_gpu_forward as forward
from test_gpu_forward import B          # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# d = 144: all fold; 528 (three passes of 256 threads, the last of 16; 33 heads of 16): 7 rows fold, 8 do not; 48: less than a
# wave.  A feed-forward of 4100: gate/up alone in variants of 16 and 32 rows, behind a normalisation of its own, between projections
# that fold theirs.  An odd number of layers and an even one leave the residual stream in either of its buffers.
# Feed-forward widths and vocabularies that are no multiple of a workgroup's four waves; windows of 1, 7, 8, 9 (a block of one
# row) and up to 32.  The prompts fill up to three chunks of 32 rows, the caches cut into two key splits and more.
@pytest.mark.parametrize("layers,d,heads,ffn,vocab,max_seq", [(1, 128, 4, 100, 301, 120), (2, 128, 2, 96, 300, 400),
                                                               (3, 144, 9, 52, 150, 120), (2, 528, 33, 60, 130, 260),
                                                               (2, 48, 3, 20, 77, 64), (2, 128, 4, 4100, 300, 120)])
def test_edges(B, layers, d, heads, ffn, vocab, max_seq):        # noqa: F811
    shape = synth.ModelShape(layers, d, heads, ffn, vocab, 0, vocab, max_seq, synth.DTYPE_F32)
    blob = forward._random_gains(shape, synth.make_weights(shape, seed=5, std=1.4 / d ** 0.5), 11)
    prompt = synth.random_tokens(max_seq // 2 + 3, 0, vocab, seed=1)
    toks = synth.random_tokens(80, 0, vocab, seed=2)
    room = min(32, max_seq - len(prompt) - 12)
    windows = [(toks[:7], 3), (toks[7:15], 2), (toks[15:16], 1), (toks[16:25], 2), (toks[30:30 + min(28, room)], 1),
               (toks[30:30 + min(29, room)], 1), (toks[40:40 + room], 1)]
    worst = forward._check_forward(B, shape, blob, prompt, windows, forward.TOL_F32)
    forward._say(f"fp32 d={d} layers={layers} worst {worst:.3e}")
