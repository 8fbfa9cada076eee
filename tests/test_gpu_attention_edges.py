"""Window attention over caches so long that a wave walks several blocks of keys (GPU only).

The check and its tolerance are those of test_gpu_forward._check_forward: logits against the fp64 oracle.  Weights of
0.1 make the scores O(1) (std about 2), so that a block that is left out or read twice shows.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_2410_01699_amd import synth  # noqa: E402

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


# several contexts, whose pointers come from the device table, in the second layer too: three images over 4126, 2573 and
# 700 positions (22 to 130 blocks of 32 in 10 splits of 4 waves: none to four blocks a wave), one query tile and two
@pytest.mark.parametrize("L", [16, 32])
def test_long_caches_of_several_images(B, L):        # noqa: F811
    shape = synth.ModelShape(2, 512, 4, 512, 512, 256, 512, 4400, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9, std=0.1)
    prompt = synth.random_tokens(4126, 0, 256, seed=1)
    lengths = [4126, 2573, 700]
    toks = np.stack([synth.random_tokens(L, 256, 512, seed=20 + b) for b in range(3)])
    om = oracle.Model(shape, blob)
    m = B.sjd_init_model(B.config_from_shape(shape), blob)
    kvs = [B.sjd_kv_create(m) for _ in lengths]
    try:
        q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        for kv, n in zip(kvs, lengths):
            B.sjd_prefill(m, kv, prompt[:n], None, B.sjd_sampler(8, 1.0), B.sjd_init(0, 0, -1), q)
        out = torch.empty((3, L, shape.v_s), dtype=torch.float32, device="cuda")
        B.sjd_forward_logits_batch(m, kvs, forward._dev(toks), L, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        om.prefill(prompt)
        for b, n in enumerate(lengths):      # (longest first: a window overwrites the oracle's rows from n on)
            err = float(np.max(np.abs(got[b] - om.forward_tokens(n, toks[b]))))
            forward._say(f"image over {n} positions, L={L}: {err:.3e}")
            assert err < forward.TOL_BF16, (n, err)
    finally:
        for kv in kvs:
            B.sjd_kv_free(kv)
        B.sjd_free_model(m)
        om.close()


# 32 rows are 32 drafts of one image or 16 of each of two.  An image's keys are split alike in both, so the first 16
# drafts have the same logits bit for bit: 32 heads of 128 (the 7B decoder's), 16 splits.
def test_same_sums_alone_and_beside_another_image(B):        # noqa: F811
    shape = synth.ModelShape(2, 4096, 32, 1024, 512, 256, 512, 2100, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9, threads=16)
    m = B.sjd_init_model(B.config_from_shape(shape), blob)
    kvs = [B.sjd_kv_create(m) for _ in range(2)]
    try:
        q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        for b, n in enumerate((1240, 900)):
            B.sjd_prefill(m, kvs[b], synth.random_tokens(n, 0, 256, seed=b), None, B.sjd_sampler(8, 1.0),
                          B.sjd_init(0, 0, -1), q)
        toks = forward._dev(synth.random_tokens(32, 256, 512, seed=5))
        alone = torch.empty((32, shape.v_s), dtype=torch.float32, device="cuda")
        two = torch.empty((2, 16, shape.v_s), dtype=torch.float32, device="cuda")
        B.sjd_forward_logits(m, kvs[0], toks, 32, alone)
        B.sjd_forward_logits_batch(m, kvs, toks, 16, two)
        torch.cuda.synchronize()
        assert torch.equal(two[0], alone[:16])
    finally:
        for kv in kvs:
            B.sjd_kv_free(kv)
        B.sjd_free_model(m)
