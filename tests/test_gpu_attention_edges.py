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

# relative error (2-norm) of the logits of several images below: values carry 16 significant bits (2^-17 each), which two layers
# with scores of std 5 raise to 4.1e-5 .. 5.1e-5; one operand half lost anywhere (8 bits) would be 2e-3
REL = 1e-4


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


# several contexts, whose pointers come from the device table, in the second layer too: three images over caches of
# different lengths, one query tile and two.  4 heads: 10 key splits a context, 22 to 130 blocks of 32 (none to four blocks
# a wave).  20 heads: 8 splits, because 10 would be two rounds of workgroups; 11 to 61 blocks.  (Weights such that the
# scores are as large in both.)
@pytest.mark.parametrize("heads,std,lengths,L", [(4, 0.1, (4126, 2573, 700), 16), (4, 0.1, (4126, 2573, 700), 32),
                                                 (20, 0.045, (1900, 1210, 333), 16), (20, 0.045, (1900, 1210, 333), 32)])
def test_long_caches_of_several_images(B, heads, std, lengths, L):        # noqa: F811
    shape = synth.ModelShape(2, 128 * heads, heads, 512, 512, 256, 512, lengths[0] + 274, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9, std=std)
    prompt = synth.random_tokens(lengths[0], 0, 256, seed=1)
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
            ref = om.forward_tokens(n, toks[b])
            err = float(np.max(np.abs(got[b] - ref)))
            rel = float(np.linalg.norm(got[b] - ref) / np.linalg.norm(ref))
            forward._say(f"{heads} heads, image over {n} positions, L={L}: {err:.3e}, 2-norm {rel:.3e}")
            assert err < forward.TOL_BF16 and rel < REL, (n, err, rel)
    finally:
        for kv in kvs:
            B.sjd_kv_free(kv)
        B.sjd_free_model(m)
        om.close()


# 32 heads of 128: workgroups of eight waves.  One to eight images cut their keys into 8, 4, 2 and 1 splits (one: the split
# kernel writes the operand planes itself); one query tile and two, whole and partial; 22 blocks of 32 at most, so waves with
# three blocks down to none.  Three images: four waves.  (Images share one long prompt, cut at different lengths.)
@pytest.fixture(scope="module")
def wide_heads(B):        # noqa: F811
    shape = synth.ModelShape(1, 4096, 32, 512, 512, 256, 512, 1280, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9, std=0.036, threads=16)
    lengths = [697, 640, 511, 333, 100, 64, 33, 2]
    prompt = synth.random_tokens(lengths[0], 0, 256, seed=1)
    om = oracle.Model(shape, blob)
    m = B.sjd_init_model(B.config_from_shape(shape), blob)
    kvs = [B.sjd_kv_create(m) for _ in lengths]
    q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
    for kv, n in zip(kvs, lengths):
        B.sjd_prefill(m, kv, prompt[:n], None, B.sjd_sampler(8, 1.0), B.sjd_init(0, 0, -1), q)
    yield shape, om, m, kvs, lengths, prompt
    for kv in kvs:
        B.sjd_kv_free(kv)
    B.sjd_free_model(m)
    om.close()


@pytest.mark.parametrize("images,L", [(1, 16), (1, 31), (2, 20), (3, 16), (4, 13), (4, 32), (8, 16), (8, 5)])
def test_heads_of_eight_waves(B, wide_heads, images, L):        # noqa: F811
    shape, om, m, kvs, lengths, prompt = wide_heads
    toks = np.stack([synth.random_tokens(L, 256, 512, seed=20 + b) for b in range(images)])
    out = torch.empty((images, L, shape.v_s), dtype=torch.float32, device="cuda")
    B.sjd_forward_logits_batch(m, kvs[:images], forward._dev(toks), L, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    om.prefill(prompt)
    for b, n in enumerate(lengths[:images]):
        ref = om.forward_tokens(n, toks[b])
        err = float(np.max(np.abs(got[b] - ref)))
        rel = float(np.linalg.norm(got[b] - ref) / np.linalg.norm(ref))
        forward._say(f"image over {n} positions, {images} x {L}: {err:.3e}, 2-norm {rel:.3e}")
        assert err < forward.TOL_BF16 and rel < REL, (n, err, rel)


# Keys and values are read with non-temporal loads where the caches of a forward may hold more than 512 MB, else with plain ones:
# the same bits either way.  A handle counts with the positions it may have reached, so a generation that has begun and may go on for
# 17000 tokens reads the same few positions the other way.  Heads of 32, 64 and 128, the latter with eight waves and (24 heads) with
# four, one query tile and two.
@pytest.mark.parametrize("layers,d,heads", [(4, 1024, 32), (2, 2048, 32), (1, 4096, 32), (2, 3072, 24)])
def test_both_ways_to_read_the_cache(B, layers, d, heads):        # noqa: F811
    n_more = 17000
    shape = synth.ModelShape(layers, d, heads, 512, 512, 256, 512, n_more + 600, synth.DTYPE_BF16)
    assert 8 * d * layers * n_more > 512 << 20 > 8 * d * layers * 600
    m = B.sjd_init_model(B.config_from_shape(shape), synth.make_weights(shape, seed=9, std=0.036, threads=16))
    kv = B.sjd_kv_create(m)
    try:
        q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        smp, init = B.sjd_sampler(8, 1.0), B.sjd_init(0, 0, -1)
        B.sjd_prefill(m, kv, synth.random_tokens(403, 0, 256, seed=1), None, smp, init, q)
        outs = []
        for _ in range(2):
            for L in (1, 16, 29):
                toks = forward._dev(synth.random_tokens(L, 256, 512, seed=L))
                outs.append(torch.empty((L, shape.v_s), dtype=torch.float32, device="cuda"))
                B.sjd_forward_logits(m, kv, toks, L, outs[-1])
            B.sjd_decode_begin(m, kv, q, n_more, 16, smp, init, 7)
        torch.cuda.synchronize()
        for a, b in zip(outs[:3], outs[3:]):
            assert torch.isfinite(a).all() and a.abs().max() > 0 and torch.equal(a, b)
    finally:
        B.sjd_kv_free(kv)
        B.sjd_free_model(m)
