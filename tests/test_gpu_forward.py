"""GPU parity: linear layers, window forward (logits), and whole generations vs the CPU oracle.

Bars: logits max-abs <= 1e-4 (fp32 models) / 2e-2 (bf16 models); in fp32 mode whole token
sequences are identical; given the GPU's own logits the verification is bit-exact in any mode.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_2410_01699_amd import synth  # noqa: E402

TOL_F32 = 1e-4
TOL_BF16 = 2e-2


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_01699_amd import binding
    return binding


def _say(msg):
    print(msg, flush=True, file=sys.stderr)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


class Gpu:
    """model + cache handles with clean-up"""

    def __init__(self, B, shape, blob):
        self.B, self.shape = B, shape
        self.m = B.sjd_init_model(B.config_from_shape(shape), blob)
        self.kv = B.sjd_kv_create(self.m)

    def close(self):
        self.B.sjd_kv_free(self.kv); self.B.sjd_free_model(self.m)

    def logits(self, tokens):
        L = len(tokens)
        out = torch.empty((L, self.shape.v_s), dtype=torch.float32, device="cuda")
        self.B.sjd_forward_logits(self.m, self.kv, _dev(np.asarray(tokens, np.int32)), L, out)
        torch.cuda.synchronize()
        return out.cpu().numpy()


# ------------------------------------------------------------------ linear layers
@pytest.mark.parametrize("dtype,M,N,K", [(0, 8, 384, 128), (0, 16, 100, 512), (0, 32, 37, 260), (0, 3, 1024, 128),
                                         (1, 16, 4608, 1536), (1, 16, 1536, 4096), (1, 32, 256, 320), (1, 5, 48, 64),
                                         (1, 16, 12288, 4096), (1, 32, 4096, 11008), (1, 16, 22016, 4096),
                                         (1, 16, 8192, 4096),
                                         # bf16 weights, fp32 activations handed over in 3 bytes per value
                                         (2, 16, 4096, 11008), (2, 32, 4096, 4096), (2, 7, 48, 96), (2, 32, 1536, 4096),
                                         (2, 21, 256, 320),
                                         # 17..32 rows of a shape whose N alone fills the chip: the span kernel (a
                                         # workgroup owns three or two weight groups for the whole reduction), also with
                                         # a reduction shorter than one k-step per wave
                                         (2, 32, 22016, 4096), (2, 21, 22016, 4096), (2, 25, 16384, 96),
                                         # more than 32 rows: the span kernel, whole (7B QKV and gate/up, 775M QKV) and in
                                         # K-slices (O at 64 rows, 775M down), the wide kernel (waves split N, K-slices
                                         # added by a second kernel: 7B O at 128 rows, down and the LM head), and
                                         # ragged sizes (rows not a multiple of 16, fewer weight groups than waves)
                                         (1, 64, 12288, 4096), (2, 128, 12288, 4096), (1, 128, 4096, 4096),
                                         (2, 64, 4096, 4096), (2, 128, 4096, 11008), (1, 64, 4096, 11008),
                                         (2, 64, 22016, 4096), (1, 128, 22016, 4096), (2, 128, 8192, 4096),
                                         (1, 96, 4608, 1536), (2, 48, 1536, 4096), (2, 33, 48, 96), (1, 100, 256, 320),
                                         (2, 77, 80, 2080)])
def test_gemm_against_fp64(B, dtype, M, N, K):
    _say(f"gemm dtype={dtype} M={M} N={N} K={K}")
    rng = np.random.default_rng(N + K)
    A = rng.standard_normal((M, K)).astype(np.float32)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    if dtype == 1:
        A16, W16 = synth.f32_to_bf16_bits(A).reshape(M, K), synth.f32_to_bf16_bits(W).reshape(N, K)
        A, W = synth.bf16_bits_to_f32(A16).reshape(M, K), synth.bf16_bits_to_f32(W16).reshape(N, K)
        dA, dW = _dev(A16.view(np.int16)), _dev(W16.view(np.int16))
    elif dtype == 2:
        # a few values whose rounding carries into the upper 16 bits or the exponent, and tiny ones
        A[0, :6] = np.array([0x3F7FFFC0, 0x3F80FF80, 0xBFFFFFFF, 0x3F800080, 0x3F800180, 0x00800000],
                            np.uint32).view(np.float32)
        W16 = synth.f32_to_bf16_bits(W).reshape(N, K)
        W = synth.bf16_bits_to_f32(W16).reshape(N, K)
        dA, dW = _dev(A), _dev(W16.view(np.int16))
        # what the kernel multiplies: A rounded to 16 significant bits, ties to even
        u = A.view(np.uint32).astype(np.uint64)
        A = ((u + 0x7F + ((u >> 8) & 1)) & 0xFFFFFF00).astype(np.uint32).view(np.float32)
    else:
        dA, dW = _dev(A), _dev(W)
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    B.sjd_gemm_test(dtype, dA, dW, M, N, K, C)
    torch.cuda.synchronize()
    got = C.cpu().numpy()
    # sampled outputs, one by one in fp64 (all of them when small)
    if M * N <= 1 << 16:
        ref = A.astype(np.float64) @ W.astype(np.float64).T
        assert np.max(np.abs(got - ref)) < 2e-5 * np.sqrt(K / 128)
    else:
        rows = rng.integers(0, M, 400); cols = rng.integers(0, N, 400)
        cols[:8] = [0, 1, 15, 16, N - 1, N - 16, N - 17, N // 2]
        for r, c in zip(rows, cols):
            ref = float(np.dot(A[r].astype(np.float64), W[c].astype(np.float64)))
            assert abs(got[r, c] - ref) < 2e-5 * np.sqrt(K / 128), (r, c)


# ------------------------------------------------------------------ window forward
def _check_forward(B, shape, blob, prompt, windows, tol, embeds=None):
    om = oracle.Model(shape, blob)
    g = Gpu(B, shape, blob)
    try:
        smp = B.sjd_sampler(8, 1.0); init = B.sjd_init(0, 0, -1)
        q_last = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        B.sjd_prefill(g.m, g.kv, prompt, embeds, smp, init, q_last)
        torch.cuda.synchronize()
        lp = om.prefill(prompt, embeds)
        P = len(prompt) + (0 if embeds is None else len(embeds))
        assert B.sjd_kv_len(g.kv) == P
        q_ref = oracle.dist(lp, 8, 1.0)
        # top-8 membership can flip on a near-tie at bf16 precision: compare through the logits instead
        worst = 0.0
        n = P
        for toks, keep in windows:
            _say(f"  window at n={n} L={len(toks)}")
            got = g.logits(toks)
            ref = om.forward_tokens(n, toks)
            err = float(np.max(np.abs(got - ref)))
            worst = max(worst, err)
            assert err < tol, (n, err)
            n += keep
            B.sjd_kv_set_len(g.kv, n)
        if tol <= TOL_F32:
            assert np.max(np.abs(q_last.cpu().numpy() - q_ref)) < 1e-5
        return worst
    finally:
        g.close(); om.close()


def test_forward_tiny_fp32(B):
    w = synth.WORKLOADS["tiny"]
    blob = synth.make_weights(w.shape, seed=0)
    prompt, _ = synth.make_prompt(w)
    toks = synth.random_tokens(64, 0, 1024, seed=3)
    windows = [(toks[0:8], 3), (toks[8:16], 8), (toks[16:17], 1), (toks[20:28], 5), (toks[30:38], 8)]
    worst = _check_forward(B, w.shape, blob, prompt, windows, TOL_F32)
    _say(f"tiny fp32 worst logit error {worst:.3e}")


def test_forward_fp32_other_head_sizes_and_large_activations(B):
    # O(1) weights so that every term matters; heads of 16 and 64; window of 32; long prompt (3 chunks)
    for heads, d in ((4, 64), (2, 128)):
        shape = synth.ModelShape(3, d, heads, 96, 300, 44, 300, 120, synth.DTYPE_F32)
        blob = synth.make_weights(shape, seed=5, std=0.12)
        prompt = synth.random_tokens(70, 0, 300, seed=1)
        toks = synth.random_tokens(40, 44, 300, seed=2)
        worst = _check_forward(B, shape, blob, prompt, [(toks[:32], 7), (toks[3:20], 17), (toks[5:6], 1)], TOL_F32)
        _say(f"fp32 d={d} heads={heads} worst {worst:.3e}")


def test_forward_small_bf16(B):
    shape = synth.ModelShape(4, 256, 4, 512, 2048, 1024, 2048, 200, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=7)
    prompt = synth.random_tokens(45, 0, 1024, seed=1)
    toks = synth.random_tokens(64, 1024, 2048, seed=2)
    worst = _check_forward(B, shape, blob, prompt, [(toks[:16], 5), (toks[16:48], 32), (toks[50:57], 7)], TOL_BF16)
    _say(f"small bf16 worst {worst:.3e}")


def _random_gains(shape, blob, seed):
    """the RMSNorm gains of a blob (all ones as generated) replaced by values in [0.5, 1.5)"""
    rng = np.random.default_rng(seed)
    for _, (off, shp) in synth.tensor_offsets(shape).items():
        if len(shp) == 1:
            g = rng.uniform(0.5, 1.5, shp[0]).astype(np.float32)
            blob[off:off + shp[0]] = g if shape.dtype == synth.DTYPE_F32 else synth.f32_to_bf16_bits(g)
    return blob


def test_forward_with_non_unit_norm_gains(B):
    """every normalisation (two per layer and the final one) with its own random gain vector: a gain
    applied at the wrong place, or the wrong layer's, shows as an error of order one"""
    # (also a RoPE base and a normalisation epsilon other than the defaults every other test uses; the
    # epsilons are of the order of mean(x^2), so that they matter)
    shape = synth.ModelShape(3, 64, 4, 96, 300, 44, 300, 120, synth.DTYPE_F32, rope_theta=50000.0, rms_eps=1e-2)
    blob = _random_gains(shape, synth.make_weights(shape, seed=5, std=0.12), 11)
    prompt = synth.random_tokens(40, 0, 300, seed=1)
    toks = synth.random_tokens(40, 44, 300, seed=2)
    worst = _check_forward(B, shape, blob, prompt, [(toks[:32], 7), (toks[3:20], 17), (toks[5:6], 1)], TOL_F32)
    _say(f"fp32 random gains worst {worst:.3e}")
    shape = synth.ModelShape(4, 256, 4, 512, 2048, 1024, 2048, 200, synth.DTYPE_BF16)
    # (weights large enough for attention scores of order one: with the 0.02 of the workloads the
    # softmax is nearly uniform and would hide a wrong score scale)
    blob = _random_gains(shape, synth.make_weights(shape, seed=7, std=0.08), 12)
    prompt = synth.random_tokens(45, 0, 1024, seed=1)
    toks = synth.random_tokens(64, 1024, 2048, seed=2)
    emb = (np.random.default_rng(3).standard_normal((5, 256)) * 0.02).astype(np.float32)
    emb = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(emb)).reshape(emb.shape)
    worst = _check_forward(B, shape, blob, prompt, [(toks[:16], 5), (toks[16:48], 32), (toks[50:57], 7)], TOL_BF16,
                           embeds=emb)
    _say(f"bf16 random gains worst {worst:.3e}")
    # d_model = 96: 6 partial sums of squares per token, rows padded to 8
    shape = synth.ModelShape(2, 96, 3, 160, 512, 0, 512, 100, synth.DTYPE_BF16, rope_theta=1e6, rms_eps=3e-3)
    blob = _random_gains(shape, synth.make_weights(shape, seed=9, std=0.05), 13)
    prompt = synth.random_tokens(33, 0, 512, seed=1)
    toks = synth.random_tokens(40, 0, 512, seed=2)
    worst = _check_forward(B, shape, blob, prompt, [(toks[:9], 9), (toks[9:40], 31)], TOL_BF16)
    _say(f"bf16 d=96 random gains worst {worst:.3e}")


def test_forward_775m_bf16(B):
    """full size of the class-conditional configuration: prompt = 1 id + 120 embedding rows"""
    w = synth.WORKLOADS["775m"]
    blob = synth.make_weights(w.shape, seed=0)
    ids, emb = synth.make_prompt(w)
    toks = synth.random_tokens(64, 0, w.shape.v_s, seed=4)
    # (the LM head, 16384 outputs, runs on the span kernel at any row count)
    worst = _check_forward(B, w.shape, blob, ids, [(toks[:16], 6), (toks[16:32], 16), (toks[32:64], 20)], TOL_BF16, embeds=emb)
    _say(f"775m bf16 worst {worst:.3e}")


# ------------------------------------------------------------------ one step, and whole generations
def test_step_matches_oracle_given_gpu_logits(B):
    """sjd_step = forward + verification: the verification applied to the GPU's own logits must be
    bit-exact in a bf16 model too, and the cache must advance by the accepted count."""
    shape = synth.ModelShape(2, 256, 4, 512, 2048, 1024, 2048, 160, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=8)
    g = Gpu(B, shape, blob)
    try:
        V, lo, L, K = shape.v_s, shape.samp_lo, 16, 300
        smp = B.sjd_sampler(K, 1.0); init = B.sjd_init(1, 16, 2047)
        osmp = oracle.Sampler(K, 1.0); oinit = oracle.Init(1, 16, 2047)
        prompt = synth.random_tokens(20, 0, 1024, seed=1)
        q_last = torch.empty(V, dtype=torch.float32, device="cuda")
        B.sjd_prefill(g.m, g.kv, prompt, None, smp, init, q_last)
        draft = torch.zeros(L, dtype=torch.int32, device="cuda")
        p_old = torch.zeros((L, V), dtype=torch.float32, device="cuda")
        B.sjd_first_window(g.m, q_last, L, init, 42, draft, p_old)
        na = torch.zeros(1, dtype=torch.int32, device="cuda")
        nd = torch.zeros(L, dtype=torch.int32, device="cuda"); pn = torch.zeros_like(p_old)
        hist = []
        n = 20
        for c in range(1, 9):
            _say(f"  step {c} n={n}")
            d_h, p_h = draft.cpu().numpy(), p_old.cpu().numpy()
            logits = g.logits(d_h)                                 # hook: same forward, no advance
            want = oracle.verify(logits, p_h, d_h, lo, osmp, oinit, len(hist), np.array(hist, np.int32), 42, c)
            B.sjd_step(g.m, g.kv, draft, p_old, L, smp, init, len(hist), 42, c, na, nd, pn)
            torch.cuda.synchronize()
            a = int(na.item())
            assert a == want[0]
            assert np.array_equal(nd.cpu().numpy(), want[1])
            assert np.array_equal(pn.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
            hist += d_h[:a].tolist()
            n += a
            assert B.sjd_kv_len(g.kv) == n
            draft, nd = nd, draft; p_old, pn = pn, p_old
    finally:
        g.close()


@pytest.mark.parametrize("L,mode,flags", [(8, 0, 0), (1, 0, 0), (4, 1, 0), (16, 0, 0), (8, 2, 0), (8, 0, 1), (4, 2, 1),
                                          (8, 3, 0), (8, 4, 0), (16, 4, 0), (5, 4, 1), (16, 3, 1)])
def test_generate_tiny_fp32_token_identity(B, L, mode, flags):
    w = synth.WORKLOADS["tiny"]
    blob = synth.make_weights(w.shape, seed=0)
    prompt, _ = synth.make_prompt(w)
    om = oracle.Model(w.shape, blob)
    g = Gpu(B, w.shape, blob)
    try:
        for seed in range(3):
            _say(f"generate tiny L={L} mode={mode} flags={flags} seed={seed}")
            osmp = oracle.Sampler(w.top_k, w.temperature); oinit = oracle.Init(mode, w.row_stride, -1, flags)
            lp = om.prefill(prompt)
            want, wst = om.generate_sjd(len(prompt), lp, w.n_image_tokens, L, osmp, oinit, seed)
            got, st = B.sjd_generate(g.m, g.kv, prompt, None, w.n_image_tokens, L, B.sjd_sampler(w.top_k, w.temperature),
                                     B.sjd_init(mode, w.row_stride, -1, flags), seed)
            assert np.array_equal(got, want), (seed, np.nonzero(got != want)[0][:5])
            assert st.steps == wst.steps
            assert list(st.accept_hist) == list(wst.accept_hist)
            if L == 1:
                lp = om.prefill(prompt)
                ar = om.generate_ar(len(prompt), lp, w.n_image_tokens, osmp, oinit, seed)
                assert np.array_equal(got, ar)                     # window 1 == ordinary AR sampling
    finally:
        g.close(); om.close()


def test_generate_greedy_equals_greedy_ar(B):
    """K = 1: SJD is deterministic Jacobi decoding and must reproduce greedy decoding exactly"""
    w = synth.WORKLOADS["tiny"]
    blob = synth.make_weights(w.shape, seed=0, std=0.05)
    prompt, _ = synth.make_prompt(w)
    om = oracle.Model(w.shape, blob)
    g = Gpu(B, w.shape, blob)
    try:
        seq = list(prompt)
        for _ in range(32):
            lg = om.forward_full(om.embed(np.array(seq, np.int32)))[-1]
            seq.append(int(np.argmax(lg)))
        want = np.array(seq[len(prompt):], np.int32)
        for L in (1, 8, 32):
            _say(f"greedy L={L}")
            got, st = B.sjd_generate(g.m, g.kv, prompt, None, 32, L, B.sjd_sampler(1, 1.0), B.sjd_init(0, 8, -1), 5)
            assert np.array_equal(got, want)
            assert st.steps <= 31
    finally:
        g.close(); om.close()


def test_generate_bf16_statistics_and_validity(B):
    """bf16 model: tokens cannot be compared one by one (logits differ in the third digit), so check
    what is unique: ids in range, row-end forcing, step accounting, determinism."""
    shape = synth.ModelShape(2, 256, 4, 512, 2048, 1024, 2048, 400, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=8)
    g = Gpu(B, shape, blob)
    try:
        prompt = synth.random_tokens(20, 0, 1024, seed=1)
        smp = B.sjd_sampler(300, 1.0); init = B.sjd_init(1, 9, 2047)
        N = 9 * 20
        a, sa = B.sjd_generate(g.m, g.kv, prompt, None, N, 16, smp, init, 3)
        b, sb = B.sjd_generate(g.m, g.kv, prompt, None, N, 16, smp, init, 3)
        assert np.array_equal(a, b) and sa.steps == sb.steps
        assert a.min() >= 1024 and a.max() < 2048
        assert np.all(a[8::9] == 2047)
        hist = np.array(sa.accept_hist[:])
        assert hist[0] == 0 and hist.sum() == sa.steps and 1 <= sa.steps <= N - 1
        assert int((hist * np.arange(65)).sum()) in (N - 1, N)
    finally:
        g.close()


def test_step_errors(B):
    w = synth.WORKLOADS["tiny"]
    blob = synth.make_weights(w.shape, seed=0)
    g = Gpu(B, w.shape, blob)
    try:
        V = w.shape.v_s
        d = torch.zeros(8, dtype=torch.int32, device="cuda"); p = torch.zeros((8, V), device="cuda")
        na = torch.zeros(1, dtype=torch.int32, device="cuda")
        smp = B.sjd_sampler(64, 1.0); init = B.sjd_init(0, 8, -1)
        B.sjd_kv_set_len(g.kv, w.shape.max_seq - 4)
        with pytest.raises(B.SjdError) as e:
            B.sjd_step(g.m, g.kv, d, p, 8, smp, init, 0, 1, 1, na, d, p)
        assert e.value.code == B.SJD_ESEQ
        with pytest.raises(B.SjdError) as e:
            B.sjd_step(g.m, g.kv, d, p, 33, smp, init, 0, 1, 1, na, d, p)
        assert e.value.code == B.SJD_EINVAL
        with pytest.raises(B.SjdError) as e:
            B.sjd_generate(g.m, g.kv, np.arange(16, dtype=np.int32), None, 1000, 8, smp, init, 0)
        assert e.value.code == B.SJD_ESEQ
        with pytest.raises(B.SjdError):
            B.sjd_init_model(B.config_from_shape(w.shape), blob[:-1])
    finally:
        g.close()


# ------------------------------------------------------------------ full size, launch configuration of the benchmark
@pytest.mark.parametrize("workload,window", [("7b_32x32", 0), ("7b_48x48", 0), ("7b_32x32", 64)])
def test_forward_and_step_7b_full_size(B, workload, window):
    """The 7B workloads at their real shape (32 layers, d=4096, 8192 sampled codes of 65536; window 16 on the
    32 x 32 grid, window 32 with a forced row-end token every 49 positions on the 48 x 48 grid, and a window
    of 64, for the span, sliced and wide projection kernels): every logit of one window against the fp64 oracle,
    then one whole sjd_step whose verification must be bit-exact given the GPU's logits."""
    import dataclasses
    w = synth.WORKLOADS[workload]
    if window:
        w = dataclasses.replace(w, window=window)
    _say(f"7b: {workload} window {w.window}: generating weights")
    blob = synth.make_weights(w.shape, seed=0, threads=16)
    ids, _ = synth.make_prompt(w)
    om = oracle.Model(w.shape, blob)
    g = Gpu(B, w.shape, blob)
    try:
        V, lo, L = w.shape.v_s, w.shape.samp_lo, w.window
        smp = B.sjd_sampler(w.top_k, w.temperature); init = B.sjd_init(w.init_mode, w.row_stride, w.eol_id)
        q_last = torch.empty(V, dtype=torch.float32, device="cuda")
        _say("7b: gpu prefill")
        B.sjd_prefill(g.m, g.kv, ids, None, smp, init, q_last)
        draft = torch.zeros(L, dtype=torch.int32, device="cuda")
        p_old = torch.zeros((L, V), dtype=torch.float32, device="cuda")
        B.sjd_first_window(g.m, q_last, L, init, 7, draft, p_old)
        torch.cuda.synchronize()
        d_h, p_h = draft.cpu().numpy(), p_old.cpu().numpy()
        got = g.logits(d_h)
        _say("7b: oracle prefill + window (fp64 on the host, about half a minute)")
        om.prefill(ids)
        ref = om.forward_tokens(len(ids), d_h)
        err = float(np.max(np.abs(got - ref)))
        _say(f"7b: worst logit error {err:.3e} (logit std {ref.std():.3f})")
        assert err < TOL_BF16
        want = oracle.verify(got, p_h, d_h, lo, oracle.Sampler(w.top_k, w.temperature),
                             oracle.Init(w.init_mode, w.row_stride, w.eol_id), 0, None, 7, 1)
        na = torch.zeros(1, dtype=torch.int32, device="cuda")
        nd = torch.zeros(L, dtype=torch.int32, device="cuda"); pn = torch.zeros_like(p_old)
        B.sjd_step(g.m, g.kv, draft, p_old, L, smp, init, 0, 7, 1, na, nd, pn)
        torch.cuda.synchronize()
        assert int(na.item()) == want[0]
        assert np.array_equal(nd.cpu().numpy(), want[1])
        assert np.array_equal(pn.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
        assert B.sjd_kv_len(g.kv) == len(ids) + want[0]

        # the launch configuration the benchmark times: the device-resident loop replaying its captured
        # iteration.  Every iteration against the oracle's verification of the same logits (taken with
        # the forward hook, which leaves the loop state alone), then the finished image token by token.
        N = 40 if w.row_stride == 32 else 60               # (the 49-token rows: past the first forced row end)
        osmp = oracle.Sampler(w.top_k, w.temperature); oinit = oracle.Init(w.init_mode, w.row_stride, w.eol_id)
        B.sjd_kv_use_graph(g.kv, True)
        B.sjd_prefill(g.m, g.kv, ids, None, smp, init, q_last)
        B.sjd_decode_begin(g.m, g.kv, q_last, N, L, smp, init, 11)
        torch.cuda.synchronize()
        d_o, p_o = oracle.first_window(q_last.cpu().numpy(), L, lo, oinit, 11)
        hist, c, done = [], 0, False
        while not done:
            c += 1
            _say(f"7b: loop iteration {c}, {len(hist)} tokens fixed")
            lg = g.logits(d_o)
            Le = min(L, N - len(hist))
            a, nd, pn = oracle.verify(lg[:Le], p_o[:Le], d_o[:Le], lo, osmp, oinit, len(hist), np.array(hist, np.int32), 11, c)
            hist += [int(t) for t in d_o[:a]]
            d_o = np.concatenate([nd, d_o[Le:]]).astype(np.int32); p_o = np.concatenate([pn, p_o[Le:]])
            done = len(hist) >= N - 1
            B.sjd_decode_steps(g.m, g.kv, 1)
            fixed, steps, gdone = B.sjd_decode_status(g.kv)
            assert fixed == len(hist) and steps == c and gdone == done, (c, fixed, len(hist))
            assert c < 2 * N
        toks, st = B.sjd_decode_result(g.kv, N)
        want_toks = np.array(hist[:N], np.int32)
        if len(want_toks) < N:
            want_toks = np.append(want_toks, d_o[0]).astype(np.int32)
        assert np.array_equal(toks, want_toks) and st.steps == c
    finally:
        g.close(); om.close()


def test_graph_replay_equals_eager_and_is_deterministic(B):
    """The decode loop replays one captured iteration; every replay must give what the kernel-by-kernel
    path gives, run after run (the loop state lives on the device, nothing is baked into the graph)."""
    shape = synth.ModelShape(3, 512, 8, 1024, 4096, 2048, 4096, 400, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9)
    g = Gpu(B, shape, blob)
    try:
        prompt = synth.random_tokens(40, 0, 2048, seed=1)
        smp = B.sjd_sampler(500, 1.0); init = B.sjd_init(0, 16, -1)
        outs = []
        for use_graph in (True, False, True):
            B.sjd_kv_use_graph(g.kv, use_graph)
            for seed in (1, 2):
                _say(f"graph={use_graph} seed={seed}")
                toks, st = B.sjd_generate(g.m, g.kv, prompt, None, 200, 16, smp, init, seed)
                outs.append((use_graph, seed, toks, st.steps))
        ref = {s: (t, n) for ug, s, t, n in outs if not ug}
        for ug, s, t, n in outs:
            assert np.array_equal(t, ref[s][0]) and n == ref[s][1], (ug, s)
        # stepping in pieces (status polled in between) gives the same stream as one go
        q_first = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        B.sjd_kv_use_graph(g.kv, True)
        B.sjd_prefill(g.m, g.kv, prompt, None, smp, init, q_first)
        B.sjd_decode_begin(g.m, g.kv, q_first, 200, 16, smp, init, 1)
        done, guard = False, 0
        while not done:
            B.sjd_decode_steps(g.m, g.kv, 3)
            fixed, steps, done = B.sjd_decode_status(g.kv)
            guard += 1
            assert guard < 200
        toks, st = B.sjd_decode_result(g.kv, 200)
        assert np.array_equal(toks, ref[1][0]) and st.steps == ref[1][1]
    finally:
        g.close()


def test_two_handles_on_two_streams(B):
    """two generations of one model, each on its own stream with its own handle, enqueued alternately
    without waiting: the weights are shared and read-only, everything else is per handle, so both must
    produce what they produce alone"""
    shape = synth.ModelShape(3, 512, 8, 1024, 4096, 2048, 4096, 300, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=9)
    m = B.sjd_init_model(B.config_from_shape(shape), blob)
    kvs = [B.sjd_kv_create(m) for _ in range(2)]
    try:
        prompts = [synth.random_tokens(30 + 11 * i, 0, 2048, seed=20 + i) for i in range(2)]
        smp = B.sjd_sampler(500, 1.0); init = B.sjd_init(4, 12, 4095)
        N, L = 12 * 10, 16
        alone = [B.sjd_generate(m, kvs[i], prompts[i], None, N, L, smp, init, 5 + i)[0] for i in range(2)]
        streams = [torch.cuda.Stream() for _ in range(2)]
        q = [torch.empty(shape.v_s, dtype=torch.float32, device="cuda") for _ in range(2)]
        for i in range(2):
            B.sjd_prefill(m, kvs[i], prompts[i], None, smp, init, q[i], stream=streams[i])
            B.sjd_decode_begin(m, kvs[i], q[i], N, L, smp, init, 5 + i, stream=streams[i])
        done, rounds = [False, False], 0
        while not all(done):
            for i in range(2):                       # a few iterations each, no synchronisation in between
                if not done[i]:
                    B.sjd_decode_steps(m, kvs[i], 3, stream=streams[i])
            for i in range(2):
                done[i] = B.sjd_decode_status(kvs[i])[2]
            rounds += 1
            assert rounds < 200
        for i in range(2):
            toks, _ = B.sjd_decode_result(kvs[i], N)
            assert np.array_equal(toks, alone[i]), i
    finally:
        for kv in kvs:
            B.sjd_kv_free(kv)
        B.sjd_free_model(m)


def test_sampled_initialisers_graph_replay(B):
    """initialisers (c) and (d) inside the captured iteration (the ring of recorded distributions lives
    on the handle): replay == kernel-by-kernel, and switching initialisers re-captures"""
    shape = synth.ModelShape(2, 256, 4, 512, 2048, 1024, 2048, 300, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=8)
    g = Gpu(B, shape, blob)
    try:
        prompt = synth.random_tokens(20, 0, 1024, seed=1)
        smp = B.sjd_sampler(300, 1.0)
        res = {}
        for use_graph in (True, False):
            B.sjd_kv_use_graph(g.kv, use_graph)
            for mode, stride in ((4, 9), (3, 9), (4, 20), (0, 9)):
                _say(f"graph={use_graph} init mode={mode} stride={stride}")
                toks, st = B.sjd_generate(g.m, g.kv, prompt, None, 9 * 20, 16, smp, B.sjd_init(mode, stride, 2047), 3)
                res[(use_graph, mode, stride)] = (toks, st.steps)
                assert np.all(toks[stride - 1::stride] == 2047)
        for mode, stride in ((4, 9), (3, 9), (4, 20), (0, 9)):
            a, b = res[(True, mode, stride)], res[(False, mode, stride)]
            assert np.array_equal(a[0], b[0]) and a[1] == b[1], (mode, stride)
    finally:
        g.close()


def test_forward_bf16_cache_of_a_1024_image(B):
    """a cache as long as the 64 x 64 grid needs (about 4200 positions: 132 blocks of 32 per head, 16 key
    splits of 8-9 blocks), windows of 16 at its far end"""
    shape = synth.ModelShape(2, 512, 4, 1024, 4096, 2048, 4096, 4256, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=12)
    prompt = synth.random_tokens(4190, 0, 2048, seed=1)
    toks = synth.random_tokens(64, 2048, 4096, seed=2)
    windows = [(toks[:16], 16), (toks[16:32], 3), (toks[32:48], 16), (toks[48:64], 1)]
    worst = _check_forward(B, shape, blob, prompt, windows, TOL_BF16)
    _say(f"bf16 4200-position cache worst {worst:.3e}")


# ------------------------------------------------------------------ long caches, wide windows, ragged ends
def test_forward_bf16_long_cache_window32(B):
    """head size 128, window 32, a cache of ~2300 positions (16 key splits, many 32-position blocks, a
    ragged last block) and windows that start at every residue of the block size"""
    shape = synth.ModelShape(2, 512, 4, 1024, 4096, 2048, 4096, 2450, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=11)
    prompt = synth.random_tokens(2290, 0, 2048, seed=1)
    toks = synth.random_tokens(160, 2048, 4096, seed=2)
    windows = [(toks[:32], 1), (toks[32:64], 31), (toks[64:96], 32), (toks[96:113], 17), (toks[113:114], 1),
               (toks[114:146], 5)]
    worst = _check_forward(B, shape, blob, prompt, windows, TOL_BF16)
    _say(f"bf16 long cache worst {worst:.3e}")


def test_forward_bf16_windows_above_32_rows(B):
    """windows of 33 .. 128 rows (span projections, whole and in K-slices; attention in query groups of 32) on a cache
    that grows past several 32-position blocks, and a prompt pre-filled in chunks of 128 rows"""
    shape = synth.ModelShape(4, 256, 4, 512, 2048, 1024, 2048, 700, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=7)
    prompt = synth.random_tokens(300, 0, 1024, seed=1)          # chunks of 128 + 128 + 44 rows
    toks = synth.random_tokens(400, 1024, 2048, seed=2)
    windows = [(toks[:64], 9), (toks[64:112], 48), (toks[112:145], 33), (toks[145:273], 128), (toks[273:370], 1),
               (toks[300:364], 64)]
    worst = _check_forward(B, shape, blob, prompt, windows, TOL_BF16)
    _say(f"bf16 wide windows worst {worst:.3e}")
    # head size 128 and 32, d_model 96 (6 partial sums of squares per token), non-unit gains
    for shape in (synth.ModelShape(2, 512, 4, 1024, 4096, 2048, 4096, 500, synth.DTYPE_BF16),
                  synth.ModelShape(2, 96, 3, 160, 512, 0, 512, 500, synth.DTYPE_BF16, rope_theta=1e6, rms_eps=3e-3)):
        blob = _random_gains(shape, synth.make_weights(shape, seed=9, std=0.05), 13)
        prompt = synth.random_tokens(150, 0, shape.samp_lo or 512, seed=1)
        toks = synth.random_tokens(300, shape.samp_lo, shape.samp_hi, seed=2)
        worst = _check_forward(B, shape, blob, prompt, [(toks[:64], 64), (toks[64:164], 7), (toks[100:228], 128)], TOL_BF16)
        _say(f"bf16 wide windows d={shape.d_model} worst {worst:.3e}")


def test_forward_bf16_7b_dims_two_layers_wide(B):
    """the 7B layer shapes with two layers: windows of 64 and 128 rows, and a 70-token prompt (one wide chunk)"""
    shape = synth.ModelShape(2, 4096, 32, 11008, 65536, 57344, 65536, 400, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=0, threads=16)
    prompt = synth.random_tokens(70, 0, 57344, seed=1)
    toks = synth.random_tokens(200, 57344, 65536, seed=2)
    worst = _check_forward(B, shape, blob, prompt, [(toks[:64], 5), (toks[64:192], 128)], TOL_BF16)
    _say(f"7b dims, 2 layers, wide windows worst {worst:.3e}")


def test_step_and_generation_with_window_64(B):
    """sjd_step with a window of 64 on a bf16 model: verification bit-exact given the GPU's logits (the accept
    scan over all 64 lanes), cache advance; then whole generations through the graph loop: valid tokens"""
    shape = synth.ModelShape(2, 256, 4, 512, 2048, 1024, 2048, 400, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=8)
    g = Gpu(B, shape, blob)
    try:
        V, lo, L, K = shape.v_s, shape.samp_lo, 64, 300
        smp = B.sjd_sampler(K, 1.0); init = B.sjd_init(1, 16, 2047)
        osmp = oracle.Sampler(K, 1.0); oinit = oracle.Init(1, 16, 2047)
        prompt = synth.random_tokens(20, 0, 1024, seed=1)
        q_last = torch.empty(V, dtype=torch.float32, device="cuda")
        B.sjd_prefill(g.m, g.kv, prompt, None, smp, init, q_last)
        draft = torch.zeros(L, dtype=torch.int32, device="cuda")
        p_old = torch.zeros((L, V), dtype=torch.float32, device="cuda")
        B.sjd_first_window(g.m, q_last, L, init, 42, draft, p_old)
        na = torch.zeros(1, dtype=torch.int32, device="cuda")
        nd = torch.zeros(L, dtype=torch.int32, device="cuda"); pn = torch.zeros_like(p_old)
        hist, n = [], 20
        for c in range(1, 7):
            _say(f"  L=64 step {c} n={n}")
            d_h, p_h = draft.cpu().numpy(), p_old.cpu().numpy()
            logits = g.logits(d_h)
            want = oracle.verify(logits, p_h, d_h, lo, osmp, oinit, len(hist), np.array(hist, np.int32), 42, c)
            B.sjd_step(g.m, g.kv, draft, p_old, L, smp, init, len(hist), 42, c, na, nd, pn)
            torch.cuda.synchronize()
            a = int(na.item())
            assert a == want[0]
            assert np.array_equal(nd.cpu().numpy(), want[1])
            assert np.array_equal(pn.cpu().numpy().view(np.uint32), want[2].view(np.uint32))
            hist += d_h[:a].tolist()
            n += a
            assert B.sjd_kv_len(g.kv) == n
            draft, nd = nd, draft; p_old, pn = pn, p_old
        # greedy decoding with a window of 64 = greedy AR of the GPU's own forward (Jacobi fixed point)
        N = 96
        t64, s64 = B.sjd_generate(g.m, g.kv, prompt, None, N, 64, B.sjd_sampler(1, 1.0), B.sjd_init(0, 16, -1), 3)
        t1, s1 = B.sjd_generate(g.m, g.kv, prompt, None, N, 1, B.sjd_sampler(1, 1.0), B.sjd_init(0, 16, -1), 3)
        assert s1.steps == N - 1 and s64.steps <= N - 1
        # (bf16 logits of a 64-row and of a 1-row forward differ in the last bits: identical unless an arg-max
        # is a near tie, which the seeds here do not hit)
        assert np.array_equal(t64, t1)
        toks, st = B.sjd_generate(g.m, g.kv, prompt, None, N, 64, smp, init, 5)
        assert toks.min() >= lo and toks.max() < shape.samp_hi and np.all(toks[15::16] == 2047)
        hist_ = np.array(list(st.accept_hist))
        assert hist_.sum() == st.steps and int((hist_ * np.arange(65)).sum()) in (N - 1, N)
    finally:
        g.close()


def test_forward_bf16_7b_dims_two_layers(B):
    """the 7B layer shapes (d 4096, 32 heads of 128, FFN 11008, 8192 sampled codes at the top of a 65536
    vocabulary) with two layers, windows of 16 and 32 rows"""
    shape = synth.ModelShape(2, 4096, 32, 11008, 65536, 57344, 65536, 200, synth.DTYPE_BF16)
    blob = synth.make_weights(shape, seed=0, threads=16)
    prompt = synth.random_tokens(70, 0, 57344, seed=1)
    toks = synth.random_tokens(64, 57344, 65536, seed=2)
    worst = _check_forward(B, shape, blob, prompt, [(toks[:16], 3), (toks[16:48], 32), (toks[48:49], 1)], TOL_BF16)
    _say(f"7b dims, 2 layers worst {worst:.3e}")


@pytest.mark.parametrize("N,L", [(1, 8), (2, 8), (5, 16), (9, 1), (33, 32)])
def test_generate_ragged_ends_fp32(B, N, L):
    """images shorter than the window, a single token, window 1: token identity with the oracle"""
    w = synth.WORKLOADS["tiny"]
    blob = synth.make_weights(w.shape, seed=0)
    prompt = synth.random_tokens(1, 0, 1024, seed=5)       # a one-token prompt
    om = oracle.Model(w.shape, blob)
    g = Gpu(B, w.shape, blob)
    try:
        osmp = oracle.Sampler(w.top_k, w.temperature); oinit = oracle.Init(1, 3, -1)
        lp = om.prefill(prompt)
        want, wst = om.generate_sjd(1, lp, N, L, osmp, oinit, 4)
        got, st = B.sjd_generate(g.m, g.kv, prompt, None, N, L, B.sjd_sampler(w.top_k, w.temperature),
                                 B.sjd_init(1, 3, -1), 4)
        assert np.array_equal(got, want)
        assert st.steps == wst.steps
    finally:
        g.close(); om.close()
