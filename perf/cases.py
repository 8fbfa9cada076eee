"""What is timed: the calls an image-generation program makes into this library, over the sizes it makes them with.

A case is one call (or, for a generation, one image) through the entry points of `paper_2410_01699_amd.binding`:

  window    Step 2 of one decoding iteration: one forward of `L` draft tokens for `images` images over `n` cached
            positions each, logits out; `guided` adds the unconditional context with `n_u` cached positions
  prefill   a prompt of `ids` token ids and `embeds` embedding rows into an empty cache, first distribution out
  verify    Steps 3-4 of one iteration from its logits: accept, resample, refresh, slide
  generate  prompt to `N` image tokens

Models are the repository's own workloads (synth.WORKLOADS) with random weights: "tiny" (fp32, 2 layers), "775m"
(24 layers, bf16) and the 7B decoder with the cache lengths of its 32 x 32, 48 x 48 and 64 x 64 grids.  A program
loads its model once, so a model is kept per process and its weights do not depend on the case's seed; prompts,
cached tokens, drafts, distributions and random streams do.
"""
from __future__ import annotations

import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from paper_2410_01699_amd import binding as B
from paper_2410_01699_amd import synth

MAX_ROWS = B.SJD_MAX_ROWS


def listed():
    return [
        # the smallest program: a whole 8 x 8 image of the two-layer fp32 decoder; bound by launches and latency
        dict(name="tiny_image", kind="generate", model="tiny", ids=16, N=64, L=8, top_k=64),
        # one iteration's forward of the 775M decoder in the middle of an image: 5-25 MB per projection
        dict(name="775m_window16", kind="window", model="775m", images=1, L=16, n=633, guided=False),
        # four images of it side by side, the way a server fills the card with a small model
        dict(name="775m_batch4", kind="window", model="775m", images=4, L=16, n=377, guided=False),
        # its prompt: one class id and 120 text-embedding rows (odd, and a mixed prompt)
        dict(name="775m_prompt121", kind="prefill", model="775m", ids=1, embeds=120, top_k=2000),
        # the auto-regressive step of the 7B decoder: one token
        dict(name="7b_token", kind="window", model="7b_32x32", images=1, L=1, n=301, guided=False),
        # the headline: a window of 16 drafts in the middle of a 32 x 32 image
        dict(name="7b_window16", kind="window", model="7b_32x32", images=1, L=16, n=583, guided=False),
        # the same late in a 64 x 64 image: the cache is what grows
        dict(name="7b_window16_long", kind="window", model="7b_64x64", images=1, L=16, n=3967, guided=False),
        # a window of 32 on the 48 x 48 grid
        dict(name="7b_window32", kind="window", model="7b_48x48", images=1, L=32, n=1239, guided=False),
        # the text-to-image setting: guidance, so two contexts of 32 drafts each in one forward
        dict(name="7b_guided32", kind="window", model="7b_48x48", images=1, L=32, n=1239, guided=True, n_u=1177),
        # the largest: eight images of 16 drafts in one forward
        dict(name="7b_batch8", kind="window", model="7b_32x32", images=8, L=16, n=583, guided=False),
        # a text prompt of 64 tokens on the 7B decoder
        dict(name="7b_prompt64", kind="prefill", model="7b_32x32", ids=64, embeds=0, top_k=2000),
        # the probabilistic test and the slide of one 7B window, from its logits
        dict(name="verify_7b", kind="verify", V=8192, L=16, top_k=2000),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _drawn(rng):
    kind = rng.choice(["window", "window", "window", "window", "prefill", "verify", "generate"])
    if kind == "generate":
        return dict(kind=kind, model="tiny", ids=rng.randint(1, 16), N=rng.randint(8, 64), L=rng.randint(1, 32), top_k=rng.choice([1, 16, 64, 200, 1024]))
    if kind == "verify":
        V = rng.choice([8192, 16384])
        return dict(kind=kind, V=V, L=rng.randint(2, 64 if V == 8192 else 32), top_k=_log_int(rng, 1, V))
    if kind == "prefill":
        model = rng.choice(["775m", "7b_32x32"])
        ids = rng.randint(1, 128)
        return dict(kind=kind, model=model, ids=ids, embeds=rng.randint(0, 128 - ids), top_k=rng.randint(2000, 8192))
    model = rng.choice(["775m", "7b_32x32", "7b_48x48", "7b_64x64"])
    images, guided = rng.choice([1, 1, 1, 2, 3, 4, 8]), rng.random() < 0.3
    contexts = images * (2 if guided else 1)
    if contexts > 8:
        images, contexts = 4, 8
    L = _log_int(rng, 1, min(B.SJD_MAX_WINDOW, 1 << int(math.log2(MAX_ROWS // contexts))))
    n = rng.randint(65, synth.WORKLOADS[model].shape.max_seq - L)
    c = dict(kind=kind, model=model, images=images, L=L, n=n, guided=guided)
    if guided:
        c["n_u"] = max(1, n - rng.randint(0, 63))
    return c


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _drawn(rng)
        if _cost(c) <= most:
            return c


# ---- what a program keeps ---------------------------------------------------------------------------------------
_models: dict = {}


def _weights(shape):
    """Random-init weights as synth.make_weights describes them (matrices N(0, 0.02^2), gains 1); large bf16 blobs
    repeat one drawn block whose length is a prime, so that no two rows of a matrix are alike."""
    if shape.n_params() < 1 << 26:
        return synth.make_weights(shape, seed=0)
    block = np.empty(16777213, np.uint16)
    synth._fill_normal(block, 0, 0, 0.02, 8)
    blob = np.empty(shape.n_params(), np.uint16)
    spans = [(o, min(o + block.size, blob.size)) for o in range(0, blob.size, block.size)]

    def fill(s):
        blob[s[0]:s[1]] = block[:s[1] - s[0]]

    with ThreadPoolExecutor(8) as ex:
        list(ex.map(fill, spans))
    for _, (off, shp) in synth.tensor_offsets(shape).items():
        if len(shp) == 1:
            blob[off:off + shp[0]] = 0x3F80
    return blob


def _model(name):
    if name not in _models:
        shape = synth.WORKLOADS[name].shape
        _models[name] = B.sjd_init_model(B.config_from_shape(shape), _weights(shape))
    return _models[name]


class _State:
    """what a program holds for one case: cache handles and buffers"""

    def __init__(self, case):
        self.case, self.kvs = case, []

    def handle(self, m):
        self.kvs.append(B.sjd_kv_create(m))
        return self.kvs[-1]

    def __del__(self):
        for kv in self.kvs:             # (waits for the device: freeing memory does)
            B.sjd_kv_free(kv)


def _ids(rng, shape, count, image):
    lo, hi = (shape.samp_lo, shape.samp_hi) if image else (0, shape.samp_lo or shape.vocab_total)
    return rng.integers(lo, hi, size=count, dtype=np.int32)


def _prompt_and_image(rng, shape, n):
    """ids of a cache of n positions: a prompt of 64, the rest image tokens"""
    p = min(64, n)
    return np.concatenate([_ids(rng, shape, p, False), _ids(rng, shape, n - p, True)])


def prepare(case, seed):
    rng = np.random.Generator(np.random.SFC64([seed, 0x5EED]))
    st = _State(case)
    kind = case["kind"]
    if kind == "verify":
        _prepare_verify(st, case, seed)
        return st
    w = synth.WORKLOADS[case["model"]]
    shape = w.shape
    st.m = _model(case["model"])
    st.init = B.sjd_init(w.init_mode, w.row_stride, w.eol_id)
    if kind == "window":
        smp = B.sjd_sampler(w.top_k, w.temperature)
        q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        for _ in range(case["images"]):
            kv = st.handle(st.m)
            B.sjd_prefill(st.m, kv, _prompt_and_image(rng, shape, case["n"]), None, smp, st.init, q)
            if case["guided"]:
                B.sjd_prefill_uncond(st.m, kv, _prompt_and_image(rng, shape, case["n_u"]), None, 3.0, smp, st.init, q)
        toks = _ids(rng, shape, case["images"] * case["L"], True)
        st.tokens = torch.from_numpy(toks).cuda().view(case["images"], case["L"])
        # (room for whole operand tiles behind the rows that are asked for: a forward computes 16 rows at a time)
        rows = torch.empty((MAX_ROWS, shape.v_s), dtype=torch.float32, device="cuda")
        st.logits = rows[:case["images"] * case["L"]].view(case["images"], case["L"], shape.v_s)
    else:
        st.smp = B.sjd_sampler(case["top_k"], w.temperature)
        st.handle(st.m)
        st.ids, st.embeds = _ids(rng, shape, case["ids"], False), None
        if case.get("embeds"):
            e = rng.standard_normal((case["embeds"], shape.d_model), dtype=np.float32) * np.float32(0.02)
            st.embeds = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(e)).reshape(e.shape)
        st.q = torch.empty(shape.v_s, dtype=torch.float32, device="cuda")
        st.seed = int(rng.integers(0, 1 << 62))
    torch.cuda.synchronize()
    return st


def _prepare_verify(st, case, seed):
    """This iteration's logits have the scale of a random-init LM head; the distributions the drafts were drawn from
    are those of an iteration before, so close that a few drafts in a row are accepted."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    L, V = case["L"], case["V"]
    st.logits = torch.randn((L, V), generator=g, device="cuda") * 1.28
    before = torch.randn((L, V), generator=g, device="cuda") * 1.28
    before[1:] = st.logits[:-1] + 0.3 * torch.randn((L - 1, V), generator=g, device="cuda")
    kth = before.topk(min(case["top_k"], V), dim=1).values[:, -1:]
    st.p_old = torch.softmax(before.masked_fill(before < kth, -math.inf), dim=1).contiguous()
    st.draft = torch.multinomial(st.p_old, 1, generator=g).view(L).to(torch.int32)
    st.n_accepted = torch.zeros(1, dtype=torch.int32, device="cuda")
    st.new_draft = torch.zeros(L, dtype=torch.int32, device="cuda")
    st.p_new = torch.zeros((L, V), device="cuda")
    st.smp, st.init = B.sjd_sampler(case["top_k"], 1.0), B.sjd_init(0, 32, -1)
    st.seed = int(torch.randint(0, 1 << 62, (1,), generator=g, device="cuda"))


def run(st):
    c = st.case
    if c["kind"] == "window":
        if c["images"] == 1:
            B.sjd_forward_logits(st.m, st.kvs[0], st.tokens, c["L"], st.logits)
        else:
            B.sjd_forward_logits_batch(st.m, st.kvs, st.tokens, c["L"], st.logits)
        return st.logits
    if c["kind"] == "prefill":
        B.sjd_prefill(st.m, st.kvs[0], st.ids, st.embeds, st.smp, st.init, st.q)
        return st.q
    if c["kind"] == "generate":
        tokens, stats = B.sjd_generate(st.m, st.kvs[0], st.ids, st.embeds, c["N"], c["L"], st.smp, st.init, st.seed)
        return tokens, stats.steps
    # the call that allocates nothing where its scratch is large enough, as a serving loop would choose
    fits = (c["L"] + 1) * c["V"] <= B.SJD_STATIC_VERIFY_FLOATS
    verify = B.sjd_verify_static if fits else B.sjd_verify
    verify(st.logits, st.p_old, st.draft, c["L"], c["V"], 0, st.smp, st.init, 0, None, st.seed, 1, st.n_accepted,
           st.new_draft, st.p_new)
    return st.n_accepted, st.new_draft, st.p_new


# ---- what a pass cannot do without ------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "verify":
        # logits and the old distributions in, the new ones out
        return {"bytes": 3.0 * 4 * case["L"] * case["V"], "flops": 10.0 * case["L"] * case["V"]}
    s = synth.WORKLOADS[case["model"]].shape
    es = 4 if s.dtype == synth.DTYPE_F32 else 2
    head = s.v_s * s.d_model
    params = s.layer_param_count() + head
    per_pos = 2 * s.n_layers * s.d_model * es                      # K and V of one cached position
    if kind == "window":
        rows = case["images"] * case["L"]
        keys = case["images"] * (case["n"] + case["L"])
        pairs = case["images"] * case["L"] * (case["n"] + (case["L"] + 1) / 2)
        if case["guided"]:
            rows *= 2
            keys += case["images"] * (case["n_u"] + case["L"])
            pairs += case["images"] * case["L"] * (case["n_u"] + (case["L"] + 1) / 2)
        return {"bytes": es * params + keys * per_pos + 4.0 * case["images"] * case["L"] * s.v_s,
                "flops": 2.0 * params * rows + 4.0 * s.n_layers * s.d_model * pairs}
    if kind == "prefill":
        # one pass over the weights, the cache written, one row of logits
        P = case["ids"] + case["embeds"]
        return {"bytes": es * params + P * per_pos + 4.0 * s.v_s,
                "flops": 2.0 * s.layer_param_count() * P + 2.0 * head + 2.0 * s.n_layers * s.d_model * P * (P + 1)}
    # a generation: the prompt, then at least N / L window forwards, each over the weights
    forwards = 1 + math.ceil((case["N"] - 1) / case["L"])
    return {"bytes": float(forwards * es * params), "flops": 2.0 * params * (case["ids"] + case["N"])}


def tolerance(case):
    if case["kind"] in ("verify", "generate"):
        # tokens, counts, and distributions made of correctly rounded operations in a fixed order
        return "exact"
    if case["kind"] == "window":
        # the same rows through kernels that add in another order differ by 2.7e-5 (775M) and 9.4e-5 (7B), at most
        # 4.6e-4 of the root mean square in one logit
        return {"rel": 4e-4, "max": 2e-3}
    # as above, and logits that close can change places at the edge of the top-2000: one such swap is 8e-3 of the
    # distribution's norm and 0.54 of its root mean square
    return {"rel": 0.03, "max": 0.9}
