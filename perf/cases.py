"""What a program built on this framework has it do, as cases that can be timed: decode steps that verify drafts, plain
decode, prefill through the verify step, filtered sampling, the sampler on a caller's own logits and the cache import /
export, over the model shapes of paper_2605_08862_amd/workloads.py at full depth and with the full vocabulary.

Everything is synthetic and made on the GPU from the seed.  A random-init decoder has a nearly flat next-token law,
under which a sampled token is decided by the last bit of the logits; a trained policy is peaked.  So the models here
are peaked: the embedding of a token dominates the residual stream, and the LM head row of token t + 1 carries a
multiple of the embedding of token t, which puts nearly all of the mass on the successor of the last token.  A draft
block is a chain of successors that breaks with probability 1 - agreement per position (the break is a uniformly random
token), so the accepted lengths are geometric, as with drafts from an earlier policy, and they follow from the inputs
and not from rounding."""
import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine

DEVICE = "cuda:0"
EMBED_STD = 32.0                 # residual stream: the token's embedding outweighs the sum of the layers' outputs
PEAK = 12.0                      # log odds of the successor token against the rest of the vocabulary
MAX_MATCH, MIN_MATCH = 4, 1      # draft lookup: longest and shortest suffix tried
POOL_MEDIAN = 8192               # tokens of a pre-generated rollout (lognormal)
MAX_CONTEXT = 32768

# per shape: most packed rows of a step and most cached tokens of a drawn case
LIMITS = {"tiny": (256, 1 << 16), "mini_bf16": (1024, 1 << 18), "s1p5b": (3900, 2000000), "s7b": (1150, 600000)}


def _step(name, shape, batch, context, k, proposal, agreement, ragged=False, spread=0.0, top_k=0, top_p=1.0):
    return dict(name=name, path="step", shape=shape, batch=batch, context=context, spread=spread, k=k, ragged=ragged,
                proposal=proposal, agreement=agreement, top_k=top_k, top_p=top_p)


def listed():
    return [
        # the float32 model on a handful of short sequences: what a test or a first integration runs; all latency
        _step("tiny_f32_b4_k4", "tiny", 4, 128, 4, "onehot", 0.6),
        # one interactive sequence on the small bf16 decoder: weights are streamed once per step
        _step("s1p5b_b1_c1000_k8", "s1p5b", 1, 1000, 8, "onehot", 0.7),
        # the end of a rollout phase, where speculation pays most: a few long sequences left, drafts from the pool
        _step("s7b_b8_c20000_k16_lookup", "s7b", 8, 20000, 16, "lookup", 0.8, spread=0.3),
        # plain decoding of a mid-sized batch (how the pool's rollouts themselves are generated)
        _step("s7b_b64_c4096_k0", "s7b", 64, 4096, 0, "onehot", 0.5),
        # uniform verify batches with a dense proposal
        _step("s1p5b_b64_c2048_k8", "s1p5b", 64, 2048, 8, "dense", 0.7),
        _step("s7b_b32_c8192_k8", "s7b", 32, 8192, 8, "dense", 0.5),
        # the long-tail batch: contexts and draft lengths differ by sequence
        _step("s7b_longtail_b128_k0to16", "s7b", 128, 4096, 16, "dense", 0.6, ragged=True, spread=1.0),
        # the widest batch: samples of 32 prompts, drafts looked up in the step
        _step("s1p5b_pool_b256_c8192_k16", "s1p5b", 256, 8192, 16, "lookup", 0.7),
        # top-k and top-p on
        _step("s1p5b_b48_c1500_k8_filtered", "s1p5b", 48, 1500, 8, "dense", 0.7, top_k=50, top_p=0.9),
        # prompts go through the verify step in chunks: forced drafts, everything is committed, nothing is sampled
        dict(name="s1p5b_prefill_b61_c512", path="prefill", shape="s1p5b", batch=61, context=512, spread=0.5, k=16),
        # a program with its own model that uses the sampler alone, without a context
        dict(name="sampler_b128_k8_v151936", path="sampler", vocab=151936, batch=128, k=8, temperature=0.8),
        # a sequence is swapped in and out of the cache
        dict(name="s1p5b_kv_swap_n1900", path="kv", shape="s1p5b", rows=1900, offset=37),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))


def draw(rng):
    path = rng.choice(["step"] * 8 + ["prefill", "sampler", "kv"])
    if path == "sampler":
        k = rng.randint(0, 16)
        return dict(path="sampler", vocab=_log_int(rng, 1000, 152064), batch=_log_int(rng, 1, 1024 // (k + 1)), k=k,
                    temperature=round(rng.uniform(0.5, 1.2), 2))
    if path == "kv":
        rows = _log_int(rng, 16, 4000)
        return dict(path="kv", shape=rng.choice(["s1p5b", "s7b"]), rows=rows, offset=rng.randint(0, 500))
    shape = rng.choice(["tiny", "mini_bf16"] + ["s1p5b"] * 4 + ["s7b"] * 4)
    max_rows, max_tokens = LIMITS[shape]
    spread = rng.choice([0.0, 0.0, 0.3, 1.0])
    k = 16 if path == "prefill" else rng.choice([0, 4, 8, 16, rng.randint(1, 16)])
    ragged = path == "step" and rng.random() < 0.4               # draft lengths uniform in 0 .. k: half the rows
    batch = _log_int(rng, 1, min(256, (2 if ragged else 1) * max_rows // (k + 1)))
    context = _log_int(rng, 64, min(MAX_CONTEXT // (4 if spread else 1), int(max_tokens / batch / math.exp(spread ** 2 / 2))))
    if path == "prefill":
        return dict(path="prefill", shape=shape, batch=batch, context=context, spread=spread, k=k)
    filtered = rng.random() < 0.15 and batch * (k + 1) <= 1024
    c = _step("", shape, batch, context, k, rng.choice(["dense", "onehot", "lookup"]) if k else "onehot",
              round(rng.uniform(0.2, 0.9), 2), ragged=ragged, spread=spread,
              top_k=rng.choice([0, 50]) if filtered else 0, top_p=rng.choice([0.9, 0.95]) if filtered else 1.0)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _normal(shape, dtype, std, g):
    return torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, std, generator=g)


def _weights(desc, g):
    """Random-init decoder in the fused layout of the engine, N(0, 0.02), with the successor structure in the LM head."""
    td = W.torch_dtype(desc)
    d, D, F, V = desc["d_model"], desc["head_dim"], desc["d_ffn"], desc["vocab"]
    Hq, Hkv, L = desc["n_q_heads"], desc["n_kv_heads"], desc["n_layers"]
    mats = lambda r, c: [_normal((r, c), td, 0.02, g) for _ in range(L)]
    ones = lambda: torch.ones(d, dtype=torch.float32, device=DEVICE)
    embed = _normal((V, d), td, EMBED_STD, g)
    lm_head = _normal((V, d), td, 0.02, g)
    # logit of the successor ~ (log V + PEAK): the final norm leaves a vector of length sqrt(d) along the embedding
    lm_head.add_(torch.roll(embed, 1, 0), alpha=(math.log(V) + PEAK) / (d * EMBED_STD))
    return {"embed": embed, "lm_head": lm_head, "final_norm": ones(), "attn_norm": [ones() for _ in range(L)],
            "wqkv": mats((Hq + 2 * Hkv) * D, d), "wo": mats(d, Hq * D), "mlp_norm": [ones() for _ in range(L)],
            "w_gate_up": mats(2 * F, d), "w_down": mats(d, F)}


def _context_lengths(case, rng):
    """Quantiles of the clipped lognormal law around the median, in random order: every seed is the same amount of work."""
    n, c, s = case["batch"], case["context"], case["spread"]
    z = np.array([NormalDist().inv_cdf((i + 0.5) / n) for i in range(n)])
    return rng.permutation(np.clip(np.rint(c * np.exp(s * z)), max(1, c // 8), min(8 * c, MAX_CONTEXT)).astype(np.int64))


def _engine(desc, ctx, k, g):
    """Engine with weights and a committed random context (K, V at the scale of projected unit-RMS rows, rounded to bf16
    where the model is; pages are filled in place, their order does not matter for independent values)."""
    eng = Engine(desc, _weights(desc, g), len(ctx), 0, B_max=len(ctx), k_max=k, slot_tokens=[int(c) + k + 1 for c in ctx],
                 page_perm_seed=int(ctx.sum()) & 0xffff)
    std = 0.02 * math.sqrt(desc["d_model"])
    for pages in eng.k_pages + eng.v_pages:
        if desc["dtype"] == B.BS_F32:
            pages.normal_(0.0, std, generator=g)
        else:
            pages.copy_(_normal(pages.shape, torch.bfloat16, std, g))
    eng.ctx_len.copy_(torch.tensor(ctx, dtype=torch.int32))
    return eng


def _chain(first, breaks, fresh, vocab):
    """Token rows [n, m]: successors of `first` [n], restarting at a fresh random token where breaks is set."""
    out = np.empty(breaks.shape, dtype=np.int64)
    cur = np.asarray(first, dtype=np.int64)
    for j in range(breaks.shape[1]):
        cur = np.where(breaks[:, j], fresh[:, j], (cur + 1) % vocab)
        out[:, j] = cur
    return out


def _pool(rng, n_prompts, agreement, vocab):
    """Rollouts of the earlier policy, 8 per prompt: chains of successors that break at random."""
    lens = np.clip(np.exp(rng.normal(math.log(POOL_MEDIAN), 1.0, 8 * n_prompts)), 256, 32768).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(lens)])
    n = int(off[-1])
    start = rng.random(n) >= agreement
    start[off[:-1]] = True
    at = np.arange(n)
    seg = np.maximum.accumulate(np.where(start, at, 0))
    toks = (rng.integers(0, vocab, n)[seg] + at - seg) % vocab
    return toks.astype(np.int32), off.astype(np.int64), (np.arange(n_prompts + 1) * 8).astype(np.int32)


def _i32(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.int32, device=DEVICE)


def _prepare_step(case, seed):
    desc = W.shape(case["shape"])
    n, k, V = case["batch"], case["k"], desc["vocab"]
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    ctx = _context_lengths(case, rng)
    eng = _engine(desc, ctx, k, g)
    st = dict(eng=eng, k=k, ctx0=_i32(ctx), slots=_i32(np.arange(n)), lookup=None, q_logits=None)
    last = rng.integers(0, V, n)
    k_b = rng.integers(0, k + 1, n) if case.get("ragged") else np.full(n, k)
    if case["path"] == "prefill":
        drafts = rng.integers(0, V, (n, k))
        st.update(last=_i32(last), drafts=_i32(drafts), draft_len=_i32(k_b), n_commit=_i32(k_b + 1))
        return st
    if case["proposal"] == "lookup":
        toks, off, prb = _pool(rng, max(1, n // 8), case["agreement"], V)
        prompt = np.minimum(np.arange(n) // 8, len(prb) - 2)
        tails = rng.integers(0, V, (n, MAX_MATCH))
        for b in np.flatnonzero(rng.random(n) < 0.8):            # 80 % of the sequences follow one of the rollouts
            r = rng.integers(prb[prompt[b]], prb[prompt[b] + 1])
            end = rng.integers(off[r] + MAX_MATCH, off[r + 1])
            tails[b] = toks[end - MAX_MATCH:end]
        eng.pool_bind(torch.from_numpy(toks), torch.from_numpy(off), torch.from_numpy(prb))
        eng.index_bind(B.bs_index_build(toks, off, prb))
        last = tails[:, -1]
        st["lookup"] = (_i32(prompt), _i32(tails))
    else:
        drafts = _chain(last, rng.random((n, k)) >= case["agreement"], rng.integers(0, V, (n, k)), V)
        st.update(drafts=_i32(drafts), draft_len=_i32(k_b))
        if case["proposal"] == "dense" and k_b.sum() > 0:
            q = _normal((int(k_b.sum()), V), W.torch_dtype(desc), 1.2, g)
            judged = np.concatenate([drafts[b, :k_b[b]] for b in range(n)])
            q[torch.arange(len(judged), device=DEVICE), torch.tensor(judged, device=DEVICE)] = math.log(V) + PEAK
            st["q_logits"] = q
    ua, us = W.uniforms(seed, n, k)
    st.update(last=_i32(last), ua=torch.tensor(ua).to(DEVICE), us=torch.tensor(us).to(DEVICE))
    if case["top_k"] > 0 or case["top_p"] < 1.0:
        eng.set_filter(case["top_k"], case["top_p"])
    return st


def _prepare_sampler(case, seed):
    n, k, V = case["batch"], case["k"], case["vocab"]
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    rows = torch.arange(n * (k + 1), device=DEVICE).view(n, k + 1)
    logits = _normal((n * (k + 1), V), torch.float32, 2.0, g)
    drafts = torch.zeros(n, k, dtype=torch.int32, device=DEVICE)
    q = None
    if k:
        q = torch.empty(n * k, V, dtype=torch.bfloat16, device=DEVICE)
        for b in range(n):                                        # a perturbed copy of the target, drafts sampled from it
            z = logits[rows[b, :k]] + _normal((k, V), torch.float32, 0.8, g)
            q[b * k:(b + 1) * k] = z
            gumbel = -torch.log(torch.empty_like(z).exponential_(generator=g))
            drafts[b] = (q[b * k:(b + 1) * k].float() + gumbel).argmax(1)
    ua, us = W.uniforms(seed, n, k)
    return dict(n=n, k=k, V=V, T=case["temperature"], logits=logits, q=q, drafts=drafts,
                draft_len=torch.full((n,), k, dtype=torch.int32, device=DEVICE), ua=torch.tensor(ua).to(DEVICE),
                us=torch.tensor(us).to(DEVICE))


def _prepare_kv(case, seed):
    desc = W.shape(case["shape"])
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    eng = _engine(desc, np.full(2, case["offset"] + case["rows"]), 0, g)
    shp = (case["rows"], desc["n_kv_heads"], desc["head_dim"])
    std = 0.02 * math.sqrt(desc["d_model"])
    return dict(eng=eng, offset=case["offset"], rows=case["rows"],
                kv=[(_normal(shp, torch.bfloat16, std, g), _normal(shp, torch.bfloat16, std, g)) for _ in range(desc["n_layers"])])


def prepare(case, seed):
    if case["path"] == "sampler":
        return _prepare_sampler(case, seed)
    if case["path"] == "kv":
        return _prepare_kv(case, seed)
    return _prepare_step(case, seed)


# ------------------------------------------------------------------------------------------------ one pass
def _run_sampler(st):
    n, k = st["n"], st["k"]
    new = lambda *s: torch.empty(s, dtype=torch.int32, device=DEVICE)
    out = dict(n_accepted=new(n), out_tokens=new(n, k + 1), n_emitted=new(n), near_tie=new(n))
    B.bs_accept_resample_logits_noalloc(n, st["V"], st["logits"], st["drafts"], st["draft_len"], k, st["q"], B.BS_BF16,
                                        st["T"], -1, True, st["ua"], st["us"], out["n_accepted"], out["out_tokens"],
                                        out["n_emitted"], out["near_tie"])
    return out


def _run_kv(st):
    eng = st["eng"]
    for l, (k, v) in enumerate(st["kv"]):
        eng.kv_write(l, 1, st["offset"], k, v)
    return [eng.kv_read(l, 1, st["offset"], st["rows"]) for l in range(len(st["kv"]))]


def run(st):
    """The cache pages of the last layer come back with the tokens: their new rows depend on all layers before it."""
    if "eng" not in st:
        return _run_sampler(st)
    if "kv" in st:
        return _run_kv(st)
    eng, k = st["eng"], st["k"]
    eng.ctx_len.copy_(st["ctx0"])                                 # every pass continues from the same committed state
    if st["lookup"] is not None:
        drafts, draft_len = eng.draft_lookup(*st["lookup"], MAX_MATCH, MIN_MATCH, k)
    else:
        drafts, draft_len = st["drafts"], st["draft_len"]
    eng.verify_step(st["slots"], st["last"], drafts, draft_len, k)
    if "n_commit" in st:                                          # prefill
        eng.kv_commit(st["slots"], st["n_commit"])
        out = {}
    else:
        out = eng.accept_resample(drafts, draft_len, k, st["ua"], st["us"], q_logits=st["q_logits"])
        eng.kv_commit(st["slots"], out["n_accepted"] + 1)
        out["draft_len"] = draft_len
    out["ctx_len"], out["k_pages"], out["v_pages"] = eng.ctx_len, eng.k_pages[-1], eng.v_pages[-1]
    return out


# ------------------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Weights, cached K/V, given logits and proposals read once, new K/V rows written once; 2 M N K of every contraction."""
    if case["path"] == "sampler":
        return {"bytes": case["vocab"] * case["batch"] * (4.0 * (case["k"] + 1) + 2.0 * case["k"]), "flops": 0.0}
    desc = W.shape(case["shape"])
    d, D, F, V, L = desc["d_model"], desc["head_dim"], desc["d_ffn"], desc["vocab"], desc["n_layers"]
    Hq, Hkv = desc["n_q_heads"], desc["n_kv_heads"]
    el = 4.0 if desc["dtype"] == B.BS_F32 else 2.0
    kv_row = 2.0 * L * Hkv * D * el
    if case["path"] == "kv":
        return {"bytes": 4.0 * kv_row * case["rows"], "flops": 0.0}
    n, s = case["batch"], case["spread"]
    drafts = n * case["k"] * (0.5 if case.get("ragged") else 0.85 if case.get("proposal") == "lookup" else 1.0)
    tokens = n * case["context"] * math.exp(min(s * s / 2, 0.36))            # mean of the clipped lognormal
    rows = n + drafts
    params = L * ((Hq + 2 * Hkv) * D * d + d * Hq * D + 3 * F * d)
    flops = 2.0 * rows * params + 4.0 * rows * tokens / n * L * Hq * D
    nbytes = params * el + kv_row * (tokens + 2 * rows) + rows * d * el
    if case["path"] == "step":
        nbytes += V * d * el + (drafts * V * el if case["proposal"] == "dense" else 0.0)
        flops += 2.0 * rows * V * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """float32 models and given logits: float32 sums.  bf16 models: float16 operands, K/V rounded to bf16 at rest (one
    rounding step of a large element is 0.03 of the root mean square).  Whole values: a uniform can fall within the
    rounding of a decision; with peaked laws that is rare, but a small output has few values."""
    if case["path"] == "kv":
        return "exact"
    if case["path"] == "sampler" or case["shape"] == "tiny":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.01}
    return {"rel": 1e-2, "max": 0.1, "differ": 0.01}
