"""GPU parity, bf16 decoders: MFMA GEMMs, ragged MFMA verify attention over the paged cache, fused
LM-head sampler.  Small shapes span several tiles and ragged tails; the 1.5B / 7B cases are two-layer
slices of the real per-layer shapes with the full vocabulary (the oracle finishes those in seconds)."""
import numpy as np
import pytest
import torch

from oracle import decoder as OD
from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine, fuse_weights
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _f64_weights(wn):
    c = lambda a: np.asarray(a, dtype=np.float64)
    return {"embed": wn["embed"], "lm_head": c(wn["lm_head"]), "final_norm": c(wn["final_norm"]),
            "layers": [{k: c(v) for k, v in lw.items()} for lw in wn["layers"]]}


def _run_case(desc, ctx_lens, k_b, k_max, seed, temperature=1.0, q_mode="dense", q_scale=0.8, perm=3,
              check_kv=True, unfused_qkv=False, after_step=None):
    """One verify step on random-filled contexts; returns stats after asserting all three tiers."""
    Bn = len(ctx_lens)
    rng = np.random.default_rng(seed)
    V = desc["vocab"]
    w = W.make_weights(desc, seed=seed)
    wn = _f64_weights(W.weights_to_numpy(w))
    eng = Engine(desc, fuse_weights(w, desc["dtype"], DEV), Bn, int(max(ctx_lens)) + k_max + 1, B_max=Bn,
                 k_max=k_max, page_perm_seed=perm)
    if unfused_qkv:
        B.bs_debug_unfused_qkv(eng.ctx, True)
    od = H.oracle_desc(desc)
    caches = []
    for b in range(Bn):
        kvs = W.context_kv(desc, int(ctx_lens[b]), seed * 100 + b)
        c = OD.SeqCache(od)
        c.fill([k.float().numpy() for k, _ in kvs], [v.float().numpy() for _, v in kvs])
        caches.append(c)
        if ctx_lens[b] > 0:
            for l, (k, v) in enumerate(kvs):
                eng.kv_write(l, b, 0, k.to(DEV), v.to(DEV))
    eng.ctx_len.copy_(H.dev_i32(ctx_lens))
    last = rng.integers(0, V, Bn)
    drafts = rng.integers(0, V, (Bn, k_max))
    k_b = np.asarray(k_b)
    blocks = H.pack_rows(last, drafts, k_b)
    ref_logits = np.concatenate([OD.verify_block(od, wn, caches[b], blocks[b]) for b in range(Bn)])
    M, Td = int(k_b.sum() + Bn), int(k_b.sum())
    q_rows = None
    if q_mode == "dense" and Td > 0:       # proposal: perturbed copy of the target logits at the judged rows
        rows = np.concatenate([np.arange(k_b[b]) + (k_b[:b].sum() + b) for b in range(Bn)]).astype(int)
        q_t = torch.tensor(ref_logits[rows] + q_scale * rng.normal(size=(Td, V)), dtype=torch.bfloat16)
        q_rows = q_t.float().numpy()
        # make most drafts plausible under q so that accept / reject / bonus all occur
        for b in range(Bn):
            for j in range(k_b[b]):
                if rng.random() < 0.8:
                    qq = OD.softmax(q_rows[k_b[:b].sum() + j])
                    drafts[b, j] = rng.choice(V, p=qq)
        blocks = H.pack_rows(last, drafts, k_b)
        for c, n in zip(caches, ctx_lens):          # redo the oracle pass with the final drafts
            c.commit(0)
        ref_logits = np.concatenate([OD.verify_block(od, wn, caches[b], blocks[b]) for b in range(Bn)])
    ua, us = W.uniforms(seed + 7, Bn, k_max)
    slots = H.dev_i32(np.arange(Bn))
    dt, dl = H.dev_i32(drafts), H.dev_i32(k_b)
    logits = eng.verify_step(slots, H.dev_i32(last), dt, dl, k_max, want_logits=True)
    if after_step is not None:
        after_step(eng)
    qdev = None if q_rows is None else q_t.to(DEV)
    out = eng.accept_resample(dt, dl, k_max, H.dev_f32(ua), H.dev_f32(us), q_logits=qdev, temperature=temperature)
    got = logits.cpu().numpy()[:M]
    err = np.abs(got - ref_logits).max()
    assert err <= H.TOL_LOGITS[W.BS_BF16], "logits max-abs %.4g" % err
    exact, near, res = H.compare_sampler(out, got, drafts, k_b, ua, us, q_rows, temperature)
    assert near <= max(1, 0.05 * Bn), (exact, near)
    if check_kv:
        for b in range(Bn):
            for l in range(desc["n_layers"]):
                k, v = eng.kv_read(l, b, int(ctx_lens[b]), int(k_b[b]) + 1)
                kr, vr = caches[b].k[l][ctx_lens[b]:], caches[b].v[l][ctx_lens[b]:]
                # both sides round to bf16 at rest: values that agree before rounding may land one bf16 step (2^-7
                # relative) apart, which exceeds the absolute bound once |x| > 2.5 (wide models)
                assert (np.abs(k.float().cpu().numpy() - kr) <= 2e-2 + 2.0 ** -7 * np.abs(kr)).all()
                assert (np.abs(v.float().cpu().numpy() - vr) <= 2e-2 + 2.0 ** -7 * np.abs(vr)).all()
    n_acc = out["n_accepted"].cpu().numpy()
    eng.kv_commit(slots, H.dev_i32(n_acc + 1))
    assert eng.ctx_len.cpu().tolist() == [int(c + n + 1) for c, n in zip(ctx_lens, n_acc)]
    assert eng.poll_status() == 0
    stats = dict(err=float(err), exact=exact, near=near, accepted=int(n_acc.sum()), drafts=Td,
                 emitted=int(out["n_emitted"].sum().item()))
    print(stats)
    eng.close()
    return stats


def test_mini_ragged_dense_q():
    desc = W.shape("mini_bf16")
    _run_case(desc, ctx_lens=[1, 63, 64, 200, 333, 0, 31, 97], k_b=[8, 0, 3, 8, 5, 2, 1, 7], k_max=8, seed=21)


def test_mini_unfused_qkv_path():
    """Head size 128 normally takes the fused QKV + rotary + append kernel; this runs the same case through
    the projection GEMM followed by the separate rotary / append kernel."""
    desc = W.shape("mini_bf16")
    _run_case(desc, ctx_lens=[1, 63, 64, 200, 333, 0, 31, 97], k_b=[8, 0, 3, 8, 5, 2, 1, 7], k_max=8, seed=21,
              unfused_qkv=True)


def test_mini_one_hot_and_temperature():
    desc = W.shape("mini_bf16")
    _run_case(desc, ctx_lens=[5, 130, 64, 257], k_b=[4, 4, 0, 2], k_max=4, seed=22, temperature=0.7, q_mode="onehot")
    _run_case(desc, ctx_lens=[5, 130, 64, 257], k_b=[4, 4, 0, 2], k_max=4, seed=23, temperature=0.0, q_mode="dense")


def test_mini_wide_groups_k16():
    """G = 7 query heads per KV head and k up to 16: 119 query rows per KV head (four MFMA row tiles)."""
    desc = W.shape("mini_bf16", n_q_heads=14, n_kv_heads=2, d_model=320, d_ffn=448, vocab=777)
    _run_case(desc, ctx_lens=[700, 40, 129, 1000, 3], k_b=[16, 0, 9, 12, 16], k_max=16, seed=24)


def test_mini_maximum_draft_length():
    """k_max = 30 (the library's maximum) with G = 3: up to 93 query rows per KV head, i.e. three of the four
    query tiles are populated and the fourth block of workgroups exits at once; ragged lengths down to 0."""
    desc = W.shape("mini_bf16")
    _run_case(desc, ctx_lens=[90, 3, 500, 64], k_b=[30, 0, 17, 29], k_max=30, seed=33)


def test_mini_many_ragged_sequences():
    """40 sequences with contexts from 0 to 900 tokens and 0..8 drafts: the attention work list cuts them into
    several hundred chunks, more than there are workgroups, so the per-XCD work queues, the partial results and
    the last-arriver merge are all exercised."""
    desc = W.shape("mini_bf16")
    rng = np.random.default_rng(35)
    ctx = [int(x) for x in rng.integers(0, 900, 40)]
    ctx[3], ctx[17] = 0, 899
    k_b = [int(x) for x in rng.integers(0, 9, 40)]
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=8, seed=35, check_kv=False)


@pytest.mark.parametrize("fill", ["full", "mixed", "plain"])
def test_wide_model_large_row_limit(fill):
    """Row limit 48 x 17 = 816 > 640 on a one-layer model that is wide enough (d = 3840) for the large-batch launch
    paths at a size the oracle still finishes in seconds: the gate/up projection in four waves, and the residual projections
    whose K split is decided on the device from the step's row count: for the O projection (K = 2048) one, two (mixed lengths, about
    430 rows) and six slabs (plain decodes only, 48 rows) of 128-row tiles.  (Row tiles that change: test_row_tile_from_the_row_count.)"""
    desc = W.shape("mini_bf16", n_layers=1, d_model=3840, n_q_heads=16, n_kv_heads=4, d_ffn=512, vocab=640)
    rng = np.random.default_rng(61)
    Bn, k_max = 48, 16
    ctx = [int(x) for x in rng.integers(0, 150, Bn)]
    k_b = {"full": [16] * Bn, "mixed": [int(x) for x in rng.integers(0, 17, Bn)], "plain": [0] * Bn}[fill]
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=k_max, seed=61, check_kv=(fill == "mixed"))


@pytest.mark.parametrize("k_b,choice", [([16] * 66, (160, 1)), ([15] * 42 + [0] * 24, (96, 2)), ([0] * 66, (160, 6))])
def test_row_tile_from_the_row_count(k_b, choice):
    """Row limit 66 x 17 = 1122: the O projection (K = 2048, 3840 columns) takes 160-row tiles of 128 columns when every block is full and when none has a
    draft, 96-row tiles of 256 columns in two slabs for 696 rows, and the device says so."""
    desc = W.shape("mini_bf16", n_layers=1, d_model=3840, n_q_heads=16, n_kv_heads=4, d_ffn=512, vocab=640)
    ctx = [int(x) for x in np.random.default_rng(62).integers(0, 150, 66)]
    seen = []
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=16, seed=62, check_kv=False, q_mode="onehot", after_step=lambda eng: seen.append(H.slab_choice(eng, 1)))
    assert seen == [choice]


def test_mini_single_sequence_edges():
    """Degenerate batches: one sequence with no draft (a single query row in the whole step), one sequence with an
    empty cache and one draft, and a batch in which no sequence has a draft (k_max = 1 is the smallest row limit)."""
    desc = W.shape("mini_bf16")
    _run_case(desc, ctx_lens=[37], k_b=[0], k_max=1, seed=71)
    _run_case(desc, ctx_lens=[0], k_b=[1], k_max=1, seed=72)
    _run_case(desc, ctx_lens=[64, 0, 5], k_b=[0, 0, 0], k_max=1, seed=73, q_mode="onehot")


def test_mini_head_dim_64():
    desc = W.shape("mini_bf16", head_dim=64, n_q_heads=8, n_kv_heads=4, vocab=4096)
    _run_case(desc, ctx_lens=[100, 513, 64], k_b=[3, 8, 8], k_max=8, seed=25)


@pytest.mark.parametrize("q_blocks,n_split", [(1, 1), (1, 3), (2, 1), (2, 2), (4, 1), (4, 5)])
def test_attention_launch_shapes_k16(q_blocks, n_split):
    """The G = 7, k = 16 case (four query tiles per KV head) under every launch shape of the attention kernel:
    one workgroup per unit with two wave groups (1 query block), two tiles per workgroup (2) and one tile per
    workgroup (4), each with one token chunk per sequence and with the longest sequence cut into several."""
    desc = W.shape("mini_bf16", n_q_heads=14, n_kv_heads=2, d_model=320, d_ffn=448, vocab=777)
    B.bs_debug_attention_shape(q_blocks, n_split)
    try:
        _run_case(desc, ctx_lens=[700, 40, 129, 1000, 3], k_b=[16, 0, 9, 12, 16], k_max=16, seed=24)
    finally:
        B.bs_debug_attention_shape(0, 0)


@pytest.mark.parametrize("q_blocks,n_split,head_dim", [(1, 1, 128), (1, 4, 128), (2, 3, 128), (1, 2, 64), (2, 1, 64)])
def test_attention_launch_shapes_k8(q_blocks, n_split, head_dim):
    """Two query tiles per KV head (G = 6, k = 8: 54 rows) as one or two query blocks, head sizes 128 and 64."""
    desc = W.shape("mini_bf16", head_dim=head_dim, n_q_heads=12, n_kv_heads=2, d_model=384, vocab=1000)
    B.bs_debug_attention_shape(q_blocks, n_split)
    try:
        _run_case(desc, ctx_lens=[1, 63, 64, 200, 333, 0], k_b=[8, 0, 3, 8, 5, 2], k_max=8, seed=31)
    finally:
        B.bs_debug_attention_shape(0, 0)


def test_slice_1p5b_full_vocab():
    """Two layers of the 1.5B shape, full 151936 vocabulary, context 2048, k = 8, dense bf16 q."""
    desc = W.shape("s1p5b", n_layers=2)
    st = _run_case(desc, ctx_lens=[2048, 2048, 1500, 2048, 17, 2048], k_b=[8, 8, 8, 0, 8, 5], k_max=8, seed=26,
                   check_kv=False)
    assert st["accepted"] > 0


def test_slice_7b_full_vocab():
    """Two layers of the 7B shape (G = 7), full 152064 vocabulary, ragged contexts and draft lengths."""
    desc = W.shape("s7b", n_layers=2)
    _run_case(desc, ctx_lens=[4096, 512, 1800], k_b=[16, 8, 0], k_max=16, seed=27, check_kv=False, q_mode="onehot")


def test_slice_7b_long_tail():
    """Configuration-4 shape on a two-layer 7B slice: contexts from the clipped lognormal range (512 .. 32768),
    ragged draft lengths 0..16, dense proposals; exercises long KV splits and the four-tile query packing."""
    desc = W.shape("s7b", n_layers=2)
    ctx = [512, 3000, 32768 - 17, 9000, 700, 20000]
    _run_case(desc, ctx_lens=ctx, k_b=[16, 0, 16, 7, 3, 11], k_max=16, seed=28, check_kv=False, q_scale=1.3)


def test_lookup_to_commit_without_host_sync():
    """Configuration-5 flow on a two-layer 1.5B slice: bs_draft_lookup writes draft_tokens / draft_len on the
    device and bs_verify_step consumes them directly (row packing is planned on the device), then one-hot
    acceptance (the paper's deterministic-draft rule) and commit.  Checked against the oracle lookup + forward."""
    from oracle.lookup import lookup as oracle_lookup
    desc = W.shape("s1p5b", n_layers=2)
    Bn, k_max, ctx = 16, 16, 300
    rng = np.random.default_rng(31)
    V = desc["vocab"]
    w = W.make_weights(desc, seed=31)
    wn = _f64_weights(W.weights_to_numpy(w))
    eng = Engine(desc, fuse_weights(w, desc["dtype"], DEV), Bn, ctx + k_max + 1, B_max=Bn, k_max=k_max, page_perm_seed=5)
    pool = W.make_pool(32, 2, 8, 2048, V, lo=64, hi=8192)
    seq_prompt, tails = W.plant_tails(33, pool, Bn, 8, 4, vocab=V)
    toks, off, prb = pool
    eng.pool_bind(torch.tensor(toks), torch.tensor(off), torch.tensor(prb))
    od = H.oracle_desc(desc)
    caches = []
    for b in range(Bn):
        kvs = W.context_kv(desc, ctx, 3100 + b)
        c = OD.SeqCache(od)
        c.fill([k.float().numpy() for k, _ in kvs], [v.float().numpy() for _, v in kvs])
        caches.append(c)
        for l, (k, v) in enumerate(kvs):
            eng.kv_write(l, b, 0, k.to(DEV), v.to(DEV))
    eng.ctx_len.fill_(ctx)
    last = tails[:, -1].copy()                       # the tail's newest token is the step's last token
    ua, us = W.uniforms(34, Bn, k_max)
    slots = H.dev_i32(np.arange(Bn))
    # device flow: no host read between the calls
    dt, dl = eng.draft_lookup(H.dev_i32(seq_prompt), H.dev_i32(tails), 4, 1, k_max)
    logits = eng.verify_step(slots, H.dev_i32(last), dt, dl, k_max, want_logits=True)
    out = eng.accept_resample(dt, dl, k_max, H.dev_f32(ua), H.dev_f32(us))
    eng.kv_commit(slots, out["n_accepted"] + 1)
    assert eng.poll_status() == 0
    # oracle flow
    drafts = np.full((Bn, k_max), -1, dtype=np.int64)
    k_b = np.zeros(Bn, dtype=np.int64)
    for b in range(Bn):
        p = seq_prompt[b]
        ref = oracle_lookup([toks[off[r]:off[r + 1]] for r in range(prb[p], prb[p + 1])], tails[b], 4, 1, k_max)
        k_b[b] = len(ref)
        drafts[b, :len(ref)] = ref
    assert dl.cpu().tolist() == k_b.tolist()
    assert (dt.cpu().numpy() == drafts).all()
    assert k_b.max() > 0 and k_b.min() == 0          # both drafted and plain sequences ride in the same launch
    blocks = H.pack_rows(last, drafts, k_b)
    ref_logits = np.concatenate([OD.verify_block(od, wn, caches[b], blocks[b]) for b in range(Bn)])
    M = int(k_b.sum() + Bn)
    got = logits.cpu().numpy()[:M]
    assert np.abs(got - ref_logits).max() <= H.TOL_LOGITS[W.BS_BF16]
    exact, near, _ = H.compare_sampler(out, got, drafts, k_b, ua, us)
    assert near <= 1
    n_acc = out["n_accepted"].cpu().numpy()
    assert eng.ctx_len.cpu().tolist() == [ctx + int(n) + 1 for n in n_acc]
    eng.close()


@pytest.mark.parametrize("which", ["w_gate_up", "wq_wk", "lm_head_weight", "kv_import"])
def test_float16_range_is_guarded(which):
    """bf16 models compute with float16 matrix operands (largest finite value 65504).  A weight matrix scaled so
    that a producer of such an operand overflows must end in saturated, finite results and BS_FAULT_RANGE in the
    status word: gated MLP activation (SwiGLU epilogue), rotated q and appended k (QKV epilogue), a weight beyond
    the range at packing time, and imported K/V rows."""
    desc = W.shape("mini_bf16")
    w = W.make_weights(desc, seed=41)
    kv_scale = 1.0
    if which == "w_gate_up":
        for lw in w["layers"]:
            lw["w_gate"] = (lw["w_gate"].float() * 2000).to(torch.bfloat16)
            lw["w_up"] = (lw["w_up"].float() * 2000).to(torch.bfloat16)
    elif which == "wq_wk":
        for lw in w["layers"]:
            lw["wq"] = (lw["wq"].float() * 2e5).to(torch.bfloat16)
            lw["wk"] = (lw["wk"].float() * 2e5).to(torch.bfloat16)
    elif which == "lm_head_weight":
        w["lm_head"][3, 5] = 1e6            # a bf16 value float16 cannot hold
    else:
        kv_scale = 1e6
    Bn, k_max = 3, 4
    eng = Engine(desc, fuse_weights(w, desc["dtype"], DEV), Bn, 256, B_max=Bn, k_max=k_max)
    torch.cuda.synchronize()
    st0 = eng.poll_status()
    assert (st0 == B.BS_FAULT_RANGE) == (which == "lm_head_weight"), st0       # set while packing, and only then
    for b in range(Bn):
        for l, (k, v) in enumerate(W.context_kv(desc, 70, 4100 + b)):
            eng.kv_write(l, b, 0, (k.float() * kv_scale).to(torch.bfloat16).to(DEV), v.to(DEV))
    if which == "kv_import":
        assert eng.poll_status() == B.BS_FAULT_RANGE
    eng.ctx_len.fill_(70)
    rng = np.random.default_rng(41)
    drafts = H.dev_i32(rng.integers(0, desc["vocab"], (Bn, k_max)))
    dl = H.dev_i32([4, 0, 2])
    slots = H.dev_i32(np.arange(Bn))
    logits = eng.verify_step(slots, H.dev_i32(rng.integers(0, desc["vocab"], Bn)), drafts, dl, k_max, want_logits=True)
    ua, us = W.uniforms(42, Bn, k_max)
    out = eng.accept_resample(drafts, dl, k_max, H.dev_f32(ua), H.dev_f32(us))
    eng.kv_commit(slots, out["n_accepted"] + 1)
    st = eng.poll_status()
    if which in ("w_gate_up", "wq_wk"):
        assert st == B.BS_FAULT_RANGE, st
    else:
        assert st == 0, st                  # the saturated weight / cache rows are ordinary finite operands
    got = logits[:9].cpu().numpy()             # M = 5 + 1 + 3 packed rows
    assert np.isfinite(got).all()
    n_emit = out["n_emitted"].cpu().numpy()
    assert ((n_emit >= 1) & (n_emit <= k_max + 1)).all()
    eng.close()
