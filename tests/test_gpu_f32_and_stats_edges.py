"""Tile edges of the float32 path (32-row / 32-column matrix tiles, K split over eight waves) against the oracle, and segment
edges of the plain-logits sampler (16 segments per row, four tokens per load, row starts of every alignment)."""
import numpy as np
import pytest
import torch

from oracle import decoder as OD
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine, fuse_weights
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_seq,vocab", [(1, 17), (31, 4096), (8, 1003), (11, 33)])     # 1, 31, 32 and 33 rows
def test_float32_step_at_tile_edges(n_seq, vocab):
    k = {8: 3, 11: 2}.get(n_seq, 0)
    desc = W.shape("tiny", vocab=vocab)
    w = W.make_weights(desc, seed=5)
    eng = Engine(desc, fuse_weights(w, desc["dtype"], DEV), 31, 64, B_max=31, k_max=3)
    wn, od = W.weights_to_numpy(w), H.oracle_desc(desc)
    rng = np.random.default_rng(n_seq)
    blk = rng.integers(0, vocab, (n_seq, k + 1))
    dl = H.dev_i32(np.full(n_seq, k))
    drafts = H.dev_i32(blk[:, 1:]) if k else None
    logits = eng.verify_step(H.dev_i32(np.arange(n_seq)), H.dev_i32(blk[:, 0]), drafts, dl, k, want_logits=True)
    got = logits[:n_seq * (k + 1)].cpu().numpy().reshape(n_seq, k + 1, vocab)
    for b in range(n_seq):
        ref = OD.verify_block(od, wn, OD.SeqCache(od), blk[b])
        assert np.abs(got[b] - ref).max() <= H.TOL_LOGITS[W.BS_F32]
    assert eng.poll_status() == 0
    eng.close()


@pytest.mark.parametrize("q_mode", ["bf16", "f32", None])
@pytest.mark.parametrize("vocab", [2, 3, 5, 63, 64, 67, 130, 8191, 16385])
def test_plain_logits_sampler_at_segment_edges(vocab, q_mode):
    desc = W.shape("tiny", n_layers=1, vocab=vocab)
    eng = Engine(desc, fuse_weights(W.make_weights(desc, seed=3), W.BS_F32, DEV), 1, 64, B_max=16, k_max=2)
    rng = np.random.default_rng(vocab)
    Bn, k = 16, 2
    k_b = rng.integers(0, k + 1, Bn)
    M, Td = int(k_b.sum() + Bn), int(k_b.sum())
    logits = rng.normal(0, 2.0, (M, vocab)).astype(np.float32)
    logits[:, vocab // 2] = logits[:, vocab - 1] = logits.max() + 1.0                   # equal maxima in two segments
    drafts = rng.integers(0, vocab, (Bn, k)).astype(np.int32)
    q = qn = None
    if q_mode:
        q = torch.tensor(rng.normal(0, 2.0, (Td, vocab)), dtype=torch.bfloat16 if q_mode == "bf16" else torch.float32)
        qn = q.float().numpy()
    ua, us = W.uniforms(vocab, Bn, k)
    for T in (0.9, 0.0):
        out = eng.accept_resample(H.dev_i32(drafts), H.dev_i32(k_b), k, H.dev_f32(ua), H.dev_f32(us),
                                  q_logits=None if q is None else q.to(DEV), logits=H.dev_f32(logits), temperature=T)
        exact, near, _ = H.compare_sampler(out, logits, drafts, k_b, ua, us, qn, T)
        assert exact + near == Bn and near <= 2
    eng.close()


@pytest.mark.parametrize("source,vocab", [("logits", 5), ("logits", 1003), ("logits", 70000), ("tiny", 4096),
                                          ("mini_bf16", 1003), ("mini_bf16", 8200)])     # 129 statistics tiles: the fold pass runs
def test_infinite_temperature_is_the_uniform_law(source, vocab):
    """1 / T = 0 is a legal scaling: p is uniform, so a one-hot draft is accepted with probability 1 / V and the sums start
    from an empty running maximum (-inf) without producing (-inf) * 0."""
    name = "tiny" if source == "logits" else source
    desc = W.shape(name, vocab=vocab, **(dict(n_layers=1) if source == "logits" else {}))
    Bn, k = 6, 3
    eng = Engine(desc, fuse_weights(W.make_weights(desc, seed=3), desc["dtype"], DEV), Bn, 64, B_max=Bn, k_max=k)
    rng = np.random.default_rng(vocab)
    blk = rng.integers(0, vocab, (Bn, k + 1))
    k_b = np.array([3, 3, 2, 1, 0, 3])
    drafts, dl = H.dev_i32(blk[:, 1:]), H.dev_i32(k_b)
    ua, us = W.uniforms(vocab, Bn, k)
    ua[0, 0] = 0.25 / vocab                                                             # accepted: below 1 / V
    M = int((k_b + 1).sum())
    if source == "logits":
        rows = rng.normal(0, 2.0, (M, vocab)).astype(np.float32)
        out = eng.accept_resample(drafts, dl, k, H.dev_f32(ua), H.dev_f32(us), logits=H.dev_f32(rows), temperature=float("inf"))
    else:
        logits = eng.verify_step(H.dev_i32(np.arange(Bn)), H.dev_i32(blk[:, 0]), drafts, dl, k, want_logits=True)
        rows = logits[:M].cpu().numpy()
        out = eng.accept_resample(drafts, dl, k, H.dev_f32(ua), H.dev_f32(us), temperature=float("inf"))
    exact, near, _ = H.compare_sampler(out, rows, blk[:, 1:], k_b, ua, us, temperature=float("inf"))
    assert exact + near == Bn and near <= 1
    assert eng.poll_status() == 0
    eng.close()


@pytest.mark.parametrize("n_ctx", [0, 1, 30, 255, 256])
def test_float32_attention_keeps_an_infinite_value(n_ctx):
    """V of the step's own row overflows in one element: the attention output is infinite there (weight > 0), not NaN, and
    finite everywhere else.  The row is the last one of its last group of tokens, which the kernel reads again as filler."""
    desc = W.shape("tiny", n_layers=1)
    w = W.make_weights(desc, seed=2)
    w["embed"][:, 0] = 0.0
    w["embed"][7, 0] = 10.0                                                             # normalised to about sqrt(d) = 16
    w["layers"][0]["wv"][0, 0] = 1e38                                                   # V of KV head 0, element 0
    eng = Engine(desc, fuse_weights(w, desc["dtype"], DEV), 1, 320, B_max=1, k_max=0)
    if n_ctx:
        rows = torch.randn(n_ctx, desc["n_kv_heads"], desc["head_dim"], device=DEV)
        eng.kv_write(0, 0, 0, rows, rows)
        eng.ctx_len.fill_(n_ctx)
    eng.verify_step(H.dev_i32([0]), H.dev_i32([7]), None, H.dev_i32([0]), 0)
    out = H.debug_buffer(eng, 4, desc["n_q_heads"] * desc["head_dim"]).cpu()
    assert out[0] == float("inf") and torch.isfinite(out[1:]).all()
    eng.close()


@pytest.mark.parametrize("vocab", [1024, 1025, 2049, 15360, 15361, 16383, 16384])      # one segment per started 1024 entries, at most 16
def test_plain_logits_sampler_where_the_segment_count_changes(vocab):
    test_plain_logits_sampler_at_segment_edges(vocab, "bf16")
