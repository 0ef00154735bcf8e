"""GPU parity of the acceptance / resampling rule alone (bs_accept_resample_logits): caller-supplied float32
logits, so every integer the device returns must equal the oracle's on the same inputs (Tier A), and the
distribution of the emitted token must be the target distribution (the paper's exactness claim, Sec. 3.2)."""
import numpy as np
import pytest
import torch
from scipy import stats
from scipy.special import softmax

from oracle import accept as OA
from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine, fuse_weights
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def eng():
    desc = W.shape("tiny")
    w = W.make_weights(desc, seed=3)
    e = Engine(desc, fuse_weights(w, desc["dtype"], DEV), 1, 64, B_max=4096, k_max=8)
    yield e
    e.close()


def _call(eng, logits, drafts, k_b, ua, us, q=None, **kw):
    k_max = drafts.shape[1]
    qd = None
    if q is not None:
        qd = torch.as_tensor(q).to(DEV)
    return eng.accept_resample(H.dev_i32(drafts), H.dev_i32(k_b), k_max, H.dev_f32(ua), H.dev_f32(us), q_logits=qd,
                               logits=H.dev_f32(logits), **kw)


@pytest.mark.parametrize("mode", ["dense_q", "one_hot"])
def test_device_output_law_is_the_target(eng, mode):
    rng = np.random.default_rng(101)
    V, Bn, rounds = 16, 4096, 25
    z = rng.normal(0, 1.5, (2, V)).astype(np.float32)
    ql = rng.normal(0, 1.5, (1, V)).astype(np.float32)
    p, q = softmax(z[0].astype(np.float64)), softmax(ql[0].astype(np.float64))
    counts = np.zeros(V)
    mism = 0
    for r in range(rounds):
        drafts = (rng.choice(V, size=(Bn, 1), p=q) if mode == "dense_q" else np.full((Bn, 1), 3)).astype(np.int32)
        ua, us = W.uniforms(7000 + r, Bn, 1)
        logits = np.tile(z, (Bn, 1))
        qrows = np.tile(ql, (Bn, 1)) if mode == "dense_q" else None
        out = _call(eng, logits, drafts, np.ones(Bn, np.int32), ua, us, q=qrows)
        first = out["out_tokens"].cpu().numpy()[:, 0]
        counts += np.bincount(first, minlength=V)
        if r < 3:       # and bit-exact against the oracle on the same inputs
            exact, near, _ = H.compare_sampler(out, logits, drafts, np.ones(Bn, int), ua, us, qrows)
            mism += near
    n = counts.sum()
    chi2 = ((counts - n * p) ** 2 / (n * p)).sum()
    assert stats.chi2.sf(chi2, df=V - 1) > 1e-4, chi2
    assert mism <= 6            # |rho - u| <= 1e-3 happens for ~0.2 % of float32 uniforms; they are counted, not hidden


def test_ragged_blocks_options_and_dtypes(eng):
    """Ragged k_b, vocabularies that are not multiples of any tile, bf16 and float32 proposals, temperature,
    greedy, EOS and emit_bonus: device integers equal the oracle's."""
    rng = np.random.default_rng(202)
    for V, T, q_mode, eos, bonus in [(1000, 1.0, "bf16", -1, True), (4096, 0.7, "f32", -1, True),
                                     (37, 1.3, None, 5, True), (513, 1.0, "f32", -1, False),
                                     (2049, 0.0, "bf16", -1, True), (50, 0.0, None, 7, True)]:
        Bn, k_max = 200, 8
        k_b = rng.integers(0, k_max + 1, Bn)
        M, Td = int(k_b.sum() + Bn), int(k_b.sum())
        logits = rng.normal(0, 2.0, (M, V)).astype(np.float32)
        drafts = rng.integers(0, V, (Bn, k_max)).astype(np.int32)
        # make a good share of drafts likely: copy the row's arg-max
        r0 = np.concatenate([[0], np.cumsum(k_b + 1)])
        for b in range(Bn):
            for j in range(k_b[b]):
                if rng.random() < 0.6:
                    drafts[b, j] = int(np.argmax(logits[r0[b] + j]))
        q = qn = None
        if q_mode and Td > 0:
            qt = torch.tensor(rng.normal(0, 2.0, (Td, V)), dtype=torch.bfloat16 if q_mode == "bf16" else torch.float32)
            q, qn = qt, qt.float().numpy()
        ua, us = W.uniforms(int(V), Bn, k_max)
        out = _call(eng, logits, drafts, k_b.astype(np.int32), ua, us, q=q, temperature=T, eos_id=eos, emit_bonus=bonus)
        exact, near, res = H.compare_sampler(out, logits, drafts, k_b, ua, us, qn, T, eos, bonus)
        assert near <= 3, (V, exact, near)
        n_emit = out["n_emitted"].cpu().numpy()
        assert sum(len(r.tokens) for r in res) == n_emit.sum() or near > 0


@pytest.mark.parametrize("dtype,n_nan", [(torch.float32, 1), (torch.float32, 4096), (torch.float32, 12288), (torch.bfloat16, 1),
                                         (torch.bfloat16, 8192)])
def test_nan_block_in_a_proposal_row_is_not_read_as_masked(dtype, n_nan):
    """A proposal row with NaN has no probabilities: its draft is accepted whatever the uniform, for one NaN as for a block of them as
    long as everything a thread has in flight at once (a block of -inf instead is a mask, and the rule applies)."""
    V, Bn = 20480, 8
    rng = np.random.default_rng(n_nan)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=DEV)
    z = torch.tensor(rng.normal(0, 1, (2 * Bn, V)), dtype=torch.float32, device=DEV)
    z[:, V - 1] = -30.0                                    # the target hardly has the draft: u = 0.5 rejects it
    q = torch.tensor(rng.normal(0, 1, (Bn, V)), dtype=dtype, device=DEV)
    for fill, accepted in ((float("nan"), 1), (-float("inf"), 0)):
        q[:, :n_nan] = fill
        new = lambda *s: torch.full(s, -7, dtype=torch.int32, device=DEV)
        n_acc, toks, n_emit, tie = new(Bn), new(Bn, 2), new(Bn), new(Bn)
        B.bs_accept_resample_logits_noalloc(Bn, V, z, i32(np.full((Bn, 1), V - 1)), i32(np.ones(Bn)), 1, q,
                                            B.BS_BF16 if dtype == torch.bfloat16 else B.BS_F32, 1.0, -1, True,
                                            torch.full((Bn, 1), 0.5, device=DEV), torch.full((Bn,), 0.5, device=DEV), n_acc, toks, n_emit, tie)
        assert n_acc.tolist() == [accepted] * Bn, fill
