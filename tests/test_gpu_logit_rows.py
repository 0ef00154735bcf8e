"""The two ways the bf16 accept step obtains the sampled rows' logits (all rows stored by the LM-head pass up to d_model / 4
packed rows, the sampled rows recomputed above that) on both sides of the line: same context, same oracle, and a context
whose row limit is above the line while the step's is below it (both buffers exist)."""
import numpy as np
import pytest
import torch

from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine, fuse_weights
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq", [12, 13, 16])        # 60, 65 and 80 rows; the line is at 64 for d_model = 256
def test_sampled_rows_from_either_source(n_seq):
    desc = W.shape("mini_bf16", vocab=1003)             # V % 4 != 0: the scalar store path
    k, B_max = 4, 16
    rng = np.random.default_rng(n_seq)
    w = W.make_weights(desc, seed=9)
    eng = Engine(desc, fuse_weights(w, desc["dtype"], "cuda:0"), B_max, 64, B_max=B_max, k_max=k)
    last, drafts = rng.integers(0, desc["vocab"], n_seq), rng.integers(0, desc["vocab"], (n_seq, k))
    k_b = rng.integers(0, k + 1, n_seq)
    ua, us = W.uniforms(3, n_seq, k)
    ua[:, :2] *= 1e-3                                    # some drafts of a flat target are accepted
    dt, dl = H.dev_i32(drafts), H.dev_i32(k_b)
    logits = eng.verify_step(H.dev_i32(np.arange(n_seq)), H.dev_i32(last), dt, dl, k, want_logits=True)
    out = eng.accept_resample(dt, dl, k, H.dev_f32(ua), H.dev_f32(us))
    rows = logits[:int((k_b + 1).sum())].cpu().numpy()
    exact, near, _ = H.compare_sampler(out, rows, drafts, k_b, ua, us)
    assert exact + near == n_seq and near <= 1
    assert eng.poll_status() == 0
    eng.close()


def test_smaller_workspaces_give_the_same_step(monkeypatch):
    """bs_create takes less than bs_workspace_bytes: with room for fewer rows of logits than the step has the sampled rows are
    recomputed, and at the smallest size small steps run on the kernels without fragment-ordered activations.  Logits equal
    within the tolerance, decisions equal to the rule on the device's own logits."""
    desc = W.shape("mini_bf16", vocab=40001)
    k, B_max = 4, 16
    weights = fuse_weights(W.make_weights(desc, seed=9), desc["dtype"], "cuda:0")
    full = B.bs_workspace_bytes(B.make_desc(desc), B_max, k)

    def engine(nbytes):
        monkeypatch.setattr(B, "bs_workspace_bytes", lambda *a: nbytes)
        return Engine(desc, weights, B_max, 64, B_max=B_max, k_max=k)

    lo, hi = full // 2, full                             # smallest size that is accepted
    while hi - lo > 256:
        mid = (lo + hi) // 2
        try:
            engine(mid).close()
            hi = mid
        except B.BsError as e:
            assert e.status == B.BS_ECAPACITY
            lo = mid
    assert full - hi > 30 * 4 * desc["vocab"]            # more than half of the 64 rows
    ref = {}
    for nbytes in (full, (full + hi) // 2, hi):
        eng = engine(nbytes)
        for n_seq in (12, 5):                            # 60 and 25 rows
            rng = np.random.default_rng(n_seq)
            last, drafts = rng.integers(0, desc["vocab"], n_seq), rng.integers(0, desc["vocab"], (n_seq, k))
            k_b = np.full(n_seq, k)
            ua, us = W.uniforms(3, n_seq, k)
            ua[:, :2] *= 1e-5
            dt, dl = H.dev_i32(drafts), H.dev_i32(k_b)
            logits = eng.verify_step(H.dev_i32(np.arange(n_seq)), H.dev_i32(last), dt, dl, k, want_logits=True)
            rows = logits[:n_seq * (k + 1)].cpu().numpy()
            for _ in range(2):                           # the accept call may be repeated: it does not use up its inputs
                out = eng.accept_resample(dt, dl, k, H.dev_f32(ua), H.dev_f32(us))
                exact, near, _ = H.compare_sampler(out, rows, drafts, k_b, ua, us)
                assert exact + near == n_seq and near <= 1
            assert np.abs(rows - ref.setdefault(n_seq, rows)).max() <= H.TOL_LOGITS[W.BS_BF16]
        assert eng.poll_status() == 0
        eng.close()
