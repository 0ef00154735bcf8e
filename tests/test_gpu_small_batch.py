"""GPU parity of the decoder layer for steps of at most 32 packed rows (one weight tile per workgroup or wave, K split over
waves and workgroups, fragment-ordered activations) at the edges of its range, and the step that is one row too large for it.

The oracle is the fp64 forward; the bound is the logit tolerance of all bf16 cases (float16 operands, 2e-2 max-abs)."""
import pytest
import torch

from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine, fuse_weights
from tests import helpers as H
from tests.test_gpu_bf16 import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ctx_lens,k_b,k_max", [
    ([77], [0], 0),                                   # one row
    ([64, 1, 200, 0], [7, 7, 7, 7], 7),               # exactly 32 rows
    ([130, 5, 63], [10, 10, 10], 10),                 # 33: the tiled kernels
    ([300, 64], [15, 3], 15),                         # row limit 32, 20 live
])
@pytest.mark.parametrize("over", [
    {},                                               # 4 K tiles for eight waves: half of them have an empty range
    dict(d_model=320, d_ffn=192, n_q_heads=6, n_kv_heads=2, vocab=777),      # odd tile counts everywhere, 3 + 3 gate/up tiles
    dict(d_model=320, d_ffn=6400, n_layers=1),        # down projection: 100 K tiles, split over workgroups
])
def test_small_row_counts(ctx_lens, k_b, k_max, over):
    desc = W.shape("mini_bf16", **over)
    _run_case(desc, ctx_lens=ctx_lens, k_b=k_b, k_max=k_max, seed=51)


@pytest.mark.parametrize("name,moved", [("tiny", ["embed", "lm_head", "wqkv", "wo", "w_gate_up", "w_down"]),
                                        ("mini_bf16", ["embed"])])
def test_weights_aligned_to_their_elements_only(name, moved):
    """Views into a larger buffer start at any element; the bits of the logits do not depend on it."""
    desc = W.shape(name)
    w = fuse_weights(W.make_weights(desc, seed=8), desc["dtype"], "cuda:0")

    def shifted(t):
        if isinstance(t, list):
            return [shifted(x) for x in t]
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:].copy_(t.reshape(-1))
        return buf[1:].view(t.shape)

    got = []
    for weights in (w, {n: shifted(t) if n in moved else t for n, t in w.items()}):
        eng = Engine(desc, weights, 2, 64, B_max=2, k_max=3)
        got.append(eng.verify_step(H.dev_i32([0, 1]), H.dev_i32([3, 4]), H.dev_i32([[5, 6, 7], [8, 9, 10]]),
                                   H.dev_i32([3, 1]), 3, want_logits=True)[:6].cpu())
        assert eng.poll_status() == 0
        eng.close()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("n_chunks", [0, 1, 3, 7])       # the rule's choice; one piece; several, merged by the last workgroup
@pytest.mark.parametrize("heads,head_dim,k_max,ctx_lens,k_b", [
    (14, 128, 16, [500], [16]),                       # G = 7: 119 query rows, four query tiles
    (14, 128, 16, [333], [8]),                        # 63 rows: the two-tile variant of the wide kernel
    (12, 128, 16, [0], [16]),                         # G = 6, empty cache
    (6, 128, 30, [700], [30]),                        # G = 3: 93 rows, 31 packed rows
    (6, 128, 30, [64], [0]),                          # three live query rows under a wide row limit
])
def test_wide_attention_in_front_of_the_small_step_kernels(heads, head_dim, k_max, ctx_lens, k_b, n_chunks):
    """At most 32 packed rows and more than 64 query rows per KV head: the wide kernel writes its rows in fragment order, from
    the workgroup itself (one chunk) and from the merge."""
    desc = W.shape("mini_bf16", n_q_heads=heads, n_kv_heads=2, head_dim=head_dim, d_model=320, vocab=777)
    B.bs_debug_attention_shape(0, n_chunks)
    try:
        _run_case(desc, ctx_lens=ctx_lens, k_b=k_b, k_max=k_max, seed=61)
    finally:
        B.bs_debug_attention_shape(0, 0)
