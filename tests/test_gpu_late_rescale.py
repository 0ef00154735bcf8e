"""GPU parity of the attention kernels where the maximum of a row's scores moves along the context: accumulators are rescaled only
when it has risen by more than a factor of 2^8.  Keys grow (by 0.5 .. 15 powers of two per 32 tokens: some rises below the bound,
some above, within a wave's tiles and between waves and chunks), shrink (the first tile holds the maximum) or jump once, late."""
import pytest
import torch

from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from tests.test_gpu_bf16 import _run_case

pytestmark = pytest.mark.gpu
PLAIN = W.context_kv


@pytest.mark.parametrize("n_chunks", [0, 3])
@pytest.mark.parametrize("k_max,heads", [(4, (6, 2)), (16, (14, 2))])         # narrow and wide kernel
@pytest.mark.parametrize("profile", ["grow", "shrink", "jump"])
def test_rows_whose_maximum_moves(monkeypatch, profile, k_max, heads, n_chunks):
    def context_kv(desc, n_tokens, seed, device="cpu"):
        t = torch.arange(n_tokens, dtype=torch.float32) / max(n_tokens - 1, 1)
        scale = {"grow": 60 * t, "shrink": 60 * (1 - t), "jump": 1 + 60 * (t > 0.8)}[profile].view(-1, 1, 1)
        return [((k.float() * scale).to(k.dtype), v) for k, v in PLAIN(desc, n_tokens, seed, device)]

    monkeypatch.setattr(W, "context_kv", context_kv)
    desc = W.shape("mini_bf16", n_layers=1, n_q_heads=heads[0], n_kv_heads=heads[1], vocab=777)
    B.bs_debug_attention_shape(0, n_chunks)
    try:
        _run_case(desc, ctx_lens=[70, 130, 333, 97, 1000, 31], k_b=[k_max, 0, k_max, 3, k_max, 1], k_max=k_max, seed=31, q_mode="onehot", check_kv=False)
    finally:
        B.bs_debug_attention_shape(0, 0)
