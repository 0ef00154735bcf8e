"""GPU parity of the decoder layer for steps of at most 32 packed rows (one weight tile per workgroup or wave, K split over
waves and workgroups, fragment-ordered activations) at the edges of its range, and the step that is one row too large for it.

The oracle is the fp64 forward; the bound is the logit tolerance of all bf16 cases (float16 operands, 2e-2 max-abs)."""
import pytest

from paper_2605_08862_amd import workloads as W
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
