"""GPU parity at the edges of the bf16 GEMM launches: the launchers choose row tiles, columns per workgroup and K splits by the row
limit and the widths.  One layer; K tiles that no ring length divides (5 and 7), widths that no column tile divides (320, 448, 12352 features,
the last wide enough for the weight-stationary gate/up tiles)."""
import numpy as np
import pytest

from paper_2605_08862_amd import workloads as W
from tests import helpers as H
from tests.test_gpu_bf16 import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_ffn,n_seq,k_max", [(448, 11, 2), (448, 16, 3), (448, 13, 4), (448, 32, 4), (448, 23, 6), (448, 39, 4), (448, 64, 4),
                                               (448, 107, 2), (448, 128, 4), (448, 43, 14), (448, 69, 16), (12352, 11, 2), (12352, 13, 4),
                                               (12352, 49, 1), (12352, 43, 2), (12352, 27, 6), (12352, 36, 6), (12352, 64, 4), (12352, 107, 2)])
def test_gemm_launches_at_row_limit(d_ffn, n_seq, k_max):
    """Row limits 33, 64, 65, 160, 161, 195, 320, 321, 640, 645 and 1173 (narrow), 33, 65, 98, 129, 189, 252, 320 and 321 (wide); full
    draft blocks, so every row of every tile is live, with two short ones at the end, so that the last tile is not full."""
    desc = W.shape("mini_bf16", n_layers=1, d_model=320, n_q_heads=14, n_kv_heads=2, d_ffn=d_ffn, vocab=777)
    rng = np.random.default_rng(n_seq)
    ctx = [int(x) for x in rng.integers(0, 70, n_seq)]
    _run_case(desc, ctx_lens=ctx, k_b=[k_max] * (n_seq - 2) + [k_max - 1, 0], k_max=k_max, seed=70 + k_max, q_mode="onehot", check_kv=(n_seq < 20))


@pytest.mark.parametrize("d_ffn", [448, 6400])
@pytest.mark.parametrize("fill", ["full", "mixed", "plain"])
def test_splits_from_the_row_count(d_ffn, fill):
    """Row limit 645: the K splits of O and down follow from the step's row count (645, about 330 and 43 rows), which the GEMM and
    the normalisation behind it read in one place; down has 7 and 100 K tiles."""
    desc = W.shape("mini_bf16", n_layers=2, d_model=320, n_q_heads=14, n_kv_heads=2, d_ffn=d_ffn, vocab=777)
    rng = np.random.default_rng(d_ffn)
    ctx = [int(x) for x in rng.integers(0, 70, 43)]
    k_b = {"full": [14] * 43, "mixed": [int(x) for x in rng.integers(0, 15, 43)], "plain": [0] * 43}[fill]
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=14, seed=91, q_mode="onehot", check_kv=fill == "mixed")


@pytest.mark.parametrize("d_model,k_b", [(320, [14] * 11 + [3] + [0] * 31), (320, [14] * 8 + [0] * 35), (2048, [0] * 43), (2048, [14] * 8 + [1] + [0] * 34),
                                         (2048, [14] * 8 + [0] * 35)])
def test_gate_up_row_blocks_with_few_live_rows(d_model, k_b):
    """Row limit 645.  Short K (four waves): 200 and 155 live rows in 64-row blocks, the blocks behind them left out.  Long K (eight waves): 43, 156 and 155 live
    rows in 96-row blocks.  (Last blocks of 128 rows with few live ones: test_gate_up_tile_of_the_row_count.)"""
    desc = W.shape("mini_bf16", n_layers=1, d_model=d_model, n_q_heads=14, n_kv_heads=2, d_ffn=6400, vocab=333)
    _run_case(desc, ctx_lens=[int(x) for x in np.random.default_rng(5).integers(0, 70, 43)], k_b=k_b, k_max=14, seed=92, q_mode="onehot", check_kv=False)


@pytest.mark.parametrize("vocab", [131072, 131401])
@pytest.mark.parametrize("n_seq,k_max", [(7, 2), (13, 4), (19, 4), (33, 3)])
def test_lm_head_columns_per_workgroup(vocab, n_seq, k_max):
    """Up to 96 rows a workgroup of the LM head takes 256 vocabulary entries while 512 workgroups hold all of them, then 320; row limits 21, 65 and 95, and
    132 (two tiles of 96, or 128, by tiles per CU).  Above 64 rows the sampled rows are computed a second time from the gathered ones."""
    desc = W.shape("mini_bf16", n_layers=1, vocab=vocab)
    ctx = [int(x) for x in np.random.default_rng(n_seq).integers(0, 70, n_seq)]
    _run_case(desc, ctx_lens=ctx, k_b=[k_max] * (n_seq - 1) + [0], k_max=k_max, seed=93, q_mode="onehot", check_kv=False)


@pytest.mark.parametrize("n_draft,choice", [(8, 1), (4, 0), (2, 2)])
def test_gate_up_rows_from_the_row_count_below_640(n_draft, choice):
    """Row limit 504, 148 column blocks of 128 features, three K tiles: the tile follows from the row count, 128 rows for 504, 96 for 280, 64 rows of 64
    features for 168."""
    desc, seen = W.shape("mini_bf16", n_layers=1, d_model=192, n_q_heads=6, n_kv_heads=2, d_ffn=18944, vocab=333), []
    _run_case(desc, ctx_lens=[int(x) for x in np.random.default_rng(6).integers(0, 70, 56)], k_b=[n_draft] * 56, k_max=8, seed=94, q_mode="onehot", check_kv=False,
              after_step=lambda eng: seen.append(H.tile_choice(eng, "glu")))
    assert seen == [choice]


@pytest.mark.parametrize("d_model,d_ffn,n_seq,k_max,live,choice", [
    (1600, 8896, 42, 16, 42, 2), (1600, 8896, 42, 16, 150, 3), (1600, 8896, 42, 16, 250, 0), (1600, 8896, 42, 16, 300, 1), (1600, 8896, 42, 16, 340, 1), (1664, 8896, 42, 16, 500, 3),
    (1600, 8896, 64, 9, 64, 0), (1664, 8896, 64, 9, 280, 0), (1664, 8896, 64, 9, 303, 1), (1600, 8896, 64, 9, 425, 2), (1664, 8896, 64, 9, 558, 3), (1600, 8896, 64, 9, 631, 4),
    (3200, 10944, 56, 8, 470, 5), (2112, 9664, 78, 8, 695, 6)])
def test_gate_up_tile_of_the_row_count(d_model, d_ffn, n_seq, k_max, live, choice):
    """Widths that 128 features do not divide (a last column block of 64; of 256: of 192), 25, 26 and 33 K tiles (1, 2 and 0 modulo three, odd and even).  Row limit 714, four waves: 64 x 64, 192 x 64 (one
    and three row blocks), 96 x 128 and 128 x 128 (rows x features), the last block of 128 with 44 live rows, computed as 64, and with 84.  Row limits 567 and 640, eight waves:
    96 (one row block and three), 128, 160, 192 and 224 rows; long K, row limits 504 and 702: 256 rows, and 128 rows x 256 features."""
    left, k_b = live - n_seq, []
    for _ in range(n_seq):
        k_b.append(min(k_max, left))
        left -= k_b[-1]
    desc, seen = W.shape("mini_bf16", n_layers=1, d_model=d_model, n_q_heads=6, n_kv_heads=2, d_ffn=d_ffn, vocab=333), []
    ctx = [int(x) for x in np.random.default_rng(11).integers(0, 70, n_seq)]
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=k_max, seed=99, q_mode="onehot", check_kv=False, after_step=lambda eng: seen.append(H.tile_choice(eng, "glu")))
    assert seen == [choice]


@pytest.mark.parametrize("n_last", [0, 1, 2, 3])
def test_normalisation_of_four_rows_per_workgroup(n_last):
    """Row limit 2176 and d <= 2048: four rows per workgroup; 1600 to 1603 live rows."""
    desc = W.shape("mini_bf16", n_layers=1, d_model=320, n_q_heads=6, n_kv_heads=2, d_ffn=448, vocab=333)
    k_b = [16] * 92 + [n_last] + [0] * 35
    _run_case(desc, ctx_lens=[int(x) for x in np.random.default_rng(8).integers(0, 40, 128)], k_b=k_b, k_max=16, seed=95, q_mode="onehot", check_kv=False)


@pytest.mark.parametrize("k_b", [[14] * 36 + [0] * 7, [14] * 41 + [13, 0], [16] * 56 + [0] * 12, [16] * 67 + [15, 0], [16] * 87 + [15, 0], [16] * 126 + [15, 0]])
def test_qkv_tiles_of_many_rows(k_b):
    """27 heads (an odd number), 18 K tiles: 64 rows of a head (547 of 645 rows), 96 (630, 1496 of 1513), 128 (964 of 1156), 160 (1156 of 1173) and 128
    rows of two heads (2159 of 2176)."""
    desc = W.shape("mini_bf16", n_layers=1, d_model=1152, n_q_heads=21, n_kv_heads=3, d_ffn=448, vocab=333)
    ctx = [int(x) for x in np.random.default_rng(9).integers(0, 70, len(k_b))]
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=max(k_b), seed=96, q_mode="onehot", check_kv=len(k_b) == 43)


@pytest.mark.parametrize("d_model,heads,k_b,choice", [(1152, (21, 3), [14] + [1] + [0] * 41, 0), (320, (6, 2), [14] * 2 + [3] + [0] * 40, 0), (1536, (42, 6), [14] * 44 + [13, 0], 5)])
def test_qkv_tiles_of_few_rows_and_of_192(d_model, heads, k_b, choice):
    """Row limits 645 and 690: 32 rows of a head for steps with few live rows (27 heads, 58 rows; ten heads, 74), 192 rows (54 heads, 24 K tiles, 675 rows)."""
    desc = W.shape("mini_bf16", n_layers=1, d_model=d_model, n_q_heads=heads[0], n_kv_heads=heads[1], d_ffn=448, vocab=333)
    ctx, seen = [int(x) for x in np.random.default_rng(9).integers(0, 70, len(k_b))], []
    _run_case(desc, ctx_lens=ctx, k_b=k_b, k_max=14, seed=98, q_mode="onehot", check_kv=True, after_step=lambda eng: seen.append(H.tile_choice(eng, "qkv")))
    assert seen == [choice]


@pytest.mark.parametrize("d_model,d_ffn,n_seq", [(1536, 8960, 48), (1536, 8960, 64), (1536, 8960, 71), (320, 18944, 20), (320, 18944, 24), (1600, 8896, 48), (1664, 8896, 63),
                                                 (1600, 8896, 30), (1664, 8896, 42)])
def test_gate_up_tiles_of_eight_waves_and_of_one_row_block(d_model, d_ffn, n_seq):
    """24 K tiles, 70 column blocks of 128 features: eight waves on 160 (423 of 432 rows), 192 (567) and, chosen by the device, 224 rows (630).  1184 columns of 16 features: one
    block of 192 and of 224 rows (171 and 207 live) with the weights in registers.  A last column block of 64 features, 25 and 26 K tiles (1 and 2 modulo three): 160 and 192 rows
    in eight waves, 96 (261 of 270 rows) and 128 (369 of 378) in four, all fixed by the row limit."""
    desc = W.shape("mini_bf16", n_layers=1, d_model=d_model, n_q_heads=6, n_kv_heads=2, d_ffn=d_ffn, vocab=333)
    ctx = [int(x) for x in np.random.default_rng(10).integers(0, 70, n_seq)]
    _run_case(desc, ctx_lens=ctx, k_b=[8] * (n_seq - 2) + [7, 0], k_max=8, seed=97, q_mode="onehot", check_kv=False)
