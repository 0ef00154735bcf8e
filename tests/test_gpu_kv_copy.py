"""Cache import / export at the edges of the page layout: ranges that start or end inside a tile of 32 tokens or a group of eight,
row tensors that are aligned to their elements only, and the range check.  Bit-exact; tokens beside the range keep their values."""
import pytest
import torch

from paper_2605_08862_amd import binding as B
from paper_2605_08862_amd import workloads as W
from paper_2605_08862_amd.runtime import Engine, fuse_weights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N_TOK = 200


@pytest.fixture(scope="module", params=[("mini_bf16", 128), ("mini_bf16", 64), ("tiny", 64)], ids=lambda p: "%s-%d" % p)
def eng(request):
    name, head_dim = request.param
    desc = W.shape(name, head_dim=head_dim, n_layers=2)
    e = Engine(desc, fuse_weights(W.make_weights(desc, seed=1), desc["dtype"], DEV), 3, N_TOK, B_max=3, k_max=0, page_perm_seed=5)
    yield e
    e.close()


def _rows(eng, n, seed, shifted=False):
    d = eng.desc
    shape = (n, d["n_kv_heads"], d["head_dim"])
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(shape, generator=g, device=DEV)
    x[x.abs() < 1e-3] = 0.5                                          # float16 holds bf16 values exactly from 6.1e-5 on
    x = x.to(W.torch_dtype(d))
    if not shifted:
        return x
    buf = torch.empty(x.numel() + 1, dtype=x.dtype, device=DEV)      # a view that starts one element into its buffer
    buf[1:].copy_(x.reshape(-1))
    return buf[1:].view(shape)


@pytest.mark.parametrize("shifted", [False, True])
@pytest.mark.parametrize("pos0", [0, 1, 7, 8, 31, 33, 63])
@pytest.mark.parametrize("n", [1, 7, 9, 65])
def test_import_replaces_its_range_and_nothing_else(eng, pos0, n, shifted):
    want = [[_rows(eng, N_TOK, 10 * l + i) for i in (0, 1)] for l in (0, 1)]
    for l in (0, 1):
        eng.kv_write(l, 1, 0, *want[l])
        eng.kv_write(l, 0, 0, *want[l])
    k, v = _rows(eng, n, 77, shifted), _rows(eng, n, 78, shifted)
    eng.kv_write(1, 1, pos0, k, v)
    before = [[t.clone() for t in w] for w in want]
    want[1][0][pos0:pos0 + n], want[1][1][pos0:pos0 + n] = k, v
    for l in (0, 1):
        for slot, ref in ((1, want[l]), (0, before[l])):             # the other layer and the other slot are untouched
            got = eng.kv_read(l, slot, 0, N_TOK)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), (l, slot)
    assert eng.poll_status() == 0


@pytest.mark.parametrize("shifted", [False, True])
@pytest.mark.parametrize("pos0,n", [(0, 200), (1, 1), (5, 3), (7, 65), (31, 2), (33, 94), (63, 130)])
def test_export_writes_its_rows_and_nothing_else(eng, pos0, n, shifted):
    k, v = _rows(eng, N_TOK, 3), _rows(eng, N_TOK, 4)
    eng.kv_write(0, 2, 0, k, v)
    row = k[0].numel()
    lead = 1 if shifted else 8                                       # 8 elements: sixteen bytes of bf16, thirty-two of float32
    out = []
    for _ in range(2):
        buf = torch.full((lead + n * row + 8,), 9.0, dtype=k.dtype, device=DEV)
        out.append((buf, buf[lead:lead + n * row].view(n, *k.shape[1:])))
    B.bs_kv_read(eng.ctx, 0, 2, pos0, n, out[0][1], out[1][1])
    for (buf, got), ref in zip(out, (k, v)):
        assert torch.equal(got, ref[pos0:pos0 + n])
        assert (buf[:lead] == 9.0).all() and (buf[lead + n * row:] == 9.0).all()
    assert eng.poll_status() == 0


@pytest.mark.parametrize("which", [0, 1])
@pytest.mark.parametrize("shifted", [False, True])
def test_import_range_check_sees_exactly_the_imported_rows(eng, which, shifted):
    """A bf16 value that float16 cannot hold is saturated and reported when its row is imported, and not looked at otherwise."""
    if eng.desc["dtype"] != B.BS_BF16:
        pytest.skip("float32 pages hold every value")
    pos0, n = 13, 22
    big = [_rows(eng, n + 2, 5, shifted), _rows(eng, n + 2, 6, shifted)]
    for i, fault in ((0, 0), (n + 1, 0), (1, B.BS_FAULT_RANGE), (n, B.BS_FAULT_RANGE)):      # just outside, just inside
        rows = [t.clone() if not shifted else t for t in big]
        keep = rows[which][i, 0, 3].item()
        rows[which][i, 0, 3] = -1e30
        B.bs_kv_write(eng.ctx, 0, 0, pos0, n, rows[0][1:n + 1], rows[1][1:n + 1])
        assert eng.poll_status() == fault, i
        got = eng.kv_read(0, 0, pos0, n)
        ref = rows[which][1:n + 1].clone()
        if fault:
            ref[i - 1, 0, 3] = -65504.0                              # the nearest bf16 value is read back
        assert torch.equal(got[which], ref) and torch.equal(got[1 - which], rows[1 - which][1:n + 1])
        rows[which][i, 0, 3] = keep
