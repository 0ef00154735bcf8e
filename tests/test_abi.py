"""CPU-only checks of the boundary: the library loads, exports every symbol the public header declares, and its
host-side validation rejects bad arguments without touching a GPU."""
import ctypes as C
import os
import re

import pytest

from paper_2605_08862_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(B.LIB_PATH):
        from paper_2605_08862_amd import build
        build.build()
    return B.lib()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "bubblespec.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(bs_[a-z_]+)\s*\(", header))
    assert declared >= {"bs_draft_lookup", "bs_verify_step", "bs_accept_resample", "bs_kv_commit"}
    for name in declared:
        assert hasattr(lib, name), name
    assert declared == set(B.EXPORTS)


def test_workspace_query_and_shape_validation(lib):
    ok = dict(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, d_ffn=1024, vocab=4096, dtype=B.BS_F32)
    assert B.bs_workspace_bytes(B.make_desc(ok), 4, 4) > 0
    for bad in (dict(ok, head_dim=96), dict(ok, d_model=100), dict(ok, n_q_heads=5, n_kv_heads=2),
                dict(ok, dtype=7), dict(ok, vocab=1)):
        assert B.bs_workspace_bytes(B.make_desc(bad), 4, 4) == 0
    assert B.bs_workspace_bytes(B.make_desc(ok), 0, 4) == 0
    assert B.bs_workspace_bytes(B.make_desc(dict(ok, d_model=16384)), 4, 4) > 0
    assert B.bs_workspace_bytes(B.make_desc(dict(ok, d_model=16384 + 64)), 4, 4) == 0     # row kept in registers
    assert B.bs_workspace_bytes(B.make_desc(ok), 4, B.BS_MAX_K + 1) == 0
    big = dict(n_layers=28, d_model=3584, n_q_heads=28, n_kv_heads=4, head_dim=128, d_ffn=18944, vocab=152064,
               dtype=B.BS_BF16)
    assert B.bs_workspace_bytes(B.make_desc(big), 128, 16) > 14e9          # holds the packed weights
    assert B.bs_workspace_bytes(B.make_desc(big), 128, 20) == 0            # 21 * 7 query rows > 128 per KV head


def test_null_arguments_are_rejected(lib):
    out = C.c_void_p()
    assert lib.bs_create(None, None, None, None, 0, 1, 1, None, C.byref(out)) == B.BS_EINVAL
    assert lib.bs_verify_step(None, 1, None, None, None, None, 0, None, None) == B.BS_EINVAL
    assert lib.bs_kv_commit(None, 1, None, None, None) == B.BS_EINVAL
    assert lib.bs_draft_lookup(None, 1, None, None, 4, 1, 4, None, None, None) == B.BS_EINVAL
    assert lib.bs_set_filter(None, 5, 0.9, None) == B.BS_EINVAL
    assert lib.bs_last_error(None) == b"null context"


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0 and "ONE GPU" in r.stderr


def test_bench_setup_guard_stops_on_non_finite_logits():
    """bench.py feeds the library's logits to torch.multinomial during set-up; a non-finite value must end the program
    on the host (SystemExit naming the step) before it reaches that device-asserting op.  Stub tensors, no GPU."""
    import torch
    import bench
    bench.check_finite(torch.zeros(3, 5), "stub")
    for bad in (float("inf"), float("-inf"), float("nan")):
        z = torch.zeros(3, 5)
        z[1, 2] = bad
        with pytest.raises(SystemExit) as e:
            bench.check_finite(z, "set-up decode step 4 of stub")
        assert "set-up decode step 4" in str(e.value) and e.value.code != 0


@pytest.mark.parametrize("name,B_max,k_max,accepted", [
    ("s7b", 128, 16, 15160072192), ("s7b", 32, 8, 14409985792), ("s7b", 64, 0, 14282450432), ("s7b", 1, 0, 14226674432),
    ("s1p5b", 256, 16, 4019766272), ("s1p5b", 64, 8, 3291568128), ("s1p5b", 1, 8, 3174217984), ("s1p5b", 61, 16, 3439172096),
    ("mini_bf16", 4, 7, 48531456), ("mini_bf16", 1, 0, 46870784), ("tiny", 4, 4, 625664)])
def test_workspace_sizes_that_were_enough_stay_enough(lib, name, B_max, k_max, accepted):
    """Workspace sizes from before accept calls kept logits: a program that laid out its memory for them is not refused, and
    the size that is asked for is at most 140 MB more.  The size is checked before anything is launched (the pointers here
    are made up, so without a GPU a call that passes the check ends in BS_EHIP)."""
    import torch
    from paper_2605_08862_amd import workloads as W
    if torch.cuda.is_available():
        pytest.skip("made-up device pointers")
    desc = W.shape(name)
    cdesc, L = B.make_desc(desc), desc["n_layers"]
    assert B.bs_workspace_bytes(cdesc, B_max, k_max) <= accepted + (140 << 20)
    ptrs = (C.c_void_p * L)(*[4096] * L)
    w = B.bs_weights(4096, 4096, 4096, ptrs, ptrs, ptrs, ptrs, ptrs, ptrs)
    kv = B.bs_kv_desc(1, 1, 1, ptrs, ptrs, 4096, 4096)
    create = lambda n: lib.bs_create(C.byref(cdesc), C.byref(w), C.byref(kv), 4096, n, B_max, k_max, None, C.byref(C.c_void_p()))
    assert create(accepted) == B.BS_EHIP
    assert create(accepted * 9 // 10) == B.BS_ECAPACITY


def test_stream_address_without_the_private_torch_functions(monkeypatch):
    import types
    import torch
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert B._stream() == 77
