"""CPU check of the compiled main loops: spills, and the order in which loads are issued.  (hipcc cross-compiles; no GPU needed.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_08862_amd import build as BLD


def stream_events(mw, nw, wn, rw, ks):
    """Loads of activations into LDS (X), of weights into registers (w) and barriers (|) of a StreamGemm loop, in the order that its
    wait counts assume: the ring's stages, then per stage (a loop of rw of them, up to rw - 1 more behind it) all steps' weights but
    the last, the barrier, the activations, the last step's weights.  The loop, and each of the stages behind it."""
    x = "X" * -(-ks * mw // wn)
    stage = "w" * ((ks - 1) * nw) + "|" + x + "w" * nw
    return [(x + "w" * (ks * nw)) * rw + "|" + stage * rw] + [stage] * (rw - 1)


def dma_events(mw, nw, wm, wn, nst):
    """Requests into LDS (X) and waits with a barrier of a DmaGemm loop: all stages but one, then a wait that leaves all but one of them in flight, and
    per stage a wait that leaves all but two in flight, with the requests of the stage whose slot is free behind it."""
    pieces, waves = 2 * (mw * wm + nw * wn), wm * wn
    ppw = -(-pieces // waves)
    return "X" * (ppw * (nst - 1)) + "<%d>" % (ppw * (nst - 2)) + "<%d>" % (ppw * (nst - 3)) + "X" * ppw


# kernels whose loops are not named in the symbol: the tiles of the declarations next to them, StreamGemm and DmaGemm
STREAMS = {"qkv_many_kernel": [(1, 1, 4, 6, 4), (2, 1, 4, 4, 4), (3, 1, 4, 3, 4), (4, 1, 4, 3, 4), (5, 1, 4, 3, 4), (6, 1, 4, 4, 2), (4, 2, 4, 2, 4)],
           "glu_w4_kernel": [(3, 2, 4, 2, 4), (4, 2, 4, 2, 4), (2, 2, 4, 2, 4), (2, 1, 4, 4, 4), (6, 1, 4, 4, 2)],
           "glu_w8_kernel": [(3, 1, 8, 3, 4), (4, 1, 8, 3, 4), (5, 1, 8, 3, 4), (6, 1, 8, 3, 4), (7, 1, 8, 2, 4), (4, 2, 8, 2, 4)]}
LOOPS = {"glu_w8_kernel": [(4, 2, 2, 4, 4)]}


def is_sequence(events, pieces):
    """Whether events are those of all the pieces, one after the other in any order (the compiler may place the stages behind a loop elsewhere)."""
    return not events if not pieces else any(events.startswith(p) and is_sequence(events[len(p):], pieces[:pieces.index(p)] + pieces[pieces.index(p) + 1:])
                                             for p in sorted(set(pieces)))


@pytest.mark.parametrize("source, kernels", [("gemm.hip", 28), ("qkv_rope.hip", 3), ("sampler.hip", 14)])
def test_weight_ring_loads_are_issued_where_they_are_written(tmp_path, source, kernels):
    """A wait for "at most N requests in flight" is right only if every request is issued where the source has it: a load that the
    compiler drops or moves past a wait would let a stage be multiplied before it has arrived.  kernels: all of the source that have such a loop."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.s"
    r = subprocess.run([hipcc, *BLD.FLAGS, "--offload-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
                        os.path.join(BLD.CSRC, source), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    spills = {n: int(s) for n, s in re.findall(r"Function Name: (\S+).*?VGPRs Spill: (\d+)", r.stderr, re.S)}
    checked = 0
    for name, body in re.findall(r"\n(_Z\S+):\s*; @.*?\n(.*?)\n\.Lfunc_end", out.read_text(), re.S):
        stream = next((v for k, v in STREAMS.items() if k in name), None)
        if not stream and not re.search(r"StreamGemmI|DmaGemmI", name):
            continue
        assert spills[name] == 0, name
        events = ""
        for line in body.split("\n"):
            line = line.strip()
            if line.startswith("buffer_load") and line.endswith(" lds"):
                events += "X"
            elif line.startswith("buffer_load_dwordx4"):
                events += "w"
            elif line.startswith("s_barrier"):
                events += "|"
        tiles = [tuple(map(int, t)) for t in re.findall(r"(?:StreamGemm|S\d*_)ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)]
        if len(tiles) == 1 or len(tiles) == 2:                # a kernel with two tiles has their loops one after the other
            orders = [tiles, tiles[::-1]]
            assert any(events.startswith("".join("".join(stream_events(*t)) for t in o)) for o in orders), (name, events)
            checked += 1
        if stream:
            dma = [re.sub(r"<\d+>", "|", dma_events(*t)) for k, v in LOOPS.items() if k in name for t in v]
            assert is_sequence(events, [p for t in stream for p in stream_events(*t)] + dma), (name, events)
            checked += 1
    assert checked == kernels, checked


@pytest.mark.parametrize("source, kernels", [("gemm.hip", 4), ("qkv_rope.hip", 1), ("attention.hip", 2)])
def test_lds_requests_are_issued_where_they_are_written(tmp_path, source, kernels):
    """The same for the loops whose operands all go through LDS (two operands of a GEMM, K/V tiles of the attention with four query tiles): the
    number of requests in front of each wait, and what the wait leaves in flight."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.s"
    r = subprocess.run([hipcc, *BLD.FLAGS, "--offload-device-only", "-S", os.path.join(BLD.CSRC, source), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    checked = 0
    for name, body in re.findall(r"\n(_Z\S+):\s*; @.*?\n(.*?)\n\.Lfunc_end", out.read_text(), re.S):
        mixed = next((v for k, v in LOOPS.items() if k in name), None)
        loops = mixed or [tuple(map(int, t)) for t in re.findall(r"DmaGemmILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)]
        head = re.search(r"attn_wide_kernelILi(\d+)E", name)
        if not loops and not head:
            continue
        events = "".join("X" if a else "<%s>" % b for a, b in re.findall(r"(buffer_load\S* [^\n]* lds\b)|;#ASMSTART\s+s_waitcnt vmcnt\((\d+)\)\s+s_barrier", body))
        if head:                                               # LPW = requests of a wave per tile; three tiles ahead, the waits of the last tiles in any order
            lpw = int(head.group(1)) // 32
            m = re.fullmatch("X{%d}((?:<\\d+>){3})X{%d}" % (3 * lpw, lpw), events)
            assert m and sorted(re.findall(r"\d+", m.group(1)), key=int) == ["0", str(lpw), str(2 * lpw)], (name, events)
        else:
            for loop in loops:
                assert events.count(dma_events(*loop)) == 1, (name, loop, events)
            assert mixed or len(events) == sum(len(dma_events(*loop)) for loop in loops), (name, events)
        checked += 1
    assert checked == kernels, checked
