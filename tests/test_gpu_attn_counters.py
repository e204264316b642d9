"""The bf16 attention's work counters, in launches that use them (more than 320 row
tiles at d 128; fewer are mapped to workgroups directly): a set build clears every
slot, a launch leaves its slot clear, launches of other layers and modes may run at
the same time, and a captured sequence replays, all with the bits of one launch after
another; sampled targets against the oracle."""

import numpy as np
import pytest
import torch

import oracle
from harness import Case, assert_close, compare_sets, synthetic_scores
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS["llama8b-8k"]
MODES = {"union": relaxkv.CONTEXT_UNION, "full": relaxkv.CONTEXT_FULL}


# more KV heads than XCDs and not a multiple of them; fewer heads than XCDs, wide groups
@pytest.mark.parametrize("T,H,H_kv,ratio", [(1000, 268, 67, 0.5), (1300, 192, 3, 0.6)])
def test_work_counters(gpu_lib, T, H, H_kv, ratio):
    w = synth.shrink(W, L=3, T_c=T, H=H, H_kv=H_kv, Qn=2)
    case = Case(w, ratio=ratio)
    a = synthetic_scores(3, T, seed=T)
    sets_ref = oracle.build_sets(oracle.select(a.astype(np.float64), case.k), T)
    tiles = case.sets.tiles
    tiles.fill_(0x5A5A5A5A)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    compare_sets(case.gpu_sets(), sets_ref)
    assert tiles.shape == (2, 3, H_kv + 1) and int(tiles.abs().sum()) == 0
    jobs = [(l, m) for l in range(3) for m in MODES]
    n = [len(r) for r in sets_ref.R]
    assert all(-(-x * (H // H_kv) // 384) * H_kv > 320 for x in n)
    fresh = [case.fresh(l, sets_ref.R[l]) for l in range(3)]

    def buffers():
        return {j: (torch.zeros(n[j[0]], H, w.d, dtype=case.q.dtype, device="cuda"),
                    torch.zeros(n[j[0]], H, device="cuda")) for j in jobs}

    def launch(j, bufs, stream=None):
        case.req.sparse_attn(case.sets, j[0], *fresh[j[0]], *bufs[j], context_mode=MODES[j[1]],
                             stream=stream)

    def same(bufs, what):
        torch.cuda.synchronize()
        for j in jobs:
            assert torch.equal(bufs[j][0], seq[j][0]) and torch.equal(bufs[j][1], seq[j][1]), (what, j)
        assert int(tiles.abs().sum()) == 0, what
    seq = buffers()
    for j in jobs:
        launch(j, seq)
    same(seq, "in turn")
    for rep in range(2):                               # interleaved, then all at once
        again = buffers()
        for j in reversed(jobs):
            launch(j, again)
        same(again, rep)
        con = buffers()
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in jobs]
        for s, j in zip(streams, jobs):
            launch(j, con, s)
        same(con, ("concurrent", rep))
    cap = buffers()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for j in jobs:
            launch(j, cap)
    for rep in range(3):
        for o, z in cap.values():
            o.fill_(float("nan"))
            z.fill_(float("nan"))
        graph.replay()
        same(cap, ("graph", rep))
        launch(jobs[rep], again)                       # the program's own work in between
        same(again, ("eager", rep))
    ts = [0, 1, n[2] // 2, n[2] - 1]
    for l, m in jobs:
        O_ref, lse_ref = case.oracle_attn(l, sets_ref, fresh[l], mode=m, targets=ts)
        assert_close(seq[(l, m)][0][ts].float().cpu().numpy(), O_ref, w, f"{m} out", rel_gate=1e-2)
        assert_close(seq[(l, m)][1][ts].cpu().numpy(), lse_ref, w, f"{m} lse")
