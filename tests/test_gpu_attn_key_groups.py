"""The bf16 attention on both sides of its key-group rule: launches of at most 320
384-row tiles (432, and 600 to 768, at d 64) split each workgroup's keys over two wave
groups, others do not.  Sampled targets (the first ones, whose contexts end inside the first key
group's keys, and the last of a ragged tile among them) against the oracle, and
the work counters are zero afterwards on both sides."""

import numpy as np
import pytest
import torch

import oracle
from harness import Case, assert_close, synthetic_scores
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS["llama8b-8k"]


# G = 4: 960 targets of 32 KV heads fill 320 tiles, 1152 of 64 heads 768.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,G,H_kv,n", [(97, 1, 32, 97), (96, 3, 32, 33), (129, 2, 5, 128), (1000, 4, 32, 960),
                                        (1000, 4, 32, 961), (1100, 5, 32, 700), (1200, 4, 64, 1152),
                                        (1200, 4, 64, 1153)])
def test_key_groups(gpu_lib, T, G, H_kv, n, d):
    w = synth.shrink(W, L=2, T_c=T, H=H_kv * G, H_kv=H_kv, d=d, Qn=2)
    case = Case(w, ratio=0.4)
    a = synthetic_scores(2, T, seed=T)
    anchors = oracle.select(a.astype(np.float64), case.k)
    assert np.array_equal(case.gpu_select(torch.from_numpy(a).cuda()), anchors)
    rng = np.random.default_rng(n + d)
    P = np.sort(rng.choice(T, size=n, replace=False))      # some with empty contexts
    t = torch.zeros(T, dtype=torch.int32, device="cuda")
    t[:n] = torch.from_numpy(P.astype(np.int32)).cuda()
    case.req.build_sets_global(case.sets, t, torch.tensor([n], dtype=torch.int32, device="cuda"))
    case.sets.counts_to_host()
    ref = oracle.build_sets_global(anchors, T, P)
    ts = sorted(set(list(range(4)) + [n // 2, n - 2, n - 1] + rng.integers(0, n, 6).tolist()))
    fresh = case.fresh(1, P)
    for mode, cm in (("union", relaxkv.CONTEXT_UNION), ("full", relaxkv.CONTEXT_FULL)):
        out, lse = case.gpu_attn(1, fresh, n, cm)
        O_ref, lse_ref = case.oracle_attn(1, ref, fresh, mode=mode, targets=ts)
        empty = np.isneginf(lse_ref)
        got, got_lse = out[ts].float().cpu().numpy(), lse[ts].cpu().numpy()
        assert np.array_equal(np.isneginf(got_lse), empty) and not got[empty].any()
        assert_close(got[~empty], O_ref[~empty], w, f"{mode} out", rel_gate=1e-2)
        assert_close(got_lse[~empty], lse_ref[~empty], w, f"{mode} lse")
        assert int(case.sets.tiles.abs().sum()) == 0


# 13, 14, 18 and 19 tiles of 32 KV heads: 416 (two key groups), 448, 576, 608 (two)
@pytest.mark.parametrize("n", [1248, 1249, 1728, 1729])
def test_key_groups_d64_lines(gpu_lib, n):
    test_key_groups(gpu_lib, 1800, 4, 32, n, 64)
