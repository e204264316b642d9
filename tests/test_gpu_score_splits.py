"""Scores where the passes take fewer keys per workgroup than a full split: context
lengths around 512-key multiples with few and many layers (the split depends on
both), in both modes, against the oracle; and the pooling over KV-head counts that
do not divide its unrolled loads."""

import pytest
import torch

import oracle
from harness import assert_close
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS["llama8b-8k"]


@pytest.mark.parametrize("L,T,H,H_kv,d,Qn", [(1, 511, 8, 8, 128, 3), (2, 513, 9, 9, 64, 40), (2, 1025, 3, 1, 128, 110),
                                             (13, 1537, 16, 2, 64, 7), (30, 2049, 8, 8, 64, 4),
                                             (2, 4096, 20, 10, 128, 17), (2, 4097, 8, 2, 128, 5)])
def test_score_splits(gpu_lib, L, T, H, H_kv, d, Qn):
    w = synth.shrink(W, L=L, T_c=T, H=H, H_kv=H_kv, d=d, Qn=Qn, std=1.0)
    q, kc, vc = synth.make_cache(w, "cuda")
    check = sorted({0, L // 2, L - 1})
    a_ref, _, lse_ref = oracle.score(synth.to_f64(q[check]), synth.to_f64(kc[check]))
    lse = torch.zeros(L, Qn, H, device="cuda")
    lse[check] = torch.from_numpy(lse_ref).float().cuda().reshape(len(check), Qn, H)
    for q_lse in (None, lse):
        req = relaxkv.Request(q, kc, vc, 0.15, q_lse=q_lse)
        a = torch.empty(L, T, device="cuda")
        req.score(req.alloc_workspace(), a)
        assert_close(a[check].cpu().numpy(), a_ref, w, "scores", rel_gate=1e-2)


# 320 rows (one chunk, its statistics merged while staging), 352 (a merge launch), eight
# splits merged while staging and nine by the launch
@pytest.mark.parametrize("L,T,H,H_kv,d,Qn", [(1, 3000, 16, 2, 64, 40), (1, 3000, 16, 2, 64, 44),
                                             (1, 32768, 6, 2, 128, 30), (1, 32769, 6, 2, 128, 30)])
def test_score_merge_sides(gpu_lib, L, T, H, H_kv, d, Qn):
    test_score_splits(gpu_lib, L, T, H, H_kv, d, Qn)
