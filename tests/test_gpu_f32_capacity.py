"""float32 attention with the largest row capacity: 2^22 rows of 64 heads on one KV
head, 2^28 (target, head) rows or 2^23 row tiles, more than one grid dimension holds
(the launch spreads them over two).  Few targets are active; they match a call
with just their rows."""

import numpy as np
import pytest
import torch

import oracle
from harness import assert_close, synthetic_scores
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu


def test_f32_largest_capacity(gpu_lib):
    T, H, d = 1 << 22, 64, 64
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GB of device memory")
    g = torch.Generator(device="cuda").manual_seed(1)
    kc = torch.randn(1, 1, T, d, device="cuda", generator=g)
    req = relaxkv.Request(torch.zeros(1, 1, H, d, device="cuda"), kc, kc, 20 / T)
    sets = req.alloc_sets()
    a = synthetic_scores(1, T, seed=3)
    req.select(torch.from_numpy(a).cuda(), sets)
    P = np.sort(np.random.default_rng(4).choice(T, size=11, replace=False)).astype(np.int32)
    t = torch.zeros(T, dtype=torch.int32, device="cuda")
    t[:len(P)] = torch.from_numpy(P).cuda()
    req.build_sets_global(sets, t, torch.tensor([len(P)], dtype=torch.int32, device="cuda"))
    sets.counts_to_host()
    n = len(P)
    q = torch.randn(n, H, d, device="cuda", generator=g)
    kv = torch.randn(n, 1, d, device="cuda", generator=g)
    out, lse = torch.empty_like(q), torch.empty(n, H, device="cuda")
    req.sparse_attn(sets, 0, q, kv, kv, out, lse)
    rows = torch.empty(T, H, d, device="cuda")        # queries and, in place, outputs
    kv_all = torch.empty(T, 1, d, device="cuda")
    lse_all = torch.empty(T, H, device="cuda")
    rows[:n], kv_all[:n] = q, kv
    req.sparse_attn(sets, 0, rows, kv_all, kv_all, rows, lse_all)
    sets.counts_to_host()
    ref = oracle.build_sets_global(oracle.select(a.astype(np.float64), req.k), T, P.astype(np.int64))
    assert len(ref.U) == int(sets.counts[0])
    w = synth.shrink(synth.WORKLOADS["tiny-2L-1k-fp32"], L=1, T_c=T, H=H, H_kv=1, d=d)
    keep = np.asarray(ref.R_u[0]) >= 0
    assert keep.any()
    assert_close(rows[:n].cpu().numpy()[keep], out.cpu().numpy()[keep], w, "out")
    assert_close(lse_all[:n].cpu().numpy()[keep], lse.cpu().numpy()[keep], w, "lse")
    assert not rows[:n][torch.from_numpy(~keep).cuda()].any()
    del rows, kv_all, lse_all
    torch.cuda.empty_cache()
