"""float32 attention and query side: what is not finite in a key or value reaches the
rows that see that position and no other.  Rows before it keep their bits, empty
contexts stay exact zeros, and the rows that see an Inf or NaN in V have it in those
elements of O (p > 0 there) and their other elements unchanged."""

import math

import numpy as np
import pytest
import torch

import oracle
from harness import Case, synthetic_scores
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS["tiny-2L-1k-fp32"]
BAD = {3: math.inf, 5: math.nan, 10: -math.inf, 63: math.inf}


def spoil(row):
    for d, x in BAD.items():
        row[..., d] = x


def compare(got, base, sees, g, G):
    """got against the finite run: rows that do not see the position, and other KV
    heads, keep their bits; the others have BAD in its elements."""
    hd = slice(g * G, (g + 1) * G)
    want = base.clone()
    for d, x in BAD.items():
        want[sees, hd, d] = x
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got.nan_to_num(nan=0., posinf=7e30, neginf=-7e30),
                       want.nan_to_num(nan=0., posinf=7e30, neginf=-7e30))


# the last one launches 32-row workgroups, the others 16-row ones
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,H,H_kv,Qn,n", [(5, 1, 1, 4, 3), (257, 10, 2, 7, 60), (300, 32, 32, 130, 150)])
def test_f32_nonfinite(gpu_lib, T, H, H_kv, Qn, n, d):
    w = synth.shrink(W, L=2, T_c=T, H=H, H_kv=H_kv, Qn=Qn, d=d)
    case = Case(w, ratio=0.3)
    G, g = H // H_kv, H_kv - 1
    a = synthetic_scores(2, T, seed=T)
    anchors = oracle.select(a.astype(np.float64), case.k)
    case.gpu_select(torch.from_numpy(a).cuda())
    P = np.sort(np.random.default_rng(n).choice(T, size=n, replace=False))
    t = torch.zeros(T, dtype=torch.int32, device="cuda")
    t[:n] = torch.from_numpy(P.astype(np.int32)).cuda()
    case.req.build_sets_global(case.sets, t, torch.tensor([n], dtype=torch.int32, device="cuda"))
    case.sets.counts_to_host()
    ref = oracle.build_sets_global(anchors, T, P)
    q, k, v = (x.clone() for x in case.fresh(1, P))
    for mode, cm in (("union", relaxkv.CONTEXT_UNION), ("full", relaxkv.CONTEXT_FULL)):
        base, lse = case.gpu_attn(1, (q, k, v), n, cm)
        lim = np.asarray(ref.R_u[1]) if mode == "union" else P
        ctx = np.asarray(ref.U) if mode == "union" else np.arange(T)
        assert not base[lim < 0].any()
        for t_bad in (n // 2, n - 1):                  # a target's fresh value, then its key
            at = int(np.searchsorted(ctx, P[t_bad]))   # its index in the context, if it is there
            there = at < len(ctx) and ctx[at] == P[t_bad]
            sees = torch.from_numpy((lim >= at) & there).cuda()
            vb = v.clone()
            spoil(vb[t_bad, g])
            got, got_lse = case.gpu_attn(1, (q, k, vb), n, cm)
            compare(got, base, sees, g, G)
            assert torch.equal(got_lse, lse)
            kb = k.clone()
            kb[t_bad, g, 1] = math.nan
            got, got_lse = case.gpu_attn(1, (q, kb, v), n, cm)
            hd = slice(g * G, (g + 1) * G)
            assert torch.equal(got[~sees], base[~sees]) and torch.equal(got_lse[~sees], lse[~sees])
            assert torch.isnan(got[sees][:, hd]).all()
        cached = [int(c) for c in ctx if c not in set(P.tolist())]
        if cached:                                     # a cached value in the middle
            at = int(np.searchsorted(ctx, cached[len(cached) // 2]))
            sees = torch.from_numpy(lim >= at).cuda()
            old = case.vc[1, g, ctx[at]].clone()
            spoil(case.vc[1, g, ctx[at]])
            got, got_lse = case.gpu_attn(1, (q, k, v), n, cm)
            case.vc[1, g, ctx[at]] = old
            compare(got, base, sees, g, G)
            assert torch.equal(got_lse, lse)

    k_q, v_q = synth.make_query_kv(w, 1, "cuda")

    def query(k_q, v_q):
        out = torch.empty(Qn, H, d, device="cuda")
        lse = torch.empty(Qn, H, device="cuda")
        case.req.query_attn(1, case.kc, case.vc, k_q, v_q, out, lse)
        return out, lse
    base, lse = query(k_q, v_q)
    tok = torch.arange(Qn, device="cuda")
    for t_bad in (0, Qn // 2, Qn - 1):
        vb = v_q.clone()
        spoil(vb[t_bad, g])
        got, got_lse = query(k_q, vb)
        compare(got, base, tok >= t_bad, g, G)
        assert torch.equal(got_lse, lse)
    kb = k_q.clone()
    kb[Qn - 1, g, 1] = math.nan
    got, got_lse = query(kb, v_q)
    assert torch.equal(got[:-1], base[:-1]) and torch.equal(got_lse[:-1], lse[:-1])
