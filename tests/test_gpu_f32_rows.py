"""The float32 kernels at the edges of their tiles: 16- and 32-row attention
workgroups (the launch rule's two sides), contexts shorter than one key block, one
key past a round of the waves' blocks, rows that do not fill a tile, empty contexts,
and fresh rows aligned to 4 bytes only; scores over the same shapes.  Every value
against the float64 oracle within the fp32 tolerance."""

import numpy as np
import pytest
import torch

import oracle
from harness import Case, assert_close, synthetic_scores
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS["tiny-2L-1k-fp32"]


def off4(t):
    """A contiguous copy of t that starts 4 bytes past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    out = buf[1:].view(t.shape)
    out.copy_(t)
    return out


# (T, H, H_kv, Qn, targets): the last two launch 32-row workgroups
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,H,H_kv,Qn,n", [(5, 1, 1, 1, 3), (33, 3, 1, 5, 33), (257, 10, 2, 3, 60),
                                           (600, 4, 4, 21, 129), (300, 32, 32, 130, 150),
                                           (540, 33, 11, 170, 151)])
def test_f32_rows(gpu_lib, T, H, H_kv, Qn, n, d):
    w = synth.shrink(W, L=2, T_c=T, H=H, H_kv=H_kv, Qn=Qn, d=d)
    case = Case(w, ratio=0.3)
    a_ref, _, _ = case.oracle_scores()
    assert_close(case.gpu_scores().cpu().numpy(), a_ref, w, "scores")
    a = synthetic_scores(2, T, seed=T)
    anchors = oracle.select(a.astype(np.float64), case.k)
    assert np.array_equal(case.gpu_select(torch.from_numpy(a).cuda()), anchors)
    P = np.sort(np.random.default_rng(n).choice(T, size=n, replace=False))
    t = torch.zeros(T, dtype=torch.int32, device="cuda")
    t[:n] = torch.from_numpy(P.astype(np.int32)).cuda()
    case.req.build_sets_global(case.sets, t, torch.tensor([n], dtype=torch.int32, device="cuda"))
    case.sets.counts_to_host()
    ref = oracle.build_sets_global(anchors, T, P)
    fresh = [off4(x) for x in case.fresh(1, P)]
    ts = sorted(set([0, 1, n - 1, n // 2] + np.random.default_rng(1).integers(0, n, 30).tolist()))
    for mode, cm in (("union", relaxkv.CONTEXT_UNION), ("full", relaxkv.CONTEXT_FULL)):
        out, lse = case.gpu_attn(1, fresh, n, cm)
        O_ref, lse_ref = case.oracle_attn(1, ref, fresh, mode=mode, targets=ts)
        empty = np.isneginf(lse_ref)
        got, got_lse = out[ts].cpu().numpy(), lse[ts].cpu().numpy()
        assert np.array_equal(np.isneginf(got_lse), empty) and not got[empty].any()
        assert_close(got[~empty], O_ref[~empty], w, f"{mode} out")
        assert_close(got_lse[~empty], lse_ref[~empty], w, f"{mode} lse")
    k_q, v_q = (off4(x) for x in synth.make_query_kv(w, 1, "cuda"))
    out = torch.empty(Qn, H, d, device="cuda")
    lse = torch.empty(Qn, H, device="cuda")
    case.req.query_attn(1, case.kc, case.vc, k_q, v_q, out, lse)
    O_ref, lse_ref = oracle.query_attn(*(synth.to_f64(x) for x in (case.q[1], case.kc[1], case.vc[1],
                                                                   k_q, v_q)))
    assert_close(out.cpu().numpy(), O_ref, w, "query out")
    assert_close(lse.cpu().numpy(), lse_ref, w, "query lse")


# The row statistics' units: 4 (the last of one key), 3 and 18 of 512 keys, each in a
# workgroup of its own or several in one (past 8, several batches), and 40 of 1024 keys.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L,T,H,H_kv,Qn", [(1, 1537, 2, 2, 1), (2, 1500, 6, 2, 30), (2, 9000, 8, 4, 130),
                                           (1, 40001, 2, 1, 2)])
def test_f32_score_units(gpu_lib, L, T, H, H_kv, Qn, d):
    w = synth.shrink(W, L=L, T_c=T, H=H, H_kv=H_kv, Qn=Qn, d=d)
    case = Case(w)
    a_ref, _, _ = case.oracle_scores()
    assert_close(case.gpu_scores().cpu().numpy(), a_ref, w, "scores")


@pytest.mark.parametrize("T", [512, 1025, 4600, 9300])
def test_f32_layer_scores_do_not_depend_on_the_other_layers(gpu_lib, T):
    """One layer (a unit per workgroup) and 64 (8 workgroups of each layer, 512 in all,
    that take every unit): the same bits."""
    w = synth.shrink(W, L=64, T_c=T, H=8, H_kv=8, Qn=5, d=64)
    q, kc, vc = synth.make_cache(w, "cuda")

    def scores(n):
        req = relaxkv.Request(q[:n], kc[:n], vc[:n], w.ratio)
        a = torch.empty(n, T, device="cuda")
        req.score(req.alloc_workspace(), a)
        return a
    assert torch.equal(scores(64)[:1], scores(1)) and torch.equal(scores(64)[:7], scores(7))


def test_f32_score_all_units_in_one_workgroup(gpu_lib):
    """33 units of 1024 keys (the last of 3), all in the one workgroup of each of 256 KV heads."""
    T, H, d = 64 * 512 + 3, 256, 64
    g = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn(1, 1, H, d, device="cuda", generator=g)
    k = torch.randn(1, H, T, d, device="cuda", generator=g)
    req = relaxkv.Request(q, k, k, 0.1)
    a = torch.empty(1, T, device="cuda")
    req.score(req.alloc_workspace(), a)
    p = torch.zeros(T, dtype=torch.float64, device="cuda")
    for h in range(H):
        p += torch.softmax(k[0, h].double() @ q[0, 0, h].double() / d ** 0.5, 0)
    ref = ((p - p.min()) / (p.max() - p.min())).cpu().numpy()
    assert_close(a[0].cpu().numpy(), ref, synth.shrink(W, T_c=T), "scores")
