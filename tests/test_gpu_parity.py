"""GPU parity of the HIP path (through the C ABI) against the float64 oracle.

Bars: index outputs bit-exact when both sides see the same fp32 scores;
scores and attention outputs within 2e-2 max-abs for bf16 inputs (plus a
normalised gate max|O - O_ref| / max|O_ref| <= 1e-2) and within 1e-5
tensor-relative for fp32 inputs.  Small workloads span several tiles with
ragged tails; the 32K planted workload is checked at full size on sampled
layers and targets, in the launch configuration the benchmark times.
"""

import math

import numpy as np
import pytest
import torch

import oracle
from harness import Case, assert_close, compare_sets, every_target_property, synthetic_scores
from paper_2609_33503_amd import relaxkv, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS
SMALL = {
    "tiny": W["tiny-2L-1k-fp32"],
    "llama-shape": synth.shrink(W["llama8b-8k"], L=3, T_c=1500),
    "qwen-shape": synth.shrink(W["qwen14b-16k"], L=3, T_c=2000),
    "qwen-planted": synth.shrink(W["qwen14b-32k-planted"], L=4, T_c=2600),
    "qwen-latent": synth.shrink(W["qwen14b-32k-latent"], L=6, T_c=2600),
    "d64-bf16": synth.shrink(W["llama8b-8k"], L=2, T_c=777, H=8, H_kv=2, d=64, Qn=24),
    "mha-bf16": synth.shrink(W["llama8b-8k"], L=2, T_c=640, H=4, H_kv=4, Qn=8),
    "fp32-d128": synth.shrink(W["tiny-2L-1k-fp32"], L=2, T_c=300, d=128, H=6, H_kv=3, Qn=5),
    # 100 query tokens x 5 heads = 500 score rows: the scoring passes take two
    # row chunks per workgroup (the column sums accumulate across chunks)
    "long-query": synth.shrink(W["qwen14b-16k"], L=2, T_c=1300, Qn=100),
    "gqa16": synth.shrink(W["llama8b-8k"], L=2, T_c=900, H=32, H_kv=2, Qn=8),
    "gqa12-d64": synth.shrink(W["llama8b-8k"], L=3, T_c=1100, H=24, H_kv=2, d=64, Qn=12),
    # more KV heads than XCDs, and a KV-head count that does not divide their number
    "kv16": synth.shrink(W["llama8b-8k"], L=2, T_c=1000, H=32, H_kv=16, Qn=8),
    "kv3": synth.shrink(W["llama8b-8k"], L=2, T_c=1000, H=12, H_kv=3, Qn=8),
    # G = 7 and G = 10 do not divide the 384 rows of an attention tile: tiles begin and
    # end inside a target's group of heads, whose context two workgroups then read
    "gqa7": synth.shrink(W["llama8b-8k"], L=3, T_c=1200, H=14, H_kv=2, Qn=8),
    "gqa10-d64": synth.shrink(W["llama8b-8k"], L=2, T_c=1000, H=20, H_kv=2, d=64, Qn=8),
}


def _pipeline(case, mode="union", check_attn=True, rel_gate=1e-2):
    w = case.w
    a_gpu = case.gpu_scores().cpu().numpy()
    a_ref, _, _ = case.oracle_scores()
    assert_close(a_gpu, a_ref, w, "scores")

    # indices bit-exact on shared fp32 scores (the oracle's, rounded to fp32)
    a32 = a_ref.astype(np.float32)
    anchors = case.gpu_select(torch.from_numpy(a32).cuda())
    anchors_ref = oracle.select(a32.astype(np.float64), case.k)
    assert np.array_equal(anchors, anchors_ref)
    sets_ref = oracle.build_sets(anchors_ref, case.T)
    got = case.gpu_sets()
    compare_sets(got, sets_ref)
    if not check_attn:
        return
    cm = relaxkv.CONTEXT_FULL if mode == "full" else relaxkv.CONTEXT_UNION
    for l in range(case.L):
        R_l = sets_ref.R[l]
        fresh = case.fresh(l, R_l)
        out, lse = case.gpu_attn(l, fresh, len(R_l), cm)
        O_ref, lse_ref = case.oracle_attn(l, sets_ref, fresh, mode=mode)
        assert_close(out.float().cpu().numpy(), O_ref, w, f"O layer {l}",
                     rel_gate=rel_gate if w.dtype == "bf16" else None)
        assert_close(lse.cpu().numpy(), lse_ref, w, f"lse layer {l}")


@pytest.mark.parametrize("name", list(SMALL))
def test_pipeline_small(gpu_lib, name):
    _pipeline(Case(SMALL[name]))


@pytest.mark.parametrize("name", ["tiny", "qwen-planted", "qwen-latent", "gqa7", "d64-bf16", "mha-bf16"])
def test_full_prefix_small(gpu_lib, name):
    _pipeline(Case(SMALL[name]), mode="full")


@pytest.mark.parametrize("ratio", [0.05, 0.30])
def test_ratio_sweep_small(gpu_lib, ratio):
    _pipeline(Case(SMALL["qwen-shape"], ratio=ratio))


def test_ratio_one_is_causal_attention(gpu_lib):
    # r = 1: every position is an anchor of every layer, so U = R_l = all and
    # the attention is plain causal attention on the fresh rows.
    w = synth.shrink(W["llama8b-8k"], L=2, T_c=333, Qn=8)
    case = Case(w, ratio=1.0)
    assert case.k == w.T_c
    _pipeline(case)


def test_minimum_context(gpu_lib):
    w = synth.shrink(W["llama8b-8k"], L=2, T_c=1, Qn=4)
    _pipeline(Case(w))
    w2 = synth.shrink(W["llama8b-8k"], L=3, T_c=100, Qn=4)
    _pipeline(Case(w2, ratio=0.0))          # k = 1


def test_supplied_lse_scoring(gpu_lib):
    w = SMALL["qwen-shape"]
    base = Case(w)
    _, p_ref, lse_ref = base.oracle_scores()
    # a larger normaliser than the cached keys alone, as a real query forward has
    lse = torch.from_numpy((lse_ref + 0.3).astype(np.float32)).cuda()
    case = Case(w, q_lse=lse)
    a_gpu = case.gpu_scores().cpu().numpy()
    a_ref, _, _ = oracle.score(synth.to_f64(case.q), synth.to_f64(case.kc),
                               row_lse=synth.to_f64(lse))
    assert_close(a_gpu, a_ref, w, "scores with supplied lse")


@pytest.mark.parametrize("kind,T_c", [("large", 1500), ("negative", 1500), ("negative", 4097)])
def test_scores_extreme_logits(gpu_lib, kind, T_c):
    """Logits far outside the unit range (tens to hundreds of log2 units): the
    row statistics must stay exact when a block's sum of exp2 would overflow
    fp32 ("large": spread of about +-150 log2 units) or underflow against the
    starting reference ("negative": every logit near -500 log2 units).  At
    T_c = 4097 the last 4096-key split holds one key, so half of each row's
    lanes meet no key there and must not pull the merged reference to 0."""
    w = synth.shrink(W["llama8b-8k"], L=2, T_c=T_c, Qn=4)
    case = Case(w)
    g = torch.Generator().manual_seed(7)
    if kind == "large":
        case.kc.mul_(4000.0)
    else:
        u = torch.randn(w.d, generator=g, dtype=torch.float64)
        u /= u.norm()
        noise = torch.randn(w.L, w.H_kv, w.T_c, w.d, generator=g, dtype=torch.float64) * 40.0
        case.q.copy_(u.expand_as(case.q).to(case.q.dtype))
        case.kc.copy_((-3925.0 * u + noise).to(case.kc.dtype))
    a_gpu = case.gpu_scores().cpu().numpy()
    a_ref, _, lse_ref = case.oracle_scores()
    assert np.abs(lse_ref).max() > 60.0          # the logits are in the extreme range
    assert_close(a_gpu, a_ref, w, f"scores ({kind} logits)")


def test_equal_keys_select_first_k(gpu_lib):
    w = synth.shrink(W["llama8b-8k"], L=2, T_c=700, Qn=4)
    case = Case(w)
    case.kc[:] = case.kc[:, :, :1, :]            # every key of a head equal
    a = case.gpu_scores()
    assert float(a.abs().max()) == 0.0
    anchors = case.gpu_select(a)
    assert anchors.tolist() == [list(range(case.k))] * 2


def test_nan_score_sets_error_word(gpu_lib):
    w = synth.shrink(W["llama8b-8k"], L=2, T_c=500, Qn=4)
    case = Case(w)
    a = torch.rand(2, 500, device="cuda")
    a[1, 17] = float("nan")
    anchors = case.gpu_select(a)
    assert anchors.min() >= 0 and anchors.max() < 500      # indices stay in range
    case.req.build_sets(case.sets)
    with pytest.raises(relaxkv.RelaxKVError) as e:
        case.sets.counts_to_host()
    assert e.value.status == relaxkv.EINVAL
    case.gpu_select(torch.rand(2, 500, device="cuda"))       # a clean call clears it
    case.req.build_sets(case.sets)
    case.sets.counts_to_host()


def test_determinism(gpu_lib):
    case = Case(SMALL["qwen-planted"])
    a1 = case.gpu_scores()
    a2 = case.gpu_scores()
    assert torch.equal(a1, a2)
    case.gpu_select(a1)
    g1 = case.gpu_sets()
    R0 = g1["R"][0]
    fresh = case.fresh(0, R0)
    o1, l1 = case.gpu_attn(0, fresh, len(R0))
    o2, l2 = case.gpu_attn(0, fresh, len(R0))
    assert torch.equal(o1, o2) and torch.equal(l1, l2)


# ---------------------------------------------------------------- full size

BIG = W["qwen14b-32k-planted"]


@pytest.fixture(scope="module")
def big_case(gpu_lib):
    return Case(BIG)


def test_full_size_scores_every_layer(big_case):
    """Scores of all 40 layers of the 32K workload against the oracle (one
    layer at a time, so the float64 copies stay small); the planted positions
    are selected in every layer."""
    a_gpu = big_case.gpu_scores().cpu().numpy()
    planted = set(synth.planted_positions(BIG).numpy().tolist())
    for l in range(BIG.L):
        a_ref, _, _ = big_case.oracle_scores([l])
        assert_close(a_gpu[[l]], a_ref, BIG, f"scores (32K, layer {l})")
        anchors_ref = oracle.select(a_ref, big_case.k)
        assert planted <= set(anchors_ref[0].tolist()), l


def test_full_size_select_and_sets_bit_exact(big_case):
    for levels in (None, 64):
        a = synthetic_scores(BIG.L, BIG.T_c, seed=11 + (levels or 0), levels=levels)
        anchors = big_case.gpu_select(torch.from_numpy(a).cuda())
        anchors_ref = oracle.select(a.astype(np.float64), big_case.k)
        assert np.array_equal(anchors, anchors_ref)
        compare_sets(big_case.gpu_sets(), oracle.build_sets(anchors_ref, BIG.T_c))


@pytest.mark.parametrize("mode", ["union", "full"])
def test_full_size_attention_sampled(big_case, mode):
    # sets from the oracle's selection on seeded scores; the GPU builds its own
    # sets from those anchors (bit-exact) and runs the benchmark's kernels.
    a = synthetic_scores(BIG.L, BIG.T_c, seed=5)
    anchors_ref = oracle.select(a.astype(np.float64), big_case.k)
    sets_ref = oracle.build_sets(anchors_ref, BIG.T_c)
    big_case.req.select(torch.from_numpy(a).cuda(), big_case.sets)
    compare_sets(big_case.gpu_sets(), sets_ref)
    cm = relaxkv.CONTEXT_FULL if mode == "full" else relaxkv.CONTEXT_UNION
    rng = np.random.default_rng(3)
    for l in (0, 19, BIG.L - 1):
        R_l = sets_ref.R[l]
        n = len(R_l)
        fresh = big_case.fresh(l, R_l)
        out, lse = big_case.gpu_attn(l, fresh, n, cm)
        ts = sorted(set([0, 1, 2, n // 2, n - 3, n - 2, n - 1] +
                        rng.integers(0, n, size=9).tolist()))
        O_ref, lse_ref = big_case.oracle_attn(l, sets_ref, fresh, mode=mode, targets=ts)
        assert_close(out[ts].float().cpu().numpy(), O_ref, BIG, f"O layer {l} ({mode})",
                     rel_gate=1e-2)
        assert_close(lse[ts].cpu().numpy(), lse_ref, BIG, f"lse layer {l} ({mode})")
        # softmax rows sum to 1 under the GPU's log-sum-exp
        t = ts[-1]
        ctx = sets_ref.U[sets_ref.U <= R_l[t]] if mode == "union" else np.arange(R_l[t] + 1)
        rank = np.full(BIG.T_c, -1)
        rank[R_l] = np.arange(n)
        qn, kn = synth.to_f64(fresh[0][t]), synth.to_f64(fresh[1])
        kc = synth.to_f64(big_case.kc[l])
        g = 0
        K = np.where((rank[ctx] >= 0)[:, None], kn[np.maximum(rank[ctx], 0), g], kc[g, ctx])
        s = K @ qn[0] / math.sqrt(BIG.d)
        assert np.exp(s - float(lse[t, 0])).sum() == pytest.approx(1.0, abs=2e-3)


def test_full_size_update_cache_bit_exact(big_case):
    """The cache update at 32K in the benchmark's launch configuration: the
    repaired layers equal the oracle's bit for bit (out of place), and layers
    that were not updated are untouched."""
    a = synthetic_scores(BIG.L, BIG.T_c, seed=5)
    sets_ref = oracle.build_sets(oracle.select(a.astype(np.float64), big_case.k), BIG.T_c)
    big_case.req.select(torch.from_numpy(a).cuda(), big_case.sets)
    compare_sets(big_case.gpu_sets(), sets_ref)
    k_out, v_out = big_case.kc.clone(), big_case.vc.clone()
    layers = (0, 19, BIG.L - 1)
    for l in layers:
        _, kn, vn = big_case.fresh(l, sets_ref.R[l])
        big_case.req.update_cache(big_case.sets, l, kn, vn, k_out, v_out)
        torch.cuda.synchronize()
        kr, vr = oracle.update_cache(l, sets_ref, synth.to_f64(kn), synth.to_f64(vn),
                                     synth.to_f64(big_case.kc[l]), synth.to_f64(big_case.vc[l]))
        assert np.array_equal(synth.to_f64(k_out[l]), kr), l
        assert np.array_equal(synth.to_f64(v_out[l]), vr), l
    others = [l for l in range(BIG.L) if l not in layers]
    assert torch.equal(k_out[others], big_case.kc[others])
    assert torch.equal(v_out[others], big_case.vc[others])


@pytest.mark.parametrize("mode,l", [("union", 19), ("full", 19), ("union", 39)])
def test_full_size_attention_every_target(big_case, mode, l):
    """Every target and head of a 32K layer (|R_l| about 27 500 targets x 40
    heads at layer 19; the 4 915 targets of the last layer, the sparsest in U,
    where tiles span the widest staircase and waves skip the most steps): the
    property check of harness.every_target_property at full size; the element-wise
    parity with the oracle is the sampled test above."""
    a = synthetic_scores(BIG.L, BIG.T_c, seed=5)
    anchors_ref = oracle.select(a.astype(np.float64), big_case.k)
    sets_ref = oracle.build_sets(anchors_ref, BIG.T_c)
    big_case.req.select(torch.from_numpy(a).cuda(), big_case.sets)
    compare_sets(big_case.gpu_sets(), sets_ref)
    every_target_property(big_case, sets_ref, l, mode)


@pytest.mark.parametrize("name,ratio,l", [("llama8b-8k", None, 0), ("qwen14b-16k", 0.30, 20)])
def test_full_size_workload_every_target(gpu_lib, name, ratio, l):
    """The same property check on every target and head of one layer of the 8K
    Llama-shaped workload (layer 0: all of U, G = 4) and of the 16K workload at
    a 30% anchor ratio, on sets from seeded scores."""
    case = Case(W[name], ratio=ratio)
    a = synthetic_scores(case.L, case.T, seed=31)
    anchors_ref = oracle.select(a.astype(np.float64), case.k)
    sets_ref = oracle.build_sets(anchors_ref, case.T)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    compare_sets(case.gpu_sets(), sets_ref)
    every_target_property(case, sets_ref, l, "union")


# ---------------------------------------------------------------- every workload at full size

@pytest.mark.parametrize("name,ratio", [("llama8b-8k", None), ("qwen14b-16k", 0.05),
                                        ("qwen14b-16k", 0.15), ("qwen14b-16k", 0.30)])
def test_full_size_workloads(gpu_lib, name, ratio):
    """Full-size workloads: scores within tolerance on every layer (on sampled
    layers for the 16K ratio points other than 0.15, whose scores are the same);
    selection and sets bit-exact on the oracle's fp32 scores of those layers (the
    other layers take seeded scores); attention on sampled targets of three
    layers, in the launch configuration the benchmark uses."""
    w = W[name]
    case = Case(w, ratio=ratio)
    L, T = case.L, case.T
    layers = [0, L // 2, L - 1]
    score_layers = list(range(L)) if ratio in (None, 0.15) else layers
    a_gpu = case.gpu_scores().cpu().numpy()
    a = synthetic_scores(L, T, seed=21)
    for l in score_layers:                           # one layer at a time (float64 copies)
        a_ref, _, _ = case.oracle_scores([l])
        assert_close(a_gpu[[l]], a_ref, w, f"scores {name} layer {l}")
        a[l] = a_ref[0].astype(np.float32)
    anchors = case.gpu_select(torch.from_numpy(a).cuda())
    anchors_ref = oracle.select(a.astype(np.float64), case.k)
    assert np.array_equal(anchors, anchors_ref)
    sets_ref = oracle.build_sets(anchors_ref, T)
    compare_sets(case.gpu_sets(), sets_ref)
    rng = np.random.default_rng(4)
    for l in layers:
        R_l = sets_ref.R[l]
        n = len(R_l)
        fresh = case.fresh(l, R_l)
        out, lse = case.gpu_attn(l, fresh, n)
        ts = sorted(set([0, n // 2, n - 1] + rng.integers(0, n, size=5).tolist()))
        O_ref, lse_ref = case.oracle_attn(l, sets_ref, fresh, targets=ts)
        assert_close(out[ts].float().cpu().numpy(), O_ref, w, f"O {name} layer {l}", rel_gate=1e-2)
        assert_close(lse[ts].cpu().numpy(), lse_ref, w, f"lse {name} layer {l}")


@pytest.mark.parametrize("name", ["qwen-planted", "tiny", "d64-bf16"])
def test_update_cache_bit_exact(gpu_lib, name):
    """The repaired cache after every layer's update equals the oracle's
    (pure data movement: bit-exact), in place and into a separate output cache."""
    w = SMALL[name]
    case = Case(w)
    a = synthetic_scores(case.L, case.T, seed=8)
    anchors_ref = oracle.select(a.astype(np.float64), case.k)
    sets_ref = oracle.build_sets(anchors_ref, case.T)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    compare_sets(case.gpu_sets(), sets_ref)
    k_out, v_out = case.kc.clone(), case.vc.clone()
    for l in range(case.L):
        R_l = sets_ref.R[l]
        _, kn, vn = case.fresh(l, R_l)
        case.req.update_cache(case.sets, l, kn, vn, k_out, v_out)
        torch.cuda.synchronize()
        kr, vr = oracle.update_cache(l, sets_ref, synth.to_f64(kn), synth.to_f64(vn),
                                     synth.to_f64(case.kc[l]), synth.to_f64(case.vc[l]))
        assert np.array_equal(synth.to_f64(k_out[l]), kr)
        assert np.array_equal(synth.to_f64(v_out[l]), vr)
    # untouched layers stay as they were when only one layer is updated in place
    R0 = sets_ref.R[0]
    _, kn, vn = case.fresh(0, R0)
    k_before = case.kc.clone()
    case.req.update_cache(case.sets, 0, kn, vn, case.kc, case.vc)
    torch.cuda.synchronize()
    assert torch.equal(case.kc[1:], k_before[1:])


@pytest.mark.parametrize("name", ["qwen-planted", "tiny"])
def test_row_capacity_clamps_and_reports(gpu_lib, name):
    """A row capacity below |R_l| (a caller that sized its buffers from a stale
    count): the attention computes exactly the first n_rows targets, writes
    nothing past them, and the device error word reports RELAXKV_ERR_ROWS, so
    relaxkv_counts_to_host returns RELAXKV_EINVAL; the cache update writes only
    the first n_rows rows.  The error word clears at the next selection."""
    w = SMALL[name]
    case = Case(w)
    a = synthetic_scores(case.L, case.T, seed=19)
    anchors_ref = oracle.select(a.astype(np.float64), case.k)
    sets_ref = oracle.build_sets(anchors_ref, case.T)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    compare_sets(case.gpu_sets(), sets_ref)
    l = 1
    R_l = sets_ref.R[l]
    n = len(R_l)
    m = n - 37
    assert m > 0
    fresh = case.fresh(l, R_l)
    cut = tuple(t[:m].contiguous() for t in fresh)
    sentinel = 7.0
    out_big = torch.full((n, w.H, w.d), sentinel, dtype=case.q.dtype, device="cuda")
    lse_big = torch.full((n, w.H), sentinel, dtype=torch.float32, device="cuda")
    for mode, cm in (("union", relaxkv.CONTEXT_UNION), ("full", relaxkv.CONTEXT_FULL)):
        out_big.fill_(sentinel)
        lse_big.fill_(sentinel)
        case.req.sparse_attn(case.sets, l, *cut, out_big[:m], lse_big[:m], context_mode=cm)
        torch.cuda.synchronize()
        assert bool((out_big[m:] == sentinel).all()) and bool((lse_big[m:] == sentinel).all())
        counts, _ = case.sets.counts_to_host(check=False)
        assert counts[case.L + 1] & relaxkv.ERR_ROWS
        with pytest.raises(relaxkv.RelaxKVError) as e:
            case.sets.counts_to_host()
        assert e.value.status == relaxkv.EINVAL
        ts = sorted({0, m // 2, m - 1})
        O_ref, lse_ref = case.oracle_attn(l, sets_ref, fresh, mode=mode, targets=ts)
        assert_close(out_big[ts].float().cpu().numpy(), O_ref, w, f"O {mode} clamped",
                     rel_gate=1e-2 if w.dtype == "bf16" else None)
        assert_close(lse_big[ts].cpu().numpy(), lse_ref, w, f"lse {mode} clamped")
    # the cache update with the same short rows writes the first m rows only
    k_out, v_out = case.kc.clone(), case.vc.clone()
    case.req.update_cache(case.sets, l, cut[1], cut[2], k_out, v_out)
    torch.cuda.synchronize()
    short = oracle.Sets(**{**sets_ref.__dict__, "R": [r[:m] if i == l else r
                                                      for i, r in enumerate(sets_ref.R)]})
    kr, vr = oracle.update_cache(l, short, synth.to_f64(cut[1]), synth.to_f64(cut[2]),
                                 synth.to_f64(case.kc[l]), synth.to_f64(case.vc[l]))
    assert np.array_equal(synth.to_f64(k_out[l]), kr)
    assert np.array_equal(synth.to_f64(v_out[l]), vr)
    # the next selection clears the word; full-capacity calls then report nothing
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    case.req.build_sets(case.sets)
    out, lse = case.gpu_attn(l, fresh, n)
    case.req.update_cache(case.sets, l, fresh[1], fresh[2], k_out, v_out)
    counts, _ = case.sets.counts_to_host()
    assert counts[case.L + 1] == 0


def test_attention_tile_counters(gpu_lib):
    """The bf16 attention's larger launches take their tiles from per-layer, per-mode
    counters in the sets buffer (test_gpu_attn_counters.py); launches of this size map
    workgroups to tiles directly.  A set build zeroes every slot whatever the buffer
    held, these launches leave them zero, every target is computed exactly once (outputs
    against the oracle on every target), and repeated launches, interleaved across
    layers and modes on one stream, give the same bits."""
    w = SMALL["qwen-planted"]
    case = Case(w)
    a = synthetic_scores(case.L, case.T, seed=23)
    sets_ref = oracle.build_sets(oracle.select(a.astype(np.float64), case.k), case.T)
    case.sets.tiles.fill_(0x5A5A5A5A)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    compare_sets(case.gpu_sets(), sets_ref)
    assert case.sets.tiles.shape == (2, case.L, w.H_kv + 1)
    assert int(case.sets.tiles.abs().sum()) == 0
    layers = [0, 1, case.L - 1]
    fresh = {l: case.fresh(l, sets_ref.R[l]) for l in layers}
    first = {}
    for rep in range(3):
        for l in layers:
            for mode, cm in (("union", relaxkv.CONTEXT_UNION), ("full", relaxkv.CONTEXT_FULL)):
                n = len(sets_ref.R[l])
                out = torch.empty(n, w.H, w.d, dtype=case.q.dtype, device="cuda")
                lse = torch.empty(n, w.H, dtype=torch.float32, device="cuda")
                case.req.sparse_attn(case.sets, l, *fresh[l], out, lse, context_mode=cm)
                if rep == 0:
                    first[(l, mode)] = (out, lse)
                else:
                    o0, s0 = first[(l, mode)]
                    assert torch.equal(out, o0) and torch.equal(lse, s0), (rep, l, mode)
        torch.cuda.synchronize()
        assert int(case.sets.tiles.abs().sum()) == 0, rep
    for (l, mode), (out, lse) in first.items():
        O_ref, lse_ref = case.oracle_attn(l, sets_ref, fresh[l], mode=mode)
        assert_close(out.float().cpu().numpy(), O_ref, w, f"O {mode} layer {l}", rel_gate=1e-2)
        assert_close(lse.cpu().numpy(), lse_ref, w, f"lse {mode} layer {l}")


def test_attention_concurrent_layers_and_modes(gpu_lib):
    """Launches for different layers, and for the two context modes of one
    layer, may run at the same time (test_gpu_attn_counters.py has those that take
    their tiles from counters): four launches on four streams with no ordering between
    them give the bits of the same launches run one after another, and every slot is
    zero afterwards."""
    w = SMALL["qwen-planted"]
    case = Case(w)
    a = synthetic_scores(case.L, case.T, seed=29)
    sets_ref = oracle.build_sets(oracle.select(a.astype(np.float64), case.k), case.T)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    compare_sets(case.gpu_sets(), sets_ref)
    jobs = [(0, relaxkv.CONTEXT_UNION), (1, relaxkv.CONTEXT_UNION), (0, relaxkv.CONTEXT_FULL),
            (case.L - 1, relaxkv.CONTEXT_FULL)]
    fresh = {l: case.fresh(l, sets_ref.R[l]) for l, _ in jobs}

    def buffers():
        return {j: (torch.empty(len(sets_ref.R[j[0]]), w.H, w.d, dtype=case.q.dtype, device="cuda"),
                    torch.empty(len(sets_ref.R[j[0]]), w.H, dtype=torch.float32, device="cuda"))
                for j in jobs}

    seq = buffers()
    for (l, cm), (out, lse) in seq.items():
        case.req.sparse_attn(case.sets, l, *fresh[l], out, lse, context_mode=cm)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in jobs]
    for rep in range(3):
        con = buffers()
        torch.cuda.synchronize()
        for s, ((l, cm), (out, lse)) in zip(streams, con.items()):
            case.req.sparse_attn(case.sets, l, *fresh[l], out, lse, context_mode=cm, stream=s)
        torch.cuda.synchronize()
        for j in jobs:
            assert torch.equal(con[j][0], seq[j][0]) and torch.equal(con[j][1], seq[j][1]), (rep, j)
        assert int(case.sets.tiles.abs().sum()) == 0, rep
    for (l, cm), (out, lse) in seq.items():
        mode = "full" if cm == relaxkv.CONTEXT_FULL else "union"
        O_ref, lse_ref = case.oracle_attn(l, sets_ref, fresh[l], mode=mode)
        assert_close(out.float().cpu().numpy(), O_ref, w, f"O {mode} layer {l}", rel_gate=1e-2)
        assert_close(lse.cpu().numpy(), lse_ref, w, f"lse {mode} layer {l}")


def test_colsum_split_does_not_change_scores(gpu_lib):
    """The column-sum pass takes 512- to 8192-key splits, whichever needs the fewest
    key-steps per CU for the problem's size; a key's column sum does not depend
    on the split, and past 4096 keys the row statistics' split is fixed.  Layer 0 of an
    8K context is scored inside a 64-layer problem (8192-key splits) and alone
    (512-key splits): the same bits in both scoring modes, and within the bf16
    tolerance of the oracle."""
    w = synth.shrink(synth.WORKLOADS["llama8b-8k"], L=64)
    q, kc, vc = synth.make_cache(w, "cuda")
    g = torch.Generator(device="cuda").manual_seed(7)
    lse = (torch.randn(w.L, w.Qn, w.H, device="cuda", generator=g) * 0.1
           + math.log(w.T_c)).float()

    def scores(n_layers, q_lse):
        req = relaxkv.Request(q[:n_layers], kc[:n_layers], vc[:n_layers], w.ratio,
                              q_lse=None if q_lse is None else q_lse[:n_layers])
        a = torch.empty(n_layers, w.T_c, dtype=torch.float32, device="cuda")
        req.score(req.alloc_workspace(), a)
        torch.cuda.synchronize()
        return a[0].cpu()

    for q_lse in (None, lse):
        a_all, a_one = scores(w.L, q_lse), scores(1, q_lse)
        assert torch.equal(a_all, a_one), "one-pass" if q_lse is not None else "self-contained"
    a_ref, _, _ = oracle.score(synth.to_f64(q[:1]), synth.to_f64(kc[:1]))
    assert_close(scores(1, None).numpy(), a_ref[0], w, "layer 0 self-contained scores")


# The longest bf16 contexts: the slab bound at 8 KV heads of d 128, and the
# context-length bound itself (T_c = 2^22) at 2 KV heads.
MAX_SHAPES = {"slab": dict(T_c=(1 << 21) - 1, H=8, H_kv=8, ratio=1e-4),
              "context": dict(T_c=1 << 22, H=2, H_kv=2, ratio=5e-5)}


@pytest.mark.parametrize("shape", list(MAX_SHAPES))
def test_maximum_bf16_context(gpu_lib, shape):
    """The longest bf16 context the attention takes at 8 KV heads of d 128:
    T_c = 2^21 - 1, so one layer's cache slab is 2^31 - 1024 elements, just under
    the 32-bit element offsets of its fills (fresh rank x H_kv d and position x d).
    Two layers at a 1e-4 anchor ratio (210 anchors each): the scores of both layers
    against the oracle, selection and every set bit-exact on shared fp32 scores,
    and every target and head of both layers in both context modes checked by the
    softmax property (layer 1's union contexts read cached rows of layer-0 anchors
    anywhere in the 2M positions; the full prefix reads every cached row)."""
    w = synth.shrink(W["llama8b-8k"], L=2, Qn=2, **MAX_SHAPES[shape])
    case = Case(w)
    assert case.k == 210
    a_gpu = case.gpu_scores().cpu().numpy()
    a_ref = np.empty((w.L, w.T_c))
    for l in range(w.L):
        a_ref[l] = oracle.score(synth.to_f64(case.q[l:l + 1]), synth.to_f64(case.kc[l:l + 1]))[0][0]
    assert_close(a_gpu, a_ref, w, "scores")
    a32 = a_ref.astype(np.float32)
    anchors = case.gpu_select(torch.from_numpy(a32).cuda())
    anchors_ref = oracle.select(a32.astype(np.float64), case.k)
    assert np.array_equal(anchors, anchors_ref)
    sets_ref = oracle.build_sets(anchors_ref, case.T)
    compare_sets(case.gpu_sets(), sets_ref)
    for l in range(w.L):
        for mode in ("union", "full"):
            every_target_property(case, sets_ref, l, mode)


@pytest.mark.parametrize("shape", list(MAX_SHAPES))
def test_maximum_bf16_context_query_and_update(gpu_lib, shape):
    """At the same longest bf16 contexts (T_c = 2^21 - 1 at 8 KV heads, 2^22 at 2): the
    query-side completion of layer 0 against the oracle, and the cache update of
    layer 1 in place: the rows of R_1 take the fresh keys and values (at cached
    offsets up to the end of the slab) and every other row and layer keeps its bits."""
    from test_gpu_query_attn import oracle_query, run_query
    w = synth.shrink(W["llama8b-8k"], L=2, Qn=2, **MAX_SHAPES[shape])
    case = Case(w)
    kq, vq, out, lse = run_query(case, 0)
    O_ref, lse_ref = oracle_query(case, 0, kq, vq)
    assert_close(out.float().cpu().numpy(), O_ref, w, "query-side O", rel_gate=1e-2)
    assert_close(lse.cpu().numpy(), lse_ref, w, "query-side lse")
    del O_ref, lse_ref

    case.gpu_select(case.gpu_scores())
    got = case.gpu_sets()
    R_1 = got["R"][1]
    assert len(R_1) == case.k
    _, kn, vn = case.fresh(1, R_1)
    kc0, vc0 = case.kc.clone(), case.vc.clone()
    case.req.update_cache(case.sets, 1, kn, vn, case.kc, case.vc)
    torch.cuda.synchronize()
    idx = torch.as_tensor(R_1, dtype=torch.int64, device="cuda")
    assert torch.equal(case.kc[1].index_select(1, idx), kn.transpose(0, 1))
    assert torch.equal(case.vc[1].index_select(1, idx), vn.transpose(0, 1))
    keep = torch.ones(w.T_c, dtype=torch.bool, device="cuda")
    keep[idx] = False
    for new, old in ((case.kc, kc0), (case.vc, vc0)):
        assert torch.equal(new[0], old[0])
        assert torch.equal(new[1][:, keep], old[1][:, keep])
    assert int(R_1.max()) > w.T_c // 2              # rows in the upper half of the slab were written
