"""What a set build does to lists it is not asked to write: the union and global
builds leave the context lists and layer means of an earlier construction as they
are, so every one of those lists can be a target list in turn."""

import numpy as np
import pytest
import torch

import oracle
from harness import synthetic_scores
from paper_2609_33503_amd import relaxkv
from test_gpu_matched_targets import compare_global_sets
from test_gpu_set_blocks import Lists

pytestmark = pytest.mark.gpu


# 200: one block of positions; 300 and 9000: several
@pytest.mark.parametrize("L,T", [(1, 200), (1, 5000), (2, 300), (3, 9000), (5, 257)])
def test_union_builds_leave_the_context_lists(gpu_lib, L, T):
    case = Lists(L, T, 0.1)
    sets = case.sets
    a = torch.from_numpy(synthetic_scores(L, T, seed=T, levels=91)).cuda()
    case.req.select(a, sets)
    case.req.build_sets_context(a, relaxkv.CONTEXT_SETS_GLOBAL, sets)
    case.req.build_sets_context(a, relaxkv.CONTEXT_SETS_LAYERWISE, sets)
    n_u = int(sets.counts[0])
    ctx, g = sets.ctx.clone(), sets.g.clone()
    anchors = sets.anchors.cpu().numpy().astype(np.int64)
    out = torch.arange(T, dtype=torch.int32, device="cuda")
    n = torch.tensor([n_u], dtype=torch.int32, device="cuda")

    def check(targets, count):
        P = targets[:count].cpu().numpy().astype(np.int64)
        case.req.build_sets_global(sets, targets, torch.full_like(n, count))
        compare_global_sets(case.got(), oracle.build_sets_global(anchors, T, P))
        assert torch.equal(sets.ctx, ctx) and torch.equal(sets.g, g)

    case.req.build_sets(sets)
    assert torch.equal(sets.ctx, ctx) and torch.equal(sets.g, g)
    check(out, T)
    for l in list(range(L)) + [0]:
        check(sets.ctx[l], n_u)
    if L > 1:                                          # a list that begins inside a row
        check(sets.ctx.view(-1)[5:5 + T], n_u - 5)


@pytest.mark.parametrize("L,T", [(1, 200), (2, 700), (3, 9000)])
def test_targets_in_an_array_the_build_writes(gpu_lib, L, T):
    """The union list as the target list, right after a new selection (U and its
    count still those of the old anchors): the build rebuilds the union first.  R_0
    in R_idx, with its count, is the same list."""
    case = Lists(L, T, 0.1)
    sets = case.sets
    for seed in (1, 2):                                # the second time U is a stale list
        a = synthetic_scores(L, T, seed=seed, levels=91)
        anchors = oracle.select(a.astype(np.float64), case.k)
        case.req.select(torch.from_numpy(a).cuda(), sets)
        if seed == 1:
            case.req.build_sets(sets)
    U = oracle.build_sets(anchors, T).U
    ref = oracle.build_sets_global(anchors, T, U)
    case.req.build_sets_global(sets, sets.U, sets.counts[:1])
    compare_global_sets(case.got(), ref)
    case.req.build_sets(sets)
    case.req.build_sets_global(sets, sets.R_idx[:T], sets.counts[1:2])
    compare_global_sets(case.got(), ref)
    # a count from the sets, a list from elsewhere, and the other way round
    P = torch.zeros(T, dtype=torch.int32, device="cuda")
    P[:len(U)] = torch.from_numpy(np.asarray(U, dtype=np.int32)).cuda()
    case.req.build_sets_global(sets, P, sets.counts[:1])
    compare_global_sets(case.got(), ref)
    case.req.build_sets_global(sets, sets.U, torch.tensor([3], dtype=torch.int32, device="cuda"))
    compare_global_sets(case.got(), oracle.build_sets_global(anchors, T, U[:3]))
