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
