"""Set building at the edges of its position blocks (256 positions up to 64 blocks,
then larger ones), for one layer up to the most layers, against the oracle, bit
for bit: the anchor union, a global target list and the per-layer contexts (whose
compact limits come from a bitmap up to 2^18 positions and a search past them)."""

import numpy as np
import pytest
import torch

import oracle
from harness import compare_sets, synthetic_scores
from paper_2609_33503_amd import relaxkv
from test_gpu_context_variants import build_both, compare_context_sets
from test_gpu_matched_targets import compare_global_sets, gpu_global_sets

pytestmark = pytest.mark.gpu


class Lists:
    """A request of L layers and T positions with its sets (no keys to speak of)."""

    def __init__(self, L, T, ratio):
        z = torch.zeros(L, 1, T, 64, dtype=torch.bfloat16, device="cuda")
        q = torch.zeros(L, 1, 1, 64, dtype=torch.bfloat16, device="cuda")
        self.L, self.T = L, T
        self.req = relaxkv.Request(q, z, z, ratio)
        self.k = self.req.k
        self.sets = self.req.alloc_sets()
        self.sets.buf.fill_(0x5A)                      # nothing relies on cleared memory

    def got(self):
        s, L = self.sets, self.L
        counts, edges = s.counts_to_host()
        off, idx, ru = (t.cpu().numpy() for t in (s.R_off, s.R_idx, s.R_u))
        nU = counts[0]
        return dict(counts=counts, edges=edges, h=s.h.cpu().numpy(), U=s.U.cpu().numpy()[:nU],
                    cidx=s.cidx.cpu().numpy(), R=[idx[off[l]:off[l + 1]] for l in range(L)],
                    R_u=[ru[off[l]:off[l + 1]] for l in range(L)],
                    src=[r[:nU] for r in s.src.cpu().numpy()], rank=s.rank.cpu().numpy())


@pytest.mark.parametrize("L,T", [(1, 1), (3, 2), (1, 255), (2, 256), (1, 257), (65, 300), (1024, 70),
                                 (2, 16384), (1, 16385), (5, 32769), (2, 131073)])
def test_set_blocks(gpu_lib, L, T):
    case = Lists(L, T, 0.1)
    a = synthetic_scores(L, T, seed=L + T, levels=53)
    anchors = oracle.select(a.astype(np.float64), case.k)
    case.req.select(torch.from_numpy(a).cuda(), case.sets)
    case.req.build_sets(case.sets)
    compare_sets(case.got(), oracle.build_sets(anchors, T))
    assert int(case.sets.tiles.abs().sum()) == 0
    rng = np.random.default_rng(T)
    for P in (np.sort(rng.choice(T, size=(T + 2) // 3, replace=False)), np.arange(T),
              np.zeros(0, dtype=np.int64)):
        compare_global_sets(gpu_global_sets(case, P), oracle.build_sets_global(anchors, T, P))


# around the layer counts where the blocks are counted by h and several layers are
# searched at a time
@pytest.mark.parametrize("L,T", [(96, 300), (97, 256), (97, 16385), (192, 700), (193, 2000), (321, 5000)])
def test_set_blocks_many_layers(gpu_lib, L, T):
    test_set_blocks(gpu_lib, L, T)


@pytest.mark.parametrize("T", [31, 33, 1025, 1 << 18, (1 << 18) + 1])
@pytest.mark.parametrize("construction", ["global", "layerwise"])
def test_context_limits(gpu_lib, T, construction):
    case = Lists(2, T, 0.05)
    a = synthetic_scores(2, T, seed=T, levels=91)
    _, ref = build_both(case, a, construction)
    compare_context_sets(case, ref, construction)


@pytest.mark.parametrize("L,T", [(1, 200), (1, 5000), (2, 300), (3, 9000)])
@pytest.mark.parametrize("row", [0, -1])
def test_targets_from_a_context_row(gpu_lib, L, T, row):
    """A target list that is a row of the sets' own context lists: the build does
    not use that row as scratch, so it gives the sets of a copy of the list, twice."""
    case = Lists(L, T, 0.1)
    a = torch.from_numpy(synthetic_scores(L, T, seed=T, levels=91)).cuda()
    case.req.select(a, case.sets)
    case.req.build_sets_context(a, relaxkv.CONTEXT_SETS_LAYERWISE, case.sets)
    n = case.sets.counts[:1]
    P = case.sets.ctx[row, :int(n)].cpu().numpy().astype(np.int64)
    ref = oracle.build_sets_global(case.sets.anchors.cpu().numpy().astype(np.int64), T, P)
    for _ in range(2):
        case.req.build_sets_global(case.sets, case.sets.ctx[row], n)
        got = case.got()
        assert [r.tolist() for r in got["R"]] == [P.tolist()] * L
        for l in range(L):
            assert got["R_u"][l].tolist() == ref.R_u[l].tolist()
            assert got["src"][l].tolist() == ref.src[l].tolist()
            assert got["edges"][l] == int(ref.edges[l])
