"""Set building with the largest blocks of positions (16384) and more than 64 of them,
the union and the target list dense, so that the blocks' sums reach their maxima:
the anchor union's sets against the oracle, and a global list's against the same
definitions in numpy (the oracle counts each target's limit by a pass over the union)."""

import numpy as np
import pytest
import torch

import oracle
from test_gpu_set_blocks import Lists

pytestmark = pytest.mark.gpu


def check(case, U, h, cidx, R, R_u):
    """The sets on the device: one list R (limits R_u) per layer, bit for bit."""
    s, L, T = case.sets, case.L, case.T
    counts, edges = s.counts_to_host()
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()   # noqa: E731
    off = np.concatenate([[0], np.cumsum([len(r) for r in R])])
    assert counts == [len(U)] + [len(r) for r in R] + [0]
    assert torch.equal(s.R_off, dev(off))
    assert torch.equal(s.U[:len(U)], dev(U)) and torch.equal(s.cidx, dev(cidx)) and torch.equal(s.h, dev(h))
    for l in range(L):
        rank = np.full(T, -1, dtype=np.int32)
        rank[R[l]] = np.arange(len(R[l]))
        assert torch.equal(s.R_idx[off[l]:off[l + 1]], dev(R[l])), l
        assert torch.equal(s.R_u[off[l]:off[l + 1]], dev(R_u[l])), l
        assert torch.equal(s.rank[l], dev(rank)), l
        assert torch.equal(s.src[l, :len(U)], dev(rank[U])), l
        assert edges[l] == int((np.asarray(R_u[l]) + 1).sum())
        assert edges[L + l] == int((np.asarray(R[l]) + 1).sum())


@pytest.mark.parametrize("L,T,ratio", [(2, (1 << 20) + 1, 0.9), (1, (1 << 20) + 16385, 0.3), (2, 1 << 22, 1.0),
                                       (97, (1 << 19) + 1, 0.3), (193, (1 << 19) + 1, 0.3)])
def test_largest_set_blocks(gpu_lib, L, T, ratio):
    case = Lists(L, T, ratio)
    rng = np.random.default_rng(T)
    anchors = np.stack([np.sort(rng.permutation(T)[:case.k]) for _ in range(L)])
    case.sets.anchors.copy_(torch.from_numpy(anchors.astype(np.int32)))
    case.sets.counts[-1] = 0                           # (the selection clears it)
    case.req.build_sets(case.sets)
    ref = oracle.build_sets(anchors, T)
    check(case, ref.U, ref.h, ref.cidx, ref.R, ref.R_u)
    for P in (np.arange(T), np.sort(rng.permutation(T)[:T // 3])):
        h = np.full(T, -1)
        h[P] = L - 1
        t = torch.zeros(T, dtype=torch.int32, device="cuda")
        t[:len(P)] = torch.from_numpy(P.astype(np.int32))
        case.req.build_sets_global(case.sets, t, torch.tensor([len(P)], dtype=torch.int32, device="cuda"))
        check(case, ref.U, h, ref.cidx, [P] * L, [np.searchsorted(ref.U, P, side="right") - 1] * L)
