"""Anchor selection at the edges of its register tiles: row lengths around every
tile size of the top-k kernel (1024-entry multiples) and past the last one, where
rows are streamed from memory.  Bit-exact against the oracle on scores with many
exact ties and signed zeros, for a single anchor, a fraction and the whole row."""

import numpy as np
import pytest
import torch

import oracle
from harness import synthetic_scores
from paper_2609_33503_amd import relaxkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 63, 64, 65, 1023, 1025, 2048, 2049, 8192, 8193, 16384, 16385,
                               32768, 32769, 49152, 49153])
def test_select_row_lengths(gpu_lib, T):
    L = 3
    z = torch.zeros(L, 1, T, 64, dtype=torch.bfloat16, device="cuda")
    q = torch.zeros(L, 1, 1, 64, dtype=torch.bfloat16, device="cuda")
    a = synthetic_scores(L, T, seed=T, levels=37)
    a[1] = np.float32(0.5)                         # one value only: the tie rule decides
    a[2] -= np.float32(0.4)                        # both signs
    for ratio in (0.0, 0.3, 1.0):
        req = relaxkv.Request(q, z, z, ratio)
        sets = req.alloc_sets()
        sets.counts[-1] = 7                        # cleared by the selection
        req.select(torch.from_numpy(a).cuda(), sets)
        assert np.array_equal(sets.anchors.cpu().numpy(),
                              oracle.select(a.astype(np.float64), req.k)), (T, ratio)
        assert int(sets.counts[-1]) == 0
    b = a.copy()
    b[2, T // 2] = np.nan                          # sets the error word, indices stay in range
    req.select(torch.from_numpy(b).cuda(), sets)
    assert int(sets.counts[-1]) == relaxkv.ERR_NAN_SCORE
    got = sets.anchors.cpu().numpy()
    assert got.min() >= 0 and got.max() < T
