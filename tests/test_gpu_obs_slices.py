"""The pair histogram's work-groups by tile pair and slice of a tile (GPU).

1 to 8 slices, ragged last tiles, positions outside the box (several periods
away), bin edges met exactly, a single bin and bins of few counts: the counts
equal the oracle's exactly.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsel,nbins", [(2, 7), (255, 1), (256, 100), (257, 100), (2900, 300), (4000, 100),
                                        (5700, 50), (8192, 100)])
def test_pair_histogram_slices(nsel, nbins):
    import torch

    from paper_1303_4523_amd.observables import PairHistogram
    rng = np.random.Generator(np.random.PCG64(nsel))
    L = 9.3
    pos = rng.uniform(-2.0 * L, 3.0 * L, size=(nsel + 5, 3))
    m = nsel // 4
    pos[:m] = np.round(pos[:m] / (L / 16)) * (L / 16)   # distances on bin edges and at L / 2
    sel = rng.permutation(nsel + 5)[:nsel]
    cls = rng.integers(0, 3, size=nsel).astype(np.int32)
    ref = oracle.pair_histogram(pos, sel, cls, 3, L, L / 2, nbins)
    H = PairHistogram(len(pos), sel, cls, 3, L, L / 2, nbins, device=0)
    H.sample(torch.tensor(pos, device="cuda"))
    assert np.array_equal(H.counts(), ref)
