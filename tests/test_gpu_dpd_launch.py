"""The pair forces and the real-space term in one launch or in two (GPU).

A step launches them together; a step whose kernels are timed launches them one
by one.  Both evaluate the same sums of the same rounded terms, so trajectories
are bitwise equal: with few charges (fewer real-space work items than blocks),
with all particles charged, on the smallest grids and on larger ones.
"""
import numpy as np
import pytest

from test_gpu_dpd import _gpu, _system, _t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,nq", [(6.5, 2), (6.5, 800), (9.0, 400), (13.0, 6400)])
def test_one_launch_or_two(L, nq, precision):
    import torch
    pos, vel, q, bonds = _system(L=L, nq=nq)
    runs = []
    for mode in ("graph", "eager", "timed"):
        d = _gpu(L, q, bonds, precision=precision)
        p, v, f = _t(pos), _t(vel), torch.empty(pos.shape, dtype=torch.float64, device="cuda")
        if mode == "eager":
            d.set_graphs(False)
        d.forces(p, v, f)
        if mode == "timed":
            d.time_kernel("dpd_pair", 64)
        d.run(p, v, f, 1, 11)
        torch.cuda.synchronize()
        assert d.status() == 0
        runs.append([x.cpu().numpy() for x in (p, v, f)] + [torch.as_tensor(d.energy()).cpu().numpy()])
        d.close()
    for r in runs[1:]:
        for a, b in zip(runs[0], r):
            assert np.array_equal(a, b)
