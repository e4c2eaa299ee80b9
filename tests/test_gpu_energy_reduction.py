"""Energies reduced by the combine kernel's last work-group or by a launch (GPU).

Up to 256 work-groups of 256 particles the last one reduces the partials, beyond
that a launch of its own does; the order of additions is the same.  Both sides of
the line, one work-group and a ragged last one: repeated evaluations on one plan
give the same bits (the count of finished work-groups is back at zero), and the
energies are the oracle's k-space and pair sums to the accuracy of the mesh.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 256, 257, 65536, 65537])
def test_last_work_group_reduces_the_energies(n):
    import torch

    from paper_1303_4523_amd import Plan
    L, alpha, Kc, r_cut, lam = 8.0, 0.6, 8, 2.0, 0.25
    rng = np.random.Generator(np.random.PCG64(n))
    pos = rng.uniform(0.0, L, size=(n, 3))
    q = np.zeros(n)
    m = min(n // 2, 200)          # charges in the first and the last work-groups
    q[:m] = 1.0
    q[n - m:] = -1.0
    ref = oracle.ewald(pos, q, L, alpha, Kc, r_cut, lam)
    plan = Plan(n, L, alpha, 8, 2.0, 32, Kc, r_cut, lam, device=0)
    tp, tq = torch.tensor(pos, device="cuda"), torch.tensor(q, device="cuda")
    runs = []
    for _ in range(5):
        F, E = plan.compute_components(tp, tq)
        runs.append(E.cpu().numpy().copy())
    assert plan.status() == 0
    plan.close()
    for E in runs[1:]:
        assert np.array_equal(E, runs[0])
    scale = sum(abs(ref[k]) for k in ("E_real", "E_recip", "E_self")) + 1e-300
    for k, name in ((0, "E_real"), (1, "E_slater"), (2, "E_recip"), (3, "E_self")):
        assert abs(runs[0][k] - ref[name]) <= 1e-8 * scale
