"""The real-space kernel's routes against the oracle's pair sum (GPU).

Grids of 2 cells per side (every candidate to the exact test), of 3 (each cell
once among the 27), cells with more charges than a block's share and more
candidates than a stage (windows), sparse systems (an item per charge), and the
four ranges of alpha r_cut of the pair function, for point and smeared charges.
The window half-width p = 8 keeps the mesh's error below 1e-12, so forces and
energies agree to the fixed point (2^-36 per pair term, at most a few thousand
terms per charge): 1e-8 of the force and energy scales.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# L, r_cut, charges, alpha, lambda
CASES = [
    (4.0, 2.0, 60, 0.4, 0.25),       # 2 cells per side
    (5.9, 2.0, 401, 0.45, 0.25),     # 2 cells per side, 50 charges per cell, windows
    (6.0, 2.0, 1, 0.45, 0.25),       # 3 cells per side (edge = r_cut), a single +- pair
    (6.3, 2.0, 4801, 0.45, 0.0),     # 178 charges per cell: shares and 13 windows
    (9.0, 1.2, 640, 0.8, 0.25),      # 7 cells per side, 2 charges per cell: segments
    (18.0, 0.9, 90, 0.5, 0.25),      # 20 cells per side: an item per charge
    (6.0, 2.0, 500, 1.3, 0.889),     # alpha r_cut = 2.6: second range
    (6.0, 2.0, 500, 1.75, 0.25),     # 3.5: third range
    (6.0, 2.0, 500, 2.4, 0.889),     # 4.8: beyond the polynomials
    (6.0, 2.0, 500, 2.4, 0.0),
]


@pytest.mark.parametrize("L,r_cut,n,alpha,lam", CASES)
def test_real_space_routes(L, r_cut, n, alpha, lam):
    import torch

    from paper_1303_4523_amd import Plan
    rng = np.random.Generator(np.random.PCG64(n))
    n += n % 2
    pos = rng.uniform(0.0, L, size=(n, 3))
    if n == 2:
        pos[1] = (pos[0] + [0.0, 0.0, 1.9]) % L
    q = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    ref = oracle.ewald(pos, q, L, alpha, 8, r_cut, lam)
    plan = Plan(n, L, alpha, 8, 2.0, 32, 8, r_cut, lam, device=0)
    F, E = plan.compute_components(torch.tensor(pos, device="cuda"), torch.tensor(q, device="cuda"))
    F, E = F.cpu().numpy(), E.cpu().numpy()
    assert plan.status() == 0
    plan.close()
    assert np.linalg.norm(F - ref["F"]) <= 1e-8 * np.linalg.norm(ref["F"])
    scale = sum(abs(ref[k]) for k in ("E_real", "E_recip", "E_self"))
    assert abs(E[0] - ref["E_real"]) <= 1e-8 * scale
    assert abs(E[1] - ref["E_slater"]) <= 1e-8 * scale


@pytest.mark.parametrize("q0", [1.0, 30.0, 100.0])
def test_real_space_terms_left_to_the_library(q0):
    """Charges so large that few (1), many (30) or all (100) of a block's pairs
    are left to the second evaluation, more than its list holds among them."""
    import torch

    from paper_1303_4523_amd import Plan
    L, r_cut, alpha, lam, n = 5.9, 2.0, 0.45, 0.25, 402
    rng = np.random.Generator(np.random.PCG64(7))
    pos = rng.uniform(0.0, L, size=(n, 3))
    q = q0 * np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    ref = oracle.ewald(pos, q, L, alpha, 8, r_cut, lam)
    plan = Plan(n, L, alpha, 8, 2.0, 32, 8, r_cut, lam, device=0)
    F, E = plan.compute_components(torch.tensor(pos, device="cuda"), torch.tensor(q, device="cuda"))
    F, E = F.cpu().numpy(), E.cpu().numpy()
    assert plan.status() == 0
    plan.close()
    assert np.linalg.norm(F - ref["F"]) <= 1e-8 * np.linalg.norm(ref["F"])
    assert abs(E[0] - ref["E_real"]) <= 1e-8 * sum(abs(ref[k]) for k in ("E_real", "E_recip", "E_self"))
