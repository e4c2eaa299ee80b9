"""The mesh passes of half-width 4 against the NumPy model of the NFFT (GPU).

A plane's charges take 4, 2 or 1 lanes each, by how many there are, in batches
of at most 512; stencils reach past the mesh on both sides of z and y; meshes of
one and of several radices, of 16 (the smallest for this half-width) to 64.  The
model evaluates the window itself, the kernels series fitted to 4e-15 of its
maximum (FP64; 1e-12 for its derivative) or to 1e-8 in FP32 arithmetic (mixed).
The tolerances leave room for the 512 stencil points, the transforms and the
fixed point: 1e-10 of the energy and 1e-9 of the forces, 1e-5 in mixed.
"""
import numpy as np
import pytest

import oracle
from oracle import nfft_mirror as nm

pytestmark = pytest.mark.gpu

# M, Kc, charges
CASES = [
    (32, 8, 2),       # most planes empty
    (32, 8, 1000),    # 63 per work-group: 4 lanes per charge
    (32, 8, 3000),    # 188: 2 lanes
    (32, 8, 5000),    # 313: 1 lane
    (32, 8, 9000),    # 563: two batches
    (16, 4, 300),     # smallest mesh, many parts
    (54, 13, 2000),   # radices 2 and 3
    (60, 14, 400),    # 3, 4 and 5
    (64, 15, 2600),   # 8 and 8
]


def _model(pos, q, L, alpha, Kc, M, ik):
    win = nm.Window("kb", 4, 2.0)
    if not ik:
        r = nm.recip_nfft(pos, q, L, alpha, Kc, M, win)
        return r["E"], r["F"]
    G = np.fft.fftn(nm.spread(pos, q, L, M, win))
    c = nm.influence(L, M, alpha, Kc, win)
    E = float((c * np.abs(G) ** 2).sum() / (2.0 * np.pi * L))
    k = np.fft.fftfreq(M, 1.0 / M)
    F = np.zeros((len(q), 3))
    for t in range(3):
        kt = k.reshape([-1 if a == t else 1 for a in range(3)])
        h = np.real(np.fft.ifftn(1j * kt * c * G)) * M ** 3
        for j in range(len(q)):
            base, offs = nm.stencil(pos[j], L, M, 4)
            i = [(base[a] + np.arange(8)) % M for a in range(3)]
            w = [win.phi(offs[a]) for a in range(3)]
            F[j, t] = -2.0 * q[j] / L ** 2 * np.einsum("abc,a,b,c", h[np.ix_(*i)], *w)
    return E, F


@pytest.mark.parametrize("ik", [False, True])
@pytest.mark.parametrize("M,Kc,n", CASES)
def test_half_width_4_routes(M, Kc, n, ik):
    import torch

    from paper_1303_4523_amd import Plan
    L, r_cut, lam = 9.0, 1.5, 0.25
    alpha = 0.6
    rng = np.random.Generator(np.random.PCG64(M * n))
    pos = rng.uniform(0.0, L, size=(n, 3))
    # at the edges of the box along y and z
    m = min(n // 2, 40)
    pos[:m, 1:] = (pos[:m, 1:] / L - 0.5) * 1e-3 * L % L
    q = np.where(np.arange(n) % 2 == 0, 1.0, -1.0) * rng.uniform(0.5, 1.5)
    E, F = _model(pos, q, L, alpha, Kc, M, ik)
    F_real = oracle.ewald(pos, q, L, alpha, 2, r_cut, lam)["F_real"]
    for precision, tol_e, tol_f in (("fp64", 1e-10, 1e-9), ("mixed", 1e-5, 1e-5)):
        plan = Plan(n, L, alpha, 4, 2.0, M, Kc, r_cut, lam, precision=precision, device=0)
        if ik:
            plan.set_force_mode("ik")
        Fg, Eg = plan.compute_components(torch.tensor(pos, device="cuda"), torch.tensor(q, device="cuda"))
        Fg, Eg = Fg.cpu().numpy(), Eg.cpu().numpy()
        assert plan.status() == 0
        plan.close()
        assert abs(Eg[2] - E) <= tol_e * abs(E)
        scale = np.linalg.norm(F) + np.linalg.norm(F_real) * 1e-3
        assert np.linalg.norm(Fg - F_real - F) <= tol_f * scale
