"""Performance cases of the library: what a program that uses it has it do.

Five kinds of work, each through the package's public classes:

* ``eval``  -- one ENUF evaluation (``Plan.compute`` or
  ``Plan.compute_components``) of a configuration: energy and forces;
* ``dpd``   -- a run of one DPD system (``DPD.run``), the state advanced in
  place, its step graphs captured beforehand;
* ``rdf``   -- the radial-distribution study: a run between two samples and
  the sample (``PairHistogram.sample``) itself;
* ``batch`` -- uneven replicas stepped together (``Batch.run``), replayed from
  the batch's graphs, with the chains' radii of gyration sampled at the end;
* ``serve`` -- densely charged systems of a request stream stepped together
  for the few steps between two membership changes (eager launches).

Systems have density 3 or 4 in a periodic cube; ENUF parameters are those of
the repository's workloads (alpha = 0.3, r_cut = 3, p = 4, M ~ 3.2 L) or the
ones its accuracy rule chooses.  ``exact`` restates the method in plain torch
FP64: the truncated Ewald sum over every |k| < Kc, minimum-image pairs, and
the DPD step with its counter-based random numbers.
"""
import math

import numpy as np
import torch

from paper_1303_4523_amd import Plan
from paper_1303_4523_amd import params
from paper_1303_4523_amd import workloads as wl
from paper_1303_4523_amd.batch import Batch
from paper_1303_4523_amd.dpd import DPD
from paper_1303_4523_amd.observables import PairHistogram, chain_rg2

DEVICE = "cuda"


def listed():
    return [
        # the smallest call: one evaluation of 300 charges, bound by launches and latency
        dict(name="eval_small_fp64", kind="eval", n=3000, charged=0.1, valency=1, precision="fp64", mode="gradient",
             delta=0.0, components=False),
        # an ordinary electrolyte, default precision, power-of-two mesh (M = 64)
        dict(name="eval_mid_fp64", kind="eval", n=24000, charged=0.1, valency=1, precision="fp64", mode="gradient",
             delta=0.0, components=False),
        # the largest of the N sweep (L = 40, M = 128) in either precision
        dict(name="eval_large_fp64", kind="eval", n=192000, charged=0.1, valency=1, precision="fp64",
             mode="gradient", delta=0.0, components=False),
        dict(name="eval_large_mixed", kind="eval", n=192000, charged=0.1, valency=1, precision="mixed",
             mode="gradient", delta=0.0, components=False),
        # a serving request evaluated alone: odd size, most beads charged, ragged mesh, energy components
        dict(name="eval_dense_mixed", kind="eval", n=60001, charged=0.7, valency=2, precision="mixed",
             mode="gradient", delta=0.0, components=True),
        # every bead charged, parameters from the accuracy rule, momentum-conserving forces
        dict(name="eval_ik_fp64", kind="eval", n=4000, charged=1.0, valency=1, precision="fp64", mode="ik",
             delta=1e-4, components=True),
        # the headline trajectory: polyelectrolyte and salt, FP64
        dict(name="dpd_24k_fp64", kind="dpd", n=24000, fraction=0.5, valency=1, precision="fp64", steps=20),
        # a small trajectory in the mixed mode, odd step count
        dict(name="dpd_small_mixed", kind="dpd", n=3333, fraction=0.25, valency=3, precision="mixed", steps=11),
        # the g(r) study's loop body: the steps between two samples, then the pair histogram
        dict(name="rdf_set3_fp64", kind="rdf", n=4000, precision="fp64", steps=25),
        # 64 uneven replicas, replayed steps
        dict(name="batch_64_mixed", kind="batch", members=64, n_min=3000, n_max=48000, precision="mixed", steps=6),
        # a few replicas in FP64
        dict(name="batch_8_fp64", kind="batch", members=8, n_min=3000, n_max=48000, precision="fp64", steps=6),
        # 16 requests of the serving stream between two membership changes
        dict(name="serve_16_mixed", kind="serve", members=16, n_min=3000, n_max=200000, precision="mixed", steps=2),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes log-uniform over each kind's range, every
    precision, force mode, charge fraction and valency."""
    kind = rng.choice(("eval", "eval", "eval", "dpd", "rdf", "batch", "serve"))
    precision = rng.choice(("fp64", "mixed"))
    if kind == "eval":
        delta = rng.choice((0.0, 0.0, 1e-3, 1e-4))
        charged = rng.choice((0.1, rng.uniform(0.05, 1.0)))
        # the charges of the largest listed evaluations bound the drawn ones
        n_max = 192000 if charged <= 0.1 else 48000
        return dict(kind=kind, n=_log_uniform(rng, 1000, n_max if delta == 0.0 else 12000), charged=charged,
                    valency=rng.choice((1, 2, 3)), precision=precision,
                    mode=rng.choice(("gradient", "gradient", "gradient", "ik")), delta=delta,
                    components=rng.random() < 0.5)
    if kind == "dpd":
        return dict(kind=kind, n=_log_uniform(rng, 1000, 48000), fraction=rng.choice((0.1, 0.25, 0.5, 1.0)),
                    valency=rng.choice((1, 2, 3)), precision=precision, steps=rng.randint(1, 24))
    if kind == "rdf":
        return dict(kind=kind, n=_log_uniform(rng, 1200, 12000), precision=precision, steps=rng.randint(5, 25))
    if kind == "batch":
        return dict(kind=kind, members=rng.randint(2, 40), n_min=rng.randint(1500, 6000),
                    n_max=rng.randint(12000, 48000), precision=precision, steps=rng.randint(1, 6))
    return dict(kind=kind, members=rng.randint(1, 10), n_min=rng.randint(1500, 6000),
                n_max=rng.randint(20000, 120000), precision=precision, steps=rng.randint(1, 2))


# ---------------------------------------------------------------------------
# Systems (seeded; the generators of the repository's workloads)
# ---------------------------------------------------------------------------
def _electrolyte(n, charged, valency, seed, velocities=False):
    L = (n / 3.0) ** (1.0 / 3.0)
    cat = int(round(charged * n / (1 + valency)))
    return wl.electrolyte(L, n, cat, valency * cat, seed, z_plus=float(valency), with_velocities=velocities)


def _mesh(L):
    """The workloads' mesh for a box of edge L: M ~ 3.2 L, Kc = M / 4 at most."""
    M = wl.mesh_size(3.2 * L)
    return wl.enuf_params(L, M=M, Kc=min(int(math.floor(0.8 * L + 1e-9)), M // 4))


def _eval_enuf(case, L):
    if case["delta"] > 0.0:
        return params.choose(L, delta=case["delta"], r_cut=3.0)
    return _mesh(L)


def _chain_system(n, fraction, valency, seed):
    L = (n / 3.0) ** (1.0 / 3.0)
    s = wl.polyelectrolyte(L, 3.0, 50, fraction, 0.1, valency, seed)
    s.meta["enuf"] = _mesh(L)
    s.meta["dpd"] = dict(wl.DPD_DEFAULTS, L=L, seed=seed)
    return s


def _systems(case, seed):
    """The systems of a dpd, rdf, batch or serve case."""
    kind = case["kind"]
    if kind == "dpd":
        return [_chain_system(case["n"], case["fraction"], case["valency"], 1000 + seed)]
    if kind == "rdf":
        L = (case["n"] / 4.0) ** (1.0 / 3.0)
        s = wl.electrolyte_set3(seed=1000 + seed, L=L, n_pairs=int(round(0.033 * case["n"])))
        s.meta["enuf"] = params.choose(L, delta=1e-4, r_cut=wl.PAPER_R_CUT, lam=wl.PAPER_LAMBDA_E)
        return [s]
    # sizes log-uniform between the bounds, the same for every seed of a case
    sizes = np.random.Generator(np.random.PCG64(case["members"]))
    out = []
    for m in range(case["members"]):
        n = int(round(math.exp(sizes.uniform(math.log(case["n_min"]), math.log(case["n_max"])))))
        sm = 1000 * (1 + seed) + m
        if kind == "batch":
            s = _chain_system(n, (0.1, 0.25, 0.5, 1.0)[m % 4], (1, 2, 3)[(m // 4) % 3], sm)
        else:
            s = _electrolyte(n, sizes.uniform(0.05, 1.0), int(sizes.integers(1, 4)), sm, velocities=True)
            s.meta["enuf"] = _mesh(s.L)
            s.meta["dpd"] = dict(wl.DPD_DEFAULTS, L=s.L, seed=sm)
        out.append(s)
    return out


# ---------------------------------------------------------------------------
# What a program has in hand before the call
# ---------------------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] == "eval":
        s = _electrolyte(case["n"], case["charged"], case["valency"], 1000 + seed)
        e = _eval_enuf(case, s.L)
        plan = Plan(s.N, s.L, e["alpha"], e["p"], e["sigma"], e["M"], e["Kc"], e["r_cut"], e["lam"],
                    precision=case["precision"])
        if case["mode"] == "ik":
            plan.set_force_mode("ik")
        return dict(case=case, plan=plan, pos=torch.tensor(s.pos, device=DEVICE), q=torch.tensor(s.q, device=DEVICE))
    systems = _systems(case, seed)
    # one allocation for the state of all systems, a slice per system
    pos = torch.tensor(np.concatenate([s.pos for s in systems]), device=DEVICE)
    vel = torch.tensor(np.concatenate([s.vel for s in systems]), device=DEVICE)
    force = torch.empty_like(pos)
    members, lo = [], 0
    for s in systems:
        d = DPD(s.L, s.q, s.meta["dpd"], bonds=s.bonds, enuf=s.meta["enuf"], precision=case["precision"])
        if case["kind"] in ("batch", "serve"):
            d.plan.set_parts(1)   # the batch fills the device
        m = (d, pos[lo:lo + s.N], vel[lo:lo + s.N], force[lo:lo + s.N])
        d.forces(*m[1:], step=0)
        members.append(m)
        lo += s.N
    state = dict(case=case, members=members, pos=pos, vel=vel, force=force, step=1)
    if case["kind"] in ("dpd", "rdf"):
        members[0][0].prepare_graphs(*members[0][1:])
    if case["kind"] == "rdf":
        s = systems[0]
        cls = np.where(s.q > 0, 1, np.where(s.q < 0, 2, 0)).astype(np.int32)
        state["hist"] = PairHistogram(s.N, np.arange(s.N), cls, 3, s.L, min(5.0, s.L / 2), 100)
    if case["kind"] in ("batch", "serve"):
        b = Batch(case["precision"], use_graph="auto" if case["kind"] == "serve" else True)
        for m in members:
            b.add(*m, first_step=1)
        state["batch"] = b
    if case["kind"] == "batch":
        state["beads"] = torch.arange(50, device=DEVICE)
        state["rg2"] = torch.zeros(len(members), dtype=torch.float64, device=DEVICE)
        state["box"] = [s.L for s in systems]
    return state


def run(state):
    """One pass; the trajectories' states advance in place."""
    case = state["case"]
    if case["kind"] == "eval":
        f = state["plan"].compute_components if case["components"] else state["plan"].compute
        return f(state["pos"], state["q"])
    out = [state["pos"], state["vel"], state["force"]]
    if case["kind"] in ("dpd", "rdf"):
        d, pos, vel, force = state["members"][0]
        d.run(pos, vel, force, state["step"], case["steps"])
        state["step"] += case["steps"]
        if case["kind"] == "rdf":
            state["hist"].sample(pos)
            out.append(state["hist"].hist)
        return out
    state["batch"].run(case["steps"])
    if case["kind"] == "batch":
        for k, (_, pos, _, _) in enumerate(state["members"]):
            chain_rg2(pos, state["beads"], state["box"][k], out=state["rg2"][k:k + 1])
        out.append(state["rg2"])
    return out


# ---------------------------------------------------------------------------
# Work that a pass cannot do without
# ---------------------------------------------------------------------------
def _elec_flops(nq, L, e):
    """Real-space pairs once each (about 60 operations), the spread and the
    gather over (2p)^3 points, and the two pruned transforms of the mesh."""
    pairs = 0.5 * nq * (nq / L ** 3) * 4.0 / 3.0 * math.pi * e["r_cut"] ** 3
    M = e["M"]
    return pairs * 60.0 + nq * (2 * e["p"]) ** 3 * 8.0 + 2 * 2.5 * M ** 3 * math.log2(M ** 3)


def work(case):
    if case["kind"] == "eval":
        n, z = case["n"], case["valency"]
        nq = int(round(case["charged"] * n / (1 + z))) * (1 + z)
        L = (n / 3.0) ** (1.0 / 3.0)
        return dict(bytes=float(32 * n + 24 * n + 40), flops=_elec_flops(nq, L, _eval_enuf(case, L)))
    nbytes = flops = 0.0
    for s in _systems(case, 0):
        rho = s.N / s.L ** 3
        nbytes += 2 * 72.0 * s.N   # the state in and out
        # each pair within R_c = 1 once, 44 operations and the random number's ten rounds
        step = 0.5 * s.N * rho * 4.0 / 3.0 * math.pi * 124.0 + _elec_flops(s.Nq, s.L, s.meta["enuf"])
        flops += case["steps"] * step
        if case["kind"] == "rdf":
            flops += 0.5 * s.N * s.N * 12.0
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------------------------------------
# The same in plain torch FP64
# ---------------------------------------------------------------------------
_CHUNK = 1 << 25   # pair matrix entries at a time


def _min_image(d, L):
    return d - L * torch.round(d / L)


def _real_space(x, q, L, e):
    """E_real, E_slater and the forces of the pairs within r_cut."""
    a, lam, rc = e["alpha"], e["lam"], e["r_cut"]
    n = x.shape[0]
    F = torch.zeros_like(x)
    er = es = 0.0
    for lo in range(0, n, max(1, _CHUNK // n)):
        xi = x[lo:lo + max(1, _CHUNK // n)]
        d2 = torch.zeros((xi.shape[0], n), dtype=x.dtype, device=x.device)
        for t in range(3):
            d2 += _min_image(xi[:, None, t] - x[None, :, t], L) ** 2
        i, j = torch.nonzero(d2 < rc * rc, as_tuple=True)
        keep = i + lo != j
        i, j = i[keep], j[keep]
        d = _min_image(xi[i] - x[j], L)
        r = d.norm(dim=1)
        qq = q[lo + i] * q[j]
        erfc = torch.erfc(a * r)
        u = erfc / r
        f = (u + 2.0 * a / math.sqrt(math.pi) * torch.exp(-(a * r) ** 2)) / r ** 2
        s = torch.zeros_like(r)
        if lam > 0.0:
            w = r / lam
            ex = torch.exp(-2.0 * w)
            s = -(1.0 + w) * ex / r
            f = f - (1.0 + 2.0 * w + 2.0 * w * w) * ex / r ** 3
        F.index_add_(0, lo + i, (qq * f)[:, None] * d)
        er += 0.5 * float((qq * (u + s)).sum())
        es += 0.5 * float((qq * s).sum())
    return er, es, F


def _reciprocal(x, q, L, e):
    """E_recip and the forces of the direct sum over 0 < |k| < Kc: structure
    factors of kz >= 0 from per-axis phases, the half space counted twice."""
    Kc, a = e["Kc"], e["alpha"]
    k = torch.arange(-Kc + 1, Kc, device=x.device)
    kd = k.to(x.dtype)
    c, s = [], []
    for t in range(3):
        th = (2.0 * math.pi / L) * x[:, t, None] * (kd if t < 2 else kd[Kc - 1:])[None, :]
        c.append(torch.cos(th))
        s.append(torch.sin(th))
    kz = kd[Kc - 1:]
    E = 0.0
    F = torch.zeros_like(x)
    for ix, kx in enumerate(k.tolist()):
        # e^{-i (kx x + ky y)} = u - i v
        u = c[0][:, ix, None] * c[1] - s[0][:, ix, None] * s[1]
        v = s[0][:, ix, None] * c[1] + c[0][:, ix, None] * s[1]
        qu, qv = (q[:, None] * u).t().contiguous(), (q[:, None] * v).t().contiguous()
        re = qu @ c[2] - qv @ s[2]
        im = -(qv @ c[2] + qu @ s[2])
        k2 = kx * kx + kd[:, None] ** 2 + kz[None, :] ** 2
        w = torch.exp(-(math.pi / (a * L)) ** 2 * k2) / torch.where(k2 > 0, k2, torch.ones_like(k2))
        w = torch.where((k2 > 0) & (k2 < Kc * Kc), w, torch.zeros_like(w)) * torch.where(kz > 0, 2.0, 1.0)[None, :]
        E += float((w * (re * re + im * im)).sum()) / (2.0 * math.pi * L)
        wr, wi = w * re, w * im
        # Im(conj(S) e^{-i k.r}) = -(Re S sin + Im S cos) per mode, weighted by k_t
        for t in range(3):
            kt = float(kx) if t == 0 else (kd[:, None] if t == 1 else kz[None, :])
            pr, pi = wr * kt, wi * kt
            g = (v @ pr + u @ pi) * c[2] + (u @ pr - v @ pi) * s[2]
            F[:, t] += (2.0 / L ** 2) * q * g.sum(dim=1)
    return E, F


def _ewald(pos, q, L, e):
    """(E_real, E_slater, E_recip, E_self) and the forces on all particles."""
    on = torch.nonzero(q != 0.0)[:, 0]
    x, c = torch.remainder(pos[on], L), q[on]
    er, es, Fr = _real_space(x, c, L, e)
    ek, Fk = _reciprocal(x, c, L, e)
    F = torch.zeros_like(pos)
    F[on] = Fr + Fk
    return (er, es, ek, -e["alpha"] / math.sqrt(math.pi) * float((c * c).sum())), F


def _theta(i, j, seed, step):
    """The pairs' uniform random numbers (Philox4x32-10 on the pair, the step and the seed)."""
    m32 = 0xFFFFFFFF
    c = [torch.minimum(i, j), torch.maximum(i, j), torch.full_like(i, step & m32), torch.full_like(i, step >> 32)]
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    u = ((c[0] << 21) | (c[1] >> 11)).to(torch.float64) / 9007199254740992.0
    return math.sqrt(3.0) * (2.0 * u - 1.0)


def _dpd_forces(s, pos, vel, q, step):
    P, L, n = s.meta["dpd"], s.L, s.N
    F = torch.zeros_like(pos)
    for lo in range(0, n, max(1, _CHUNK // n)):
        xi = pos[lo:lo + max(1, _CHUNK // n)]
        d2 = torch.zeros((xi.shape[0], n), dtype=pos.dtype, device=pos.device)
        for t in range(3):
            d2 += _min_image(xi[:, None, t] - pos[None, :, t], L) ** 2
        i, j = torch.nonzero((d2 < 1.0) & (d2 > 0.0), as_tuple=True)
        i = i + lo
        keep = i != j
        i, j = i[keep], j[keep]
        d = _min_image(pos[i] - pos[j], L)
        r = d.norm(dim=1)
        d = d / r[:, None]
        w = 1.0 - r
        ev = ((vel[i] - vel[j]) * d).sum(dim=1)
        mag = P["a"] * w - P["gamma"] * w * w * ev + P["sigma"] * w * _theta(i, j, P["seed"], step) / math.sqrt(P["dt"])
        F.index_add_(0, i, mag[:, None] * d)
    if s.bonds is not None and len(s.bonds):
        b = torch.tensor(s.bonds, device=pos.device)
        d = _min_image(pos[b[:, 0]] - pos[b[:, 1]], L)
        r = d.norm(dim=1)
        f = (-P["k_bond"] * (r - P["r0_bond"]) / r)[:, None] * d
        F.index_add_(0, b[:, 0], f)
        F.index_add_(0, b[:, 1], -f)
    return F + P["kappa"] * _ewald(pos, q, L, s.meta["enuf"])[1]


def _trajectory(s, steps):
    P = s.meta["dpd"]
    pos, vel = torch.tensor(s.pos, device=DEVICE), torch.tensor(s.vel, device=DEVICE)
    q = torch.tensor(s.q, device=DEVICE)
    F = _dpd_forces(s, pos, vel, q, 0)
    for step in range(1, 1 + steps):
        v0 = vel + P["lam"] * P["dt"] * F
        vel = vel + 0.5 * P["dt"] * F
        pos = torch.remainder(pos + P["dt"] * vel, s.L)
        F = _dpd_forces(s, pos, v0, q, step)
        vel = vel + 0.5 * P["dt"] * F
    return pos, vel, F


def exact(case, seed):
    """What ``run`` returns, in plain FP64; None where the direct sums take too long."""
    if case["kind"] == "eval":
        s = _electrolyte(case["n"], case["charged"], case["valency"], 1000 + seed)
        e = _eval_enuf(case, s.L)
        if float(s.Nq) ** 2 > 2e10 or s.Nq * float(2 * e["Kc"]) ** 3 > 2e10:
            return None
        (er, es, ek, eself), F = _ewald(torch.tensor(s.pos, device=DEVICE), torch.tensor(s.q, device=DEVICE), s.L, e)
        if case["components"]:
            return [F, torch.tensor([er, es, ek, eself, 0.0 if case["mode"] == "ik" else ek], dtype=torch.float64)]
        return [F, torch.tensor([er + ek + eself], dtype=torch.float64)]
    systems = _systems(case, seed)
    if sum(float(s.N) ** 2 + 100.0 * s.N * (2 * s.meta["enuf"]["Kc"]) for s in systems) * (1 + case["steps"]) > 3e10:
        return None
    if any(s.Nq * float(2 * s.meta["enuf"]["Kc"]) ** 3 * case["steps"] > 1e11 for s in systems):
        return None
    pos, vel, F = (torch.cat(x) for x in zip(*[_trajectory(s, case["steps"]) for s in systems]))
    # the histogram's counts (which accumulate over passes) and the radii of gyration are left to the other bounds
    return [pos, vel, F] + [None] * (case["kind"] in ("rdf", "batch"))
