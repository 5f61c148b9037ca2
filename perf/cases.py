"""Performance cases: the calls that programs make on this package, over the sizes they make them.

    listed()            the named cases
    draw(rng)           one more case from the same ranges
    prepare(case, seed) what a program holds before the call, on the GPU, made from the seed
    run(state)          one pass through the public entry points, and what it returns
    work(case)          bytes and flops that a pass cannot do without
    exact(case, seed)   the same outputs in plain 64-bit torch (None: too large, or whole numbers)

Kinds of case:
    score    energy, forces and charges of one new structure from a cold start (charges 0, new
             neighbour lists): scoring a data set, one structure after another on one buffer
    md       a short piece of NVE or NVT dynamics, charges equilibrated at every step
    coupled  the same with the charge-dependent covalent coupling
    relax    FIRE relaxation steps at fixed cell
    serve    a burst of uneven requests through the batching server
    fit      a fitting step: energies, forces and charges of a batch of structures and the
             gradient of the loss in the 56 parameters
    removal  removal energies of surface atoms (the desorption test)
    rings    ring statistics of a carbon sheet
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1802_07871_amd as ct
from ctbop_inputs import generators as G
from ctbop_inputs import params as PR
from paper_1802_07871_amd.autograd import ctbop_efq
from paper_1802_07871_amd.serving import Server


def listed():
    return [
        # the smallest call: a molecule-sized cluster, all latency and launches
        {"name": "score_cluster_12", "kind": "score", "form": "cluster", "n": 12, "c_frac": 0.75, "density": 2.6,
         "fp64": False},
        # an ordinary request of the serving mix, odd-sized, periodic, in the FP64 build
        {"name": "score_cell_1999", "kind": "score", "form": "cell", "n": 1999, "c_frac": 0.7, "density": 2.9,
         "fp64": True},
        # the largest request of the serving mix
        {"name": "score_cell_20000", "kind": "score", "form": "cell", "n": 20000, "c_frac": 0.6, "density": 2.6,
         "fp64": False},
        # small-system dynamics: 3C-SiC, 4x4x4 cells at 300 K
        {"name": "md_crystal_512", "kind": "md", "form": "crystal", "nx": 4, "ny": 4, "nz": 4, "temp": 300.0,
         "nvt": False, "steps": 30, "fp64": False},
        # growth-simulation-like NVT of a 4H-SiC slab, 24 x 24 cells x 16 bilayers
        {"name": "md_slab_nvt_36864", "kind": "md", "form": "slab", "nx": 24, "ny": 24, "nz": 16, "temp": 2500.0,
         "nvt": True, "steps": 10, "fp64": False},
        # the benchmark slab: 160 x 160 cells x 10 bilayers, stepped, depleted, 2500 K
        {"name": "md_slab_1m", "kind": "md", "form": "stepped", "nx": 160, "ny": 160, "nz": 10, "temp": 2500.0,
         "nvt": False, "steps": 5, "fp64": False},
        # dynamics with the charge-dependent coupling on a stepped slab of the paper's growth-cell size
        {"name": "coupled_slab_18086", "kind": "coupled", "form": "stepped", "nx": 24, "ny": 24, "nz": 8,
         "temp": 2500.0, "nvt": False, "steps": 5, "fp64": False},
        # FIRE relaxation of a slab with its bottom held
        {"name": "relax_slab_1920", "kind": "relax", "form": "slab", "nx": 10, "ny": 6, "nz": 8, "steps": 25,
         "fp64": False},
        # a burst of requests, 8 to 20,000 atoms, half clusters and half periodic cells
        {"name": "serve_48", "kind": "serve", "count": 48, "nmin": 8, "nmax": 20000, "mix": 1002},
        # one fitting step over a batch of crystals, sheets and amorphous carbon
        {"name": "fit_12", "kind": "fit", "count": 12, "nmin": 64, "nmax": 2000, "mix": 1003, "fp64": False},
        # the desorption test on the stepped slab of the paper's growth-cell size
        {"name": "removal_18086", "kind": "removal", "nx": 24, "ny": 24, "nz": 8, "count": 32},
        # ring statistics of a million-atom sheet
        {"name": "rings_graphene_1m", "kind": "rings", "nx": 500, "ny": 500, "defects": 400},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("score", "score", "score", "md", "md", "md", "coupled", "relax", "serve", "fit", "removal",
                       "rings"))
    if kind == "score":
        return {"kind": kind, "form": rng.choice(("cluster", "cell")), "n": _log(rng, 8, 20000),
                "c_frac": round(rng.uniform(0.5, 0.9), 3), "density": round(rng.uniform(2.0, 3.2), 3),
                "fp64": rng.random() < 0.25}
    if kind in ("md", "coupled", "relax"):
        form = rng.choice(("crystal", "slab", "stepped"))
        most = 250 if kind == "md" else 100          # in-plane cells of a slab: up to 10^5 - 10^6 atoms
        if form == "crystal":
            k = _log(rng, 2, 24)
            nx, ny, nz = k, k, k
        else:
            area = _log(rng, 9, most * 40)
            nx = max(3, int(round(math.sqrt(area) * rng.uniform(0.8, 1.25))))
            ny = max(2, int(round(area / nx)))
            nz = rng.choice((4, 6, 8, 10, 12)) if form == "slab" else rng.choice((8, 10, 12))
        if kind == "relax":
            return {"kind": kind, "form": form, "nx": nx, "ny": ny, "nz": nz, "steps": rng.randint(10, 30),
                    "fp64": rng.random() < 0.25}
        return {"kind": kind, "form": form, "nx": nx, "ny": ny, "nz": nz,
                "temp": float(rng.choice((300.0, 1000.0, 2000.0, 2500.0))),
                "nvt": kind == "md" and rng.random() < 0.5, "steps": rng.randint(3, 10),
                "fp64": kind == "md" and rng.random() < 0.2}
    if kind == "serve":
        return {"kind": kind, "count": rng.randint(4, 48), "nmin": 8, "nmax": _log(rng, 200, 20000),
                "mix": rng.randrange(1 << 16)}
    if kind == "fit":
        return {"kind": kind, "count": rng.randint(2, 12), "nmin": 64, "nmax": _log(rng, 200, 2000),
                "mix": rng.randrange(1 << 16), "fp64": rng.random() < 0.25}
    if kind == "removal":
        return {"kind": kind, "nx": rng.randint(6, 24), "ny": rng.randint(4, 24), "nz": 8, "count": rng.randint(8, 32)}
    return {"kind": kind, "nx": _log(rng, 12, 500), "ny": _log(rng, 8, 500), "defects": rng.randint(1, 12)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
FQ_KAPPA = 0.5
NVT_TAU = 25.0


def _slab(case, seed):
    stepped = case.get("form", "stepped") == "stepped"
    s = G.slab_4h(case["nx"], case["ny"], case["nz"], step=stepped, deplete=0.3 if stepped else 0.0, seed=seed)
    s.pos = s.pos + np.random.default_rng(seed + 1).normal(0.0, 0.03, size=s.pos.shape)
    return s


def _structures(case, seed):
    """The case's structure (a list of them for serve and fit), on the host."""
    kind = case["kind"]
    if kind == "score":
        return G.random_system(case["n"], case["c_frac"], case["density"], case["form"] == "cell", seed)
    if kind in ("md", "coupled", "relax"):
        s = G.zincblende(case["nx"], sigma=0.05, seed=seed) if case["form"] == "crystal" else _slab(case, seed)
        if kind == "relax":
            return s
        s.vel = G.maxwell_velocities(s.types, case["temp"], seed + 2, s.fixed)
        return s
    if kind == "rings":
        return G.graphene(case["nx"], case["ny"], case["defects"], seed, sigma=0.04)
    if kind == "serve":
        # (the mix fixes sizes and compositions, the seed the positions)
        reqs = G.serving_requests(case["count"], case["mix"], case["nmin"], case["nmax"])
        return [G.request_structure(dict(r, seed=seed + 7919 * k)) for k, r in enumerate(reqs)]
    if kind == "fit":
        batch = G.fit_batch(case["count"], case["mix"], case["nmin"], case["nmax"])
        rng = np.random.default_rng(seed)
        for s in batch:
            s.pos = s.pos + rng.normal(0.0, 0.02, s.pos.shape)
        return batch
    return _slab(case, seed)


def _candidates(s, case, seed):
    top = np.flatnonzero(s.meta["layer"] == s.meta["layer"].max())
    return np.sort(np.random.default_rng(seed + 3).permutation(top)[:case["count"]]).astype(np.int32)


def _fit_targets(structs, seed):
    """Trial parameters (up to 5 % off) and the reference energies, forces and charges of the batch."""
    rng = np.random.default_rng(seed + 4)
    th = PR.load() * (1.0 + 0.05 * rng.uniform(-1.0, 1.0, 56))
    for t in range(2):                               # keep S above R, angles and masses as they are
        for k in (4, 5, 10, 17, 25):
            th[26 * t + k] = PR.load()[26 * t + k]
    th[54] = PR.load()[54]
    ref = [(-6.0 * s.n * rng.uniform(0.9, 1.1), rng.normal(0.0, 2.0, (s.n, 3)), rng.normal(0.0, 0.3, s.n))
           for s in structs]
    return th, ref


def _gpu(a, dtype):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _on_gpu(s):
    d = {"pos": _gpu(s.pos, torch.float64), "types": _gpu(s.types, torch.int32), "box": s.box, "pbc": s.pbc,
         "fixed": s.fixed}
    if s.vel is not None:
        d["vel"] = _gpu(s.vel, torch.float64)
    return d


def prepare(case, seed):
    kind = case["kind"]
    s = _structures(case, seed)
    st = {"case": case}
    if kind == "serve":
        st["pot"] = ct.Potential(PR.load())
        st["server"] = Server(st["pot"], 4 << 30, max_slots=256)
        st["requests"] = [(r.pos, r.types, r.box, r.pbc) for r in s]
        return st
    if kind == "fit":
        th, ref = _fit_targets(s, seed)
        st["pot"] = ct.Potential(th, fp64=case["fp64"])
        st["theta"] = torch.tensor(th, dtype=torch.float64, requires_grad=True)
        st["batch"] = [_on_gpu(x) for x in s]
        st["ref"] = [(e, _gpu(f, torch.float64), _gpu(q, torch.float64)) for e, f, q in ref]
        return st
    if kind == "removal":
        st["pot"] = ct.Potential(PR.load())
        st["s"] = s
        st["cand"] = _candidates(s, case, seed)
        return st
    st["pot"] = ct.Potential(PR.load(), fp64=case.get("fp64", False),
                             fq_kappa=FQ_KAPPA if kind == "coupled" else 0.0)
    st["sys"] = st["pot"].system(s.n, s.box, s.pbc)
    st.update(_on_gpu(s))
    return st


def run(st):
    case = st["case"]
    kind, pot = case["kind"], st["pot"]
    if kind == "score":
        E, F, q, _ = pot.compute(st["pos"], st["types"], st["box"], st["pbc"], warm=False, force_rebuild=True,
                                 sysbuf=st["sys"])
        return {"E": E, "F": F, "q": q}
    if kind in ("md", "coupled"):
        a = (st["pos"], st["vel"], st["types"], st["box"], st["pbc"], 0.5, case["steps"])
        if case["nvt"]:
            x, v, F, q, th, chain, _ = pot.md_run_nvt(*a, T=case["temp"], tau=NVT_TAU, fixed=st["fixed"],
                                                      sysbuf=st["sys"])
            return {"x": x, "v": v, "F": F, "q": q, "thermo": th, "chain": chain}
        x, v, F, q, th, _ = pot.md_run(*a, fixed=st["fixed"], sysbuf=st["sys"])
        return {"x": x, "v": v, "F": F, "q": q, "thermo": th}
    if kind == "relax":
        x, F, q, trace, k, fm, conv, _ = pot.relax_fire(st["pos"], st["types"], st["box"], st["pbc"], fmax=1e-3,
                                                        max_steps=case["steps"], fixed=st["fixed"], sysbuf=st["sys"])
        return {"x": x, "F": F, "q": q, "trace": trace, "fmax": fm, "steps": k, "converged": conv}
    if kind == "serve":
        srv = st["server"]
        tickets = [srv.submit(*r) for r in st["requests"]]
        got = srv.wait_all(tickets)
        return {"E": np.array([got[t]["E"] for t in tickets]), "F": np.concatenate([got[t]["F"] for t in tickets]),
                "q": np.concatenate([got[t]["q"] for t in tickets])}
    if kind == "fit":
        theta = st["theta"]
        theta.grad = None
        loss, energies = 0.0, []
        for s, (e0, f0, q0) in zip(st["batch"], st["ref"]):
            E, F, q = ctbop_efq(theta, s["pos"], s["types"], s["box"], s["pbc"], pot)
            loss = loss + _loss(E, F, q, e0, f0, q0)
            energies.append(E.detach())
        loss.backward()
        return {"grad": theta.grad, "loss": loss.detach(), "E": torch.stack(energies)}
    if kind == "removal":
        s = st["s"]
        E, dE, _ = pot.removal_energies(s.pos, s.types, s.box, s.pbc, st["cand"])
        return {"E": E, "dE": dE}
    r = pot.rings(st["pos"], st["types"], st["box"], st["pbc"], r_bond=1.7, sysbuf=st["sys"])
    return {"counts": r["counts"], "bonds": r["bonds"], "chain_bonds": r["chain_bonds"], "hist": r["hist"]}


def _loss(E, F, q, e0, f0, q0):
    n = q.numel()
    return ((F - f0) ** 2).mean() + ((E - e0) / n) ** 2 + ((q - q0) ** 2).mean()


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def _atoms(case):
    kind = case["kind"]
    if kind == "score":
        return case["n"]
    if kind == "rings":
        return 4 * case["nx"] * case["ny"]
    if kind in ("serve", "fit"):                     # mean of the log-uniform sizes
        lo, hi = case["nmin"], max(case["nmax"], case["nmin"] + 1)
        return case["count"] * (hi - lo) / math.log(hi / lo)
    if case.get("form") == "crystal":
        return 8 * case["nx"] ** 3
    return 4 * case["nx"] * case["ny"] * case["nz"]


def work(case):
    """Per evaluation: positions and types in, forces and charges out; each unordered Coulomb pair's
    kernel once for the matrix and once with its derivative (~80 flops), a product with the matrix per
    solver iteration (two flops an entry; ~40 iterations from a cold start, ~22 from the previous
    step), and ~600 flops per atom and bond pair of the covalent part."""
    kind, n = case["kind"], _atoms(case)
    pairs = n * 170                                  # ordered, inside 8 A
    io = n * (3 * 8 + 4 + 3 * 8 + 8)

    def evaluation(iters):
        return pairs * (40 + 2 * iters) + n * 12 * 600

    if kind == "rings":
        return {"bytes": n * 28, "flops": n * 200}
    if kind in ("md", "coupled"):
        k = case["steps"]
        return {"bytes": io + 2 * 24 * n, "flops": evaluation(30) + k * evaluation(22)}
    if kind == "relax":
        return {"bytes": io, "flops": evaluation(30) + case["steps"] * evaluation(22)}
    if kind == "removal":
        return {"bytes": 28 * n, "flops": evaluation(40) + case["count"] * evaluation(34)}
    if kind == "fit":
        return {"bytes": io + 32 * n, "flops": 4 * evaluation(40)}
    return {"bytes": io, "flops": evaluation(40)}


# ---------------------------------------------------------------------------
# the same outputs in plain 64-bit torch
# ---------------------------------------------------------------------------
ACC = 9.648533212e-3                                 # (eV/A)/amu in A/fs^2
KB = 8.617333262e-5


def _pairs(x, box, pbc, cut):
    """Ordered pairs closer than cut, images included, sorted by the first atom: i, j, image shift."""
    n = len(x)
    b = torch.as_tensor(box, dtype=torch.float64, device=x.device)
    inv = torch.linalg.inv(b.cpu()).to(x.device)
    width = 1.0 / torch.linalg.vector_norm(inv, dim=0)
    wrap = torch.floor((x[:, :, None] * inv[None]).sum(1)) * torch.as_tensor(np.asarray(pbc, float), device=x.device)
    home = (wrap[:, :, None] * b[None]).sum(1)       # x - home lies in the cell along the periodic vectors
    y = x - home
    reach = [int(cut / float(width[a])) + 1 if pbc[a] else 0 for a in range(3)]
    rows = max(1, int(4e7) // n)
    out = []
    for r0 in range(0, n, rows):
        yi = y[r0:r0 + rows]
        for a in range(-reach[0], reach[0] + 1):
            for c in range(-reach[1], reach[1] + 1):
                for d in range(-reach[2], reach[2] + 1):
                    sh = a * b[0] + c * b[1] + d * b[2]
                    r2 = (y[None, :, 0] + (sh[0] - yi[:, 0, None])) ** 2
                    r2 += (y[None, :, 1] + (sh[1] - yi[:, 1, None])) ** 2
                    r2 += (y[None, :, 2] + (sh[2] - yi[:, 2, None])) ** 2
                    near = torch.nonzero((r2 < cut * cut) & (r2 > 1e-12))
                    i, j = near[:, 0] + r0, near[:, 1]
                    out.append((i, j, sh[None] + home[i] - home[j]))
    i, j, sh = (torch.cat([o[k] for o in out]) for k in range(3))
    order = torch.argsort(i, stable=True)
    return i[order], j[order], sh[order]


class _Exact:
    """Energy, forces and charges of one structure; x may move as long as the pair list covers it."""

    def __init__(self, types, box, pbc, theta, kappa=0.0, slack=0.5):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.t = torch.as_tensor(np.asarray(types), dtype=torch.int64, device=self.dev)
        self.box, self.pbc, self.kappa, self.slack = box, pbc, kappa, slack
        self.th = theta if torch.is_tensor(theta) else torch.tensor(theta, dtype=torch.float64)
        self.th = self.th.to(self.dev)
        self.x0 = None

    def _species(self, k):
        return torch.stack([self.th[k], self.th[26 + k]])

    def _mix(self, k, geo):
        s = self._species(k)
        return torch.sqrt(s[:, None] * s[None, :]) if geo else 0.5 * (s[:, None] + s[None, :])

    def _list(self, x):
        if self.x0 is None or float((x - self.x0).abs().max()) > 0.25 * self.slack:
            self.x0 = x.detach().clone()
            self.pi, self.pj, self.ps = _pairs(self.x0, self.box, self.pbc, float(self.th[54]) + self.slack)

    def _coulomb(self, x, near):
        i, j, sh = near
        d = x[j] + sh - x[i]
        r = torch.sqrt((d * d).sum(1))
        gam = self._species(23)
        g3 = (gam[self.t[i]] * gam[self.t[j]]) ** -1.5
        u = r / self.th[54]
        taper = (1 - u) ** 4 * (1 + 4 * u + 10 * u ** 2 + 20 * u ** 3)
        return self.th[53] * taper * (r ** 3 + g3) ** (-1.0 / 3.0)

    def _covalent(self, x, near):
        """Attractive and repulsive halves per ordered bond: (i, j, 1/2 fc fR, 1/2 fc b fA)."""
        i, j, sh = near
        n, K = len(x), int(torch.bincount(i, minlength=len(x)).max()) if len(i) else 0
        if K == 0:
            z = torch.zeros(0, dtype=torch.float64, device=self.dev)
            return i, j, z, z
        start = torch.searchsorted(i, torch.arange(n, device=self.dev))
        col = torch.arange(len(i), device=self.dev) - start[i]
        ti, tj = self.t[i], self.t[j]
        d = x[j] + sh - x[i]
        r = torch.sqrt((d * d).sum(1))
        mix = torch.ones(2, 2, dtype=torch.float64, device=self.dev) + \
            (self.th[52] - 1.0) * (1.0 - torch.eye(2, dtype=torch.float64, device=self.dev))
        A, B = self._mix(0, True)[ti, tj], (self._mix(1, True) * mix)[ti, tj]
        l1, l2 = self._mix(2, False)[ti, tj], self._mix(3, False)[ti, tj]
        Rc, Sc = self._mix(4, True)[ti, tj], self._mix(5, True)[ti, tj]
        fc = torch.where(r <= Rc, torch.ones_like(r), 0.5 + 0.5 * torch.cos(math.pi * (r - Rc) / (Sc - Rc)))
        shape = (n, K)
        D = torch.zeros(*shape, 3, dtype=torch.float64, device=self.dev).index_put((i, col), d / r[:, None])
        Rr = torch.ones(shape, dtype=torch.float64, device=self.dev).index_put((i, col), r)
        Fc = torch.zeros(shape, dtype=torch.float64, device=self.dev).index_put((i, col), fc)
        Dk, Rk, Fk = D[i], Rr[i], Fc[i]              # per bond: its centre's bonds
        other = torch.ones(len(i), K, dtype=torch.float64, device=self.dev)
        other[torch.arange(len(i), device=self.dev), col] = 0.0
        cos = (Dk * (d / r[:, None])[:, None, :]).sum(2)
        zh = []
        for ch in (7, 14):
            p = [self._species(ch + k)[ti] for k in range(7)]    # gamma, c, d, h, n, g, alpha
            u = p[3][:, None] - cos
            w = p[0][:, None] * (1 + (p[1] / p[2])[:, None] ** 2 * u ** 2 / (p[2][:, None] ** 2 + u ** 2))
            ex = torch.exp((p[6][:, None] * (r[:, None] - Rk)) ** 3)
            z = (other * Fk * w * ex).sum(1)
            some = z > 0
            zh.append(p[5] + torch.where(some, torch.where(some, z, torch.ones_like(z)) ** p[4], torch.zeros_like(z)))
        pw, sig = self.th[55], self._species(6)[ti]
        g1, g2 = self._species(12)[ti], self._species(19)[ti]
        b = ((zh[0] ** -pw + zh[1] ** -pw) / (g1 ** -pw + g2 ** -pw)) ** (1.0 / (2.0 * sig * pw))
        return i, j, 0.5 * fc * A * torch.exp(-l1 * r), 0.5 * fc * b * B * torch.exp(-l2 * r)

    def _near(self, x, cut):
        d = x[self.pj] + self.ps - x[self.pi]
        k = torch.nonzero((d * d).sum(1) < cut * cut if not torch.is_tensor(cut) or cut.dim() == 0 else
                          (d * d).sum(1) < cut ** 2)[:, 0]
        return self.pi[k], self.pj[k], self.ps[k]

    def __call__(self, x, Q=0.0, graph=False, q0=None):
        x = x.detach()
        self._list(x)
        n = len(x)
        with torch.no_grad():
            far = self._near(x, self.th[54].detach())
            near = self._near(x, self._mix(5, True)[self.t[self.pi], self.t[self.pj]].detach())
        J, chi = self._species(22)[self.t], self._species(21)[self.t]
        with torch.set_grad_enabled(graph):
            C = self._coulomb(x, far)
            if n <= 2600:
                H = torch.diag(J).index_put((far[0], far[1]), C, accumulate=True)
                both = torch.linalg.solve(H, torch.stack([-chi, torch.ones_like(chi)], 1))
                q = both[:, 0] + both[:, 1] * (Q - both[:, 0].sum()) / both[:, 1].sum()
            else:
                q = self._cg(C, far, J, -chi, Q, q0)
        if self.kappa > 0:
            with torch.no_grad():
                bi, bj, _, att = self._covalent(x, near)
                q = self._newton(C, far, J, chi, q, bi, bj, 2.0 * att)
        xg = x.clone().requires_grad_(True)
        i, j, rep, att = self._covalent(xg, near)
        if self.kappa > 0:
            att = att * torch.exp(-self.kappa * (q[i] - q[j]) ** 2)
        E = rep.sum() - att.sum() + 0.5 * (q[far[0]] * q[far[1]] * self._coulomb(xg, far)).sum()
        E = E + (self._species(24)[self.t] + chi * q + 0.5 * J * q * q).sum()
        F = -torch.autograd.grad(E, xg, create_graph=graph, retain_graph=graph)[0]
        if graph:
            # total energy derivative in the parameters: q is stationary, so its own graph adds mu sum(dq) = 0
            return E, F, q
        return E.detach(), F.detach(), q.detach()

    @staticmethod
    def _apply(C, far, J, v):
        return J * v + torch.zeros_like(v).index_add_(0, far[0], C * v[far[1]])

    def _cg(self, C, far, J, rhs, Q, q0, extra=None, tol=1e-13, maxit=400):
        """Projected Jacobi-preconditioned CG for (H + extra) q = rhs + mu, sum q = Q."""
        n = len(J)
        apply = (lambda v: self._apply(C, far, J, v)) if extra is None else \
            (lambda v: self._apply(C, far, J, v) + extra(v))
        q = torch.full_like(J, Q / n) if q0 is None else q0 + (Q - q0.sum()) / n
        m = 1.0 / J
        r = rhs - apply(q)
        r = r - r.mean()
        p, rho = None, None
        for _ in range(maxit):
            z = m * r
            z = z - m * (z.sum() / m.sum())
            new = (r * z).sum()
            p = z if p is None else z + (new / rho) * p
            rho = new
            s = apply(p)
            a = rho / (p * s).sum()
            q = q + a * p
            r = r - a * s
            r = r - r.mean()
            if float(torch.sqrt((r * r).mean())) < tol:
                break
        return q + (Q - q.sum()) / n

    def _newton(self, C, far, J, chi, q, bi, bj, c):
        """Charges with the coupling energy -1/2 sum c exp(-kappa (q_i - q_j)^2) added."""
        kap = self.kappa
        for _ in range(20):
            d = q[bi] - q[bj]
            f = c * kap * torch.exp(-kap * d * d)
            g = self._apply(C, far, J, q) + chi
            g = g.index_add(0, bi, f * d).index_add(0, bj, -f * d)
            g = g - g.mean()
            if float(torch.sqrt((g * g).mean())) < 1e-12:
                break
            h = f * (1 - 2 * kap * d * d)

            def extra(v):
                w = h * (v[bi] - v[bj])
                return torch.zeros_like(v).index_add_(0, bi, w).index_add_(0, bj, -w)

            q = q + self._cg(C, far, J, -g, 0.0, torch.zeros_like(q), extra, tol=1e-13)
        return q


def _t(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float64, device="cuda" if torch.cuda.is_available() else "cpu")


def _exact_md(case, s):
    ex = _Exact(s.types, s.box, s.pbc, PR.load(), FQ_KAPPA if case["kind"] == "coupled" else 0.0, slack=1.0)
    x, v = _t(s.pos), _t(s.vel)
    mass = _t(np.where(s.types == 0, PR.load()[25], PR.load()[51]))[:, None]
    mob = _t(np.ones(s.n) if s.fixed is None else ~s.fixed)[:, None]
    dt, nvt, M = 0.5, case["nvt"], 3
    xi, vxi = [0.0] * M, [0.0] * M
    nm = int(mob.sum())
    nf, kT = 3.0 * nm - (3.0 if nm == s.n else 0.0), KB * case["temp"]
    Qm = [(nf if k == 0 else 1.0) * kT * NVT_TAU ** 2 for k in range(M)]

    def kinetic():
        return float((0.5 * mass * v * v * (mob if nvt else 1.0)).sum()) / ACC

    def half(K):
        h = 0.5 * dt
        g = (lambda k, K: (2 * K - nf * kT) / Qm[0] if k == 0 else (Qm[k - 1] * vxi[k - 1] ** 2 - kT) / Qm[k])
        vxi[M - 1] += 0.5 * h * g(M - 1, K)
        for k in range(M - 2, -1, -1):
            e = math.exp(-0.25 * h * vxi[k + 1])
            vxi[k] = (vxi[k] * e + 0.5 * h * g(k, K)) * e
        sc = math.exp(-h * vxi[0])
        K *= sc * sc
        for k in range(M):
            xi[k] += h * vxi[k]
        for k in range(M - 1):
            e = math.exp(-0.25 * h * vxi[k + 1])
            vxi[k] = (vxi[k] * e + 0.5 * h * g(k, K)) * e
        vxi[M - 1] += 0.5 * h * g(M - 1, K)
        return sc

    def scaled(sc):
        return v * (1.0 + (sc - 1.0) * mob)

    def row(E):
        K = kinetic()
        if not nvt:
            return [float(E), K]
        eth = nf * kT * xi[0] + sum(0.5 * Qm[k] * vxi[k] ** 2 + (kT * xi[k] if k else 0.0) for k in range(M))
        return [float(E), K, float(E) + K + eth]

    E, F, q = ex(x)
    thermo = [row(E)]
    for _ in range(case["steps"]):
        if nvt:
            v = scaled(half(kinetic()))
        v = v + mob * (0.5 * dt * ACC) * F / mass
        x = x + dt * mob * v
        E, F, q = ex(x, q0=q)
        v = v + mob * (0.5 * dt * ACC) * F / mass
        if nvt:
            v = scaled(half(kinetic()))
        thermo.append(row(E))
    out = {"x": x, "v": v, "F": F, "q": q, "thermo": np.array(thermo)}
    if nvt:
        out["chain"] = np.array(xi + vxi)
    return out


def _exact_relax(case, s):
    ex = _Exact(s.types, s.box, s.pbc, PR.load())
    x = _t(s.pos)
    v = torch.zeros_like(x)
    mass = _t(np.where(s.types == 0, PR.load()[25], PR.load()[51]))[:, None]
    mob = _t(np.ones(s.n) if s.fixed is None else ~s.fixed)[:, None]
    dt, alpha, npos = 0.5, 0.1, 0
    E, F, q = ex(x)
    f = mob * F
    trace, fm = [float(E)], float(torch.sqrt((f * f).sum(1).max()))
    P = vv = ff = 0.0
    for k in range(case["steps"]):
        if fm < 1e-3:
            break
        cv, cf = 1.0, 0.0
        if k > 0:
            cv, cf = 1.0 - alpha, alpha * math.sqrt(vv) / math.sqrt(ff)
            if P > 0.0:
                npos += 1
                if npos > 5:
                    dt, alpha = min(dt * 1.1, 5.0), alpha * 0.99
            else:
                dt, alpha, npos, cv, cf = dt * 0.5, 0.1, 0, 0.0, 0.0
        v = cv * v + cf * f + (0.5 * dt * ACC) * f / mass
        x = x + dt * v
        E, F, q = ex(x, q0=q)
        f = mob * F
        v = v + (0.5 * dt * ACC) * f / mass
        P, vv, ff = float((f * v).sum()), float((v * v).sum()), float((f * f).sum())
        fm = float(torch.sqrt((f * f).sum(1).max()))
        trace.append(float(E))
    return {"x": x, "F": F, "q": q, "trace": np.array(trace), "fmax": fm, "steps": None, "converged": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "rings" or (kind in ("md", "coupled", "relax") and _atoms(case) * case["steps"] > 4e5):
        return None
    s = _structures(case, seed)
    if kind == "score":
        E, F, q = _Exact(s.types, s.box, s.pbc, PR.load())(_t(s.pos))
        return {"E": float(E), "F": F, "q": q}
    if kind in ("md", "coupled"):
        return _exact_md(case, s)
    if kind == "relax":
        return _exact_relax(case, s)
    if kind == "serve":
        got = [_Exact(r.types, r.box, r.pbc, PR.load())(_t(r.pos)) for r in s]
        return {"E": np.array([float(g[0]) for g in got]), "F": torch.cat([g[1] for g in got]),
                "q": torch.cat([g[2] for g in got])}
    if kind == "fit":
        th, ref = _fit_targets(s, seed)
        theta = torch.tensor(th, dtype=torch.float64, requires_grad=True)
        total, energies = 0.0, []
        for r, (e0, f0, q0) in zip(s, ref):
            E, F, q = _Exact(r.types, r.box, r.pbc, theta)(_t(r.pos), graph=True)
            loss = _loss(E, F, q, e0, _t(f0), _t(q0))
            loss.backward()
            total += float(loss)
            energies.append(float(E))
        return {"grad": theta.grad, "loss": torch.tensor(total, dtype=torch.float64), "E": torch.tensor(energies, dtype=torch.float64)}
    ex = _Exact(s.types, s.box, s.pbc, PR.load(), slack=0.01)
    x = _t(s.pos)
    E0, _, q = ex(x)
    dE = []
    pairs = (ex.pi, ex.pj, ex.ps, ex.t)
    for c in _candidates(s, case, seed).tolist():
        keep = torch.ones(s.n, dtype=torch.bool, device=x.device)
        keep[c] = False
        k = keep[pairs[0]] & keep[pairs[1]]
        ex.pi, ex.pj, ex.ps, ex.t = pairs[0][k], pairs[1][k], pairs[2][k], pairs[3][keep]
        ex.pi, ex.pj = ex.pi - (ex.pi > c).long(), ex.pj - (ex.pj > c).long()
        ex.x0 = x[keep]
        dE.append(float(ex(x[keep], q0=q[keep])[0] - E0))
    return {"E": float(E0), "dE": np.array(dE)}
