"""Measured cases: what a user of this library has it do, through its Python binding.

Kinds of case
  apply     y = H x on one sector (rank order, or the grouped order the solvers iterate in)
  ground    ground state of one sector: energy and eigenvector
  lowest    the k lowest energies of one sector, counted with multiplicity
  batched   the lowest energy of every sector of an impurity, all advanced together
  green     impurity Green function of one eigenstate by two continued fractions

A case names the model family, its size, the sector and the options; the model's
free parameters (bath energies, hybridisations, U) and the vectors come from the
seed.  Precisions: "fp64", and "fp32" = FP32-stored vectors ("FP32-mixed").

`exact` is an independent dense-tensor evaluation in 64 bits: operator strings on
enumerated bit strings with torch indexing, and a plain fully reorthogonalised
Lanczos iteration on top of it.
"""
import math

import numpy as np
import torch

from paper_1004_3354_amd import ed, models

DEV = "cuda"
BETA = 10.0   # inverse temperature of the Matsubara points of the Green function
NZ = 64


# ------------------------------------------------------------------ cases ----

def listed():
    return [
        # one impurity and seven bath levels, half filling: the smallest sector in use,
        # where a product is one short launch
        dict(name="apply-aim8-fp64", kind="apply", model="aim", size=8, nup=4, ndn=4, prec="fp64", order="rank"),
        # three orbitals with three bath levels each: the sector a DMFT loop spends its time in
        dict(name="apply-kan12-fp64", kind="apply", model="kan", size=12, nup=6, ndn=6, prec="fp64", order="rank"),
        # off half filling, unequal spins, in the order a caller's own vectors have
        dict(name="apply-kan15-rank-fp64", kind="apply", model="kan", size=15, nup=6, ndn=8, prec="fp64",
             order="rank"),
        # the benchmark's product
        dict(name="apply-kan15-fp32", kind="apply", model="kan", size=15, nup=7, ndn=7, prec="fp32",
             order="grouped"),
        # the 4x4 Hubbard lattice: connected move graphs, no grouped order
        dict(name="apply-hub4x4-fp32", kind="apply", model="hub", size=16, nup=8, ndn=8, prec="fp32", order="rank"),
        # the largest sector one GPU is asked to hold
        dict(name="apply-kan18-fp32", kind="apply", model="kan", size=18, nup=9, ndn=9, prec="fp32",
             order="grouped"),
        # a one-band impurity solved with the default options
        dict(name="ground-aim8-fp64", kind="ground", model="aim", size=8, nup=4, ndn=4, prec="fp64", reorth=2,
             basis=0, keep=0),
        # a three-orbital impurity sector with two-pass reorthogonalisation and the planned basis
        dict(name="ground-kan12-fp64", kind="ground", model="kan", size=12, nup=6, ndn=6, prec="fp64", reorth=2,
             basis=0, keep=0),
        # the benchmark's time to E0: implicit restarts, one basis read for both projections
        dict(name="ground-kan15-fp32", kind="ground", model="kan", size=15, nup=7, ndn=7, prec="fp32", reorth=3,
             basis=14, keep=4),
        # several levels of a lattice sector, deflated one after another
        dict(name="lowest4-hub4x3-fp64", kind="lowest", model="hub", size=12, nup=6, ndn=6, prec="fp64", k=4,
             reorth=2, basis=24, keep=8),
        # every sector of the 12-site impurity at once, as the thermal average needs them
        dict(name="batched-kan12-fp32", kind="batched", model="kan", size=12, nup=0, ndn=0, prec="fp32", reorth=3,
             basis=20, keep=8),
        # Green function of the 15-site impurity's ground state
        dict(name="green-kan15-fp32", kind="green", model="kan", size=15, nup=7, ndn=7, prec="fp32", m=100),
    ]


LATTICE = {6: (3, 2), 8: (4, 2), 9: (3, 3), 12: (4, 3), 16: (4, 4)}


def _sizes(model):
    return {"aim": range(4, 17), "kan": (6, 9, 12, 15, 18), "hub": tuple(LATTICE)}[model]


def _sector(rng, model, lo, hi):
    """A sector with lo <= D <= hi, its dimension spread over the logarithm."""
    t = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    near = [(n, a, b) for n in _sizes(model) for a in range(1, n) for b in range(1, n)
            if t / 2 <= math.comb(n, a) * math.comb(n, b) <= min(2 * t, hi)]
    # the fillings that matter lie around one half
    near = [c for c in near if abs(2 * c[1] - c[0]) <= c[0] // 2 + 1 and abs(2 * c[2] - c[0]) <= c[0] // 2 + 1] or near
    return rng.choice(near)


def draw(rng):
    kind = rng.choice(["apply"] * 5 + ["ground"] * 3 + ["lowest", "batched", "green", "green"])
    prec = rng.choice(["fp64", "fp32"])
    model = rng.choice(["aim", "kan", "kan", "hub"])
    c = dict(kind=kind, model=model, prec=prec)
    if kind == "apply":
        order = rng.choice(["rank", "grouped"]) if model != "hub" else "rank"
        n, a, b = _sector(rng, model, 1.0e3, 1.0e9 if order == "grouped" else 2.0e8)
        c.update(size=n, nup=a, ndn=b, order=order)
    elif kind == "ground":
        n, a, b = _sector(rng, model, 1.0e3, 4.2e7 if prec == "fp32" else 8.0e6)
        keep = rng.choice([0, 4, 8])
        c.update(size=n, nup=a, ndn=b, reorth=rng.choice([2, 3]), keep=keep, basis=rng.randint(14, 40) if keep else 0)
    elif kind == "lowest":
        n, a, b = _sector(rng, model, 1.0e3, 9.0e5)
        c.update(size=n, nup=a, ndn=b, k=rng.randint(2, 5), reorth=2, keep=8, basis=rng.randint(18, 40))
    elif kind == "batched":
        model = rng.choice(["aim", "kan"])
        keep = rng.choice([0, 4, 8])
        c.update(model=model, size=rng.randint(6, 11) if model == "aim" else rng.choice([6, 9, 12]), nup=0, ndn=0,
                 reorth=rng.choice([2, 3]), keep=keep, basis=rng.randint(16, 40) if keep else 60)
    else:
        model = rng.choice(["aim", "kan"])
        n, a, b = _sector(rng, model, 1.0e3, 1.0e6)
        c.update(model=model, size=n, nup=a, ndn=b, m=rng.randint(40, 120))
    return c


# ------------------------------------------------------------------ inputs ----

def _model(c, seed):
    """Physical parameters of the case's model: the distributions of the benchmark workloads."""
    rng = np.random.default_rng(seed)
    n = c["size"]
    if c["model"] == "aim":
        return {"model": "aim", "Ns": n, "U": float(rng.uniform(1.5, 2.5)), "eps_d": -1.0,
                "eps_k": rng.uniform(-2.0, 2.0, n - 1).tolist(), "V": rng.uniform(0.2, 0.6, n - 1).tolist()}
    if c["model"] == "hub":
        lx, ly = LATTICE[n]
        return {"model": "hubbard", "Ns": n, "lx": lx, "ly": ly, "t": 1.0, "U": float(rng.uniform(3.0, 5.0)),
                "periodic": True}
    nb, U, J = n // 3 - 1, 2.3, 0.4
    up = U - 2.0 * J
    return {"model": "kanamori", "Ns": n, "M": 3, "n_b": nb, "U": U, "J": J, "Up": up, "Jp_sf": J, "Jp_ph": J,
            "eps_imp": [-(U / 2.0 + (2.0 * up - J))] * 3, "eps_bath": rng.uniform(-3.0, 3.0, (3, nb)).tolist(),
            "V": rng.uniform(0.1, 0.5, (3, nb)).tolist()}


def _dim(c):
    return math.comb(c["size"], c["nup"]) * math.comb(c["size"], c["ndn"])


def _vector(n, dtype, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn(n, generator=g, device=DEV, dtype=dtype)


def _prec(c):
    return ed.ED_FP64 if c["prec"] == "fp64" else ed.ED_FP32


def _dtype(c):
    return torch.float64 if c["prec"] == "fp64" else torch.float32


def _tol(c):
    return 1e-12 if c["prec"] == "fp64" else 1e-7


def _opts(c):
    return ed.options(tol=_tol(c), reorth=c["reorth"], max_basis=c["basis"], keep=c["keep"], max_iter=3000)


def _ham(p, nup, ndn, prec):
    return ed.Hamiltonian(p, ed.Basis(int(p["Ns"]), nup, ndn), prec)


def _tuned(H, dtype):
    """The first product on a handle chooses its schedule; a program's later ones do not."""
    x = torch.zeros(H.D, dtype=dtype, device=DEV)
    H.apply(x, torch.empty_like(x))
    return H


def _matsubara():
    return 1j * math.pi * (2 * np.arange(NZ) + 1) / BETA


def prepare(case, seed):
    c, n = case, case["size"]
    p = models.params_from_model(_model(c, seed))
    s = {"case": c}
    if c["kind"] == "batched":
        s["hams"] = [_ham(p, a, b, _prec(c)) for a in range(n + 1) for b in range(n + 1)]
        s["seed"] = seed
        s["opts"] = _opts(c)
        return s
    H = _ham(p, c["nup"], c["ndn"], _prec(c))
    s["H"] = H
    if c["kind"] == "apply":
        if c["order"] == "grouped":
            s["H"] = H.grouped() or H
        s["x"] = _vector(H.D, _dtype(c), seed)
        s["y"] = torch.empty_like(s["x"])
        _tuned(s["H"], _dtype(c))
    elif c["kind"] in ("ground", "lowest"):
        s["x"] = _vector(H.D, _dtype(c), seed)
        s["opts"] = _opts(c)
        if c["kind"] == "ground":
            s["psi"] = torch.empty_like(s["x"])
        _tuned(H.grouped() or H, _dtype(c))
    else:
        # a well converged eigenvector, held in the run's precision
        h = H if c["prec"] == "fp64" else _ham(p, c["nup"], c["ndn"], ed.ED_FP64)
        psi = torch.empty(h.D, dtype=torch.float64, device=DEV)
        opts = ed.options(tol=1e-12, reorth=3, max_basis=min(20, h.D), keep=min(6, h.D - 2), max_iter=3000)
        s["e0"], _ = h.lanczos_ground(_vector(h.D, torch.float64, seed), opts, psi=psi)
        s["psi"] = psi.to(_dtype(c))
        s["Hp"] = _tuned_pair(_ham(p, c["nup"] + 1, c["ndn"], _prec(c)), _dtype(c))
        s["Hm"] = _tuned_pair(_ham(p, c["nup"] - 1, c["ndn"], _prec(c)), _dtype(c))
    return s


def _tuned_pair(H, dtype):
    _tuned(H.grouped() or H, dtype)
    return H


def run(state):
    c = state["case"]
    if c["kind"] == "apply":
        state["H"].apply(state["x"], state["y"])
        return state["y"]
    if c["kind"] == "ground":
        e, _ = state["H"].lanczos_ground(state["x"], state["opts"], psi=state["psi"])
        return {"E": np.float64(e), "psi": state["psi"]}
    if c["kind"] == "lowest":
        e, _ = state["H"].lowest(c["k"], state["x"], state["opts"])
        return e
    if c["kind"] == "batched":
        e, _ = ed.lanczos_ground_batched(state["hams"], state["opts"], seed=state["seed"])
        return e
    g, _ = ed.green_function(state["H"], state["e0"], state["psi"], state["Hp"], state["Hm"], 0, 0, _matsubara(),
                             m=c["m"])
    # the fractions carry the precision of the vectors they were built from
    return g if c["prec"] == "fp64" else g.astype(np.complex64)


# -------------------------------------------------------------------- work ----

def work(case):
    """One read of x and one write of y per product; a solver step besides reads the
    stored vectors once and writes the new one.  Steps are nominal: about 60 for a
    ground state, as many again for each further level, m for a continued fraction."""
    c, el = case, 8 if case["prec"] == "fp64" else 4
    n = c["size"]
    hops = {"aim": n, "kan": n, "hub": 2 * n}[c["model"]] + (6 if c["model"] == "kan" else 0)
    if c["kind"] == "batched":
        D = float(4 ** n)
        return {"bytes": 60 * (2 + 10) * D * el, "flops": 60 * (2 * hops + 40) * D}
    D = float(_dim(c))
    if c["kind"] == "apply":
        return {"bytes": 2 * D * el, "flops": 2 * hops * D}
    if c["kind"] == "green":
        Dp = math.comb(n, c["nup"] + 1) * math.comb(n, c["ndn"])
        Dm = math.comb(n, c["nup"] - 1) * math.comb(n, c["ndn"])
        return {"bytes": (2 + 4) * c["m"] * float(Dp + Dm) * el, "flops": c["m"] * (2 * hops + 10) * float(Dp + Dm)}
    steps = 60 * c.get("k", 1)
    return {"bytes": steps * (2 + 10) * D * el, "flops": steps * (2 * hops + 40) * D}


# ------------------------------------------------------------------- exact ----

def _states(ns, n):
    s = torch.arange(1 << ns, dtype=torch.int64, device=DEV)
    c = torch.zeros_like(s)
    for i in range(ns):
        c += (s >> i) & 1
    return s[c == n]


def _move(st, dst, src):
    """(rows reached, rows left, sign) of c+_dst c_src on one spin's states."""
    f = torch.nonzero((((st >> src) & 1) == 1) & (((st >> dst) & 1) == 0)).reshape(-1)
    s = st[f]
    lo, hi = min(src, dst), max(src, dst)
    par = torch.zeros_like(s)
    for i in range(lo + 1, hi):
        par += (s >> i) & 1
    t = torch.searchsorted(st, s ^ (1 << src) ^ (1 << dst))
    return t, f, (1 - 2 * (par & 1)).to(torch.float64)


class _Exact:
    """H of one sector as operator strings, in 64 bits."""

    def __init__(self, p, nup, ndn):
        ns = int(p["Ns"])
        self.st = [_states(ns, nup), _states(ns, ndn)]
        self.shape = (len(self.st[0]), len(self.st[1]))
        self.D = self.shape[0] * self.shape[1]
        occ = [torch.stack([((st >> i) & 1).to(torch.float64) for i in range(ns)], 1) for st in self.st]
        self.e = []
        for s in range(2):
            w = torch.from_numpy(np.asarray(p["w_ss"][s])).to(DEV)
            eps = torch.from_numpy(np.asarray(p["eps"][s])).to(DEV)
            self.e.append(occ[s] @ eps + ((occ[s] @ w) * occ[s]).sum(1))
        self.nw = occ[0] @ torch.from_numpy(np.asarray(p["w_ud"])).to(DEV)
        self.nd = occ[1].t().contiguous()
        self.hops = [[], []]
        for s in range(2):
            for i in range(ns):
                for j in range(ns):
                    h = float(p["hop"][s][i][j])
                    if i != j and h != 0.0:
                        t, f, g = _move(self.st[s], i, j)
                        self.hops[s].append((t, f, h * g))
        self.x = []
        for typ, m, mp, coef in p["xterms"]:
            # both printed strings equal minus (up move mp -> m) (down move): see the anticommutations
            a = _move(self.st[0], m, mp)
            b = _move(self.st[1], mp, m) if typ == models.SPIN_FLIP else _move(self.st[1], m, mp)
            self.x.append((a, b, -float(coef)))

    def apply(self, x):
        X = x.reshape(self.shape)
        Y = torch.empty_like(X)
        rows = max(1, (1 << 27) // self.shape[1])
        for r in range(0, self.shape[0], rows):
            q = slice(r, r + rows)
            Y[q] = (self.nw[q] @ self.nd + self.e[0][q, None] + self.e[1][None, :]) * X[q]
        for t, f, a in self.hops[0]:
            for r in range(0, len(t), rows):
                q = slice(r, r + rows)
                Y[t[q]] += a[q, None] * X[f[q]]
        for t, f, a in self.hops[1]:
            for r in range(0, self.shape[0], rows):
                Y[r:r + rows].index_add_(1, t, X[r:r + rows].index_select(1, f) * a)
        for (tu, fu, su), (td, fd, sd), c in self.x:
            for r in range(0, len(tu), rows):
                q = slice(r, r + rows)
                V = X[fu[q]].index_select(1, fd) * (c * su[q, None] * sd[None, :])
                Z = Y[tu[q]]
                Z.index_add_(1, td, V)
                Y[tu[q]] = Z
        return Y.reshape(-1)


def _lanczos(H, v0, steps, locked=(), tol=1e-13):
    """Fully reorthogonalised Lanczos from v0; stops when the lowest Ritz pair has converged to tol."""
    V = torch.empty((min(steps, H.D - len(locked)) + 1, H.D), dtype=torch.float64, device=DEV)

    def clean(w, k):
        for _ in range(2):
            for l in locked:
                w = w - l * torch.dot(l, w)
            if k:
                w = w - V[:k].t() @ (V[:k] @ w)
        return w
    w = clean(v0.clone(), 0)
    n0 = float(torch.linalg.vector_norm(w))
    V[0] = w / n0
    al, be = [], []
    for j in range(V.shape[0] - 1):
        w = H.apply(V[j])
        al.append(float(torch.dot(V[j], w)))
        w = clean(w, j + 1)
        b = float(torch.linalg.vector_norm(w))
        be.append(b)
        if b < 1e-12 or j == V.shape[0] - 2:
            break
        if tol and j % 8 == 7:
            t, z = np.linalg.eigh(np.diag(al) + np.diag(be[:j], 1) + np.diag(be[:j], -1))
            if abs(b * z[-1, 0]) < tol * max(1.0, abs(t[0])):
                break
        V[j + 1] = w / b
    k = len(al)
    t, z = np.linalg.eigh(np.diag(al) + np.diag(be[:k - 1], 1) + np.diag(be[:k - 1], -1))
    z0 = z[:, 0] * (1.0 if z[0, 0] >= 0 else -1.0)
    psi = torch.from_numpy(z0).to(DEV) @ V[:k]
    return t[0], psi / torch.linalg.vector_norm(psi), al, be, n0 * n0


def _resolvent(H, phi, m, e0, sign, z):
    if float(torch.linalg.vector_norm(phi)) == 0.0:
        return 0.0 * z
    _, _, al, be, n2 = _lanczos(H, phi, m, tol=0.0)
    d = z - sign * (al[-1] - e0)
    for a, b in zip(reversed(al[:-1]), reversed(be[:len(al) - 1])):
        d = z - sign * (a - e0) - b * b / d
    return n2 / d


def _ladder(Hs, Hd, dagger, psi):
    """c+_0 or c_0 of spin up: site 0 is the first mode, so there is no sign."""
    out = torch.zeros(Hd.shape, dtype=torch.float64, device=DEV)
    f = torch.nonzero((Hs.st[0] & 1) == (0 if dagger else 1)).reshape(-1)
    out[torch.searchsorted(Hd.st[0], Hs.st[0][f] ^ 1)] = psi.reshape(Hs.shape)[f]
    return out.reshape(-1)


def exact(case, seed):
    c = case
    p = models.params_from_model(_model(c, seed))
    if c["kind"] == "batched":
        n = c["size"]
        if n > 7:
            return None   # minutes, one sector after another
        e = []
        for a in range(n + 1):
            for b in range(n + 1):
                H = _Exact(p, a, b)
                e.append(_lanczos(H, _vector(H.D, torch.float64, 1), 120)[0])
        return np.array(e)
    if c["kind"] != "apply" and _dim(c) > 1.0e6:
        return None
    H = _Exact(p, c["nup"], c["ndn"])
    if c["kind"] == "apply":
        x = _vector(H.D, _dtype(c), seed).double()
        if c["order"] == "rank" or c["model"] == "hub":
            return H.apply(x)
        # the grouped order is a reordering of each spin's states
        g = _ham(p, c["nup"], c["ndn"], _prec(c)).grouped()
        if g is None:
            return H.apply(x)
        pu, pd = (torch.from_numpy(g.grouped_order(s)).to(DEV).long() for s in range(2))
        del g
        X = torch.empty(H.shape, dtype=torch.float64, device=DEV)
        X[:, pd] = x.reshape(H.shape)
        iu = torch.empty_like(pu)
        iu[pu] = torch.arange(len(pu), device=DEV)
        Y = H.apply(X[iu].reshape(-1)).reshape(H.shape)
        del X
        return Y[pu].index_select(1, pd).reshape(-1)
    v0 = _vector(H.D, _dtype(c) if c["kind"] != "green" else torch.float64, seed).double()
    if c["kind"] == "ground":
        e, psi, _, _, _ = _lanczos(H, v0, 400)
        # the sign an implicit restart leaves is not fixed by the start vector
        return {"E": e, "psi": psi if c["keep"] == 0 and c["prec"] == "fp64" else None}
    if c["kind"] == "lowest":
        e, lock = [], []
        for i in range(c["k"]):
            t, psi, _, _, _ = _lanczos(H, v0 if i == 0 else _vector(H.D, torch.float64, i), 400, lock)
            e.append(t)
            lock.append(psi)
        return np.sort(np.array(e))
    e0, psi, _, _, _ = _lanczos(H, v0, 400)
    if c["prec"] == "fp32":
        psi = psi.float().double()
    z, g = _matsubara(), 0.0
    for d, sign in ((1, 1), (-1, -1)):
        Hx = _Exact(p, c["nup"] + d, c["ndn"])
        g = g + _resolvent(Hx, _ladder(H, Hx, d == 1, psi), min(c["m"], Hx.D), e0, sign, z)
    return g
