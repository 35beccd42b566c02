"""Timed cases of the library: what its users call, over the sizes they call it with.

Every case names an entry point ("do"), a lattice, a sector (n_up, n_dn) and the
options of the call.  Lattices: "ring" (lx sites), "torus" (lx x ly, periodic),
"tprime" (the torus with both diagonals at t' = -0.3: two amplitude classes) and
"random" (a ring with an amplitude of its own on every bond).  The sectors are
those of the benchmark and the tests: the 8-site and 14-site rings, the 3 x 4 and
4 x 4 tori, and the 10 to 12 site rings of a batch.

prepare() builds the handles and makes the vectors from the seed on the device,
run() is one call, exact() the same quantity from plain torch and numpy in 64
bits (its own basis, its own Lanczos iteration).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1204_3425_amd as hb

DEV = "cuda"


# ------------------------------------------------------------------ lattices

def _bonds(case):
    """(edges, amplitudes or None) of a case's lattice."""
    kind, lx, ly = case["lattice"], case["lx"], case["ly"]
    if kind in ("ring", "random"):
        pairs = [(i, (i + 1) % lx) for i in range(lx)]
    else:
        pairs = []
        for y in range(ly):
            for x in range(lx):
                pairs += [(x + lx * y, (x + 1) % lx + lx * y), (x + lx * y, x + lx * ((y + 1) % ly))]
    nn = _unique(pairs)
    if kind == "random":
        return nn, np.random.RandomState(lx).uniform(0.5, 1.5, len(nn)).tolist()
    if kind != "tprime":
        return nn, None
    diag = []
    for y in range(ly):
        for x in range(lx):
            diag += [(x + lx * y, (x + 1) % lx + lx * ((y + s) % ly)) for s in (1, -1)]
    both = _unique(nn + diag)
    return both, [1.0] * len(nn) + [-0.3] * (len(both) - len(nn))


def _unique(pairs):
    seen, out = set(), []
    for i, j in pairs:
        key = (min(i, j), max(i, j))
        if i != j and key not in seen:
            seen.add(key)
            out.append((i, j))
    return out


def _sites(case):
    return case["lx"] * case["ly"]


def _dims(case):
    n = _sites(case)
    return math.comb(n, case["n_up"]), math.comb(n, case["n_dn"])


# --------------------------------------------------------------------- cases

def _case(name, do, lattice, lx, ly, n_up, n_dn, U, **more):
    return dict(name=name, do=do, lattice=lattice, lx=lx, ly=ly, n_up=n_up, n_dn=n_dn, U=U, **more)


def listed():
    return [
        # y = H x as a caller's own iteration drives it: the smallest sector in
        # use (one call is launches and host work), 11.8 million states in
        # single precision, and the largest, 165.6 million states in double
        _case("apply_ring8_fp64", "apply", "ring", 8, 1, 4, 4, 4.0, mixed=False),
        _case("apply_ring14_fp32", "apply", "ring", 14, 1, 7, 7, 4.0, mixed=True),
        _case("apply_4x4_fp64", "apply", "torus", 4, 4, 8, 8, 8.0, mixed=False),
        # the same call with an amplitude per bond: the t-t' square lattice away
        # from half filling, and disordered hopping on an odd sector
        _case("apply_4x4_tprime_fp64", "apply", "tprime", 4, 4, 6, 6, 6.0, mixed=False),
        _case("apply_ring14_random_fp64", "apply", "random", 14, 1, 7, 6, 4.0, mixed=False),
        # a ground state with its vector, from the energy test's own stop: a
        # teaching-size ring, and the sector a parameter scan runs thousands of times
        _case("solve_ring8_fp64", "solve", "ring", 8, 1, 4, 4, 4.0, steps=35),
        _case("solve_3x4_fp64", "solve", "torus", 3, 4, 6, 6, 4.0, steps=75),
        # a fixed count of Lanczos steps of the largest sector, energy and coefficients only
        _case("steps_4x4_fp64", "steps", "torus", 4, 4, 8, 8, 8.0, steps=20),
        # the lowest states of one sector (the gap and the levels above it)
        _case("lowest4_3x4_fp64", "lowest", "torus", 3, 4, 4, 4, 4.0, k=4, steps=90),
        # site densities and correlations of a state
        _case("observables_4x4", "observables", "torus", 4, 4, 6, 6, 6.0),
        # real-time evolution of a complex state
        _case("propagate_3x4", "propagate", "torus", 3, 4, 6, 5, 4.0, n_steps=4, krylov=16),
        # many small solves in one call (a sweep over U and the filling), mixed precision
        _case("batch64_rings_mixed", "batch", "ring", 12, 1, 6, 6, 8.0, count=64, mixed=True, steps=60),
    ]


def _sectors(do):
    """Lattices and sectors that draw() chooses from, with the bounds of the sector size."""
    rings = [("ring", n, 1, u, d) for n in range(8, 15) for u in range(n // 2 - 2, n // 2 + 1)
             for d in range(n // 2 - 2, n // 2 + 1)]
    t34 = [("torus", 3, 4, u, d) for u in range(3, 9) for d in range(3, 9)]
    t44 = [("torus", 4, 4, u, d) for u in range(3, 9) for d in range(3, 9)]
    if do == "apply":
        return rings + t34 + t44, 4900, 100e6
    if do == "bonds":
        tp = [("tprime", 4, 4, u, d) for u in range(3, 7) for d in range(3, 7)]
        tp += [("tprime", 3, 4, u, d) for u in range(3, 7) for d in range(3, 7)]
        rd = [("random", n, 1, u, d) for n in range(10, 15) for u in range(n // 2 - 2, n // 2 + 1)
              for d in range(n // 2 - 2, n // 2 + 1)]
        return tp + rd, 20e3, 64e6
    if do == "solve":
        return rings + t34, 1000, 12e6
    if do == "steps":
        return t44, 1e6, 100e6
    if do == "lowest":
        return rings + t34, 1000, 1e6
    if do == "propagate":
        return rings + t34, 4900, 1e6
    return rings + t34 + t44, 4900, 64e6  # observables


def draw(rng):
    do = rng.choice(["apply", "apply", "bonds", "solve", "steps", "lowest", "observables", "propagate", "batch"])
    U = round(rng.uniform(2.0, 10.0), 3)
    if do == "batch":
        return dict(do="batch", lattice="ring", lx=12, ly=1, n_up=6, n_dn=6, U=U, count=rng.randint(9, 63),
                    mixed=rng.random() < 0.5, steps=60)
    pool, lo, hi = _sectors(do)
    target = rng.uniform(math.log(lo), math.log(hi))

    def off(s):
        n = s[1] * s[2]
        return abs(math.log(math.comb(n, s[3]) * math.comb(n, s[4])) - target)

    near = sorted(pool, key=off)[:6]
    kind, lx, ly, nu, nd = rng.choice(near)
    c = dict(do="apply" if do == "bonds" else do, lattice=kind, lx=lx, ly=ly, n_up=nu, n_dn=nd, U=U)
    if do in ("apply", "bonds"):
        c["mixed"] = rng.random() < 0.4
    elif do == "solve":
        c["steps"] = 75
    elif do == "steps":
        c["steps"] = rng.randint(10, 20)
    elif do == "lowest":
        c.update(k=rng.randint(2, 4), steps=90)
    elif do == "propagate":
        c.update(n_steps=rng.randint(1, 4), krylov=rng.randint(10, 20))
    return c


# ------------------------------------------------------- inputs and the call

TOL = 1e-10     # energy test of the solves
MAX_ITER = 400


def _build(case):
    edges, amps = _bonds(case)
    if amps is not None:
        return hb.hubbard_build_bonds(_sites(case), edges, amps, case["n_up"], case["n_dn"], case["U"])
    return hb.hubbard_build(_sites(case), edges, case["n_up"], case["n_dn"], 1.0, case["U"])


def _uniform(n, seed, dtype=torch.float64):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.rand(n, generator=g, device=DEV, dtype=dtype).mul_(2).sub_(1)


def _batch_cases(case, seed):
    """The solves of a batch: rings of 10 to 12 sites at and below half filling, U in [0, 2 U]."""
    r = np.random.RandomState(seed % (2**31))
    out = []
    for i in range(case["count"]):
        n = int(r.randint(10, 13))
        out.append(dict(lattice="ring", lx=n, ly=1, n_up=int(r.randint(n // 2 - 2, n // 2 + 1)),
                        n_dn=int(r.randint(n // 2 - 2, n // 2 + 1)), U=float(r.uniform(0.0, 2.0 * case["U"]))))
    return out


def prepare(case, seed):
    do = case["do"]
    st = {"case": case, "seed": seed}
    if do == "batch":
        st["hs"] = [_build(c) for c in _batch_cases(case, seed)]
        st["seeds"] = [seed + i for i in range(case["count"])]
        return st
    h = st["h"] = _build(case)
    if do == "apply":
        hb.hubbard_set_precision(h, hb.HUBBARD_MIXED if case["mixed"] else hb.HUBBARD_FP64)
        st["x"] = _uniform(h.dim, seed, torch.float32 if case["mixed"] else torch.float64)
        st["y"] = torch.empty_like(st["x"])
    elif do == "solve":
        st["psi"] = torch.empty(h.dim, dtype=torch.float64, device=DEV)
    elif do == "lowest":
        st["psi"] = torch.empty((case["k"], h.dim), dtype=torch.float64, device=DEV)
    elif do == "observables":
        st["psi"] = _uniform(h.dim, seed)
        st["psi"] /= st["psi"].norm()
    elif do == "propagate":
        st["re"], st["im"] = _uniform(h.dim, seed), _uniform(h.dim, seed + 1)
        nrm = torch.sqrt(st["re"].square().sum() + st["im"].square().sum())
        st["re"] /= nrm
        st["im"] /= nrm
    return st


def run(st):
    case, do = st["case"], st["case"]["do"]
    if do == "apply":
        hb.hubbard_apply(st["h"], st["x"], st["y"])
        return st["y"]
    if do == "solve":
        r = hb.hubbard_lanczos_ex(st["h"], tol=TOL, max_iter=MAX_ITER, seed=st["seed"], psi=st["psi"], history=False)
        return {"E0": r["E0"], "psi": st["psi"]}
    if do == "steps":
        r = hb.hubbard_lanczos_ex(st["h"], tol=-1.0, max_iter=case["steps"], seed=st["seed"])
        return {"E0": r["E0"], "a": r["a"], "b": r["b"], "e": r["e_hist"]}
    if do == "lowest":
        E, _ = hb.hubbard_lowest_states(st["h"], case["k"], tol=TOL, max_iter=MAX_ITER, seed=st["seed"], psi=st["psi"])
        return {"E": E, "psi": st["psi"]}
    if do == "observables":
        return hb.hubbard_observables(st["h"], st["psi"])
    if do == "propagate":
        r = hb.hubbard_propagate(st["h"], st["re"], st["im"], 0.1 * case["n_steps"], case["n_steps"], case["krylov"])
        return {"re": st["re"], "im": st["im"], "energy": r["energy"]}
    rs = hb.hubbard_lanczos_batch(st["hs"], tol=TOL, max_iter=MAX_ITER, seeds=st["seeds"],
                                  precision=hb.HUBBARD_MIXED if case["mixed"] else hb.HUBBARD_FP64)
    return {"E0": np.array([r["E0"] for r in rs])}


def work(case):
    """One pass's least traffic and arithmetic: an H.v reads x and writes y, a
    Lanczos step reads the two vectors of the recurrence and writes one, a
    resident basis is read once more for the state, a propagation works on two halves."""
    do = case["do"]
    if do == "batch":
        tot = {"bytes": 0.0, "flops": 0.0}
        for c in _batch_cases(case, 1):
            w = work(dict(c, do="steps", steps=case["steps"]))
            tot["bytes"] += w["bytes"] * (0.5 if case["mixed"] else 1.0)
            tot["flops"] += w["flops"]
        return tot
    du, dd = _dims(case)
    dim, es = float(du) * dd, 4 if case.get("mixed") else 8
    n, ne = _sites(case), len(_bonds(case)[0])

    def hops(k):
        return 2.0 * ne * math.comb(n - 2, k - 1) / math.comb(n, k) if 0 < k < n else 0.0

    hv = dim * (2 * (hops(case["n_up"]) + hops(case["n_dn"])) + 2)
    if do == "apply":
        return {"bytes": 2 * dim * es, "flops": hv}
    if do == "steps":
        return {"bytes": 3 * dim * es * case["steps"], "flops": (hv + 8 * dim) * case["steps"]}
    if do == "solve":
        return {"bytes": 4 * dim * es * case["steps"], "flops": (hv + 10 * dim) * case["steps"]}
    if do == "lowest":
        k = case["k"]
        return {"bytes": (4 * k + k * (k - 1) / 2) * dim * es * case["steps"],
                "flops": (k * (hv + 10 * dim) + 4 * dim * k * (k - 1) / 2) * case["steps"]}
    if do == "observables":
        return {"bytes": dim * es, "flops": 2 * dim * n}
    m = case["n_steps"] * case["krylov"]
    return {"bytes": 2 * 4 * dim * es * m, "flops": 2 * (hv + 12 * dim) * m}


# --------------------------------------------- the same in plain 64-bit torch

class _Ref:
    """H of one sector as index arrays over the dim_up x dim_dn view."""

    def __init__(self, case):
        n = _sites(case)
        edges, amps = _bonds(case)
        self.dev = DEV if torch.cuda.is_available() else "cpu"
        words = np.arange(1 << n, dtype=np.int64)
        pop = np.zeros(1 << n, dtype=np.int64)
        for i in range(n):
            pop += (words >> i) & 1
        self.hop, self.bits = [], []
        for k in (case["n_up"], case["n_dn"]):
            s = words[pop == k]
            rank = np.zeros(1 << n, dtype=np.int64)
            rank[s] = np.arange(len(s))
            per = []
            for b, (i, j) in enumerate(edges):
                lo, hi = min(i, j), max(i, j)
                at = np.nonzero(((s >> i) & 1) != ((s >> j) & 1))[0]
                to = rank[s[at] ^ ((1 << i) | (1 << j))]
                between = s[at] & (((1 << hi) - 1) ^ ((1 << (lo + 1)) - 1))
                f = -(1.0 if amps is None else amps[b]) * (1.0 - 2.0 * (pop[between] & 1))
                per.append(tuple(torch.from_numpy(v).to(self.dev) for v in (at, to, f)))
            self.hop.append(per)
            self.bits.append(torch.from_numpy(np.stack([(s >> i) & 1 for i in range(n)])).to(self.dev, torch.float64))
        self.du, self.dd = (b.shape[1] for b in self.bits)
        self.dim, self.U = self.du * self.dd, case["U"]

    def apply(self, x):
        x = x.view(self.du, self.dd)
        y = torch.empty_like(x)
        for r in range(0, self.du, 2048):  # U times the doubly occupied sites
            y[r:r + 2048] = self.U * (self.bits[0][:, r:r + 2048].T @ self.bits[1]) * x[r:r + 2048]
        for at, to, f in self.hop[0]:
            for r in range(0, len(at), 2048):
                y[at[r:r + 2048]] += f[r:r + 2048, None] * x[to[r:r + 2048]]
        for r in range(0, self.du, 2048):
            for at, to, f in self.hop[1]:
                y[r:r + 2048].index_add_(1, at, f * x[r:r + 2048].index_select(1, to))
        return y.view(-1)

    def start(self, seed):
        """2 u - 1 with u from SplitMix64's output J + 1."""
        out = torch.empty(self.dim, dtype=torch.float64, device=self.dev)
        with np.errstate(over="ignore"):
            for a in range(0, self.dim, 1 << 24):
                b = min(self.dim, a + (1 << 24))
                z = np.uint64(seed) + np.arange(a + 1, b + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
                z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
                z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
                z ^= z >> np.uint64(31)
                out[a:b] = torch.from_numpy(2.0 * ((z >> np.uint64(11)).astype(np.float64) * 2.0**-53) - 1.0)
        return out

    def lanczos(self, f1, tol, steps, lower=(), vector=True):
        """E0, psi, a, b, E_j of the three-term iteration, every vector projected off `lower`."""
        def off(q):
            for p in lower:
                q = q - (p @ q) * p
            return q

        f = off(f1 / f1.norm())
        f = first = f / f.norm()
        prev, beta, a, b, e, kept = None, 0.0, [], [], [], []
        while True:
            if vector:
                kept.append(f)
            q = self.apply(f)
            if prev is not None:
                q -= beta * prev
            al = float(q @ f)
            q = off(q.sub_(al * f))
            beta = float(q.norm())
            a.append(al)
            b.append(beta)
            w, v = np.linalg.eigh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
            e.append(w[0])
            if (tol >= 0 and len(e) > 1 and abs(e[-1] - e[-2]) <= tol * max(1.0, abs(e[-1]))) or len(a) == steps:
                break
            prev, f = f, q / beta
        if not vector:
            return e[-1], None, a, b, e
        psi = sum(float(c) * g for c, g in zip(v[:, 0], kept))
        psi = off(psi)
        psi = psi / psi.norm()
        return e[-1], psi if float(psi @ first) > 0 else -psi, a, b, e


def exact(case, seed):
    do = case["do"]
    if do == "batch":
        E = []
        for i, c in enumerate(_batch_cases(case, seed)):
            ref = _Ref(c)
            E.append(ref.lanczos(ref.start(seed + i), 1e-13, MAX_ITER, vector=False)[0])
        return {"E0": np.array(E)}
    ref = _Ref(case)
    if do == "apply":
        return ref.apply(_uniform(ref.dim, seed, torch.float32 if case["mixed"] else torch.float64).double())
    if do == "solve":
        E0, psi, *_ = ref.lanczos(ref.start(seed), TOL, MAX_ITER)
        return {"E0": float(E0), "psi": psi}
    if do == "steps":
        E0, _, a, b, e = ref.lanczos(ref.start(seed), -1.0, case["steps"], vector=False)
        return {"E0": float(E0), "a": np.array(a), "b": np.array(b), "e": np.array(e)}
    if do == "lowest":
        E, psis = [], []
        for i in range(case["k"]):
            e0, psi, *_ = ref.lanczos(ref.start(seed + i), TOL, MAX_ITER, psis)
            E.append(e0)
            psis.append(psi)
        return {"E": np.array(E), "psi": torch.stack(psis)}
    if do == "observables":
        psi = _uniform(ref.dim, seed)
        psi /= psi.norm()
        w = psi.square().view(ref.du, ref.dd)
        u, d = ref.bits
        ru, rd = w.sum(1), w.sum(0)
        tot = float(ru.sum())
        ud = (u @ (w @ d.T)) / tot
        corr = torch.stack([(u * ru) @ u.T / tot, (d * rd) @ d.T / tot, ud])
        return {"dens": torch.stack([u @ ru, d @ rd]) / tot, "corr": corr, "docc": float(ud.diagonal().sum())}
    re, im = _uniform(ref.dim, seed), _uniform(ref.dim, seed + 1)
    nrm = torch.sqrt(re.square().sum() + im.square().sum())
    re, im = re / nrm, im / nrm
    energy = []
    for k in range(case["n_steps"] + 1):
        energy.append(float((re @ ref.apply(re) + im @ ref.apply(im)) / (re @ re + im @ im)))
        if k == case["n_steps"]:
            break
        for _ in range(2):  # exp(-i H dt) by its power series, dt = 0.05
            tr, ti = re, im
            for m in range(1, 60):
                tr, ti = ref.apply(ti) * (0.05 / m), ref.apply(tr) * (-0.05 / m)
                re, im = re + tr, im + ti
                if float(tr.norm() + ti.norm()) < 1e-18:
                    break
    return {"re": re, "im": im, "energy": np.array(energy)}
