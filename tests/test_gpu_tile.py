"""The one-launch H.v of small and medium sectors at its edges, and the Lanczos
and Krylov steps built on it, against the oracle.

Shapes: rows of one element, of little more than one wave and of little more than
one pass of the workgroup, a single row and few rows (several
workgroups share a row's columns), up rows of no hop, of fewer than the eight
hops loaded ahead and of more than sixteen, odd dense rows and strided rows in
both precisions, and per-bond handles (entries in slots of one amplitude each)
with two classes, with a class per bond, and with more than 16 slots.

Tolerance as for every H.v of this library: FP64 1e-13 of the largest element;
FP32 (terms + 1) 2^-24 times the largest sum of magnitudes a row can have.
"""
import itertools
import math

import numpy as np
import pytest

import oracle
import workload

torch = pytest.importorskip("torch")
hb = pytest.importorskip("paper_1204_3425_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _complete(n):
    return [(i, j) for i in range(n) for j in range(i + 1, n)]


def _amps(edges, classes, seed):
    v = np.random.default_rng(seed).uniform(-1.5, 1.5, classes)
    return [float(v[k % classes]) for k in range(len(edges))]


CASES = [
    # name, sites, edges, n_up, n_dn, amplitude classes (0: one amplitude)
    ("one_column", 12, workload.ring(12), 6, 0, 0),
    ("one_row", 12, workload.ring(12), 0, 6, 0),
    ("one_state", 4, workload.ring(4), 0, 4, 0),
    ("66_columns", 12, workload.torus(3, 4), 5, 2, 0),
    ("84_columns", 9, workload.chain(9), 4, 3, 0),
    ("few_rows", 15, workload.ring(15), 1, 7, 0),               # 15 rows of 6,435 columns: shared rows
    ("two_spans", 13, workload.ring(13), 2, 4, 0),              # 78 rows of 715 columns
    ("odd_3432x3003", 14, workload.ring(14), 7, 6, 0),
    ("wide_row", 16, workload.torus(4, 4), 2, 8, 0),            # FP64 rows of more than half the LDS
    ("up_rows_of_36", 12, _complete(12), 6, 2, 0),
    ("up_rows_of_72", 17, _complete(17), 8, 1, 0),
    ("two_classes", 12, workload.torus(3, 4), 4, 5, 2),
    ("class_per_bond", 11, workload.ring(11), 5, 6, 11),
    ("66_slots", 12, _complete(12), 3, 5, 66),
    ("class_per_bond_few_rows", 13, workload.ring(13), 1, 6, 13),
]


@pytest.mark.parametrize("precision", [hb.HUBBARD_FP64, hb.HUBBARD_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name,sites,edges,nu,nd,ncls", CASES, ids=[c[0] for c in CASES])
def test_one_launch_apply(name, sites, edges, nu, nd, ncls, precision):
    print("tile", name, precision, flush=True)
    U = 3.0
    amps = _amps(edges, ncls, sites) if ncls else None
    h = hb.hubbard_build_bonds(sites, edges, amps, nu, nd, U) if amps else hb.hubbard_build(sites, edges, nu, nd, 1.0, U)
    m = oracle.Model(sites, edges, nu, nd, amps if amps else 1.0, U)
    hb.hubbard_set_precision(h, precision)
    info = hb.hubbard_info(h)
    dt = torch.float64 if precision == hb.HUBBARD_FP64 else torch.float32
    x = workload.random_vector(h.dim, 77).astype(np.float64 if precision == hb.HUBBARD_FP64 else np.float32)
    ref = m.apply(x.astype(np.float64))
    if precision == hb.HUBBARD_FP64:
        tol = 1e-13 * max(1.0, np.abs(ref).max())
    else:
        terms = 1 + info["w_up"] + info["w_dn"]
        big = max(abs(U) * sites, max(map(abs, amps)) if amps else 1.0)
        tol = terms * 2.0**-24 * big * terms * np.abs(x).max()
    xd = torch.from_numpy(x).to(DEV)
    y = torch.full_like(xd, 7.0)
    hb.hubbard_apply(h, xd, y)
    torch.cuda.synchronize()
    assert np.abs(y.double().cpu().numpy() - ref).max() <= tol
    # strided rows (where the handle takes them): the same bits, the padding untouched
    if amps and ncls > 4:
        return
    for ld in (h.dim_dn + 3, info["ld_pref"]):
        xs = torch.full((h.dim_up, ld), float("nan"), dtype=dt, device=DEV)
        xs[:, :h.dim_dn] = xd.view(h.dim_up, h.dim_dn)
        ys = torch.full((h.dim_up, ld + 2), -5.0, dtype=dt, device=DEV)
        hb.hubbard_apply_ld(h, xs, ld, ys, ld + 2)
        torch.cuda.synchronize()
        assert torch.equal(ys[:, :h.dim_dn].reshape(-1), y)
        assert bool((ys[:, h.dim_dn:] == -5.0).all())


def test_one_launch_apply_infinite_element():
    """An infinite element of x reaches exactly the rows and columns it hops to:
    slots past a row's last hop, which repeat that hop's row, add nothing."""
    h = hb.hubbard_build(10, workload.ring(10), 5, 4, 1.0, 0.0)
    m = oracle.Model(10, workload.ring(10), 5, 4, 1.0, 0.0)
    x = np.zeros(h.dim)
    x[h.dim // 3] = np.inf
    marker = np.zeros(h.dim)
    marker[h.dim // 3] = 1.0
    xd = torch.from_numpy(x).to(DEV)
    y = torch.empty_like(xd)
    hb.hubbard_apply(h, xd, y)
    torch.cuda.synchronize()
    got, want = y.cpu().numpy(), m.apply(marker)
    hit = want != 0.0
    hit[h.dim // 3] = False  # the element itself: 0 * inf in the interaction term
    assert np.array_equal(np.isinf(got) & hit, hit)
    assert np.array_equal(np.sign(got[hit]), np.sign(want[hit]))
    rest = ~hit
    rest[h.dim // 3] = False
    assert np.all(got[rest] == 0.0)


STEP_CASES = [
    # name, sites, edges, n_up, n_dn, amplitude classes
    ("ring8", 8, workload.ring(8), 4, 4, 0),
    ("odd_792x924", 12, workload.torus(3, 4), 5, 6, 0),
    # 4,845 rows: more partial sums than the update adds up itself
    ("4845_rows", 20, workload.ring(20), 4, 1, 0),
    ("few_rows_shared", 13, workload.ring(13), 1, 6, 0),
    # a class per bond: rows of 462 elements (not on 16 bytes when dense)
    ("class_per_bond", 11, workload.ring(11), 5, 6, 11),
]


@pytest.mark.parametrize("name,sites,edges,nu,nd,ncls", STEP_CASES, ids=[c[0] for c in STEP_CASES])
def test_one_launch_steps(name, sites, edges, nu, nd, ncls):
    """Twelve steps against the oracle's Alg. 1.  Each a_j, b_{j+1} carries the
    rounding of its sums, about sqrt(dim) eps of |H|, forward through the
    recurrence: 64 sqrt(dim) eps relative, as for every coefficient test.  The
    vectors kept in slots, in the three work vectors (basis limit 0) and moved
    from the one to the other in mid-run give the same bits."""
    print("steps", name, flush=True)
    amps = _amps(edges, ncls, sites) if ncls else None
    h = hb.hubbard_build_bonds(sites, edges, amps, nu, nd, 3.0) if amps else hb.hubbard_build(sites, edges, nu, nd, 1.0, 3.0)
    m = oracle.Model(sites, edges, nu, nd, amps if amps else 1.0, 3.0)
    ref = m.lanczos(oracle.start_vector(5, m.dim), tol=-1.0, max_iter=40, want_psi=True)
    psi = torch.empty(h.dim, dtype=torch.float64, device=DEV)
    r = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=40, seed=5, psi=psi)
    tol = 64 * np.sqrt(h.dim) * np.finfo(float).eps
    scale = np.abs(ref["a"][:12]).max() + ref["b"][:12].max()
    assert np.abs(r["a"][:12] - ref["a"][:12]).max() <= tol * scale
    assert np.abs(r["b"][:12] - ref["b"][:12]).max() <= tol * scale
    assert abs(r["E0"] - ref["E0"]) <= 1e-12 * max(1.0, abs(ref["E0"]))
    assert r["psi_resident"] == 1
    ld = (h.dim_dn + 63) // 64 * 64
    for limit in (0, 33 * h.dim_up * ld * 8):  # no slots; one chunk of 32 vectors for 40 steps
        hb.hubbard_set_basis_limit(h, limit)
        again = torch.empty_like(psi)
        q = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=40, seed=5, psi=again)
        assert q["psi_resident"] == 0
        assert np.array_equal(q["a"], r["a"]) and np.array_equal(q["b"], r["b"])
        assert float((again - psi).abs().max()) <= 1e-12
    # both precisions of one handle share its kept buffers
    mixed = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=12, seed=5, precision=hb.HUBBARD_MIXED)
    assert np.abs(mixed["a"] - ref["a"][:12]).max() <= 1e-4 * scale
    assert np.array_equal(hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=40, seed=5)["a"], r["a"])


@pytest.mark.parametrize("k", [2, 3, 4, 5, 7])
def test_one_launch_deflated_steps(k):
    """One to six lower states: one, two and up to four are projected out inside
    the two launches, more by the separate projection.  A ring of 9 sites with
    random amplitudes has no degenerate levels (spacing above 1e-3)."""
    print("deflated", k, flush=True)
    edges = workload.ring(9)
    amps = _amps(edges, 9, 31)
    h = hb.hubbard_build_bonds(9, edges, amps, 3, 2, 2.0)
    m = oracle.Model(9, edges, 3, 2, amps, 2.0)
    w, V = m.lowest_states(k)
    psi = torch.empty((k, h.dim), dtype=torch.float64, device=DEV)
    E, _ = hb.hubbard_lowest_states(h, k, tol=1e-14, max_iter=600, psi=psi)
    assert np.abs(E - w).max() <= 1e-10 * max(1.0, np.abs(w).max())
    P = psi.cpu().numpy()
    assert np.abs(P @ P.T - np.eye(k)).max() <= 1e-12


def test_one_launch_deflated_steps_rows_that_fill_the_lds():
    """Rows of 20,349 doubles leave 1,040 bytes of LDS, less than the sums of a step
    with four lower vectors take: one and two are projected out in the step's
    launches, three and four by their own.  Free fermions on an open chain, levels
    -2 cos(pi j / 22) (spacing of the lowest states above 0.04): energies within
    1e-10, orthonormal to 1e-12, residuals below 1e-6."""
    n, nu, nd, k = 21, 1, 5, 5
    print("deflated, 20,349 columns", flush=True)
    lv = [-2.0 * math.cos(math.pi * j / (n + 1)) for j in range(1, n + 1)]
    w = np.sort(np.add.outer(lv, [sum(c) for c in itertools.combinations(lv, nd)]).ravel())[:k]
    h = hb.hubbard_build(n, workload.chain(n), nu, nd, 1.0, 0.0)
    psi = torch.empty((k, h.dim), dtype=torch.float64, device=DEV)
    E, res = hb.hubbard_lowest_states(h, k, tol=1e-14, max_iter=800, psi=psi)
    assert np.abs(np.array(E) - w).max() <= 1e-10 * max(1.0, np.abs(w).max())
    P = psi.cpu().numpy()
    assert np.abs(P @ P.T - np.eye(k)).max() <= 1e-12
    assert max(r["residual"] for r in res) <= 1e-6


def test_one_launch_propagation_many_rows():
    """A Krylov step on 4,845 rows (the partial sums reduced first), against the
    power series of exp(-i H t) from the oracle's H.v (terms below 1e-17)."""
    h = hb.hubbard_build(20, workload.ring(20), 4, 1, 1.0, 3.0)
    m = oracle.Model(20, workload.ring(20), 4, 1, 1.0, 3.0)
    g = np.random.default_rng(3)
    psi = g.uniform(-1, 1, h.dim) + 1j * g.uniform(-1, 1, h.dim)
    psi /= np.linalg.norm(psi)
    want, term = psi.copy(), psi.copy()
    for n in range(1, 40):
        term = -1j * 0.1 / n * (m.apply(np.ascontiguousarray(term.real)) + 1j * m.apply(np.ascontiguousarray(term.imag)))
        want = want + term
        if np.linalg.norm(term) < 1e-17:
            break
    re, im = torch.from_numpy(psi.real.copy()).to(DEV), torch.from_numpy(psi.imag.copy()).to(DEV)
    r = hb.hubbard_propagate(h, re, im, 0.1, 1, 20)
    got = re.cpu().numpy() + 1j * im.cpu().numpy()
    assert r["err_est"] <= 1e-13
    assert np.linalg.norm(got - want) <= 1e-11


@pytest.mark.parametrize("ncls", [0, 2, 8], ids=["uniform", "two_classes", "class_per_bond"])
@pytest.mark.parametrize("e", [-498, -370, 370, 498])
def test_one_launch_steps_of_tiny_and_huge_couplings(e, ncls):
    """H scaled by a power of two scales every product and sum of a step exactly
    while all of them are normal numbers, and the squared norms are up to 2^+-500
    couplings: the coefficients, energies and the evolution over the scaled time
    are those of the unscaled H to rounding (the stop test, absolute below 1, is
    off; the vector of a scaled H is the same vector)."""
    print("couplings times 2 **", e, ncls, flush=True)
    f = 2.0**e
    edges = workload.ring(8)
    amps = _amps(edges, ncls, 8) if ncls else [1.0] * len(edges)
    got = []
    for c in (1.0, f):
        h = hb.hubbard_build_bonds(8, edges, [c * a for a in amps], 4, 3, 3.0 * c)
        psi = torch.empty(h.dim, dtype=torch.float64, device=DEV)
        r = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=30, seed=5, psi=psi)
        E, _ = hb.hubbard_lowest_states(h, 3, tol=-1.0, max_iter=30, seed=5)
        g = torch.Generator(device=DEV)
        g.manual_seed(4)
        re = torch.rand(h.dim, generator=g, dtype=torch.float64, device=DEV) - 0.5
        im = torch.rand(h.dim, generator=g, dtype=torch.float64, device=DEV) - 0.5
        p = hb.hubbard_propagate(h, re, im, 0.25 / c, 2, 16)
        got.append((r["a"] / c, r["b"] / c, psi.cpu().numpy(), E / c, re.cpu().numpy(), im.cpu().numpy(), p["energy"] / c))
    for one, scaled in zip(*got):
        assert np.abs(scaled - one).max() <= 1e-11 * max(1.0, np.abs(one).max())


def test_kept_buffers_two_streams_and_a_batch_of_one_handle():
    """A handle's kept buffers are not shared by work in flight: solves on two
    streams in turn, and the same handle several times in one batch."""
    h = hb.hubbard_build(10, workload.ring(10), 5, 5, 1.0, 4.0)
    psi = torch.empty(h.dim, dtype=torch.float64, device=DEV)
    first = hb.hubbard_lanczos_ex(h, tol=1e-10, seed=9, psi=psi)
    want = psi.clone()
    side = torch.cuda.Stream()
    for s in (side, torch.cuda.current_stream(), side):
        with torch.cuda.stream(s):
            psi.zero_()
            r = hb.hubbard_lanczos_ex(h, tol=1e-10, seed=9, psi=psi)
        s.synchronize()
        assert np.array_equal(r["a"], first["a"]) and torch.equal(psi, want)
    one = hb.hubbard_lanczos_batch([h], tol=1e-10, seeds=[9])[0]
    for r in hb.hubbard_lanczos_batch([h, h, h], tol=1e-10, seeds=[9, 9, 9]):
        assert r["E0"] == one["E0"] and r["n_iter"] == one["n_iter"]
