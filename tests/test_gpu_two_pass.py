"""The two-pass H.v where sectors are too large for the one-launch form, at rows
whose 128-byte slabs are whole lines, whole half lines, or neither (results then
stored through the L2), with counts of slabs that the eight XCDs do not share
evenly, in dense and strided rows: H.v and the first Lanczos steps against the
oracle.

Tolerance: H.v FP64 1e-13 of the largest element, FP32 (terms + 1) 2^-24 times the
largest sum of magnitudes of a row; coefficients 64 sqrt(dim) eps of |H|.
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

CASES = [
    # sites, edges, n_up, n_dn
    (17, workload.ring(17), 5, 5),       # 6,188 columns: FP64 rows on 32 bytes, 387 slabs
    (16, workload.torus(4, 4), 6, 5),    # 4,368 columns: on 128 bytes, 273 slabs
    (15, workload.torus(3, 5), 7, 6),    # 5,005 columns: dense rows on 8 bytes
    (16, workload.torus(4, 4), 5, 6),    # 8,008 columns: on 64 bytes
]


@pytest.mark.parametrize("sites,edges,nu,nd", CASES, ids=["6188", "4368", "5005", "8008"])
def test_two_pass_sectors(sites, edges, nu, nd):
    print("two pass", sites, nu, nd, flush=True)
    U = 3.0
    h = hb.hubbard_build(sites, edges, nu, nd, 1.0, U)
    assert h.dim * 8 > 192 << 20
    m = oracle.Model(sites, edges, nu, nd, 1.0, U)
    x = workload.random_vector(h.dim, 77).astype(np.float64)
    ref = m.apply(x)
    info = hb.hubbard_info(h)
    xd = torch.from_numpy(x).to(DEV)
    y = torch.full_like(xd, 7.0)
    hb.hubbard_apply(h, xd, y)
    torch.cuda.synchronize()
    assert np.abs(y.cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    ld = info["ld_pref"]
    xs = torch.full((h.dim_up, ld), float("nan"), dtype=torch.float64, device=DEV)
    xs[:, :h.dim_dn] = xd.view(h.dim_up, h.dim_dn)
    ys = torch.full((h.dim_up, ld + 2), -5.0, dtype=torch.float64, device=DEV)
    hb.hubbard_apply_ld(h, xs, ld, ys, ld + 2)
    torch.cuda.synchronize()
    assert torch.equal(ys[:, :h.dim_dn].reshape(-1), y)
    assert bool((ys[:, h.dim_dn:] == -5.0).all())
    # single precision
    hb.hubbard_set_precision(h, hb.HUBBARD_MIXED)
    y32 = torch.empty(h.dim, dtype=torch.float32, device=DEV)
    hb.hubbard_apply(h, xd.float(), y32)
    torch.cuda.synchronize()
    terms = 1 + info["w_up"] + info["w_dn"]
    ref32 = m.apply(x.astype(np.float32).astype(np.float64))
    assert np.abs(y32.double().cpu().numpy() - ref32).max() <= terms * 2.0**-24 * U * sites * terms * np.abs(x).max()
    # the fused step
    want = m.lanczos(oracle.start_vector(5, m.dim), tol=-1.0, max_iter=4)
    got = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=4, seed=5, precision=hb.HUBBARD_FP64)
    tol = 64 * np.sqrt(h.dim) * np.finfo(float).eps * (np.abs(want["a"]).max() + want["b"].max())
    assert np.abs(got["a"] - want["a"]).max() <= tol and np.abs(got["b"] - want["b"]).max() <= tol


def _two(edges, n):
    """The first n bonds at 1, the others at -0.3."""
    return [1.0] * n + [-0.3] * (len(edges) - n)


TPRIME, _ = workload.torus_tprime(4, 4, 1.0, -0.3)
CLASS_CASES = [
    # sites, edges, amplitudes, n_up, n_dn
    (16, TPRIME, _two(TPRIME, 32), 6, 5),                                    # even rows on 128 bytes
    (15, workload.torus(3, 5), _two(workload.torus(3, 5), 15), 7, 6),        # 6,435 rows; dense rows on 8 bytes
    (17, workload.ring(17), [1.0 if k % 2 else 0.6 for k in range(17)], 5, 6),  # 12,376 columns: FP64 pairs do not fit
    (16, TPRIME, _two(TPRIME, 63), 6, 5),                                    # more than 32 hops of one class
]


@pytest.mark.parametrize("sites,edges,amps,nu,nd", CLASS_CASES, ids=["tprime", "odd_rows", "long_rows", "uneven"])
def test_two_pass_two_classes(sites, edges, amps, nu, nd):
    """Two amplitude classes, sorted by class where a row's hops of each fit, else by
    the class bits of each entry; the residual of a short solve as well."""
    print("two classes", sites, nu, nd, flush=True)
    U = 3.0
    h = hb.hubbard_build_bonds(sites, edges, amps, nu, nd, U)
    assert h.dim * 8 > 192 << 20
    m = oracle.Model(sites, edges, nu, nd, amps, U)
    info = hb.hubbard_info(h)
    x = workload.random_vector(h.dim, 78).astype(np.float64)
    ref = m.apply(x)
    xd = torch.from_numpy(x).to(DEV)
    y = torch.full_like(xd, 7.0)
    hb.hubbard_apply(h, xd, y)
    torch.cuda.synchronize()
    assert np.abs(y.cpu().numpy() - ref).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    ld = info["ld_pref"]
    xs = torch.full((h.dim_up, ld), float("nan"), dtype=torch.float64, device=DEV)
    xs[:, :h.dim_dn] = xd.view(h.dim_up, h.dim_dn)
    ys = torch.full((h.dim_up, ld + 2), -5.0, dtype=torch.float64, device=DEV)
    hb.hubbard_apply_ld(h, xs, ld, ys, ld + 2)
    torch.cuda.synchronize()
    assert np.abs((ys[:, :h.dim_dn].reshape(-1) - y).cpu().numpy()).max() <= 1e-13 * max(1.0, np.abs(ref).max())
    assert bool((ys[:, h.dim_dn:] == -5.0).all())
    if h.dim * 4 > 192 << 20:
        hb.hubbard_set_precision(h, hb.HUBBARD_MIXED)
        y32 = torch.empty(h.dim, dtype=torch.float32, device=DEV)
        hb.hubbard_apply(h, xd.float(), y32)
        torch.cuda.synchronize()
        terms = 1 + info["w_up"] + info["w_dn"]
        ref32 = m.apply(x.astype(np.float32).astype(np.float64))
        assert np.abs(y32.double().cpu().numpy() - ref32).max() <= terms * 2.0**-24 * U * sites * terms * np.abs(x).max()
    want = m.lanczos(oracle.start_vector(5, m.dim), tol=-1.0, max_iter=4, want_psi=True)
    psi = torch.empty(h.dim, dtype=torch.float64, device=DEV)
    got = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=4, seed=5, precision=hb.HUBBARD_FP64, psi=psi)
    tol = 64 * np.sqrt(h.dim) * np.finfo(float).eps * (np.abs(want["a"]).max() + want["b"].max())
    assert np.abs(got["a"] - want["a"]).max() <= tol and np.abs(got["b"] - want["b"]).max() <= tol
    p = psi.cpu().numpy()
    res = np.linalg.norm(m.apply(p) - got["E0"] * p)
    assert abs(got["residual"] - res) <= 1e-9 * max(1.0, res)


DIAG = workload.torus_tprime(4, 4, 1.0, 1.0)[0]
ACROSS = [(i, 10 + j) for i in range(10) for j in range(10)]
STEP_CASES = [
    # sites, edges, n_up, n_dn, precision: the layouts of the up-spin entries
    (16, workload.torus(4, 4), 6, 5, hb.HUBBARD_FP64),   # one line of 32 slots
    (16, DIAG, 6, 5, hb.HUBBARD_FP64),                   # up rows of 48 hops: two lines
    (20, ACROSS, 10, 2, hb.HUBBARD_FP64),                # up rows of 100 hops: entries by block
    (16, workload.torus(4, 4), 6, 6, hb.HUBBARD_MIXED),
    (16, DIAG, 6, 6, hb.HUBBARD_MIXED),
    (20, ACROSS, 10, 3, hb.HUBBARD_MIXED),
]
IDS = ["line-fp64", "two_lines-fp64", "blocks-fp64", "line-mixed", "two_lines-mixed", "blocks-mixed"]


def _coefficients_agree(got, want, h, precision):
    scale = np.abs(want["a"]).max() + want["b"].max()
    tol = 1e-4 if precision == hb.HUBBARD_MIXED else 64 * np.sqrt(h.dim) * np.finfo(float).eps
    assert np.abs(got["a"] - want["a"]).max() <= tol * scale
    assert np.abs(got["b"] - want["b"]).max() <= tol * scale


@pytest.mark.parametrize("sites,edges,nu,nd,precision", STEP_CASES, ids=IDS)
def test_two_pass_steps_against_the_batched_engine(sites, edges, nu, nd, precision):
    """The fused two-pass step on sectors too large for the one-launch form against
    the batched engine's step, which shares no kernel with it.  The sign of site 0's
    orbital flipped turns the bonds of site 0 to -t, two amplitude classes, and the
    start vector with it: the coefficients stay."""
    print("two-pass steps", sites, nu, nd, precision, flush=True)
    h = hb.hubbard_build(sites, edges, nu, nd, 1.0, 3.0)
    assert h.dim * (8 if precision == hb.HUBBARD_FP64 else 4) > 160 << 20
    opt = dict(tol=-1.0, max_iter=12, precision=precision)
    want = hb.hubbard_lanczos_batch([h], seeds=[11], history=True, **opt)[0]
    _coefficients_agree(hb.hubbard_lanczos_ex(h, seed=11, **opt), want, h, precision)
    f = torch.empty(h.dim, dtype=torch.float64, device=DEV)
    hb.hubbard_start_raw(11, h.dim, f)
    flip = [torch.from_numpy(1.0 - 2.0 * (hb.hubbard_export_basis(h, s) & 1)).to(DEV) for s in (0, 1)]
    f.view(h.dim_up, h.dim_dn).mul_(flip[0][:, None]).mul_(flip[1][None, :])
    hb.hubbard_free(h)
    h = hb.hubbard_build_bonds(sites, edges, [-1.0 if 0 in e else 1.0 for e in edges], nu, nd, 3.0)
    _coefficients_agree(hb.hubbard_lanczos_ex(h, start=f, **opt), want, h, precision)


@pytest.mark.parametrize("sites,edges,nu,nd,precision", [STEP_CASES[0], STEP_CASES[2], STEP_CASES[3]],
                         ids=[IDS[0], IDS[2], IDS[3]])
def test_two_pass_psi_resident_replayed_and_moved(sites, edges, nu, nd, precision):
    """psi from the resident vectors (formed in their slots with entry lines, copied
    to them without), from the replay, and from a run that leaves its 32 slots
    midway: the coefficients bit for bit, the vectors to 1e-12."""
    print("two-pass psi", sites, nu, nd, precision, flush=True)
    h = hb.hubbard_build(sites, edges, nu, nd, 1.0, 3.0)
    ld, es = hb.hubbard_info(h)["ld_pref"], 8 if precision == hb.HUBBARD_FP64 else 4
    runs = []
    for limit in (2**62, 0, 33 * h.dim_up * ld * es):
        hb.hubbard_set_basis_limit(h, limit)
        psi = torch.empty(h.dim, dtype=torch.float64, device=DEV)
        r = hb.hubbard_lanczos_ex(h, tol=-1.0, max_iter=36, seed=5, precision=precision, psi=psi)
        assert r["psi_resident"] == (limit == 2**62)
        runs.append((r, psi))
    for r, psi in runs[1:]:
        assert np.array_equal(r["a"], runs[0][0]["a"]) and np.array_equal(r["b"], runs[0][0]["b"])
        assert float((psi - runs[0][1]).abs().max()) <= 1e-12


@pytest.mark.parametrize("nu,nd,k,precision", [(6, 5, 4, hb.HUBBARD_FP64), (7, 6, 3, hb.HUBBARD_MIXED)],
                         ids=["fp64", "mixed"])
def test_two_pass_deflated_steps(nu, nd, k, precision):
    """Lower states projected out of two-pass steps (one and two in the fused step,
    three by launches of their own): free fermions on an open chain of 16 sites,
    levels -2 cos(pi j / 17), no degenerate levels among the lowest.  Energies
    within 1e-10 (mixed 1e-6) of their size, FP64 states orthonormal to 1e-12."""
    print("two-pass deflated", nu, nd, k, precision, flush=True)
    lv = [-2.0 * math.cos(math.pi * j / 17) for j in range(1, 17)]
    low = [sorted(sum(c) for c in itertools.combinations(lv, n))[:k] for n in (nu, nd)]
    w = np.sort(np.add.outer(*low).ravel())[:k]
    h = hb.hubbard_build(16, workload.chain(16), nu, nd, 1.0, 0.0)
    fp64 = precision == hb.HUBBARD_FP64
    assert h.dim * (8 if fp64 else 4) > 160 << 20
    psi = torch.empty((k, h.dim), dtype=torch.float64, device=DEV)
    E, res = hb.hubbard_lowest_states(h, k, tol=1e-13 if fp64 else 1e-9, max_iter=600, precision=precision, psi=psi)
    assert np.abs(np.array(E) - w).max() <= (1e-10 if fp64 else 1e-6) * np.abs(w).max()
    if fp64:
        G = np.array([[float(torch.dot(psi[i], psi[j])) for j in range(k)] for i in range(k)])
        assert np.abs(G - np.eye(k)).max() <= 1e-12
        assert max(r["residual"] for r in res) <= 1e-4


@pytest.mark.parametrize("sites,edges,nu,nd,precision", STEP_CASES, ids=IDS)
def test_two_pass_apply_on_misaligned_vectors(sites, edges, nu, nd, precision):
    """Vectors that start one element past 16 bytes: the same product as on aligned
    ones to the bound of any two orders of its sums, nothing written beside it."""
    print("two-pass, one element off", sites, nu, nd, precision, flush=True)
    h = hb.hubbard_build(sites, edges, nu, nd, 1.0, 3.0)
    hb.hubbard_set_precision(h, precision)
    fp64 = precision == hb.HUBBARD_FP64
    if not fp64 and h.dim * 4 <= 192 << 20:
        pytest.skip("one-launch form")
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    x = torch.rand(h.dim + 2, generator=g, dtype=torch.float64 if fp64 else torch.float32, device=DEV) - 0.5
    y, off = torch.empty_like(x[:h.dim]), torch.full_like(x, 7.0)
    hb.hubbard_apply(h, x[1:-1].clone(), y)
    hb.hubbard_apply(h, x[1:-1], off[1:-1])
    info = hb.hubbard_info(h)
    terms = 1 + info["w_up"] + info["w_dn"]
    tol = terms * (2.0**-53 if fp64 else 2.0**-24) * 0.5 * (3.0 * sites + info["w_up"] + info["w_dn"])
    assert float((off[1:-1] - y).abs().max()) <= 2 * tol
    assert float(off[0]) == 7.0 and float(off[-1]) == 7.0
