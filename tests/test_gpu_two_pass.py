"""The two-pass H.v where sectors are too large for the one-launch form, at rows
whose 128-byte slabs are whole lines, whole half lines, or neither (results then
stored through the L2), with counts of slabs that the eight XCDs do not share
evenly, in dense and strided rows: H.v and the first Lanczos steps against the
oracle.

Tolerance: H.v FP64 1e-13 of the largest element, FP32 (terms + 1) 2^-24 times the
largest sum of magnitudes of a row; coefficients 64 sqrt(dim) eps of |H|.
"""
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
