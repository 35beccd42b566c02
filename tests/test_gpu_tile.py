"""The one-launch H.v of small and medium sectors at its edges, against the oracle.

Shapes: rows of one element, of little more than one wave and of little more than
one pass of the workgroup, a single row and few rows (several
workgroups share a row's columns), up rows of no hop, of fewer than the eight
hops loaded ahead and of more than sixteen, odd dense rows and strided rows in
both precisions, and per-bond handles (entries in slots of one amplitude each)
with two classes, with a class per bond, and with more than 16 slots.

Tolerance as for every H.v of this library: FP64 1e-13 of the largest element;
FP32 (terms + 1) 2^-24 times the largest sum of magnitudes a row can have.
"""
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
