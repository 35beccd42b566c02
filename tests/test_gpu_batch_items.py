"""The batched engine's work items at their edges: one column and thousands of
rows to an item, odd row counts (the last pair is half empty), one to several
64-column chunks, up and down rows of more hops than are loaded ahead, rows too
long for pairs in one or both precisions beside rows that are not, a descriptor
table rebuilt when half of its instances have stopped, and a Ritz value of more
steps than its LDS copy holds.

Tolerance as for every Lanczos coefficient: 64 sqrt(dim) eps of |H| in FP64, 1e-4
of |H| in mixed precision; an instance's bits do not depend on the others.
"""
import numpy as np
import pytest

import oracle
import workload

torch = pytest.importorskip("torch")
hb = pytest.importorskip("paper_1204_3425_amd")

pytestmark = pytest.mark.gpu

DIAG = workload.torus_tprime(4, 4, 1.0, 1.0)[0]

CASES = [
    # sites, edges, n_up, n_dn
    (14, workload.ring(14), 7, 0),       # 3,432 rows of one column
    (12, workload.torus(3, 4), 5, 2),    # 792 x 66
    (11, workload.ring(11), 4, 5),       # 330 x 462
    (9, workload.chain(9), 1, 4),        # 9 x 126
    (16, DIAG, 3, 3),                    # down rows of three groups of eight hops
    (16, DIAG, 5, 1),                    # up rows of up to 40 hops
    (13, workload.ring(13), 2, 6),       # 1,716 columns: pairs in FP32 only
    (14, workload.ring(14), 1, 7),       # 3,432 columns: no pairs
    (16, DIAG, 1, 5),                    # 4,368 columns of up to 40 hops
]
TINY = [(3, workload.ring(3), 1, 1), (4, workload.ring(4), 4, 0), (4, workload.ring(4), 1, 1), (5, workload.ring(5), 1, 1)]


@pytest.mark.parametrize("precision", [hb.HUBBARD_FP64, hb.HUBBARD_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("pick", [slice(0, 6), slice(0, 9)], ids=["pairs", "long_rows_too"])
def test_batch_items(pick, precision):
    cases = CASES[pick] + 3 * TINY  # the twelve tiny sectors stop first
    print("batch items", len(cases), precision, flush=True)
    hs = [hb.hubbard_build(*c, 1.0, 3.0) for c in cases]
    seeds = list(range(40, 40 + len(cases)))
    opt = dict(tol=-1.0, max_iter=40, precision=precision, history=True)
    mix = hb.hubbard_lanczos_batch(hs, seeds=seeds, **opt)
    for c, h, seed, g in zip(cases, hs, seeds, mix):
        m = oracle.Model(*c, 1.0, 3.0)
        ref = m.lanczos(oracle.start_vector(seed, m.dim), tol=-1.0, max_iter=40)
        n = 12 if h.dim > 100 else min(h.dim, 4)  # before a tiny sector's Krylov space ends
        scale = np.abs(ref["a"][:n]).max() + ref["b"][:n].max()
        tol = 1e-4 if precision == hb.HUBBARD_MIXED else 64 * np.sqrt(h.dim) * np.finfo(float).eps
        assert np.abs(g["a"][:n] - ref["a"][:n]).max() <= tol * scale, c
        if h.dim > 1:
            assert np.abs(g["b"][:n] - ref["b"][:n]).max() <= tol * scale, c
        alone = hb.hubbard_lanczos_batch([h], seeds=[seed], **opt)[0]
        assert alone["n_iter"] == g["n_iter"] and alone["E0"] == g["E0"], c
        assert np.array_equal(alone["a"], g["a"]) and np.array_equal(alone["b"], g["b"]), c


def test_batch_ritz_value_of_many_steps():
    """600 steps: the Ritz value of every step is the lowest eigenvalue of T_m, from
    the LDS copy and from the recorded coefficients."""
    h = hb.hubbard_build(10, workload.ring(10), 4, 5, 1.0, 3.0)
    r = hb.hubbard_lanczos_batch([h], tol=-1.0, max_iter=600, precision=hb.HUBBARD_FP64, seeds=[3], history=True)[0]
    assert r["n_iter"] == 600
    from scipy.linalg import eigh_tridiagonal
    for m in (1, 2, 3, 17, 100, 511, 512, 513, 600):
        w = eigh_tridiagonal(r["a"][:m], r["b"][:m - 1], eigvals_only=True, select="i", select_range=(0, 0))[0]
        assert abs(r["e_hist"][m - 1] - w) <= 1e-13 * max(1.0, np.abs(r["a"][:m]).max() + 2 * r["b"][:m].max()), m


NARROW = [
    # sites, edges, n_up, n_dn: rows a wave takes several pairs of at a time, and some it does not
    (13, workload.ring(13), 6, 0),       # 1,716 rows of one column
    (12, workload.torus(3, 4), 5, 1),    # 12 columns, 170 rows to an item, an odd last pair
    (16, DIAG, 3, 1),                    # 16 columns, down rows of one, up rows of three groups of eight
    (17, workload.ring(17), 4, 16),      # 17 columns
    (8, workload.ring(8), 4, 2),         # 28 columns
    (7, workload.ring(7), 3, 4),         # 35 columns: one pair at a time
    (15, workload.ring(15), 1, 7),       # long rows beside them
]


@pytest.mark.parametrize("precision", [hb.HUBBARD_FP64, hb.HUBBARD_MIXED], ids=["fp64", "mixed"])
def test_batch_of_narrow_rows(precision):
    """Each sector alone and all of them in one batch: the coefficients of the oracle,
    and the same bits either way."""
    print("narrow rows", precision, flush=True)
    hs = [hb.hubbard_build(*c, 1.0, 3.0) for c in NARROW]
    seeds = list(range(60, 60 + len(hs)))
    opt = dict(tol=-1.0, max_iter=10, precision=precision, history=True)
    for c, h, seed, g in zip(NARROW, hs, seeds, hb.hubbard_lanczos_batch(hs, seeds=seeds, **opt)):
        m = oracle.Model(*c, 1.0, 3.0)
        ref = m.lanczos(oracle.start_vector(seed, m.dim), tol=-1.0, max_iter=10)
        scale = np.abs(ref["a"]).max() + ref["b"].max()
        tol = 1e-4 if precision == hb.HUBBARD_MIXED else 64 * np.sqrt(h.dim) * np.finfo(float).eps
        assert np.abs(g["a"] - ref["a"]).max() <= tol * scale, c
        assert np.abs(g["b"] - ref["b"]).max() <= tol * scale, c
        alone = hb.hubbard_lanczos_batch([h], seeds=[seed], **opt)[0]
        assert np.array_equal(alone["a"], g["a"]) and np.array_equal(alone["b"], g["b"]), c
