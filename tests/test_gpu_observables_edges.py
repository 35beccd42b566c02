"""Site observables at the edges of the accumulation's tiles, against the oracle:
odd rows (8-byte loads) and a psi that starts on 8 but not on 16 bytes, one
column, one row, rows that are no multiple of the 16 a workgroup takes at once,
columns just past a tile of 128 (64 above 16 sites), and rows of more tiles than
workgroups (several tiles of columns per workgroup).

Tolerance: the sums of non-negative terms carry at most their length times eps
relative; every value is at most 1 (the correlations) after the division:
1e-12 as for the other observables tests.
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
    # name, sites, n_up, n_dn
    ("odd_35x21", 7, 3, 2),
    ("one_column", 9, 4, 0),
    ("one_row", 9, 0, 4),
    ("one_state", 6, 6, 0),
    ("17_rows_of_136", 17, 1, 2),
    ("130_columns_odd", 13, 2, 4),       # 78 rows of 715
    ("792x924", 12, 5, 6),
    ("many_tiles", 20, 1, 8),            # 20 rows of 125,970: 1,969 tiles of 64 columns
]


@pytest.mark.parametrize("name,sites,nu,nd", CASES, ids=[c[0] for c in CASES])
def test_observables_edges(name, sites, nu, nd):
    print("observables", name, flush=True)
    edges = workload.chain(sites)
    h = hb.hubbard_build(sites, edges, nu, nd, 1.0, 2.0)
    m = oracle.Model(sites, edges, nu, nd, 1.0, 2.0)
    v = workload.random_vector(h.dim, 11)
    buf = torch.empty(h.dim + 1, dtype=torch.float64, device=DEV)
    o = m.observables(v)
    for off in (0, 1):
        psi = buf[off:off + h.dim]
        psi.copy_(torch.from_numpy(v))
        g = hb.hubbard_observables(h, psi)
        assert np.abs(g["dens"] - o["dens"]).max() <= 1e-12
        assert np.abs(g["corr"] - o["corr"]).max() <= 1e-12
        assert abs(g["docc"] - o["docc"]) <= 1e-12 * max(1.0, nu * nd)
        n = hb.hubbard_observables_noalloc(h, psi)
        assert np.abs(n["corr"] - g["corr"]).max() <= 1e-12


def test_observables_non_finite_state_is_refused():
    h = hb.hubbard_build(8, workload.ring(8), 4, 3, 1.0, 2.0)
    v = torch.zeros(h.dim, dtype=torch.float64, device=DEV)
    for bad in (float("inf"), float("nan")):
        v[5] = bad
        with pytest.raises(hb.HubbardError):
            hb.hubbard_observables(h, v)
