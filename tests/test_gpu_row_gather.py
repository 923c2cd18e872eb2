"""The row gather with 1, 2, 4 and 8 rows to a wave.  Their choice depends on
the number of rows and of cells per tet alone, so a mesh takes each of them
when vertices that no tet uses are added to it; every node adds its
contributions in the same order whatever the choice, so the rows of the
mesh's own vertices are the same bit for bit, and the first are those of the
FP64 oracle."""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.gpu_common import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


# cells of the grid, hexahedra of the body; element sizes of 0.7, 1.4, 2.6 and 4
# cells: up to 8, 27 and more than 64 cells a tet, boxes of 27 to 1,500 nodes
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("cells,hexes", [(12, (9, 7, 8)), (17, (6, 5, 5)), (26, (5, 4, 4)), (24, (3, 2, 3))])
def test_rows_do_not_depend_on_rows_per_wave(dev, cells, hexes, prec):
    import torch
    from paper_1810_13046_amd import Coupling
    say(f"[gpu] row gather {cells} {hexes} {prec}")
    rng = np.random.default_rng(cells)
    b = wl.box_body("b", (0.5, 0.42, 0.46), (0.5, 0.5, 0.5), hexes, 0.2, rng)
    faces = [np.linspace(0.0, 1.0, cells + 1)] * 3
    n = b.X.shape[0]
    tets = to_dev(b.tets, torch.int32, dev)
    R = oracle.assemble(faces, b.X, b.tets)
    want = None
    # 3 n_vert rows: 1, 1 or 2, 2, 4 and (or 4) 8 rows a wave
    for n_vert in (n, 1900, 3300, 6600, 9000):
        X = np.full((n_vert, 3), 0.5)
        X[:n] = b.X
        c = Coupling(faces, to_dev(X, torch.float64, dev), tets, precision=prec)
        got = [c.export_csr(d) for d in range(3)]
        for d, (rp, col, val) in enumerate(got):
            assert np.all(rp[n:] == rp[n])
            if want is None:
                B = R.B[d].tocsr()
                B.sort_indices()
                rows = np.repeat(np.arange(n), np.diff(rp))
                ref = np.asarray(B[rows, col]).ravel()
                tol = 1e-12 if prec == "fp64" else 1e-5
                assert np.linalg.norm(val - ref) <= tol * np.linalg.norm(ref), d
                assert abs(val.sum() - B.sum()) <= tol * abs(B).sum(), d
            else:
                assert np.array_equal(rp[:n + 1], want[d][0]), (d, n_vert)
                assert np.array_equal(col, want[d][1]) and np.array_equal(val, want[d][2]), (d, n_vert)
        if want is None:
            want = got
