"""B^d and B^dT of small operators: the counting transpose of all components
together (tiles of 4,096 lattice nodes) and the scans that go through one
block up to 16,384 entries, at the edges of both: lattices just below, at and
beyond whole tiles, vertex counts around the short scan's limit (unused
vertices make empty rows), no elements at all, and the planar coupling.
Exact: B^dT is the transpose of the exported B^d, entry for entry."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as wl
from tests.gpu_common import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


def check(c, n_comp, n_vert):
    for d in range(n_comp):
        brp, bcol, bval = c.export_csr(d)
        rp, col, val, rm = c.export_csr(d, transposed=True)
        assert brp.shape == (n_vert + 1,) and brp[0] == 0 and np.all(np.diff(brp) >= 0)
        B = sp.csr_matrix((bval, bcol, brp), shape=(n_vert, c.n_fluid[d]))
        T = B.T.tocsr()
        touched = np.flatnonzero(np.diff(T.indptr))
        T = T[touched]
        T.sort_indices()
        assert np.array_equal(rm, touched) and np.array_equal(rp, T.indptr), d
        assert np.array_equal(col, T.indices) and np.array_equal(val, T.data), d


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("cells,n_vert", [((15, 16, 16), 0), ((16, 16, 16), 0), ((31, 33, 37), 16383),
                                          ((24, 24, 24), 16384), ((24, 24, 24), 16385),
                                          ((64, 48, 40), 70001)])
def test_counting_transpose(dev, cells, n_vert, prec):
    import torch
    from paper_1810_13046_amd import Coupling
    say(f"[gpu] counting transpose {cells} {n_vert} {prec}")
    rng = np.random.default_rng(sum(cells) + n_vert)
    b = wl.box_body("b", (0.5, 0.4, 0.45), (0.5, 0.5, 0.5), (5, 4, 4), 0.2, rng)
    X, tets = b.X, b.tets
    if n_vert:  # the mesh's vertices spread over more, most of them unused
        at = np.sort(rng.choice(n_vert, X.shape[0], replace=False))
        at[-1] = n_vert - 1
        Y = np.full((n_vert, 3), 0.5)
        Y[at] = X
        X, tets = Y, at[tets].astype(np.int32)
    c = Coupling([np.linspace(0.0, 1.0, n + 1) for n in cells], to_dev(X, torch.float64, dev),
                 to_dev(tets, torch.int32, dev), precision=prec)
    check(c, 3, X.shape[0])
    c.reassemble(to_dev(X + 0.01, torch.float64, dev))
    check(c, 3, X.shape[0])


@pytest.mark.parametrize("dim", [2, 3])
def test_no_elements(dev, dim):
    import torch
    from paper_1810_13046_amd import Coupling
    c = Coupling([np.linspace(0.0, 1.0, 9)] * dim, torch.full((7, dim), 0.5, dtype=torch.float64,
                                                              device=dev),
                 torch.zeros((0, dim + 1), dtype=torch.int32, device=dev))
    check(c, dim, 7)


@pytest.mark.parametrize("cells", [(63, 64), (64, 64), (200, 130)])
def test_planar(dev, cells):
    import torch
    from paper_1810_13046_amd import Coupling
    rng = np.random.default_rng(cells[0])
    g = np.stack(np.meshgrid(np.linspace(0.25, 0.75, 12), np.linspace(0.3, 0.7, 9),
                             indexing="ij"), -1)
    g += 0.005 * rng.standard_normal(g.shape)
    k = np.arange(g[..., 0].size).reshape(g.shape[:2])
    a, b, c_, d = k[:-1, :-1].ravel(), k[1:, :-1].ravel(), k[1:, 1:].ravel(), k[:-1, 1:].ravel()
    tris = np.concatenate([np.stack([a, b, c_], 1), np.stack([a, c_, d], 1)])
    c = Coupling([np.linspace(0.0, 1.0, n + 1) for n in cells],
                 to_dev(g.reshape(-1, 2), torch.float64, dev), to_dev(tris, torch.int32, dev))
    check(c, 2, g.shape[0] * g.shape[1])
