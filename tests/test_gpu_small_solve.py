"""Two kernels at their edges.  The one-block mass solve (up to 512 vertices,
a row for every four of 1,024 threads): one row, the edges of its rounds, the
first size that takes a launch per iteration, rows of few and of many
entries, against the oracle's direct solve of the same right-hand side.  The
planar row gather (16 lanes to a row): vertices of more than 16 triangles,
boxes of less and of much more than 16 nodes, against the planar oracle."""
import numpy as np
import pytest

import oracle
import workloads as wl
from oracle import plane
from tests.gpu_common import rel_fro, require_gpu, say, sparse_rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


# 8, 18, 256, 448, 510, 512, 513 vertices; the solve stops at 1e-13 (1e-7): the
# mass matrix's condition (some 30) above it, and float results
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("hexes", [(1, 1, 1), (2, 1, 2), (3, 7, 7), (6, 7, 7), (16, 4, 5), (7, 7, 7),
                                   (18, 2, 8)])
def test_mass_solve(dev, hexes, prec):
    import torch
    from paper_1810_13046_amd import Coupling
    say(f"[gpu] block solve {hexes} {prec}")
    rng = np.random.default_rng(sum(hexes))
    b = wl.box_body("b", (0.5, 0.42, 0.46), (0.5, 0.5, 0.5), hexes, 0.2, rng)
    faces = [np.linspace(0.0, 1.0, 11)] * 3
    c = Coupling(faces, to_dev(b.X, torch.float64, dev), to_dev(b.tets, torch.int32, dev),
                 precision=prec)
    R = oracle.assemble(faces, b.X, b.tets)
    u = [rng.standard_normal(s) for s in c.lattice_shapes]
    got, info = c.velocity([to_dev(a, c.dtype, dev) for a in u], mass="consistent",
                           rtol=1e-13 if prec == "fp64" else 1e-7, maxit=500, with_info=True)
    e = rel_fro(got.cpu().numpy(), oracle.transfer_velocity(R, u, "consistent"))
    say(f"  {b.X.shape[0]} vertices: {e:.1e}, {info.iterations}")
    assert e <= (1e-11 if prec == "fp64" else 2e-5)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("spokes,cells", [(3, 9), (15, 12), (16, 40), (17, 40), (40, 90)])
def test_planar_rows(dev, spokes, cells, prec):
    import torch
    from paper_1810_13046_amd import Coupling
    say(f"[gpu] planar rows {spokes} {cells} {prec}")
    a = 2 * np.pi * np.arange(spokes) / spokes
    ring = np.stack([np.cos(a), np.sin(a)], 1)
    X = np.concatenate([[[0.5, 0.5]], 0.5 + 0.2 * ring, 0.5 + 0.35 * ring])
    k = np.arange(spokes)
    n = (k + 1) % spokes
    tris = np.concatenate([np.stack([0 * k, 1 + k, 1 + n], 1),
                           np.stack([1 + k, 1 + spokes + k, 1 + spokes + n], 1),
                           np.stack([1 + k, 1 + spokes + n, 1 + n], 1)])
    faces = [np.linspace(0.0, 1.0, cells + 1), np.linspace(0.0, 1.0, cells + 3)]
    c = Coupling(faces, to_dev(X, torch.float64, dev), to_dev(tris, torch.int32, dev),
                 precision=prec)
    R = plane.assemble(faces, X, tris.astype(np.int32))
    for d in range(2):
        rp, col, val = c.export_csr(d)
        import scipy.sparse as sp
        B = sp.csr_matrix((val, col, rp), shape=R.B[d].shape)
        assert all(np.all(np.diff(col[i:j]) > 0) for i, j in zip(rp[:-1], rp[1:]))
        assert sparse_rel(B, R.B[d])[0] <= (1e-12 if prec == "fp64" else 1e-5), d
