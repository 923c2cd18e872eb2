"""The shape terms from stored moments with 16, 8, 4 and 1 lanes for each
(component, tet): the choice follows the number of tets and of cells per tet,
so the meshes below take one each (and 16 at their edges: tets in one cell,
tets with more pairs than lanes).  Against the coupling that keeps no moments
and integrates the pieces again by quadrature (exact for these integrands
too): rounding only, 1e-10 in double; float moments, weights and terms
carry some 1e-6 relative to the gradient's norm, 2e-5 leaves room for the
cancellation in its sums."""
import numpy as np
import pytest

import workloads as wl
from tests.gpu_common import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("cells,hexes", [(6, (5, 4, 3)), (40, (3, 2, 3)), (48, (7, 6, 6)),
                                         (16, (10, 9, 8)), (24, (16, 12, 10)), (48, (30, 28, 26))])
def test_shape_terms(dev, cells, hexes, prec):
    import torch
    from paper_1810_13046_amd import Coupling
    say(f"[gpu] shape lanes {cells} {hexes} {prec}")
    rng = np.random.default_rng(cells)
    b = wl.box_body("b", (0.5, 0.42, 0.46), (0.5, 0.5, 0.5), hexes, 0.2, rng)
    faces = [np.linspace(0.0, 1.0, cells + 1)] * 3
    X, tets = to_dev(b.X, torch.float64, dev), to_dev(b.tets, torch.int32, dev)
    n = b.X.shape[0]
    g = rng.standard_normal((3, n))
    f_s = rng.standard_normal((3, n))
    got = []
    for pr, store in ((prec, True), ("fp64", False)):
        c = Coupling(faces, X, tets, precision=pr, store_pieces=store)
        r = np.random.default_rng(7)
        u = [to_dev(r.standard_normal(s), c.dtype, dev) for s in c.lattice_shapes]
        gf = [to_dev(r.standard_normal(s), c.dtype, dev) for s in c.lattice_shapes]
        us = c.velocity(u, mass="lumped")
        out = []
        # one adjoint, then both in one pass
        gX = torch.zeros((n, 3), dtype=torch.float64, device=dev)
        gd, fd = to_dev(g, c.dtype, dev), to_dev(f_s, c.dtype, dev)
        c.velocity_vjp(gd, u_f=u, u_s=us, mass="lumped", g_X=gX)
        out.append(gX.cpu().numpy())
        gX = torch.zeros((n, 3), dtype=torch.float64, device=dev)
        c.vjp(gd, gf, u_f=u, u_s=us, f_s=fd, mass="lumped", alpha=0.7, g_X=gX)
        out.append(gX.cpu().numpy())
        got.append(out)
    for a, ref in zip(*got):
        e = np.linalg.norm(a - ref) / np.linalg.norm(ref)
        say(f"  {e:.1e}")
        assert e <= (1e-10 if prec == "fp64" else 2e-5)
