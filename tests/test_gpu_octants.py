"""FP64 grid couplings integrated from boundary integrals: element sizes at
the edges of the rule (one cell to more than six cells per axis, where the
clipped path takes over), ties with the cell planes, the dual multipliers and
chunked assemblies, against the oracle at the FP64 tolerances (1e-12 for
B and the transfers, 1e-10 for gradients)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_common import gpu_csr, rel_fro, require_gpu, say, sparse_rel, to_dev

pytestmark = pytest.mark.gpu


def mesh(size, snap, n=(3, 2, 2), cells=32):
    """A jittered block of hexahedra of `size` cells, its nodes moved to
    half-cell positions where snap."""
    rng = np.random.default_rng(int(10 * size) + snap)
    ext = np.array(n) * size / cells
    b = wl.box_body("b", ext, (0.5, 0.51, 0.49), n, 0.15, rng)
    X = np.round(2 * cells * b.X) / (2 * cells) if snap else b.X
    return X, b.tets


@pytest.mark.parametrize("size,snap,dual,items", [
    (0.3, False, False, 0), (1.0, True, False, 0), (2.0, True, False, 0), (2.6, False, True, 0),
    (2.6, False, False, 40), (4.2, False, False, 0), (5.6, False, False, 0)])
def test_octant_assembly(size, snap, dual, items, monkeypatch):
    import torch
    dev = require_gpu()
    if items:
        monkeypatch.setenv("IBVT_CHUNK_ITEMS", str(items))
    from paper_1810_13046_amd import Coupling
    faces = [wl.uniform_faces(32), wl.stretched_faces(32, 1.5), wl.uniform_faces(32)]
    X, T = mesh(size, snap)
    say(f"[gpu] octants size={size} snap={snap} dual={dual} items={items}")
    c = Coupling(faces, to_dev(X, torch.float64, dev), to_dev(T, torch.int32, dev), dual=dual,
                 consistent=False)
    R = oracle.assemble(faces, X, T, dual=dual)
    assert abs(c.info()["pieces"] - R.stats["pieces"]) <= max(4, R.stats["pieces"] // 100)
    for d in range(3):
        fro, mx = sparse_rel(gpu_csr(c, d, oracle.n_fluid(faces, d)), R.B[d])
        assert fro <= 1e-12 and mx <= 1e-12
    rng = np.random.default_rng(3)
    u = [rng.standard_normal(oracle.lattice_shape(faces, d)[::-1]) for d in range(3)]
    g = rng.standard_normal((3, X.shape[0]))
    ud = [to_dev(v, torch.float64, dev) for v in u]
    us = c.velocity(ud)
    assert rel_fro(us.cpu().numpy(), oracle.transfer_velocity(R, u)) <= 1e-12
    gu = [torch.zeros_like(v) for v in ud]
    gX = torch.zeros((X.shape[0], 3), dtype=torch.float64, device=dev)
    c.velocity_vjp(to_dev(g, torch.float64, dev), u_f=ud, u_s=us, g_uf=gu, g_X=gX)
    want = oracle.velocity_vjp(R, u, g)
    assert rel_fro(gX.cpu().numpy(), want[1]) <= 1e-10
    c.free()
