"""FP64 grid couplings with tets past the limits of the boundary integrals:
cells much narrower than their neighbours, flat tets and wide ones are clipped,
beside others that are not, against the oracle at the FP64 tolerances (1e-12
for B, 1e-10 for gradients) and against the clip's own counts."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_common import gpu_csr, rel_fro, require_gpu, say, sparse_rel, to_dev

pytestmark = pytest.mark.gpu


def coupling(faces, X, T, dev, **kw):
    import torch
    from paper_1810_13046_amd import Coupling
    return Coupling(faces, to_dev(X, torch.float64, dev), to_dev(T, torch.int32, dev),
                    consistent=False, **kw)


def jumped(jump):
    """16 cells on [0, 1], the middle three `jump` times narrower."""
    w = np.where(abs(np.arange(16) - 8) <= 1, 1.0 / jump, 1.0)
    f = np.concatenate([[0.0], np.cumsum(w)])
    return f / f[-1], 1.0 / f[-1]


@pytest.mark.parametrize("axes,jump", [(1, 10), (1, 100), (1, 1000), (3, 10), (3, 100), (3, 1000)])
def test_spacing_jumps(axes, jump):
    import torch
    dev = require_gpu()
    f, wide = jumped(jump)
    faces = [f if e < axes else wl.uniform_faces(16) for e in range(3)]
    centre = [0.5 * (a[8] + a[9]) for a in faces]
    ext = np.array([1.6 * (wide if e < axes else 1 / 16) for e in range(3)])
    b = wl.box_body("b", ext, centre, (1, 1, 1), 0.0, np.random.default_rng(0))
    say(f"[gpu] octant limits: axes={axes} jump={jump}")
    c = coupling(faces, b.X, b.tets, dev)
    R = oracle.assemble(faces, b.X, b.tets)
    for d in range(3):
        fro, mx = sparse_rel(gpu_csr(c, d, oracle.n_fluid(faces, d)), R.B[d])
        assert fro <= 1e-12 and mx <= 1e-12
    rng = np.random.default_rng(3)
    u = [rng.standard_normal(oracle.lattice_shape(faces, d)[::-1]) for d in range(3)]
    g = rng.standard_normal((3, b.X.shape[0]))
    ud = [to_dev(v, torch.float64, dev) for v in u]
    us = c.velocity(ud)
    gu = [torch.zeros_like(v) for v in ud]
    gX = torch.zeros((b.X.shape[0], 3), dtype=torch.float64, device=dev)
    c.velocity_vjp(to_dev(g, torch.float64, dev), u_f=ud, u_s=us, g_uf=gu, g_X=gX)
    assert rel_fro(gX.cpu().numpy(), oracle.velocity_vjp(R, u, g)[1]) <= 1e-10
    assert c.info()["subtets"] > 0
    c.free()


@pytest.mark.parametrize("size", [0.7, 2.5, 5.0])
@pytest.mark.parametrize("flat", [1e-2, 1e-3, 1e-4, 1e-6])
def test_flat_tets_keep_the_clips_pieces(size, flat):
    """Tets apart, their fourth vertex `flat` of the size off the others'
    plane: as many pieces and entries as a mixed coupling, which clips the
    same tets in double."""
    dev = require_gpu()
    rng = np.random.default_rng(int(10 * size))
    faces = [wl.uniform_faces(32)] * 3
    base = np.array([[0, 0, 0], [1, 0, 0], [0.2, 0.9, 0], [0.5, 0.4, flat]]) * size / 32
    X = []
    for _ in range(60):
        R = np.linalg.qr(rng.standard_normal((3, 3)))[0]
        X.append(base @ R + 0.25 + 0.5 * rng.random(3))
    X, T = np.concatenate(X), np.arange(240).reshape(60, 4)
    say(f"[gpu] octant limits: size={size} flat={flat}")
    c, m = coupling(faces, X, T, dev), coupling(faces, X, T, dev, precision="fp32")
    assert c.info()["pieces"] == m.info()["pieces"]
    for d in range(3):
        a, b = c.export_csr(d), m.export_csr(d)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    c.free()
    m.free()


@pytest.mark.parametrize("items", [0, 40])
def test_wide_tets_beside_small_ones(items, monkeypatch):
    """A block of 0.8-cell elements and one of eight-cell elements: the first
    as if it were alone, bit for bit, the second clipped; then moved until
    none and until all are wide."""
    import torch
    dev = require_gpu()
    if items:
        monkeypatch.setenv("IBVT_CHUNK_ITEMS", str(items))
    faces = [wl.uniform_faces(32), wl.stretched_faces(32, 1.5), wl.uniform_faces(32)]
    small = wl.box_body("a", np.array([3, 2, 2]) * 0.8 / 32, (0.3, 0.4, 0.5), (3, 2, 2), 0.1,
                        np.random.default_rng(1))
    wide = wl.box_body("b", np.array([8, 8, 8]) / 32, (0.7, 0.6, 0.5), (1, 1, 1), 0.0,
                       np.random.default_rng(2))
    say(f"[gpu] octant limits: wide beside small, items={items}")
    ns = small.X.shape[0]
    T = np.concatenate([small.tets, wide.tets + ns])

    def check(c, X):
        R = oracle.assemble(faces, X, T)
        for d in range(3):
            fro, mx = sparse_rel(gpu_csr(c, d, oracle.n_fluid(faces, d)), R.B[d])
            assert fro <= 1e-12 and mx <= 1e-12
        assert abs(c.info()["pieces"] - R.stats["pieces"]) <= 4
        return c.info()["subtets"]

    X = np.concatenate([small.X, wide.X])
    c, alone = coupling(faces, X, T, dev), coupling(faces, small.X, small.tets, dev)
    some = check(c, X)
    assert some > 0 and alone.info()["subtets"] == 0
    for d in range(3):
        rp, col, val = c.export_csr(d)
        r2, c2, v2 = alone.export_csr(d)
        assert np.array_equal(rp[:ns + 1], r2)
        assert np.array_equal(col[:rp[ns]], c2) and np.array_equal(val[:rp[ns]], v2)
    def shrunk(factor):
        Y = X.copy()
        Y[ns:] = (Y[ns:] - [0.7, 0.6, 0.5]) * factor + [0.7, 0.6, 0.5]
        return Y

    for Y, want in ((shrunk(0.1), "none"), (X, "some"), ((X - 0.5) * 0.1 + 0.5, "none"),
                    ((X - 0.5) * 1.1 + 0.5, "some")):
        c.reassemble(to_dev(Y, torch.float64, dev))
        got = check(c, Y)
        assert (got == 0) == (want == "none")
    c.free()
    alone.free()


def test_piece_store_overflow_beside_boundary_integrals():
    """Long tets cut in more sub-tetrahedra than the store first holds (3.25 a
    pair), beside small elements: both are integrated again."""
    dev = require_gpu()
    rng = np.random.default_rng(4)
    faces = [wl.uniform_faces(32)] * 3
    small = wl.box_body("a", np.array([3, 2, 2]) * 0.8 / 32, (0.3, 0.4, 0.5), (3, 2, 2), 0.1, rng)
    rod = np.array([[0, 0, 0], [0, 1.9, 1.9], [24, 0, 1.9], [24, 1.9, 0]]) / 32
    X = [rod + (0.05 + rng.random(3) * [0.15, 0.8, 0.8]) for _ in range(60)]
    ns = small.X.shape[0]
    T = np.concatenate([small.tets, ns + np.arange(240).reshape(60, 4)])
    X = np.concatenate([small.X, *X])
    c, alone = coupling(faces, X, T, dev), coupling(faces, small.X, small.tets, dev)
    i = c.info()
    clipped = i["pairs"] - alone.info()["pairs"]
    say(f"[gpu] octant limits: overflow, {clipped} clipped pairs, {i['subtets']} sub-tetrahedra")
    assert i["subtets"] > 3.25 * clipped + 1024
    R = oracle.assemble(faces, X, T)
    assert abs(i["pieces"] - R.stats["pieces"]) <= 4
    for d in range(3):
        fro, mx = sparse_rel(gpu_csr(c, d, oracle.n_fluid(faces, d)), R.B[d])
        assert fro <= 1e-12 and mx <= 1e-12
    for d in range(3):
        assert np.array_equal(c.export_csr(d)[2][:c.export_csr(d)[0][ns]], alone.export_csr(d)[2])
    c.free()
    alone.free()
