"""B^T's row arrays hold the fluid nodes B touches, not what they could be: the
same mesh and cells in a lattice of many more nodes takes the same memory
between assemblies (coupling_release_scratch gives the rest back)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as wl
from gpu_common import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


def check_transpose(c, d):
    rp, col, val = c.export_csr(d)
    trp, tcol, tval, rm = c.export_csr(d, True)
    n = int(np.prod(c.lattice_shapes[d]))
    want = sp.csr_matrix((val, col, rp), shape=(c.n_vert, n)).T.tocsr()
    want.sort_indices()
    assert np.array_equal(np.flatnonzero(np.diff(want.indptr)), rm)
    assert np.array_equal(want.indptr[rm], trp[:-1]) and trp[-1] == want.nnz
    assert np.array_equal(want.indices, tcol) and np.array_equal(want.data, tval)


@pytest.mark.parametrize("hexes,size,cells,more", [(20, 1.6, 40, 60), (14, 3.0, 48, 72)])
def test_rows_of_bt_are_not_sized_by_the_lattice(hexes, size, cells, more):
    """20: through the buckets, 14: through the counting sort; `more` cells on
    each side."""
    import torch
    from paper_1810_13046_amd import Coupling
    dev = require_gpu()
    h = 1.0 / cells
    b = wl.box_body("b", (hexes * size * h,) * 3, (0.5,) * 3, (hexes,) * 3, 0.1,
                    np.random.default_rng(hexes))
    held, rows = [], []
    for pad in (0, more):
        faces = [np.arange(-pad, cells + pad + 1) * h] * 3
        c = Coupling(faces, to_dev(b.X, torch.float64, dev), to_dev(b.tets, torch.int32, dev),
                     precision="fp32", consistent=False)
        c.release_scratch()
        i = c.info()
        check_transpose(c, 1)
        held.append(i["device_bytes"])
        rows.append(i["touched"])
        say(f"[gpu] transpose memory: pad={pad} nnz={i['nnz']} touched={i['touched']} "
            f"held={i['device_bytes']}")
        c.free()
    assert 12 * sum(i["nnz"]) > 32 << 20  # what the arrays could take
    assert np.allclose(rows[0], rows[1], rtol=0.01)
    assert abs(held[1] - held[0]) <= 8 << 20


def test_counts_waited_for_on_a_planar_grid():
    """A planar operator of more than 32 MiB of possible rows, both components
    in one launch, twice."""
    import torch
    from paper_1810_13046_amd import Coupling
    dev = require_gpu()
    n, cells = 400, 1600
    g = np.arange(n + 1) * 1.5 / cells + 0.1
    X = np.stack([a.ravel() for a in np.meshgrid(g, g, indexing="xy")], 1)
    X += (np.random.default_rng(2).random(X.shape) - 0.5) * 0.2 / cells
    k = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).ravel()
    T = np.concatenate([np.stack([k, k + 1, k + n + 2], 1), np.stack([k, k + n + 2, k + n + 1], 1)])
    c = Coupling([np.linspace(0, 1, cells + 1)] * 2, to_dev(X, torch.float64, dev),
                 to_dev(T, torch.int32, dev), consistent=False)
    assert 12 * sum(map(min, c.info()["nnz"], c.n_fluid)) > 32 << 20
    say(f"[gpu] transpose memory: planar nnz={c.info()['nnz']} touched={c.info()['touched']}")
    for _ in range(2):
        for d in range(2):
            check_transpose(c, d)
        c.reassemble(to_dev(X + 0.3 / cells, torch.float64, dev))
    c.free()
