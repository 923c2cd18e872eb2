"""B^T's row arrays hold the fluid nodes B touches, not what they could be: the
same mesh and cells in a lattice of many more nodes takes the same memory
between assemblies (coupling_release_scratch gives the rest back)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as wl
from gpu_common import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


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
        rp, col, val = c.export_csr(1)
        trp, tcol, tval, rm = c.export_csr(1, True)
        n = int(np.prod(c.lattice_shapes[1]))
        want = sp.csr_matrix((val, col, rp), shape=(c.n_vert, n)).T.tocsr()
        want.sort_indices()
        assert np.array_equal(np.flatnonzero(np.diff(want.indptr)), rm)
        assert np.array_equal(want.indptr[rm], trp[:-1]) and trp[-1] == want.nnz
        assert np.array_equal(want.indices, tcol) and np.array_equal(want.data, tval)
        held.append(i["device_bytes"])
        rows.append(i["touched"])
        say(f"[gpu] transpose memory: pad={pad} nnz={i['nnz']} touched={i['touched']} "
            f"held={i['device_bytes']}")
        c.free()
    assert 12 * sum(i["nnz"]) > 32 << 20  # what the arrays could take
    assert np.allclose(rows[0], rows[1], rtol=0.01)
    assert abs(held[1] - held[0]) <= 8 << 20
