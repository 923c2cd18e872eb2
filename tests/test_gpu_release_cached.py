"""What freed couplings leave with the library goes back without a handle."""
import gc

import numpy as np
import pytest

import workloads as wl
from gpu_common import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


def test_release_without_a_coupling():
    import torch
    from paper_1810_13046_amd import Coupling, release_cached
    dev = require_gpu()
    gc.collect()

    def free_bytes():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    def use(n):
        b = wl.box_body("b", (0.5, 0.42, 0.46), (0.5, 0.5, 0.5), (n + 2, n - 2, n), 0.2,
                        np.random.default_rng(5))
        Coupling([np.linspace(0.0, 1.0, 2 * n + 5)] * 3, to_dev(b.X, torch.float64, dev),
                 to_dev(b.tets, torch.int32, dev)).free()
    use(4)  # loads the library's code and its static scratch
    release_cached()
    before = free_bytes()
    use(34)
    kept = before - free_bytes()
    release_cached()
    left = before - free_bytes()
    say(f"[gpu] release_cached: kept {kept}, then {left}")
    assert kept > 256 << 20
    assert left <= 64 << 20
    release_cached()  # nothing kept: no error
