"""Few samples in the tiers of one sample a workgroup, around the ids these take at a time: cycles of
more nodes than the second tier holds (the hash tier, in LDS in the persistent form and in HBM in the
captured one), and a hub row above every bound but the bitmap tier's.  Bit for bit with the oracle."""
import numpy as np
import pytest

import oracle
from paper_1709_03565_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


@pytest.mark.parametrize("form", [0, 2])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 15, 16, 17, 1100])
@pytest.mark.parametrize("kind", ["cycle", "hub"])
def test_few_samples(skis, kind, T, form):
    print("late tiers", kind, T, form, flush=True)
    if kind == "cycle":
        n = 1500
        src, dst, w = (np.arange(n) + 1) % n, np.arange(n), np.ones(n, np.float32)
    else:
        n = (1 << 20) + 10 # node 0's row is above the second and the hash tier's bound
        src, dst, w = np.arange(1, n), np.zeros(n - 1, np.int64), np.full(n - 1, 1e-5, np.float32)
    T = min(T, 17) if kind == "hub" else T
    rp, col, w = inputs.edges_to_in_csr(n, src, dst, w)
    ora = oracle.build_sketch(rp, col, w, seed=3, j0=0, j1=T, nthreads=8)
    sk = skis.build_sketch(rp, col, w, T, 3, form=form)
    sp, nodes, roots, probed = (x.cpu().numpy() for x in sk.export())
    assert np.array_equal(sp, ora.sample_ptr) and np.array_equal(nodes, ora.nodes)
    assert np.array_equal(roots, ora.roots) and np.array_equal(probed.astype(np.uint64), ora.probed)
    assert sk.info().tier_samples == ((0, 0, T, 0) if kind == "cycle" else (0, 0, 0, T))
