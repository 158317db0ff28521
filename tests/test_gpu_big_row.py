"""A caller's big_row is taken as 2^22 at most: a hub row of 2^22 edges stays in the first tier, one
edge more sends the sample on to the last, in the persistent and the captured form; the samples are
the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
MOST = 1 << 22


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


@pytest.mark.parametrize("form", [0, 2])
@pytest.mark.parametrize("deg", [MOST, MOST + 1])
def test_bound(skis, deg, form):
    print("big row", deg, form, flush=True)
    T = 12
    rp = np.zeros(deg + 2, np.int32) # node 0 has every other node as in-neighbour
    rp[1:] = deg
    col = np.arange(1, deg + 1, dtype=np.int32)
    w = np.full(deg, 1e-6, np.float32)
    ora = oracle.build_sketch(rp, col, w, seed=2, j0=0, j1=T, nthreads=8)
    sk = skis.build_sketch(rp, col, w, T, 2, form=form, big_row=0xFFFFFFFF)
    sp, nodes, roots, probed = (x.cpu().numpy() for x in sk.export())
    assert np.array_equal(sp, ora.sample_ptr) and np.array_equal(nodes, ora.nodes)
    assert np.array_equal(roots, ora.roots) and np.array_equal(probed.astype(np.uint64), ora.probed)
    inf = sk.info()
    assert inf.tier_samples == ((T, 0, 0, 0) if deg == MOST else (0, 0, 0, T))
