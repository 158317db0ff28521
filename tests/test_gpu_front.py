"""The sampler's front (slots of 44 nodes) from the count of samples it takes on, at its slots' sizes:
cycles of up to 64 nodes whose rows share a threshold or do not, one sample below its count, at it and
past it.  Bit for bit with the oracle."""
import numpy as np
import pytest

import oracle
from paper_1709_03565_amd import inputs

pytestmark = pytest.mark.gpu
FRONT_MIN = 1 << 20


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


@pytest.mark.parametrize("T", [FRONT_MIN - 1, FRONT_MIN, FRONT_MIN + 17])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("size", [3, 43, 44, 45, 64])
def test_sizes(skis, size, mixed, T):
    print("front", size, mixed, T, flush=True)
    rng = np.random.Generator(np.random.PCG64(size))
    v = np.arange(3 * size)
    ring = v // size * size
    src = np.concatenate([ring + (v + 1) % size, ring + (v + rng.integers(2, size, v.size)) % size])
    src = np.where(src == np.concatenate([v, v]), ring[0] + np.concatenate([ring, ring]) + (np.concatenate([v, v]) + 1) % size, src)
    w = np.concatenate([np.ones(v.size), np.full(v.size, 0.01 if mixed else 1.0)]).astype(np.float32)
    rp, col, w = inputs.edges_to_in_csr(3 * size, src, np.concatenate([v, v]), w)
    ora = oracle.build_sketch(rp, col, w, seed=3, j0=0, j1=T, nthreads=8)
    sk = skis.build_sketch(rp, col, w, T, 3, build_inverse_index=0)
    sp, nodes, roots, probed = (x.cpu().numpy() for x in sk.export())
    assert np.array_equal(sp, ora.sample_ptr) and np.array_equal(nodes, ora.nodes)
    assert np.array_equal(roots, ora.roots) and np.array_equal(probed.astype(np.uint64), ora.probed)
    assert sum(sk.info().tier_samples) == T


@pytest.mark.parametrize("T,chunk", [(FRONT_MIN + 17, FRONT_MIN), (FRONT_MIN + 17, FRONT_MIN - 1), (2 * FRONT_MIN + 5, 1 << 18)])
def test_captured_chunks(skis, T, chunk):
    """The captured form takes the front by the ids of a chunk, not of the build."""
    print("front chunks", T, chunk, flush=True)
    g = inputs.chung_lu_graph(3000, 24000, 2.1, 31, "wc", cache=False)
    a = skis.build_sketch(g.row_ptr, g.col, g.w, T, 3, build_inverse_index=0)
    b = skis.build_sketch(g.row_ptr, g.col, g.w, T, 3, build_inverse_index=0, form=2, chunk_samples=chunk)
    for x, y in zip(a.export(), b.export()):
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())
    assert a.info().deferred == b.info().deferred and sum(b.info().tier_samples) == T
