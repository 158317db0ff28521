"""A degenerate sketch (Gamma = 0, no samples) built without the inverse index: the entry points that
take it -- the allocation-free estimate and the service -- answer cov 0 and the size of the set."""
import numpy as np
import pytest

from paper_1709_03565_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


@pytest.mark.parametrize("index", [0, 1])
def test_no_samples(skis, index):
    print("no samples", index, flush=True)
    n = 6000
    rp = np.minimum(np.arange(n + 1), n - 1).astype(np.int32)
    col = np.arange(1, n, dtype=np.int32)
    sk = skis.build_sketch(rp, col, np.zeros(n - 1, np.float32), 100, 1, build_inverse_index=index)
    assert sk.status == skis.SKIS_WDEGENERATE
    sets = [[0], [], [5, 5, n - 1], np.arange(4096), np.arange(5000)]
    set_ptr, set_nodes = inputs.sets_to_csr(sets)
    want = [float(len(np.unique(s))) for s in sets]
    cov, est = (x.cpu().numpy() for x in sk.estimate_noalloc(set_ptr, set_nodes))
    assert not cov.any() and list(est) == want
    srv = skis.Server(sk)
    cov, est, _ = srv.replay(set_ptr, set_nodes, np.zeros(len(sets)))
    srv.close()
    assert not cov.any() and list(est) == want
