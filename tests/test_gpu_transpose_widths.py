"""The node -> samples transpose at the edges of its two-pass form: node counts around the powers of
two where a digit's width, a kernel's width or the form changes, entries on both sides of the smallest
count it takes, and a node that is in every sample (its half of the ids fills several chunks)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


def _graph(n, hub):
    """A ring of in-edges of weight 1/2; hub: every other node has an in-edge of weight 1 from it."""
    v = np.arange(n, dtype=np.int64)
    deg = 1 + (v != hub) * (hub >= 0)
    rp = np.concatenate([[0], np.cumsum(deg)])
    col = np.empty(rp[-1], np.int32)
    w = np.empty(rp[-1], np.float32)
    col[rp[:-1]], w[rp[:-1]] = (v - 1) % n, 0.5
    if hub >= 0:
        second = rp[:-1][v != hub] + 1
        col[second], w[second] = hub, 1.0
    return rp.astype(np.int32), col, w


CASES = [(256, 40000, -1), (257, 20000, -1), (257, 3000, -1), (512, 20000, 300), (1 << 14, 40000, 77),
         ((1 << 14) + 1, 40000, -1), (1 << 20, 300000, 5), ((1 << 20) + 1, 1 << 20, 1 << 20), (1 << 20, 100000, -1),
         (1 << 22, 1 << 19, (1 << 22) - 1), ((1 << 22) + 1, 1 << 19, 9), (1 << 22, 1 << 17, 3)]


@pytest.mark.parametrize("n,T,hub", CASES)
def test_inverse(skis, n, T, hub):
    rp, col, w = _graph(n, hub)
    sk = skis.build_sketch(rp, col, w, T, 7)
    sp, nodes, _, _ = (x.cpu().numpy() for x in sk.export())
    npt, samples = (x.cpu().numpy() for x in sk.inverse())
    owner = np.repeat(np.arange(T, dtype=np.int32), np.diff(sp))
    assert np.array_equal(npt, np.concatenate([[0], np.cumsum(np.bincount(nodes, minlength=n))]))
    assert np.array_equal(samples, owner[np.argsort(nodes, kind="stable")])
