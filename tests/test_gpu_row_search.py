"""The searches of a row from a guess (first live in-edge, LT pick) where the guess is far off or at
an end, and the running sums of long rows of equal weights: rows led by one heavy edge, ended by
one, of zeros around one, of weights that rise or fall by decades, of one to 9000 edges.  Bit for bit
with the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
N = 10000


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


def _row(kind, k, rng):
    w = np.full(k, 0.4 / k)
    if kind == "first":
        w[0] = 0.5
    elif kind == "last":
        w[-1] = 0.5
    elif kind == "one":
        w[:] = 0.0
        w[k // 3] = 0.9
    elif kind == "rise":
        w = 0.4 * np.logspace(-6, 0, k) / np.logspace(-6, 0, k).sum()
    elif kind == "fall":
        w = 0.4 * np.logspace(0, -6, k) / np.logspace(0, -6, k).sum()
    elif kind == "random":
        w = rng.random(k) / k
    elif kind == "full":
        w[:] = 1.0 / k
    return w


def _graph(kind):
    rng = np.random.default_rng(3)
    lens = [1, 2, 3, 4, 5, 8, 17, 64, 128, 129, 1024, 1025, 3071, 3072, 3073, 3136, 6145, 9000] + [7] * 200
    lens = np.array(lens + [1] * (N - len(lens)))
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows = np.repeat(np.arange(N), lens)
    # mostly towards the long rows, so that walks meet them again
    col = np.where(rng.random(rp[-1]) < 0.7, rng.integers(0, 220, rp[-1]), rng.integers(0, N, rp[-1]))
    col = np.where(col == rows, (col + 1) % N, col).astype(np.int32)
    w = np.concatenate([_row(kind, int(k), rng) for k in lens]).astype(np.float32)
    return rp, col, w


KINDS = ["equal", "first", "last", "one", "rise", "fall", "random", "full"]


@pytest.mark.parametrize("kind", KINDS)
def test_first_live_edge(skis, kind):
    rp, col, w = _graph(kind)
    T = 20000
    ora = oracle.build_sketch(rp, col, w, seed=9, j0=0, j1=T, nthreads=4)
    sp, nodes, roots, probed = (x.cpu().numpy() for x in skis.build_sketch(rp, col, w, T, 9).export())
    assert np.array_equal(sp, ora.sample_ptr) and np.array_equal(nodes, ora.nodes)
    assert np.array_equal(roots, ora.roots) and np.array_equal(probed.astype(np.uint64), ora.probed)


@pytest.mark.parametrize("kind", KINDS)
def test_lt_pick_and_sums(skis, kind):
    rp, col, w = _graph(kind)
    out = skis.preprocess(rp, col, w, model=1)
    S, q, status = oracle.row_sums_lt(rp, w)
    assert status == oracle.OK
    assert np.array_equal(out["P"].cpu().numpy(), S) and np.array_equal(out["q"].cpu().numpy(), q)
    T = 20000
    ora = oracle.build_sketch(rp, col, w, seed=9, j0=0, j1=T, nthreads=4, model=1)
    sp, nodes, roots, probed = (x.cpu().numpy() for x in skis.build_sketch(rp, col, w, T, 9, model=1).export())
    assert np.array_equal(sp, ora.sample_ptr) and np.array_equal(nodes, ora.nodes)
    assert np.array_equal(roots, ora.roots) and np.array_equal(probed.astype(np.uint64), ora.probed)
