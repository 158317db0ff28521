"""Greedy at the edges of its tiles (2048 nodes) and of its two forms (one workgroup for sketches of
up to 2^19 entries, the launches beyond), with samples above 512 nodes, ties and k up to n: the
same seeds, marginals, coverage and estimate as the oracle's."""
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


def _check(skis, rp, col, w, T, ks, seed=6, ris=0):
    n = len(rp) - 1
    sk = skis.build_sketch(rp, col, w, T, seed)
    sp, nodes, _, _ = (x.cpu().numpy() for x in sk.export())
    _, q = oracle.row_prefix(rp, w)
    Gamma = sk.info().Gamma
    for k in ks:
        seeds, marg, cov, est = sk.greedy(k)
        oseeds, omarg, ocov, oest = oracle.greedy(n, sp, nodes, q, Gamma, k)
        assert np.array_equal(seeds.cpu().numpy(), oseeds)
        assert np.array_equal(marg.cpu().numpy().astype(np.uint64), omarg)
        assert cov == ocov and abs(est - oest) <= 1e-12 * abs(oest)
    return sk


@pytest.mark.parametrize("n", [3, 2047, 2048, 2049, 4096, 6200])
@pytest.mark.parametrize("T", [1, 900, 60_000])
def test_tile_edges(skis, n, T):
    print("tiles", n, T, flush=True)
    m = min(8 * n, n * (n - 1))
    g = inputs.chung_lu_graph(n, m, 2.1, 41, "wc", cache=False)
    sk = _check(skis, g.row_ptr, g.col, g.w, T, [1, min(n, 60)])
    print(sk.info().entries, flush=True)


def test_ties_and_all_nodes(skis):
    # weight-1 cycles: every node of a cycle has the same delta, and one pick covers them all
    print("ties", flush=True)
    size, rings = 30, 9
    v = np.arange(size * rings)
    src = (v // size) * size + (v + 1) % size
    rp, col, w = inputs.edges_to_in_csr(len(v), src, v, np.ones(len(v), np.float32))
    _check(skis, rp, col, w, 500, [1, 9, len(v)])
    _check(skis, rp, col, w, 40_000, [9, len(v)]) # past 2^19 entries: the launches


@pytest.mark.parametrize("T", [700, 3000])
def test_samples_above_512_nodes(skis, T):
    # samples of hundreds to thousands of nodes: the grid (or the workgroup) takes each together
    print("big samples", T, flush=True)
    g = inputs.chung_lu_graph(8000, 80000, 2.1, 77, "wc", cache=False)
    w = np.minimum(g.w * 1.6, 1.0).astype(np.float32)
    sk = _check(skis, g.row_ptr, g.col, w, T, [1, 40])
    sizes = np.diff(sk.export()[0].cpu().numpy())
    assert (sizes > 512).any() and (sizes < 512).any()
