"""Estimates by the three routes a set can take -- the LDS hash of a light set, the windows of a
heavy one, the chunked path above 4096 entries -- at the sizes where one route ends and the next
begins, mixed in one call, against the oracle (Cov exact, the estimate to 1e-12 relative)."""
import numpy as np
import pytest

import oracle
from paper_1709_03565_amd import inputs

pytestmark = pytest.mark.gpu

HASH_MAX = 10922  # list entries of a light set's members


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


def _check(skis, rp, col, w, T, sets, seed=4):
    n = len(rp) - 1
    ora = oracle.build_sketch(rp, col, w, seed=seed, j0=0, j1=T, nthreads=4)
    _, q = oracle.row_prefix(rp, w)
    sk = skis.build_sketch(rp, col, w, T, seed)
    set_ptr, set_nodes = inputs.sets_to_csr(sets)
    ocov, oest = oracle.estimate(n, ora.sample_ptr, ora.nodes, q, ora.Gamma, set_ptr=set_ptr, set_nodes=set_nodes)
    first = None
    for call in (sk.estimate, sk.estimate_noalloc, sk.estimate):
        cov, est = (x.cpu().numpy() for x in call(set_ptr, set_nodes))
        assert np.array_equal(cov.astype(np.uint64), ocov)
        assert np.all(np.abs(est - oest) <= 1e-12 * np.abs(oest))
        first = est if first is None else first
        assert np.array_equal(first, est)
    # alone as in the mix
    for i in range(0, len(sets), max(1, len(sets) // 7)):
        c, e = sk.estimate(*inputs.sets_to_csr([sets[i]]))
        assert int(c[0]) == int(ocov[i]) and float(e[0]) == first[i]
    return sk


def _star(leaves, hubs):
    """`hubs` nodes each with an edge of weight 1 to every leaf... as in-edges of the leaves: a
    leaf's sample holds the leaf and all hubs, so a hub's list is every sample."""
    dst = np.repeat(np.arange(hubs, hubs + leaves), hubs)
    src = np.tile(np.arange(hubs), leaves)
    return inputs.edges_to_in_csr(hubs + leaves, src, dst, np.ones(len(src), np.float32))


@pytest.mark.parametrize("T", [1, 31, HASH_MAX - 1, HASH_MAX, HASH_MAX + 1, 32768, 32769, 65537, 200_003])
def test_lists_at_the_routes_ends(skis, T):
    # one hub's list holds T entries; two hubs' 2T, all of them repeats
    print("route ends", T, flush=True)
    rp, col, w = _star(50, 2)
    sets = [[0], [1], [0, 1], [0, 0, 1, 1], [10], [0, 10, 11], [], list(range(2, 52)), list(range(52))]
    _check(skis, rp, col, w, T, sets)


@pytest.mark.parametrize("count", [1, 1024, 1025])
def test_sets_of_all_routes_in_one_call(skis, count):
    print("mixed", count, flush=True)
    g = inputs.chung_lu_graph(6000, 48000, 2.0, 23, "wc", cache=False)
    rng = np.random.Generator(np.random.PCG64(count))
    top = np.argsort(-np.bincount(g.col, minlength=g.n), kind="stable").astype(np.int32)
    sets = []
    for i in range(count):
        kind = i % 5 if count > 1 else 1
        if kind == 0:
            sets.append(rng.choice(g.n, int(rng.integers(1, 60)), replace=False))
        elif kind == 1: # hubs: heavy
            sets.append(top[rng.integers(0, 40, int(rng.integers(1, 50)))])
        elif kind == 2: # many members, more than one chunk of 1024, repeats among them
            sets.append(rng.integers(0, g.n, 1500))
        elif kind == 3 and i % 100 == 3: # above one set's LDS: the chunked path
            sets.append(rng.integers(0, g.n, 4097 + i))
        else:
            sets.append(np.zeros(0, np.int32))
    _check(skis, g.row_ptr, g.col, g.w, 150_001, sets)


def test_refused_sets(skis):
    import torch
    print("refused", flush=True)
    rp, col, w = _star(50, 2)
    sk = skis.build_sketch(rp, col, w, 1000, 1)
    nodes = torch.zeros(8, dtype=torch.int32)
    for ptr in ([0, 5, 3], [-1, 2], [0, 2, 1, 8], [3, 2]):
        for call in (sk.estimate, sk.estimate_noalloc):
            with pytest.raises(skis.SkisError) as e:
                call(torch.tensor(ptr), nodes)
            assert e.value.code == skis.SKIS_EINVAL
    for bad in (-1, 52, 2**31 - 1):
        for call in (sk.estimate, sk.estimate_noalloc):
            with pytest.raises(skis.SkisError) as e:
                call(torch.tensor([0, 1, 3]), torch.tensor([0, 1, bad], dtype=torch.int32))
            assert e.value.code == skis.SKIS_EINVAL
    c, _ = sk.estimate(torch.tensor([0, 1]), nodes) # and the next call is answered
    assert int(c[0]) == 1000
