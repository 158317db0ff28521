"""Greedy on sketches of up to 2^19 entries, where the first rounds are the whole device's and the rest
one workgroup's: entries just below and above the least for that, up to the most, k up to and past the
eight rounds that may all be the device's, hubs first, samples of the graph's size, and a graph without
hubs -- the oracle's seeds, marginals, coverage and estimate, and nothing written past the k picks."""
import ctypes

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


def _check(skis, sk, g_rp, g_w, ks):
    import torch
    n = len(g_rp) - 1
    sp, nodes, _, _ = (x.cpu().numpy() for x in sk.export())
    _, q = oracle.row_prefix(g_rp, g_w)
    Gamma = sk.info().Gamma
    for k in ks:
        seeds = torch.full((k + 64,), -7, dtype=torch.int32, device="cuda")
        marg = torch.full((k + 64,), -7, dtype=torch.int64, device="cuda")
        cov, est = ctypes.c_uint64(), ctypes.c_double()
        st = skis.lib().skis_greedy_max_cover(sk._h, k, ctypes.c_void_p(seeds.data_ptr()), ctypes.c_void_p(marg.data_ptr()),
                                              ctypes.byref(cov), ctypes.byref(est),
                                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == skis.SKIS_OK
        oseeds, omarg, ocov, oest = oracle.greedy(n, sp, nodes, q, Gamma, k)
        seeds, marg = seeds.cpu().numpy(), marg.cpu().numpy()
        assert np.array_equal(seeds[:k], oseeds) and np.array_equal(marg[:k].astype(np.uint64), omarg)
        assert cov.value == ocov and abs(est.value - oest) <= 1e-12 * abs(oest)
        assert (seeds[k:] == -7).all() and (marg[k:] == -7).all()


@pytest.mark.parametrize("entries", [60_000, 65_000, 66_500, 130_000, 500_000, 560_000])
@pytest.mark.parametrize("n,m,weights", [(2000, 40000, "wc"), (15000, 60000, "wc"), (30000, 200000, "tri")])
def test_entries(skis, n, m, weights, entries):
    g = inputs.chung_lu_graph(n, m, 2.0, 3, weights, cache=False)
    p = skis.build_sketch(g.row_ptr, g.col, g.w, 20000, 5).info()
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, max(1, int(20000 * entries / p.entries)), 5)
    print("handover", n, weights, entries, sk.info().entries, flush=True)
    _check(skis, sk, g.row_ptr, g.w, [1, 2, 3, 7, 8, 9, 16, 60])


def test_no_hubs(skis):
    # every node in two others' rows: small samples, no pick lowers many entries
    print("no hubs", flush=True)
    n = 20000
    v = np.arange(n)
    rp, col, w = inputs.edges_to_in_csr(n, np.concatenate([(v + 1) % n, (v + 17) % n]), np.concatenate([v, v]),
                                        np.full(2 * n, 0.3, np.float32))
    sk = skis.build_sketch(rp, col, w, 60000, 5)
    assert 65536 < sk.info().entries < 1 << 19
    _check(skis, sk, rp, w, [1, 2, 6, 9, 40])
