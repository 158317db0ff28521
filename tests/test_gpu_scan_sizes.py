"""The prefix sums at the edges of their one-workgroup form (4096 values a tile, up to 32768): node counts
around them, whose alias tables are built from three such sums.  Bit for bit with the oracle."""
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


@pytest.mark.parametrize("n", [2, 63, 65, 4095, 4096, 4097, 8193, 32767, 32768, 32769, 65537])
def test_alias_table(skis, n):
    g = inputs.chung_lu_graph(n, 6 * n if n > 2 else 2, 2.1, 5, "tri", cache=False)
    out = skis.preprocess(g.row_ptr, g.col, g.w)
    _, q = oracle.row_prefix(g.row_ptr, g.w)
    W, C, _ = oracle.root_weights(q)
    thr, alias = oracle.alias_build(W, C)
    assert out["C"] == C and out["Gamma"] == oracle.gamma_total(q)
    assert np.array_equal(out["thr"].cpu().numpy().astype(np.uint64), thr)
    assert np.array_equal(out["alias"].cpu().numpy(), alias)
    T = min(n, 40000)
    ora = oracle.build_sketch(g.row_ptr, g.col, g.w, seed=2, j0=0, j1=T, nthreads=4)
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, T, 2)
    sp, nodes, _, _ = (x.cpu().numpy() for x in sk.export())
    npt, samples = (x.cpu().numpy() for x in sk.inverse())
    assert np.array_equal(sp, ora.sample_ptr) and np.array_equal(nodes, ora.nodes)
    assert np.array_equal(npt, np.concatenate([[0], np.cumsum(np.bincount(nodes, minlength=n))]))
    assert np.array_equal(samples, np.repeat(np.arange(T, dtype=np.int32), np.diff(sp))[np.argsort(nodes, kind="stable")])
