"""skis_estimate_noalloc over its chunks of 1024 sets: light, heavy and large sets in the first, the
last or both, an error met in a later chunk, sets that are all empty without a node array -- equal to
skis_estimate bit for bit, and the call after a refused one is answered."""
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


@pytest.mark.parametrize("count", [1, 1023, 1024, 1025, 2050])
def test_chunks(skis, count):
    import torch
    print("chunks", count, flush=True)
    g = inputs.workload_graph("cl15k_wc")
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, 60000, 1)
    hubs = np.argsort(-np.diff(sk.inverse()[0].cpu().numpy()), kind="stable")[:20].astype(np.int32)
    rng = np.random.Generator(np.random.PCG64(count))
    base = [rng.choice(g.n, int(rng.integers(0, 8)), replace=False) for _ in range(count)]
    large = rng.choice(g.n, 4500, replace=False)
    for heavy_at, large_at in ((None, None), (0, None), (-1, None), (None, -1), (0, -1), (-1, 0)):
        sets = list(base)
        if large_at is not None:
            sets[large_at] = large
        if heavy_at is not None:
            sets[heavy_at] = hubs
        p, x = inputs.sets_to_csr(sets)
        cov, est = (t.cpu().numpy() for t in sk.estimate(p, x))
        c, e = (t.cpu().numpy() for t in sk.estimate_noalloc(p, x))
        assert np.array_equal(c, cov) and np.array_equal(e, est)
    bad = torch.as_tensor(p).clone()
    bad[-1] = bad[-2] - 1
    for ptr, nodes in ((bad, torch.as_tensor(x)), (torch.as_tensor(p), torch.as_tensor(np.append(x[:-1], g.n)))):
        if count > 1 or nodes[-1] == g.n:
            with pytest.raises(skis.SkisError) as err:
                sk.estimate_noalloc(ptr, nodes)
            assert err.value.code == skis.SKIS_EINVAL
    c, e = (t.cpu().numpy() for t in sk.estimate_noalloc(p, x))
    assert np.array_equal(c, cov) and np.array_equal(e, est)
    # no node array: every set must be empty
    none = torch.zeros(count + 1, dtype=torch.int64)
    c, e = sk.estimate_noalloc(none, torch.zeros(0, dtype=torch.int32))
    assert not c.any() and not e.any()
    none[-1] = 3
    with pytest.raises(skis.SkisError) as err:
        sk.estimate_noalloc(none, torch.zeros(0, dtype=torch.int32))
    assert err.value.code == skis.SKIS_EINVAL
