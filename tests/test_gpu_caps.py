"""Limits on device memory (max_device_bytes) that sufficed before the sampler's second tier took more
workgroups a CU and the row records came: they suffice again, and the sketch under the limit is the
one without.  The limits are what the earlier version needed on a device of 256 CUs."""
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


@pytest.mark.parametrize("n,m,weights,T,limit,options", [
    (15000, 60000, "wc", 200_000, 615_970_000, {}),
    (15000, 60000, "wc", 200_000, 579_320_000, dict(staging_entries=1 << 16)),
    (15000, 60000, "wc", 200_000, 1_906_800_000, dict(form=1)),
    (15000, 60000, "wc", 200_000, 1_333_700_000, dict(form=2)),
    (1_000_000, 1000, "wc", 1000, 155_820_000, dict(staging_entries=1 << 16)),
    (1_000_000, 1000, "wc", 1000, 215_820_000, dict(form=1)),
    (1_000_000, 1000, "wc", 1000, 1_744_700_000, dict(form=2)),
    (1_000_000, 1000, "lt", 1000, 120_170_000, {}),
    (4_000_000, 100, "tri", 5000, 663_860_000, dict(staging_entries=1 << 16)),
])
def test_limits(skis, n, m, weights, T, limit, options):
    print("limit", n, m, weights, T, options, flush=True)
    g = inputs.chung_lu_graph_device(n, m, 2.3, 3, weights)
    model = 1 if weights == "lt" else 0
    a = skis.build_sketch(*g, T, 5, model=model, max_device_bytes=limit, **options)
    b = skis.build_sketch(*g, T, 5, model=model, **options)
    for x, y in zip(a.export(), b.export()):
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())


def test_many_sets_under_a_limit(skis):
    # 8 bytes of scratch a set would be more than the limit leaves
    import torch
    g = inputs.workload_graph("cl15k_wc")
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, 1000, 1, staging_entries=1 << 16, max_device_bytes=122_000_000)
    sets = inputs.random_sets(g.n, 20, 10, seed=3)
    hubs = np.argsort(-np.diff(sk.inverse()[0].cpu().numpy()), kind="stable")[:40].astype(np.int32)
    sets[11] = hubs
    p, x = inputs.sets_to_csr(sets)
    cov, est = (t.cpu().numpy() for t in sk.estimate(p, x))
    Q = (1 << 24) + 3 # the sets at the ends of rounds, the others empty
    at = [0, 1, 65534, 65535, 65536, 65537, 131071, 131072, 5_000_000, 1 << 23, (1 << 24) - 1, 1 << 24, Q - 2, Q - 1]
    size = torch.zeros(Q + 1, dtype=torch.int64)
    order = [i % 20 for i in range(len(at))]
    for pos, i in zip(at, order):
        size[pos + 1] = len(sets[i])
    nodes = np.concatenate([sets[i] for i in order]).astype(np.int32)
    c, e = sk.estimate(torch.cumsum(size, 0).cuda(), torch.as_tensor(nodes))
    assert np.array_equal(c[at].cpu().numpy(), cov[order]) and np.array_equal(e[at].cpu().numpy(), est[order])
    c[at] = 0
    e[at] = 0
    assert not c.any() and not e.any()
