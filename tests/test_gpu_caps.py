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
