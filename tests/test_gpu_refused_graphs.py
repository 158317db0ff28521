"""Row offsets that are no graph's -- far below zero, where a row's length wraps to a large one, past
the edges, out of order -- are refused before any edge is read by them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LOW, HIGH = -2**31, 2**31 - 1


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


@pytest.mark.parametrize("value", [LOW, LOW + 1, LOW + 1500, LOW + 4000, -1, HIGH, 5001])
@pytest.mark.parametrize("at", [0, 1, 40, 99, 100])
def test_row_offsets(skis, at, value):
    print("offsets", at, value, flush=True)
    n, m = 100, 5000
    rp = np.arange(n + 1, dtype=np.int32) * (m // n)
    col = (np.repeat(np.arange(n), m // n) + 1).astype(np.int32) % n
    w = np.full(m, 0.01, np.float32)
    rp[at] = value
    for model in (0, 1):
        with pytest.raises(skis.SkisError) as e:
            skis.preprocess(rp, col, w, model=model)
        assert e.value.code == skis.SKIS_EINVAL
        with pytest.raises(skis.SkisError) as e:
            skis.build_sketch(rp, col, w, 10, 1, model=model)
        assert e.value.code == skis.SKIS_EINVAL
