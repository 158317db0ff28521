"""Preprocessing of 2^31 - 1 edges, the most there can be: a long row whose last chunk of edges would end
past 2^31 (35 GB of device memory)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("last", [1500, 3 * 3072 + 5])
def test_last_row(last, model):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    from paper_1709_03565_amd import skis
    print("last edges", last, model, flush=True)
    m, rows = 2**31 - 1, 2_100_000
    each = (m - last) // rows
    rp = torch.arange(rows + 1, dtype=torch.int64, device="cuda") * each
    rp[rows] = m - last
    rp = torch.cat([rp, torch.tensor([m], device="cuda")]).to(torch.int32)
    col = torch.zeros(m, dtype=torch.int32, device="cuda") # row 0's in-neighbour is node 1, the others' node 0
    col[:each] = 1
    w = torch.full((m,), 1e-7, dtype=torch.float32, device="cuda")
    w[m - last:] = torch.rand(last, device="cuda") * 1e-5
    out = skis.preprocess(rp, col, w, model=model)
    wl = w[m - last:].cpu().numpy().astype(np.float64)
    want = np.add.accumulate(wl) if model else np.multiply.accumulate(1.0 - wl)
    assert np.array_equal(out["P"][m - last:].cpu().numpy(), want)
    q = out["q"].cpu().numpy()
    assert q[-1] == (1.0 - want[-1] if model else want[-1])
    first = np.full(each, np.float64(np.float32(1e-7)))
    assert np.array_equal(out["P"][:each].cpu().numpy(), np.add.accumulate(first) if model else np.multiply.accumulate(1.0 - first))
    del out, rp, col, w
    torch.cuda.empty_cache()
    skis.release_cached_memory()
