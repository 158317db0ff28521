"""Sets of more members than a workgroup holds, through the service (members read from host memory, a
chunk ahead) and through skis_estimate: at the ends of chunks and of the clearing steps, with repeats
within and across chunks, several times over on the same slots."""
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


def test_large_sets(skis):
    print("large sets", flush=True)
    g = inputs.chung_lu_graph(30000, 60000, 2.3, 5, "wc", cache=False)
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, 3000, 1)
    rng = np.random.default_rng(2)
    sets = [rng.choice(g.n, k, replace=False).astype(np.int32) for k in (4097, 5120, 8191, 8192, 8193, 12288, 12289, g.n)]
    sets.append(np.tile(rng.choice(g.n, 700, replace=False).astype(np.int32), 13)) # each id in every chunk
    sets.append(np.full(9000, 17, np.int32))
    sets += [rng.choice(g.n, 5, replace=False).astype(np.int32) for _ in range(4)]
    set_ptr, set_nodes = inputs.sets_to_csr(sets)
    cov, est = (x.cpu().numpy() for x in sk.estimate(set_ptr, set_nodes))
    sp, nodes = (x.cpu().numpy() for x in sk.export()[:2])
    sample = np.repeat(np.arange(len(sp) - 1), np.diff(sp))
    for i, s in enumerate(sets):
        assert int(cov[i]) == len(np.unique(sample[np.isin(nodes, s)]))
    c, e = (x.cpu().numpy() for x in sk.estimate_noalloc(set_ptr, set_nodes))
    assert np.array_equal(c, cov) and np.array_equal(e, est)
    srv = skis.Server(sk, pipeline_depth=2, max_batch_queries=8)
    for _ in range(4):
        c, e, _ = srv.replay(set_ptr, set_nodes, np.zeros(len(sets)))
        assert np.array_equal(c, cov.astype(np.uint64)) and np.array_equal(e, est)
    srv.close()


@pytest.mark.parametrize("options", [dict(max_batch_entries=9000, max_large_sets=1), dict(max_batch_queries=4096),
                                     dict(pipeline_depth=1), dict(max_batch_entries=1 << 20, max_large_sets=64)])
def test_held_batches_go(skis, options):
    """Bursts in which large sets, entries or nothing fill a batch that is held back."""
    print("held", options, flush=True)
    g = inputs.chung_lu_graph(30000, 60000, 2.3, 5, "wc", cache=False)
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, 3000, 1)
    rng = np.random.default_rng(3)
    sets = [rng.choice(g.n, 5000 if i % 7 in (2, 3) else 900 if i % 5 == 1 else 3, replace=False).astype(np.int32) for i in range(80)]
    set_ptr, set_nodes = inputs.sets_to_csr(sets)
    cov, est = (x.cpu().numpy() for x in sk.estimate(set_ptr, set_nodes))
    srv = skis.Server(sk, **options)
    for at in (np.zeros(80), np.arange(80) * 2.0, np.arange(80) * 40.0):
        c, e, _ = srv.replay(set_ptr, set_nodes, at)
        assert np.array_equal(c, cov.astype(np.uint64)) and np.array_equal(e, est)
    assert srv.stats()["queries"] == 240
    srv.close()
