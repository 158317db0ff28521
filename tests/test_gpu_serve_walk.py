"""The service's walk at its edges: sets whose members' lists hold just what the LDS hash takes and
one entry more, a wave's share of entries and one more, 1024, 1025 and 4096 members, duplicates; served
several times over (a bitmap left unclean would show), equal to skis_estimate of the set."""
import numpy as np
import pytest

from paper_1709_03565_amd import inputs

pytestmark = pytest.mark.gpu
HASH_MAX, SHARE = 10922, 512


@pytest.fixture(scope="module")
def skis():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1709_03565_amd import skis as s
    return s


def _with_entries(deg, order, total):
    """Distinct nodes whose list lengths add up to `total` (greedily, then by the short lists)."""
    out, left = [], total
    for v in order:
        if 0 < deg[v] <= left:
            out.append(v)
            left -= deg[v]
        if not left or len(out) == 4096:
            break
    return np.array(out, np.int32), total - left


@pytest.mark.parametrize("T", [20000, 100000])
def test_walk(skis, T):
    g = inputs.workload_graph("cl15k_wc")
    sk = skis.build_sketch(g.row_ptr, g.col, g.w, T, 1)
    deg = np.diff(sk.inverse()[0].cpu().numpy())
    rng = np.random.default_rng(2)
    desc = np.argsort(-deg, kind="stable")
    desc = desc[deg[desc] < 4000] # no hubs
    sets, hit = [], 0
    for total in (HASH_MAX, HASH_MAX + 1, 22 * SHARE, 22 * SHARE + 1, 16 * SHARE * 3, 16 * SHARE * 3 + 63, 60000):
        s, got = _with_entries(deg, desc, total)
        hit += got == total
        sets.append(rng.permutation(s).astype(np.int32))
    assert hit >= 5
    few = np.flatnonzero(deg < 20)
    for k in (1, 1023, 1024, 1025, 4096):
        sets.append(rng.choice(few if k > 1 else desc[:9], k, replace=False).astype(np.int32))
    sets.append(np.concatenate([sets[1], sets[1], sets[6][:50]]).astype(np.int32)[:4096])
    assert max(int(deg[s].sum()) for s in sets) < 1 << 18
    set_ptr, set_nodes = inputs.sets_to_csr(sets)
    cov, est = (x.cpu().numpy() for x in sk.estimate(set_ptr, set_nodes))
    srv = skis.Server(sk, pipeline_depth=2, max_batch_queries=8)
    for _ in range(4):
        c, e, _ = srv.replay(set_ptr, set_nodes, np.zeros(len(sets)))
        assert np.array_equal(c, cov.astype(np.uint64)) and np.array_equal(e, est)
    srv.close()
