"""RobustPrune of a small batch, whose nodes get four waves each, keeps what Eq. 1 keeps of their candidate lists, in order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _keep(x, v, cand, deg):
    """Eq. 1 over candidates in ascending (distance, id) order; distances as the library rounds them."""
    def dist(a, b):
        return np.float32(np.sum((x[a] - x[b]).astype(np.float64) ** 2))
    kept = []
    for c in cand:
        if c != v and len(kept) < deg and not any(dist(s, c) <= dist(v, c) for s in kept):
            kept.append(c)
    return kept


# d: 1 .. 12 chunks a lane, with and without a rest; degrees below and above the rows that LDS holds, up to a full wave;
# candidates: fewer than a step of eight, not a multiple of it, several steps
@pytest.mark.parametrize("d,P,deg,efc", [(32, 8, 8, 6), (256, 16, 64, 203), (260, 20, 16, 100), (768, 32, 48, 120), (1024, 32, 64, 77),
                                         (1536, 64, 40, 90), (2048, 64, 24, 64), (3072, 64, 32, 50)])
def test_first_batch(d, P, deg, efc):
    """The first batch after the initial nodes: its candidate lists come from pag_insertion_candidates, its neighbours from a
    build that ends with it.  Reverse edges change records of older nodes only, those of the batch's own are as they were pruned."""
    import torch
    from paper_2603_06660_amd import FLAG_KEEP_ORDER, FLAG_NO_PES, PagIndex
    first = min(efc, 100)
    m = max(1, first // 2)
    n = first + m
    rng = np.random.default_rng(d)
    # around a few centres, so that candidates occlude each other after different numbers of kept ones
    base = torch.from_numpy((rng.standard_normal((n, d)) + 1.5 * rng.standard_normal((5, d))[rng.integers(0, 5, n)]).astype(np.float32)).cuda()
    kw = dict(metric="l2", max_degree=deg, num_subspaces=P, ef_construction=efc, seed=11, flags=FLAG_KEEP_ORDER | FLAG_NO_PES)
    old, new = PagIndex.build(base[:first].contiguous(), capacity=n, **kw), PagIndex.build(base, **kw)
    x, adj = new.export()["vectors"], new.export()["adj"].reshape(n, deg)
    ids, _, count, *_ = old.insertion_candidates(base[first:].contiguous(), efc)
    differ = 0
    for i in range(min(m, 16)):
        want = _keep(x, first + i, [int(c) for c in ids[i][:int(count[i])]], deg)
        got = [int(a) for a in adj[first + i] if a != 0xFFFFFFFF]
        differ += got != want
    assert differ == 0                # sums in another order differ by one part in 2^50: ties at 2^24 do not occur in these draws
    old.close(); new.close()
