"""The shortest searches, which get several waves per query like all others: against one wave per query, and in the construction of an
index against the oracle."""
import numpy as np
import pytest

from test_gpu_build_parity import _assert_same_index, _oracle_on

pytestmark = pytest.mark.gpu


# K, efS, working set (0: by K): one to 23 nodes, a working set of one; graphs of a single node, of fewer than the working set holds, of many
@pytest.mark.parametrize("n,K,efS,b", [(1, 1, 1, 0), (7, 1, 1, 0), (7, 7, 20, 0), (3000, 1, 1, 0), (3000, 1, 3, 1), (3000, 1, 9, 2), (3000, 10, 10, 0),
                                       (3000, 1, 15, 0), (3000, 10, 23, 0)])
def test_answers(n, K, efS, b):
    import torch
    from paper_2603_06660_amd import PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator("cuda").manual_seed(n + efS)
    ix = PagIndex.build(torch.randn(n, 96, generator=g, device="cuda"), metric="l2", max_degree=16, num_subspaces=8, ef_construction=40, seed=4)
    ix.set_search_options(b, 0)
    q = torch.randn(4 * cus + 1, 96, generator=g, device="cuda")
    assert ix.search_layout(q.shape[0], K, efS)[0] == 1
    ids, dists = (t.clone() for t in ix.search(q, K, efS))
    for nq, waves in ((1, 12), (cus, 12), (cus + 1, 8), (2 * cus, 8), (2 * cus + 1, 4), (4 * cus, 4)):
        assert ix.search_layout(nq, K, efS)[0] == waves
        i, d = ix.search(q[:nq].contiguous(), K, efS)
        assert torch.equal(i, ids[:nq]) and torch.equal(d, dists[:nq]), nq
    ix.close()


@pytest.mark.parametrize("efC", [1, 2, 5, 15])
@pytest.mark.parametrize("subbatch", [0, 1])
def test_construction(orc, efC, subbatch):
    import torch
    from paper_2603_06660_amd import FLAG_KEEP_ORDER, PagIndex
    n, deg, P = 300, 12, 8
    base = np.random.default_rng(efC).standard_normal((n, 64)).astype(np.float32)
    gix = PagIndex.build(torch.from_numpy(base).cuda(), metric="l2", max_degree=deg, num_subspaces=P, ef_construction=efC,
                         insert_subbatch=subbatch, seed=61, flags=FLAG_KEEP_ORDER)
    ex = gix.export()
    kw = dict(pes_every=1) if subbatch else dict(max_batch=n)
    _assert_same_index(ex, _oracle_on(orc, ex, np.arange(n), base, deg=deg, P=P, efC=efC, pes=True, **kw), "efC %d" % efC)
    gix.close()
