"""Distances of zero, rows stored twice, NaN and infinite queries: searches with several waves per query, which compare their keys as
doubles, answer like those with one, which compare them as integers."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def index_and_queries():
    import torch
    from paper_2603_06660_amd import PagIndex
    g = torch.Generator("cuda").manual_seed(1)
    x = torch.randn(3000, 128, generator=g, device="cuda")
    x[1000:1100] = x[:100]
    x[2000:2010] = 0
    ix = PagIndex.build(x, metric="l2", max_degree=32, num_subspaces=16, ef_construction=60, seed=4)
    near = torch.cat([x[:150], x[995:1050], x[1995:2020], x[:40] * 1e-22, x[:20] * 1e18])
    odd = x[:8].clone()
    odd[0, 3], odd[1, 5], odd[2, 7], odd[3, 7] = float("nan"), -float("nan"), float("inf"), -float("inf")
    odd[4] = 3e38
    yield ix, near, odd
    ix.close()


# one and two members of W per lane, at and below the slot's end; above 128 nodes up to four and up to eight, with slots before the first and without
@pytest.mark.parametrize("K,efS", [(1, 64), (10, 64), (64, 200), (100, 300), (129, 129), (200, 600), (256, 300), (257, 600), (512, 1200)])
@pytest.mark.parametrize("kind", ["near", "odd"])
def test_values(index_and_queries, kind, K, efS):
    import torch
    ix, near, odd = index_and_queries
    q = near if kind == "near" else odd
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    many = q.repeat(4 * cus // q.shape[0] + 2, 1)[:4 * cus + 1].contiguous()
    assert ix.search_layout(many.shape[0], K, efS)[0] == 1
    ids, dists = (t.clone() for t in ix.search(many, K, efS))
    assert kind == "odd" or bool((dists == 0).any())
    for nq in (8, cus, 2 * cus, 3 * cus):
        assert ix.search_layout(nq, K, efS)[0] > 1
        i, d = ix.search(many[:nq].contiguous(), K, efS)
        assert torch.equal(i, ids[:nq]), nq
        assert bool(((d == dists[:nq]) | (d.isnan() & dists[:nq].isnan())).all()), nq
