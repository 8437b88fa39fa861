"""Small batches are searched by several waves per query, large ones by one: the two have to agree bit for bit.

The reference is the one-wave search, which tests/test_gpu_one_wave.py compares with the oracle: the same queries, repeated until
the batch is too large for teams.  The plan of each batch is asserted beside its answers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

COUNTERS = ("queries", "hops", "tests", "passes", "exact", "rounds", "rf_overflow", "rt_overflow")


def _rows(n, d, seed, metric):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((n, d), dtype=np.float32) * (np.arange(1, d + 1) ** -0.3).astype(np.float32)
    if metric == "ip":
        x /= np.linalg.norm(x, axis=1, keepdims=True)
    return x


def _count(ix, fn):
    ix.reset_counters()
    ids, dists = fn()
    c = ix.counters()
    return ids.cpu().numpy(), dists.cpu().numpy(), {k: c[k] for k in COUNTERS}


def _compare(ix, q, K, efS, sizes, search=None, waves=None, flags=0):
    """`waves`: per size, how many work on a query; None: more than one."""
    import torch
    from paper_2603_06660_amd import FLAG_EXACT_TEST_COUNT
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    qd = torch.from_numpy(q).cuda()
    many = qd.repeat((4 * cus) // q.shape[0] + 2, 1)[:4 * cus + 1].contiguous()
    assert ix.search_layout(many.shape[0], K, efS)[0] == 1
    ix.set_search_options(0, flags)
    ref_i, ref_d = (x.cpu().numpy() for x in ix.search(many, K, efS))
    ix.set_search_options(0, flags | FLAG_EXACT_TEST_COUNT)             # counters only: a long one-wave search tests some seen nodes
    _, _, ac = _count(ix, lambda: ix.search(many, K, efS))
    for at, nq in enumerate(sizes):
        got = ix.search_layout(nq, K, efS)[0]
        assert got == waves[at] if waves else got > 1, (nq, got)
        part = many[:nq].contiguous()
        ix.set_search_options(0, flags)
        gi, gd = (x.cpu().numpy() for x in (search or ix.search)(part, K, efS))
        assert np.array_equal(gi, ref_i[:nq]), "nq %d: ids differ in %d slots" % (nq, int((gi != ref_i[:nq]).sum()))
        assert np.array_equal(gd, ref_d[:nq]), "nq %d: distances differ" % nq
        if search is None:
            # the counters of the same queries, one wave each: the whole batch less what follows them
            ix.set_search_options(0, flags | FLAG_EXACT_TEST_COUNT)
            _, _, gc = _count(ix, lambda: ix.search(part, K, efS))
            rest = torch.cat([part, many]).contiguous()
            _, _, rc = _count(ix, lambda: ix.search(rest, K, efS))
            assert gc == {k: rc[k] - ac[k] for k in COUNTERS}, nq
    ix.set_search_options(0, flags)


# n, d, subspaces, degree, metric, half, K, efS: chunks of a row per lane 1 .. 12 with and without a tail, code words
# 2 / 4 / 8, register slots of W 1 / 2 / 4 / 8 / 16, exact LDS hash and bitmap, degrees up to a full wave; then the waves per query
# that up to one and up to two queries per CU get (four where the registers of two teams of eight do not fit a CU)
CASES = [
    (3000, 32, 8, 16, "l2", False, 1, 16, 12, 8),
    (3000, 128, 16, 32, "l2", False, 10, 64, 12, 8),
    (3000, 256, 16, 32, "ip", False, 10, 600, 12, 8),
    (2500, 260, 20, 24, "ip", False, 64, 300, 12, 8),
    (2500, 384, 24, 40, "l2", False, 65, 200, 12, 8),
    (4000, 768, 32, 32, "ip", False, 128, 512, 12, 8),
    (4000, 768, 32, 32, "ip", True, 10, 400, 12, 8),
    (2500, 1024, 32, 48, "ip", True, 129, 400, 12, 8),
    (2500, 1280, 40, 64, "ip", False, 10, 1500, 12, 8),
    (2000, 1536, 64, 48, "cos", False, 50, 768, 12, 8),
    (2000, 2048, 64, 33, "ip", False, 300, 900, 12, 4),
    (1500, 2304, 64, 32, "ip", True, 20, 100, 12, 4),
    (1500, 3072, 64, 32, "ip", False, 10, 128, 12, 4),
    (1500, 3072, 64, 32, "ip", True, 10, 200, 12, 4),
    (3000, 96, 8, 32, "l2", False, 600, 1200, 8, 4),
    (3000, 768, 32, 32, "ip", False, 1000, 3000, 8, 4),
]


@pytest.mark.parametrize("n,d,P,deg,metric,half,K,efS,one_per_cu,two_per_cu", CASES)
def test_team_equals_one_wave(n, d, P, deg, metric, half, K, efS, one_per_cu, two_per_cu):
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS, PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ix = PagIndex.build(torch.from_numpy(_rows(n, d, 1, metric)).cuda(), metric=metric, max_degree=deg, num_subspaces=P,
                        ef_construction=60, flags=FLAG_FP16_VECTORS if half else 0, seed=3)
    q = _rows(2 * cus, d, 2, metric)
    _compare(ix, q, K, efS, (1, 3, cus, cus + 1, 2 * cus), waves=(one_per_cu,) * 3 + (two_per_cu,) * 2)
    ix.close()


def test_team_of_four():
    """More queries than two per CU."""
    import torch
    from paper_2603_06660_amd import PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    d = 768
    ix = PagIndex.build(torch.from_numpy(_rows(4000, d, 5, "ip")).cuda(), metric="ip", max_degree=32, num_subspaces=32,
                        ef_construction=60, seed=3)
    q = _rows(700, d, 6, "ip")
    for K, efS, sizes in ((10, 128, (2 * cus + 1, 5 * cus // 2)), (64, 400, (2 * cus + 1, 3 * cus, 4 * cus)), (100, 400, (5 * cus // 2,))):
        _compare(ix, q, K, efS, sizes, waves=(4,) * len(sizes))
    ix.close()


@pytest.mark.parametrize("via", ["searcher", "static", "no_prt", "tiny_seen_set", "few_nodes"])
def test_team_variants(via):
    """A searcher's view (which drops repeated ids), the allocation-free entry point, the search without the projection
    test, a seen set that overflows, and an index with fewer nodes than the working set holds."""
    import torch
    from paper_2603_06660_amd import FLAG_NO_PRT, PagIndex
    n, d = (40 if via == "few_nodes" else 3000), 128
    ix = PagIndex.build(torch.from_numpy(_rows(n, d, 8, "l2")).cuda(), metric="l2", max_degree=32, num_subspaces=16,
                        ef_construction=60, seed=4)
    q = _rows(300, d, 9, "l2")
    K, efS = (40 if via == "few_nodes" else 20), 200
    if via == "searcher":
        s = ix.searcher()
        _compare(ix, q, K, efS, (1, 200, 300), search=s.search)
        s.close()
    elif via == "static":
        def static(part, k, ef):
            out = (torch.empty(part.shape[0], k, dtype=torch.int64, device="cuda"), torch.empty(part.shape[0], k, device="cuda"))
            return ix.search_static(part, k, ef, out)
        _compare(ix, q, K, efS, (1, 200, 300), search=static)
    else:
        if via == "tiny_seen_set":
            ix.set_seen_capacity_log2(6)
        _compare(ix, q, K, efS, (1, 200, 300), flags=FLAG_NO_PRT if via == "no_prt" else 0)
    ix.close()
