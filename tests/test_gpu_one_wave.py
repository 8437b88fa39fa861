"""The search with one wave per query, which large batches get, against the oracle: the queries of the parity tests repeated until
no team is planned.  Every repetition has to give the oracle's answers, and the counters are the oracle's times the repetitions."""
import threading

import numpy as np
import pytest

import pag_workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COUNTERS = (("hops", "hops"), ("passes", "passes"), ("exact", "exact"), ("rounds", "rounds"), ("rf_overflow", "rf_over"),
            ("rt_overflow", "rt_over"))


@pytest.fixture(scope="module")
def index(cfg1_oracle_index):
    from paper_2603_06660_amd import PagIndex
    o = cfg1_oracle_index
    ix = PagIndex.from_arrays(o.vec, o.adj, o.a, o.c, o.e2, o.codes, o.rot, o.cb, o.entry, metric="l2")
    yield ix
    ix.close()


def _repeat(q):
    """-> the queries, repeated, on the device; how often"""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    times = 4 * cus // len(q) + 1
    return torch.from_numpy(np.tile(q, (times, 1))).cuda(), times


def _parity(ix, oix, q, K, efS, b=0, flags=0, oflags=0, search=None):
    """`flags`: of the library, kept set; `oflags`: of the oracle.  -> the oracle's counters"""
    from paper_2603_06660_amd import FLAG_EXACT_TEST_COUNT
    many, times = _repeat(q)
    oi, od, oc = oix.search(q, K, efS, b=b, flags=oflags)
    try:
        ix.set_search_options(b, flags)
        assert ix.search_layout(many.shape[0], K, efS)[0] == 1
        ix.reset_counters()
        gi, gd = (search or ix.search)(many, K, efS)
        gc = ix.counters()
        gi, gd = gi.cpu().numpy().reshape(times, *oi.shape), gd.cpu().numpy().reshape(times, *od.shape)
        assert np.array_equal(gi, np.broadcast_to(gi[0], gi.shape)) and np.array_equal(gd, np.broadcast_to(gd[0], gd.shape))
        assert np.array_equal(gi[0], oi)
        assert np.all(np.abs(gd[0][oi >= 0] - od[oi >= 0]) <= 1e-5 * od[oi >= 0]) and np.array_equal(np.isinf(gd[0]), oi < 0)
        if search is None:
            for k_g, k_o in COUNTERS:
                assert gc[k_g] == times * oc[k_o], (k_g, gc[k_g], oc[k_o])
            width = b if b else max(10, K)
            if width + 8 * max(efS, width) <= 1024:     # exact on-chip seen set: unseen neighbours only
                assert gc["tests"] == times * oc["tests"]
            else:                                       # and seen ones that the second level would have recognised
                assert gc["tests"] >= times * oc["tests"]
                ix.set_search_options(b, flags | FLAG_EXACT_TEST_COUNT)
                ix.reset_counters()
                xi, xd = ix.search(many, K, efS)
                gx = ix.counters()
                assert np.array_equal(xi.cpu().numpy()[:len(q)], gi[0]) and np.array_equal(xd.cpu().numpy()[:len(q)], gd[0])
                for k_g, k_o in COUNTERS + (("tests", "tests"),):
                    assert gx[k_g] == times * oc[k_o], (k_g, gx[k_g], oc[k_o])
    finally:
        ix.set_search_options(0, 0)
    return oc


@pytest.mark.parametrize("efS", [10, 32, 64, 200])
def test_search(cfg1_small, cfg1_oracle_index, index, efS):
    w, base, q, gt, gtk = cfg1_small
    _parity(index, cfg1_oracle_index, q, w.K, efS)


@pytest.mark.parametrize("K,efS,b", [(100, 256, 0), (50, 128, 0), (200, 400, 0), (129, 129, 0), (500, 700, 0), (1000, 1000, 0), (1000, 2500, 0),
                                     (10, 512, 512), (10, 900, 300), (64, 1024, 1024)])
def test_large_working_sets(cfg1_small, cfg1_oracle_index, index, K, efS, b):
    w, base, q, gt, gtk = cfg1_small
    _parity(index, cfg1_oracle_index, q[:48], K, efS, b=b)


@pytest.mark.parametrize("efS", [64, 300])                          # exact hash and its spill; bitmap behind the Bloom filter
def test_seen_set_spills(cfg1_small, cfg1_oracle_index, index, efS):
    w, base, q, gt, gtk = cfg1_small
    index.set_seen_capacity_log2(6)
    try:
        _parity(index, cfg1_oracle_index, q, w.K, efS)
        assert index.counters()["seen_spills"] > 0
        _parity(index, cfg1_oracle_index, q[::-1].copy(), w.K, efS)     # the waves left clean bitmaps
    finally:
        index.set_seen_capacity_log2(0)


def test_without_the_projection_test(orc, cfg1_small, cfg1_oracle_index, index):
    from paper_2603_06660_amd import FLAG_NO_PRT
    w, base, q, gt, gtk = cfg1_small
    many, times = _repeat(q)
    try:
        index.set_search_options(48, FLAG_NO_PRT)
        assert index.search_layout(many.shape[0], 10, 48)[0] == 1
        gi, gd = index.search(many, 10, 48)
    finally:
        index.set_search_options(0, 0)
    oi, od, _ = cfg1_oracle_index.search(q, 10, 48, b=48, flags=orc.NO_PRT)
    assert np.array_equal(gi.cpu().numpy(), np.tile(oi, (times, 1)))
    assert np.allclose(gd.cpu().numpy(), np.tile(od, (times, 1)), rtol=1e-5)


def test_searcher_and_static(cfg1_small, cfg1_oracle_index, index):
    """A searcher's view drops ids that a record lists twice; the allocation-free entry point has its own bitmaps."""
    w, base, q, gt, gtk = cfg1_small
    s = index.searcher()

    def static(many, K, efS):
        out = (torch.empty(many.shape[0], K, dtype=torch.int64, device="cuda"), torch.empty(many.shape[0], K, device="cuda"))
        return index.search_static(many, K, efS, out)

    for search in (s.search, static):
        for K, efS in ((w.K, 64), (w.K, 300), (100, 256)):
            _parity(index, cfg1_oracle_index, q, K, efS, search=search)
            torch.cuda.synchronize()
    s.close()


@pytest.mark.parametrize("deg", [32, 48])
def test_search_while_inserting(orc, deg):
    """Large batches answered while pag_insert grows the index: every (id, distance) pair is a real one, and afterwards
    searcher and oracle agree.  With 48 neighbours the id row of a record spans two cache lines."""
    from paper_2603_06660_amd import PagIndex
    w = wl.workload(1, n=40000, nq=200)
    base, q = wl.make(w, "base"), wl.make(w, "query")
    n0 = 20000
    bd = torch.from_numpy(base).cuda()
    many, times = _repeat(q)
    gix = PagIndex.build(bd[:n0].contiguous(), metric="l2", max_degree=deg, num_subspaces=w.P, ef_construction=200, seed=31, capacity=w.n)
    srch = gix.searcher()
    assert gix.search_layout(many.shape[0], w.K, 64)[0] == 1
    extra = bd[n0:].contiguous()
    torch.cuda.synchronize()
    err = []

    def grow():
        try:
            gix.insert(extra)
        except Exception as ex:          # pragma: no cover
            err.append(ex)

    t = threading.Thread(target=grow)
    t.start()
    answers = []
    while t.is_alive() and len(answers) < 1000:
        answers.append(srch.search(many, w.K, 64))
    t.join()
    torch.cuda.synchronize()
    assert not err and answers, err
    bq, bb = torch.from_numpy(q).cuda().double(), bd.double()
    for ids, dists in answers[:: max(1, len(answers) // 10)]:
        assert int(ids.min()) >= 0 and int(ids.max()) < w.n and bool((dists[:, 1:] >= dists[:, :-1]).all())
        srt = ids.sort(dim=1).values
        assert bool((srt[:, 1:] != srt[:, :-1]).all())
        exact = ((bq.repeat(times, 1)[:, None, :] - bb[ids]) ** 2).sum(-1)
        assert bool(((dists.double() - exact).abs() <= 1e-4 * exact + 1e-5).all())
    i1, d1 = srch.search(many, w.K, 64)
    ex = gix.export()
    oix = orc.OracleIndex(ex["vectors"], ex["adj"], ex["a"], ex["c"], ex["e2"], ex["codes"], ex["rotation"], ex["codebooks"], ex["entry"],
                          metric=ex["metric"])
    oi, _, _ = oix.search(q, w.K, 64)
    assert (i1.cpu().numpy() == np.tile(oi, (times, 1))).mean() >= 0.999
    srch.close()
    gix.close()
