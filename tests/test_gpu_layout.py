"""How searches are laid out on the GPU: waves per query and queries resident at a time."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# What the registers of the one-wave kernel have to leave room for, in waves per CU.  Short searches where the on-chip memory
# would bound a long one below that.
@pytest.mark.parametrize("d,P,half,K,efS,per_cu", [
    (256, 64, False, 10, 16, 20), (768, 32, False, 10, 1024, 16), (768, 32, True, 10, 1024, 20),
    (1280, 40, True, 10, 1024, 12), (1280, 32, True, 100, 1024, 12), (1536, 64, False, 10, 1024, 12),
    (1792, 64, True, 400, 1024, 8), (2048, 32, False, 100, 1024, 12), (2304, 48, True, 10, 1024, 12), (2560, 64, False, 400, 1024, 8),
    (2816, 32, True, 10, 1024, 12), (2816, 64, True, 10, 1024, 8), (2816, 64, True, 400, 1024, 8),
    (3072, 64, False, 10, 1024, 8), (3072, 64, False, 100, 128, 8), (3072, 64, False, 200, 1024, 8), (3072, 64, True, 400, 1024, 8)])
def test_resident_queries_of_large_batches(d, P, half, K, efS, per_cu):
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS, PagIndex
    base = torch.from_numpy(np.random.default_rng(d).standard_normal((420, d), dtype=np.float32)).cuda()
    ix = PagIndex.build(base, metric="l2", max_degree=16, num_subspaces=P, ef_construction=20, flags=FLAG_FP16_VECTORS if half else 0)
    waves, resident = ix.search_layout(1 << 20, K, efS)
    ix.close()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert waves == 1 and resident >= per_cu * cus, (waves, resident / cus)


def test_reserved_room_does_not_change_the_plan():
    """Rows that an index has room for are not rows that a search reads."""
    import torch
    from paper_2603_06660_amd import PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    d, layouts = 768, []
    base = torch.from_numpy(np.random.default_rng(d).standard_normal((500, d), dtype=np.float32)).cuda()
    for capacity in (0, (512 << 20) // (4 * d) + 1):
        ix = PagIndex.build(base, metric="l2", max_degree=16, num_subspaces=32, ef_construction=20, capacity=capacity)
        layouts.append([ix.search_layout(nq, K, 128) for nq in (1, cus, 2 * cus, 5 * cus // 2, 3 * cus, 4 * cus) for K in (10, 100)])
        ix.close()
    assert layouts[0] == layouts[1] and layouts[0][8][0] == 4       # 3 to a CU, whatever the graph's size


def test_workspaces_are_sized_by_the_batch():
    """A small batch takes the seen-set bitmaps of its own queries, not of all that the GPU could hold at a time, also where it
    gets one wave per query, and its answers stay right when the next batches are larger."""
    import torch
    from paper_2603_06660_amd import PagIndex
    d, capacity = 16, 1 << 20
    rng = np.random.default_rng(3)
    rows = lambda n: torch.from_numpy(rng.standard_normal((n, d), dtype=np.float32)).cuda()
    kw = dict(metric="l2", max_degree=8, num_subspaces=4, ef_construction=20)
    base = rows(2000)
    ix, small = PagIndex.build(base, capacity=capacity, **kw), PagIndex.build(base, **kw)
    q = rows(3000)
    ix.search(q[:8], 1, 10)                                             # everything but the bitmaps' growth
    few = 4 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    for nq, waves in ((100, 12), (few, 1)):
        assert ix.search_layout(nq, 1, 10) == (waves, nq)
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        ix.search(q[:nq], 1, 10)
        torch.cuda.synchronize()
        assert free0 - torch.cuda.mem_get_info()[0] <= nq * capacity // 8 + (16 << 20)
    s = ix.searcher()
    for nq, K, efS in ((100, 1, 10), (300, 10, 900), (3000, 10, 900), (50, 10, 900), (40, 300, 400), (2000, 300, 400)):
        want = small.search(q[:nq], K, efS)
        for search in (ix.search, s.search):
            got = search(q[:nq], K, efS)
            torch.cuda.synchronize()
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (nq, K, efS)
    s.close(); ix.close(); small.close()


def test_waves_follow_what_the_gpu_is_searching():
    """A single query gets a team while nothing else is searched, one wave while a large batch is, and a team beside a batch
    that fills the GPU (it has its turn between two of them)."""
    import threading
    import torch
    from paper_2603_06660_amd import PagIndex
    rng = np.random.default_rng(5)
    rows = lambda n: torch.from_numpy(rng.standard_normal((n, 128), dtype=np.float32)).cuda()
    ix = PagIndex.build(rows(4000), metric="l2", max_degree=32, num_subspaces=16, ef_construction=60, seed=2)
    other = PagIndex.build(rows(500), metric="l2", max_degree=16, num_subspaces=16, ef_construction=30, seed=2)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    q = rows(12 * cus)
    many = q.repeat(10, 1)
    one = [x.clone() for x in other.search(q[:1].contiguous(), 10, 200)]
    assert ix.search_layout(q.shape[0], 10, 20000)[1] == q.shape[0] and ix.search_layout(many.shape[0], 10, 20000)[1] < many.shape[0]
    s = other.searcher()
    for batch, efS, want in ((q, 20000, 1), (many, 3000, 12)):
        assert other.search_layout(1, 10, 200)[0] == 12
        started = threading.Event()
        busy = threading.Thread(target=lambda: (started.set(), ix.search(batch, 10, efS)))
        seen, got = [], []
        busy.start()
        started.wait()
        while busy.is_alive():                              # nothing in here waits for the stream of the batch
            seen.append(other.search_layout(1, 10, 200)[0])
            got.append(s.search(q[:1], 10, 200))
        busy.join()
        torch.cuda.synchronize()
        assert want in seen and (want == 1 or set(seen) == {12}), seen
        assert all(torch.equal(i, one[0]) and torch.equal(d, one[1]) for i, d in got)       # the same answer either way
    assert other.search_layout(1, 10, 200)[0] > 1
    s.close(); other.close(); ix.close()
