"""Working sets of 129 to 512 nodes, which a team keeps sorted over several slots of a lane and single waves keep unsorted: the same answers.

Sizes at the edges of slots (64 nodes), of groups of four slots and of the kernels' ranges (256, 512), fewer nodes than the set holds, searches
of one and of several rounds, and rows of lengths with 1 to 3 and more chunks.  The one-wave search is compared with the oracle in
tests/test_gpu_one_wave.py; ids and distances have to be equal bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rows(m, d, seed):
    import torch
    rng = np.random.default_rng(seed)
    return torch.from_numpy(rng.standard_normal((m, d), dtype=np.float32) * (np.arange(1, d + 1) ** -0.3).astype(np.float32)).cuda()


@pytest.mark.parametrize("n,d,deg,half,K,efS", [
    (2000, 64, 16, False, 129, 129), (2000, 128, 32, False, 191, 400), (2000, 128, 32, False, 192, 800), (2000, 260, 33, False, 193, 193),
    (2000, 768, 32, False, 256, 700), (2000, 768, 32, True, 255, 600), (2000, 96, 64, False, 257, 300), (2000, 520, 24, False, 320, 1000),
    (2000, 128, 32, False, 321, 321), (2000, 1536, 32, False, 384, 500), (2000, 128, 32, True, 449, 900), (2000, 64, 32, False, 511, 1100),
    (2000, 128, 48, False, 512, 1600), (400, 64, 16, False, 399, 399), (130, 64, 16, False, 129, 500)])
def test_answers(n, d, deg, half, K, efS):
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS, PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(n + d + K)
    rows = lambda m: torch.from_numpy(rng.standard_normal((m, d), dtype=np.float32) * (np.arange(1, d + 1) ** -0.3).astype(np.float32)).cuda()
    base, q = rows(n), rows(2 * cus)
    ix = PagIndex.build(base, metric="l2", max_degree=deg, num_subspaces=max(p for p in (8, 16, 20, 26) if d % p == 0), ef_construction=60,
                        flags=FLAG_FP16_VECTORS if half else 0, seed=3)
    many = q.repeat(3, 1)[:4 * cus + 1].contiguous()
    assert ix.search_layout(many.shape[0], K, efS)[0] == 1
    want = [x.clone() for x in ix.search(many, K, efS)]
    layouts = set()
    for nq in (1, 5, cus, cus + 1, 2 * cus, 2 * cus + 1):
        layouts.add(ix.search_layout(nq, K, efS)[0])
        ids, dists = ix.search(many[:nq].contiguous(), K, efS)
        assert torch.equal(ids, want[0][:nq]) and torch.equal(dists, want[1][:nq]), nq
    assert max(layouts) == 12 and min(layouts) in (4, 8), layouts
    ix.close()


# rows of one to four chunks, read in all three ways: of working sets of up to 256 nodes the registers leave room for four teams of four on a CU
@pytest.mark.parametrize("d,half,K,efS", [(128, False, 200, 400), (128, True, 129, 300), (512, False, 256, 256), (768, False, 150, 600), (768, True, 200, 200),
                                          (1024, False, 250, 500), (1024, True, 192, 400), (1536, True, 200, 300), (2048, True, 129, 129)])
def test_four_teams_a_cu(d, half, K, efS):
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS, PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ix = PagIndex.build(_rows(2000, d, d), metric="l2", max_degree=32, num_subspaces=max(16, d // 32), ef_construction=60,
                        flags=FLAG_FP16_VECTORS if half else 0, seed=3)
    q = _rows(4 * cus + 1, d, d + 1)
    assert ix.search_layout(4 * cus + 1, K, efS)[0] == 1
    want = [x.clone() for x in ix.search(q, K, efS)]
    for nq, waves in ((2 * cus, 8), (3 * cus + 1, 4), (4 * cus, 4)):
        assert ix.search_layout(nq, K, efS) == (waves, nq)
        ids, dists = ix.search(q[:nq].contiguous(), K, efS)
        assert torch.equal(ids, want[0][:nq]) and torch.equal(dists, want[1][:nq]), nq
    ix.close()


# a working set larger than K, by the index and by a searcher, whose hops look for repeated ids
@pytest.mark.parametrize("b", [129, 200, 256, 257, 400, 512])
@pytest.mark.parametrize("via", ["index", "searcher"])
def test_working_sets_above_K(b, via):
    import torch
    from paper_2603_06660_amd import PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ix = PagIndex.build(_rows(3000, 128, 7), metric="l2", max_degree=32, num_subspaces=16, ef_construction=60, search_b=b, seed=3)
    q = _rows(4 * cus + 1, 128, 8)
    s = ix.searcher() if via == "searcher" else ix
    for K, efS in ((1, 2 * b + 5), (20, b), (128, 3 * b)):
        assert ix.search_layout(4 * cus + 1, K, efS)[0] == 1
        want = [x.clone() for x in s.search(q, K, efS)]
        for nq in (3, cus, 2 * cus):
            assert ix.search_layout(nq, K, efS)[0] > 1
            ids, dists = s.search(q[:nq].contiguous(), K, efS)
            torch.cuda.synchronize()
            assert torch.equal(ids, want[0][:nq]) and torch.equal(dists, want[1][:nq]), (K, nq)
    if via == "searcher":
        s.close()
    ix.close()
