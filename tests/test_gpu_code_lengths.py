"""Edge codes of 8, 16 and 32 bytes, read by teams by their own length (rows of one chunk, up to 128 nodes) and as two 16-byte reads (all others): the answers
of the search with one wave per query, which has a kernel for each length.  Odd degrees: the last neighbour's codes stand alone in their 16 bytes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,P,deg", [(32, 8, 16), (64, 16, 33), (128, 16, 1), (96, 24, 17), (128, 32, 64), (192, 48, 31), (256, 64, 33), (264, 12, 15), (512, 64, 17)])
@pytest.mark.parametrize("half", [False, True])
def test_answers(d, P, deg, half):
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS, PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(d + P + deg)
    rows = lambda m: torch.from_numpy(rng.standard_normal((m, d), dtype=np.float32) * (np.arange(1, d + 1) ** -0.3).astype(np.float32)).cuda()
    ix = PagIndex.build(rows(1500), metric="l2", max_degree=deg, num_subspaces=P, ef_construction=60, flags=FLAG_FP16_VECTORS if half else 0, seed=3)
    q = rows(4 * cus + 1)
    for K, efS in ((10, 64), (10, 500), (100, 300), (150, 300)):
        assert ix.search_layout(q.shape[0], K, efS)[0] == 1
        want = [x.clone() for x in ix.search(q, K, efS)]
        for nq in (1, cus, 2 * cus, 3 * cus):
            assert ix.search_layout(nq, K, efS)[0] > 1
            ids, dists = ix.search(q[:nq].contiguous(), K, efS)
            assert torch.equal(ids, want[0][:nq]) and torch.equal(dists, want[1][:nq]), (K, efS, nq)
    ix.close()
