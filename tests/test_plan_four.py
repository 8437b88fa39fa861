"""Teams of four where more than two and up to four queries come to a CU (tests/test_plan.py has the rule): the answers."""
import numpy as np
import pytest

@pytest.mark.gpu
# n, d, subspaces, degree, metric, half, K, efS
@pytest.mark.parametrize("n,d,P,deg,metric,half,K,efS", [(1024, 32, 8, 16, "l2", False, 1, 4), (60, 128, 16, 32, "l2", False, 10, 10),
                                                         (500, 768, 32, 32, "ip", False, 10, 128), (3000, 128, 16, 32, "l2", False, 10, 64),
                                                         (3000, 260, 20, 24, "ip", False, 64, 100), (2500, 768, 32, 32, "ip", True, 128, 128),
                                                         (2000, 1536, 64, 48, "cos", False, 50, 120), (2500, 96, 8, 64, "l2", False, 150, 300)])
def test_answers(n, d, P, deg, metric, half, K, efS):
    """The same queries in a batch that is too large for teams, whose searches have one wave."""
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS, PagIndex
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(n + d)
    rows = lambda m: torch.from_numpy(rng.standard_normal((m, d), dtype=np.float32) * (np.arange(1, d + 1) ** -0.3).astype(np.float32)).cuda()
    base, q = rows(n), rows(4 * cus + 1)
    if metric == "ip":
        base, q = base / base.norm(dim=1, keepdim=True), q / q.norm(dim=1, keepdim=True)
    ix = PagIndex.build(base, metric=metric, max_degree=deg, num_subspaces=P, ef_construction=60, flags=FLAG_FP16_VECTORS if half else 0, seed=3)
    assert ix.search_layout(q.shape[0], K, efS)[0] == 1
    want = [x.clone() for x in ix.search(q, K, efS)]
    for nq in (2 * cus + 1, 3 * cus):
        assert ix.search_layout(nq, K, efS)[0] == 4, nq
        ids, dists = ix.search(q[:nq].contiguous(), K, efS)
        assert torch.equal(ids, want[0][:nq]) and torch.equal(dists, want[1][:nq]), nq
    ix.close()
