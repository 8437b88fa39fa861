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
