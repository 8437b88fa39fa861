"""The search of an insertion with one wave per vector, as large batches are searched: R_L and H(v) against the oracle and against teams."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("efC", [40, 100, 250])
def test_one_wave_candidates(orc, cfg1_small, cfg1_oracle_index, efC):
    import torch
    from paper_2603_06660_amd import PagIndex
    w, base, q, gt, gtk = cfg1_small
    oix = cfg1_oracle_index
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(efC)
    # more vectors than teams are planned for: near the index's, so that their lists differ
    x = (base[rng.integers(0, len(base), 4 * cus + 40)] + 0.1 * rng.standard_normal((4 * cus + 40, w.d))).astype(np.float32)
    gix = PagIndex.from_arrays(oix.vec, oix.adj, oix.a, oix.c, oix.e2, oix.codes, oix.rot, oix.cb, oix.entry, metric="l2", ef_construction=efC)
    one = gix.insertion_candidates(torch.from_numpy(x).cuda(), efC)
    part = 3 * cus
    for a, b in zip(one, gix.insertion_candidates(torch.from_numpy(x[:part]).cuda(), efC)):      # four waves per vector
        assert np.array_equal(a[:part], b)
    ci, ck, cn, hi, hk, hn = one
    sample = range(0, len(x), 23)
    qr, _ = oix.prepare(x[list(sample)])
    n_pes = 0
    for k, i in enumerate(sample):
        oi, ok, ohi, ohk, _ = oix.index_search(qr[k], efC)
        assert cn[i] == len(oi) and ci[i, :cn[i]].tolist() == oi.tolist(), i
        assert np.all(np.abs(ck[i, :cn[i]] - ok) <= 1e-5 * ok)
        assert hn[i] == len(ohi) and hi[i, :hn[i]].tolist() == ohi.tolist(), i
        assert np.all(np.abs(hk[i, :hn[i]] - ohk) <= 1e-5 * ohk)
        n_pes += len(ohi)
    assert n_pes > 0
    gix.close()
