"""RobustPrune with four waves and with one wave per node: both keep what Eq. 1 keeps of a candidate list, in order, and the same."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PER_CU = {1: 0, 2: 0, 3: 0, 4: 32, 6: 8, 8: 0, 12: 3}        # chunks of a row: nodes per CU up to which four waves take a node; 0: always


def test_rule(tmp_path):
    (tmp_path / "plan.cpp").write_text('#include <cstdio>\n#include "pag_plan.h"\nint main() { for (uint32_t c : {1, 2, 3, 4, 6, 8, 12})\n'
                                       '    std::printf("%lld ", (long long)(pag_prune_line(c, 256) == PAG_ANY_BATCH ? 0 : pag_prune_line(c, 256))); }\n')
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_06660_amd", "csrc"),
                           str(tmp_path / "plan.cpp"), "-o", str(tmp_path / "plan")])
    assert [int(x) for x in subprocess.check_output([str(tmp_path / "plan")], text=True).split()] == [256 * x for x in PER_CU.values()]


def _chunks(d):
    return next(c for c in PER_CU if c >= -(-d // 256))


def _rows_in_lds(d, m, cus, deg):
    """Kept rows that a node's four waves hold on the chip."""
    room = min(65536, 163840 // min(-(-m // cus), 4) - 512)
    return min((room - 544) // (1024 * _chunks(d)) - 1, deg)


def _keep(x, v, cand, deg):
    """Eq. 1 over candidates in ascending (distance, id) order; distances as the library rounds them."""
    kept = []
    for c in cand:
        if c == v or len(kept) == deg:
            continue
        dv = np.float32(np.sum((x[c] - x[v]).astype(np.float64) ** 2))
        if not kept or not (np.sum((x[kept] - x[c]).astype(np.float64) ** 2, axis=1).astype(np.float32) <= dv).any():
            kept.append(c)
    return kept


def _grown(base, old, batches, flags=0, **kw):
    """An index of the first `old` rows, and what batches of these sizes become that follow it, each on a copy of its own.  Reverse
    edges change records of older nodes only, those of the batch's own are as they were pruned."""
    from paper_2603_06660_amd import FLAG_KEEP_ORDER, FLAG_NO_PES, PagIndex
    kw, flags = dict(metric="l2", seed=11, **kw), FLAG_KEEP_ORDER | FLAG_NO_PES | flags
    ix = PagIndex.build(base[:old].contiguous(), flags=flags, **kw)
    e = ix.export()
    ix.close()
    arrays = [e[k] for k in ("vectors", "adj", "a", "c", "e2", "codes", "rotation", "codebooks", "entry")]
    out = []
    for m in batches:
        ix = PagIndex.from_arrays(*arrays, metric="l2", ef_construction=kw["ef_construction"], capacity=old + m, flags=flags, insert_subbatch=m)
        cand = ix.insertion_candidates(base[old:old + m][::max(1, m // 24)].contiguous(), kw["ef_construction"])
        ix.insert(base[old:old + m].contiguous())
        assert ix.counters()["relinked_batches"] == 0
        ex = ix.export()
        ix.close()
        out.append((ex["vectors"], ex["adj"].reshape(old + m, kw["max_degree"])[old:], cand))
    return out


def _check(x, adj, cand, old, m, deg):
    """The sampled nodes against Eq. 1; how many neighbours each kept."""
    ids, _, count, *_ = cand
    for k, i in enumerate(range(0, m, max(1, m // 24))):
        want = _keep(x, old + i, [int(c) for c in ids[k][:int(count[k])]], deg)
        # sums in another order differ by one part in 2^50: ties at 2^24 do not occur in these draws
        assert [int(a) for a in adj[i] if a != 0xFFFFFFFF] == want, i
    return (adj != 0xFFFFFFFF).sum(axis=1)


@pytest.mark.gpu
# d: 1 .. 12 chunks a lane, with and without a rest; batches in which one to four nodes share a CU; candidates: fewer than a step of
# eight, not a multiple of it, several steps.  `fills`: some node keeps as many as its degree allows, and more than the LDS holds where that is less
@pytest.mark.parametrize("d,P,deg,efc,m,half,fills", [(32, 8, 8, 6, 40, False, False), (64, 8, 10, 90, 800, False, True), (256, 16, 64, 203, 300, False, False),
                                                      (260, 20, 16, 150, 800, False, True), (768, 32, 20, 120, 900, False, True), (768, 32, 24, 120, 520, True, True),
                                                      (1024, 32, 18, 117, 260, False, True), (1024, 32, 18, 117, 1100, False, True), (1536, 64, 12, 90, 600, False, True),
                                                      (2048, 64, 12, 100, 800, False, True), (3072, 64, 10, 90, 24, False, True), (3072, 64, 10, 90, 768, False, True)])
def test_four_waves(d, P, deg, efc, m, half, fills):
    import torch
    from paper_2603_06660_amd import FLAG_FP16_VECTORS
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert not PER_CU[_chunks(d)] or m <= PER_CU[_chunks(d)] * cus
    old = max(2 * m, 300)
    base = torch.from_numpy(np.random.default_rng(d + m).standard_normal((old + m, d), dtype=np.float32)).cuda()
    (x, adj, cand), = _grown(base, old, [m], flags=FLAG_FP16_VECTORS if half else 0, max_degree=deg, num_subspaces=P, ef_construction=efc)
    kept = _check(x, adj, cand, old, m, deg)
    assert not fills or kept.max() == deg
    assert not fills or deg <= _rows_in_lds(d, m, cus, 64) or kept.max() > _rows_in_lds(d, m, cus, deg)


@pytest.mark.gpu
# row lengths that have both; more neighbours kept than either holds in LDS
@pytest.mark.parametrize("d,P,deg,efc", [(772, 4, 20, 40), (1040, 40, 24, 60), (1536, 64, 24, 60), (2064, 43, 16, 60), (3072, 64, 16, 60)])
def test_one_wave_and_four(d, P, deg, efc):
    """The same nodes in the largest batch that gets four waves per node and in one that is a node too large for that."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    line = PER_CU[_chunks(d)] * cus
    old = 2 * (line + 1)
    base = torch.from_numpy(np.random.default_rng(d).standard_normal((old + line + 1, d), dtype=np.float32)).cuda()
    kw = dict(max_degree=deg, num_subspaces=P, ef_construction=efc)
    (x, four, cand), (y, one, cand1) = _grown(base, old, [line, line + 1], **kw)
    kept = _check(x, four, cand, old, line, deg)
    _check(y, one, cand1, old, line + 1, deg)
    assert np.array_equal(four, one[:line])
    assert kept.max() > max(4, 16 // _chunks(d)) and kept.max() > _rows_in_lds(d, line, cus, deg)
