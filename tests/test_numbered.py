"""Which workgroup takes which query of a batch that is larger than the launch: the rule on the CPU, the answers on the GPU."""
import heapq
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "pag_plan.h"
// arguments: bytes of LDS, of a CU; or nq groups sure
int main(int n, char** v) {
    if (n == 3) std::printf("%u\n", pag_lds_room(atoi(v[1]), atoi(v[2])));
    else std::printf("%llu\n", (unsigned long long)pag_numbered(strtoull(v[1], 0, 10), strtoull(v[2], 0, 10), strtoull(v[3], 0, 10)));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_06660_amd", "csrc"),
                           str(d / "plan.cpp"), "-o", str(d / "plan")])
    return lambda *a: int(subprocess.check_output([str(d / "plan")] + [str(x) for x in a], text=True))


# as measured with workgroups that do nothing but wait
@pytest.mark.parametrize("bytes_,room", [(5120, 32), (5121, 25), (6144, 25), (8192, 18), (11520, 14), (11904, 12), (12800, 12), (32384, 4), (0, 128)])
def test_lds_is_handed_out_in_pieces(rule, bytes_, room):
    assert rule(bytes_, 163840) == room


def _end(nq, groups, places, numbered):
    """When the batch ends, with searches of one unit each: a workgroup searches until no query is left, the next one takes its place."""
    taken, free, waiting, end = numbered, [0.0] * places, list(range(groups)), 0
    heapq.heapify(free)
    running = []                                            # (time, workgroup) at which a workgroup asks for its next query
    while waiting or running:
        while waiting and free:
            t, g = heapq.heappop(free), waiting.pop(0)
            if numbered:
                heapq.heappush(running, (t + 1, g))
                end = max(end, t + 1)
            else:
                heapq.heappush(running, (t, g))
        t, g = heapq.heappop(running)
        if taken < nq:
            taken += 1
            heapq.heappush(running, (t + 1, g))
            end = max(end, t + 1)
        else:
            heapq.heappush(free, t)
    return end


@pytest.mark.parametrize("nq,groups,sure,want", [(3328, 3328, 3072, 3328), (100, 128, 64, 128), (4000, 3328, 3328, 3328), (4000, 3328, 3327, 0), (10000, 3334, 4096, 3334)])
def test_rule(rule, nq, groups, sure, want):
    assert rule(nq, groups, sure) == want


@pytest.mark.parametrize("nq,groups,places", [(40, 33, 30), (66, 33, 30), (33, 33, 30), (40, 30, 30), (99, 33, 32)])
def test_no_query_is_kept_for_the_end(rule, nq, groups, places):
    assert _end(nq, groups, places, rule(nq, groups, places)) == -(-nq // min(places, groups))


@pytest.mark.gpu
# efS and K: the footprint with K = 100 lets the GPU hold fewer waves than it is asked to; with K = 10 all find a place
@pytest.mark.parametrize("K,efS", [(100, 120), (10, 40)])
def test_answers(K, efS):
    """A batch of two rounds that nearly fill the GPU against the same queries in batches of one."""
    import torch
    from paper_2603_06660_amd import PagIndex
    rng = np.random.default_rng(K)
    scale = (np.arange(1, 769) ** -0.3).astype(np.float32)
    rows = lambda m: torch.from_numpy(rng.standard_normal((m, 768), dtype=np.float32) * scale).cuda()
    ix = PagIndex.build(rows(1500), metric="l2", max_degree=32, num_subspaces=32, ef_construction=60, seed=5)
    waves, room = ix.search_layout(1 << 20, K, efS)
    assert waves == 1
    q = rows(2 * room - 50)
    want = [tuple(t.clone() for t in ix.search(q[s:s + 1500].contiguous(), K, efS)) for s in range(0, q.shape[0], 1500)]
    ids, dists = ix.search(q, K, efS)
    assert torch.equal(ids, torch.cat([w[0] for w in want])) and torch.equal(dists, torch.cat([w[1] for w in want]))
    ix.close()
