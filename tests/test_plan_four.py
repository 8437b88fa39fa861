"""Teams of four where more than two and up to four queries come to a CU: the rule on the CPU, the answers on the GPU."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "pag_plan.h"
// arguments: nq others b ef nodes waves_per_cu; a CU holds that many waves of the kernel, 160 KB of LDS; 256 CUs
int main(int, char** v) {
    pag_team_request r = {};
    r.nq = strtoull(v[1], 0, 10); r.others = strtoull(v[2], 0, 10); r.b = atoi(v[3]); r.ef = atoi(v[4]);
    const uint32_t per_cu = atoi(v[6]);
    r.d = 128; r.num_cu = 256; r.lds_per_cu = 163840; r.most_waves = 12;
    r.hlog = 9; r.blog = r.b + 8 * std::max(r.ef, r.b) > 1024 ? 15 : 0;
    pag_team_plan p;
    auto lds = [&](uint32_t h, uint32_t bl) { return 6144u + (4u << h) + (bl ? (1u << bl) / 8 : 0u); };
    auto resident = [&](uint32_t w, uint32_t bytes, int* n) { *n = pag_resident((int)std::min(per_cu / w, 163840 / bytes), 256, w); return 0; };
    const int rc = pag_plan_four(r, strtoull(v[5], 0, 10), lds, resident, &p);
    std::printf("%d %u %u\n", rc, p.waves, p.waves > 1 ? p.lds : 0);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_06660_amd", "csrc"),
                           str(d / "plan.cpp"), "-o", str(d / "plan")])

    def run(*a):
        rc, waves, lds = (int(x) for x in subprocess.check_output([str(d / "plan")] + [str(x) for x in a], text=True).split())
        assert rc == 0 and 4 * (lds + 512) <= 163840          # four of them fit a CU
        return waves
    return run


# nq, others, b, ef, nodes, waves a CU holds
@pytest.mark.parametrize("args,want", [((512, 0, 10, 32, 10000, 16), 1), ((513, 0, 10, 32, 10000, 16), 4), ((1024, 0, 100, 10, 10000, 16), 4),
                                       ((1025, 0, 10, 128, 10000, 16), 1), ((100, 500, 10, 64, 10000, 16), 4), ((1000, 25, 10, 64, 10000, 16), 1),
                                       ((1000, 0, 10, 64, 1023, 16), 1), ((1000, 0, 10, 64, 1024, 16), 4), ((768, 0, 300, 300, 10000, 12), 4),
                                       ((769, 0, 300, 300, 10000, 12), 1), ((600, 0, 10, 100000, 10000, 16), 4), ((600, 0, 10, 64, 10000, 3), 1)])
def test_rule(plan, args, want):
    assert plan(*args) == want


@pytest.mark.gpu
# n, d, subspaces, degree, metric, half, K, efS
@pytest.mark.parametrize("n,d,P,deg,metric,half,K,efS", [(1024, 32, 8, 16, "l2", False, 1, 4), (3000, 128, 16, 32, "l2", False, 10, 64),
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
