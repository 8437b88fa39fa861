"""The rules that choose a search's plan, compiled for the CPU: they see sizes only, and an occupancy that the test makes up."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "pag_plan.h"
// arguments: nq others b ef waves_per_cu; a CU holds that many waves of the kernel, 160 KB of LDS; 256 CUs
// or: calls queries, for pag_queries_beside; or one number, for pag_resident: of a single wave, of a team;
// or d half b ef nq waves room and two more, for pag_paced
int main(int n, char** v) {
    if (n == 3) { std::printf("0 %llu\n", (unsigned long long)pag_queries_beside(strtoull(v[1], 0, 10), strtoull(v[2], 0, 10))); return 0; }
    if (n == 2) { std::printf("%d %d\n", pag_resident(atoi(v[1]), 256, 1), pag_resident(atoi(v[1]), 256, 4)); return 0; }
    if (n == 10) { std::printf("%d\n", (int)pag_paced(atoi(v[1]), atoi(v[2]) != 0, atoi(v[3]), atoi(v[4]), atoi(v[5]), atoi(v[6]), atoi(v[7]))); return 0; }
    pag_team_request r = {};
    r.nq = strtoull(v[1], 0, 10); r.others = strtoull(v[2], 0, 10); r.b = atoi(v[3]); r.ef = atoi(v[4]);
    const uint32_t per_cu = atoi(v[5]);
    r.num_cu = 256; r.lds_per_cu = 163840; r.most_waves = 12;
    r.hlog = 9; r.blog = r.b + 8 * std::max(r.ef, r.b) > 1024 ? 15 : 0;
    pag_team_plan p;
    auto lds = [&](uint32_t h, uint32_t bl) { return 6144u + (4u << h) + (bl ? (1u << bl) / 8 : 0u); };
    auto resident = [&](uint32_t w, uint32_t bytes, int* n) { *n = pag_resident((int)std::min(per_cu / w, 163840 / bytes), 256, w); return 0; };
    const int rc = pag_plan_team(r, lds, resident, &p);
    std::printf("%d %u\n", rc, p.waves);
}
"""


@pytest.fixture(scope="module")
def waves(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_06660_amd", "csrc"),
                           str(d / "plan.cpp"), "-o", str(d / "plan")])

    def beside(calls, queries):
        return int(subprocess.check_output([str(d / "plan"), str(calls), str(queries)], text=True).split()[1])

    def run(nq, others=0, b=10, ef=256, per_cu=16):
        rc, w = subprocess.check_output([str(d / "plan")] + [str(x) for x in (nq, others, b, ef, per_cu)], text=True).split()
        assert rc == "0"
        return int(w)
    run.beside = beside
    run.paced = lambda *a: bool(int(subprocess.check_output([str(d / "plan")] + [str(int(x)) for x in a] + ["paced", ""], text=True)))
    run.resident = lambda per_cu: [int(x) for x in subprocess.check_output([str(d / "plan"), str(per_cu)], text=True).split()]
    return run


@pytest.mark.parametrize("nq,others,want", [(1, 0, 12), (256, 0, 12), (257, 0, 8), (512, 0, 8), (513, 0, 4), (1024, 0, 4), (1025, 0, 1)])
def test_waves_of_a_call_alone(waves, nq, others, want):
    assert waves(nq, others) == want


# what another call searches meanwhile counts like queries of this one: the sum decides
@pytest.mark.parametrize("nq,others,want", [(64, 192, 12), (64, 193, 8), (256, 256, 8), (256, 768, 4), (256, 769, 1), (1, 1024, 1),
                                            (512, 1536, 1), (1, 10000, 1)])
def test_waves_beside_other_calls(waves, nq, others, want):
    assert waves(nq, others) == want


# more than two queries to a CU: four waves for searches of any length and working sets of any size, as long as all queries are resident
@pytest.mark.parametrize("b,ef", [(10, 1), (10, 127), (10, 100000), (64, 256), (128, 1000), (256, 300)])
def test_four_waves(waves, b, ef):
    assert [waves(nq, b=b, ef=ef) for nq in (513, 1024, 1025)] == [4, 4, 1]
    assert [waves(nq, b=b, ef=ef, per_cu=15) for nq in (513, 768, 769, 1024)] == [4, 4, 1, 1]
    assert waves(513, b=b, ef=ef, per_cu=11) == 1


@pytest.mark.parametrize("calls,queries,want", [(0, 0, 0), (1, 64, 64), (3, 1000, 1000), (7, 448, 192), (7, 1792, 768), (15, 3 * 2 ** 31, 3 * 2 ** 31 // 5)])
def test_calls_beyond_the_hardware_queues_wait(waves, calls, queries, want):
    assert waves.beside(calls, queries) == want


# per_cu: waves that the registers of the made-up kernel leave room for on a CU
@pytest.mark.parametrize("nq,per_cu,want", [(1, 12, 12), (1, 11, 11), (256, 4, 4), (256, 3, 1), (1, 0, 1), (512, 16, 8), (512, 15, 4), (512, 12, 4),
                                              (512, 8, 4), (512, 7, 1)])
def test_a_team_that_does_not_fit_is_not_planned(waves, nq, per_cu, want):
    assert waves(nq, per_cu=per_cu) == want


def test_a_single_wave_is_always_resident(waves):
    assert waves.resident(0) == [256, 0] and waves.resident(-1) == [256, 0] and waves.resident(3) == [768, 768]


# d, 16-bit, b, efS, queries, waves launched, waves that the GPU holds
@pytest.mark.parametrize("want,args", [(True, (768, False, 10, 1408, 10000, 3334, 4096)), (True, (768, False, 64, 256, 4097, 3072, 4096)),
                                       (True, (1024, False, 10, 256, 3100, 1550, 3072)), (False, (768, False, 10, 1408, 4200, 2100, 4096)),
                                       (False, (768, False, 10, 1408, 4096, 4096, 4096)), (False, (768, False, 10, 255, 10000, 3334, 4096)),
                                       (False, (768, False, 65, 1408, 10000, 3334, 4096)), (False, (764, False, 10, 1408, 10000, 3334, 4096)),
                                       (False, (768, True, 10, 1408, 10000, 3334, 4096)), (False, (768, False, 10, 1408, 10000, 64, 4096)),
                                       (False, (1536, False, 10, 1408, 10000, 64, 3072))])
def test_pacing(waves, want, args):
    """Long fp32 rows, small working sets, long searches, and a GPU that stays full: a batch of which the scratch array of the
    allocation-free entry point holds few waves does not keep it so."""
    assert waves.paced(*args) == want
