"""The orthogonal transform of an index is the same, bit for bit, whichever way the library orthogonalises it.

The library's host routine, compiled for the CPU by itself, is held against a reference in Python; the transform of a built index,
which the GPU orthogonalised from d = 192 on, against the host routine on the same matrix."""
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "pag_random.h"
int main(int, char** v) {          // seed d file
    const uint32_t d = atoi(v[2]);
    std::vector<double> g((size_t)d * d);
    pag_random::draw_normals(pag_random::Rng(strtoull(v[1], 0, 10), 1), g);
    pag_random::orthonormalise(g, d);
    FILE* f = fopen(v[3], "wb");
    for (double x : g) { const float y = (float)x; fwrite(&y, 4, 1, f); }
    return fclose(f);
}
"""


@pytest.fixture(scope="module")
def host_routine(tmp_path_factory):
    at = tmp_path_factory.mktemp("transform")
    (at / "host.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-pthread", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2603_06660_amd", "csrc"), str(at / "host.cpp"), "-o", str(at / "host")])

    def run(seed, d):
        subprocess.check_call([str(at / "host"), str(seed), str(d), str(at / "q")])
        return np.fromfile(at / "q", np.float32).reshape(d, d)
    return run

MASK = (1 << 64) - 1


def _normals(seed, count):
    """SplitMix64 (stream 1 of the seed) and Box-Muller, as the library draws Q's Gaussian matrix."""
    state = (seed * 0x9E3779B97F4A7C15 + 0xD1B54A32D192ED03 + 0x2545F4914F6CDD1D) & MASK
    out = np.empty(count)

    def uniform():
        nonlocal state
        state = (state + 0x9E3779B97F4A7C15) & MASK
        z = state
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & MASK
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & MASK
        return (float((z ^ (z >> 31)) >> 11) + 0.5) * (1.0 / 9007199254740992.0)

    for i in range(count):
        u1, u2 = uniform(), uniform()
        out[i] = math.sqrt(-2.0 * math.log(u1)) * math.cos(6.283185307179586476925 * u2)
    return out


def _orthonormalise(g):
    """Classical Gram-Schmidt with one re-orthogonalisation pass; row j of g is column j of the Gaussian matrix.  Sums run
    in index order (vectorised over the independent ones only)."""
    d = g.shape[0]
    for j in range(d):
        for _ in range(2 if j else 0):
            s = np.zeros(j)
            for k in range(d):
                s = s + g[:j, k] * g[j, k]
            for i in range(j):
                g[j] = g[j] - s[i] * g[i]
        n = 0.0
        for x in g[j].tolist():
            n = n + x * x
        g[j] = g[j] / math.sqrt(n)
    return g.astype(np.float32)


def test_reference_is_orthogonal():
    q = _orthonormalise(_normals(9, 48 * 48).reshape(48, 48)).astype(np.float64)
    assert np.abs(q @ q.T - np.eye(48)).max() < 1e-6


@pytest.mark.parametrize("d", [4, 48, 128, 300])                     # 300: columns that several threads share
def test_host_routine(host_routine, d):
    got, want = host_routine(77 + d, d), _orthonormalise(_normals(77 + d, d * d).reshape(d, d))
    # the logarithms and cosines are the same C library's; where they are not, a last bit of fp64 in the matrix can tip the
    # rounding to fp32 of about one entry in 2^29 / 100
    assert (got != want).mean() <= 1e-6 and np.all(np.abs(got - want) <= np.spacing(np.abs(want)))


@pytest.mark.gpu
# below and above the line at 192, chunks of 64 with and without a rest, more than one element per thread of the normalisation (1024)
@pytest.mark.parametrize("d", [128, 188, 192, 196, 256, 260, 1028])
def test_transform_bits(host_routine, d):
    import torch
    from paper_2603_06660_amd import PagIndex
    seed = 1234 + d
    base = torch.from_numpy(np.random.default_rng(d).standard_normal((64, d), dtype=np.float32)).cuda()
    ix = PagIndex.build(base, metric="l2", max_degree=8, num_subspaces=4, ef_construction=20, seed=seed)
    got = ix.export()["rotation"]
    ix.close()
    assert np.array_equal(got, host_routine(seed, d))


@pytest.mark.gpu
def test_build_without_room_for_the_workspace():
    """The orthogonalisation's workspace (16 d^2 bytes) does not fit the memory that is left, the index does: the host
    orthogonalises instead, to the same bits."""
    import torch
    from paper_2603_06660_amd import PagIndex
    d = 2560
    base = torch.from_numpy(np.random.default_rng(d).standard_normal((64, d), dtype=np.float32)).cuda()

    def rotation():
        ix = PagIndex.build(base, metric="l2", max_degree=8, num_subspaces=16, ef_construction=20, seed=7)
        r = ix.export()["rotation"]
        ix.close()
        return r

    want = rotation()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    filler = []
    try:
        for block in (1 << 30, 48 << 20):                   # until there is less than 48 MB in one piece
            while True:
                try:
                    filler.append(torch.empty(block, dtype=torch.uint8, device="cuda"))
                except torch.OutOfMemoryError:
                    break
        filler.pop()                                        # 48 to 96 MB are left
        torch.cuda.empty_cache()
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(16 * d * d, dtype=torch.uint8, device="cuda")
        assert np.array_equal(rotation(), want)
    finally:
        filler.clear()
        torch.cuda.empty_cache()
