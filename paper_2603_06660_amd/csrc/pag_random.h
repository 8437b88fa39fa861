// Random structures of the method, drawn on the host once per index (Sec. 3.1; Alg. 1): what the orthogonal transform Q
// from the Haar measure (Gaussian matrix, Gram-Schmidt with re-orthogonalisation) and the codebooks (per subspace,
// independently rotated cross-polytopes) are made of.  No HIP, so that it can be compiled for a CPU.
// Counter-based generator: SplitMix64 on (seed, stream, counter) + Box-Muller.
#pragma once

#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <system_error>
#include <thread>
#include <vector>

namespace pag_random {

struct Rng {
    uint64_t state;
    explicit Rng(uint64_t seed, uint64_t stream) : state(seed * 0x9E3779B97F4A7C15ull + stream * 0xD1B54A32D192ED03ull + 0x2545F4914F6CDD1Dull) {}
    uint64_t next() {
        uint64_t z = (state += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }
    double uniform() { return ((double)(next() >> 11) + 0.5) * (1.0 / 9007199254740992.0); }
    double normal() {
        const double u1 = uniform(), u2 = uniform();
        return sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925 * u2);
    }
};

// fn(lo, hi) over parts of [0, count), on up to eight host threads; parts whose thread cannot be started run on this one
template <class F>
inline void on_threads(size_t count, F&& fn) {
    const size_t threads = std::max(1u, std::min(8u, std::thread::hardware_concurrency()));
    auto from = [&](size_t t) { return count * t / threads; };
    struct Joined {
        std::vector<std::thread> all;
        ~Joined() { for (auto& t : all) t.join(); }
    } started;
    started.all.reserve(threads);
    size_t t = 1;
    try {
        for (; t < threads; ++t) started.all.emplace_back(fn, from(t), from(t + 1));
    } catch (const std::system_error&) {
    }
    fn(size_t(0), from(1));
    if (t < threads) fn(from(t), count);
}

// Fills g with normals, two draws each, in order.  The generator's state advances by a constant per draw, so several
// threads can start where their part of g begins.
inline void draw_normals(const Rng& first, std::vector<double>& g) {
    auto part = [&](size_t lo, size_t hi) {
        Rng rng = first;
        rng.state += 2ull * lo * 0x9E3779B97F4A7C15ull;
        for (size_t i = lo; i < hi; ++i) g[i] = rng.normal();
    };
    if (g.size() < (1u << 16)) part(0, g.size());
    else on_threads(g.size(), part);
}

// Orthonormalise the columns of the dim x dim Gaussian matrix g (column-major) in place:
// classical Gram-Schmidt with one re-orthogonalisation pass, both inner loops split over threads where they are long.
inline void orthonormalise(std::vector<double>& g, uint32_t dim) {
    std::vector<double> proj(dim);
    for (uint32_t j = 0; j < dim; ++j) {
        double* aj = &g[(size_t)j * dim];
        auto project = [&](size_t lo, size_t hi) {
            for (size_t i = lo; i < hi; ++i) {
                const double* qi = &g[i * dim];
                double s = 0.0;
                for (uint32_t k = 0; k < dim; ++k) s += qi[k] * aj[k];
                proj[i] = s;
            }
        };
        auto subtract = [&](size_t lo, size_t hi) {
            for (uint32_t i = 0; i < j; ++i) {
                const double* qi = &g[(size_t)i * dim];
                const double p = proj[i];
                for (size_t k = lo; k < hi; ++k) aj[k] -= p * qi[k];
            }
        };
        for (int pass = 0; pass < 2 && j > 0; ++pass) {
            if (j < 256) { project(0, j); subtract(0, dim); }
            else { on_threads(j, project); on_threads(dim, subtract); }
        }
        double nrm = 0.0;
        for (uint32_t k = 0; k < dim; ++k) nrm += aj[k] * aj[k];
        nrm = sqrt(nrm);
        for (uint32_t k = 0; k < dim; ++k) aj[k] /= nrm;
    }
}

}  // namespace pag_random
