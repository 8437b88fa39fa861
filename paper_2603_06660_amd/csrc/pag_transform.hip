// The random orthogonal transform Q of an index (Sec. 3.1; Alg. 1): classical Gram-Schmidt with one
// re-orthogonalisation pass over a Gaussian matrix, on the GPU.  Every sum runs in index order with a
// rounding after each product and each addition, as a plain loop on the host would compute it, so that a
// seed gives the same Q wherever the orthogonalisation runs.
//
// What bounds it is the latency of fp64 additions: a column's projections (over all earlier columns), its update (over
// all of its elements) and its norm are chains of dependent additions, and a column needs the one before it finished.
//   The chains of 16 neighbours belong to one workgroup (gs_panel): eight waves fetch and multiply, a ninth adds from LDS
//     and does nothing else, so that a step costs it one addition and half an LDS read.  (A wave that fetched, broadcast
//     its factors and multiplied besides took 17 us for chains of 768, this takes 7.)
//   The first pass works with the columns as drawn, so it does not wait for the column before: 16 columns at a time are
//     projected on everything finished before them in one launch, and as each of the 16 is finished the others are projected
//     on it (k_gs_finish).  What is left for each column is the second pass and its norm: three launches instead of five.
// d = 768: 48 ms as five launches a column, 21.5 ms now (7 us a projection, 5.5 an update, 14 the norm and the block's first pass;
// at 8 clocks an addition the chains alone are 9 ms); 300 ms on eight host threads.
// The matrix is kept twice, in pairs of rows and in pairs of columns, so that neighbouring threads read neighbouring
// addresses in both.
#include "pag_internal.h"

namespace {

constexpr u32 GS_BLOCK = 16;                 // chains of a workgroup, columns of a block
constexpr u32 GS_CHUNK = 128;                // steps between two barriers
constexpr u32 GS_LOADERS = 512;              // threads that fetch and multiply; one more wave adds
constexpr u32 GS_THREADS = GS_LOADERS + 64;
constexpr u32 GS_ITEMS = GS_CHUNK / 2 * GS_BLOCK / GS_LOADERS;      // pairs that one of them has in a chunk
constexpr u32 GS_AHEAD = 4;                  // chunks on their way

// where element k of vector i lies: pairs of k side by side, then i (`rows`); pairs of i, then k (`cols`)
__device__ __forceinline__ u64 in_rows(u32 i, u32 k, u32 ld) { return ((u64)(k / 2) * ld + i) * 2 + (k & 1); }
__device__ __forceinline__ u64 in_cols(u32 i, u32 k, u32 ld) { return ((u64)(i / 2) * ld + k) * 2 + (i & 1); }

// LDS traffic only: loads from memory stay in flight
__device__ __forceinline__ void gs_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A chunk of this lane's chain: products in pairs, GS_BLOCK chains side by side.
template <bool SUB>
__device__ __forceinline__ double gs_add(const double2* products, double acc) {
    constexpr u32 G = 8;
    double2 v[2][G];
#pragma unroll
    for (u32 t = 0; t < G; ++t) v[0][t] = products[t * GS_BLOCK];
#pragma unroll
    for (u32 g = 0; g < GS_CHUNK / 2 / G; ++g) {
        if (g + 1 < GS_CHUNK / 2 / G) {
#pragma unroll
            for (u32 t = 0; t < G; ++t) v[(g + 1) & 1][t] = products[((g + 1) * G + t) * GS_BLOCK];
        }
#pragma unroll
        for (u32 t = 0; t < G; ++t) {
            const double2 p = v[g & 1][t];
            acc = SUB ? acc - p.x : acc + p.x;
            acc = SUB ? acc - p.y : acc + p.y;
        }
    }
    return acc;
}

// Chains c = 0 .. 15: acc (+/-)= m[(p * ld + c)].{x,y} * factor[p].{x,y} over p = 0 .. count / 2 - 1, in order; count is a
// multiple of GS_CHUNK.  Lanes 0 .. 15 of the last wave pass their acc and receive the sums; the other threads' results mean
// nothing.  products: LDS, two chunks.
template <bool SUB>
__device__ __forceinline__ double gs_panel(const double2* m, u32 ld, const double2* factor, u32 count, double acc, double2* products) {
    const u32 chunks = count / GS_CHUNK, chain = threadIdx.x % GS_BLOCK, pair = threadIdx.x / GS_BLOCK;
    if (threadIdx.x < GS_LOADERS) {
        double2 v[GS_AHEAD][GS_ITEMS], f[GS_AHEAD][GS_ITEMS];
        auto fetch = [&](u32 g, double2 (&fv)[GS_ITEMS], double2 (&ff)[GS_ITEMS]) {
#pragma unroll
            for (u32 t = 0; t < GS_ITEMS; ++t) {
                const u32 p = g * (GS_CHUNK / 2) + t * (GS_LOADERS / GS_BLOCK) + pair;
                fv[t] = m[(u64)p * ld + chain];
                ff[t] = factor[p];
            }
        };
#pragma unroll
        for (u32 a = 0; a < GS_AHEAD; ++a) fetch(a < chunks ? a : chunks - 1, v[a], f[a]);
        for (u32 g0 = 0; g0 < chunks; g0 += GS_AHEAD) {
#pragma unroll
            for (u32 a = 0; a < GS_AHEAD; ++a) {
                const u32 g = g0 + a;
                if (g < chunks) {
                    double2* to = products + (g & 1) * (GS_CHUNK / 2 * GS_BLOCK);
#pragma unroll
                    for (u32 t = 0; t < GS_ITEMS; ++t)
                        to[(t * (GS_LOADERS / GS_BLOCK) + pair) * GS_BLOCK + chain] = make_double2(v[a][t].x * f[a][t].x, v[a][t].y * f[a][t].y);
                    if (g + GS_AHEAD < chunks) fetch(g + GS_AHEAD, v[a], f[a]);
                    gs_barrier();
                }
            }
        }
    } else {
        for (u32 g = 0; g < chunks; ++g) {
            gs_barrier();            // chunk g is complete; the loaders are one chunk ahead from here on
            acc = gs_add<SUB>(products + (g & 1) * (GS_CHUNK / 2 * GS_BLOCK) + chain, acc);
        }
    }
    return acc;
}

// the thread that holds chain c of a workgroup's panel, or -1
__device__ __forceinline__ int gs_chain() {
    const int c = (int)threadIdx.x - (int)GS_LOADERS;
    return c >= 0 && c < (int)GS_BLOCK ? c : -1;
}

// proj[y][i] = <vector i, column y of the block> for all i of `rows` (zeros where vector i is not finished)
__global__ void __launch_bounds__(GS_THREADS) k_gs_project(const double* __restrict__ rows, u32 ld, const double* __restrict__ cur,
                                                           double* __restrict__ proj) {
    __shared__ __align__(16) double2 products[2 * (GS_CHUNK / 2) * GS_BLOCK];
    const u32 i0 = blockIdx.x * GS_BLOCK;
    const double s = gs_panel<false>((const double2*)rows + i0, ld, (const double2*)(cur + (u64)blockIdx.y * ld), ld, 0.0, products);
    const int c = gs_chain();
    if (c >= 0) proj[(u64)blockIdx.y * ld + i0 + c] = s;
}

// column y of the block -= sum_i proj[y][i] * vector i, i ascending; proj is zero where vector i is not finished
__global__ void __launch_bounds__(GS_THREADS) k_gs_update(const double* __restrict__ cols, u32 ld, u32 count, double* __restrict__ cur,
                                                          const double* __restrict__ proj) {
    __shared__ __align__(16) double2 products[2 * (GS_CHUNK / 2) * GS_BLOCK];
    const u32 k0 = blockIdx.x * GS_BLOCK;
    const int c = gs_chain();
    double* at = cur + (u64)blockIdx.y * ld + k0;
    const double a = gs_panel<true>((const double2*)cols + k0, ld, (const double2*)(proj + (u64)blockIdx.y * ld), count, c >= 0 ? at[c] : 0.0, products);
    if (c >= 0) at[c] = a;
}

// The block's columns as drawn: `cur` (column after column) is worked on, `drawn` (pairs of k, then the column) stays.
__global__ void __launch_bounds__(256) k_gs_begin(const double* __restrict__ cols, u32 j0, u32 ld, double* __restrict__ cur, double* __restrict__ drawn) {
    const u32 k = blockIdx.x * 256 + threadIdx.x, c = blockIdx.y;
    if (k >= ld) return;
    const double x = cols[in_cols(j0 + c, k, ld)];
    cur[(u64)c * ld + k] = x;
    drawn[in_rows(c, k, GS_BLOCK)] = x;
}

// Column j = j0 + c to unit length: it is finished, into both layouts and into row j of Q.  The first pass of the block's later
// columns over it.
__global__ void __launch_bounds__(GS_THREADS) k_gs_finish(double* __restrict__ cols, double* __restrict__ rows, u32 j0, u32 c, u32 dim, u32 ld,
                                                          double* __restrict__ cur, const double* __restrict__ drawn, float* __restrict__ rot) {
    extern __shared__ __align__(16) unsigned char smem[];
    double2* products = (double2*)smem;                              // two chunks
    double* a = (double*)(products + 2 * (GS_CHUNK / 2) * GS_BLOCK);     // [ld]
    __shared__ double norm, on_it[GS_BLOCK];
    const u32 j = j0 + c;
    for (u32 k = threadIdx.x; k < ld; k += GS_THREADS) a[k] = cur[(u64)c * ld + k];
    __syncthreads();
    if (threadIdx.x >= GS_LOADERS) {
        const double2* pairs = (const double2*)a;
        double s = 0.0;
        for (u32 p0 = 0; p0 < ld / 2; p0 += 16) {                     // ld is a multiple of GS_CHUNK
            double2 v[16];
#pragma unroll
            for (u32 t = 0; t < 16; ++t) v[t] = pairs[p0 + t];
#pragma unroll
            for (u32 t = 0; t < 16; ++t) {
                s = s + v[t].x * v[t].x;
                s = s + v[t].y * v[t].y;
            }
        }
        if (threadIdx.x == GS_LOADERS) norm = sqrt(s);
    }
    __syncthreads();
    const double n = norm;
    for (u32 k = threadIdx.x; k < ld; k += GS_THREADS) {
        const double x = a[k] / n;
        a[k] = x;
        cols[in_cols(j, k, ld)] = x;
        rows[in_rows(j, k, ld)] = x;
        if (k < dim) rot[(u64)j * dim + k] = (float)x;
    }
    if (c + 1 >= GS_BLOCK || j + 1 >= dim) return;
    __syncthreads();
    const double s = gs_panel<false>((const double2*)drawn, GS_BLOCK, (const double2*)a, ld, 0.0, products);
    const int mine = gs_chain();
    if (mine >= 0) on_it[mine] = s;
    __syncthreads();
    for (u32 k = threadIdx.x; k < ld; k += GS_THREADS) {
        double x[GS_BLOCK];
#pragma unroll
        for (u32 other = 1; other < GS_BLOCK; ++other)
            if (other > c) x[other] = cur[(u64)other * ld + k];
#pragma unroll
        for (u32 other = 1; other < GS_BLOCK; ++other)
            if (other > c) cur[(u64)other * ld + k] = x[other] - on_it[other] * a[k];
    }
}

__global__ void __launch_bounds__(256) k_gs_lay_out(const double* __restrict__ g, u32 dim, u32 ld, double* __restrict__ cols) {
    const u32 k = blockIdx.x * 256 + threadIdx.x, i = blockIdx.y;
    if (k < dim) cols[in_cols(i, k, ld)] = g[(u64)i * dim + k];
}

}  // namespace

// g (host): the dim x dim Gaussian matrix, column after column; rot (dev): Q, row j = column j of the result
int pag_orthonormalise(hipStream_t s, const double* g, u32 dim, float* rot) {
    const u32 ld = (dim + GS_CHUNK - 1) / GS_CHUNK * GS_CHUNK;
    double* ws = nullptr;
    struct Release { double*& p; ~Release() { if (p) (void)hipFree(p); } } release{ws};
    const u64 matrix = (u64)ld * ld, block = (u64)GS_BLOCK * ld, doubles = 2 * matrix + 3 * block;
    hipError_t e = hipMalloc((void**)&ws, doubles * sizeof(double));
    if (e != hipSuccess) { pag_set_error(std::string("hipMalloc (transform): ") + hipGetErrorString(e)); return PAG_ENOMEM; }
    double *cols = ws, *rows = ws + matrix, *cur = ws + 2 * matrix, *drawn = cur + block, *proj = drawn + block;
    int rc;
    if ((rc = pag_launch_zero_u32(s, (u32*)ws, doubles * 2))) return rc;
    // the matrix arrives column after column in the place of `rows`, is laid out in `cols`, and `rows` starts empty
    PAG_HIP(hipMemcpyAsync(rows, g, (size_t)dim * dim * 8, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_gs_lay_out, dim3((dim + 255) / 256, dim), dim3(256), 0, s, rows, dim, ld, cols);
    if ((rc = pag_launch_zero_u32(s, (u32*)rows, matrix * 2))) return rc;
    const u32 finish_lds = 2 * (GS_CHUNK / 2) * GS_BLOCK * (u32)sizeof(double2) + ld * (u32)sizeof(double);
    for (u32 j0 = 0; j0 < dim; j0 += GS_BLOCK) {
        // vectors i < j0 are finished: j0 is a multiple of GS_BLOCK, a count of vectors is rounded up to whole chunks
        auto chunks = [&](u32 count) { return (count + GS_CHUNK - 1) / GS_CHUNK * GS_CHUNK; };
        hipLaunchKernelGGL(k_gs_begin, dim3((ld + 255) / 256, GS_BLOCK), dim3(256), 0, s, cols, j0, ld, cur, drawn);
        if (j0 > 0) {
            hipLaunchKernelGGL(k_gs_project, dim3(j0 / GS_BLOCK, GS_BLOCK), dim3(GS_THREADS), 0, s, rows, ld, cur, proj);
            hipLaunchKernelGGL(k_gs_update, dim3(ld / GS_BLOCK, GS_BLOCK), dim3(GS_THREADS), 0, s, cols, ld, chunks(j0), cur, proj);
        }
        for (u32 c = 0; c < GS_BLOCK && j0 + c < dim; ++c) {
            const u32 j = j0 + c;
            if (j > 0) {
                hipLaunchKernelGGL(k_gs_project, dim3((j + GS_BLOCK - 1) / GS_BLOCK), dim3(GS_THREADS), 0, s, rows, ld, cur + (u64)c * ld, proj);
                hipLaunchKernelGGL(k_gs_update, dim3(ld / GS_BLOCK), dim3(GS_THREADS), 0, s, cols, ld, chunks(j), cur + (u64)c * ld, proj);
            }
            hipLaunchKernelGGL(k_gs_finish, dim3(1), dim3(GS_THREADS), finish_lds, s, cols, rows, j0, c, dim, ld, cur, drawn, rot);
        }
    }
    PAG_HIP(hipGetLastError());
    PAG_HIP(hipStreamSynchronize(s));
    return PAG_OK;
}
