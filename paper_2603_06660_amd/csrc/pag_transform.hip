// The random orthogonal transform Q of an index (Sec. 3.1; Alg. 1): classical Gram-Schmidt with one
// re-orthogonalisation pass over a Gaussian matrix, on the GPU.  Every sum runs in index order with a
// rounding after each product and each addition, as a plain loop on the host would compute it, so that a
// seed gives the same Q wherever the orthogonalisation runs.
//
// A column's projections (all earlier columns at once) and its update (all of its elements at once) are
// chains of dependent additions: what bounds them is the latency of an fp64 addition and of the loads, not
// bandwidth.  A thread therefore owns a chain and has up to 2 GS_CHUNK values on their way while it adds
// the last ones, two values to a load; the matrix is kept twice, in pairs of rows and in pairs of columns,
// so that neighbouring threads read neighbouring addresses in both.  What a chain is multiplied with is the
// same for all threads: each lane fetches one factor of a chunk, and they are broadcast from there (from LDS
// they cost a wait each: 24 against 17 us for a chain of 768).
// d = 768: 300 ms on eight host threads, 48 ms here (17 us a projection, 10 us an update, 8 us a normalisation).
#include "pag_internal.h"

namespace {

constexpr u32 GS_CHUNK = 64;

// where element k of vector i lies: pairs of k side by side, then i (`rows`); pairs of i, then k (`cols`)
__device__ __forceinline__ u64 in_rows(u32 i, u32 k, u32 ld) { return ((u64)(k / 2) * ld + i) * 2 + (k & 1); }
__device__ __forceinline__ u64 in_cols(u32 i, u32 k, u32 ld) { return ((u64)(i / 2) * ld + k) * 2 + (i & 1); }

// the factor that lane t holds, in every lane
__device__ __forceinline__ double gs_from_lane(double x, int t) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), t), __builtin_amdgcn_readlane(__double2loint(x), t));
}

// One chain: acc = step(acc, value, factor) over the pairs m[0], m[ld], ... of `count` (a multiple of GS_CHUNK) values;
// factor(k) is read once per wave
template <class Factor, class Step>
__device__ __forceinline__ double gs_chain(const double2* __restrict__ m, u32 ld, u32 count, Factor&& factor, double acc, Step&& step) {
    double2 v[2][GS_CHUNK / 2];
    double f[2];
    auto load = [&](double2 (&to)[GS_CHUNK / 2], double& fl, u32 k0) {
        fl = factor(k0 + threadIdx.x);
#pragma unroll
        for (u32 t = 0; t < GS_CHUNK / 2; ++t) to[t] = m[(u64)(k0 / 2 + t) * ld];
    };
    auto add = [&](const double2 (&of)[GS_CHUNK / 2], double fl) {
#pragma unroll
        for (u32 t = 0; t < GS_CHUNK / 2; ++t) {
            acc = step(acc, of[t].x, gs_from_lane(fl, 2 * t));
            acc = step(acc, of[t].y, gs_from_lane(fl, 2 * t + 1));
        }
    };
    load(v[0], f[0], 0);
    for (u32 k0 = 0; k0 < count; k0 += 2 * GS_CHUNK) {
        if (k0 + GS_CHUNK < count) load(v[1], f[1], k0 + GS_CHUNK);
        add(v[0], f[0]);
        if (k0 + GS_CHUNK < count) {
            if (k0 + 2 * GS_CHUNK < count) load(v[0], f[0], k0 + 2 * GS_CHUNK);
            add(v[1], f[1]);
        }
    }
    return acc;
}

// proj[i] = <column i, column j> for the finished columns i < j; `rows` holds zeros for the others
__global__ void __launch_bounds__(64) k_gs_project(const double* __restrict__ rows, const double* __restrict__ cols, u32 j, u32 ld,
                                                   double* __restrict__ proj) {
    const u32 i = blockIdx.x * 64 + threadIdx.x;
    proj[i] = gs_chain((const double2*)rows + i, ld, ld, [&](u32 k) { return cols[in_cols(j, k, ld)]; }, 0.0,
                       [](double s, double v, double a) { return s + v * a; });
}

// column j -= sum_i proj[i] * column i, i ascending; proj is zero from j on
__global__ void __launch_bounds__(64) k_gs_update(double* __restrict__ cols, u32 j, u32 ld, const double* __restrict__ proj) {
    const u32 count = (j + GS_CHUNK - 1) / GS_CHUNK * GS_CHUNK;
    const u32 k = blockIdx.x * 64 + threadIdx.x;
    const double a = gs_chain((const double2*)cols + k, ld, count, [&](u32 i) { return proj[i]; }, cols[in_cols(j, k, ld)],
                              [](double s, double v, double p) { return s - p * v; });
    cols[in_cols(j, k, ld)] = a;
}

// column j to unit length; it is finished then: into `rows`, and into row j of Q as fp32
__global__ void __launch_bounds__(1024) k_gs_normalise(double* __restrict__ cols, double* __restrict__ rows, u32 j, u32 dim, u32 ld,
                                                       float* __restrict__ rot) {
    extern __shared__ double a[];
    __shared__ double norm;
    for (u32 k = threadIdx.x; k < ld; k += 1024) a[k] = cols[in_cols(j, k, ld)];
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (u32 k0 = 0; k0 < ld; k0 += 16) {
            double v[16];
#pragma unroll
            for (u32 t = 0; t < 16; ++t) v[t] = a[k0 + t];
#pragma unroll
            for (u32 t = 0; t < 16; ++t) s = s + v[t] * v[t];
        }
        norm = sqrt(s);
    }
    __syncthreads();
    const double n = norm;
    for (u32 k = threadIdx.x; k < ld; k += 1024) {
        const double x = a[k] / n;
        cols[in_cols(j, k, ld)] = x;
        rows[in_rows(j, k, ld)] = x;
        if (k < dim) rot[(u64)j * dim + k] = (float)x;
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
    const u64 matrix = (u64)ld * ld;
    hipError_t e = hipMalloc((void**)&ws, (2 * matrix + ld) * sizeof(double));
    if (e != hipSuccess) { pag_set_error(std::string("hipMalloc (transform): ") + hipGetErrorString(e)); return PAG_ENOMEM; }
    double *cols = ws, *rows = ws + matrix, *proj = ws + 2 * matrix;
    int rc;
    if ((rc = pag_launch_zero_u32(s, (u32*)ws, (2 * matrix + ld) * 2))) return rc;
    // the matrix arrives column after column in the place of `rows`, is laid out in `cols`, and `rows` starts empty
    PAG_HIP(hipMemcpyAsync(rows, g, (size_t)dim * dim * 8, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_gs_lay_out, dim3((dim + 255) / 256, dim), dim3(256), 0, s, rows, dim, ld, cols);
    if ((rc = pag_launch_zero_u32(s, (u32*)rows, matrix * 2))) return rc;
    for (u32 j = 0; j < dim; ++j) {
        if (j > 0)
            for (int pass = 0; pass < 2; ++pass) {
                hipLaunchKernelGGL(k_gs_project, dim3((j + 63) / 64), dim3(64), 0, s, rows, cols, j, ld, proj);
                hipLaunchKernelGGL(k_gs_update, dim3(ld / 64), dim3(64), 0, s, cols, j, ld, proj);
            }
        hipLaunchKernelGGL(k_gs_normalise, dim3(1), dim3(1024), ld * sizeof(double), s, cols, rows, j, dim, ld, rot);
    }
    PAG_HIP(hipGetLastError());
    PAG_HIP(hipStreamSynchronize(s));
    return PAG_OK;
}
