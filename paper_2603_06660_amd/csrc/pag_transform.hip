// The random orthogonal transform Q of an index (Sec. 3.1; Alg. 1): classical Gram-Schmidt with one
// re-orthogonalisation pass over a Gaussian matrix, on the GPU.  Every sum runs in index order with a
// rounding after each product and each addition, as a plain loop on the host would compute it, so that a
// seed gives the same Q wherever the orthogonalisation runs.
//
// A column's projections (all earlier columns at once) and its update (all of its elements at once) are
// chains of dependent additions: what bounds them is the latency of an fp64 addition and of the loads, not
// bandwidth.  A thread therefore owns a chain and asks for GS_CHUNK values before it adds them; the matrix
// is kept twice, by columns and by rows, so that neighbouring threads read neighbouring addresses in both.
// d = 768: 300 ms on eight host threads, 33 ms here.
#include "pag_internal.h"

namespace {

constexpr u32 GS_CHUNK = 64;

// proj[i] = <column i, column j> for the finished columns i < j; `rows` holds zeros for the others
__global__ void __launch_bounds__(64) k_gs_project(const double* __restrict__ rows, const double* __restrict__ col_j, u32 ld,
                                                   double* __restrict__ proj) {
    const u32 i = blockIdx.x * 64 + threadIdx.x;
    double s = 0.0;
    for (u32 k0 = 0; k0 < ld; k0 += GS_CHUNK) {
        double v[GS_CHUNK];
#pragma unroll
        for (u32 t = 0; t < GS_CHUNK; ++t) v[t] = rows[(u64)(k0 + t) * ld + i];
#pragma unroll
        for (u32 t = 0; t < GS_CHUNK; ++t) s = s + v[t] * col_j[k0 + t];
    }
    proj[i] = s;
}

// column j -= sum_i proj[i] * column i, i ascending; proj is zero from j on
__global__ void __launch_bounds__(64) k_gs_update(double* __restrict__ cols, u32 j, u32 ld, const double* __restrict__ proj) {
    const u32 k = blockIdx.x * 64 + threadIdx.x;
    double a = cols[(u64)j * ld + k];
    for (u32 i0 = 0; i0 < j; i0 += GS_CHUNK) {
        double v[GS_CHUNK];
#pragma unroll
        for (u32 t = 0; t < GS_CHUNK; ++t) v[t] = cols[(u64)(i0 + t) * ld + k];
#pragma unroll
        for (u32 t = 0; t < GS_CHUNK; ++t) a = a - proj[i0 + t] * v[t];
    }
    cols[(u64)j * ld + k] = a;
}

// column j to unit length; it is finished then: into `rows`, and into row j of Q as fp32
__global__ void __launch_bounds__(1024) k_gs_normalise(double* __restrict__ cols, double* __restrict__ rows, u32 j, u32 dim, u32 ld,
                                                       float* __restrict__ rot) {
    extern __shared__ double a[];
    __shared__ double norm;
    for (u32 k = threadIdx.x; k < ld; k += 1024) a[k] = cols[(u64)j * ld + k];
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
        cols[(u64)j * ld + k] = x;
        rows[(u64)k * ld + j] = x;
        if (k < dim) rot[(u64)j * dim + k] = (float)x;
    }
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
    PAG_HIP(hipMemcpy2DAsync(cols, (size_t)ld * 8, g, (size_t)dim * 8, (size_t)dim * 8, dim, hipMemcpyHostToDevice, s));
    for (u32 j = 0; j < dim; ++j) {
        if (j > 0)
            for (int pass = 0; pass < 2; ++pass) {
                hipLaunchKernelGGL(k_gs_project, dim3((j + 63) / 64), dim3(64), 0, s, rows, cols + (u64)j * ld, ld, proj);
                hipLaunchKernelGGL(k_gs_update, dim3(ld / 64), dim3(64), 0, s, cols, j, ld, proj);
            }
        hipLaunchKernelGGL(k_gs_normalise, dim3(1), dim3(1024), ld * sizeof(double), s, cols, rows, j, dim, ld, rot);
    }
    PAG_HIP(hipGetLastError());
    PAG_HIP(hipStreamSynchronize(s));
    return PAG_OK;
}
