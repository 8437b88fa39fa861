// Query / data preparation kernels: normalisation (cosine), rotation by the fixed orthogonal
// transform Q (Alg. 1 and Alg. 2, rotation step) and the projection tables
// (Alg. 2, projection-table step).  All sums are fp64 sums of exact fp32 x fp32 products,
// rounded once to fp32, so that they agree with a plain fp64 evaluation to the last bit in all
// but a vanishing fraction of the outputs.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <string>

#include "pag_internal.h"

namespace {

typedef double double4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------
// Rotation: OUT[i][j] = fl32( sum_k X[i][k] * R[j][k] ),  X [rows x d], R [d x d] row-major.
// The one dense contraction of the path: fp64 MFMA (v_mfma_f64_16x16x4).  A workgroup of four waves computes
// 16 NT x 16 NT outputs; the waves share out the k range in chunks of 16 and add their partial sums through LDS at the end.
// An operand wants row (lane % 16) and k (lane / 16) from each lane; which four k's make up one MFMA does not
// matter as long as both operands agree, so a lane reads 16 consecutive bytes of its row and feeds their four elements to
// four MFMAs: operands go from memory to registers without LDS or barriers, and the next chunk's are on their way while
// one is multiplied.
// Large batches are bound by the matrix cores (0.6 of the fp64 rate of a large product), small ones by the length of the
// k loop, which the four waves cut to a quarter.
// ---------------------------------------------------------------------------------------
template <int NT>
__global__ void __launch_bounds__(256) k_rotate(const float* __restrict__ X, u64 rows, u32 d,
                                                const float* __restrict__ R, float* __restrict__ OUT) {
    __shared__ double part[2][NT * NT * 4 * 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const u64 m0 = (u64)blockIdx.y * (16 * NT);
    const u32 n0 = blockIdx.x * (16 * NT);
    const u32 k_lane = 4u * ((u32)lane >> 4);
    const float* xp[NT];
    const float* rp[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const u64 row = m0 + 16 * i + (lane & 15);
        xp[i] = X + (row < rows ? row : rows - 1) * d;      // rows and columns past the end are computed and dropped
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const u32 col = n0 + 16 * j + (lane & 15);
        rp[j] = R + (u64)(col < d ? col : d - 1) * d;
    }
    double4_t acc[NT][NT];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (double4_t){0.0, 0.0, 0.0, 0.0};
    float4 a[NT], b[NT];
    auto load = [&](u32 k0) {
        const u32 k = k0 + k_lane;                           // d is a multiple of four: 16 bytes lie inside or outside
        const bool in = k < d;
#pragma unroll
        for (int i = 0; i < NT; ++i) a[i] = in ? *(const float4*)(xp[i] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j] = in ? *(const float4*)(rp[j] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    load(16u * w);
    for (u32 k0 = 16u * w; k0 < d; k0 += 64) {
        float4 ca[NT], cb[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) ca[i] = a[i];
#pragma unroll
        for (int j = 0; j < NT; ++j) cb[j] = b[j];
        if (k0 + 64 < d) load(k0 + 64);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double av[NT], bv[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) av[i] = (double)(e == 0 ? ca[i].x : e == 1 ? ca[i].y : e == 2 ? ca[i].z : ca[i].w);
#pragma unroll
            for (int j = 0; j < NT; ++j) bv[j] = (double)(e == 0 ? cb[j].x : e == 1 ? cb[j].y : e == 2 ? cb[j].z : cb[j].w);
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
    }
    // waves 2, 3 -> 0, 1, then 1 -> 0
#pragma unroll
    for (int step = 2; step > 0; step >>= 1) {
        if (w >= step && w < 2 * step) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) part[w - step][((i * NT + j) * 4 + r) * 64 + lane] = acc[i][j][r];
        }
        __syncthreads();
        if (w < step) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] += part[w][((i * NT + j) * 4 + r) * 64 + lane];
        }
        __syncthreads();
    }
    if (w != 0) return;
    // accumulator layout of the 16x16 f64 tile: register r of lane l holds row l/16 + 4*r, column l%16
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const u64 row = m0 + i * 16 + (lane >> 4) + 4 * r;
                const u32 col = n0 + j * 16 + (lane & 15);
                if (row < rows && col < d) OUT[row * d + col] = (float)acc[i][j][r];
            }
}

// tables[row][l][j] = fl32( sum_k r_jl[k] * q_l[k] ), k ascending; rows l >= P are zero padding.
// A thread keeps one reference vector r_jl in registers and takes `per` rows with it: the codebook, whose vectors lie
// side by side in a wave, is read once per workgroup and not once per query (10,000 x 32 tables of 32-element subspaces:
// 318 us when every thread fetched its vector for one product).  DS: elements held at a time.
template <u32 DS>
__global__ void __launch_bounds__(256) k_tables(const float* __restrict__ qrot, u64 rows, u32 d, u32 P,
                                                u32 Ppad, u32 dsub, const float* __restrict__ cb, u32 per,
                                                float* __restrict__ tables) {
    const u32 lj = blockIdx.x * 256 + threadIdx.x, l = lj / PAG_NCODE;      // Ppad * 16 is a multiple of 256
    const u64 row0 = (u64)blockIdx.y * per, row1 = row0 + per < rows ? row0 + per : rows;
    const bool real = l < P;
    const float* r = cb + (u64)(real ? lj : 0u) * dsub;
    float rv[DS];
#pragma unroll
    for (u32 k = 0; k < DS; ++k) rv[k] = k < dsub ? r[k] : 0.f;
    for (u64 row = row0; row < row1; ++row) {
        const float* q = qrot + row * d + (u64)(real ? l : 0u) * dsub;
        double acc = 0.0;
        if (dsub <= DS) {
            float qv[DS];
#pragma unroll
            for (u32 k = 0; k < DS; ++k) qv[k] = k < dsub ? q[k] : 0.f;
#pragma unroll
            for (u32 k = 0; k < DS; ++k)
                if (k < dsub) acc = __builtin_fma((double)rv[k], (double)qv[k], acc);
        } else {
            for (u32 k = 0; k < dsub; ++k) acc = __builtin_fma((double)r[k], (double)q[k], acc);
        }
        tables[row * Ppad * PAG_NCODE + lj] = real ? (float)acc : 0.f;
    }
}

// The same, one product per thread and little in registers, so that up to TABLE_BLOCKS_AT_ONCE workgroups are on the chip
// together.
constexpr u64 TABLE_BLOCKS_AT_ONCE = 2048;           // eight on each of 256 CUs
__global__ void __launch_bounds__(256) k_tables_few(const float* __restrict__ qrot, u32 d, u32 P, u32 Ppad, u32 dsub,
                                                    const float* __restrict__ cb, float* __restrict__ tables) {
    const u32 gid = blockIdx.x * 256 + threadIdx.x, per_row = Ppad * PAG_NCODE;
    const u32 row = gid / per_row, lj = gid % per_row, l = lj / PAG_NCODE;
    double acc = 0.0;
    if (l < P) {
        const float* r = cb + (u64)lj * dsub;
        const float* q = qrot + (u64)row * d + (u64)l * dsub;
        for (u32 k = 0; k < dsub; ++k) acc = __builtin_fma((double)r[k], (double)q[k], acc);
    }
    tables[gid] = (float)acc;
}

// out = x / ||x||, one wave per row; norm from an fp64 sum of squares.
__global__ void __launch_bounds__(64) k_normalise(const float* __restrict__ X, u64 rows, u32 d,
                                                  float* __restrict__ out) {
    const u64 row = blockIdx.x;
    if (row >= rows) return;
    const int lane = threadIdx.x;
    const float* x = X + row * d;
    double s = 0.0;
    for (u32 k = lane; k < d; k += 64) s = __builtin_fma((double)x[k], (double)x[k], s);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    double nrm = sqrt(s);
    if (nrm == 0.0) nrm = 1.0;
    for (u32 k = lane; k < d; k += 64) out[row * d + k] = (float)((double)x[k] / nrm);
}

// float -> __half (round to nearest even) or __half -> float (exact), one element per thread
__global__ void __launch_bounds__(256) k_convert(const void* __restrict__ src, u32 src_half, void* __restrict__ dst,
                                                 u32 dst_half, u64 count) {
    const u64 i = (u64)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const float v = src_half ? __half2float(((const __half*)src)[i]) : ((const float*)src)[i];
    if (dst_half) ((__half*)dst)[i] = __float2half_rn(v);
    else ((float*)dst)[i] = v;
}

__global__ void __launch_bounds__(256) k_zero_u32(u32* p, u64 count) {
    const u64 i = (u64)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// ---------------------------------------------------------------------------------------
// Query order.  The waves take the queries of a batch a few thousand at a time; when the queries that run side by
// side search the same part of the graph, part of their rows comes from the memory-side cache instead of HBM.  The
// batch is therefore taken in the order of its projections onto its direction of largest spread, found by two steps
// of the power iteration from the best of ORDER_CAND stored vectors (the first entry nodes, i.e. random data
// points: the one along which the batch varies most).  Results do not depend on the order.
// ---------------------------------------------------------------------------------------
constexpr u32 ORDER_CAND = 16;

// dirs[k] = stored vector of entry[k] as fp32, norm2[k] = its squared length
__global__ void __launch_bounds__(64) k_order_dirs(pag_vecs vec, const u32* __restrict__ entry, float* __restrict__ dirs,
                                                   float* __restrict__ norm2) {
    const u32 k = blockIdx.x, d = vec.d;
    const u32 id = entry[k];
    float acc = 0.f;
    for (u32 c = threadIdx.x; c < d / 4; c += 64) {
        const float4 x = pag_vload4(vec, id, c);
        ((float4*)(dirs + (u64)k * d))[c] = x;
        acc += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (threadIdx.x == 0) norm2[k] = acc;
}

// proj[row][k] = <q_row, dirs[k]>, one wave per row
__global__ void __launch_bounds__(64) k_order_project(const float* __restrict__ qrot, u64 rows, u32 d, const float* __restrict__ dirs,
                                                      u32 ncand, float* __restrict__ proj) {
    const u64 row = blockIdx.x;
    if (row >= rows) return;
    const int lane = threadIdx.x;
    float acc[ORDER_CAND];
#pragma unroll
    for (u32 k = 0; k < ORDER_CAND; ++k) acc[k] = 0.f;
    for (u32 c = lane; c < d / 4; c += 64) {
        const float4 q = ((const float4*)(qrot + row * d))[c];
#pragma unroll
        for (u32 k = 0; k < ORDER_CAND; ++k)
            if (k < ncand) {
                const float4 x = ((const float4*)(dirs + (u64)k * d))[c];
                acc[k] += q.x * x.x + q.y * x.y + q.z * x.z + q.w * x.w;
            }
    }
#pragma unroll
    for (u32 k = 0; k < ORDER_CAND; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
        if ((u32)lane == k) proj[row * ORDER_CAND + k] = acc[k];
    }
}

// the candidate with the largest variance of the projections per unit length -> *best
__global__ void __launch_bounds__(1024) k_order_pick(const float* __restrict__ proj, u64 rows, u32 ncand, const float* __restrict__ norm2,
                                                     u32* __restrict__ best, float* __restrict__ pbar) {
    __shared__ double s1[1024], s2[1024];
    const u32 t = threadIdx.x, k = t % ORDER_CAND;
    double a = 0.0, b = 0.0;
    for (u64 r = t / ORDER_CAND; r < rows; r += 1024 / ORDER_CAND) {
        const double v = (double)proj[r * ORDER_CAND + k];
        a += v; b += v * v;
    }
    s1[t] = a; s2[t] = b;
    __syncthreads();
    for (u32 step = 512; step >= ORDER_CAND; step >>= 1) {       // threads t and t + step hold the same candidate
        if (t < step) { s1[t] += s1[t + step]; s2[t] += s2[t + step]; }
        __syncthreads();
    }
    if (t == 0) {
        u32 arg = 0;
        double top = -1.0;
        for (u32 c = 0; c < ncand; ++c) {
            const double n2 = (double)norm2[c];
            const double var = n2 > 0.0 ? (s2[c] - s1[c] * s1[c] / (double)rows) / n2 : 0.0;
            if (var > top) { top = var; arg = c; }
        }
        *best = arg;
        *pbar = (float)(s1[arg] / (double)rows);
    }
}

__global__ void __launch_bounds__(256) k_order_keys(const float* __restrict__ proj, u64 rows, const u32* __restrict__ best,
                                                    float* __restrict__ keys, u32* __restrict__ vals) {
    const u64 r = (u64)blockIdx.x * 256 + threadIdx.x;
    if (r >= rows) return;
    keys[r] = proj[r * ORDER_CAND + *best];
    vals[r] = (u32)r;
}

// One step of the power iteration towards the batch's direction of largest spread: v' = sum_i (p_i - pbar) q_i, the
// centred batch applied to its own projections (the sum of the weights is zero, so the mean of the batch drops out).
// k_order_back: partial sums over ORDER_CHUNKS row chunks, one column per thread, together with the column sums of
// the batch; k_order_finish: v' and the mean of the next projections, <mean row, v'>.
constexpr u32 ORDER_CHUNKS = 64;

__global__ void __launch_bounds__(256) k_order_back(const float* __restrict__ qrot, u64 rows, u32 d, const float* __restrict__ p,
                                                    const float* __restrict__ pbar, float* __restrict__ part_v,
                                                    float* __restrict__ part_m) {
    const u32 j = blockIdx.x * 256 + threadIdx.x;
    if (j >= d) return;
    const u64 per = (rows + ORDER_CHUNKS - 1) / ORDER_CHUNKS;
    const u64 r0 = (u64)blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
    const float mean = *pbar;
    float av = 0.f, am = 0.f;
    for (u64 r = r0; r < r1; ++r) {
        const float x = qrot[r * d + j];
        av += (p[r] - mean) * x;
        am += x;
    }
    part_v[(u64)blockIdx.y * d + j] = av;
    part_m[(u64)blockIdx.y * d + j] = am;
}

__global__ void __launch_bounds__(1024) k_order_finish(const float* __restrict__ part_v, const float* __restrict__ part_m, u64 rows, u32 d,
                                                       float* __restrict__ v, float* __restrict__ pbar) {
    __shared__ double red[1024];
    double dot = 0.0;
    for (u32 j = threadIdx.x; j < d; j += 1024) {
        double a = 0.0, m = 0.0;
        for (u32 c = 0; c < ORDER_CHUNKS; ++c) { a += (double)part_v[(u64)c * d + j]; m += (double)part_m[(u64)c * d + j]; }
        v[j] = (float)a;
        dot += (double)(float)a * (m / (double)rows);
    }
    red[threadIdx.x] = dot;
    __syncthreads();
    for (u32 step = 512; step > 0; step >>= 1) {
        if (threadIdx.x < step) red[threadIdx.x] += red[threadIdx.x + step];
        __syncthreads();
    }
    if (threadIdx.x == 0) *pbar = (float)red[0];
}

// p[row] = <q_row, v>, one wave per row
__global__ void __launch_bounds__(64) k_order_project1(const float* __restrict__ qrot, u64 rows, u32 d, const float* __restrict__ v,
                                                       float* __restrict__ p) {
    const u64 row = blockIdx.x;
    if (row >= rows) return;
    float acc = 0.f;
    for (u32 c = threadIdx.x; c < d / 4; c += 64) {
        const float4 q = ((const float4*)(qrot + row * d))[c];
        const float4 x = ((const float4*)v)[c];
        acc += q.x * x.x + q.y * x.y + q.z * x.z + q.w * x.w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (threadIdx.x == 0) p[row] = acc;
}

}  // namespace

int pag_order_queries(pag_index* ix, const float* qrot, u64 nq, const u32** order) {
    *order = nullptr;
    const u32 ncand = std::min<u32>(ORDER_CAND, ix->n_entry);
    if (ncand == 0 || nq < 2 || nq >= (1ull << 31)) return PAG_OK;
    hipStream_t s = ix->stream;
    const u32 d = ix->L.d;
    size_t sort_bytes = 0;
    PAG_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, sort_bytes, (const float*)nullptr, (float*)nullptr, (const u32*)nullptr,
                                               (u32*)nullptr, (int)nq, 0, 32, s));
    // words: proj [nq * 16] | keys in [nq] | keys out [nq] | numbers [nq] | order [nq] | dirs [16 * d] | norm2 [16] |
    //        best, mean [16] | v [d] | partial sums [2 * 64 * d] | sort
    const u64 o_keys = nq * ORDER_CAND, o_keys2 = o_keys + nq, o_vals = o_keys2 + nq, o_order = o_vals + nq, o_dirs = o_order + nq;
    const u64 o_norm = o_dirs + (u64)ORDER_CAND * d, o_best = o_norm + ORDER_CAND, o_v = o_best + 16, o_part = o_v + d;
    const u64 o_sort = (o_part + 2ull * ORDER_CHUNKS * d + 63) / 64 * 64;   // 256-byte aligned
    const u64 need = o_sort + (sort_bytes + 3) / 4;
    if (ix->ws_order_cap < need) {
        if (ix->ws_order) (void)hipFree(ix->ws_order);
        ix->ws_order = nullptr; ix->ws_order_cap = 0;
        hipError_t e = hipMalloc((void**)&ix->ws_order, need * 4);
        if (e != hipSuccess) { pag_set_error(std::string("hipMalloc (query order): ") + hipGetErrorString(e)); return PAG_ENOMEM; }
        ix->ws_order_cap = need;
    }
    u32* w = ix->ws_order;
    float* proj = (float*)w;
    float* dirs = (float*)(w + o_dirs);
    float* norm2 = (float*)(w + o_norm);
    hipLaunchKernelGGL(k_order_dirs, dim3(ncand), dim3(64), 0, s, pag_vecs_of(ix), ix->entry, dirs, norm2);
    hipLaunchKernelGGL(k_order_project, dim3((unsigned)nq), dim3(64), 0, s, qrot, nq, d, dirs, ncand, proj);
    float* pbar = (float*)(w + o_best + 1);
    float* keys = (float*)(w + o_keys);
    float* v = (float*)(w + o_v);
    float* part_v = (float*)(w + o_part);
    float* part_m = part_v + (u64)ORDER_CHUNKS * d;
    hipLaunchKernelGGL(k_order_pick, dim3(1), dim3(1024), 0, s, proj, nq, ncand, norm2, w + o_best, pbar);
    hipLaunchKernelGGL(k_order_keys, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s, proj, nq, w + o_best, keys, w + o_vals);
    // two steps from the best stored vector reach the direction of largest spread to within a percent of its variance
    for (int it = 0; it < 2; ++it) {
        hipLaunchKernelGGL(k_order_back, dim3((d + 255) / 256, ORDER_CHUNKS), dim3(256), 0, s, qrot, nq, d, keys, pbar, part_v, part_m);
        hipLaunchKernelGGL(k_order_finish, dim3(1), dim3(1024), 0, s, part_v, part_m, nq, d, v, pbar);
        hipLaunchKernelGGL(k_order_project1, dim3((unsigned)nq), dim3(64), 0, s, qrot, nq, d, v, keys);
    }
    PAG_HIP(hipGetLastError());
    PAG_HIP(hipcub::DeviceRadixSort::SortPairs((void*)(w + o_sort), sort_bytes, (const float*)(w + o_keys), (float*)(w + o_keys2),
                                               (const u32*)(w + o_vals), w + o_order, (int)nq, 0, 32, s));
    *order = w + o_order;
    return PAG_OK;
}

template <int NT>
static void launch_rotate(hipStream_t s, const float* X, u64 rows, u32 d, const float* rot, float* out) {
    const u64 by = (rows + 16 * NT - 1) / (16 * NT);
    // gridDim.y is limited to 65535: walk the rows in slabs
    const u64 slab = 65535ull;
    for (u64 y0 = 0; y0 < by; y0 += slab) {
        const u64 ny = by - y0 < slab ? by - y0 : slab;
        const u64 r0 = y0 * 16 * NT;
        const u64 nrows = rows - r0 < ny * 16 * NT ? rows - r0 : ny * 16 * NT;
        dim3 grid((d + 16 * NT - 1) / (16 * NT), (unsigned)ny);
        hipLaunchKernelGGL(k_rotate<NT>, grid, dim3(256), 0, s, X + r0 * d, nrows, d, rot, out + r0 * d);
    }
}

int pag_launch_rotate(hipStream_t s, const float* X, u64 rows, u32 d, const float* rot, float* out) {
    if (rows == 0) return PAG_OK;
    // 32 x 32 outputs per workgroup if that gives every CU (256) one, else 16 x 16.  Larger tiles read less from L2 but
    // leave fewer waves to cover the loads (10,000 x 1024: 64 x 64 530 us, 32 x 32 440 us; staged through LDS 490 us).
    // One row of 768 takes 6 us (45 us as a loop over LDS tiles), 250 rows of 3072 120 us (330 us).
    const u64 blocks = ((rows + 31) / 32) * ((d + 31) / 32);
    if (blocks >= 256) launch_rotate<2>(s, X, rows, d, rot, out);
    else launch_rotate<1>(s, X, rows, d, rot, out);
    PAG_HIP(hipGetLastError());
    return PAG_OK;
}

int pag_launch_tables(hipStream_t s, const float* qrot, u64 rows, const pag_layout& L, const float* cb,
                      float* tables) {
    if (rows == 0) return PAG_OK;
    const u32 bx = L.Ppad * PAG_NCODE / 256;
    if (rows * bx <= TABLE_BLOCKS_AT_ONCE) {
        // No slower here (1,024 x 1024: 89 us of preparation against 97; 2,048 x 128: 20 against 24), and the search that follows
        // is placed better: after workgroups that had to wait for registers (74 to 203 a thread below, two to six
        // workgroups on a CU) 1,024 waves land on 945 of the 1,024 SIMDs, 80 of them with two, after these on all of them
        // (1,024 queries of 50,000 x 1024, efS 512: 3.0 against 2.7 ms).
        hipLaunchKernelGGL(k_tables_few, dim3((unsigned)(rows * bx)), dim3(256), 0, s, qrot, L.d, L.P, L.Ppad, L.dsub, cb, tables);
        PAG_HIP(hipGetLastError());
        return PAG_OK;
    }
    // enough workgroups for eight on every CU before a thread takes a second row; at most 32 rows
    const u32 per = (u32)std::min<u64>(32, std::max<u64>(1, rows * bx / 2048));
    const u64 slab = 65535ull * per;                         // gridDim.y is limited to 65535
    for (u64 r0 = 0; r0 < rows; r0 += slab) {
        const u64 n = rows - r0 < slab ? rows - r0 : slab;
        const dim3 grid(bx, (unsigned)((n + per - 1) / per));
        const float* q = qrot + r0 * L.d;
        float* t = tables + r0 * L.Ppad * PAG_NCODE;
        if (L.dsub <= 16) hipLaunchKernelGGL(k_tables<16>, grid, dim3(256), 0, s, q, n, L.d, L.P, L.Ppad, L.dsub, cb, per, t);
        else if (L.dsub <= 32) hipLaunchKernelGGL(k_tables<32>, grid, dim3(256), 0, s, q, n, L.d, L.P, L.Ppad, L.dsub, cb, per, t);
        else hipLaunchKernelGGL(k_tables<48>, grid, dim3(256), 0, s, q, n, L.d, L.P, L.Ppad, L.dsub, cb, per, t);
    }
    PAG_HIP(hipGetLastError());
    return PAG_OK;
}

int pag_launch_normalise(hipStream_t s, const float* X, u64 rows, u32 d, float* out) {
    if (rows == 0) return PAG_OK;
    hipLaunchKernelGGL(k_normalise, dim3((unsigned)rows), dim3(64), 0, s, X, rows, d, out);
    PAG_HIP(hipGetLastError());
    return PAG_OK;
}

int pag_launch_convert(hipStream_t s, const void* src, u32 src_half, void* dst, u32 dst_half, u64 count) {
    const u64 step = 1ull << 30;
    for (u64 o = 0; o < count; o += step) {
        const u64 c = count - o < step ? count - o : step;
        hipLaunchKernelGGL(k_convert, dim3((unsigned)((c + 255) / 256)), dim3(256), 0, s,
                           (const void*)((const char*)src + o * (src_half ? 2 : 4)), src_half,
                           (void*)((char*)dst + o * (dst_half ? 2 : 4)), dst_half, c);
    }
    PAG_HIP(hipGetLastError());
    return PAG_OK;
}

int pag_launch_zero_u32(hipStream_t s, u32* p, u64 count) {
    if (count == 0) return PAG_OK;
    hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count);
    PAG_HIP(hipGetLastError());
    return PAG_OK;
}
