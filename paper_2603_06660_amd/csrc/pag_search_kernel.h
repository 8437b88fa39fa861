// PRT-TFB best-first search (Alg. 2, Sec. 3.3).  In k_search one wavefront owns one query from the entry nodes to the final
// top-K; in k_search_team the waves of a workgroup share a query (see run_team; pag_plan.h has the rule).  Included by the
// instantiation units pag_search_nq*_cw*.hip and pag_search_team_nq*.hip.
//
// Wave-level data placement (64 lanes; a team's wave 0 holds W, R_L and the rings, its wave 1 keeps the seen set):
//   query        registers, NQ float4 per lane (element chunk c*64+lane)
//   W            registers, NW slots per lane (b <= 64 NW).  Up to 128 nodes (NW <= 2), and up to 512 in a team: sorted ascending
//                by key, rank r in slot r/64 of lane r%64 (above 128 nodes the last slots are used).  Else: unsorted, entry i in slot i/64 of lane i%64; the node to
//                expand and the farthest member are found by wave-wide minima / maxima, the farthest one is cached
//   R_L          up to 128 nodes: registers, same placement (capacity K <= b); above: the front of a per-wave HBM buffer
//   table T      LDS, float [Ppad][16]
//   seen set     short searches: LDS open-addressing hash of node ids (exact; overflows into a
//                per-wave HBM bitmap).  Long searches: every id goes to the per-wave HBM bitmap,
//                an LDS Bloom filter says which lookups can skip it, and the LDS table is a
//                direct-mapped cache of recently admitted ids (most re-encounters are recent)
//   R_F, R_T     rings (power-of-two buffers, the last b pushes are valid): LDS, or per-wave HBM
//                buffers for working sets above 128 nodes, which are pushed to rarely and read
//                once per round
//   SA, SB       scratch for scatters and sorts: LDS for working sets of up to 128 nodes; above, two per-wave HBM buffers
//                that are touched at round ends only (SA holds R_L in front and sorts R_L + W, SB sorts the rings)
// A key packs (dist bits << 32) | (id << 1) | visited, so that unsigned comparison orders by
// (dist, id); distances are sums of squares, hence non-negative and monotone as bit patterns.
//
// One hop evaluates the projection test for all neighbours of u at once, lane s <-> neighbour
// slot s, against the threshold read when u is popped; the hop's passers enter W as if they
// were admitted one after another in ascending (dist, id) order: the b smallest of W + passers
// stay, displaced W members go to R_T (largest first), passers that do not fit go to R_F
// (smallest first).  One wave by itself merges a sorted W by ranks, a team's wave 0 inserts one
// passer after another, a step of one lane each; an unsorted W takes them one replacement at a time.
#pragma once

#include "pag_internal.h"
#include "pag_wave.h"

#include <type_traits>

namespace pagk {

__device__ __forceinline__ u32 rdlane(u32 v, int l) { return (u32)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ u64 rdlane64(u64 v, int l) {
    u32 lo = rdlane((u32)v, l), hi = rdlane((u32)(v >> 32), l);
    return ((u64)hi << 32) | lo;
}
// Orders the LDS accesses of one wavefront: its LDS operations execute in program order, so all that traffic between its lanes
// needs is that the compiler keeps the accesses in place and that the LDS queue has drained.  Unlike __syncthreads() this does
// not wait for global loads in flight (prefetched records, seen-set words), which is the point.  Between the waves of a team
// stands team_barrier.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// the value that lane l holds, in every lane
__device__ __forceinline__ double lane_value(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

__device__ __forceinline__ u32 uniform(u32 v) { return (u32)__builtin_amdgcn_readfirstlane((int)v); }

__device__ __forceinline__ u32 hash_slot(u32 id, u32 hlog) { return (id * 2654435761u) >> (32 - hlog); }

// BUCKETS (teams): the table is probed in buckets of four slots that fill from the front.  One 16-byte read tells nearly all, where the
// longest run of 32 lanes that probe slot by slot takes several reads, one after the other (37 queries of 1M x 768 1,268 -> 1,233 us,
// 512 x 768 in 16 bits 1,332 -> 1,293).  Single waves fill the GPU and wait for the LDS rather than for one read after the
// other: there a read of one slot stays the better one.
template <bool BUCKETS>
__device__ __forceinline__ bool hash_contains(const u32* H, u32 hlog, u32 id) {
    const u32 mask = (1u << hlog) - 1;
    u32 p = hash_slot(id, hlog);
    if constexpr (BUCKETS) {
        p &= ~3u;
        for (;;) {
            const uint4 v = *(const uint4*)(H + p);
            if (v.x == id || v.y == id || v.z == id || v.w == id) return true;
            if (v.w == PAG_EMPTY) return false;
            p = (p + 4) & mask;
        }
    } else {
        for (;;) {
            const u32 v = H[p];
            if (v == id) return true;
            if (v == PAG_EMPTY) return false;
            p = (p + 1) & mask;
        }
    }
}

template <bool BUCKETS>
__device__ __forceinline__ void hash_insert(u32* H, u32 hlog, u32 id) {
    const u32 mask = (1u << hlog) - 1;
    u32 p = hash_slot(id, hlog);
    if constexpr (BUCKETS) {
        p &= ~3u;
        const uint4 v = *(const uint4*)(H + p);
        p += v.x == PAG_EMPTY ? 0u : v.y == PAG_EMPTY ? 1u : v.z == PAG_EMPTY ? 2u : 3u;
    }
    for (;;) {
        const u32 old = atomicCAS(&H[p], PAG_EMPTY, id);
        if (old == PAG_EMPTY || old == id) return;
        p = (p + 1) & mask;
    }
}

// Bloom filter over the ids that live in the HBM bitmap (two hash functions, LDS bit array):
// "no" is definite, so most lookups of unseen nodes never touch HBM.
__device__ __forceinline__ bool bloom_maybe(const u32* B, u32 blog, u32 id) {
    const u32 h1 = (id * 0x9E3779B1u) >> (32 - blog), h2 = (id * 0x85EBCA77u) >> (32 - blog);
    return ((B[h1 >> 5] >> (h1 & 31)) & (B[h2 >> 5] >> (h2 & 31)) & 1u) != 0;
}
__device__ __forceinline__ void bloom_set(u32* B, u32 blog, u32 id) {
    const u32 h1 = (id * 0x9E3779B1u) >> (32 - blog), h2 = (id * 0x85EBCA77u) >> (32 - blog);
    atomicOr(&B[h1 >> 5], 1u << (h1 & 31));
    atomicOr(&B[h2 >> 5], 1u << (h2 & 31));
}

// The rank of this lane's key among the n <= 64 of lanes 0 .. n - 1 (the other lanes: the largest key): broadcast four at a
// time, their comparisons do not wait for each other, nor for LDS.
__device__ __forceinline__ u32 rank_among(u64 k, u32 n) {
    u32 r = 0;
    for (u32 j = 0; j < n; j += 4) {
        u64 o[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) o[g] = rdlane64(k, (int)j + g);     // beyond n: the largest key, smaller than none
#pragma unroll
        for (int g = 0; g < 4; ++g) r += (o[g] < k) ? 1u : 0u;
    }
    return r;
}

// dst[rank] = src[i], rank = number of smaller keys; keys are distinct.  Quadratic: for short lists.
__device__ __forceinline__ void rank_sort(const u64* src, u64* dst, u32 n, int lane) {
    if (n <= 64) {
        const u64 k = (u32)lane < n ? src[lane] : PAG_KEY_INVALID;
        const u32 r = rank_among(k, n);
        if ((u32)lane < n) dst[r] = k;
        return;
    }
    for (u32 i = lane; i < n; i += 64) {
        const u64 k = src[i];
        u32 r = 0;
        for (u32 j = 0; j < n; ++j) r += (src[j] < k) ? 1u : 0u;
        dst[r] = k;
    }
}

// In-place ascending bitonic sort of S[0, n) in LDS by one wave; S has room for n rounded up to a power
// of two (the tail is padded with the largest key).
__device__ __forceinline__ void bitonic_sort(u64* S, u32 n, int lane) {
    u32 N = 64;
    while (N < n) N <<= 1;
    for (u32 i = n + lane; i < N; i += 64) S[i] = PAG_KEY_INVALID;
    lds_sync();
    for (u32 k = 2; k <= N; k <<= 1)
        for (u32 j = k >> 1; j > 0; j >>= 1) {
            for (u32 t = lane; t < N / 2; t += 64) {
                const u32 i = ((t & ~(j - 1)) << 1) | (t & (j - 1));   // bit j clear
                const u32 l = i | j;
                const u64 x = S[i], y = S[l];
                if ((x > y) == ((i & k) == 0)) { S[i] = y; S[l] = x; }
            }
            lds_sync();
        }
}

// Ascending bitonic sort of 64 * NS keys held in registers, key e in slot e / 64 of lane e % 64 (pad with the
// largest key).  Compare-exchange steps at distances below 64 go across lanes (one exchange per slot), those at
// distances of 64 and more pair up slots of the same lane.  No memory is touched.
template <int NS, int D>
__device__ __forceinline__ void bitonic_slot_step(u64 (&x)[NS], u32 k) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if ((s & D) == 0) {
            const bool asc = ((64u * (u32)s) & k) == 0;
            const u64 a = x[s], b = x[s | D];
            const u64 lo = a < b ? a : b, hi = a < b ? b : a;
            x[s] = asc ? lo : hi;
            x[s | D] = asc ? hi : lo;
        }
}

template <int NS>
__device__ __forceinline__ void bitonic_registers(u64 (&x)[NS], int lane) {
    for (u32 k = 2; k <= 64u * NS; k <<= 1) {
        // slot distance D pairs keys 64 D apart: part of the stages k >= 128 D
        if constexpr (NS >= 32) { if (k >= 16u * 128u) bitonic_slot_step<NS, 16>(x, k); }
        if constexpr (NS >= 16) { if (k >= 8u * 128u) bitonic_slot_step<NS, 8>(x, k); }
        if constexpr (NS >= 8) { if (k >= 4u * 128u) bitonic_slot_step<NS, 4>(x, k); }
        if constexpr (NS >= 4) { if (k >= 2u * 128u) bitonic_slot_step<NS, 2>(x, k); }
        if constexpr (NS >= 2) { if (k >= 128u) bitonic_slot_step<NS, 1>(x, k); }
        for (u32 j = (k >> 1) < 32u ? (k >> 1) : 32u; j > 0; j >>= 1) {
            const bool lower = ((u32)lane & j) == 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const u64 other = (u64)__shfl_xor((unsigned long long)x[s], (int)j, 64);
                const bool asc = ((64u * (u32)s + (u32)lane) & k) == 0;
                const u64 lo = x[s] < other ? x[s] : other, hi = x[s] < other ? other : x[s];
                x[s] = (lower == asc) ? lo : hi;
            }
        }
    }
}

// Sorts the n keys in `a` ascending and returns where the result lives.  Working sets whose lists
// are always short (by_ranks) go through the rank sort into `b`; the others sort in place, and
// their `b` does not exist.
__device__ __forceinline__ const u64* sort_keys(u64* a, u64* b, u32 n, bool by_ranks, int lane) {
    if (by_ranks) {
        rank_sort(a, b, n, lane);
        lds_sync();
        return b;
    }
    bitonic_sort(a, n, lane);
    return a;
}

// Optional per-phase timers (diagnostic builds only): every mark first drains all outstanding
// memory operations, so the phases are timed as if they did not overlap.
#ifdef PAG_PHASE_TIMERS
#define PAG_MARK(i)                                                  \
    do {                                                             \
        __builtin_amdgcn_s_waitcnt(0);                               \
        const u64 t__ = wall_clock64();                              \
        s_phase[i] += t__ - t_last;                                  \
        t_last = t__;                                                \
    } while (0)
#else
#define PAG_MARK(i) do {} while (0)
#endif

// S = sum_l T[l][code_l] over the CW * 8 subspaces of one neighbour, added in increasing l.
// The LDS gathers of G subspaces are issued together, then consumed in order.  `t_base` is the
// LDS byte address of T, a multiple of 64, so that "4 * code" can be OR-ed into it and the row
// offset 64 * l rides in the instruction.
typedef __attribute__((address_space(3))) const float* lds_cfloat_ptr;
template <int CW, int N, int G = 16>
__device__ __forceinline__ float table_sum(u32 t_base, const u32 (&cwv)[N]) {
    float S = 0.f;
#pragma unroll
    for (int k = 0; k < CW; k += G / 8) {
        float t[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const u32 wd = cwv[k + j / 8];
            const int sh = 4 * (j % 8) - 2;
            const u32 x = sh < 0 ? wd << 2 : wd >> sh;
            t[j] = ((lds_cfloat_ptr)(uintptr_t)((x & 60u) | t_base))[(k * 8 + j) * PAG_NCODE];
        }
#pragma unroll
        for (int j = 0; j < G; ++j) S = S + t[j];
    }
    return S;
}

// NQ: chunks of a stored vector per lane (a chunk is what one lane loads at once); NW: entries of
// W / R_L per lane; VM: how the store is read -- 0: fp32, 16-byte chunks of 4 elements; 1: 16-bit
// floats, 16-byte chunks of 8 elements; 2: 16-bit floats, 8-byte chunks of 4 elements (for row
// lengths that would leave half of the lanes idle in the last 16-byte chunk); 16-bit values are
// widened to fp32 on use; CW: dwords of 4-bit codes per neighbour (2, 4 or 8 for up to 16, 32 or
// 64 subspaces).
// TEAM: the workgroup has several waves that work on one query (see run_team()).  CW is then the most that is supported,
// the index's own count is read at run time.
template <int NQ, int NW, int VM, int CW, bool TEAM = false>
struct Wave {
    static constexpr bool HALF = VM != 0;
    static constexpr int EPC = VM == 1 ? 8 : 4;     // elements per chunk
    using Chunk = std::conditional_t<VM == 2, uint2, uint4>;
    // constant for the kernel
    const SearchArgs A;
    int lane;
    const int wave, nwaves;         // TEAM: this wave's number in its workgroup, and how many there are
    float* T;
    u32 t_base;                     // LDS byte address of T
    u32* H;
    u32* BL;
    u64 *SA, *SB, *RF, *RT;
    u32* bitmap;
    // per query
    static constexpr int QV = NQ * EPC / 4;         // float4 registers holding the query
    static constexpr bool RINGS_IN_HBM = NW > 2;    // matches the host's LDS carve-up
    static constexpr bool BIG = NW > 2;             // large working sets
    // W is kept sorted: up to 128 nodes, by a team up to 512; else see merge_unsorted
    static constexpr bool SORTED = NW <= 2 || (TEAM && NW <= 8);
    u64 wmax;                       // W not sorted: key of its farthest member, valid while nW == b
    u64 nx_key;                     // W not sorted: key of the node to expand next (PAG_KEY_INVALID: W has no unvisited node)
    bool nx_known;                  // W not sorted: nx_key is up to date
    u32 open_slot;                  // W sorted, above 128 nodes: the slots before this one hold no unvisited member
    u64 GM, GU;                     // W not sorted: lane s < NW holds slot s's farthest member (0: slot empty) and its closest
                                    // unvisited member (PAG_KEY_INVALID: none); the other lanes hold 0 / PAG_KEY_INVALID
    float4 q[QV];
    u64 W[NW];
    u64 RL[NW > 2 ? 1 : NW];        // unused for large working sets: their R_L is SA[0, nRL)
    u32 nW, nRL;
    u64 done[NW > 2 ? 1 : NW];      // TEAM, wave 0: W of the last round, if it has yet to enter R_L, ...
    u32 n_done;                     // ... how many keys that are
    u32 cntF, hdF, cntT, hdT;       // rings: valid entries (<= b) and total pushes; slot = push number & ring mask
    u32 n_hash, n_spill;
    u32 n_cand;                     // indexing mode: entries of R_L written so far
    u32 round;                      // TEAM, wave 0: rounds finished
    u32 posted_node;                // TEAM, wave 0: the node to expand next
    u32 scr_id;                     // TEAM, wave 1: the neighbours last screened
    float pf_sum; bool pf_summed;   // TEAM: the code sums of the record in pf_*, once they are computed
    // The last TAILS chunk rows of the NQ may lie partly or wholly beyond the end of a row (the host
    // picks NQ = the rows needed, or one more where that count is not instantiated): per such chunk the
    // index this lane reads (0 if past the end) and a mask (all ones if inside the row, else zero)
    static constexpr int TAILS = NQ >= 5 ? 2 : 1;
    u32 tail_idx[TAILS];
    u32 tail_mask[TAILS];
    // Where the third wave on a SIMD leaves no register for a row waiting unmasked (see pag_search_occupancy) the values
    // past the end are replaced right after the request: 16-bit rows of 2304 at 8,000 queries 0.95 of that with 40 dwords
    // spilled, of 2816 0.7 with 85
    static constexpr bool MASK_EARLY = !TEAM && (VM == 2 ? NQ == 10 || (NQ == 12 && CW < 8) : VM == 0 && NQ == 8 && NW == 2);
    // adjacency record requested ahead of time for the node that will be expanded next
    u32 nx_id;                      // whose record pf_* holds (PAG_EMPTY: none)
    u32 pf_id, pf_cw[CW];
    float pf_a, pf_c;
    // TEAM: what the waves of a workgroup share (LDS), see run_team()
    u32* team;                      // words TM_* below
    u64 Hk;                         // indexing: PES buffer H(v), lane i = i-th closest surviving node (Alg. 1)
    // statistics (wave-uniform)
    u32 s_hops, s_tests, s_passes, s_exact, s_rounds, s_rf, s_rt, s_spill, s_queries;
#ifdef PAG_PHASE_TIMERS
    u64 s_phase[6];
    u64 t_last;
#endif

    __device__ Wave(const SearchArgs& a, unsigned char* smem, int ln, int wv = 0, int nw = 1)
        : A(a), lane(ln), wave(wv), nwaves(nw) {
        T = (float*)smem;
        t_base = (u32)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
        H = (u32*)(smem + a.off_hash);
        BL = (u32*)(smem + a.off_bloom);
        SA = (u64*)(smem + a.off_sa);
        SB = (u64*)(smem + a.off_sb);
        if constexpr (RINGS_IN_HBM) {
            RF = a.rings + (u64)blockIdx.x * 3 * (u64)(a.ring_mask + 1);
            RT = RF + (a.ring_mask + 1);
            SA = RT + (a.ring_mask + 1);      // R_L of large working sets: b <= ring_mask + 1 keys
            SB = nullptr;
        } else {
            RF = (u64*)(smem + a.off_rf);
            RT = (u64*)(smem + a.off_rt);
        }
        team = (u32*)(smem + a.off_team);
        bitmap = a.bitmap + (u64)blockIdx.x * a.bitmap_words;
#pragma unroll
        for (int t = 0; t < TAILS; ++t) {
            const u32 idx = (u32)(NQ - TAILS + t) * 64 + (u32)ln;
            const bool tail_ok = idx * (u32)EPC < a.d;
            tail_idx[t] = tail_ok ? idx : 0u;
            tail_mask[t] = tail_ok ? 0xFFFFFFFFu : 0u;
        }
        s_hops = s_tests = s_passes = s_exact = s_rounds = s_rf = s_rt = s_spill = s_queries = 0;
#ifdef PAG_PHASE_TIMERS
        for (int i = 0; i < 6; ++i) s_phase[i] = 0;
        t_last = wall_clock64();
#endif
    }

    // Wave priorities within the SIMD, used with the 16-bit store only: requesting rows comes first (3),
    // then the screening that leads to the requests (2), then the distance arithmetic (1), and the
    // bookkeeping of the merge last (0).  With short rows this is worth 9 %; with fp32 rows, where
    // memory throughput binds, it is not (and costs 1 % on long rows), so there it is left out.
    __device__ __forceinline__ void set_priority(int p) const {
        if constexpr (HALF) {
            if (p == 3) __builtin_amdgcn_s_setprio(3);
            else if (p == 2) __builtin_amdgcn_s_setprio(2);
            else if (p == 1) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
    }

    // lane s < deg reads neighbour slot s of node u: id, a, c and its chunk of 4-bit codes.  The
    // other lanes read slot 0 and get an empty id (their a, c and codes are never used), so the
    // loads sit in straight-line code and can stay in flight across whatever follows.
    __device__ __forceinline__ u32 load_id(u32 u) const {
        const bool in = (u32)lane < A.deg;
        const u32 raw = ((const u32*)(A.rec + (u64)u * A.rec_bytes))[in ? (u32)lane : 0u];
        return in ? raw : PAG_EMPTY;
    }
    __device__ __forceinline__ void load_edges(u32 u, float& ea, float& ec, u32 (&cwv)[CW]) const {
        const uint8_t* rec = A.rec + (u64)u * A.rec_bytes;
        const u32 sl = (u32)lane < A.deg ? (u32)lane : 0u;
        ea = ((const float*)(rec + A.off_a))[sl];
        ec = ((const float*)(rec + A.off_c))[sl];
        const u32* cp = (const u32*)(rec + A.off_codes) + sl * (u32)CW;    // 16-byte aligned section
        if constexpr (TEAM && NQ == 1 && NW <= 2) {
            // Short rows come from the caches, a hop waits for its estimates, and a read that the codes do not need delays them: each length has its own
            // (50k rows of 32 to 256 values, 8- and 16-byte codes, 1 to 1,000 queries, K 10 and 100: 0.97 to 1.01 of the time with the two reads
            // below, 0.99 on average; one query of 128-d, K 10, efS 512 813 -> 795 us, 1,000 queries with K 100 861 -> 851.  32-byte codes, 256-d: 0.97 to
            // 1.02).  Above 128 nodes the two reads are as good or better here too (0.97 to 1.02, 1.00 on average).
            // Every word is written on every path, else the arrays would not stay in registers.
            const u32* tp = (const u32*)(rec + A.off_codes) + sl * A.cw;
            uint4 t = make_uint4(0, 0, 0, 0), v = t;
            if (A.cw == 2) {
                const uint2 w = *(const uint2*)tp;
                t.x = w.x; t.y = w.y;
            } else {
                t = *(const uint4*)tp;
                if (A.cw == 8) v = *(const uint4*)(tp + 4);
            }
            cwv[0] = t.x; cwv[1] = t.y; cwv[2] = t.z; cwv[3] = t.w;
            cwv[4] = v.x; cwv[5] = v.y; cwv[6] = v.z; cwv[7] = v.w;
        } else if constexpr (TEAM) {
            // Two 16-byte reads whatever the length of the codes, in straight-line code (8 bytes: of a pair of neighbours; the section is
            // 16-byte aligned and the record has room behind an odd last one).  A read by length took 0.98 to 1.03 times
            // the time with 32-byte codes and longer rows, one query of 1536-d, 2304-d and 3072-d 1.02 to 1.03; 0.98 to 1.01 with shorter codes.
            const bool pairs = A.cw == 2;
            const uint8_t* tp = rec + A.off_codes + (pairs ? (sl >> 1) * 16u : sl * A.cw * 4u);
            const uint4 t = *(const uint4*)tp, v = *(const uint4*)(tp + (A.cw == 8 ? 16u : 0u));
            const bool upper = pairs && (sl & 1u);
            cwv[0] = upper ? t.z : t.x; cwv[1] = upper ? t.w : t.y; cwv[2] = t.z; cwv[3] = t.w;
            cwv[4] = v.x; cwv[5] = v.y; cwv[6] = v.z; cwv[7] = v.w;
        } else if constexpr (CW == 2) {
            const uint2 t = *(const uint2*)cp;
            cwv[0] = t.x; cwv[1] = t.y;
        } else {
#pragma unroll
            for (int k = 0; k < CW; k += 4) {
                const uint4 t = *(const uint4*)(cp + k);
                cwv[k] = t.x; cwv[k + 1] = t.y; cwv[k + 2] = t.z; cwv[k + 3] = t.w;
            }
        }
    }
    __device__ __forceinline__ void load_record(u32 u, u32& id, float& ea, float& ec, u32 (&cwv)[CW]) const {
        id = load_id(u);
        load_edges(u, ea, ec, cwv);
    }

    // The node expanded next is the unvisited entry with the smallest rank after the merge: either the
    // first unvisited member of W or the smallest passer.  Both are known before W is physically
    // rebuilt, so its adjacency record is requested here and arrives while the merge completes.
    __device__ __forceinline__ void request_next(const u32 (&cntW)[NW], bool pass, u32 cP, u32 rP, u32 id_lane) {
        const u32 b = A.b;
        u32 best_r = 0xFFFFFFFFu, best_id = PAG_EMPTY;
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            const u32 idx = s * 64 + lane;
            const u32 r = idx + cntW[s];
            const u64 m = __ballot(idx < nW && !(W[s] & 1ull) && r < b);
            if (m && best_r == 0xFFFFFFFFu) {
                const int l = __ffsll((long long)m) - 1;
                best_r = rdlane(r, l);
                best_id = rdlane((u32)(W[s] & 0xFFFFFFFFull), l) >> 1;
            }
        }
        const u64 m2 = __ballot(pass && cP == 0 && rP < b);
        if (m2) {
            const int l = __ffsll((long long)m2) - 1;
            const u32 r2 = rdlane(rP, l);
            if (r2 < best_r) { best_r = r2; best_id = rdlane(id_lane, l); }
        }
        nx_id = best_id;
        if (best_id != PAG_EMPTY) load_record(best_id, pf_id, pf_a, pf_c, pf_cw);
    }

    // exact keys ||q - x_id||^2 (Alg. 2, exact-distance step) for the lanes in `mask`;
    // lane p receives the key of its own id.  Differences in fp32, squares summed in fp64,
    // one rounding to fp32 at the end.  Two buffers of GB vectors each alternate: while one is
    // reduced the other one's loads are in flight.  No load sits inside a branch (a buffer without
    // a passer left simply re-reads the last row), which keeps the wait counts exact.
    static constexpr int GB = NQ * (int)sizeof(Chunk) <= 64 ? 2 : 1;

    // Branch-free row load: only the last TAILS chunks can run past the row; there the lane re-reads
    // chunk 0 (in bounds), so no load ever sits inside a branch and the loads of several rows stay in
    // flight together.  The values read past the end are replaced by zeros where they are used
    // (lane_partial): doing it here waits for the row right after asking for it.
    __device__ __forceinline__ void load_vec(Chunk (&v)[NQ], u32 id) const {
        const Chunk* p = (const Chunk*)((const char*)A.vec + (u64)id * A.d * (HALF ? 2 : 4));
#pragma unroll
        for (int c = 0; c < NQ - TAILS; ++c) v[c] = p[c * 64 + lane];
#pragma unroll
        for (int t = 0; t < TAILS; ++t) {
            v[NQ - TAILS + t] = p[tail_idx[t]];
            if constexpr (MASK_EARLY) v[NQ - TAILS + t] = masked(v[NQ - TAILS + t], tail_mask[t]);
        }
    }

    __device__ __forceinline__ static Chunk masked(Chunk x, u32 m) {
        x.x &= m; x.y &= m;
        if constexpr (VM != 2) { x.z &= m; x.w &= m; }
        return x;
    }
    __device__ __forceinline__ Chunk inside_row(Chunk x, int c) const {
        return !MASK_EARLY && c >= NQ - TAILS ? masked(x, tail_mask[c - (NQ - TAILS)]) : x;
    }

    // sum over this lane's elements of fl32(q - x)^2, accumulated in fp64
    __device__ __forceinline__ double lane_partial(const Chunk (&v)[NQ]) const {
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            const Chunk x = inside_row(v[c], c);
            if constexpr (VM == 1) {
                const float2 x0 = __half22float2(*(const __half2*)&x.x), x1 = __half22float2(*(const __half2*)&x.y);
                const float2 x2 = __half22float2(*(const __half2*)&x.z), x3 = __half22float2(*(const __half2*)&x.w);
                const float d0 = q[2 * c].x - x0.x, d1 = q[2 * c].y - x0.y, d2 = q[2 * c].z - x1.x, d3 = q[2 * c].w - x1.y;
                const float d4 = q[2 * c + 1].x - x2.x, d5 = q[2 * c + 1].y - x2.y;
                const float d6 = q[2 * c + 1].z - x3.x, d7 = q[2 * c + 1].w - x3.y;
                a = __builtin_fma((double)d0, (double)d0, a); a = __builtin_fma((double)d1, (double)d1, a);
                a = __builtin_fma((double)d2, (double)d2, a); a = __builtin_fma((double)d3, (double)d3, a);
                a = __builtin_fma((double)d4, (double)d4, a); a = __builtin_fma((double)d5, (double)d5, a);
                a = __builtin_fma((double)d6, (double)d6, a); a = __builtin_fma((double)d7, (double)d7, a);
            } else if constexpr (VM == 2) {
                const float2 x0 = __half22float2(*(const __half2*)&x.x), x1 = __half22float2(*(const __half2*)&x.y);
                const float d0 = q[c].x - x0.x, d1 = q[c].y - x0.y, d2 = q[c].z - x1.x, d3 = q[c].w - x1.y;
                a = __builtin_fma((double)d0, (double)d0, a); a = __builtin_fma((double)d1, (double)d1, a);
                a = __builtin_fma((double)d2, (double)d2, a); a = __builtin_fma((double)d3, (double)d3, a);
            } else {
                const float dx = q[c].x - __uint_as_float(x.x), dy = q[c].y - __uint_as_float(x.y);
                const float dz = q[c].z - __uint_as_float(x.z), dw = q[c].w - __uint_as_float(x.w);
                a = __builtin_fma((double)dx, (double)dx, a);
                a = __builtin_fma((double)dy, (double)dy, a);
                a = __builtin_fma((double)dz, (double)dz, a);
                a = __builtin_fma((double)dw, (double)dw, a);
            }
        }
        return a;
    }

    // request the rows of the next GB passers (or, when none is left, the last row again)
    __device__ __forceinline__ void issue(Chunk (&buf)[GB][NQ], int (&pl)[GB], u64& m, int& last, u32 id_lane) const {
        set_priority(3);
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            pl[g] = -1;
            if (m) { last = __ffsll((long long)m) - 1; m &= m - 1; pl[g] = last; }
            load_vec(buf[g], rdlane(id_lane, last));
        }
        set_priority(1);
    }

    __device__ __forceinline__ void reduce(const Chunk (&buf)[GB][NQ], const int (&pl)[GB], float& mine) const {
        double acc[GB];
#pragma unroll
        for (int g = 0; g < GB; ++g) acc[g] = lane_partial(buf[g]);
        const double tot = fold_sum<GB>(acc);
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            const double t = __hiloint2double((int)rdlane((u32)__double2hiint(tot), g * (64 / GB)),
                                              (int)rdlane((u32)__double2loint(tot), g * (64 / GB)));
            if (lane == pl[g]) mine = (float)t;
        }
    }

    __device__ __forceinline__ float exact_keys(u32 id_lane, u64 mask) {
        float mine = 0.f;
        Chunk va[GB][NQ], vb[GB][NQ];
        int pa[GB], pb[GB];
        u64 m = mask;
        int last = __ffsll((long long)mask) - 1;
        int left = __popcll(mask);
        const bool paced = (A.flags & PAG_SEARCH_PACED) != 0;
        issue(va, pa, m, last, id_lane);
        for (;;) {
            // the scheduling barriers keep the requests for one buffer ahead of the arithmetic on the other
            if (paced) __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
            issue(vb, pb, m, last, id_lane);
            __builtin_amdgcn_sched_barrier(0);
            reduce(va, pa, mine);
            left -= GB;
            if (left <= 0) break;
            if (paced) __builtin_amdgcn_s_waitcnt(0x0F70);
            issue(va, pa, m, last, id_lane);
            __builtin_amdgcn_sched_barrier(0);
            reduce(vb, pb, mine);
            left -= GB;
            if (left <= 0) break;
        }
        return mine;
    }

    // the hop's passers enter the seen set
    __device__ __forceinline__ void mark_seen(u32 id_lane, u32 np, bool pass) {
        if (A.blog != 0) {
            // long searches: every node goes to the bitmap and the Bloom filter; the LDS table keeps the
            // most recently admitted id per slot (a hit there is definite)
            if (pass) {
                H[hash_slot(id_lane, A.hlog)] = id_lane;
                atomicOr(&bitmap[id_lane >> 5], 1u << (id_lane & 31));
                bloom_set(BL, A.blog, id_lane);
            }
            n_spill += np; s_spill += np;
        } else {
            // short searches: exact open-addressing hash, kept at most half full; beyond that the bitmap
            const bool spill = (n_hash + np) > (1u << (A.hlog - 1));
            if (pass) {
                if (!spill) hash_insert<TEAM>(H, A.hlog, id_lane);
                else atomicOr(&bitmap[id_lane >> 5], 1u << (id_lane & 31));
            }
            if (spill) { n_spill += np; s_spill += np; } else n_hash += np;
        }
    }

    // Admission of the lanes in `mask` (ids in id_lane): exact keys, seen-set insertion, merge into W.
    __device__ __forceinline__ void admit(u32 id_lane, u64 mask) {
        const u32 np = (u32)__popcll(mask);
        if (np == 0) {
            set_priority(0);
            if constexpr (BIG) {
                look_ahead();
            } else {
                u32 zero[NW];
#pragma unroll
                for (int s = 0; s < NW; ++s) zero[s] = 0;
                request_next(zero, false, 0, 0, id_lane);
            }
            return;
        }
        const bool pass = (mask >> lane) & 1ull;
        PAG_MARK(2);
        const float dist = exact_keys(id_lane, mask);
        set_priority(0);
        PAG_MARK(3);
        mark_seen(id_lane, np, pass);
        merge(id_lane, mask, np, pass, dist);
        PAG_MARK(4);
    }

    // What a merge of the hop's passers into a sorted W comes to, before anything is moved.
    struct Ranks {
        u64 pk;                         // my passer's key
        u32 cntW[NW];                   // passers closer than my members of W
        u32 cP, rP;                     // my passer's rank among the passers and in the merged list
    };
    __device__ __forceinline__ void rank(Ranks& R, u32 id_lane, u64 mask, bool pass, float dist) const {
        R.pk = pass ? (((u64)__float_as_uint(dist) << 32) | ((u64)id_lane << 1)) : PAG_KEY_INVALID;
#pragma unroll
        for (int s = 0; s < NW; ++s) R.cntW[s] = 0;
        u32 cP = 0, cPW = 0;
        for (u64 m = mask; m;) {
            const int p = __ffsll((long long)m) - 1;
            m &= m - 1;
            const u64 k = rdlane64(R.pk, p);
            u32 c = 0;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                // keys are distinct, so one comparison tells both sides (an empty slot counts as larger)
                const bool lt = W[s] < k;
                c += (u32)__popcll(__ballot(lt));
                R.cntW[s] += lt ? 0u : 1u;
            }
            cP += (k < R.pk) ? 1u : 0u;
            if (lane == p) cPW = c;
        }
        R.cP = cP;
        R.rP = cP + cPW;
    }

    // the passers into a sorted W, as ranked
    __device__ __forceinline__ void settle(const Ranks& R, u32 np, bool pass) {
        const u32 b = A.b;
        const u32 total = nW + np;
        const u32 nW2 = total < b ? total : b;
        const u32 n_ins = (u32)__popcll(__ballot(pass && R.rP < b)); // passers that enter W
        const u32 n_f = np - n_ins;                                // false positives -> R_F
        const u32 n_ej = nW + n_ins - nW2;                         // displaced members -> R_T
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            const u32 idx = s * 64 + lane;
            if (idx < nW) {
                const u32 r = idx + R.cntW[s];
                if (r < b) SA[r] = W[s];
                else RT[(hdT + (nW - 1 - idx)) & A.ring_mask] = W[s];   // largest first
            }
        }
        if (pass) {
            if (R.rP < b) SA[R.rP] = R.pk;
            else {
                const u32 oi = R.cP - n_ins;                        // smallest first
                if (oi + b >= n_f) RF[(hdF + oi) & A.ring_mask] = R.pk;  // older ones would be overwritten anyway
            }
        }
        if (n_ej) {
            if (cntT + n_ej > b) s_rt += cntT + n_ej - b;
            cntT = cntT + n_ej < b ? cntT + n_ej : b;
            hdT += n_ej;
        }
        if (n_f) {
            if (cntF + n_f > b) s_rf += cntF + n_f - b;
            cntF = cntF + n_f < b ? cntF + n_f : b;
            hdF += n_f;
        }
        lds_sync();
#pragma unroll
        for (int s = 0; s < NW; ++s) {
            const u32 idx = s * 64 + lane;
            W[s] = idx < nW2 ? SA[idx] : PAG_KEY_INVALID;
        }
        nW = nW2;
        lds_sync();
    }

    // the hop's passers, with their exact distances, into W (see the head of this file)
    __device__ __forceinline__ void merge(u32 id_lane, u64 mask, u32 np, bool pass, float dist) {
        s_exact += np;
        if constexpr (BIG) {
            merge_unsorted(id_lane, mask, np, pass, dist);
        } else {
            Ranks R;
            rank(R, id_lane, mask, pass, dist);
            request_next(R.cntW, pass, R.cP, R.rP, id_lane);
            settle(R, np, pass);
        }
    }

    // ---- working sets above 128 nodes (NW >= 4): W is kept unsorted, in teams above 512 ----
    // Keeping up to 1024 keys sorted by rank costs a pass over all NW slots per passer and a round trip of the
    // whole set through LDS per hop.  What a hop needs of W is only its closest unvisited member, its farthest
    // member and the replacement of that one; the order of the rest matters at the round's end alone, where
    // everything is sorted anyway.

    // Keys are distance bits over (id << 1 | visited): an extreme key is found in two 32-bit steps -- the extreme
    // distance, then the extreme low word among the members at that distance -- each a handful of DPP
    // instructions, where a 64-bit reduction moves and compares register pairs.
    // W's slots (one register per lane each) keep their extremes in GM / GU, so that finding W's farthest member or
    // its closest unvisited one is a reduction over NW <= 16 lanes, and a change of one member costs a reduction over
    // that member's slot alone, reached through a uniform branch.

    // farthest member of slot S (0 if the slot is empty)
    template <int S>
    __device__ __forceinline__ u64 slot_max() const {
        const bool valid = (u32)(S * 64 + lane) < nW;
        const u32 hi = valid ? (u32)(W[S] >> 32) : 0u;
        const u32 mh = wave_extreme_u32<true>(hi);
        const u32 lo = (valid && hi == mh) ? (u32)W[S] : 0u;
        return ((u64)mh << 32) | wave_extreme_u32<true>(lo);
    }

    // closest unvisited member of slot S (PAG_KEY_INVALID if there is none)
    template <int S>
    __device__ __forceinline__ u64 slot_min_unvisited() const {
        const bool ok = (u32)(S * 64 + lane) < nW && !(W[S] & 1ull);
        const u32 hi = ok ? (u32)(W[S] >> 32) : 0xFFFFFFFFu;
        const u32 mh = wave_extreme_u32<false>(hi);
        const u32 lo = (ok && hi == mh) ? (u32)W[S] : 0xFFFFFFFFu;      // distances are finite: no member carries mh = ~0
        return ((u64)mh << 32) | wave_extreme_u32<false>(lo);
    }

    // extreme over the slots: lanes 0 .. NW - 1 of GM (MAX) or GU
    template <bool MAX>
    __device__ __forceinline__ u64 over_slots(u64 v) const {
        const u32 neutral = MAX ? 0u : 0xFFFFFFFFu;
        const u32 mh = row0_extreme_u32<MAX>((u32)(v >> 32));
        const u32 lo = (u32)(v >> 32) == mh ? (u32)v : neutral;
        return ((u64)mh << 32) | row0_extreme_u32<MAX>(lo);
    }

    // runs f(slot) for the one slot g (uniform), with the slot number as a compile-time constant; found by halving
    template <int LO = 0, int HI = NW, class F>
    __device__ __forceinline__ void at_slot(int g, F&& f) {
        if constexpr (HI - LO == 1) {
            f(std::integral_constant<int, LO>{});
        } else {
            constexpr int MID = (LO + HI) / 2;
            if (g < MID) at_slot<LO, MID>(g, f);
            else at_slot<MID, HI>(g, f);
        }
    }

    // W sorted, above 128 nodes: its closest unvisited member, and that one's slot in open_slot
    __device__ __forceinline__ u64 closest_open() {
        u64 k = PAG_KEY_INVALID;
#pragma unroll
        for (int s = 0; s < NW; ++s)
            if ((u32)s >= open_slot && k == PAG_KEY_INVALID) {
                const u64 m = __ballot(!(W[s] & 1ull));
                open_slot = (u32)s;
                if (m) k = rdlane64(W[s], __ffsll((long long)m) - 1);
            }
        return k;
    }

    // finds the node that will be expanded next and requests its adjacency record
    __device__ __forceinline__ void look_ahead() {
        nx_key = over_slots<false>(GU);
        nx_known = true;
        nx_id = PAG_EMPTY;
        if (nx_key != PAG_KEY_INVALID) {
            nx_id = (u32)(nx_key & 0xFFFFFFFFull) >> 1;
            load_record(nx_id, pf_id, pf_a, pf_c, pf_cw);
        }
    }

    // Admission into an unsorted W.  The hop's passers are taken in ascending (dist, id) order, exactly as Alg. 2
    // admits them one after the other: while W has room a passer is appended; then a passer closer than W's
    // farthest member takes that member's place and the member goes to R_T; the first passer that is not closer
    // ends it -- the farthest member can only have come closer since, and the remaining passers are no smaller --,
    // and that passer and all after it go to R_F.
    __device__ __forceinline__ void merge_unsorted(u32 id_lane, u64 mask, u32 np, bool pass, float dist) {
        const u32 b = A.b;
        if constexpr (TEAM) nx_known = false;
        const u64 pk = pass ? (((u64)__float_as_uint(dist) << 32) | ((u64)id_lane << 1)) : PAG_KEY_INVALID;
        // rank of my passer among the hop's passers (keys are distinct)
        u32 cP = 0;
        for (u64 m = mask; m;) {
            const int p = __ffsll((long long)m) - 1;
            m &= m - 1;
            cP += (rdlane64(pk, p) < pk) ? 1u : 0u;
        }
        u32 n_ej = 0, j = 0;
        for (; j < np; ++j) {
            const int src = __ffsll((long long)__ballot(pass && cP == j)) - 1;
            const u64 k = rdlane64(pk, src);
            if (nW < b) {
                const int slot = (int)(nW >> 6), ln = (int)(nW & 63u);
                at_slot(slot, [&](auto S_) { constexpr int S = decltype(S_)::value; if (lane == ln) W[S] = k; });
                if (lane == slot) { GM = k > GM ? k : GM; GU = k < GU ? k : GU; }
                nW++;
                if (nW == b) wmax = over_slots<true>(GM);
            } else if (k < wmax) {
                // the farthest member leaves for R_T (pushes of one hop: farthest first), the passer takes its place
                if (lane == 0) RT[(hdT + n_ej) & A.ring_mask] = wmax;
                n_ej++;
                const int g = __ffsll((long long)__ballot(GM == wmax)) - 1;       // its slot
                at_slot(g, [&](auto S_) {
                    constexpr int S = decltype(S_)::value;
                    if (W[S] == wmax) W[S] = k;
                    const u64 m = slot_max<S>();
                    if (lane == S) GM = m;
                });
                // the slot's closest unvisited member: the one that left was it only if it was the slot's last
                if (lane == g) GU = (GU == wmax) ? k : (k < GU ? k : GU);
                wmax = over_slots<true>(GM);
            } else {
                break;
            }
        }
        const u32 n_f = np - j;                                     // false positives -> R_F, smallest first
        if (pass && cP >= j) {
            const u32 oi = cP - j;
            if (oi + b >= n_f) RF[(hdF + oi) & A.ring_mask] = pk;   // older ones would be overwritten anyway
        }
        if (n_ej) {
            if (cntT + n_ej > b) s_rt += cntT + n_ej - b;
            cntT = cntT + n_ej < b ? cntT + n_ej : b;
            hdT += n_ej;
        }
        if (n_f) {
            if (cntF + n_f > b) s_rf += cntF + n_f - b;
            cntF = cntF + n_f < b ? cntF + n_f : b;
            hdF += n_f;
        }
        if constexpr (!TEAM) look_ahead();
    }

    // The query into registers, its table into LDS, the LDS levels of the seen set empty; the waves of a team share the
    // LDS part out.
    __device__ __forceinline__ void begin_query(u32 qi) {
        const u32 d = A.d, tid = (u32)(wave * 64 + lane), step = 64u * (u32)nwaves;
        const float4* qp = (const float4*)(A.qrot + (u64)qi * d);
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
            const u32 idx = c * 64 + lane;
            if constexpr (VM == 1) {
                const bool in = c < NQ - TAILS || idx * 8 < d;
                q[2 * c] = in ? qp[2 * idx] : make_float4(0.f, 0.f, 0.f, 0.f);
                q[2 * c + 1] = in ? qp[2 * idx + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
                q[c] = (c < NQ - TAILS || idx * 4 < d) ? qp[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        const float4* tp = (const float4*)(A.tables + (u64)qi * A.Ppad * PAG_NCODE);
        for (u32 i = tid; i < A.Ppad * PAG_NCODE / 4; i += step) ((float4*)T)[i] = tp[i];
        const uint4 e4 = make_uint4(PAG_EMPTY, PAG_EMPTY, PAG_EMPTY, PAG_EMPTY);
        for (u32 i = tid; i < (1u << A.hlog) / 4; i += step) ((uint4*)H)[i] = e4;
        if (A.blog) {
            const uint4 z4 = make_uint4(0, 0, 0, 0);
            for (u32 i = tid; i < (1u << A.blog) / 128; i += step) ((uint4*)BL)[i] = z4;
        }
    }

    __device__ __forceinline__ void reset_lists() {
#pragma unroll
        for (int s = 0; s < NW; ++s) W[s] = !(BIG && SORTED) ? PAG_KEY_INVALID : (u32)s < first_slot() ? BEFORE_ALL : BEHIND_ALL;
        open_slot = 0;
#pragma unroll
        for (int s = 0; s < (BIG ? 1 : NW); ++s) RL[s] = PAG_KEY_INVALID;
        nW = nRL = n_done = 0;
        cntF = hdF = cntT = hdT = 0;
        n_hash = n_spill = 0;
        Hk = PAG_KEY_INVALID;
        nx_id = PAG_EMPTY;
        wmax = 0; nx_key = PAG_KEY_INVALID; nx_known = false;
        GM = 0ull; GU = PAG_KEY_INVALID;
        n_cand = 0;
        round = 0;
    }

    // Marks the closest unvisited member of W visited and returns its key; PAG_KEY_INVALID: there is none.
    __device__ __forceinline__ u64 pop() {
        const u32 b = A.b;
        u64 ukey = PAG_KEY_INVALID;
        if constexpr (BIG && SORTED) {
            ukey = closest_open();
            if (ukey == PAG_KEY_INVALID) return ukey;
            at_slot((int)open_slot, [&](auto S_) { constexpr int S = decltype(S_)::value; if (W[S] == ukey) W[S] |= 1ull; });
        } else if constexpr (BIG) {
            if (!nx_known) nx_key = over_slots<false>(GU);
            nx_known = false;
            if (nx_key == PAG_KEY_INVALID) return nx_key;
            PAG_MARK(5);
            ukey = nx_key;
            const int g = __ffsll((long long)__ballot(GU == ukey)) - 1;        // its slot
            at_slot(g, [&](auto S_) {
                constexpr int S = decltype(S_)::value;
                if (W[S] == ukey) W[S] |= 1ull;
                const u64 m = slot_min_unvisited<S>();
                if (lane == S) GU = m;
            });
            if (GM == ukey) GM |= 1ull;                                         // it may be its slot's farthest too
            if (nW == b && (wmax | 1ull) == (ukey | 1ull)) wmax |= 1ull;
        } else {
            int us = -1, ul = 0;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                const u64 m = __ballot(idx < nW && !(W[s] & 1ull));
                if (us < 0 && m) { us = s; ul = __ffsll((long long)m) - 1; }
            }
            if (us < 0) return ukey;
            PAG_MARK(5);
#pragma unroll
            for (int s = 0; s < NW; ++s)
                if (s == us) {
                    ukey = rdlane64(W[s], ul);
                    if (lane == ul) W[s] |= 1ull;
                }
        }
        s_hops++;
        return ukey;
    }

    // key of W's farthest member; PAG_KEY_INVALID while W is not full
    __device__ __forceinline__ u64 farthest() const {
        if (nW != A.b) return PAG_KEY_INVALID;
        if constexpr (BIG && SORTED) {
            return rdlane64(W[NW - 1], (int)((A.b - 1) & 63u));
        } else if constexpr (BIG) {
            return wmax;
        } else {
            const u32 wr = A.b - 1;
            u64 k = 0;
#pragma unroll
            for (int s = 0; s < NW; ++s)
                if ((int)(wr >> 6) == s) k = rdlane64(W[s], wr & 63);
            return k;
        }
    }

    // threshold ||z_max - q||^2 of a hop (Eq. 4); +inf while W is not full
    __device__ __forceinline__ static float threshold(u64 far) {
        return far == PAG_KEY_INVALID ? __builtin_inff() : __uint_as_float((u32)(far >> 32));
    }

    // The projection test's input for all neighbours of a node at distance Du: their estimates, and which of them are
    // candidates (in the graph and not known to be seen) and unseen.  Dmax is the threshold or, where that is not known
    // yet, a bound above it: it only decides which neighbours of a long search are looked up in the second level.
    __device__ __forceinline__ void screen(u32 id, float ea, float ec, const u32 (&cwv)[CW], float Du, float Dmax, float& est, bool& cand,
                                           bool& unseen) {
        const bool in_graph = id != PAG_EMPTY && id < A.n_limit;
        // seen-set lookup.  Short searches: the exact LDS hash, then the bitmap word if the hash has
        // overflowed, requested now and consumed after the table sums.  Long searches: the LDS cache of
        // recent ids now; the Bloom filter and the bitmap only for the neighbours that pass the test
        // (a bitmap read costs more than the table sums of the seen neighbours it would spare).
        cand = in_graph;
        if (cand) cand = A.blog != 0 ? H[hash_slot(id, A.hlog)] != id : !hash_contains<TEAM>(H, A.hlog, id);
        u32 bm_word = 0;
        if (A.blog == 0 && n_spill && cand)
            bm_word = __hip_atomic_load(&bitmap[id >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // counting mode of long searches: the second level is consulted for every neighbour, before the
        // test, so that `tests` counts the unseen neighbours only (same results, more bitmap reads)
        const bool resolve_first = A.blog != 0 && (A.flags & PAG_FLAG_EXACT_TEST_COUNT);
        if (resolve_first) {
            u32 wd = 0;
            if (cand && bloom_maybe(BL, A.blog, id))
                wd = __hip_atomic_load(&bitmap[id >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            cand = cand && !((wd >> (id & 31)) & 1u);
        }
        // projection test: S = sum_l T[l][code_l] (increasing l), est = D_u + c - 2 a S
        est = 0.f;
        const bool want_pes = A.pes != nullptr;   // indexing: every neighbour's estimate feeds Eq. 5
        if (!(A.flags & PAG_FLAG_NO_PRT)) {
            float S = 0.f;
            if (cand || (want_pes && in_graph)) {
                S = table_sum<CW>(t_base, cwv);
            }
            est = __builtin_fmaf(-2.0f * ea, S, Du + ec);
        }
        if (A.blog != 0 && !resolve_first) {
            // long searches: only neighbours that pass the test are looked up in the Bloom filter and the bitmap
            const bool maybe = cand && ((A.flags & PAG_FLAG_NO_PRT) || est < Dmax) && bloom_maybe(BL, A.blog, id);
            if (maybe) bm_word = __hip_atomic_load(&bitmap[id >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        unseen = cand && !((bm_word >> (id & 31)) & 1u);
        if (A.blog == 0) cand = unseen;
    }

    __device__ __forceinline__ bool passes(bool unseen, float est, float Dmax) const {
        return unseen && ((A.flags & PAG_FLAG_NO_PRT) || est < Dmax);
    }

    // PES screening (Eq. 5): max_i (cos theta_i / cos beta_i - delta_i) < 0 for all neighbours
    // <=> every estimate est_i exceeds D_u, i.e. no neighbour of u looks closer to v than
    // u itself.  Then u -> v is a candidate edge; H(v) keeps the closest `deg` such nodes.
    __device__ __forceinline__ void screen_pes(u32 id, float est, u64 ukey) {
        const bool in_graph = id != PAG_EMPTY && id < A.n_limit;
        const float Du = __uint_as_float((u32)(ukey >> 32));
        if (__ballot(in_graph && !(est > Du)) == 0ull) {
            const u64 key = (ukey & ~1ull);
            const u32 pos = (u32)__popcll(__ballot(Hk < key));
            const u64 up = __shfl_up(Hk, 1, 64);
            if ((u32)lane == pos) Hk = key;
            else if ((u32)lane > pos) Hk = up;
        }
    }

    // searches that overlap an insertion: a record read between two states of a reverse-edge pass may
    // list one node in two slots; the first slot stands, the merge needs distinct keys
    __device__ __forceinline__ bool first_of_id(u32 id, bool pass) const {
        const u64 all = __ballot(pass);
        u64 again = 0;
        for (u64 m = all; m;) {
            const int p = __ffsll((long long)m) - 1;
            m &= m - 1;
            const u64 same = __ballot(id == rdlane(id, p)) & m;      // slots behind p only are left in m
            m &= ~same;
            again |= same;
        }
        return !((again >> lane) & 1ull);
    }

    // ---- round end (Alg. 2): W -> R_L, clear W; merge + sort rings; refill W; rest -> R_T ----
    __device__ __forceinline__ void end_round(u32 qi) {
        const u32 b = A.b;
        nx_id = PAG_EMPTY;
        if (A.cand) {
            // indexing: R_L has room for every round's W (capacity efC >= Rmax * b and b <= 128 are enforced by the host: above,
            // a team's sorted W lies in other slots, and to compute its ranks here costs its hops 1 to 18 % in spilled registers)
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                if (idx < nW && n_cand + idx < A.cand_cap) A.cand[(u64)qi * A.cand_cap + n_cand + idx] = W[s];
            }
            n_cand = n_cand + nW < A.cand_cap ? n_cand + nW : A.cand_cap;
        } else if constexpr (BIG) {
            // R_L <- best K of R_L + W: R_L (sorted, SA[0, nRL) in HBM) and W are sorted together in registers
            u64 x[2 * NW];
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                x[s] = (SORTED ? rank_at(s) : idx) < nW ? W[s] : PAG_KEY_INVALID;
                x[NW + s] = idx < nRL ? SA[idx] : PAG_KEY_INVALID;
            }
            bitonic_registers<2 * NW>(x, lane);
            const u32 n = nRL + nW;
            nRL = n < A.K ? n : A.K;
#pragma unroll
            for (int s = 0; s < NW; ++s) {                  // K <= b <= 64 NW
                const u32 idx = s * 64 + lane;
                if (idx < nRL) SA[idx] = x[s];
            }
        } else if constexpr (TEAM) {
            // kept until the others are busy with rows (see keep_best)
#pragma unroll
            for (int s = 0; s < NW; ++s) done[s] = W[s];
            n_done = nW;
        } else {
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                if (idx < nRL) SA[idx] = RL[s];
                if (idx < nW) SA[nRL + idx] = W[s];
            }
            lds_sync();
            const u32 n = nRL + nW;
            const u64* S = sort_keys(SA, SB, n, 2 * b <= PAG_RANK_SORT_MAX, lane);
            nRL = n < A.K ? n : A.K;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                RL[s] = idx < nRL ? S[idx] : PAG_KEY_INVALID;
            }
            lds_sync();
        }
        if constexpr (BIG) {
            // this wave's own stores (ring pushes, R_L) must have landed before other lanes read them
            __threadfence();
            const u32 n = cntF + cntT;                       // <= 2b <= 128 NW
            u64 x[2 * NW];
#pragma unroll
            for (int s = 0; s < 2 * NW; ++s) {
                const u32 i = s * 64 + lane;
                u64 k = PAG_KEY_INVALID;
                if (i < cntF) k = RF[(hdF - cntF + i) & A.ring_mask];
                else if (i < n) k = RT[(hdT - cntT + (i - cntF)) & A.ring_mask];
                x[s] = k;
            }
            bitonic_registers<2 * NW>(x, lane);
            nW = n < b ? n : b;
            if constexpr (!SORTED) {
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const u32 idx = s * 64 + lane;
                    W[s] = idx < nW ? x[s] : PAG_KEY_INVALID;
                }
                // W is sorted now: a slot's farthest member is its last, its closest unvisited one the first unvisited
                GM = 0ull; GU = PAG_KEY_INVALID;
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const u32 first = s * 64;
                    if (nW > first) {
                        const u32 cnt = nW - first < 64u ? nW - first : 64u;
                        const u64 far = rdlane64(W[s], (int)cnt - 1);
                        const u64 open = __ballot((u32)lane < cnt && !(W[s] & 1ull));
                        const u64 near = open ? rdlane64(W[s], __ffsll((long long)open) - 1) : PAG_KEY_INVALID;
                        if (lane == s) { GM = far; GU = near; }
                    }
                }
                wmax = nW == b ? over_slots<true>(GM) : 0ull;
                nx_known = false;
            }
            const u32 rest = n - nW;                         // <= b; written worst first
#pragma unroll
            for (int s = 0; s < 2 * NW; ++s) {
                const u32 e = s * 64 + lane;
                if (e >= nW && e < n) RT[n - 1 - e] = x[s];
            }
            if constexpr (SORTED) {
                // W to its slots, through the memory of R_F, which is empty now
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const u32 idx = s * 64 + lane;
                    if (idx < b) RF[idx] = idx < nW ? x[s] : BEHIND_ALL;
                }
                __threadfence();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < NW; ++s) {
                    const u32 at = rank_at(s);
                    const u64 k = __hip_atomic_load(&RF[at < b ? at : 0u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    W[s] = at < b ? k : (u32)s < first_slot() ? BEFORE_ALL : BEHIND_ALL;
                }
                open_slot = 0;
            }
            cntT = rest; hdT = rest;
            cntF = 0; hdF = 0;
        } else if (TEAM && cntF + cntT <= 64) {
            // in registers: one key a lane
            const u32 n = cntF + cntT;
            u64 x = PAG_KEY_INVALID;
            if ((u32)lane < cntF) x = RF[(hdF - cntF + lane) & A.ring_mask];
            else if ((u32)lane < n) x = RT[(hdT - cntT + (lane - cntF)) & A.ring_mask];
            const u32 r = rank_among(x, n);
            if ((u32)lane < n) SA[r] = x;
            lds_sync();
            if ((u32)lane < n) x = SA[lane];
            nW = n < b ? n : b;
            W[0] = (u32)lane < nW ? x : PAG_KEY_INVALID;
#pragma unroll
            for (int s = 1; s < NW; ++s) W[s] = PAG_KEY_INVALID;
            if ((u32)lane >= nW && (u32)lane < n) RT[n - 1 - lane] = x;      // the rest, worst first
            cntT = hdT = n - nW;
            cntF = 0; hdF = 0;
            lds_sync();
        } else {
            for (u32 i = lane; i < cntF; i += 64) SA[i] = RF[(hdF - cntF + i) & A.ring_mask];
            for (u32 i = lane; i < cntT; i += 64) SA[cntF + i] = RT[(hdT - cntT + i) & A.ring_mask];
            lds_sync();
            const u32 n = cntF + cntT;
            const u64* S = sort_keys(SA, SB, n, 2 * b <= PAG_RANK_SORT_MAX, lane);
            nW = n < b ? n : b;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                W[s] = idx < nW ? S[idx] : PAG_KEY_INVALID;
            }
            const u32 rest = n - nW;                         // <= b; written worst first
            for (u32 j = lane; j < rest; j += 64) RT[j] = S[n - 1 - j];
            cntT = rest; hdT = rest;
            cntF = 0; hdF = 0;
            lds_sync();
        }
    }

    __device__ __forceinline__ void write_results(u32 qi) const {
        if (A.cand) {
            if (wave == 0 && lane == 0) A.cand_cnt[qi] = n_cand;
            // the buffer H(v) is kept where the screening is done
            if (A.pes && wave == (TEAM ? 1 : 0) && (u32)lane < A.deg) A.pes[(u64)qi * A.deg + lane] = Hk;
        } else if (wave == 0) {
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 idx = s * 64 + lane;
                if (idx < A.K) {
                    long long oid = -1;
                    float od = __builtin_inff();
                    if (idx < nRL) {
                        u64 key;
                        if constexpr (BIG) key = SA[idx];
                        else key = RL[s];
                        oid = (long long)((u32)(key & 0xFFFFFFFFull) >> 1);
                        od = A.out_scale * __uint_as_float((u32)(key >> 32));
                    }
                    A.out_ids[(u64)qi * A.K + idx] = oid;
                    A.out_dists[(u64)qi * A.K + idx] = od;
                }
            }
        }
    }

    // a spilled query leaves its bitmap clean for the next one
    __device__ __forceinline__ void clear_bitmap() const {
        uint4* bm = (uint4*)bitmap;
        const uint4 z = make_uint4(0, 0, 0, 0);
        for (u64 i = wave * 64 + lane; i < A.bitmap_words / 4; i += 64 * nwaves) bm[i] = z;
        __threadfence();
    }

    // entry nodes base .. base + 63 (Alg. 2, entry step): this lane's id, or PAG_EMPTY
    __device__ __forceinline__ u32 entry_node(u32 base, u32 ne) const {
        const u32 i = base + lane;
        u32 id = PAG_EMPTY;
        if (i < ne) id = A.entry[i];
        return id != PAG_EMPTY && id < A.n_limit ? id : PAG_EMPTY;
    }

    // one query, one wave
    __device__ __forceinline__ void run_query(u32 qi) {
        begin_query(qi);
        reset_lists();
        __syncthreads();
        s_queries++;
        // ---- b entry nodes (Alg. 2, entry step) ----
        const u32 ne = A.n_entry < A.b ? A.n_entry : A.b;
        for (u32 base = 0; base < ne; base += 64) {
            const u32 id = entry_node(base, ne);
            admit(id, __ballot(id != PAG_EMPTY));
        }
        // ---- rounds ----
        for (u32 r = 0; r < A.Rmax; ++r) {
            if (nW == 0) break;
            s_rounds++;
            for (;;) {
                const u64 ukey = pop();
                if (ukey == PAG_KEY_INVALID) break;
                set_priority(2);   // screening leads to the next loads: ahead of other waves' bookkeeping
                const u32 u = (u32)(ukey & 0xFFFFFFFFull) >> 1;
                const float Dmax = threshold(farthest());      // read once per hop
                PAG_MARK(0);
                // adjacency record of u: normally already on its way (see request_next)
                u32 id;
                float ea, ec;
                u32 cwv[CW];
                if (u == nx_id) {
                    id = pf_id; ea = pf_a; ec = pf_c;
#pragma unroll
                    for (int k = 0; k < CW; ++k) cwv[k] = pf_cw[k];
                } else {
                    load_record(u, id, ea, ec, cwv);
                }
                nx_id = PAG_EMPTY;
                PAG_MARK(1);
                float est;
                bool cand, unseen;
                screen(id, ea, ec, cwv, __uint_as_float((u32)(ukey >> 32)), Dmax, est, cand, unseen);
                bool pass = passes(unseen, est, Dmax);
                if (A.pes != nullptr) screen_pes(id, est, ukey);
                if (A.flags & PAG_SEARCH_DISTINCT) {
                    const bool first = first_of_id(id, pass);
                    pass = pass && first;
                    cand = cand && first;
                }
                const u64 pmask = __ballot(pass);
                s_tests += (u32)__popcll(__ballot(cand));
                s_passes += (u32)__popcll(pmask);
                admit(id, pmask);
            }
            end_round(qi);
        }
        write_results(qi);
        if (n_spill) clear_bitmap();
    }

    // ---- several waves on one query (TEAM) ----
    // With few queries the GPU waits for one hop after the other, and a single wave adds up the hop's trips to memory
    // (record, rows two at a time, next record) and all of its bookkeeping, at one instruction per 4 to 10 clocks.  Here
    // wave 0 keeps W and the rings, wave 1 the seen set, wave 2 computes the estimates, and the other waves fetch the rows; in teams of
    // less than six wave 0 computes those estimates that have time, and wave 2 fetches rows besides.  A hop has two phases between barriers:
    //   rows    every wave reads the node's neighbours, their estimates and the threshold from LDS and derives the
    //           passers, whose rows are fetched all at once, their records behind them.  Meanwhile wave 0 does what the last
    //           hop left it (ring pushes, a finished round's entry into R_L), wave 1 enters the passers into the seen set, and the
    //           neighbours of W's closest unvisited member are screened ahead;
    //   lists   wave 0 enters the passers that are closer than W's farthest member and pops the next node.  Which node that will
    //           be is known before: the closest passer, if it enters W and is closer than W's closest unvisited member (half of
    //           the hops at b = 10), else that member, whose neighbours are screened already; a passer's are screened now.
    //           Only the threshold has to wait.
    // Where a round has ended in between (every eleventh hop at b = 10) the node is another one, and it is screened in a phase
    // of its own.
    // 37 queries, 1M x 768, efS 512: 5.85 us a hop with one wave, 2.2 with twelve (4,900 clocks: rows 2,600, of which a trip to
    // memory is 1,200 and wave 1's seen set 1,700, wave 0's lists 1,400, the rest reading what is posted, barriers).  While every row wave also
    // ranked its passers against W for a merge by scatter through LDS, and a record was first asked for when its node was
    // expanded, it was 2.6.
    enum : u32 {
        TM_QUERY = 0,                                  // query number, PAG_EMPTY: no more
        TM_SPILLED,                                    // wave 1: the search has used its bitmap
        // four words wave 0: the node to expand (PAG_EMPTY: the search is over) and its distance, W's farthest
        TM_NODE = 4, TM_NODE_DIST, TM_FAR_LO, TM_FAR_HI,
        // two words wave 0: W's closest unvisited member after that (PAG_EMPTY: none); wave 1: the node whose neighbours are screened
        TM_SECOND = 8, TM_SECOND_DIST, TM_SCREENED,
        TM_ID = 64,                                    // wave 1, per neighbour slot: id (PAG_EMPTY: not an unseen node)
        TM_EST = 128,                                  // wave 2, per neighbour slot: estimate
        TM_KEY = 192                                   // u64: keys of the hop's passers, in slot order
    };
    static_assert(TM_KEY + 128 <= PAG_TEAM_WORDS, "team words");

    // raw barrier: unlike __syncthreads() it leaves global loads in flight
    __device__ __forceinline__ void team_barrier() const {
        lds_sync();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    // whether the estimates have a wave of their own
    __device__ __forceinline__ bool split() const { return nwaves >= 6; }

    __device__ __forceinline__ u32 team_index(u64 mask) const { return (u32)__popcll(mask & ((1ull << lane) - 1)); }
    __device__ __forceinline__ u64* team_keys() const { return (u64*)(team + TM_KEY); }

    // the smallest key of the hop's np passers; PAG_KEY_INVALID: there are none
    __device__ __forceinline__ u64 closest_passer(u32 np) const {
        if (np == 0) return PAG_KEY_INVALID;
        const u64 k = (u32)lane < np ? team_keys()[lane] : PAG_KEY_INVALID;
        const u32 hi = (u32)(k >> 32);
        if (np <= 16) {
            const u32 mh = row0_extreme_u32<false>(hi);
            return ((u64)mh << 32) | row0_extreme_u32<false>(hi == mh ? (u32)k : 0xFFFFFFFFu);
        }
        const u32 mh = wave_extreme_u32<false>(hi);
        return ((u64)mh << 32) | wave_extreme_u32<false>(hi == mh ? (u32)k : 0xFFFFFFFFu);
    }

    // This wave's share of the rows of the lanes in `mask`, at most TR of them in flight at a time.  The rows of a wave are reduced
    // together: one row alone is a chain of dependent instructions.
    static constexpr int TR = NQ * (int)sizeof(Chunk) <= 48 ? 4 : (NQ * (int)sizeof(Chunk) <= 96 ? 2 : 1);

    // R rows of this wave, those of passers at, at + step, ...: they are asked for in straight-line code.  With a request in a branch of its own
    // the compiler waits for an earlier row before it: of four rows the third and the fourth came a trip to memory
    // later (1,000 queries of 1M x 768 1.161 -> 1.122 ms, 250 x 3072 1.442 -> 1.366, 512 x 768 in 16 bits 1.379 -> 1.332).
    template <int R, bool AHEAD>
    __device__ __forceinline__ void rows_at(u32 id_lane, u32 mine, u32 at, u32 step, u32& touched) const {
        constexpr int G = R == 3 ? 4 : R;
        const u32 line = (u32)lane * 128u < A.rec_bytes ? (u32)lane * 128u : 0u;
        Chunk v[R][NQ];
        u32 id[R], word[R];
#pragma unroll
        for (int g = 0; g < R; ++g) id[g] = rdlane(id_lane, __ffsll((long long)__ballot(mine == at + (u32)g * step)) - 1);
#pragma unroll
        for (int g = 0; g < R; ++g) load_vec(v[g], id[g]);
        if constexpr (AHEAD) {
#pragma unroll
            for (int g = 0; g < R; ++g) word[g] = *(const u32*)(A.rec + (u64)id[g] * A.rec_bytes + line);
        }
        __builtin_amdgcn_sched_barrier(0);
        double acc[G];
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = 0.0;
#pragma unroll
        for (int g = 0; g < R; ++g) acc[g] = lane_partial(v[g]);
        const double tot = fold_sum<G>(acc);                // lanes g * 64 / G ...: the total of row g
        const u32 g = (u32)lane / (64 / G);
        u32 my_id = id[0];
#pragma unroll
        for (u32 i = 1; i < R; ++i) {
            u32 other = id[i];
            asm volatile("" : "+v"(other));                 // or the compiler indexes the ids in scratch
            my_id = g == i ? other : my_id;
        }
        if ((u32)lane % (64 / G) == 0 && g < (u32)R) {
            const u32 bits = __float_as_uint((float)tot);       // a NaN of either sign: the largest distance
            team_keys()[at + g * step] = ((u64)(bits < 0x7FC00000u ? bits : 0x7FC00000u) << 32) | ((u64)my_id << 1);
        }
        if constexpr (AHEAD) {
#pragma unroll
            for (int g = 0; g < R; ++g) touched |= word[g];
        }
    }

    // Half of the nodes that are expanded are passers of the hop before: AHEAD asks for a row's record behind it, one lane per
    // 128-byte line, so that the caches have it when the node is screened (teams of six and more: smaller ones fill the GPU, and
    // then the traffic costs more).  Returns something of it, to be waited for later.
    template <bool AHEAD>
    __device__ __forceinline__ u32 team_rows(u32 id_lane, u64 mask) const {
        const u32 first = AHEAD ? 3u : 2u;                  // the first wave that fetches rows
        const u32 n = (u32)__popcll(mask), step = (u32)nwaves - first;
        const u32 mine = ((mask >> lane) & 1ull) ? team_index(mask) : PAG_EMPTY;
        u32 touched = 0;
        for (u32 at = (u32)wave - first; at < n; at += TR * step) {
            if (TR < 2 || at + step >= n) rows_at<1, AHEAD>(id_lane, mine, at, step, touched);
            else if (TR < 4 || at + 2 * step >= n) { if constexpr (TR >= 2) rows_at<2, AHEAD>(id_lane, mine, at, step, touched); }
            else if (at + 3 * step >= n) { if constexpr (TR >= 4) rows_at<3, AHEAD>(id_lane, mine, at, step, touched); }
            else if constexpr (TR >= 4) rows_at<4, AHEAD>(id_lane, mine, at, step, touched);
        }
        return touched;
    }

    // key of W's closest unvisited member, which stays unvisited
    __device__ __forceinline__ u64 peek() {
        if constexpr (BIG && SORTED) {
            return closest_open();
        } else if constexpr (BIG) {
            if (!nx_known) nx_key = over_slots<false>(GU);
            nx_known = true;
            return nx_key;
        } else {
            u64 k = PAG_KEY_INVALID;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u64 m = __ballot((u32)(s * 64 + lane) < nW && !(W[s] & 1ull));
                if (m && k == PAG_KEY_INVALID) k = rdlane64(W[s], __ffsll((long long)m) - 1);
            }
            return k;
        }
    }

    // wave 0: what the other waves need to know of W
    __device__ __forceinline__ void post(u64 node, u64 far, u64 second) {
        const u32 n = posted_node = node != PAG_KEY_INVALID ? (u32)node >> 1 : PAG_EMPTY;
        if (lane == 0) {
            const u32 s = second != PAG_KEY_INVALID ? (u32)second >> 1 : PAG_EMPTY;
            *(uint4*)(team + TM_NODE) = make_uint4(n, (u32)(node >> 32), (u32)far, (u32)(far >> 32));
            *(uint2*)(team + TM_SECOND) = make_uint2(s, (u32)(second >> 32));
        }
    }

    // wave 0: R_L <- the best K of R_L and the W of the last round
    __device__ __forceinline__ void keep_best() {
        if constexpr (!BIG) {
            if (n_done == 0) return;
            double w[NW];
            u64 kth = PAG_KEY_INVALID;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                w[s] = __longlong_as_double((long long)((u32)(s * 64 + lane) < nRL ? RL[s] : BEHIND_ALL));
                if (nRL == A.K && (int)((A.K - 1) >> 6) == s) kth = rdlane64(RL[s], (int)((A.K - 1) & 63u));
            }
            u32 n = 0;
#pragma unroll
            for (int s = 0; s < NW; ++s) {
                const u32 enter = (u32)__popcll(__ballot((u32)(s * 64 + lane) < n_done && done[s] < kth));      // done is sorted
                const double d = __longlong_as_double((long long)done[s]);
                for (u32 i = 0; i < enter; ++i) (void)insert(w, lane_value(d, (int)i));
                n += enter;
            }
            nRL = nRL + n < A.K ? nRL + n : A.K;
#pragma unroll
            for (int s = 0; s < NW; ++s) RL[s] = (u32)(s * 64 + lane) < nRL ? (u64)__double_as_longlong(w[s]) : PAG_KEY_INVALID;
            n_done = 0;
        }
    }

    // wave 0: pops the next node, through as many round ends as that takes, and posts it
    __device__ __forceinline__ void post_next(u32 qi) {
        u64 ukey = PAG_KEY_INVALID;
        while (round < A.Rmax && nW != 0) {
            ukey = pop();
            if (ukey != PAG_KEY_INVALID) break;
            keep_best();
            end_round(qi);
            round++;
            if (round < A.Rmax && nW != 0) s_rounds++;
        }
        post(ukey, farthest(), ukey != PAG_KEY_INVALID ? peek() : PAG_KEY_INVALID);
    }

    // wave 0, sorted W: the hop's np passers, whose keys lie in LDS, in two parts: W itself, ...
    // (Working sets of 129 to 512 nodes were unsorted here too.  A passer cost them a reduction over one slot, one over all
    // slots and a search for the member that leaves, all one after the other; to step to the next lane is four slots at a time and needs no
    // search.  Unsorted -> sorted, 50k x 768, one query / 256 / 512: K 150, efS 600 1778 -> 1170 us, 1832 -> 1226, 2134 -> 1448 (with the eight waves that the
    // registers allow now); K 300, efS 1200 3437 -> 2867, 3518 -> 2916, 4225 -> 3790; K 500, efS 1500 4217 -> 3459, 4385 -> 3600, 5143 -> 4574.  Every length of
    // rows and store that there is a kernel for, 128-d to 3072-d, K 150 to 256: 1.28 to 1.78 times as fast up to one query a CU, 1.15 to 1.68 up to two; K 300 to 500
    // 1.17 to 1.50, 1.02 to 1.32.  With sixteen slots the registers spill inside the hop: 300 queries, K 1000 17.9 ms unsorted, 19.2 sorted.)
    // A passer takes its place by one comparison of every member, and those behind it step to the next lane (470 clocks a hop; by
    // ranks and a scatter through LDS 840, with the counting in the row waves besides).  The keys are
    // compared as doubles, whose order is theirs (the distance word of a key is at most that of a NaN, 0x7FC00000, see
    // rows_at: no key is a NaN or an infinity as a double), in one instruction each.
    static constexpr int OW = NW < 2 ? NW : 2;          // the slots that lose members: a hop has 64 passers at most
    struct Merge {
        u64 oldW[OW], pk, far;
        u32 nW, np;
    };
    // Above 128 nodes rank r lies in slot first_slot() + r / 64, so that the farthest member of a full W is in the last slot; places
    // without a member count as visited.
    static constexpr u64 BEHIND_ALL = 0x7FEFFFFFFFFFFFFFull;       // a place behind the last member: the largest double
    static constexpr u64 BEFORE_ALL = 0xBFF0000000000001ull;       // the places of slots before the first: below 0
    __device__ __forceinline__ u32 first_slot() const { return BIG ? (u32)NW - (A.b + 63u) / 64u : 0u; }
    __device__ __forceinline__ u32 rank_at(int s) const { return ((u32)s - first_slot()) * 64u + (u32)lane; }       // of slots before the first: huge
    template <bool FIRST>
    __device__ __forceinline__ static double from_below(double x, double first) {      // lane l: x of lane l - 1; lane 0: first, or 0
        constexpr int WAVE_SHR1 = 0x138;
        const int lo = __builtin_amdgcn_update_dpp(FIRST ? __double2loint(first) : 0, __double2loint(x), WAVE_SHR1, 0xF, 0xF, !FIRST);
        const int hi = __builtin_amdgcn_update_dpp(FIRST ? __double2hiint(first) : 0, __double2hiint(x), WAVE_SHR1, 0xF, 0xF, !FIRST);
        return __hiloint2double(hi, lo);
    }
    // Four slots at a time where there are many, those before k's place left alone; returns the first slot that may have changed.
    __device__ __forceinline__ static u32 insert(double (&w)[NW], double k) {
        if constexpr (NW <= 2) {
            double below[NW];
            below[0] = from_below<false>(w[0], 0.0);
#pragma unroll
            for (int s = 1; s < NW; ++s) below[s] = from_below<true>(w[s], lane_value(w[s - 1], 63));
#pragma unroll
            for (int s = 0; s < NW; ++s) w[s] = fmin(w[s], fmax(below[s], k));
            return 0;
        } else {
            constexpr int STEP = 4;
            u32 slot = NW - STEP;
            bool here = true;
#pragma unroll
            for (int g = NW - STEP; g >= 0; g -= STEP) {
                if (g < NW - STEP) here = here && k < lane_value(w[g + STEP - 1], 63);
                if (here) {
#pragma unroll
                    for (int s = g + STEP - 1; s >= g; --s) w[s] = fmin(w[s], fmax(from_below<true>(w[s], s > 0 ? lane_value(w[s > 0 ? s - 1 : 0], 63) : -1.0), k));
                    slot = (u32)g;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            return slot;
        }
    }
    __device__ __forceinline__ void merge_w(Merge& M, u32 np) {
        M.pk = (u32)lane < np ? team_keys()[lane] : PAG_KEY_INVALID;
        M.np = np; M.nW = nW;
        double w[NW];
#pragma unroll
        for (int s = 0; s < OW; ++s) M.oldW[s] = W[NW - OW + s];
#pragma unroll
        for (int s = 0; s < NW; ++s)
            w[s] = __longlong_as_double((long long)(BIG || (u32)(s * 64 + lane) < nW ? W[s] : BEHIND_ALL));
        const double pk = __longlong_as_double((long long)M.pk);
        const u64 far0 = farthest();
        for (u64 m = __ballot((u32)lane < np && M.pk < far0); m; m &= m - 1) {
            const u32 slot = insert(w, lane_value(pk, __ffsll((long long)m) - 1));
            if (BIG && slot < open_slot) open_slot = slot;
        }
        nW = nW + np < A.b ? nW + np : A.b;
#pragma unroll
        for (int s = 0; s < NW; ++s) W[s] = BIG || (u32)(s * 64 + lane) < nW ? (u64)__double_as_longlong(w[s]) : PAG_KEY_INVALID;
        if (BIG && (u32)lane > ((A.b - 1) & 63u)) W[NW - 1] = BEHIND_ALL;       // pushed out of a full W
        M.far = farthest();
    }
    // ... and what it pushes to the rings: displaced members to R_T (largest first), passers that do not fit to R_F (smallest first)
    __device__ __forceinline__ void merge_rings(const Merge& M) {
        const u32 b = A.b;
        const u64 fails = __ballot((u32)lane < M.np && M.pk > M.far);
        const u32 n_f = (u32)__popcll(fails);
        const u32 n_ej = M.nW + (M.np - n_f) - (M.nW + M.np < b ? M.nW + M.np : b);
        if (n_ej) {
#pragma unroll
            for (int s = 0; s < OW; ++s) {
                const u32 idx = rank_at(NW - OW + s);
                if (idx < M.nW && M.oldW[s] > M.far) RT[(hdT + (M.nW - 1 - idx)) & A.ring_mask] = M.oldW[s];
            }
            if (cntT + n_ej > b) s_rt += cntT + n_ej - b;
            cntT = cntT + n_ej < b ? cntT + n_ej : b;
            hdT += n_ej;
        }
        if (n_f) {
            u32 oi = 0;
            for (u64 m = fails; m; m &= m - 1) oi += rdlane64(M.pk, __ffsll((long long)m) - 1) < M.pk ? 1u : 0u;
            if (((fails >> lane) & 1ull) && oi + b >= n_f) RF[(hdF + oi) & A.ring_mask] = M.pk;  // older ones would be overwritten anyway
            if (cntF + n_f > b) s_rf += cntF + n_f - b;
            cntF = cntF + n_f < b ? cntF + n_f : b;
            hdF += n_f;
        }
    }

    // which of a node's neighbours are unseen
    __device__ __forceinline__ bool find_unseen(u32 id) const {
        bool cand = id != PAG_EMPTY && id < A.n_limit;
        u32 word = 0;
        if (A.blog != 0) {
            // the second level is consulted for every neighbour that the first does not know: the estimates, which
            // could spare some, are computed by another wave meanwhile
            cand = cand && H[hash_slot(id, A.hlog)] != id;
            if (cand && bloom_maybe(BL, A.blog, id))
                word = __hip_atomic_load(&bitmap[id >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            if (cand) cand = !hash_contains<TEAM>(H, A.hlog, id);
            if (n_spill && cand) word = __hip_atomic_load(&bitmap[id >> 5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return cand && !((word >> (id & 31)) & 1u);
    }

    // sum_l T[l][code_l] of a node's neighbours
    __device__ __forceinline__ float code_sum(const u32 (&cwv)[CW]) const {
        if (A.flags & PAG_FLAG_NO_PRT) return 0.f;
        if (A.cw == 2) return table_sum<2>(t_base, cwv);
        if (A.cw == 4) return table_sum<4, CW, 32>(t_base, cwv);
        return table_sum<8, CW, 32>(t_base, cwv);
    }

    // The screening of a node's neighbours; SEEN and EST: which half of it this wave does.  What it needs of the record of
    // W's closest unvisited member is kept in the prefetch registers (nx_id: whose), the sums with it: that member is often
    // expanded some hops later.
    template <bool SEEN, bool EST>
    __device__ __forceinline__ void fetch_screen(u32 u) {
        if (u == nx_id) return;
        nx_id = u;
        if constexpr (SEEN) pf_id = load_id(u);
        if constexpr (EST) { load_edges(u, pf_a, pf_c, pf_cw); pf_summed = false; }
    }
    __device__ __forceinline__ void sum_codes() {
        if (!pf_summed) pf_sum = code_sum(pf_cw);
        pf_summed = true;
    }
    __device__ __forceinline__ void put_unseen(u32 id, bool unseen) {
        scr_id = id;
        team[TM_ID + lane] = unseen ? id : PAG_EMPTY;
    }
    __device__ __forceinline__ void put_estimate(float Du, float ea, float ec, float sum) {
        team[TM_EST + lane] = __float_as_uint(__builtin_fmaf(-2.0f * ea, sum, Du + ec));
    }
    // ... of a node whose record is not at hand
    template <bool SEEN, bool EST>
    __device__ __forceinline__ void screen_node(u32 u, float Du) {
        u32 id = PAG_EMPTY;
        float ea, ec;
        u32 cwv[CW];
        if constexpr (SEEN) id = load_id(u);
        if constexpr (EST) {
            load_edges(u, ea, ec, cwv);
            put_estimate(Du, ea, ec, code_sum(cwv));
        }
        if constexpr (SEEN) put_unseen(id, find_unseen(id));
    }

    // One wave of the workgroup: queries until the batch is drained.  Each role is compiled by itself, so that the
    // registers hold what that role needs.
    enum Role { LISTS, SEEN, ESTIMATES, ROWS_AHEAD, LISTS_FEW, ROWS };       // teams of six and more: the first four; smaller ones: LISTS_FEW, SEEN, ROWS
    template <Role ROLE>
    __device__ __forceinline__ void run_team() {
        constexpr bool KEEPS_LISTS = ROLE == LISTS || ROLE == LISTS_FEW, KEEPS_SEEN = ROLE == SEEN;
        constexpr bool AHEAD = ROLE == ROWS_AHEAD, FETCH = ROLE == ROWS || AHEAD;
        // the estimates of the neighbours of W's closest unvisited member, computed ahead: wave 2, in small teams wave 0
        constexpr bool ESTIMATE = ROLE == ESTIMATES || ROLE == LISTS_FEW;
        // those of a node whose record is not at hand: wave 2, in small teams too, whose rows are done then
        constexpr bool MAY_ESTIMATE = ROLE == ESTIMATES || ROLE == ROWS;
        const bool estimates = ROLE == ESTIMATES || (ROLE == ROWS && wave == 2);
        for (u32 take = 0;; ++take) {
            // or what begins and ends a query is computed before all of them and held in registers all along (3072-d 18 -> 2 spilled, 1536-d
            // 12 -> 0; with the reads of codes above 250 x 3072 1,380 -> 1,318 us, K 1000 18.9 -> 17.9 ms)
            asm volatile("" : "+v"(lane));
            if constexpr (KEEPS_LISTS) {
                u32 qi = take == 0 ? blockIdx.x : next_query();
                if (qi >= A.nq) qi = PAG_EMPTY;
                else if (A.order) qi = A.order[qi];
                if (lane == 0) team[TM_QUERY] = qi;
            }
            team_barrier();
            const u32 qi = uniform(team[TM_QUERY]);
            if (qi == PAG_EMPTY) break;
            begin_query(qi);
            reset_lists();
            team_barrier();
            if constexpr (KEEPS_LISTS) s_queries++;
            // ---- b entry nodes ----
            const u32 ne = A.n_entry < A.b ? A.n_entry : A.b;
            for (u32 base = 0; base < ne; base += 64) {
                const u32 id = entry_node(base, ne);
                const bool pass = id != PAG_EMPTY;
                const u64 mask = __ballot(pass);
                if (mask == 0ull) continue;
                const u32 np = (u32)__popcll(mask);
                if constexpr (FETCH) (void)team_rows<AHEAD>(id, mask);
                if constexpr (KEEPS_SEEN) mark_seen(id, np, pass);
                team_barrier();
                if constexpr (KEEPS_LISTS) {
                    s_exact += np;
                    if constexpr (SORTED) {
                        Merge M;
                        merge_w(M, np);                // no more than b in all: nothing for the rings
                    } else {
                        merge_unsorted(id, mask, np, pass, __uint_as_float((u32)(team_keys()[pass ? team_index(mask) : 0u] >> 32)));
                    }
                }
                team_barrier();
            }
            if constexpr (KEEPS_LISTS) {
                if (nW != 0) s_rounds++;
                post_next(qi);
            }
            if (KEEPS_SEEN && lane == 0) team[TM_SCREENED] = PAG_EMPTY;
            team_barrier();
            // ---- hops ----
            bool owed = false;                         // wave 0: a merge whose ring pushes are outstanding
            Merge M;
            for (;;) {
                PAG_MARK(0);
                // all that wave 0 and the screening have left, asked for at once
                uint4 posted = *(const uint4*)(team + TM_NODE), more = *(const uint4*)(team + TM_SECOND);
                u32 id = team[TM_ID + lane];
                float est = __uint_as_float(team[TM_EST + lane]);
                asm volatile("" : "+v"(posted.x), "+v"(posted.y), "+v"(posted.z), "+v"(posted.w), "+v"(more.x), "+v"(more.y), "+v"(more.z), "+v"(id), "+v"(est));
                const u32 u = uniform(posted.x), du = uniform(posted.y);
                if (u == PAG_EMPTY) break;
                const u64 far = ((u64)uniform(posted.w) << 32) | uniform(posted.z);
                const u32 second = uniform(more.x), second_d = uniform(more.y);
                // TM_SCREENED stays as it is until all waves have read it: it is written again after the rows
                if (uniform(more.z) != u) {
                    if constexpr (KEEPS_SEEN) screen_node<true, false>(u, __uint_as_float(du));
                    if constexpr (MAY_ESTIMATE) { if (estimates) screen_node<false, true>(u, __uint_as_float(du)); }
                    team_barrier();
                    id = team[TM_ID + lane];
                    est = __uint_as_float(team[TM_EST + lane]);
                }
                bool pass = passes(id != PAG_EMPTY, est, threshold(far));
                if (A.flags & PAG_SEARCH_DISTINCT) { const bool first = first_of_id(id, pass); pass = pass && first; }
                const u64 mask = __ballot(pass);
                const u32 np = (u32)__popcll(mask);
                PAG_MARK(2);
                bool unseen = false;                   // of the neighbours of `second`
                u32 touched = 0;
                if constexpr (KEEPS_SEEN) {
                    if (A.pes != nullptr) screen_pes(scr_id, est, ((u64)du << 32) | ((u64)u << 1));
                }
                if constexpr (KEEPS_SEEN || ESTIMATE) {
                    if (second != PAG_EMPTY) fetch_screen<KEEPS_SEEN, ESTIMATE>(second);
                }
                if constexpr (FETCH) touched = team_rows<AHEAD>(id, mask);
                if constexpr (KEEPS_SEEN) {
                    s_tests += (u32)__popcll(__ballot(id != PAG_EMPTY));
                    s_passes += np;
                    if (np) mark_seen(id, np, pass);
                    if (second != PAG_EMPTY) unseen = find_unseen(pf_id);
                }
                if constexpr (KEEPS_LISTS) {
                    if (owed) merge_rings(M);
                    keep_best();
                }
                if constexpr (ESTIMATE) {
                    if (second != PAG_EMPTY) sum_codes();
                }
                PAG_MARK(1);
                team_barrier();
                PAG_MARK(3);
                if constexpr (AHEAD) asm volatile("" :: "v"(touched));
                if constexpr (KEEPS_LISTS) {
                    s_exact += np;
                    if constexpr (SORTED) {
                        owed = np != 0;
                        if (np) merge_w(M, np);
                        const u64 next = pop();
                        if (next != PAG_KEY_INVALID) {
                            post(next, owed ? M.far : farthest(), peek());
                        } else {
                            if (owed) merge_rings(M);
                            owed = false;
                            post_next(qi);
                        }
                    } else {
                        owed = false;
                        if (np) merge_unsorted(id, mask, np, pass, __uint_as_float((u32)(team_keys()[pass ? team_index(mask) : 0u] >> 32)));
                        post_next(qi);
                    }
                }
                if (KEEPS_SEEN || (MAY_ESTIMATE && estimates)) {
                    const u64 first = closest_passer(np);
                    const u64 next2 = second != PAG_EMPTY ? ((u64)second_d << 32) | ((u64)second << 1) : PAG_KEY_INVALID;
                    const bool passer = first < far && first < next2;
                    const u64 next = passer ? first : next2;
                    const u32 node = uniform(next != PAG_KEY_INVALID ? (u32)next >> 1 : PAG_EMPTY);
                    if (KEEPS_SEEN && lane == 0) team[TM_SCREENED] = node;
                    const float Du = __uint_as_float((u32)(next >> 32));
                    if (passer) {
                        if constexpr (KEEPS_SEEN) screen_node<true, false>(node, Du);
                        if constexpr (MAY_ESTIMATE) screen_node<false, true>(node, Du);
                    } else if (node != PAG_EMPTY) {
                        if constexpr (KEEPS_SEEN) put_unseen(pf_id, unseen);
                        if constexpr (ROLE == ESTIMATES) put_estimate(Du, pf_a, pf_c, pf_sum);
                    }
                }
                if constexpr (ROLE == LISTS_FEW) {
                    if (second != PAG_EMPTY && posted_node == second) put_estimate(__uint_as_float(second_d), pf_a, pf_c, pf_sum);
                }
                PAG_MARK(4);
                team_barrier();
            }
            if constexpr (KEEPS_LISTS) keep_best();
            if constexpr (KEEPS_LISTS || KEEPS_SEEN) write_results(qi);
            if constexpr (KEEPS_SEEN) {
                if (n_spill) __threadfence();        // its bit-sets have landed before others clear
                if (lane == 0) team[TM_SPILLED] = n_spill ? 1u : 0u;
            }
            team_barrier();
            if (uniform(team[TM_SPILLED])) clear_bitmap();
        }
    }

    // the next query that no workgroup has (A.nq and above: there is none)
    __device__ __forceinline__ u32 next_query() const {
        if (A.numbered >= A.nq) return A.nq;
        u32 qi = 0;
        if (lane == 0) qi = A.numbered + atomicAdd(A.qcounter, 1u);
        return uniform(qi);
    }

    __device__ __forceinline__ void flush_stats() {
        u64* line = A.counters + (u64)(blockIdx.x % PAG_CTR_COPIES) * CTR_LINE;
        // one counter a lane
        u32 v = 0;
        auto put = [&](int counter, u32 x) {
            asm volatile("" : "+v"(x));          // or the compiler indexes the members in scratch, and with them all of this object
            v = lane == counter ? x : v;
        };
        put(CTR_QUERIES, s_queries); put(CTR_HOPS, s_hops); put(CTR_TESTS, s_tests); put(CTR_PASSES, s_passes); put(CTR_EXACT, s_exact);
        put(CTR_ROUNDS, s_rounds); put(CTR_RF_OVER, s_rf); put(CTR_RT_OVER, s_rt); put(CTR_SPILLS, s_spill);
        if (lane <= CTR_SPILLS && v) atomicAdd(&line[lane], (u64)v);
#ifdef PAG_PHASE_TIMERS
        if (lane == 0)
            for (int i = 0; i < 6; ++i) atomicAdd(&line[CTR_PHASE0 + i], s_phase[i]);
#endif
    }
};

// Waves per SIMD that the registers have to leave room for.
// Short rows: four (five where a row takes one chunk of fp32 or 8-byte chunks), at up to 21 dwords of spill (up to 56 with
// 16-byte chunks of 16-bit rows).  Working sets above 128 nodes hold W in 4 NW registers per lane: three up to 512 nodes, two
// for 1024 (a third wave there spills W and costs 50 %).
// Long rows: left to itself the compiler keeps the two rows in flight in as many registers as it likes and gives up a wave for
// them; with the line stated it spills at most 24 dwords.  Kernel times with and without, 1,030 to 8,000 queries: 3072-d at
// K 200 5.16 -> 3.53 ms, 2560-d at K 400 1.4-1.5 times as fast, 16-bit rows of 1280 1.0-1.47 times, of 2816 at K 400 1.2-1.6.
// Up to one wave per SIMD it costs fp32 rows of 3072 5 % (900 queries, efS 512: 4.48 -> 4.73 ms; masked early 4.94).
constexpr int pag_search_occupancy(int nq, int nw, int vm, int cw) {
    if (nq <= 4) {
        if (nw > 2) return nw >= 16 ? 2 : 3;
        return nq > 3 ? 1 : (vm == 2 || (nq == 1 && vm == 0)) ? 5 : 4;
    }
    if (nw > 2) return nw >= 16 || (nw == 8 && nq == 12 && vm == 0) ? 1 : 2;
    if (vm == 2) return nq == 8 || (nq == 12 && cw == 8) ? 2 : 3;      // two rows to a buffer at eight chunks
    return vm == 0 && (nq == 6 || (nq == 8 && nw == 2)) ? 3 : 2;
}

// Persistent waves: every wave begins with the query of its own number, if all are resident at once, and pulls further ones from one
// counter until the batch is drained, so long and short searches balance themselves; the loop ends for every wave once the counter passes nq.
template <int NQ, int NW, int VM, int CW>
__attribute__((amdgpu_waves_per_eu(pag_search_occupancy(NQ, NW, VM, CW), 8)))
__global__ void __launch_bounds__(64) k_search(const SearchArgs A) {
    extern __shared__ __align__(64) unsigned char smem[];   // the table sits first: see table_sum
    const int lane = threadIdx.x;
    Wave<NQ, NW, VM, CW> w(A, smem, lane);
    for (u32 qi = A.numbered ? blockIdx.x : w.next_query(); qi < A.nq; qi = w.next_query()) w.run_query(A.order ? A.order[qi] : qi);
    w.flush_stats();
}

// The same with several waves per query, for batches that would leave the GPU mostly idle.
// Registers: 128 a lane, four waves per SIMD, where the rows in flight, the query and W allow it: working sets of up to 128 nodes with fp32
// rows spill none of them, 16-bit ones up to 4, with six 8-byte chunks 22; 129 to 256 nodes 14 to 36, at their ends of rounds above all.
// With 168 there, rows of 128-d to 1024-d and 16-bit ones to 2048, K 150 and 200: up to one query a CU 1.00 to 0.97 of the time, 700 queries 1.00 to
// 0.92, but up to two a CU 1.12 to 1.23 of it (teams of four instead of eight), 1,000 queries 1.33 to 1.74 (one wave each).  Else the 168 that twelve waves
// leave: none or 2 spilled, 16-bit rows in six 16-byte chunks 39, of 3072 42 (with 128 every wave felt it: one query per CU 1.17 times
// as fast as one wave, 1.35 with 168, two per CU 0.85), working sets of 257 to 512 nodes 38 to 93.
template <int NQ, int NW, int VM>
__attribute__((amdgpu_waves_per_eu(NW <= 4 && (NQ <= 4 || (NW <= 2 && NQ == 6 && VM != 1)) ? 4 : 2, 8)))
__global__ void __launch_bounds__(64 * pag_team_max(NW)) k_search_team(const SearchArgs A) {
    extern __shared__ __align__(64) unsigned char smem[];
    Wave<NQ, NW, VM, PAG_MAX_CW, true> w(A, smem, (int)(threadIdx.x & 63), (int)uniform(threadIdx.x >> 6), (int)(blockDim.x >> 6));
    typedef decltype(w) Wv;
    if (w.wave == 0) {
        if (w.split()) w.template run_team<Wv::LISTS>();
        else w.template run_team<Wv::LISTS_FEW>();
        w.flush_stats();
    } else if (w.wave == 1) {
        w.template run_team<Wv::SEEN>();
        w.flush_stats();
    } else if (w.split()) {
        if (w.wave == 2) w.template run_team<Wv::ESTIMATES>();
        else w.template run_team<Wv::ROWS_AHEAD>();
    } else {
        w.template run_team<Wv::ROWS>();
    }
}

}  // namespace pagk

// Which ways of reading the store occur with NQ chunks per lane: 16-bit rows are read in 8-byte chunks where their number
// of 256-element chunk rows is odd, else in 16-byte chunks of 512 elements, of which 3,072 elements need six.
constexpr bool pag_search_reached(int nq, int vm) { return vm == 0 || (vm == 1 ? nq <= 6 : nq != 2 && nq != 4); }

// One translation unit per (NQ, CW) defines the selector below: the kernels for every number of
// W / R_L entries per lane (working sets of up to 64, 128, 256, 512, 1024 nodes) and the three ways of reading the store.
typedef void (*pag_search_fn)(const SearchArgs);
#define PAG_SEARCH_INSTANCES(NQ, CW)                                                                  \
    template <int VM>                                                                                 \
    static pag_search_fn pag_search_by_nw(int nw) {                                                   \
        switch (nw) {                                                                                 \
            case 1: return (pag_search_fn)pagk::k_search<NQ, 1, VM, CW>;                              \
            case 2: return (pag_search_fn)pagk::k_search<NQ, 2, VM, CW>;                              \
            case 4: return (pag_search_fn)pagk::k_search<NQ, 4, VM, CW>;                              \
            case 8: return (pag_search_fn)pagk::k_search<NQ, 8, VM, CW>;                              \
            case 16: return (pag_search_fn)pagk::k_search<NQ, 16, VM, CW>;                            \
            default: return nullptr;                                                                  \
        }                                                                                             \
    }                                                                                                 \
    pag_search_fn pag_search_fn_nq##NQ##_cw##CW(int nw, int vm) {                                     \
        if (vm == 0) return pag_search_by_nw<0>(nw);                                                  \
        if constexpr (pag_search_reached(NQ, 1)) { if (vm == 1) return pag_search_by_nw<1>(nw); }     \
        if constexpr (pag_search_reached(NQ, 2)) { if (vm == 2) return pag_search_by_nw<2>(nw); }     \
        return nullptr;                                                                               \
    }
// the same for the kernels with several waves per query (one translation unit per NQ)
#define PAG_SEARCH_TEAM_INSTANCES(NQ)                                                                 \
    template <int VM>                                                                                 \
    static pag_search_fn pag_search_by_nw(int nw) {                                                   \
        switch (nw) {                                                                                 \
            case 1: return (pag_search_fn)pagk::k_search_team<NQ, 1, VM>;                             \
            case 2: return (pag_search_fn)pagk::k_search_team<NQ, 2, VM>;                             \
            case 4: return (pag_search_fn)pagk::k_search_team<NQ, 4, VM>;                             \
            case 8: return (pag_search_fn)pagk::k_search_team<NQ, 8, VM>;                             \
            case 16: return (pag_search_fn)pagk::k_search_team<NQ, 16, VM>;                           \
            default: return nullptr;                                                                  \
        }                                                                                             \
    }                                                                                                 \
    pag_search_fn pag_search_team_fn_nq##NQ(int nw, int vm) {                                         \
        if (vm == 0) return pag_search_by_nw<0>(nw);                                                  \
        if constexpr (pag_search_reached(NQ, 1)) { if (vm == 1) return pag_search_by_nw<1>(nw); }     \
        if constexpr (pag_search_reached(NQ, 2)) { if (vm == 2) return pag_search_by_nw<2>(nw); }     \
        return nullptr;                                                                               \
    }
