// Which plan a search gets: arithmetic on sizes, without HIP, so that it can be checked on a CPU.
#pragma once

#include <stdint.h>

#include <algorithm>

// How many queries the GPU holds, from the workgroups of `waves` waves that the occupancy query grants a CU.  A single wave is
// launched whatever the answer, a team only if it fits.
inline int pag_resident(int per_cu, int num_cu, uint32_t waves) { return std::max(per_cu, waves == 1 ? 1 : 0) * num_cu; }

struct pag_team_request {
    uint64_t nq;             // queries of the call
    uint64_t others;         // queries of other calls that the GPU searches beside them, see pag_queries_beside
    uint32_t b, ef;
    uint32_t num_cu, lds_per_cu;
    uint32_t hlog, blog;     // the seen set of the one-wave search
    uint32_t seen_fixed;     // its size is the caller's choice
    uint32_t most_waves;     // that the kernel is built for
};

struct pag_team_plan {
    uint32_t waves;          // 1: no team
    uint32_t hlog, blog;     // of the team's seen set
    uint32_t lds;            // bytes
};

// Of `calls` other calls under way with `queries` queries in all, how many are searched side by side with a new one: HIP gives a
// process four hardware queues, what is beyond waits.  (Eight searchers with 64 queries each, 200k x 768, efS 256: 247,000
// queries/s when all seven others count, 276,000 when three do.)
inline uint64_t pag_queries_beside(uint64_t calls, uint64_t queries) { return calls <= 3 ? queries : queries * 3 / calls; }

// A team of `most` waves, or of as many less in steps of `step` as leave every query resident where `share` queries share a CU, but not of less
// than four; `waves` stays as it is if there is no such team.
template <class Lds, class Resident>
int pag_fit_team(const pag_team_request& r, uint32_t share, uint32_t most, uint32_t step, Lds&& lds_bytes, Resident&& resident, pag_team_plan* p) {
    const uint64_t load = r.nq + r.others;
    const uint32_t length = std::max(r.ef, r.b);                    // nodes that a search expands, about
    const uint32_t room = r.lds_per_cu / share - 512;
    // The seen set: an exact hash of everything the search is expected to compute, if the LDS holds it half full;
    // otherwise the bitmap behind a Bloom filter of 16 bits per node, as far as the LDS goes.
    uint32_t hlog = r.hlog, blog = r.blog;
    const uint64_t expected = r.b + 8ull * length;
    uint32_t lg = 9;
    while ((1ull << lg) < 2 * expected && lg < 16) ++lg;
    if (!r.seen_fixed && (1ull << lg) >= 2 * expected && lds_bytes(lg, 0u) <= room) {
        hlog = lg; blog = 0;
    } else if (blog) {
        while (blog < 20 && (1ull << blog) < 16 * expected && lds_bytes(hlog, blog + 1) <= room) ++blog;
    }
    const uint32_t lds = lds_bytes(hlog, blog);
    if (lds > room) return 0;
    // as many waves as leave every query resident
    for (uint32_t waves = most; waves >= 4; waves -= step) {
        int rc, n = 0;
        if ((rc = resident(waves, lds, &n))) return rc;
        if ((uint64_t)n < load) continue;
        p->waves = waves; p->hlog = hlog; p->blog = blog; p->lds = lds;
        return 0;
    }
    return 0;
}

// Batches that leave the GPU mostly idle with one wave per query get several (a team); `share` queries then share a CU.
// `waves` stays 1 where one wave is the better plan.
//   lds_bytes(hlog, blog): LDS of a team with that seen set; resident(waves, lds, &n): error code, teams that the GPU holds at a time
//
// What decides is not the call alone but the queries under way on the GPU: a team takes a large part of a CU, and teams of
// several calls would wait for each other where smaller teams or single waves run side by side.  Four searchers with 256 queries
// each (200k x 768, efS 256): 302,000 queries/s when every call plans as if it were alone, 482,000 with one wave per query,
// 661,000 with what the sum asks for; with 1,000 queries each 706,000, 1,158,000 and 1,186,000, with 16 each 73,000, 39,000 and 73,000.
//
// The shortest searches gain like all others (whole calls of 10 nodes with one wave -> a team; one query: 5k x 32 68 -> 48 us, 5k x 128
// 88 -> 57, 50k x 768 91 -> 55, 12k x 3072 159 -> 99; 256 queries: 90 -> 60, 96 -> 63, 176 -> 98, 323 -> 234; 512: 91 -> 61, 97 -> 65, 199 -> 124).
// The lines, with kernel times of one wave -> a team (100,000 rows, efS 128, unless stated) as they were when the lines were drawn:
//   one query per CU: up to 12 waves.  128-d 474 -> 310 us, 768-d 650 -> 365, 3072-d 1068 -> 605 (256 queries); a single
//     query 375 -> 242, 491 -> 271, 777 -> 414
//   two per CU: 8 waves, where the registers of the kernel allow 16 on a CU.  128-d 508 -> 401 us, 768-d 704 -> 492,
//     1536-d 995 -> 747 (512 queries).  Where they allow twelve, teams of four, of which three fit: two teams of six are granted but
//     run one after the other.  Whole calls with one wave / six / four, 512 queries: 3072-d at efS 128 1183 / 1363 / 1051 us, at efS 512 3348 /
//     4048 / 2930, K 200 2993 / 3974 / 2614, 16-bit 1267 / 1404 / 997, 3528 / 4105 / 2717, 3113 / 4472 / 2583; K 400 of 50k x 768 4367 /
//     5271 / 3108, K 200 and 400 of 20k x 1536 2482 / 2994 / 1840, 4822 / 5682 / 3420 (all with W unsorted above 128 nodes).  Working sets of 129 to 256
//     nodes with rows of up to four chunks allow sixteen: four -> eight, W sorted, 512 queries of 50k x 128 / 768 / 1024, K 150, efS 600 1470 -> 1247,
//     1644 -> 1440, 1858 -> 1565, K 200, efS 800 1875 -> 1588, 2067 -> 1813, 2329 -> 1955, 16-bit 768 and 30k x 2048 1.16 to 1.23 times as
//     fast.  Where they allow eight (working sets above 512), four, too:
//     K 600 and 1000 of 50k x 768 6883 -> 5523, 10696 -> 8595
//   up to four per CU: 4 waves, where the registers of the kernel let every query be resident (all four of short rows and working sets
//     of up to 256 nodes, three of long rows and of up to 512, none above).  Whole calls with one wave -> four, working sets of 129 to 256 nodes,
//     1,000 queries, K 150, efS 600 / K 200, efS 800: 50k x 128 2414 -> 1817, 3141 -> 2287 us, 768 3170 -> 2106, 4110 -> 2621, 1024 3391 -> 2460, 4360 ->
//     3034, 16-bit 768 3312 -> 2150, 4298 -> 2696, 30k x 2048 4957 -> 3173, 6292 -> 3930; smaller ones: 1,024 queries of
//     5k x 32 / 128 at efS 10 91 -> 72, 102 -> 74 us, 50k x 768 at efS 10 / 24 247 -> 178, 345 -> 307, 16-bit 244 -> 180, 380 -> 318, 20k x
//     1536 345 -> 280, 471 -> 386; 768 queries of 50k x 768 at efS 128 / 512 755 -> 485, 2523 -> 1563, K 300 3431 -> 2736, of 12k x 3072
//     at efS 16 / 512 670 -> 642, 3729 -> 3568, K 400 5897 -> 5144, 16-bit 669 -> 593, 3718 -> 3017, 5917 -> 5126.  Small graphs, 1,024 queries: 120 x 128
//     at efS 10 / 64 68 -> 58, 166 -> 137, K 100 182 either way; 500 x 768 at efS 10 / 128 146 -> 122, 480 -> 340
template <class Lds, class Resident>
int pag_plan_team(const pag_team_request& r, Lds&& lds_bytes, Resident&& resident, pag_team_plan* p) {
    const uint64_t cus = r.num_cu, load = r.nq + r.others;
    uint32_t share, most, step;
    p->waves = 1;
    if (load <= cus) {
        share = 1; most = 12; step = 1;
    } else if (load <= 2 * cus) {
        share = 2; most = 8; step = 4;
    } else if (load <= 4 * cus) {
        share = 4; most = 4; step = 4;
    } else {
        return 0;
    }
    return pag_fit_team(r, share, std::min(most, r.most_waves), step, lds_bytes, resident, p);
}

// The largest batch of new nodes whose RobustPrune has four waves per node, for rows of `chunks` 16-byte chunks a lane (1, 2, 3, 4, 6, 8, 12).
// Four waves finish a node sooner and keep more of its rows on the chip; one wave per node leaves the CU to more nodes, which counts
// where their rows come from HBM and their candidates are few to a kept row.  Prune phase of whole builds, one wave -> four:
//   up to 768-d any batch gains.  100,000 rows in batches of 2,048 / 16,384: 128-d 22.4 -> 17.4, 15.2 -> 13.6 ms, 768-d 34.9 -> 25.2, 22.1 ->
//     19.1; 300,000 in 16,384: 256-d, degree 64 21.3 -> 18.3 (65,536: 18.6 -> 17.1), 512-d 45.8 -> 41.5, 768-d, degree 16 / 64 34.0 -> 30.2,
//     74.9 -> 63.6; 1M in 16,384: 128-d 59.7 -> 56.7, 768-d 357 -> 341
//   1024-d up to 32 nodes a CU.  300,000 rows, degree 48, batches of 4,096 / 8,192 / 16,384: 117 -> 97, 93 -> 86, 81 -> 80, degree 32
//     73.9 -> 72.2 at 8,192, 66.2 -> 68.0 at 16,384; 1M, degree 48, in 16,384: 651 -> 687
//   1280-d and 1536-d up to 8.  300,000 x 1280 in 2,048 / 4,096: 166 -> 147, 119 -> 130; 300,000 x 1536 326 -> 293, 234 -> 256 (16,384: 179 -> 225)
//   2048-d any batch.  200,000 rows in 2,048 / 4,096 / 16,384: 164 -> 129, 127 -> 114, 106 -> 101
//   longer ones up to 3.  100,000 x 2560 in 512 / 1,024: 287 -> 202, 154 -> 171; 200,000 x 3072 in 512 / 768: 588 -> 394, 413 -> 359;
//     30,000 x 3072 in 768 / 1,024: 64 -> 59, 51 -> 57
constexpr uint64_t PAG_ANY_BATCH = ~0ull;
constexpr uint64_t pag_prune_line(uint32_t chunks, uint32_t num_cu) {
    return chunks <= 3 || chunks == 8 ? PAG_ANY_BATCH : (uint64_t)num_cu * (chunks == 4 ? 32 : chunks == 6 ? 8 : 3);
}

// How many workgroups with that LDS a CU really holds.  It is handed out in pieces of 1,280 bytes, which the occupancy query does not
// know: workgroups that only wait, with 11,904 bytes each, run twelve at a time and not thirteen, with 6,144 25 and not 26 (every size
// from 5 to 40 KB).
inline uint32_t pag_lds_room(uint32_t bytes, uint32_t lds_per_cu) { return lds_per_cu / std::max(1280u, (bytes + 1279) / 1280 * 1280); }

// How many of a batch's queries go to the workgroup of their number instead of being taken from a counter, of `groups` workgroups that
// are launched and `sure` that have room at a time.  The counter costs 14 ns a query, done one after the other at the start of a
// batch (4,000 queries of 100,000 x 768, efS 10, all resident: 515 us with it, 459 without).  But a workgroup that finds no place before another one
// ends keeps the query of its number until then, and where the others go on to the rest of the batch that is its end (search phase of
// 200,000 rows built with efC 200 / 100, 13 workgroups of 768-d and 11 of 128-d a CU launched, 12 and 10 held, by number -> by counter: 768-d
// 150 -> 144 / 83 -> 75 ms, 128-d efC 100 59 -> 54; 6,600 queries of 100,000 x 768, K 100, efS 300: 6.34 -> 5.99 ms).  A batch
// without a rest has no such end: a workgroup is done with its one query, and the next has its place.
inline uint64_t pag_numbered(uint64_t nq, uint64_t groups, uint64_t sure) { return groups >= nq || groups <= sure ? groups : 0; }

// Whether a wave of the one-wave search waits for the rows it has asked for before it asks for the next ones.  With the GPU full
// from beginning to end, more long rows in flight only make the waves evict each other's from the memory-side cache.  `room`:
// waves the GPU holds, `waves`: that are launched.  Kernel time without : with, over batches of 4,200 to 10,000 queries and searches
// of 300 to 1,408 nodes: 1M and 60k x 768 1.00 to 1.02 with at least 3/4 of the waves, 0.99 below; 400k x 1024 1.00 to 1.02, 60k and
// 200k x 1536 0.99 to 1.03, 100k x 3072 0.99 to 1.01.  It loses with shorter rows (1M x 128 0.94 to 1.0, 700k x 384 0.97 to 0.99,
// 400k x 640 0.97 to 1.01), 16-bit ones (1M x 768 0.97 to 1.0), larger working sets (1M x 768, K 100: 0.96 to 1.0) and batches of
// one round (0.95 to 1.0).
inline bool pag_paced(uint32_t d, bool half, uint32_t b, uint32_t ef, uint64_t nq, uint64_t waves, uint64_t room) {
    return !half && d >= 768 && b <= 64 && ef >= 256 && nq > room && (d >= 1024 ? 2 * waves >= room : 4 * waves >= 3 * room);
}
