// Run lengths of the 3-D marching kernels: which planes a workgroup walks, by
// grid and by batch.  Host arithmetic only.
#pragma once

#include <algorithm>

#include "../../include/ch.h"

#ifndef CH_WBLK_MAX
#define CH_WBLK_MAX 2048         // most strip workgroups per instance (larger grids loop over strips)
#endif
                                 // <= 8 * CH_BLOCK partials per instance (sum_partials)
#ifndef CH_MARCH_L
#define CH_MARCH_L 16            // planes per run of the 3-D marching matvec
#endif

// Rows (y) of the x-y block of a marching workgroup: 8 in FP64 (two x per
// thread), 16 in FP32 (four x per thread); the block is 64 wide.
constexpr int march_rows(int prec) { return prec == CH_FP64 ? 8 : 16; }

// Planes per z-run of the FP32 DCGS2 matvec: of the lengths CH_MARCH_L ..
// 2 CH_MARCH_L, the one whose work items (64 x 16 blocks times runs) fill the
// largest share of whole rounds of co-resident workgroups, the shorter on
// ties.  The kernel holds three workgroups per CU at its register count, so
// 256 CUs hold 768: at 256^3 runs of 16 give 1024 items (a second round a
// third full), runs of 22 give 768.  Only while every item has a workgroup
// of its own at CH_MARCH_L (at most CH_WBLK_MAX items): beyond that the
// workgroups loop over items, rounds no longer follow the item count, and
// longer runs were slower (384^3, 512^3).
constexpr unsigned MARCH_SLOTS_FP32 = 256u * 3u;

inline int march_len_fp32(int n) {
    const unsigned nxy = (unsigned)((n + 63) / 64) * (unsigned)((n + 15) / 16);
    if ((unsigned long long)nxy * (unsigned)((n + CH_MARCH_L - 1) / CH_MARCH_L) > CH_WBLK_MAX) return CH_MARCH_L;
    int best = CH_MARCH_L;
    unsigned long long bi = 0, br = 1;   // items and rounds of the best length so far
    for (int L = CH_MARCH_L; L <= 2 * CH_MARCH_L; ++L) {
        const unsigned long long items = (unsigned long long)nxy * (unsigned)((n + L - 1) / L);
        const unsigned long long rounds = (items + MARCH_SLOTS_FP32 - 1) / MARCH_SLOTS_FP32;
        if (items * br > bi * rounds) {
            best = L;
            bi = items;
            br = rounds;
        }
    }
    return best;
}

// Planes per z-run of the FP64 kernels (matvec, estimate pass, LIM stage, LIM
// estimate): 16 on large grids, down to 1 where 16 leave CUs without work.  A
// plane step is a chain (a load, two stencil passes, the dot phase, a
// barrier), so a grid that gives a CU one workgroup takes as long as its run:
// 18 steps of about 0.9 us in a LIM stage at L = 16, however small the grid.  More
// workgroups on a CU share its time: a step of w of them takes about
// 0.55 + 0.19 w of these units (w <= 4, the occupancy), so the length that
// minimises L + 4 (the two planes on either side) times that, summed over the
// rounds of workgroups, is taken, the longer on ties (fewer rim planes).
// Measured, EE2 step of dimension 30 with its trace and LIM step of order 19 (37
// stages), L = 16 and the length picked: 32^3 2270 -> 907 us and 733 -> 324
// (L = 1); 97^3 2769 -> 2053 and 743 -> 586 (4); 128^3 4189 -> 3817 and 811 ->
// 704 (4); 160^3 7684 -> 7309 and 1193 -> 1063 (10); 192^3 12280 -> 11883 and
// 1515 -> 1447 (14).  From 2048 workgroups at L = 16 on (256^3) every shorter
// length was slower.  The rule is for a grid alone; batches group runs (march_group).
inline int march_len_fp64(int n) {
    const unsigned nxy = (unsigned)((n + 63) / 64) * (unsigned)((n + 7) / 8);
    int best = CH_MARCH_L;
    unsigned bt = ~0u;
    for (int L = CH_MARCH_L; L >= 1; --L) {
        const unsigned long long items = (unsigned long long)nxy * (unsigned)((n + L - 1) / L);
        if (items > CH_WBLK_MAX) break;   // at CH_MARCH_L: the workgroups loop over items
        const unsigned w = (unsigned)((items + 255) / 256), last = w % 4;
        const unsigned t = (unsigned)(L + 4) * (w / 4 * 131 + (last ? 55 + 19 * last : 0));
        if (t < bt) {
            best = L;
            bt = t;
        }
    }
    return best;
}

inline int march_len(int n, int prec) { return prec == CH_FP64 ? march_len_fp64(n) : march_len_fp32(n); }

// ... and under a launch shape of `wblk` workgroups: the shortest runs from that
// length on that give every workgroup one run, CH_MARCH_L where none does (the workgroups
// then loop over runs, and the short ones cost two planes on either side each:
// 32^3 with 8 workgroups, two steps 1830 us EE2 and 1420 LIM with runs of 16, 2950 and 4090 with runs of 1).
inline int march_len_set(int n, int prec, int wblk) {
    int L = march_len(n, prec);
    if (prec != CH_FP64) return L;
    const long long nxy = (long long)((n + 63) / 64) * ((n + 7) / 8);
    while (L < CH_MARCH_L && nxy * ((n + L - 1) / L) > wblk) ++L;
    return L;
}

// Workgroups of a grid whose workgroups walk `grp` runs each.
inline int march_groups(int n, int zlen, int grp) {
    return ((n + 63) / 64) * ((n + 7) / 8) * (((n + zlen - 1) / zlen + grp - 1) / grp);
}

// x-y blocks of an FP64 grid times its planes.
inline long long march_planes(int n) { return (long long)((n + 63) / 64) * ((n + 7) / 8) * n; }

// Runs that a workgroup of an FP64 batch walks one after the other (1 for a
// grid alone, for which march_len_fp64 is made).  Short runs pay where a grid leaves CUs
// idle; in a batch the other members fill them, and the two planes on either side of
// every run only cost.  planes: march_planes summed over the batch.  As many planes as leave two
// workgroups per CU (512), at most 16 in a LIM table and 8 in an EE2 one, whose runs of four
// and more are left as they are (8 planes against 4: 4 x 97^3 6690 -> 7090 us).
// Two steps, us, runs as of a grid alone and grouped: LIM 64 x 32^3 2886 -> 1555, 300 x 32^3
// 11641 -> 5527, 16 x 64^3 1888 -> 1383, 8 x 128^3 5313 -> 4304, 2 x 32^3 418 (one run);
// EE2 64 x 32^3 5198 -> 4173, 300 x 32^3 22064 -> 16351, 40 x 48^3 6943 -> 6459.
inline int march_group(int n, int zlen, long long planes, bool lim) {
    if (!lim && zlen >= 4) return 1;
    const int want = (int)std::min<long long>(lim ? 16 : 8, planes / 512);
    return std::max(1, std::min(want / zlen, (n + zlen - 1) / zlen));
}
