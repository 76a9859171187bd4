// Which variant of a kernel runs and how the work is split: rules on sizes, modes and the number of SIMDs alone, in plain
// C++, so that they can be compiled and checked without a GPU.
#pragma once
#include <algorithm>
#include <stdint.h>

typedef uint64_t u64;
typedef uint32_t u32;

#define GT_TP 21                             // lanes of a party in a wavefront (the wavefront model)
#define GT_INFER_LANES(NW) ((NW) * GT_TP)
#define GT_INFER_OCT(NW) (4 * (NW))          // groups of a workgroup of k_infer at most: 13 KB of LDS per wavefront, 16 with thresholds, two per SIMD (at most 20)
#define GT_AHEAD_OCT(NQ) (4 * (NQ))          // groups of a tile of k_infer_ahead at most: 39 KB of LDS per NQ, 155 KB on a compute unit
#define GT_XY_COLS 5                         // adjacent product columns of a wavefront's step of k_xy
#define GT_XY_FEAT 32                        // features of a workgroup of k_xy at most
#define GT_YROWS 16                          // rows of the class columns' tiles where they have their own: GT_MAX_K
enum { GM_STORE = 0, GM_COMMON = 1, GM_ROWS = 2 };      // modes of the equality grid, see k_eqgrid

// Column ranges per tile of an equality grid.  A wavefront per item (tile, range); every range
// replays the row's part, which costs as much as 2.5 steps (3 PRF blocks, the opening, the atomic
// adds).  Items that fill the two wavefronts per SIMD a whole number of times leave no nearly empty
// last wave; a SIMD with one wavefront takes 0.6 of the time of one with two.  Measured with 1, 3,
// 5, 6 ranges for 200,003 rows x 100 columns: 446, 309, 287, 285 us; with 7, 14, 21, 28 ranges for
// 48,842 rows x 294 columns of their own: 199, 199, 203, 221 us.
// Inner products (sums: how many, 0: none): more than one range costs the launch that completes the sums, against one range, whose
// wavefronts, alone on a SIMD, take 0.82 of the time of two with paired additions (the sums of many short ranges meet at the same words,
// which is why 0.6 is the better line there: 445 rows x 669 columns 29 us in 341 ranges, 51 in 683).  140,244 rows x 32 columns: 92
// in one, 61 and 11 in two; x 8 columns 31 in one, 22 and 11 in two.  Two columns in one range and in two, with that launch: 13 rows 12.2
// and 12.2 us, 30,000 rows 13.2 and 14.6 (three columns: 15.5 either way, 45,753 rows 16.4 in one, 17.4 in three); of their own (fetched meanwhile) 13 rows 1.3 us less in two, 3,000 rows 1.4, 10,000 0.7, 30,000 0.9
// more; two sums, 13 to 20,000 rows 3 to 3.5 us less in two (one range completes the sums of eight rows per lane), 30,000 0.9
// less, 60,000 3.7 more.
// Wavefronts per SIMD: two, or three of 168 registers with the rows' opened values in LDS (shared arrays and the leaf one-hot; own rows gain
// nothing by it).  Three take 1.37 of the time of two for a step of each, two of them 1.05, one 0.66, and the row's part 3.3 steps: 1,000,000 x 64
// 593 us and 533; 200,003 x 100 in 5 ranges 213 and 196, 48,842 x 64 in the 7 ranges that fill two per SIMD 46.5 and 50.2, in ten 62.5 and 49.3;
// 89,221 x 28 in 3 and 5 ranges 49.1 and 50.5.  Half a step more whatever the length, which decides where little else differs: 49,820 x 49, 6 and 10
// ranges 41.2 and 43.5, 100,666 x 25, 3 and 5 43.7 and 46.4, 127,049 x 18, 2 and 4 45.7 and 47.7, but 25,221 x 390, 13 and 20 101.5 and 98.6.  More than 32 ranges only of
// 22 columns on, where the sums' atomic adds count less: 8,477 x 733 in 40 and 60 ranges 72 and 77, 4,061 x 939 in 81 and 118 58 and 68, 9,027 x 1,044, 36 and 55
// (of 19) 99 and 103, 9,993 x 1,159, 34 and 51 (of 23) 116 and 112, 12,735 x 1,463, 26 and 40 180 and 166, 5,980 x 2,920, 56 and 84 168 and 159; and at most
// 100: 3,152 x 3,492, 106 and 159 (of 22) 113 either way.
struct ColumnRanges { u64 n; u32 waves; };
static inline ColumnRanges column_ranges(u64 simds, int mode, int sums, u64 ntile, u64 nsteps)
{
    // in units of a step of two wavefronts, 3 us
    const double launch = sums == 0 ? 0.0 : sums == 2 ? 0.5 + 0.006 * (double)ntile : (mode == GM_ROWS ? 1.2 : 1.6) + 0.003 * (double)ntile;
    ColumnRanges best = { 1, 2 };
    double best_cost = 0;
    for (u32 waves = 2; waves <= (mode == GM_ROWS || sums == 2 ? 2 : 3); waves++) {
        const u64 fills2[] = { 0, 1, 2, 4, 6, 8 }, fills3[] = { 0, 3, 6, 9, 12 };   // wavefronts per SIMD; 0: one range
        for (u32 i = 0; i < (waves == 2 ? 6u : 5u); i++) {
            const u64 f = waves == 2 ? fills2[i] : fills3[i];
            u64 n = std::min<u64>(nsteps, std::max<u64>(1, f * simds / ntile));
            const u64 len = (nsteps + n - 1) / n;
            n = (nsteps + len - 1) / len;
            const u64 items = ntile * n, full = items / (waves * simds), rest = items % (waves * simds);
            if (waves == 3 && (items <= 2 * simds || (n > 32 && (len < 22 || n > 100)))) continue;
            const double last = rest == 0 ? 0.0 : waves == 2 ? (rest > simds ? 1.0 : n == 1 && sums ? 0.82 : 0.6)
                                : rest > 2 * simds ? 1.37 : rest > simds ? 1.05 : 0.66;
            const double cost = ((waves == 2 ? 1.0 : 1.37) * (double)full + last) * ((double)len + (waves == 2 ? 2.5 : 3.3)) + (n > 1 ? launch : 0.0) + (waves == 2 ? 0.0 : 0.5);
            if (best_cost == 0 || cost < best_cost) { best_cost = cost; best = { n, waves }; }
        }
    }
    return best;
}

// Split of an equality grid: gpt groups of 8 samples x rps adjacent columns per step and wavefront, ntile tiles, nkc ranges of
// kchunk columns each.  alone: the variant without issue priorities (see chacha8).  sums: GM_STORE writes the tiles of the sums, too.
// waves: wavefronts per SIMD that the variant's registers are cut for.
struct GridShape { u32 rps, gpt, kchunk, nkc; u64 ntile; bool alone; u32 waves; };
static inline GridShape grid_shape(u64 simds, int mode, int ndot, bool sums, u32 w, u64 N8)
{
    GridShape s;
    // A wavefront covers 21 groups of 8 samples of one column per step.  The leaf one-hot grid takes
    // four groups (the 32 samples of a sample block) of five adjacent columns, eight of two (at most three
    // columns) or twenty of one: the 32-byte pieces that it stores per limb then lie side by side.
    s.rps = mode != GM_STORE || w == 1 ? 1 : (w <= 3 ? 2 : 5);
    s.gpt = s.rps == 1 ? (mode == GM_STORE ? 20 : GT_TP) : (s.rps == 2 ? 8 : 4);
    const u64 nsteps = ((u64)w + s.rps - 1) / s.rps;
    s.ntile = (N8 / 8 + s.gpt - 1) / s.gpt;
    const ColumnRanges ranges = column_ranges(simds, mode, mode == GM_STORE ? 0 : ndot, s.ntile, nsteps);
    const u64 nkc = ranges.n;
    s.kchunk = (u32)(((nsteps + nkc - 1) / nkc) * s.rps);
    s.nkc = (u32)(((u64)w + s.kchunk - 1) / s.kchunk);
    // wavefronts that have their SIMD to themselves, or a single step per item (1.5 * 10^6 rows x 1 column: 76 us, 83 with
    // priorities); inner products over up to three columns whose last wavefronts are alone (360,000 rows, 2,143 tiles, x 2, 3, 6 columns: 31,
    // 37, 54 us, 35, 40, 54 with them; 534,134 rows, 3,180 tiles: 40, 47, 70 and 40, 45, 60); and the grid that writes a level's tiles and their sums for many samples: what it gains by priorities the
    // contraction behind it loses, which reads tiles that were written in a different order.  Grid + contraction without and with them, 16, 32,
    // 64 nodes: 60,000 samples x 122 columns 37 + 78, 54 + 78, 86 + 109 us and 32 + 78, 46 + 79, 73 + 113; 140,244: 75 + 182, 113 + 195,
    // 190 + 273 and 73 + 195, 110 + 213, 187 + 298; 400,000: 173 + 500, 281 + 531, 493 + 659 and 161 + 519, 271 + 553, 493 + 663.
    // These run with two wavefronts per SIMD, whichever the ranges were priced for: without priorities three gain nothing (the level's grid of 10^6 samples x 64
    // nodes 2.45 ms with two, 2.50 with three).  Their ranges stay as priced: 135,000 samples x 128 and 256 nodes 284 and 543 us in one, 218 and 406 in two.
    const u64 items = s.ntile * s.nkc, rest = items % (2 * simds);
    s.alone = items <= simds || s.kchunk <= s.rps || (mode != GM_STORE && s.kchunk <= 3 && items > 2 * simds && rest && rest <= simds) || (sums && N8 > 131072);
    s.waves = s.alone ? 2 : ranges.waves;
    return s;
}

// Up to eight nodes all columns run on the narrow tiles, where x holds the columns: every component of a column is then
// fetched once for the three parties, and no row is padding but those below 8.  48,842 x 590 columns with 1, 2, 4, 8 nodes:
// 215, 199, 198, 204 us on the wide tiles, 172, 135, 139, 150 on the narrow ones; 50,000 x 34: 33 and 31-32; with 16 nodes, two narrow
// tiles, 205 and 260.  Not with few samples and many columns, where the adds of a tile's sums count (a wide tile adds 64 columns
// at a time): 8 nodes, 500 samples x 2,408 columns 15 and 18 us, x 8,002 42 and 56; 1,500 x 2,408 27 and 29; beyond the line,
// 2,100 samples: x 2,408 36 and 37, x 8,002 121 and 115; 3,000 x 2,408 44 and 44.
// xcols: x holds the columns (CountArgs); nh nodes, nblk blocks of 32 samples, ncol columns.
static inline bool count_few(bool xcols, u64 nh, u64 nblk, u64 ncol) { return xcols && nh <= 8 && (nblk > 64 || ncol <= 64); }

// Whether a level's one-hot of split decisions (partition by products: np nodes before it, d features) is written as limb bytes by the launch
// that tests, a line per byte, or as words that a second launch turns into limbs.  d, np*d: one launch, the two: 20, 10,240 9.0 and 9.9 us, 20,480 16.7 and
// 10.9; 30, 15,360 10.0 and 10.4; 64, 16,384 8.4 and 10.2, 32,768 12.8 and 11.6; 300, 9,600 5.9 and 10.1, 38,400 15.2 and 11.4, 307,200 86 and 38; few
// nodes write few bytes of a line: 2,000, 32,000 9.7 and 11.6, 64,000 14.1 and 13.3; 4,000, 32,000 10.8 and 12.6; but 10,000, 10,000 18.0 and 16.7.
static inline bool onehot_bytes(u64 simds, u64 np, u64 d) { return np * d <= (np <= 16 ? 32 : 16) * simds && d <= 4096; }

// Whether a level's node split (n words) loads its words before the block function instead of after it.  On a full chip the registers
// count more: 249,856 words 18.7 us with the loads after it, 20.0 before, 604,160 46.4 and 55.1, but 156,672 14.4 and 13.3.  So do the copies that the
// same launch makes of the same words, where the columns' tiles that the level has read (tile_bytes) leave nothing of them in the 256 MB of the last-level
// cache: 48,842 samples x 306 columns (450 MB), 612 to 78,336 words 11.4 to 13.2 and 12.3 to 14.1; 5,000 samples (46 MB) 10.3 to 12.2 and 10.1 to 11.8.
static inline bool split_early(u64 n, u64 tile_bytes) { return n <= 163840 && tile_bytes <= (u64)256 << 20; }

// Whether equality tests of n elements take tiles of 40, see k_eq_pair: from as many of these on as there are SIMDs (both sides there).
static inline bool eq_pairs(u64 simds, u64 n) { return n >= 40 * simds; }

// Rows of a training's tiles (nodes of the level before the last, columns, a multiple of 32 and of 64) and whether the columns are kept once per component, with the
// sums own + next on the nodes: whichever way needs less memory, and with it traffic.
struct TileRows { u64 nodes, cols; bool comps; };
static inline TileRows tile_rows(u32 H, u64 ncol)
{
    TileRows r;
    r.cols = (ncol + 63) / 64 * 64 + 64;
    r.nodes = H ? std::max<u64>(32, (((u64)1 << H) / 2 + 31) / 32 * 32) : 0;
    r.comps = 3 * r.nodes + 3 * r.cols + 6 * GT_YROWS <= 6 * r.cols;
    return r;
}

// k_xy: features in equal parts of at most 32 (whole rows of 256 bytes), tk each; more parts where the blocks of 32 samples are few, down to a step for each wavefront
// (267 x 22: 11 us in three parts, 13 in one; 10^6 x 64 in parts of 16 2.97 ms, of 32 2.49).  items: a block x a part, groups: workgroups.
struct XySplit { u32 tk; u64 items, groups; };
static inline XySplit xy_split(u64 simds, u64 N8, u32 d, u32 K)
{
    XySplit s;
    const u64 blocks = (N8 / 8 + 3) / 4, cus = std::max<u64>(1, simds / 4);
    const u32 parts = (u32)std::max<u64>((d + GT_XY_FEAT - 1) / GT_XY_FEAT, std::min<u64>(((u64)d * K + 4 * GT_XY_COLS - 1) / (4 * GT_XY_COLS), cus / blocks));
    s.tk = (d + parts - 1) / parts;
    s.items = blocks * ((d + s.tk - 1) / s.tk);
    s.groups = std::min<u64>(s.items, 3 * cus);
    return s;
}

// Kernel and tile of an inference: the 21 lanes of a party per wavefront (pair of wavefronts, k_infer_ahead) are split into noct
// groups of 8 instances x ncol columns per step.  Where all tiles are on the chip at once: k_infer_ahead with 84, 42 or
// 21 lanes per party.  Otherwise k_infer in workgroups of one wavefront with at most four groups: a wavefront waits for no
// other one, and its loads touch the lines of at most 32 rows of instances at a time (50,000 instances of 20 features,
// depth 6, thresholds: 405 us in workgroups of four, 308 in single ones; 50,000 x 294, depth 6: 2.74 and 1.64 ms (1.42 since a component is read once); 16 trees of
// depth 5 on 5,003 x 30: 570 and 437 us); of two or four for some tiles that the caller asks for.
// simds: of the device; lgi: log2 of the instances per workgroup that the caller asks for, 0: none; ngrp: groups of 8 instances.
// The cost, in steps of k_infer on a full SIMD.  k_infer: an access costs 2.4 beside its steps (PRF blocks of its own, the
// opening, the sums), a comparison 0.4 and 0.4 for every instance of a group that a lane takes; a wavefront alone on its
// SIMD takes 0.84 of the time of two; and where the rows of all groups at work exceed the L2s, a step of few columns waits for
// lines that it had before.  k_infer_ahead: 3.6 for a launch, 0.1 and 0.1 more for every 21 lanes an access (barriers), 0.32 a
// step, 0.41 with thresholds, 0.27 for every instance of a half group that a lane compares; all but the launch times
// 2.2 where the chip is full.  Fitted to 53 batches and forests of 1 to 700,000 instances while k_infer read six planes and held the rows' opened
// values; of 22 batches of k_infer as it is, this picks within 1 % of the best of all shapes on average, 7 % at worst (300,000 x 8, depth 12: 4 groups are faster).
struct InferShape { u32 nq, nw, noct; };                // nq: k_infer_ahead<., nq>; else nw wavefronts of k_infer
// whether single wavefronts of k_infer add up their sums through LDS, see group_sums
static inline bool staged_sums(u32 noct, bool has_thr) { return noct == 1 && !has_thr; }
static inline InferShape infer_shape(u64 simds, u32 lgi, u64 ngrp, u32 ntrees, u32 H, u32 d, bool has_thr)
{
    InferShape best = { 0, 1, 1 };
    double best_cost = 0;
    const auto steps = [&](u64 ncol) {
        u64 n = H * ((d + ncol - 1) / ncol);
        for (u32 h = 0; h <= H; h++) n += (((u64)1 << h) + ncol - 1) / ncol;
        return (double)n;
    };
    const auto forced = [&](u32 noct) { return !lgi || noct == (1u << lgi) / 8; };
    const auto take = [&](u32 nq, u32 nw, u32 noct, double cost) { if (best_cost == 0 || cost < best_cost) { best_cost = cost; best = { nq, nw, noct }; } };
    for (u32 nq = 4; nq >= 1; nq /= 2)
        for (u32 noct = 1; noct <= GT_AHEAD_OCT(nq); noct++) {
            const u64 items = (ngrp + noct - 1) / noct * ntrees, ncol = GT_INFER_LANES(nq) / noct;
            if (!forced(noct) || items > simds / nq) continue;
            const double chain = (0.11 + 0.093 * nq) * (2 * H + 1) + (has_thr ? 0.41 : 0.32) * steps(ncol) + (has_thr ? 0.27 * (double)(H * ((4 + ncol - 1) / ncol)) : 0.0);
            take(nq, 0, noct, 3.6 + chain * (1.0 + 1.17 * (double)(items * nq) / (double)simds));
        }
    // a lone label: k_infer's start and end count beside its one access, which its cost above leaves out (137, 2,699, 12,110 instances
    // 11.4, 12.5, 13.6 us; k_infer_ahead 8.6, 8.7, 9.6)
    if (H == 0 && best.nq) return best;
    // A tile that the caller asks for: the fewest wavefronts whose steps do not fetch the rows' 128-byte lines more than twice,
    // unless the rows stay in the L2s or are of less than 48 columns (300,000 x 150, depth 4, tiles of 32: 4.2 ms with one, 3.8 with four; tiles of
    // 64: 5.8 with two; but 208,758 x 30, depth 3: 522 us with one, 595 with two, 1,052 with four; of depth 12, where the tree's
    // steps divide by the wavefronts as well, 20.3 ms with one, 18.5 with two), and of rows of 250 columns on at least 21 a step once
    // the wavefronts fill the chip (208,758 x 373, depth 3, tiles of 32: 4.14 ms with 10, two wavefronts, 3.79 with 21, four; of 16: 3.65 and 3.45,
    // thresholds 4.12 and 3.64; of 200 columns 2.23 and 2.30, 1.99 and 2.02; 25,000 x 300, 782 tiles of 32: 468 us with 10, 484 with 21).
    u32 nw = 1;
    const u32 ask = lgi ? (1u << lgi) / 8 : 0;
    if (ask) {
        const bool in_l2 = ngrp * 8 * d * 24 <= (u64)8 << 20;          // three planes are read; up to 16 MB 40 batches took the same time either way
        const u64 tiles = (ngrp + ask - 1) / ask * ntrees;
        const auto more = [&](u32 ncol) {
            return !in_l2 && (((d >= 48 || H >= 10) && (d + ncol - 1) / ncol > 2 * ((d + 15) / 16)) || (d >= 250 && ncol < GT_TP && tiles * nw > 2 * simds));
        };
        while (nw < 4 && (ask > GT_INFER_OCT(nw) || more(GT_INFER_LANES(nw) / ask))) nw *= 2;
    }
    for (u32 noct = 1; noct <= GT_INFER_OCT(nw); noct++) {
        if (!forced(noct)) continue;
        const u64 items = (ngrp + noct - 1) / noct * ntrees, ncol = GT_INFER_LANES(nw) / noct;
        double units = 2.4 * (2 * H + 1) + steps(ncol) + (has_thr ? H * (0.4 + 0.4 * (double)((8 + ncol - 1) / ncol)) : 0.0);
        const double at_work = std::min(8.0 * noct, 4.0 * (double)(items * noct) / (double)simds);    // groups per compute unit
        if (d > 16 && ncol < 16 && at_work > 18.0) units += 0.27 * H * (double)((d + ncol - 1) / ncol);
        const u64 waves = items * nw, full = waves / (2 * simds), rest = waves % (2 * simds);
        const double last = rest == 0 ? 0.0 : rest <= simds ? 0.84 : full ? 0.84 + 0.16 * (double)(rest - simds) / (double)simds : 1.0;
        take(0, nw, noct, units * ((double)full + last));
    }
    return best;
}
