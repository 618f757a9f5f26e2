// Rules of the fill that are plain arithmetic on sizes.  C++ without HIP, so that the host tests can call them.
#pragma once

namespace ckpt_rules {

// Upper bounds of the block product (stage 1 of gemm_kernel).  A tile has nq middle splits, k = 0 .. nq - 1.  KS slices
// of waves share them, and sixteen lanes of a slice, x = 0 .. 15, fetch the bounds of one split each.  Any splits give a
// valid upper bound; more of them, and better ones, give a tighter one.

// With more splits than this slice 0 asks finished neighbours which splits they took.  The answer is a trip to memory
// before the gather, which tiles of few splits do not pay back.  us a solve with 17, 25, 33, 49 and 65:
//   64 x 96 stages, 2048 slots 3501, 3501, 3508, 3519, 3533;  128 x 96, 1024 slots 3822, 3827, 3815, 3842, 3852
//   8 x 128, 1024 slots 774.4, 773.2, 771.5, 769.8, 768.4;  16 x 48, 1024 slots 211.3, 210.8, 210.1, 210.3, 210.3
constexpr int kAsk = 33;

// The split of a lane that asks nobody, evenly spread over the tile.  Where slice 0 asks, its lanes 12 .. 15 take four places
// and the other slices the rest.  Where nobody asks, all slices share the places: with 16 KS splits and fewer every
// split is taken, and the slices fetch different ones.  (When slice 1 of 2 took the places of slice 0 again: 16 x 48 stages, 1024
// slots 214.0 us and 213.1 so; 8 x 96, 2048 slots 666.7 and 662.8; 10 x 56, 1500 slots 257.5 and 256.1.)
constexpr int spread_split(int x, int slice, int KS, int nq) {
    const int others = KS > 1 ? KS - 1 : 1;
    if (nq <= kAsk) return (2 * (16 * slice + x) + 1) * nq / (32 * KS);
    if (slice > 0) return (2 * (16 * (slice - 1) + x) + 1) * nq / (32 * others);
    return (2 * (x - 12) + 1) * nq / 8;
}

// The split that an asked neighbour took, from the number of its candidate: q + 1 for split q, i + 1 for C_all of row i, 0 for
// none.  Lanes 0 .. 7 ask row qlo, lanes 8 .. 11 the rows above it.  Lanes whose neighbour took none of the tile's splits take one of
// twelve spread places, but C_all of row qlo reads like split qlo, the first of the tile, and is left so: lanes
// that agree gather fewer lines, and with places of their own no batch was faster (8 x 192 stages, 4096 slots 4433 us,
// 4427 with places; 3 x 254, 1500 slots 2075, 2070; 1 x 192, 4096 slots 1134, 1134; 1 x 254, 1500 slots 1646, 1653).
constexpr int asked_split(int x, int number, int qlo, int nq) {
    const int k = number - 1 - qlo;
    return k < 0 || k >= nq ? x * nq / 12 : k;
}

// Whether the rows that the block product of one diagonal stores, five bytes a cell of tiles x 64 rows of `pitch` columns for B
// chains, are stored as passing through the caches (nontemporal).  That is for batches split over streams: the launches of
// all groups are in flight together, and what they store pushes operands out of the caches long before the row
// kernels read it back.  The line is half of the 256 MB memory-side cache.  us a solve with all rows of the batch passing, those of
// diagonals from 128 MB on, from 192 MB on, and none:
//   first diagonal 446 MB: 128 x 96 stages, 1024 slots 3603, 3604, 3617, 3720
//   432 MB: 64 x 96, 2048 slots 3080, 3080, 3083, 3140
//   351 MB: 12 x 192, 4096 slots 5074, 5081, 5096, 5131
//   209 MB: 200 x 40, 1024 slots 785, 786, 788, 791
//   160 MB: 60 x 30, 4096 slots 554.6, 552.8, 553.7, 554.1
//   157 MB, little over the size from which batches are split: 16 x 254, 1000 slots 5386, 5386, 5393, 5401
// Batches that only the caller splits, four groups, all passing and none from 128 MB on:
//   117 MB: 4 x 192, 4096 slots 2229, 2218;  84 MB: 40 x 60, 1024 slots 515, 509;  54 MB: 8 x 96, 2048 slots 675, 668
constexpr bool rows_pass(int tiles, int pitch, int B) { return 320LL * tiles * pitch * B >= 128LL * 1000 * 1000; }

// Whether all tiles of a solve are one launch whose work-groups wait for each other's data (flow_kernel), or two launches a
// diagonal.  One launch has no gaps between diagonals and a quarter of the instructions a row step, but a work-group
// of four waves for every 64 columns of a tile, and it evaluates every feasible split: it pays while the chip is not full.
// `wide` counts the work-groups of the first diagonal; `wide * nblk` grows with the splits that bounds would have dropped, which
// they do better in tables of 1100 columns and more.  (Chains that chain_pays takes come here only where the caller asks for one
// group.)  us a solve, two launches a diagonal and one:
//   one block: 14 x 7 stages, 780 slots (182 by that measure) 20 and 16;  67 x 8, 184 slots (201) 15 and 14;  100 x 6, 810 slots (1300) 20 and 24
//   two: 67 x 9, 524 slots (1206) 45 and 38;  126 x 16, 315 slots (1260) 44 and 44;  65 x 15, 829 slots (1690) 52 and 59
//   three: 37 x 20, 1074 slots (1887) 93 and 76;  19 x 24, 2245 slots (2052) 97 and 100;  77 x 24, 791 slots (3003) 98 and 106
//   more, without samples: 5 x 53, 777 slots (455) 233 and 112;  6 x 53, 1295 slots (882) 246 and 134;  33 x 63, 410 slots (1848) 369 and 210;  38 x 49, 794 slots
//   (3458) 330 and 295;  112 x 29, 470 slots (3584) 147 and 155;  185 x 26, 390 slots (5180) 180 and 216
//   wide tables, wide * nblk: 4 x 129, 1389 slots (25 k) 740 and 544;  1 x 192, 4096 slots (37 k) 1072 and 1128;  2 x 165, 3436 slots (48 k) 1160 and 1256
//   narrow ones: 15 x 121, 665 slots (42 k) 888 and 778;  25 x 162, 317 slots (55 k) 1611 and 1290;  30 x 122, 463 slots (61 k) 1203 and 1208
// With samples of the finished cells (see uses_bounds) splits are dropped by bounds in that launch too, and it pays for wider batches of
// four blocks and more, longer chains more than short ones (their lists are longer):
//   20 x 39, 2671 slots, five blocks (4200) 276 and 270;  41 x 82, 677 slots (4961) 794 and 746;  43 x 35, 1500 slots (5160) 265 and 274;
//   59 x 56, 884 slots (5782) 484 and 516;  56 x 57, 774 slots, eight blocks (5824) 565 and 560;  116 x 106, 196 slots (6496) 1689 and 1611;
//   24 x 138, 993 slots (6912) 2071 and 2065;  wider batches are split over streams: 8 x 192, 4096 slots (12480) 3609 and 5001
constexpr bool flow_pays(int nblk, int chunks, long long B, bool samples) {
    const long long wide = B * chunks * nblk;
    if (samples && nblk >= 4) return wide <= (nblk < 8 ? 4500 : 7000);
    if (nblk < 4) return wide <= (nblk == 1 ? 224 : nblk == 2 ? 1200 : 2000);
    return wide <= 3500 && wide * nblk <= (chunks >= 18 ? 33000 : 60000);
}

// Byte offset in flow_kernel that lies beyond every row: the column of a cell that does not exist, negative where it is the left side of
// a difference, and the shift of an entry that reads nothing.  A column less a shift has to stay a 32-bit number with both,
// and beyond every row with one of them; flow_pays takes no table of more than 1125 chunks.
constexpr int kFar = 0x3f000000;

// Whether it drops splits by bounds: where there are enough of them.  us a solve without and with, four to seven blocks by the same measure:
//   4 x 50 stages, 2004 slots (896) 134 and 144;  6 x 48, 2048 slots (1188) 132 and 139;  12 x 48, 1024 slots (1224) 120 and 117;
//   10 x 33, 1700 slots (1350) 110 and 111;  5 x 45, 3000 slots (1410) 153 and 158;  14 x 42, 1024 slots (1428) 128 and 121;  14 x 50, 900 slots
//   (1470) 155 and 141;  16 x 48, 1024 slots (1632) 143 and 134;  9 x 33, 2500 slots (1800) 136 and 134;  36 x 56, 643 slots (2772) 263 and 225
// Eight blocks and more, before what belongs to the rows was read early without bounds (4 % of some): 8 x 58, 1659 slots (1664) 208 and 194;
// 1 x 139, 1609 slots (468) 357 and 324;  4 x 112, 1967 slots (1736) 475 and 371; narrow tables lose a little, 7 x 236, 263 slots 1104 and 1155.
constexpr bool flow_bounds(int nblk, int chunks, long long B, bool samples) {
    return samples && (nblk >= 8 || (nblk >= 4 && B * chunks * nblk >= 1420));
}

// Samples of the finished cells: of every kG columns the last one, sample k is column kG k + kG - 1.  Sub-chunk kk holds columns
// kG kk .. kG kk + kG - 1.  Costs do not rise with m, so the operands of a split of shift `shift` are, in all columns of the
// sub-chunk, at most (first column, upper bounds) what the samples of *_below say and at least (last column) what those of *_above say.
// Below zero: no sample, the operand is infeasible.
constexpr int kG = 16;
constexpr int left_below(int kk) { return kk - 1; }
constexpr int right_below(int kk, int shift) { return ((kk * kG + 1 - shift) >> 4) - 1; }
constexpr int left_above(int kk) { return kk; }
constexpr int right_above(int kk, int shift) { return (kk * kG + kG - 1 - shift) >> 4; }

// Chunks of 64 columns below its own that a work-group of flow_kernel waits for at other tiles, by the chain's largest shift:
// those of the operands, column m0 - reach at the lowest, and where it reads samples for upper bounds too, column
// m0 - reach - 15 at the lowest (m0 - 1 without shifts).
constexpr int operand_chunks(int reach) { return (reach + 63) >> 6; }
constexpr int sample_chunks(int reach) { return (reach + kG - 1 + 63) >> 6; }

// Rows of the threshold tables that a work-group of precompute_kernel writes.  Few, where work-groups are too few to fill the
// chip and each is a serial chain of rows; more, where what a work-group costs to start and its reads of the chain count.
// us with 4, 8, 16 and 32 rows, by the number of work-groups with 4:
//   1 x 24 stages (6) 3.2, 3.2, 3.4, 4.1;  10 x 50 (130) 4.2, 4.4, 5.2, 6.7;  3 x 254 (192) 4.2, 4.5, 5.1, 6.7;  8 x 192 (384) 6.6, 7.6, 7.3, 9.4
//   64 x 96 (1536) 9.6, 8.5, 7.8, 9.0;  256 x 24 (1536) 8.1, 6.6, 6.3, 6.6;  700 x 64 (11200) 11.8, 10.2, 9.0, 10.0;  20000 x 8 (40000) 29, 23, 23, 23
constexpr int precompute_rows(int L, long long B) { return B * ((L + 3) / 4) <= 1024 ? 4 : 16; }

// Whether a solve is one launch with a work-group per chain (chain_kernel): up to so many stages, a thread for every column, and all
// rows but the first have to fit into LDS.  A column's instructions grow with the cube of the stages and are one thread's: longer
// chains are better cut into tiles, unless they are many.  us a solve by the kernels of longer chains and by this one:
//   1 x 8 stages, 64 slots 10.0 and 7.2;  67 x 8, 184 slots 12.5 and 7.9;  60 x 8, 1000 slots 21 and 12;  3000 x 8, 300 slots 58 and 37
//   1 x 10, 300 slots 21.8 and 12.4;  10 x 9, 900 slots 29 and 15;  3000 x 12, 200 slots 147 and 102;  1 x 13, 500 slots 25.4 and 20.7;
//   200 x 13, 500 slots 49 and 23;  1000 x 13, 60 slots 58 and 21
// From 14 stages on a few chains lose.  Many gain, in narrow tables (which this line leaves out: it goes by stages and columns only):
//   1 x 14, 60 slots 18.8 and 20.5;  40 x 14, 120 slots 20.9 and 22.5;  100 x 14, 300 slots 32.7 and 25.9;  600 x 14, 188 slots 44.3 and 45.2;
//   600 x 14, 380 slots 80.3 and 72.4;  2000 x 14, 60 slots 86.7 and 46.7
//   1 x 15, 188 slots 20.3 and 25.2;  300 x 15, 188 slots 37.5 and 52.3;  2000 x 15, 188 slots 104 and 200;  2000 x 15, 60 slots 87.4 and 54.5
//   1 x 16, 60 slots 18.8 and 27.1;  300 x 16, 300 slots 53.9 and 64.6;  600 x 16, 60 slots 37.1 and 31.5;  2000 x 16, 60 slots 85.4 and 63.9
constexpr int kChainStages = 13;
constexpr long long kChainLds = 156 * 1024;  // of a compute unit's 160 KB; the static arrays take 2
constexpr long long chain_lds(int L, int pitch) { return 4LL * (L * (L - 1) / 2) * pitch; }
// Row of cell (q, q) in LDS, cell (q, j) stands j - q rows further; the first row of the table (q = 0) is not kept.
constexpr int chain_row(int L, int q) { return (q - 1) * L - q * (q - 1) / 2; }
constexpr bool chain_pays(int L, int pitch) { return L <= kChainStages && pitch <= 1024 && chain_lds(L, pitch) <= kChainLds; }

}  // namespace ckpt_rules
