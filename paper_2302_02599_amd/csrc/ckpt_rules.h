// Rules of the fill that are plain arithmetic on sizes.  C++ without HIP, so that the host tests can call them.
#pragma once

namespace ckpt_rules {

// Upper bounds of the block product (stage 1 of gemm_kernel).  A tile has nq middle splits, k = 0 .. nq - 1.  KS slices
// of waves share them, and sixteen lanes of a slice, x = 0 .. 15, fetch the bounds of one split each.  Any splits give a
// valid upper bound; more of them, and better ones, give a tighter one.

// With more splits than this slice 0 asks finished neighbours which splits they took.
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

}  // namespace ckpt_rules
