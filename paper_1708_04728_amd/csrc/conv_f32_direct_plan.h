// Which layers conv_f32_direct.hip takes, with which tiles.  Plain functions of numbers, so that the same lines run in the launcher and on the host.
#pragma once
#include "conv_f32_pieces_plan.h"

namespace dr {

// Tiles of filters x 128 pixels; microseconds of a tile: fixed + slices * slice, fitted to 150 strided layers (6, 5 and 7 % off)
constexpr int DIRECT_TILES = 3, DIRECT_BN = 128;
struct DirectTile { int bm; double fixed, slice; };
constexpr DirectTile direct_tile[DIRECT_TILES] = {{128, 9.4, 1.34}, {96, 6.9, 1.30}, {64, 3.8, 1.14}};

constexpr long direct_count(const PiecesLayer& l, const DirectTile& t)
{
    return ((long)l.K + t.bm - 1) / t.bm * (((long)l.N * l.P * l.Q + DIRECT_BN - 1) / DIRECT_BN);
}

// The fastest tile of a layer by itself; us: the time it takes
inline int direct_best(const PiecesLayer& l, int cus, double* us)
{
    int best = -1;
    for (int i = 0; i < DIRECT_TILES; ++i) {
        const double t = 2.5 + ceil((double)direct_count(l, direct_tile[i]) / cus) * (direct_tile[i].fixed + pieces_slices(l) * direct_tile[i].slice);
        if (best < 0 || t < *us) { best = i; *us = t; }
    }
    return best;
}

// Layers of nine taps and more, strided in both directions, with more than 64 filters, where the other fp32 kernels use tiles of 32 filters (K % 64 from 1 to 32), whose
// strided rows cost them most; from 1.9 units of the operations at 125 TFLOP/s (filters in whole 32) on.  Of 36 such layers on rectified operands all gain, 1.04 to 3.2
// (3x3 96 -> 208 on 56 x 56 x 99 3.09, 160 -> 288 on 28 x 28 x 52 1.48, 64 -> 96 on 64 x 64 x 69 1.11).  Beyond the line 0.2 to 2.2.
// Whole tiles of 64 filters stay there: of 30 that a line at 1.2 units would take 7 lose (3x3 and 5x5; 5x5 96 -> 192 on 27 x 27 x 128 215 us there, 248 here; 96 -> 256 on
// 27 x 27 x 256 541 and 588) and 23 gain 1.07 to 2.0, and a gain measured alone need not hold between other layers: 96 -> 256 on 28 x 28 x 128 gains 1.10 alone, while
// AlexNet's slim blocks, whose second convolution it is, took 360 us with the other kernel and 389 with this one.
// Strides of 1 in one direction and fewer taps: 0.85 to 1.1 (2x4 112 -> 66 on 78 x 82 x 12 67 and 80).  1x1 layers gain nothing: 130 of them 0.66 to 1.1.
inline bool direct_pays(const PiecesLayer& l, int cus)
{
    if (l.sh == 1 || l.sw == 1 || l.R * l.S < 9 || l.C % 16 != 0 || l.K <= 64 || (long)l.P * l.Q > 65536) return false;
    if ((l.K + 31) / 32 * 32 >= (l.K + 63) / 64 * 64) return false;
    const double least = 2e-6 * l.N * l.P * l.Q * ((l.K + 31) / 32 * 32.0) * l.C * l.R * l.S / 125.0;
    double us = 0;
    direct_best(l, cus, &us);
    return us < 1.9 * least;
}

}  // namespace dr
