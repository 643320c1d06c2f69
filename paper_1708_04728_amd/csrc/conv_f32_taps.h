// Which filter blocks conv_f32_taps.hip takes for a layer, and whether its stores reach the layer's outputs.  Plain constant expressions, so that
// the same lines run in the launcher and on the host.
#pragma once

namespace dr {

constexpr int TAPS_BN = 128;                             // pixels per tile: 32 per multiplying wave

// Blocks of 32 filters per workgroup: the number that pads the filter count least, the larger one of two
constexpr int taps_tm(int K)
{
    int best = 1;
    for (int tm = 2; tm <= 3; ++tm)
        if ((K + tm * 32 - 1) / (tm * 32) * tm <= (K + best * 32 - 1) / (best * 32) * best) best = tm;
    return best;
}

// A store's offset counts from the first image of its tile, the filter's plane within its block as the scalar part.  The outputs have to end within
// 2 GiB, and so do the planes of the filters that a block is rounded up to: a lane without an output stores at an offset that the
// hardware compares with the bytes left behind the scalar part, which has to lie inside the buffer.
constexpr bool taps_store_fits(int K, int y_ctot, int P, int Q)
{
    const double plane = (double)P * Q * 4.0;
    return ((double)TAPS_BN / ((double)P * Q) + 2) * y_ctot * plane < 2147483648.0 && 32.0 * taps_tm(K) * plane < 2147483648.0;
}

}  // namespace dr
