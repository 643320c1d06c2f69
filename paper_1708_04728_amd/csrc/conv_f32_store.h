// Whether the short form of conv_f32.hip's store reaches a layer's outputs.  Plain constant expressions, so that the same lines run in the launcher and on
// the host.
#pragma once

namespace dr {

// Offsets are counted from a tile's first image: its images, of up to `pixels` pixels' worth, times the channels of the widest tensor (output or residual)
// below 2 GiB.  A row's plane is the scalar part of an offset, and beside it the lanes without an output -- rows that a block of 32 is rounded up to -- are
// sent out of range, which they are only for sure where the scalar part lies inside the 2 GiB that the buffer spans: 3 planes for a store (each eight
// filters have a buffer of their own), 27 for a residual.
constexpr bool store_tile_fits(int ctot, int P, int Q, bool residual, int pixels = 128)
{
    const double plane = (double)P * Q * 4.0;
    return (pixels + 2.0 * P * Q) * (double)ctot * 4.0 < 2147483648.0 && (residual ? 27.0 : 3.0) * plane < 2147483647.0;
}

}  // namespace dr
