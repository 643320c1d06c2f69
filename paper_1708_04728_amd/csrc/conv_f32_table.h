// One-word entries of the table k -> (offset of x[0][c][r][s], tap) that conv_f32.hip keeps in LDS.  Plain constant expressions, so
// that the same lines run in the kernel and on the host.
#pragma once

namespace dr {

// 5 bits of tap (31: beyond the contraction), 26 bits of offset in elements: the sign bit stays clear.
constexpr int TAB1_OFFSET_BITS = 26, TAB1_NO_TAP = 31;

constexpr int tab1_entry(int offset, int tap) { return offset << 5 | tap; }
constexpr int tab1_offset(int entry) { return (int)((unsigned)entry >> 5); }
constexpr int tab1_tap(int entry) { return entry & 31; }

// Whether every entry of an R x S filter on C planes of H x W fits.  The largest one bounds it, not the tensor: with padding a filter may be
// taller than the map, and its last rows then start behind the last plane (31 x 1 on one row of 9 million pixels: 30 rows further).
constexpr bool tab1_fits(int C, int H, int W, int R, int S)
{
    return (long)R * S <= 31 && (C - 1) * ((long)H * W) + (long)(R - 1) * W + S - 1 < (1l << TAB1_OFFSET_BITS);
}

}  // namespace dr
