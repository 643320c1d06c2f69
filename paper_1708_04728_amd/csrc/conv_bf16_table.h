// Where a chunk of the contraction -- 8 channels of a tap, 16 bytes -- lies: the entries of the tables that conv_bf16_small.hip and
// conv_bf16_wide.hip keep in LDS, and the masks they are tested with.  Plain constant expressions, so that the same lines run in
// the kernels and on the host.
#pragma once

namespace dr {

// A chunk's offset from the first pixel of an output's window, and a pixel's window from the tensor's first element, in bytes modulo 2^32.
// Neither has to fit 31 bits: with padding a window may begin before the tensor, and a filter row then lies 2 GiB or more behind it while
// the sum of the two is inside the tensor.  Whether a chunk exists is therefore a bit of its mask and not of its offset.
constexpr unsigned chunk_offset(int r, int chunk, int W, int C) { return (unsigned)r * (unsigned)W * (unsigned)C * 2u + (unsigned)chunk * 16u; }
constexpr unsigned window_offset(int img, int ih0, int iw0, int H, int W, int C)
{
    return (((unsigned)img * (unsigned)H + (unsigned)ih0) * (unsigned)W + (unsigned)iw0) * (unsigned)C * 2u;
}

// Bits of a chunk's mask: its tap column s (0..8), its filter row r (9 + 0..15); the sign bit alone: beyond the contraction.  Bits of a
// window's mask: the columns and rows that lie outside the image, and the sign bit.  A chunk is read where the two have no bit in common.
constexpr unsigned CHUNK_NONE = 0x80000000u, WINDOW_NONE = 0xFFFFFFFFu;      // WINDOW_NONE: no such output
constexpr unsigned chunk_mask(bool exists, int r, int s) { return exists ? (0x200u << r) | (1u << s) : CHUNK_NONE; }
constexpr bool chunk_exists(unsigned mask) { return (int)mask >= 0; }
constexpr unsigned bits(int lo, int hi) { return hi >= lo ? (2u << hi) - (1u << lo) : 0u; }      // lo..hi set
constexpr int smaller(int a, int b) { return a < b ? a : b; }
constexpr int larger(int a, int b) { return a > b ? a : b; }
constexpr unsigned window_mask(bool exists, int ih0, int iw0, int R, int S, int H, int W)
{
    return ~(bits(larger(0, -iw0), smaller(S - 1, W - 1 - iw0)) | bits(larger(0, -ih0), smaller(R - 1, H - 1 - ih0)) << 9) | (exists ? 0u : WINDOW_NONE);
}

// Slices of 8 chunks of a contraction: row_chunks from filter row to filter row.  They run on across filter rows (row_chunks: a row's chunks)
// where that saves slices; else every row starts one (rounded up to whole slices).
inline int chunk_slices(int R, int S, int C, int* row_chunks)
{
    const int run = S * (C / 8), spr = (run + 7) / 8, flat = (R * run + 7) / 8;
    const bool on = run >= 8 && flat < R * spr;
    *row_chunks = on ? run : spr * 8;
    return on ? flat : R * spr;
}

}  // namespace dr
