// What the tiled fp32 convolution kernels share: their arguments, loads and stores through buffer descriptors, and the store of a wave's sums.
#pragma once
#include <algorithm>

#include "conv_bf16_dev.h"
#include "conv_f32_store.h"
#include "dr_internal.h"

namespace dr {
namespace {

struct KArgs {
    const float* x;
    const float* w;
    const float* bias;
    const float* res;
    float* y;
    ConvGeom g;
    int grid_m, grid_n;
    int x_bytes, w_bytes;   // sizes of the x and w tensors (both < 2 GiB, checked by the launcher)
    int w_krsc;             // filters are in KRSC order (else KCRS)
    int row_groups;         // CF = false: k runs over (c, r, groups of 4 taps), see the header
    // Stacked convolution (Eq. (12): several filter banks on one input) whose filter ranges go to different tensors:
    // filter m < split_end[0] goes to destination 0, m < split_end[1] to destination 1, ... (unused ends hold INT_MAX).
    // Element (img, m, pix) of destination d lies at y_seg[d][(img * ctot_seg[d] + m) * P * Q + pix] (the host has
    // folded the destination's channel offset and the range's first filter into y_seg).  nsplit <= 1: everything to destination 0.
    int nsplit;
    int far_store;          // destinations or offsets that the short form of the store does not take (see store_fits)
    int split_end[3];
    float* y_seg[4];
    int ctot_seg[4];
    float* part;            // partial sums [splits][K][Ng] of a split contraction, or NULL
    int splits, slices_per_split;
};

__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

__device__ __forceinline__ void buf_store(float v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
#endif
}

// The store of one column of a 32x32 block, element by element: any destinations, any size
__device__ __forceinline__ void store_far(const KArgs& a, const f32x16& acc, int mh, int img, int pix)
{
    const ConvGeom& g = a.g;
    const size_t PQ = (size_t)g.P * g.Q;
#pragma unroll 1
    for (int v = 0; v < 16; ++v) {
        const int m = mh + (v >> 2) * 8 + (v & 3);
        if (m >= g.K) continue;
        float o = acc[0];
#pragma unroll
        for (int u = 1; u < 16; ++u) o = v == u ? acc[u] : o;
        if (a.bias) o += a.bias[m];
        if (a.res) o += a.res[((size_t)img * g.res_ctot + m) * PQ + pix];
        if (g.relu) o = fmaxf(o, 0.f);
        const int d = (m >= a.split_end[0]) + (m >= a.split_end[1]) + (m >= a.split_end[2]);
        float* const yd = d == 0 ? a.y_seg[0] : d == 1 ? a.y_seg[1] : d == 2 ? a.y_seg[2] : a.y_seg[3];
        const int ct = d == 0 ? a.ctot_seg[0] : d == 1 ? a.ctot_seg[1] : d == 2 ? a.ctot_seg[2] : a.ctot_seg[3];
        yd[((size_t)img * ct + m) * PQ + pix] = o;
    }
}

// The sums of a wave's TM x TN blocks of 32x32, rows from mw and columns from nw on; n0: the tile's first column
template <int TM, int TN, bool SPLIT>
__device__ __forceinline__ void store_tile(const KArgs& a, const f32x16 (&acc)[TM][TN], int mw, int nw, int n0)
{
    constexpr int OOB = (int)0x80000000;
    const ConvGeom& g = a.g;
    const int PQ = g.P * g.Q, half = (threadIdx.x >> 5) & 1, l32 = threadIdx.x & 31;
    // Accumulator register v of a 32x32 tile holds row 8*(v/4) + 4*half + v%4, column l32.  Addresses are a descriptor that starts at
    // the tile's first image, a per-lane offset and the row as scalar offset; lanes without an output, and rows beyond the last filter, store
    // outside the descriptor.  Nothing per element but the bias, the ReLU and the store: with a branch each for bias, residual and destination
    // (16 dependent loads, some 50 instructions per element, which fp32 matrix instructions of other waves do not overlap with) the store took as
    // long as six to eight slices.  GoogLeNet's 3a on 32 images, slim: its first level 24.3 -> 20.2 us, the module 99.7 -> 92.9; 4c on 64 images
    // 166 -> 158.5; 3x3 32 -> 256 on 30 x 45 x 9 with what follows it 44.1 -> 42.1; AlexNet's 5x5, 150 slices, 1 % or less.
    const int img0 = n0 / PQ;
    const __amdgpu_buffer_rsrc_t rbias = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, a.bias ? g.K * 4 : 0, 0x00020000);
    // the biases of all blocks first: a load behind stores would be waited for together with them (a wave by itself on its matrix core spent 21 000 cycles on the
    // store of 64 x 64 outputs, as long as ten slices of products)
    f32x4 bias[TM][4];
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                bias[i][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (__builtin_amdgcn_readfirstlane(mw + i * 32) + half * 4 + q * 8) * 4, 0, 0));
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = nw + j * 32 + l32;
        const int img = n / PQ, pix = n - img * PQ;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = __builtin_amdgcn_readfirstlane(mw + i * 32), mh = mb + half * 4;
            const bool whole = mb + 32 <= g.K;                // (wave-uniform)
            if constexpr (SPLIT) {
                const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void*)(a.part + (size_t)blockIdx.y * g.K * g.Ng), 0, 0x7FFFFFFF, 0x00020000);
                const int vp = n < g.Ng ? (mh * g.Ng + n) * 4 : OOB;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = (v >> 2) * 8 + (v & 3);
                    buf_store(acc[i][j][v], rp, whole || mh + row < g.K ? vp : OOB, row * g.Ng * 4);
                }
                continue;
            }
            if (a.far_store) {
                if (n < g.Ng) store_far(a, acc[i][j], mh, img, pix);
                continue;
            }
            f32x4 o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = bias[i][q];
#pragma unroll
            for (int v = 0; v < 16; ++v) o[v >> 2][v & 3] += acc[i][j][v];
            if (a.res) {
                const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc((void*)(a.res + (size_t)img0 * g.res_ctot * PQ), 0, 0x7FFFFFFF, 0x00020000);
                const int vr = n < g.Ng ? (((img - img0) * g.res_ctot + mh) * PQ + pix) * 4 : OOB;
                float res[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = (v >> 2) * 8 + (v & 3);
                    res[v] = buf_load(rr, whole || mh + row < g.K ? vr : OOB, row * PQ * 4);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) o[v >> 2][v & 3] += res[v];
            }
            if (g.relu) {
#pragma unroll
                for (int v = 0; v < 16; ++v) o[v >> 2][v & 3] = fmaxf(o[v >> 2][v & 3], 0.f);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // rows mb + 8 q .. + 7 have one destination (wave-uniform)
                const int m8 = mb + q * 8, d = (m8 >= a.split_end[0]) + (m8 >= a.split_end[1]) + (m8 >= a.split_end[2]);
                const int ct = d == 0 ? a.ctot_seg[0] : d == 1 ? a.ctot_seg[1] : d == 2 ? a.ctot_seg[2] : a.ctot_seg[3];
                float* const yd = d == 0 ? a.y_seg[0] : d == 1 ? a.y_seg[1] : d == 2 ? a.y_seg[2] : a.y_seg[3];
                const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)(yd + (size_t)img0 * ct * PQ + (size_t)m8 * PQ), 0, 0x7FFFFFFF, 0x00020000);
                const int vy = n < g.Ng ? (((img - img0) * ct + half * 4) * PQ + pix) * 4 : OOB;
#pragma unroll
                for (int e = 0; e < 4; ++e) buf_store(o[q][e], ry, whole || mh + q * 8 + e < g.K ? vy : OOB, e * PQ * 4);
            }
        }
    }
}

// The short form of the store: offsets that fit (conv_f32_store.h), and ranges of filters with a destination each that start at multiples of 8 (a lane's half
// holds four filters of every eight).
inline bool store_fits(const KArgs& a, int pixels)
{
    int ctot = a.g.res_ctot;
    for (int d = 0; d < 4; ++d) ctot = std::max(ctot, a.ctot_seg[d]);
    for (int d = 0; d < 3; ++d)
        if (a.split_end[d] != 0x7FFFFFFF && a.split_end[d] % 8 != 0) return false;
    return store_tile_fits(ctot, a.g.P, a.g.Q, a.res != nullptr, pixels);
}

// Destinations of a (stacked) layer, tensor sizes.
inline KArgs conv_f32_args(const ConvGeom& g, const float* x, const float* w, const float* bias, const float* residual, float* y, const ConvSplit* split,
                            int pixels = 128)      // of a tile
{
    KArgs a;
    a.x = x; a.w = w; a.bias = bias; a.res = residual; a.y = y; a.g = g;
    a.grid_m = a.grid_n = 0;
    a.row_groups = 0;
    a.part = nullptr;
    a.splits = a.slices_per_split = 0;
    a.nsplit = 0;
    for (int d = 0; d < 4; ++d) { a.y_seg[d] = nullptr; a.ctot_seg[d] = 0; if (d < 3) a.split_end[d] = 0x7FFFFFFF; }
    a.y_seg[0] = y + (size_t)g.y_coff * g.P * g.Q;
    a.ctot_seg[0] = g.y_ctot;
    if (split && split->n > 1) {
        a.nsplit = split->n;
        const long PQ = (long)g.P * g.Q;
        int start = 0;
        for (int d = 0; d < split->n && d < 4; ++d) {
            const ConvDest& s = split->dst[d];
            a.y_seg[d] = (float*)s.y + ((long)s.c_offset - start) * PQ;
            a.ctot_seg[d] = s.ctot;
            start += s.k;
            if (d < 3 && d + 1 < split->n) a.split_end[d] = start;
        }
    }
    a.x_bytes = (int)((size_t)g.N * g.C * g.H * g.W * 4);
    a.w_bytes = (int)((size_t)g.K * g.Kg * 4);
    a.w_krsc = g.w_krsc;
    a.far_store = !store_fits(a, pixels);
    return a;
}

}  // namespace
}  // namespace dr
