// fp32 operands as three bf16 pieces: the device code that the kernels on them share (conv_f32_pieces.hip has the arithmetic and what it measures).
#pragma once
#include "conv_f32_dev.h"
#include "f32_pieces.h"

namespace dr {
namespace {

// The pieces of eight operands, scaled, to LDS, one `stride` behind the other
__device__ __forceinline__ void put_pieces(const float (&v)[8], unsigned char* at, int stride)
{
    float t[8];
    u32x4 p[3];
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = v[e] * PIECES_SCALE;
    split8(t, p[0], p[1], p[2]);
#pragma unroll
    for (int e = 0; e < 3; ++e) *reinterpret_cast<u32x4*>(at + e * stride) = p[e];
}

// One block of 32 x 32 outputs by fp32 matrix instructions, straight from memory: for operands that three bf16 pieces do not hold.  Lane half h: channel c + h.
__device__ __forceinline__ f32x16 exact_block(const KArgs& a, int m, int n, int half)
{
    const ConvGeom& g = a.g;
    const int HW = g.H * g.W, PQ = g.P * g.Q;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, a.w_bytes, 0x00020000);
    const int nn = n < g.Ng ? n : 0, img = nn / PQ, pix = nn - img * PQ, p = pix / g.Q, q = pix - p * g.Q, ih0 = p * g.sh - g.ph, iw0 = q * g.sw - g.pw;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int r = 0; r < g.R; ++r)
        for (int s = 0; s < g.S; ++s) {
            const bool ok = (n < g.Ng) & ((unsigned)(ih0 + r) < (unsigned)g.H) & ((unsigned)(iw0 + s) < (unsigned)g.W);
            const int xo = ok ? ((img * g.C + half) * HW + (ih0 + r) * g.W + iw0 + s) * 4 : OOB;
            const int wo = m < g.K ? (m * g.Kg + (r * g.S + s) * g.C + half) * 4 : OOB;
#pragma unroll 2
            for (int c = 0; c < g.C; c += 2) {
                const float fa = buf_load(rw, wo, c * 4), fb = buf_load(rx, xo, c * HW * 4);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa, fb, acc, 0, 0, 0);
            }
        }
    return acc;
}

// Whole blocks: a store per element whose filter is the scalar offset, with a descriptor for every eight
template <int TM, int TN>
__device__ __forceinline__ void store_whole(const KArgs& a, const f32x16 (&acc)[TM][TN], const f32x4 (&bias)[TM][4], int mw, int nw, int img0, unsigned long long by_pq)
{
    const int half = (threadIdx.x >> 5) & 1, l32 = threadIdx.x & 31;
    const int PQ = a.g.P * a.g.Q, plane = PQ * 4;
    int img[TN], pix[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int o = nw + j * 32 + l32 - img0 * PQ;
        img[j] = div_small(o, by_pq);
        pix[j] = (half * 4 * PQ + o - img[j] * PQ) * 4;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int m8 = mw + i * 32 + q * 8, ct = a.ctot_seg[0];
            const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)(a.y_seg[0] + ((size_t)img0 * ct + m8) * PQ), 0, 0x7FFFFFFF, 0x00020000);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int vy = nw + j * 32 + l32 < a.g.Ng ? img[j] * ct * plane + pix[j] : OOB;
                f32x4 v = bias[i][q];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += acc[i][j][q * 4 + e];
                if (a.g.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) buf_store(v[e], ry, vy, e * plane);
            }
        }
}

// The end of a tile for a multiplying wave: the two sums, bias, ReLU, the store.  Rows from mw and columns from nw on; img0: the tile's first image.  Whether a block
// of 32 x 32 is computed again depends on its own sums alone, so that a layer has the same bits in tiles of any size.
template <int TM, int TN>
__device__ __forceinline__ void finish_tile(const KArgs& a, f32x16 (&acc)[TM][TN], const f32x16 (&small)[TM][TN], int mw, int nw, int n0, int img0,
                                            unsigned long long by_pq)
{
    const int half = (threadIdx.x >> 5) & 1, l32 = threadIdx.x & 31;
    // (the biases before any store: a load behind stores is waited for together with them)
    f32x4 bias[TM][4];
    const __amdgpu_buffer_rsrc_t rbias = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, a.bias ? a.g.K * 4 : 0, 0x00020000);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[i][q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (mw + i * 32 + half * 4 + q * 8) * 4, 0, 0));
    unsigned bad = 0;                            // blocks that pieces do not hold (no residual here, which a second store would find changed in place)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float z = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][j][v] += small[i][j][v];
                z = __builtin_fmaf(acc[i][j][v], 0.f, z);
                acc[i][j][v] *= PIECES_UNSCALE;
            }
            bad |= __any(z != 0.f) ? 1u << (i * TN + j) : 0u;
        }
    if (a.far_store || mw + TM * 32 > a.g.K) store_tile<TM, TN, false>(a, acc, mw, nw, n0);
    else store_whole<TM, TN>(a, acc, bias, mw, nw, img0, by_pq);
    if (bad == 0) return;
    // (over what has just been stored)
    __builtin_amdgcn_s_waitcnt(0);
#pragma unroll 1
    for (int b = 0; b < TM * TN; ++b) {
        if (!(bad >> b & 1)) continue;
        const int m = mw + b / TN * 32, n = nw + b % TN * 32 + l32, img = n / (a.g.P * a.g.Q);
        const f32x16 one = exact_block(a, m + l32, n, half);
        if (n < a.g.Ng) store_far(a, one, m + half * 4, img, n - img * a.g.P * a.g.Q);
    }
}

// ---- a stream of tiles whose operands are cut slice by slice
// A slice is STEPS k-steps of 16; LDS holds two of them, of each operand for each piece and each 8 k a run of rows (filters or pixels), 16 bytes each.
template <int ROWS, int STEPS> struct CutLayout {
    static constexpr int CHUNK = ROWS * 16 + 16, PIECE = 2 * STEPS * CHUNK, BYTES = 3 * PIECE;
};
template <int BM, int BN, int STEPS> constexpr int cut_stage() { return CutLayout<BM, STEPS>::BYTES + CutLayout<BN, STEPS>::BYTES; }

// The multiplying waves' part of a tile of `slices` slices, its first slice in stage `stage`: behind the barrier that ends its writing
template <int WGM, int WGN, int TM, int TN, int STEPS>
__device__ __forceinline__ void multiply_tile(const unsigned char* const lds, int slices, int& stage, f32x16 (&acc)[TM][TN], f32x16 (&small)[TM][TN])
{
    using LA = CutLayout<WGM * TM * 32, STEPS>;
    using LB = CutLayout<WGN * TN * 32, STEPS>;
    constexpr int STAGE = LA::BYTES + LB::BYTES;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5, l32 = lane & 31, wm = wave / WGN, wn = wave % WGN;
    u32x4 fa[2][TM][3], fb[2][TN][3];
    int a_rd = half * LA::CHUNK + (wm * TM * 32 + l32) * 16 + stage * STAGE, b_rd = LA::BYTES + half * LB::CHUNK + (wn * TN * 32 + l32) * 16 + stage * STAGE;
    auto read = [&](int ks, auto set_c, int e) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_c)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[SET][i][e] = *reinterpret_cast<const u32x4*>(lds + a_rd + e * LA::PIECE + ks * 2 * LA::CHUNK + i * 512);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[SET][j][e] = *reinterpret_cast<const u32x4*>(lds + b_rd + e * LB::PIECE + ks * 2 * LB::CHUNK + j * 512);
    };
    auto multiply = [&](auto set_c, int x, int y) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_c)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (x + y) small[i][j] = mfma(fa[SET][i][x], fb[SET][j][y], small[i][j]);
                else acc[i][j] = mfma(fa[SET][i][0], fb[SET][j][0], acc[i][j]);
    };
    auto step = [&](auto set_c, int next_ks) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_c)::value;
        multiply(set_c, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        read(next_ks, IC<1 - SET>{}, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(set_c, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        read(next_ks, IC<1 - SET>{}, 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(set_c, 1, 0);
        __builtin_amdgcn_sched_barrier(0);
        read(next_ks, IC<1 - SET>{}, 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(set_c, 1, 1);
        multiply(set_c, 0, 2);
        multiply(set_c, 2, 0);
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = small[i][j][v] = 0.f;
#pragma unroll
    for (int e = 0; e < 3; ++e) read(0, IC<0>{}, e);
    auto turn = [&]() __attribute__((always_inline)) {       // every wave has read the stage; the other one is complete
        const int d = stage ? -STAGE : STAGE;
        a_rd += d; b_rd += d;
        stage ^= 1;
        ring_barrier();
    };
    for (int k = 0; k < slices; ++k) {
        step(IC<0>{}, 1);
        turn();
        step(IC<1>{}, 0);                        // (after the tile's last slice it reads what is read again)
    }
}

}  // namespace
}  // namespace dr
