// bf16 convolution of small layers: few images, or a few thousand output pixels.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (r, s, c)
//
// What bounds such a layer is not arithmetic and not bandwidth but the chain of dependent steps inside one workgroup: the
// streaming kernel (conv_bf16_dma.hip) walks the contraction in slices of 64, and with a tile or less per compute unit every
// slice costs it 0.4 us (its waves send the slice's loads, wait for older ones, meet, read operands and multiply one after
// the other) while most compute units stand idle.  Here
//   * the tile is as small as the layer leaves compute units for: 32 x 32, 64 x 32 or 64 x 64;
//   * some waves multiply and do nothing else, others send the loads; they meet once per stage of two slices.  The multiplying waves
//     use the 16 x 16 x 32 instruction, which adds in the order of the 32 x 32 x 16 one (compared bit by bit on the card), so that the
//     results are the bits of the streaming kernel; four waves then read the operands of a 32 x 32 tile from LDS at once.  (Sharing the
//     contraction among the waves adds the products in another order: a few outputs in ten thousand round the other way, and 25
//     layers later the class probabilities of GoogLeNet differ by 1 to 3 %.)
//   * where a chunk of the contraction lies is worked out once, by the multiplying waves while the loading waves decode their pixels: a
//     table in LDS, chunk -> {offset, mask}.  A load then costs its wave half a dozen instructions.  Decoding chunk by chunk in every
//     loading wave was what bounded the kernel before: with every load and every multiplication taken out the slice still took
//     0.16 of its 0.2 us.  The loading waves are still on the path of every stage: an instruction or a branch more between the barrier
//     and the loads shows (two more: 2 to 7 %), so the addresses are worked out before it;
//   * two groups of loading waves send a slice each of a stage;
//   * one launch takes several layers (the second steps of an inception module, say): a launch costs 3 to 4 us on a
//     stream whatever it does, as much as the layer itself.  A job may also be a 3x3 max-pooling layer, which a
//     module's pooling branch needs beside the other branches' first steps.
// Measured in chains of dependent launches of one layer (3.1 us of which are the launch), one wave per 32 x 32 block and four loading waves that
// decode -> the table and two loading groups -> addresses ready before the barrier: 3x3 160 -> 320 on one 14 x 14 image 8.5 -> 5.7 -> 5.4 us,
// 5x5 32 -> 512 6.2 -> 4.6 -> 4.4, 1x1 832 -> 624 on 7 x 7 5.4 -> 4.4 -> 3.9, 3x3 96 -> 128 on 28 x 28 x 8 (64 x 64 tiles, one per compute unit) 8.2 -> 6.8 -> 6.6;
// the slim GoogLeNet on one image 151 -> 128 -> 124 us.
// What bounds it now: 0.10 us per slice for tiles of 32 x 32 and, at two tiles of 64 x 64 per compute unit, the path from L2 into LDS (32 loads
// of 1 KiB per pair of slices, about 24 cycles each).
//
// Operands travel as in the streaming kernel: 16-byte buffer loads that write LDS, lanes outside the tensor or in the padding at
// an offset the hardware answers with zeros, chunk j of row r stored at chunk j ^ ((r >> 1) & 7) so that loads and operand
// reads are free of bank conflicts.
#include <algorithm>

#include "dr_internal.h"
#include "dr_store.h"
#include "conv_bf16_dev.h"

namespace dr {
namespace {

constexpr int SMALL_TABLE = 2048;                        // chunks of 8 contraction elements that the table holds (16 KB of LDS)

struct SmallJob {
    const uint16_t* x;
    const uint16_t* w;                                   // NULL: a max-pooling layer (3x3)
    const float* bias;
    const uint16_t* res;
    uint16_t* y_seg[4];                                  // destinations of the filter ranges (see ConvSplit), y_seg[0] alone otherwise
    int ctot_seg[4], split_end[3];
    int res_ctot;
    int C, H, W, K, R, S, sh, sw, ph, pw, P, Q, Kg, Ng, relu;
    int x_bytes, w_bytes;
    int stem_hp, stem_wp;                                // padded 4-channel input copy (see launch_conv_bf16_stem), 0: ordinary input
    int pointwise, tabled;                               // 1x1 at stride 1; the table holds the contraction
    int c8, run_chunks;                                  // 16-byte chunks per tap, per filter row
    int row_chunks;                                      // chunks from filter row to filter row of the slices: run_chunks, or rounded up to whole slices
    int slices;
    unsigned magic_c8, magic_row;
    unsigned long long m_pq, m_q;
    int n_tiles, tiles;                                  // pixel tiles; tiles in all
    int vec;                                             // whole groups of 8 filters, 16-byte accesses of output, residual and bias aligned
};
struct SmallArgs {
    int first[SMALL_GROUP_MAX];                          // first workgroup of each job (a multiple of 8); beyond the last: INT_MAX
    SmallJob job[SMALL_GROUP_MAX];
};

// How a loading wave finds a chunk: by the table; 1x1 filters at stride 1, where the chunks lie side by side; worked out chunk by chunk for a
// contraction that the table does not hold (about 20 instructions more per slice and wave; the streaming kernel, which took these layers once,
// needs twice as long: 7x7 512 -> 4096 on one pixel 113 us there, 56 here; 3x3 2048 -> 512 on 7 x 7 87 and 41)
enum { TABLE, POINTWISE, LONG };

// Keeps the computation of v before what follows
__device__ __forceinline__ void keep(int& v) { asm volatile("" : "+v"(v)); }

// 3x3 max-pooling of one job: an item is one 16-byte channel group of an output pixel
__device__ __forceinline__ void pool_items(const SmallJob& j, int block)
{
    const int item = block * (int)blockDim.x + (int)threadIdx.x;
    if (item >= j.Ng * j.c8) return;
    const int n = item / j.c8, cv = item - n * j.c8;
    const int img = div_small(n, j.m_pq), pix = n - img * j.P * j.Q, p = div_small(pix, j.m_q), q = pix - p * j.Q;
    const int h0 = p * j.sh - j.ph, w0 = q * j.sw - j.pw;
    const uint16_t* xb = j.x + (size_t)img * j.H * j.W * j.C + cv * 8;
    u32x4 raw[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int h = h0 + t / 3, w = w0 + t % 3;
        raw[t] = u32x4{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};      // -inf
        if ((unsigned)h < (unsigned)j.H && (unsigned)w < (unsigned)j.W) raw[t] = *reinterpret_cast<const u32x4*>(xb + ((size_t)h * j.W + w) * j.C);
    }
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float lo = __uint_as_float(raw[0][e] << 16), hi = __uint_as_float(raw[0][e] & 0xFFFF0000u);
#pragma unroll
        for (int t = 1; t < 9; ++t) {
            lo = fmaxf(lo, __uint_as_float(raw[t][e] << 16));
            hi = fmaxf(hi, __uint_as_float(raw[t][e] & 0xFFFF0000u));
        }
        o[e] = pack_bf16x2(lo, hi);
    }
    *reinterpret_cast<u32x4*>(j.y_seg[0] + (size_t)n * j.C + cv * 8) = o;
}

// A tile of 16 TM WM filters x 16 TN WN pixels: WM x WN multiplying waves with TM x TN blocks of 16 x 16 each, LG groups of four loading
// waves, a slice of each stage for every group, three stages in LDS.
template <int TM, int TN, int WM, int WN, int LG>
__global__ __launch_bounds__((WM * WN + 4 * LG) * 64) void conv_bf16_small_kernel(const SmallArgs args)
{
    constexpr int NS = 3, G = LG;                                            // stages in LDS; slices of a stage, one per loading group
    constexpr int CW = WM * WN, BM = WM * TM * 16, BN = WN * TN * 16, A_PER = BM / 32, B_PER = BN / 32, SLICE = (BM + BN) * 128, STAGE = G * SLICE;
    constexpr int L = A_PER + B_PER;                                         // a wave's loads for a stage
    static_assert(BM % 32 == 0 && BN % 32 == 0 && (NS - 1) * L < 63, "loads in flight");
    __shared__ __attribute__((aligned(1024))) unsigned char ring[NS * STAGE];
    __shared__ __attribute__((aligned(16))) u32x2 table[SMALL_TABLE];      // chunk of the contraction -> {offset, mask}

    // ---- the job and the tile.  Workgroup b runs on die b & 7; a die takes a contiguous range of tiles, filter block by filter
    // block, so that the pixel tiles of one filter block read it from one L2.  (The job is copied: left in the argument
    // buffer, every field would be read again behind each wait.)
    static_assert(SMALL_GROUP_MAX == 4, "jobs");
    const int ji = ((int)blockIdx.x >= args.first[1]) + ((int)blockIdx.x >= args.first[2]) + ((int)blockIdx.x >= args.first[3]);
    const SmallJob j = args.job[ji];
    const int b = (int)blockIdx.x - args.first[ji], die = b & 7, s_die = b >> 3, per = j.tiles >> 3, odd = j.tiles & 7;
    if (s_die >= per + (die < odd ? 1 : 0)) return;
    const int t = die * per + min(die, odd) + s_die;
    if (!j.w) { pool_items(j, t); return; }
    const int mt = t / j.n_tiles, nt = t - mt * j.n_tiles;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slices = j.slices, stages = (slices + G - 1) / G;

    // Iteration k, for every wave: at the barrier stage k has landed and stage k - 1 has been read; behind it the multiplying waves
    // read stage k and multiply stage k - 1, the loading waves send stage k + NS - 1 into the LDS stage k - 1 has left.
    if (wave >= CW) {
        // ---- loading: pass i of this wave fills rows 32 i + lrow of an operand
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)j.x, 0, j.x_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)j.w, 0, j.w_bytes, 0x00020000);
        const int lw = (wave - CW) & 3, lg = (wave - CW) >> 2, lrow = lw * 8 + (lane >> 3), lc = (lane & 7) ^ ((lrow >> 1) & 7);
        int a_voff[A_PER];
        unsigned b_base[B_PER], b_mask[B_PER];           // windows of the pixels (conv_bf16_table.h)
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int m = mt * BM + i * 32 + lrow;
            a_voff[i] = m < j.K ? (m * j.Kg + lc * 8) * 2 : OOB;
        }
#pragma unroll
        for (int i = 0; i < B_PER; ++i) {
            const int n = nt * BN + i * 32 + lrow;
            const bool in = n < j.Ng;
            if (j.pointwise) {                           // output pixel n reads input pixel n
                b_base[i] = window_offset(0, 0, n, 0, 0, j.C);
                b_mask[i] = in ? CHUNK_NONE : WINDOW_NONE;
            } else {
                const int nn = in ? n : 0;
                const int img = div_small(nn, j.m_pq), pix = nn - img * j.P * j.Q, p = div_small(pix, j.m_q), q = pix - p * j.Q;
                if (j.stem_wp) {                         // chunk lc of a slice: pixel pair lc & 3 of window row lc >> 2; nothing lies outside the copy
                    b_base[i] = ((img * j.stem_hp + p * j.sh + (lc >> 2)) * j.stem_wp + q * j.sw + 2 * (lc & 3)) * 8;
                    b_mask[i] = in ? CHUNK_NONE : WINDOW_NONE;
                    continue;
                }
                const int ih0 = p * j.sh - j.ph, iw0 = q * j.sw - j.pw;
                b_base[i] = window_offset(img, ih0, iw0, j.H, j.W, j.C);
                b_mask[i] = window_mask(in, ih0, iw0, j.R, j.S, j.H, j.W);
            }
        }
        // The slices one after the other.  The loading waves are on the path of every stage, so the addresses are there before the barrier, and the
        // next slice's are worked out behind the loads.  (A copy of the code for each way to find a chunk; within it, one: a launch of
        // this kernel finds the instruction cache cold.)
        auto send = [&](auto way_c) __attribute__((always_inline)) {
            constexpr int WAY = decltype(way_c)::value;
            // wave-uniform position of this wave's next slice: its number, its filter row (LONG) and chunk in the row, its filters' offset, its place in the ring
            int ld_s = lg, ld_r = 0, ld_j0 = 0, soff_a = 0, ld_slot = lg;
            auto next_slice = [&]() __attribute__((always_inline)) {
                ld_j0 += 8;
                soff_a += 128;
                if (WAY == POINTWISE) return;
                if (WAY == LONG ? ld_j0 >= j.row_chunks : ld_j0 == j.row_chunks) {
                    ld_j0 = WAY == LONG ? ld_j0 - j.row_chunks : 0;
                    ++ld_r;
                    soff_a += (j.run_chunks - j.row_chunks) * 16;
                }
            };
            if (lg) next_slice();
            const unsigned tab_rd = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)table + lc * 8;
            auto entry = [&]() __attribute__((always_inline)) {
                if constexpr (WAY == TABLE) return ds_read8(tab_rd + ld_s * 64);
                else if constexpr (WAY == POINTWISE) return u32x2{chunk_offset(0, ld_j0 + lc, 0, 0), chunk_mask(ld_j0 + lc < j.c8, 0, 0)};
                else {                                   // chunk ld_j0 + lc of row ld_r, or of the row behind it where the slices run on
                    const int jl = ld_j0 + lc, over = jl >= j.row_chunks, jr = over ? jl - j.row_chunks : jl, r = ld_r + over;
                    const int s = j.c8 == 1 ? jr : (int)__umulhi((unsigned)jr, j.magic_c8);
                    return u32x2{chunk_offset(ld_r, jr, j.W, j.C) + (over ? chunk_offset(1, 0, j.W, j.C) : 0u), chunk_mask(r < j.R && jr < j.run_chunks, r, s)};
                }
            };
            if (WAY == TABLE) ring_barrier();            // the table is complete
            u32x2 e = entry();
            for (int k = 1 - NS; k + NS - 1 < stages; ++k) {
                if (WAY == TABLE) { wait_lgkm<0>(); touch(e); }
                int va[A_PER], vb[B_PER];
                const bool ok = chunk_exists(e[1]);
#pragma unroll
                for (int i = 0; i < A_PER; ++i) { va[i] = ok ? a_voff[i] : OOB; keep(va[i]); }
#pragma unroll
                for (int i = 0; i < B_PER; ++i) { vb[i] = (b_mask[i] & e[1]) == 0 ? (int)(b_base[i] + e[0]) : OOB; keep(vb[i]); }
                // A stage's slice beyond the last one begins behind the filters, and of few filters behind the whole tensor: OOB is only sure to be
                // out of range beside a scalar offset inside the buffer, since the hardware compares with the bytes that are left behind that.
                const int soff = min(soff_a, j.w_bytes);
                unsigned char* const sa = ring + ld_slot * SLICE + lw * 1024;
                unsigned char* const sb = sa + BM * 128;
                if (k >= 0) {
                    wait_vmcnt<(NS - 2) * L>();
                    ring_barrier();
                }
#pragma unroll
                for (int i = 0; i < A_PER; ++i) load_to_lds16(rw, sa + i * 4096, va[i], soff);
#pragma unroll
                for (int i = 0; i < B_PER; ++i) load_to_lds16(rx, sb + i * 4096, vb[i], 0);
                ld_s += LG;
                if (WAY == TABLE) e = entry();           // (after the last slice: entries of the table that nobody uses)
#pragma unroll
                for (int v = 0; v < LG; ++v) next_slice();
                if (WAY != TABLE) e = entry();
                ld_slot = ld_slot + LG == NS * G + lg ? lg : ld_slot + LG;
            }
            if (WAY == TABLE) { wait_lgkm<0>(); touch(e); }      // (the registers of the entry read ahead stay its own until it has arrived)
        };
        if (j.pointwise) send(IC<POINTWISE>{});
        else if (j.tabled) send(IC<TABLE>{});
        else send(IC<LONG>{});
        // the last two stages, already on their way
        if (stages > 1) { wait_vmcnt<L>(); ring_barrier(); }
        wait_vmcnt<0>();
        ring_barrier();
        return;
    }

    // ---- the table: entry e = 8 slice + chunk of the slice
    if (j.tabled) {
        for (int e = tid; e < stages * G * 8; e += CW * 64)
            table[e] = chunk_entry(e, j.R, j.W, j.C, j.c8, j.run_chunks, j.row_chunks, j.magic_row, j.magic_c8, j.stem_wp != 0);
        ring_barrier();
    }

    // ---- multiplying: blocks of 16 filters x 16 pixels, 32 elements of the contraction per instruction: lane = row lane & 15 of either operand,
    // eight elements from 8 (lane >> 4) on; result register v = filter 4 (lane >> 4) + v of pixel lane & 15
    const int quad = lane >> 4, l16 = lane & 15, m0 = (wave % WM) * TM * 16, n0 = (wave / WM) * TN * 16;
    const int m_lane = mt * BM + m0 + quad * 4, n_lane = nt * BN + n0 + l16;
    f32x4 bias[TM];
    u32x2 res[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        bias[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j.vec && j.bias && m_lane + i * 16 < j.K) bias[i] = *reinterpret_cast<const f32x4*>(j.bias + m_lane + i * 16);       // (vec: whole groups of 8 filters)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            const int n = n_lane + jn * 16;
            res[i][jn] = u32x2{0u, 0u};
            if (j.vec && j.res && n < j.Ng && m_lane + i * 16 < j.K) res[i][jn] = *reinterpret_cast<const u32x2*>(j.res + (size_t)n * j.res_ctot + m_lane + i * 16);
        }
    }
    const unsigned ring_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
    const unsigned lane_x = (quad << 4) ^ (((l16 >> 1) & 7) << 4);
    const unsigned a_rd = ring_lds + (m0 + l16) * 128 + lane_x, b_rd = ring_lds + BM * 128 + (n0 + l16) * 128 + lane_x;
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) acc[i][jn] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 fa[2 * G][TM], fb[2 * G][TN], na[2 * G][TM], nb[2 * G][TN];
    auto multiply = [&](int n) __attribute__((always_inline)) {             // the first n slices of the stage in registers
#pragma unroll
        for (int ks = 0; ks < 2 * G; ++ks) {
            if (ks >= 2 && ks % 2 == 0 && ks / 2 >= n) break;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jn = 0; jn < TN; ++jn)
                    acc[i][jn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[ks][i]), __builtin_bit_cast(bf16x8, fb[ks][jn]), acc[i][jn], 0, 0, 0);
        }
    };
    int stage = 0;
    for (int k = 0; k < stages; ++k) {
        ring_barrier();
#pragma unroll
        for (int ks = 0; ks < 2 * G; ++ks) {
            const unsigned at = stage * STAGE + (ks >> 1) * SLICE;
            const unsigned pa = (a_rd + at) ^ ((ks & 1) * 64), pb = (b_rd + at) ^ ((ks & 1) * 64);
            na[ks][0] = ds_read16<0>(pa);
            if constexpr (TM > 1) na[ks][1] = ds_read16<2048>(pa);
            nb[ks][0] = ds_read16<0>(pb);
            if constexpr (TN > 1) nb[ks][1] = ds_read16<2048>(pb);
        }
        if (k) multiply(G);
        wait_lgkm<0>();
#pragma unroll
        for (int ks = 0; ks < 2 * G; ++ks) {
#pragma unroll
            for (int i = 0; i < TM; ++i) { touch(na[ks][i]); fa[ks][i] = na[ks][i]; }
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) { touch(nb[ks][jn]); fb[ks][jn] = nb[ks][jn]; }
        }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    multiply(slices - (stages - 1) * G);                     // (slices beyond the last were sent as zeros)

    // ---- the store: a lane has four consecutive filters of a pixel
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int mb = m_lane + i * 16;
        if (mb >= j.K) continue;
        const bool s1 = mb >= j.split_end[0], s2 = mb >= j.split_end[1], s3 = mb >= j.split_end[2];      // (ends: multiples of 8)
        uint16_t* const base = s3 ? j.y_seg[3] : s2 ? j.y_seg[2] : s1 ? j.y_seg[1] : j.y_seg[0];
        const int ctot = s3 ? j.ctot_seg[3] : s2 ? j.ctot_seg[2] : s1 ? j.ctot_seg[1] : j.ctot_seg[0];
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            const int n = n_lane + jn * 16;
            if (n >= j.Ng) continue;
            uint16_t* const yb = base + (size_t)n * ctot;
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = acc[i][jn][e];
            if (j.vec) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] += bias[i][e];
                if (j.res) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        o[2 * e] += __uint_as_float(res[i][jn][e] << 16);
                        o[2 * e + 1] += __uint_as_float(res[i][jn][e] & 0xFFFF0000u);
                    }
                }
                if (j.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = fmaxf(o[e], 0.f);
                }
                *reinterpret_cast<u32x2*>(yb + mb) = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
                continue;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (mb + e >= j.K) break;
                float v = o[e] + (j.bias ? j.bias[mb + e] : 0.f);
                if (j.res) v += bf16_to_f32(j.res[(size_t)n * j.res_ctot + mb + e]);
                if (j.relu) v = fmaxf(v, 0.f);
                yb[mb + e] = f32_to_bf16(v);
            }
        }
    }
}

SmallJob small_job(const ConvSmall& c, int bm, int bn, int nth)
{
    const ConvGeom& g = c.g;
    SmallJob j{};
    j.x = (const uint16_t*)c.x; j.w = (const uint16_t*)c.w; j.bias = c.bias; j.res = (const uint16_t*)c.res;
    j.res_ctot = g.res_ctot;
    j.C = g.C; j.H = g.H; j.W = g.W; j.K = g.K; j.R = g.R; j.S = g.S; j.sh = g.sh; j.sw = g.sw; j.ph = g.ph; j.pw = g.pw;
    j.P = g.P; j.Q = g.Q; j.Kg = g.Kg; j.Ng = g.Ng; j.relu = g.relu;
    j.c8 = g.C / 8;
    j.m_pq = ((1ull << 40) + (unsigned)(g.P * g.Q) - 1) / (unsigned)(g.P * g.Q);
    j.m_q = ((1ull << 40) + (unsigned)g.Q - 1) / (unsigned)g.Q;
    if (!c.w) {                                          // max-pooling
        j.y_seg[0] = (uint16_t*)c.y;
        j.tiles = (g.Ng * j.c8 + nth - 1) / nth;
        return j;
    }
    j.stem_hp = c.stem_hp; j.stem_wp = c.stem_wp;
    j.x_bytes = c.stem_wp ? (int)((size_t)g.N * c.stem_hp * c.stem_wp * 8) : (int)((size_t)g.N * g.C * g.H * g.W * 2);
    j.w_bytes = (int)((size_t)g.K * g.Kg * 2);
    j.pointwise = g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    j.run_chunks = g.S * j.c8;
    j.slices = chunk_slices(g.R, g.S, g.C, &j.row_chunks);
    j.tabled = !j.pointwise && (j.slices + 3) * 8 <= SMALL_TABLE;      // (+ 3: the last stage's second slice, and one entry read ahead by each group)
    j.magic_c8 = (unsigned)((0x100000000ull + j.c8 - 1) / j.c8);
    j.magic_row = (unsigned)((0x100000000ull + j.row_chunks - 1) / j.row_chunks);
    j.n_tiles = (g.Ng + bn - 1) / bn;
    j.tiles = j.n_tiles * ((g.K + bm - 1) / bm);
    j.vec = g.K % 8 == 0 && aligned16(c.bias) && (!c.res || (g.res_ctot % 8 == 0 && aligned16(c.res)));
    set_destinations(j, c.split, (uint16_t*)c.y, g.y_ctot, g.y_coff);
    if (c.split && c.split->n > 1) {
        for (int d = 0; d < c.split->n; ++d) j.vec = j.vec && c.split->dst[d].ctot % 8 == 0 && c.split->dst[d].c_offset % 8 == 0 && aligned16(c.split->dst[d].y);
    } else {
        j.vec = j.vec && g.y_ctot % 8 == 0 && g.y_coff % 8 == 0 && aligned16(c.y);
    }
    return j;
}

}  // namespace

// Tiles of bm x bn of a group of layers.
static long small_tiles(const ConvSmall* jobs, int n, int bm, int bn)
{
    long t = 0;
    for (int i = 0; i < n; ++i)
        if (jobs[i].w) t += ((long)jobs[i].g.Ng + bn - 1) / bn * ((jobs[i].g.K + bm - 1) / bm);
    return t;
}

// As long as the layer's 64 x 64 tiles fit the device at two workgroups per compute unit, 1x1 filters at one (their contraction is
// short).  Between one tile per compute unit and two, this kernel and the streaming one: 3x3 80 -> 24 on 24 x 26 x 29 6.9 and 8.7 us, 5x5 136 -> 24 on
// 25 x 26 x 37 19.6 and 27.5, 3x3 64 -> 84 on 23 x 25 x 24 10.3 and 10.7, with three slices up to a fifth the other way (3x3 16 -> 20 on 35 x 37 x 58 at
// stride 2 6.8 and 5.5); 1x1 96 -> 22 on 96 x 97 x 2 6.1 and 4.7, 280 -> 21 on 83 x 86 x 3 7.2 and 5.8.  Beyond two: 3x3 64 -> 23 on 34 x 36 x 29
// 13.2 and 8.9, 3x3 104 -> 26 on 29 x 30 x 42 16.6 and 12.6.  Channels: as many as a tap is found exactly for by a multiplication (the kernel's LONG).
bool conv_bf16_small_takes(const ConvGeom& g, const void* x, const void* w)
{
    const long tiles = ((long)g.Ng + 63) / 64 * ((g.K + 63) / 64);
    return conv_bf16_dma_eligible(g, x, w) && (g.R * g.S == 1 || g.C <= 1 << 17) && tiles <= (g.R * g.S > 1 ? 2 : 1) * device_cus();
}

// Several layers whose 64 x 64 tiles are more than five for four compute units are better off side by side in wide tiles (conv_bf16_wide.hip), kernel trace:
// 1x1 .. 3x3 of GoogLeNet's 4a slim on 12 images (333 tiles) 8.2 us here, 7.8 there, on 19 (531) 11.4 and 7.9; 4c on 37 (912) 16.8 and 12.4; 4e fused
// on 12 (333) 11.2 and 10.3; 5b slim on 64 (784) 21.8 and 16.2.  Fewer: 5a slim on 25 (260) 9.3 and 10.2, 4c slim on 12 (296) 8.9 and 9.2, 5b slim on 25 (320)
// 11.3 and 12.6.
bool conv_bf16_small_crowded(const ConvSmall* jobs, int n)
{
    int convs = 0;
    for (int i = 0; i < n; ++i) convs += jobs[i].w != nullptr;
    return convs > 1 && 4 * small_tiles(jobs, n, 64, 64) > 5 * device_cus();
}

template <int TM, int TN, int WM, int WN, int LG>
static int launch_group(const ConvSmall* jobs, int n, hipStream_t st)
{
    constexpr int NTH = (WM * WN + 4 * LG) * 64;
    SmallArgs a{};
    int blocks = 0;
    for (int i = 0; i < SMALL_GROUP_MAX; ++i) {
        a.first[i] = i < n ? blocks : 0x7FFFFFFF;
        if (i >= n) continue;
        a.job[i] = small_job(jobs[i], WM * TM * 16, WN * TN * 16, NTH);
        blocks += (a.job[i].tiles + 7) / 8 * 8;
    }
    hipLaunchKernelGGL((conv_bf16_small_kernel<TM, TN, WM, WN, LG>), dim3((unsigned)blocks), dim3(NTH), 0, st, a);
    return check_launch("conv_bf16_small");
}

// The smallest tile that leaves every compute unit at most one.  Stages of two slices, three in flight; eight loading waves.  Sixteen waves of
// 16 x 16 and 32 x 16 for the larger tiles (64 x 32: blocks of 32 x 16 were no faster).  Two 64 x 64 tiles to a compute unit -- layers that share the
// launch, and by themselves those that wide tiles do not take: four waves of 32 x 32 and four loading ones, three stages of one slice
// (24 -> 88 5x5 on 31 x 45 x 9, when it came here by itself, 7.8 us; eight waves of 32 x 16 8.3; stages of two slices, two in flight 10.6: too few loads on their way).
int launch_conv_bf16_small(const ConvSmall* jobs, int n, hipStream_t st)
{
    if (small_tiles(jobs, n, 32, 32) <= device_cus()) return launch_group<1, 1, 2, 2, 2>(jobs, n, st);
    if (small_tiles(jobs, n, 64, 32) <= device_cus()) return launch_group<1, 1, 4, 2, 2>(jobs, n, st);
    // 1, 3 or 5 slices: half of the last stage of two would be empty, and four waves start sooner than eight (one slice: 1x1 32 -> 528 on 19 x 19 x 15 at
    // stride 2 4.3 us in stages of two, 3.95 so; three: 3x3 16 -> 344 on 41 x 44 4.5 and 4.3; 1x1 at stride 1 3.7 and 3.65; two slices 3.8 and
    // 3.9, four 4.4 and 4.4, six and more the larger stages)
    int most = 0, row_chunks;
    for (int i = 0; i < n; ++i)
        if (jobs[i].w) most = std::max(most, chunk_slices(jobs[i].g.R, jobs[i].g.S, jobs[i].g.C, &row_chunks));
    if (small_tiles(jobs, n, 64, 64) <= device_cus()) return most % 2 && most <= 5 ? launch_group<2, 2, 2, 2, 1>(jobs, n, st) : launch_group<2, 1, 2, 4, 2>(jobs, n, st);
    // a layer by itself: wide tiles, which two to a compute unit beat only by sharing the launch (3x3 144 -> 288 on 14 x 14 x 19 10.8 us here, 10.4 there,
    // 160 -> 320 on 7 x 7 x 128 13.4 and 11.3)
    const ConvSmall& j = jobs[0];
    if (n == 1 && j.w && !j.stem_wp && conv_bf16_wide_takes(j.g, j.x, j.w, j.res, j.y, j.split))
        return launch_conv_bf16_wide(j.g, (const uint16_t*)j.x, (const uint16_t*)j.w, j.bias, (uint16_t*)j.y, st, j.split);
    return launch_group<2, 2, 2, 2, 1>(jobs, n, st);
}

}  // namespace dr
