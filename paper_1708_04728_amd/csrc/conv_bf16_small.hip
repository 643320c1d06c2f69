// bf16 convolution of small layers: few images, or a few hundred to a few thousand output pixels.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (r, s, c)
//
// What bounds such a layer is not arithmetic and not bandwidth but the chain of dependent steps inside one workgroup: the
// streaming kernel (conv_bf16_dma.hip) walks the whole contraction in slices of 64 with a barrier in each, and with a
// tile or less per compute unit every slice costs a trip to the caches (about 0.4 us: 3x3 filters on 112 channels, 16
// slices, 10 us on one image) while most compute units stand idle.  Here
//   * a tile is one 32 x 32 block of the matrix instructions, four times as many workgroups as with 64 x 64 tiles;
//   * the NW = 8 or 4 waves of a workgroup share the CONTRACTION of that tile: wave w takes the w-th share of the slices, with a
//     ring of two slices of its own in LDS, so that no wave waits for another and 16 slices are in flight per compute unit;
//     the partial sums meet in LDS once, are added in wave order (the same bits from run to run) and stored with bias,
//     residual and ReLU applied;
//   * one launch takes several layers (the second steps of an inception module, say): a launch costs 3 to 4 us on a
//     stream whatever it does, as much as the layer itself.  A job may also be a 3x3 max-pooling layer, which a
//     module's pooling branch needs beside the other branches' first steps.
// Measured in chains of dependent launches, streaming kernel -> this one: 3x3 160 -> 320 on one 14 x 14 image 12.4 -> 6.7 us (of
// which 3.3 are the launch), 1x1 832 -> 192 on 7 x 7 6.8 -> 4.5 us; the slim GoogLeNet on one image 272 -> 151 us.
// What bounds it now: a wave's slice takes 0.4 us however many are in flight (8 loads, 8 operand reads and 4 dependent matrix
// instructions of one wave), 15 cycles of the load path per KiB once 8 waves share it.
//
// Operands travel as in the streaming kernel: 16-byte buffer loads that write LDS, lanes outside the tensor or in the padding at
// an offset the hardware answers with zeros, chunk j of row r stored at chunk j ^ ((r >> 1) & 7) so that loads and operand
// reads are free of bank conflicts.
#include "dr_internal.h"
#include "dr_store.h"
#include "conv_bf16_dev.h"

namespace dr {
namespace {

struct SmallJob {
    const uint16_t* x;
    const uint16_t* w;                                   // NULL: a max-pooling layer (3x3)
    const float* bias;
    const uint16_t* res;
    uint16_t* y_seg[4];                                  // destinations of the filter ranges (see ConvSplit), y_seg[0] alone otherwise
    int ctot_seg[4], split_end[3];
    int nsplit, res_ctot;
    int C, H, W, K, R, S, sh, sw, ph, pw, P, Q, Kg, Ng, relu;
    int x_bytes, w_bytes;
    int tap, flat, pointwise;                                       // slices: whole taps (C % 64 == 0); running on from filter row to filter row
    int c8, run_chunks, spr, slices;                     // chunks per tap, per filter row; slices per filter row, per tile
    unsigned magic_c8;
    unsigned long long m_pq, m_q;
    int n_tiles, tiles, first;                           // pixel tiles; tiles in all; first workgroup (a multiple of 8)
    int vec_bias;                                        // the bias can be read 16 bytes at a time
    int vec;                                             // 8-byte stores (and residual reads) are aligned
};
struct SmallArgs {
    int n;
    SmallJob job[SMALL_GROUP_MAX];
};

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

// TM x TN blocks of 32 x 32 per tile, NW waves (shares of the contraction), NS slices in flight per wave.
template <int TM, int TN, int NW, int NS>
__global__ __launch_bounds__(NW * 64) void conv_bf16_small_kernel(const SmallArgs args)
{
    constexpr int A_PER = TM * 4, B_PER = TN * 4, L = A_PER + B_PER, STAGE = L * 1024, BM = TM * 32, BN = TN * 32;
    static_assert(TM * TN * 4096 <= NS * STAGE && NS >= 1 && NS <= 4 && (NS - 1) * L < 63, "bad configuration");
    __shared__ __attribute__((aligned(1024))) unsigned char ring[NW * NS * STAGE];

    // ---- the job and the tile.  Workgroup b runs on die b & 7; a die takes a contiguous range of tiles, filter block by filter
    // block, so that the pixel tiles of one filter block read it from one L2.
    int ji = 0;
    while (ji + 1 < args.n && (int)blockIdx.x >= args.job[ji + 1].first) ++ji;
    const SmallJob& j = args.job[ji];
    const int b = (int)blockIdx.x - j.first, die = b & 7, s_die = b >> 3, per = j.tiles >> 3, odd = j.tiles & 7;
    if (s_die >= per + (die < odd ? 1 : 0)) return;
    const int t = die * per + min(die, odd) + s_die;
    if (!j.w) { pool_items(j, t); return; }
    const int mt = t / j.n_tiles, nt = t - mt * j.n_tiles;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned ring_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
    unsigned char* const my_ring = ring + wave * (NS * STAGE);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)j.x, 0, j.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)j.w, 0, j.w_bytes, 0x00020000);

    // ---- loader: pass i fills rows 8 i .. 8 i + 7 of an operand; the lane's row there is 8 i + lrow and its chunk lc[i & 1]
    const int lrow = lane >> 3;
    const int lc[2] = {(lane & 7) ^ (lrow >> 1), (lane & 7) ^ (lrow >> 1) ^ 4};
    int a_voff[A_PER], b_base[B_PER];
    unsigned b_mask[B_PER];                              // bits 0..15: tap s is OUTSIDE the image row; bits 16..31: filter row r is inside
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
        const int m = mt * BM + i * 8 + lrow;
        a_voff[i] = m < j.K ? (m * j.Kg + lc[i & 1] * 8) * 2 : OOB;
    }
    if (j.pointwise) {                                   // output pixel n reads input pixel n
#pragma unroll
        for (int i = 0; i < B_PER; ++i) {
            const int n = nt * BN + i * 8 + lrow;
            b_base[i] = (n * j.C + lc[i & 1] * 8) * 2;
            b_mask[i] = n < j.Ng ? 0x1FFFEu : 0xFFFFu;
        }
    } else {
#pragma unroll
        for (int i = 0; i < B_PER; ++i) {
            const int n = nt * BN + i * 8 + lrow;
            const bool in = n < j.Ng;
            const int nn = in ? n : 0;
            const int img = div_small(nn, j.m_pq), pix = nn - img * j.P * j.Q, p = div_small(pix, j.m_q), q = pix - p * j.Q;
            const int ih0 = p * j.sh - j.ph, iw0 = q * j.sw - j.pw;
            b_base[i] = (((img * j.H + ih0) * j.W + iw0) * j.C + lc[i & 1] * 8) * 2;
            const unsigned wv = bit_range(max(0, -iw0), min(j.S - 1, j.W - 1 - iw0));
            const unsigned hv = in ? bit_range(max(0, -ih0), min(j.R - 1, j.H - 1 - ih0)) : 0u;
            b_mask[i] = (~wv & 0xFFFFu) | (hv << 16);
        }
    }

    // ---- this wave's slices and the cursor of the next one to load
    const int s0 = j.slices * wave / NW, count = j.slices * (wave + 1) / NW - s0;
    int ld_r, ld_s = 0, ld_j0;                           // filter row, tap (tap mode), first chunk of the slice in the tap / row
    if (j.tap) {
        const int per_tap = j.c8 >> 3, tap = s0 / per_tap;
        ld_j0 = (s0 - tap * per_tap) * 8;
        ld_r = tap / j.S; ld_s = tap - ld_r * j.S;
    } else if (j.flat) {
        ld_r = s0 * 8 / j.run_chunks; ld_j0 = s0 * 8 - ld_r * j.run_chunks;
    } else {
        ld_r = s0 / j.spr; ld_j0 = (s0 - ld_r * j.spr) * 8;
    }
    auto issue_slice = [&](int stage) __attribute__((always_inline)) {
        unsigned char* sa = my_ring + stage * STAGE;
        unsigned char* sb = sa + A_PER * 1024;
        if (j.tap) {
            const int soff_a = ((ld_r * j.S + ld_s) * j.c8 + ld_j0) * 16, off = (ld_r * j.W + ld_s) * j.C * 2 + ld_j0 * 16;
            const unsigned want = 1u << (16 + ld_r), sel = want | (1u << ld_s);
#pragma unroll
            for (int i = 0; i < A_PER; ++i) load_to_lds16(rw, sa + i * 1024, a_voff[i], soff_a);
#pragma unroll
            for (int i = 0; i < B_PER; ++i) load_to_lds16(rx, sb + i * 1024, (b_mask[i] & sel) == want ? b_base[i] + off : OOB, 0);
            ld_j0 += 8;
            if (ld_j0 == j.c8) {
                ld_j0 = 0;
                if (++ld_s == j.S) { ld_s = 0; ++ld_r; }
            }
            return;
        }
        // slices along a filter row's run of S C values; with `flat` they run on into the next row, whose filters follow in memory
        const int soff_a = (ld_r * j.run_chunks + ld_j0) * 16, run_off = ld_r * j.W * j.C * 2 + ld_j0 * 16;
        const int wrap_off = (j.W * j.C - j.run_chunks * 8) * 2;
        const bool more = j.flat && ld_r + 1 < j.R;
        int sh[2], off[2];
        bool wrap[2], ok[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int jl0 = ld_j0 + lc[e];
            wrap[e] = jl0 >= j.run_chunks;
            ok[e] = !wrap[e] || more;
            const int jl = wrap[e] ? jl0 - j.run_chunks : jl0;
            sh[e] = 31 - (j.c8 == 1 ? jl : (int)__umulhi((unsigned)jl, j.magic_c8));     // the chunk's tap, at most 15 where it counts
            off[e] = run_off + (wrap[e] ? wrap_off : 0);
        }
        const int bit = 16 + ld_r, next_bit = (17 + ld_r) & 31;
#pragma unroll
        for (int i = 0; i < A_PER; ++i) load_to_lds16(rw, sa + i * 1024, ok[i & 1] ? a_voff[i] : OOB, soff_a);
#pragma unroll
        for (int i = 0; i < B_PER; ++i) {
            const bool row_in = (b_mask[i] >> (wrap[i & 1] ? next_bit : bit)) & 1u;
            const bool tap_out = (b_mask[i] << sh[i & 1]) & 0x80000000u;
            load_to_lds16(rx, sb + i * 1024, ok[i & 1] && row_in && !tap_out ? b_base[i] + off[i & 1] : OOB, 0);
        }
        ld_j0 += 8;
        if (ld_j0 >= j.run_chunks) { ld_j0 = j.flat ? ld_j0 - j.run_chunks : 0; ++ld_r; }
    };
    // (one copy of the loader's code, here and in the loop: a launch of this kernel finds the instruction cache cold)
    // ---- what the store needs, requested while the slices travel.  A tile's 4 TM TN groups of 8 filters x 32 pixels go round the
    // waves; group u is filters 8 (u % 4) of block (u / 4 % TM, u / 4 / TM)
    constexpr int UNITS = 4 * TM * TN, PER = (UNITS + NW - 1) / NW;
    f32x4 bias[PER];
    uint2 res[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int u = wave + k * NW, blk = u >> 2, n = nt * BN + blk / TM * 32 + l32, m0 = mt * BM + blk % TM * 32 + (u & 3) * 8 + half * 4;
        bias[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        res[k] = make_uint2(0u, 0u);
        if (u < UNITS && n < j.Ng && m0 < j.K) {
            if (j.vec_bias) bias[k] = *reinterpret_cast<const f32x4*>(j.bias + m0);
            if (j.res && j.vec && m0 + 3 < j.K) res[k] = *reinterpret_cast<const uint2*>(j.res + (size_t)n * j.res_ctot + m0);
        }
    }

    // ---- the wave's share of the contraction
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][jn][v] = 0.f;
    const unsigned lane_x = (half << 4) ^ (((l32 >> 1) & 7) << 4);
    const unsigned a_rd = ring_lds + wave * (NS * STAGE) + l32 * 128 + lane_x;
    int stage = 0, ld_stage = 0;
    for (int k = 1 - NS; k < count; ++k) {
        if (k + NS - 1 < count) {
            issue_slice(ld_stage);
            ld_stage = ld_stage + 1 == NS ? 0 : ld_stage + 1;
        }
        if (k < 0) continue;
        const unsigned pa = a_rd + stage * STAGE, pb = pa + A_PER * 1024;
        // slice k has landed; the loads of the slices behind it may be pending
        const int behind = min(count - 1 - k, NS - 1);
        if (NS > 3 && behind == 3) wait_vmcnt<(NS > 3 ? 3 : 0) * L>();
        else if (NS > 2 && behind == 2) wait_vmcnt<(NS > 2 ? 2 : 0) * L>();
        else if (NS > 1 && behind == 1) wait_vmcnt<(NS > 1 ? 1 : 0) * L>();
        else wait_vmcnt<0>();
        u32x4 fa[4][TM], fb[4][TN];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            fa[ks][0] = ds_read16<0>(pa ^ (ks * 32));
            if constexpr (TM > 1) fa[ks][1] = ds_read16<4096>(pa ^ (ks * 32));
            fb[ks][0] = ds_read16<0>(pb ^ (ks * 32));
            if constexpr (TN > 1) fb[ks][1] = ds_read16<4096>(pb ^ (ks * 32));
        }
        auto step = [&](auto ks_c) __attribute__((always_inline)) {
            constexpr int KS = decltype(ks_c)::value;
            wait_lgkm<(3 - KS) * (TM + TN)>();
#pragma unroll
            for (int i = 0; i < TM; ++i) touch(fa[KS][i]);
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) touch(fb[KS][jn]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jn = 0; jn < TN; ++jn)
                    acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[KS][i]), __builtin_bit_cast(bf16x8, fb[KS][jn]), acc[i][jn], 0, 0, 0);
        };
        step(IC<0>{}); step(IC<1>{}); step(IC<2>{}); step(IC<3>{});
        stage = stage + 1 == NS ? 0 : stage + 1;
    }

    // ---- the partial sums meet: registers 4 g .. 4 g + 3 of a lane (filters 8 g + 4 half ..) at [wave][block][g][lane]
    f32x4* const mine = reinterpret_cast<f32x4*>(my_ring);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                mine[((jn * TM + i) * 4 + g) * 64 + lane] = f32x4{acc[i][jn][4 * g], acc[i][jn][4 * g + 1], acc[i][jn][4 * g + 2], acc[i][jn][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int u = wave + k * NW, blk = u >> 2, n = nt * BN + blk / TM * 32 + l32, m0 = mt * BM + blk % TM * 32 + (u & 3) * 8 + half * 4;
        if (u >= UNITS || n >= j.Ng || m0 >= j.K) continue;
        f32x4 o = reinterpret_cast<const f32x4*>(ring)[u * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) o += reinterpret_cast<const f32x4*>(ring + w * (NS * STAGE))[u * 64 + lane];
        if (j.vec_bias) o += bias[k];
        else if (j.bias)
            for (int e = 0; e < 4 && m0 + e < j.K; ++e) o[e] += j.bias[m0 + e];
        uint16_t* yb = j.y_seg[0] + (size_t)n * j.ctot_seg[0];
        if (j.nsplit > 1) {
            const bool s1 = m0 >= j.split_end[0], s2 = m0 >= j.split_end[1], s3 = m0 >= j.split_end[2];
            uint16_t* base = s3 ? j.y_seg[3] : s2 ? j.y_seg[2] : s1 ? j.y_seg[1] : j.y_seg[0];
            yb = base + (size_t)n * (s3 ? j.ctot_seg[3] : s2 ? j.ctot_seg[2] : s1 ? j.ctot_seg[1] : j.ctot_seg[0]);
        }
        if (j.vec && m0 + 3 < j.K) {
            o[0] += __uint_as_float(res[k].x << 16); o[1] += __uint_as_float(res[k].x & 0xFFFF0000u);
            o[2] += __uint_as_float(res[k].y << 16); o[3] += __uint_as_float(res[k].y & 0xFFFF0000u);
            if (j.relu) {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = fmaxf(o[e], 0.f);
            }
            *reinterpret_cast<uint2*>(yb + m0) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
            continue;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (m0 + e >= j.K) break;
            float v = o[e];
            if (j.res) v += bf16_to_f32(j.res[(size_t)n * j.res_ctot + m0 + e]);
            if (j.relu) v = fmaxf(v, 0.f);
            yb[m0 + e] = f32_to_bf16(v);
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
    for (int d = 0; d < 3; ++d) j.split_end[d] = 0x7FFFFFFF;
    if (!c.w) {                                          // max-pooling
        j.y_seg[0] = (uint16_t*)c.y;
        j.tiles = (g.Ng * j.c8 + nth - 1) / nth;
        return j;
    }
    j.x_bytes = (int)((size_t)g.N * g.C * g.H * g.W * 2);
    j.w_bytes = (int)((size_t)g.K * g.Kg * 2);
    j.tap = g.C % 64 == 0;
    j.pointwise = g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    j.run_chunks = g.S * j.c8;
    j.spr = (j.run_chunks + 7) / 8;
    j.slices = g.R * j.spr;
    const int flat_slices = (g.R * j.run_chunks + 7) / 8;
    if (!j.tap && j.run_chunks >= 8 && flat_slices < j.slices) { j.flat = 1; j.slices = flat_slices; }
    j.magic_c8 = (unsigned)((0x100000000ull + j.c8 - 1) / j.c8);
    j.n_tiles = (g.Ng + bn - 1) / bn;
    j.tiles = j.n_tiles * ((g.K + bm - 1) / bm);
    j.vec_bias = c.bias && g.K % 4 == 0 && ((uintptr_t)c.bias & 15) == 0;
    j.nsplit = c.split && c.split->n > 1 ? c.split->n : 0;
    j.vec = !c.res || (g.res_ctot % 4 == 0 && ((uintptr_t)c.res & 7) == 0);
    auto dest = [&](int d, uint16_t* y, int ctot, int coff, int start) {
        j.y_seg[d] = y + coff - start;
        j.ctot_seg[d] = ctot;
        j.vec = j.vec && ctot % 4 == 0 && coff % 4 == 0 && start % 4 == 0 && ((uintptr_t)y & 7) == 0;
    };
    if (j.nsplit) {
        int start = 0;
        for (int d = 0; d < j.nsplit; ++d) {
            dest(d, (uint16_t*)c.split->dst[d].y, c.split->dst[d].ctot, c.split->dst[d].c_offset, start);
            start += c.split->dst[d].k;
            if (d + 1 < j.nsplit) j.split_end[d] = start;
        }
    } else {
        dest(0, (uint16_t*)c.y, g.y_ctot, g.y_coff, 0);
    }
    return j;
}

}  // namespace

// 32 x 32 tiles of a layer
static long small_tiles(const ConvGeom& g) { return ((long)g.Ng + 31) / 32 * ((g.K + 31) / 32); }

// Several taps: as long as the tiles fit the device at two workgroups of four waves per compute unit (measured in a chain of
// dependent launches, 3x3 filters on 96..160 channels, streaming kernel -> this one: 28 x 28 x 3 images, 296 and 444 tiles,
// 9.4 -> 7.6 us; 14 x 14 x 8 images, 490 tiles, 12.5 -> 9.6 us; 666 tiles 9.2 -> 11.3 us).
// 1x1 filters: the contraction has to be long enough to be worth sharing (480 channels 6.2 -> 4.5 us, 192 channels
// 3.8 -> 4.2 us), and the line is drawn by pixels alone so that it does not depend on how filters are banked together.
bool conv_bf16_small_takes(const ConvGeom& g, const void* x, const void* w)
{
    if (!conv_bf16_dma_eligible(g, x, w)) return false;
    if (g.R * g.S == 1) return g.Ng <= 1024 && g.C > 256;
    return small_tiles(g) <= 2 * device_cus();
}

template <int TM, int TN, int NW, int NS>
static int launch_group(const ConvSmall* jobs, int n, hipStream_t st)
{
    SmallArgs a{};
    a.n = n;
    int blocks = 0;
    for (int i = 0; i < n; ++i) {
        a.job[i] = small_job(jobs[i], TM * 32, TN * 32, NW * 64);
        a.job[i].first = blocks;
        blocks += (a.job[i].tiles + 7) / 8 * 8;
    }
    hipLaunchKernelGGL((conv_bf16_small_kernel<TM, TN, NW, NS>), dim3((unsigned)blocks), dim3(NW * 64), 0, st, a);
    return check_launch("conv_bf16_small");
}

int launch_conv_bf16_small(const ConvSmall* jobs, int n, hipStream_t st)
{
    // eight shares while there is at most one tile per compute unit, else four, which leave room for a second workgroup;
    // 1x1 filters always four (the sums must not depend on what else is in the group)
    long tiles = 0;
    bool pointwise = false;
    for (int i = 0; i < n; ++i)
        if (jobs[i].w) { tiles += small_tiles(jobs[i].g); pointwise = pointwise || jobs[i].g.R * jobs[i].g.S == 1; }
    return tiles <= device_cus() && !pointwise ? launch_group<1, 1, 8, 2>(jobs, n, st) : launch_group<1, 1, 4, 2>(jobs, n, st);
}

}  // namespace dr
