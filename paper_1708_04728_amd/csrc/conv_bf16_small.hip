// bf16 convolution of small layers: few images, or a few thousand output pixels.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (r, s, c)
//
// What bounds such a layer is not arithmetic and not bandwidth but the chain of dependent steps inside one workgroup: the
// streaming kernel (conv_bf16_dma.hip) walks the contraction in slices of 64, and with a tile or less per compute unit every
// slice costs it 0.4 us (its waves send the slice's loads, wait for older ones, meet, read operands and multiply one after
// the other) while most compute units stand idle.  Here
//   * the tile is as small as the layer leaves compute units for: 32 x 32, 64 x 32 or 64 x 64;
//   * one wave per 32 x 32 block multiplies and does nothing else; four other waves send the loads.  They meet once per slice.
//     The slices are multiplied in the same order as in the streaming kernel, so the results are the same bits.  (Sharing the
//     contraction among eight waves was faster still, 6.2 against 8.9 us on the layer below, but adds the products in
//     another order: a few outputs in ten thousand round the other way, and 25 layers later the class probabilities of
//     GoogLeNet differ by 1 to 3 %.)
//   * one launch takes several layers (the second steps of an inception module, say): a launch costs 3 to 4 us on a
//     stream whatever it does, as much as the layer itself.  A job may also be a 3x3 max-pooling layer, which a
//     module's pooling branch needs beside the other branches' first steps.
// Measured in chains of dependent launches, streaming kernel -> this one: 3x3 160 -> 320 on one 14 x 14 image 12.3 -> 8.9 us (of
// which 3.3 are the launch), 5x5 32 -> 512 9.0 -> 5.9 us, 1x1 832 -> 624 on 7 x 7 7.3 -> 5.6 us, 3x3 96 -> 128 on 28 x 28 x 8
// 9.4 -> 8.2 us; the slim GoogLeNet on one image, wall time of a pass among others, 272 -> 151 us.
// What bounds it now: about 0.2 us per slice -- a wave takes 300 cycles to read a slice's 8 KB of operands from LDS and a load that
// writes LDS takes its sender about 50, so neither more slices in flight nor eight loading waves nor reads dealt out between
// the matrix instructions made it faster.
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
    int stem_hp, stem_wp;                                // padded 4-channel input copy (see launch_conv_bf16_stem), 0: ordinary input
    int tap, flat, pointwise;                                       // slices: whole taps (C % 64 == 0); running on from filter row to filter row
    int c8, run_chunks, spr, slices;                     // chunks per tap, per filter row; slices per filter row, per tile
    unsigned magic_c8;
    unsigned long long m_pq, m_q;
    int n_tiles, tiles, first;                           // pixel tiles; tiles in all; first workgroup (a multiple of 8)
    int vec;                                             // whole groups of 8 filters, 16-byte accesses of output, residual and bias aligned
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

// CM x CN multiplying waves with one block of 32 x 32 each, four loading waves, NS slices in LDS.
template <int CM, int CN, int NS>
__global__ __launch_bounds__((CM * CN + 4) * 64) void conv_bf16_small_kernel(const SmallArgs args)
{
    constexpr int CW = CM * CN, LW = 4, BM = CM * 32, BN = CN * 32, A_PER = CM, B_PER = CN, L = A_PER + B_PER, STAGE = (BM + BN) * 128;
    static_assert((NS - 1) * L < 63, "loads in flight");
    __shared__ __attribute__((aligned(1024))) unsigned char ring[NS * STAGE];

    // ---- the job and the tile.  Workgroup b runs on die b & 7; a die takes a contiguous range of tiles, filter block by filter
    // block, so that the pixel tiles of one filter block read it from one L2.  (The job is copied: left in the argument
    // buffer, every field would be read again behind each wait.)
    int ji = 0;
    while (ji + 1 < args.n && (int)blockIdx.x >= args.job[ji + 1].first) ++ji;
    const SmallJob j = args.job[ji];
    const int b = (int)blockIdx.x - j.first, die = b & 7, s_die = b >> 3, per = j.tiles >> 3, odd = j.tiles & 7;
    if (s_die >= per + (die < odd ? 1 : 0)) return;
    const int t = die * per + min(die, odd) + s_die;
    if (!j.w) { pool_items(j, t); return; }
    const int mt = t / j.n_tiles, nt = t - mt * j.n_tiles;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slices = j.slices;

    // Iteration k, for every wave: at the barrier slice k has landed and slice k - 1 has been read; behind it the multiplying waves
    // read slice k and multiply slice k - 1, the loading waves send slice k + NS - 1 into the stage slice k - 1 has left.
    if (wave >= CW) {
        // ---- loading: pass i of this wave fills rows 32 i + lrow of an operand
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)j.x, 0, j.x_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)j.w, 0, j.w_bytes, 0x00020000);
        const int lw = wave - CW, lrow = lw * 8 + (lane >> 3), lc = (lane & 7) ^ ((lrow >> 1) & 7);
        int a_voff[A_PER], b_base[B_PER];
        unsigned b_mask[B_PER];                          // bits 0..15: tap s is OUTSIDE the image row; bits 16..31: filter row r is inside
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
                b_base[i] = (n * j.C + lc * 8) * 2;
                b_mask[i] = in ? 0x1FFFEu : 0xFFFFu;
            } else {
                const int nn = in ? n : 0;
                const int img = div_small(nn, j.m_pq), pix = nn - img * j.P * j.Q, p = div_small(pix, j.m_q), q = pix - p * j.Q;
                if (j.stem_wp) {                         // chunk lc of a slice: pixel pair lc & 3 of window row lc >> 2; nothing lies outside the copy
                    b_base[i] = ((img * j.stem_hp + p * j.sh + (lc >> 2)) * j.stem_wp + q * j.sw + 2 * (lc & 3)) * 8;
                    b_mask[i] = in ? 0xFFFFFEu : 0xFFFFu;
                    continue;
                }
                const int ih0 = p * j.sh - j.ph, iw0 = q * j.sw - j.pw;
                b_base[i] = (((img * j.H + ih0) * j.W + iw0) * j.C + lc * 8) * 2;
                const unsigned wv = bit_range(max(0, -iw0), min(j.S - 1, j.W - 1 - iw0));
                const unsigned hv = in ? bit_range(max(0, -ih0), min(j.R - 1, j.H - 1 - ih0)) : 0u;
                b_mask[i] = (~wv & 0xFFFFu) | (hv << 16);
            }
        }
        int ld_r = 0, ld_s = 0, ld_j0 = 0, ld_stage = 0;     // filter row, tap (tap mode), first chunk of the next slice in the tap / row
        auto issue_slice = [&]() __attribute__((always_inline)) {
            unsigned char* sa = ring + ld_stage * STAGE + lw * 1024;
            unsigned char* sb = sa + BM * 128;
            ld_stage = ld_stage + 1 == NS ? 0 : ld_stage + 1;
            if (j.tap) {
                const int soff_a = ((ld_r * j.S + ld_s) * j.c8 + ld_j0) * 16, off = (ld_r * j.W + ld_s) * j.C * 2 + ld_j0 * 16;
                const unsigned want = 1u << (16 + ld_r), sel = want | (1u << ld_s);
#pragma unroll
                for (int i = 0; i < A_PER; ++i) load_to_lds16(rw, sa + i * 4096, a_voff[i], soff_a);
#pragma unroll
                for (int i = 0; i < B_PER; ++i) load_to_lds16(rx, sb + i * 4096, (b_mask[i] & sel) == want ? b_base[i] + off : OOB, 0);
                ld_j0 += 8;
                if (ld_j0 == j.c8) {
                    ld_j0 = 0;
                    if (++ld_s == j.S) { ld_s = 0; ++ld_r; }
                }
                return;
            }
            // slices along a filter row's run of S C values; with `flat` they run on into the next row, whose filters follow in memory
            const int soff_a = (ld_r * j.run_chunks + ld_j0) * 16, run_off = ld_r * j.W * j.C * 2 + ld_j0 * 16;
            const bool more = j.flat && ld_r + 1 < j.R;
            const int jl0 = ld_j0 + lc;
            const bool wrap = jl0 >= j.run_chunks, ok = !wrap || more;
            const int jl = wrap ? jl0 - j.run_chunks : jl0;
            const int sh = 31 - (j.c8 == 1 ? jl : (int)__umulhi((unsigned)jl, j.magic_c8));     // the chunk's tap, at most 15 where it counts
            const int off = run_off + (wrap ? (j.W * j.C - j.run_chunks * 8) * 2 : 0);
            const int bit = (16 + ld_r + (wrap ? 1 : 0)) & 31;
#pragma unroll
            for (int i = 0; i < A_PER; ++i) load_to_lds16(rw, sa + i * 4096, ok ? a_voff[i] : OOB, soff_a);
#pragma unroll
            for (int i = 0; i < B_PER; ++i) {
                const bool row_in = (b_mask[i] >> bit) & 1u, tap_out = (b_mask[i] << sh) & 0x80000000u;
                load_to_lds16(rx, sb + i * 4096, ok && row_in && !tap_out ? b_base[i] + off : OOB, 0);
            }
            ld_j0 += 8;
            if (ld_j0 >= j.run_chunks) { ld_j0 = j.flat ? ld_j0 - j.run_chunks : 0; ++ld_r; }
        };
        // (one copy of the loader's code: a launch of this kernel finds the instruction cache cold)
        for (int k = 1 - NS; k <= slices; ++k) {
            if (k >= 0) {
                const int behind = min(slices - 1 - k, NS - 2);      // slices requested behind slice k
                if (behind == NS - 2) wait_vmcnt<(NS - 2) * L>();
                else if (NS > 4 && behind >= NS / 2) wait_vmcnt<(NS > 4 ? NS / 2 : 0) * L>();
                else if (NS > 3 && behind >= 2) wait_vmcnt<(NS > 3 ? 2 : 0) * L>();
                else if (behind == 1) wait_vmcnt<L>();
                else wait_vmcnt<0>();
                ring_barrier();
            }
            if (k + NS - 1 < slices) issue_slice();
        }
        return;
    }

    // ---- multiplying: block (cm, cn) of the tile
    const int half = lane >> 5, l32 = lane & 31, cm = wave % CM, cn = wave / CM;
    const int n = nt * BN + cn * 32 + l32, m_lane = mt * BM + cm * 32 + half * 8;     // after the store's lane exchange: filters m_lane + 16 qp ..
    f32x4 bias[2][2];
    u32x4 res[2];
#pragma unroll
    for (int qp = 0; qp < 2; ++qp) {
        const int mb = m_lane + qp * 16;
        bias[qp][0] = bias[qp][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        res[qp] = u32x4{0u, 0u, 0u, 0u};
        if (j.vec && n < j.Ng && mb < j.K) {             // (vec: whole groups of 8 filters)
            if (j.bias) {
                bias[qp][0] = *reinterpret_cast<const f32x4*>(j.bias + mb);
                bias[qp][1] = *reinterpret_cast<const f32x4*>(j.bias + mb + 4);
            }
            if (j.res) res[qp] = *reinterpret_cast<const u32x4*>(j.res + (size_t)n * j.res_ctot + mb);
        }
    }
    const unsigned ring_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
    const unsigned lane_x = (half << 4) ^ (((l32 >> 1) & 7) << 4);
    const unsigned a_rd = ring_lds + (cm * 32 + l32) * 128 + lane_x, b_rd = ring_lds + BM * 128 + (cn * 32 + l32) * 128 + lane_x;
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    u32x4 fa[4], fb[4];
    auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[ks]), __builtin_bit_cast(bf16x8, fb[ks]), acc, 0, 0, 0);
    };
    int stage = 0;
    for (int k = 0; k < slices; ++k) {
        ring_barrier();
        u32x4 na[4], nb[4];
        const unsigned pa = a_rd + stage * STAGE, pb = b_rd + stage * STAGE;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            na[ks] = ds_read16<0>(pa ^ (ks * 32));
            nb[ks] = ds_read16<0>(pb ^ (ks * 32));
        }
        if (k) multiply();
        wait_lgkm<0>();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) { touch(na[ks]); touch(nb[ks]); fa[ks] = na[ks]; fb[ks] = nb[ks]; }
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    ring_barrier();
    multiply();

    // ---- the store: as in the streaming kernel
#pragma unroll
    for (int qp = 0; qp < 2; ++qp) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[qp * 8 + e]), __float_as_uint(acc[qp * 8 + 4 + e]), false, false);
            o[e] = __uint_as_float(sw[0]);
            o[4 + e] = __uint_as_float(sw[1]);
        }
        const int mb = m_lane + qp * 16;
        if (n >= j.Ng || mb >= j.K) continue;
        uint16_t* yb = j.y_seg[0] + (size_t)n * j.ctot_seg[0];
        if (j.nsplit > 1) {
            const bool s1 = mb >= j.split_end[0], s2 = mb >= j.split_end[1], s3 = mb >= j.split_end[2];
            uint16_t* base = s3 ? j.y_seg[3] : s2 ? j.y_seg[2] : s1 ? j.y_seg[1] : j.y_seg[0];
            yb = base + (size_t)n * (s3 ? j.ctot_seg[3] : s2 ? j.ctot_seg[2] : s1 ? j.ctot_seg[1] : j.ctot_seg[0]);
        }
        if (j.vec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += bias[qp][e >> 2][e & 3];
            if (j.res) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[2 * e] += __uint_as_float(res[qp][e] << 16);
                    o[2 * e + 1] += __uint_as_float(res[qp][e] & 0xFFFF0000u);
                }
            }
            if (j.relu) {
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = fmaxf(o[e], 0.f);
            }
            u32x4 pk;
#pragma unroll
            for (int e = 0; e < 4; ++e) pk[e] = pack_bf16x2(o[2 * e], o[2 * e + 1]);
            *reinterpret_cast<u32x4*>(yb + mb) = pk;
            continue;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (mb + e >= j.K) break;
            float v = o[e] + (j.bias ? j.bias[mb + e] : 0.f);
            if (j.res) v += bf16_to_f32(j.res[(size_t)n * j.res_ctot + mb + e]);
            if (j.relu) v = fmaxf(v, 0.f);
            yb[mb + e] = f32_to_bf16(v);
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
    j.stem_hp = c.stem_hp; j.stem_wp = c.stem_wp;
    j.x_bytes = c.stem_wp ? (int)((size_t)g.N * c.stem_hp * c.stem_wp * 8) : (int)((size_t)g.N * g.C * g.H * g.W * 2);
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
    j.nsplit = c.split && c.split->n > 1 ? c.split->n : 0;
    j.vec = g.K % 8 == 0 && aligned16(c.bias) && (!c.res || (g.res_ctot % 8 == 0 && aligned16(c.res)));
    auto dest = [&](int d, uint16_t* y, int ctot, int coff, int start) {
        j.y_seg[d] = y + coff - start;
        j.ctot_seg[d] = ctot;
        j.vec = j.vec && ctot % 8 == 0 && coff % 8 == 0 && aligned16(y);
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

// Tiles of bm x bn of a group of layers.
static long small_tiles(const ConvSmall* jobs, int n, int bm, int bn)
{
    long t = 0;
    for (int i = 0; i < n; ++i)
        if (jobs[i].w) t += ((long)jobs[i].g.Ng + bn - 1) / bn * ((jobs[i].g.K + bm - 1) / bm);
    return t;
}

// As long as the layer's 64 x 64 tiles fit the device at two workgroups per compute unit, 1x1 filters at one (their contraction is
// short and the larger tiles then win: 480 -> 304 on 14 x 14 x 19, 295 tiles, 7.7 against 8.5 us; 3x3 144 -> 288, 295 tiles too,
// 13.6 against 13.5).
bool conv_bf16_small_takes(const ConvGeom& g, const void* x, const void* w)
{
    const long tiles = ((long)g.Ng + 63) / 64 * ((g.K + 63) / 64);
    return conv_bf16_dma_eligible(g, x, w) && tiles <= (g.R * g.S > 1 ? 2 : 1) * device_cus();
}

template <int CM, int CN, int NS>
static int launch_group(const ConvSmall* jobs, int n, hipStream_t st)
{
    constexpr int NTH = (CM * CN + 4) * 64;
    SmallArgs a{};
    a.n = n;
    int blocks = 0;
    for (int i = 0; i < n; ++i) {
        a.job[i] = small_job(jobs[i], CM * 32, CN * 32, NTH);
        a.job[i].first = blocks;
        blocks += (a.job[i].tiles + 7) / 8 * 8;
    }
    hipLaunchKernelGGL((conv_bf16_small_kernel<CM, CN, NS>), dim3((unsigned)blocks), dim3(NTH), 0, st, a);
    return check_launch("conv_bf16_small");
}

int launch_conv_bf16_small(const ConvSmall* jobs, int n, hipStream_t st)
{
    // the smallest tile that leaves every compute unit at most one
    if (small_tiles(jobs, n, 32, 32) <= device_cus()) return launch_group<1, 1, 4>(jobs, n, st);
    if (small_tiles(jobs, n, 64, 32) <= device_cus()) return launch_group<2, 1, 4>(jobs, n, st);
    return launch_group<2, 2, 4>(jobs, n, st);
}

}  // namespace dr
