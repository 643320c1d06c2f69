// fp32 convolution of small layers (NCHW; filters in KRSC order, or 1x1): few images, or a few thousand output pixels.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (r, s, c)
//
// The kernel of conv_f32.hip gives a workgroup a 64 x 64 tile and walks the whole contraction with it, a barrier per slice; a layer
// with a tile or less per compute unit then runs at the latency of its slices (18 slices of 3x3 filters on 64 channels: 20 us
// for 8 us of matrix work, most compute units idle).  Here a tile is one 32 x 32 block, and the NW waves of a workgroup
// share its contraction.  The slices (16 channels of one tap each) are cut into SHARES runs; a wave takes one or two of them with
// a ring of two slices of its own in LDS, so that no wave waits for another; the partial sums meet in LDS once, are added in a
// fixed order and stored with bias, residual and ReLU.  Runs and order are the same however many waves there are, so a
// layer's bits do not depend on what shares its launch.  One launch takes several layers (the convolutions at one depth of an
// inception module).
//
// Operands.  v_mfma_f32_32x32x2_f32 takes one k from each half of the wave: half h holds the slice's channels 8 h .. 8 h + 7.  Both
// operands are loaded into LDS directly: the filters 16 rows of 64 bytes per load (filter rows read straight into registers, 64
// different lines per load, cost 70 % more), the activations one channel plane of 32 consecutive pixels per half and load,
// laid down in the lane order in which they are read.  Lanes in the padding or beyond the tensor load at an offset outside
// the buffer and get zeros.
#include "dr_internal.h"
#include <type_traits>

#include "dr_store.h"
#include "conv_bf16_dev.h"

namespace dr {
namespace {

constexpr int BK = 16;                                   // channels per slice
constexpr int SLICE = 2 * 32 * BK * 4;                   // bytes of one slice of both operands
constexpr int SHARES = 8;                                // runs of slices with a partial sum each, summed in pairs

struct SmallJobF {
    const float *x, *w, *bias, *res;
    float* y_seg[4];                                     // destinations of the filter ranges (see ConvSplit), y_seg[0] alone otherwise
    int ctot_seg[4], split_end[3];
    int nsplit, res_ctot;
    int C, H, W, K, S, sh, sw, ph, pw, Q, PQ, Kg, Ng, relu;
    int x_bytes, w_bytes;
    int per_tap, slices;                                 // slices per tap, per tile
    int n_tiles, tiles, first;                           // pixel tiles; tiles in all; first workgroup (a multiple of 8)
};
struct SmallArgsF {
    int n;
    SmallJobF job[SMALL_GROUP_MAX];
};

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// the dwords 256 OFF and 256 (OFF + 1) bytes behind addr (see ds_read16 for the wait)
template <int OFF>
__device__ __forceinline__ u32x2 ds_read2_planes(unsigned addr)
{
    u32x2 v;
    asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=&v"(v) : "v"(addr), "n"(OFF), "n"(OFF + 1));
    return v;
}

// NW waves, each with SHARES / NW runs of the contraction one after the other; NS slices in flight per wave
// (at least two waves per SIMD: the compiler then keeps the sums in ordinary registers, without copies between loops)
template <int NW, int NS>
__global__ __launch_bounds__(NW * 64, 2) void conv_f32_small_kernel(const SmallArgsF args)
{
    __shared__ __attribute__((aligned(1024))) unsigned char ring[NW * NS * SLICE];     // filters; the partial sums at the end
    constexpr int PER_WAVE = SHARES / NW;
    static_assert((PER_WAVE == 1 || PER_WAVE == 2) && NS * SLICE >= 4096, "a wave's partial sums take 4 KiB");

    // the job and the tile; a die (workgroup id & 7) takes a contiguous range of tiles, filter block by filter block
    int ji = 0;
    while (ji + 1 < args.n && (int)blockIdx.x >= args.job[ji + 1].first) ++ji;
    const SmallJobF j = args.job[ji];
    const int b = (int)blockIdx.x - j.first, die = b & 7, s_die = b >> 3, per = j.tiles >> 3, odd = j.tiles & 7;
    if (s_die >= per + (die < odd ? 1 : 0)) return;
    const int t = die * per + min(die, odd) + s_die;
    const int mt = t / j.n_tiles, nt = t - mt * j.n_tiles;

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)j.x, 0, j.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)j.w, 0, j.w_bytes, 0x00020000);

    const int n = nt * 32 + l32, HW4 = j.H * j.W * 4;
    const bool n_ok = n < j.Ng;
    const int nn = n_ok ? n : 0, img = nn / j.PQ, pix = nn - img * j.PQ, p = pix / j.Q, q = pix - p * j.Q;
    const int ih0 = n_ok ? p * j.sh - j.ph : -(1 << 30), iw0 = q * j.sw - j.pw;
    const int b_base = (img * j.C + half * 8) * HW4 + (p * j.sh - j.ph) * j.W * 4 + iw0 * 4;
    // filters: a load fills 16 rows of 64 bytes, chunk c of row r at c ^ ((r >> 2) & 3); this lane fetches one chunk of rows lrow, lrow + 16
    const int lrow = lane >> 2, lchunk = (lane & 3) ^ ((lane >> 4) & 3);
    int a_voff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = mt * 32 + i * 16 + lrow;
        a_voff[i] = m < j.K ? (m * j.Kg + lchunk * 4) * 4 : OOB;
    }
    unsigned char* const my_ring = ring + wave * (NS * SLICE);
    const unsigned ring_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)my_ring, a_lane = l32 * 64;
    const unsigned chunk0 = ((2 * half) ^ ((l32 >> 2) & 3)) * 16, chunk1 = ((2 * half + 1) ^ ((l32 >> 2) & 3)) * 16;

    // this wave's slices, the first of its second run, and the position of the next one to load
    const int s0 = j.slices * (wave * PER_WAVE) / SHARES, count = j.slices * ((wave + 1) * PER_WAVE) / SHARES - s0;
    const int second = PER_WAVE == 2 ? j.slices * (wave * 2 + 1) / SHARES - s0 : count;
    int tap = s0 / j.per_tap, ld_c = s0 - tap * j.per_tap;
    int ld_r = tap / j.S, ld_s = tap - ld_r * j.S;
    f32x16 sum[PER_WAVE];
#pragma unroll
    for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) sum[i][v] = 0.f;
    int stage = 0, ld_stage = 0, k = 1 - NS;
    // (a loop and registers per run: where one loop changes from run to run the compiler copies the sums in every slice, 15 % slower, and
    // where one set of registers is emptied in between the wave waits for its matrix instructions)
    auto multiply = [&](f32x16& acc, int end) __attribute__((always_inline)) {
        for (; k < end; ++k) {
            if (k + NS - 1 < count) {
                unsigned char* const dst = my_ring + ld_stage * SLICE;
                const int soff_a = (tap * j.C + ld_c * BK) * 4;
#pragma unroll
                for (int i = 0; i < 2; ++i) load_to_lds16(rw, dst + i * 1024, a_voff[i], soff_a);
                const bool in = (unsigned)(ih0 + ld_r) < (unsigned)j.H && (unsigned)(iw0 + ld_s) < (unsigned)j.W;
                const int voff = in ? b_base + (ld_r * j.W + ld_s) * 4 : OOB;
                int soff = ld_c * BK * HW4;
#pragma unroll
                for (int i = 0; i < 8; ++i, soff += HW4) load_to_lds4(rx, dst + 2048 + i * 256, voff, soff);
                ld_stage = ld_stage + 1 == NS ? 0 : ld_stage + 1;
                if (++ld_c == j.per_tap) {
                    ld_c = 0; ++tap;
                    if (++ld_s == j.S) { ld_s = 0; ++ld_r; }
                }
            }
            if (k < 0) continue;
            const int behind = min(count - 1 - k, NS - 1);   // slice k has landed; the loads of the slices behind it may be pending
            if (NS > 3 && behind == 3) wait_vmcnt<(NS > 3 ? 3 : 0) * 10>();
            else if (NS > 2 && behind == 2) wait_vmcnt<(NS > 2 ? 2 : 0) * 10>();
            else if (behind == 1) wait_vmcnt<10>();
            else wait_vmcnt<0>();
            const unsigned rd = ring_lds + stage * SLICE;
            u32x4 a0 = ds_read16<0>(rd + a_lane + chunk0), a1 = ds_read16<0>(rd + a_lane + chunk1);
            u32x2 bv[4];
            bv[0] = ds_read2_planes<8>(rd + lane * 4);
            bv[1] = ds_read2_planes<10>(rd + lane * 4);
            bv[2] = ds_read2_planes<12>(rd + lane * 4);
            bv[3] = ds_read2_planes<14>(rd + lane * 4);
            wait_lgkm<0>();
            touch(a0); touch(a1);
#pragma unroll
            for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(bv[i]));
#pragma unroll
            for (int i = 0; i < 8; ++i)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(i < 4 ? a0[i & 3] : a1[i & 3]), __uint_as_float(bv[i >> 1][i & 1]), acc, 0, 0, 0);
            stage = stage + 1 == NS ? 0 : stage + 1;
        }
    };
    if constexpr (PER_WAVE == 2) multiply(sum[0], second);
    multiply(sum[PER_WAVE - 1], count);

    // the runs' sums are added pair by pair, then the pairs in order.  Registers 4 g .. 4 g + 3 of a lane are filters 8 g + 4 half .. + 3 of
    // the block
    f32x16 acc = sum[0];
    if constexpr (PER_WAVE == 2) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] += sum[PER_WAVE - 1][v];
    }
    f32x4* const mine = reinterpret_cast<f32x4*>(my_ring);
#pragma unroll
    for (int g = 0; g < 4; ++g) mine[g * 64 + lane] = f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    __syncthreads();
    if (wave >= 4 || !n_ok) return;
    auto sum_of = [&](int w) __attribute__((always_inline)) { return reinterpret_cast<const f32x4*>(ring + w * (NS * SLICE))[wave * 64 + lane]; };
    auto pair = [&](int i) __attribute__((always_inline)) { return PER_WAVE == 2 ? sum_of(i) : sum_of(2 * i) + sum_of(2 * i + 1); };
    f32x4 o = pair(0);
#pragma unroll
    for (int i = 1; i < SHARES / 2; ++i) o += pair(i);
    const int m0 = mt * 32 + wave * 8 + half * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int m = m0 + e;
        if (m >= j.K) break;
        float v = o[e] + (j.bias ? j.bias[m] : 0.f);
        if (j.res) v += j.res[((size_t)img * j.res_ctot + m) * j.PQ + pix];
        if (j.relu) v = fmaxf(v, 0.f);
        float* base = j.y_seg[0];
        int ct = j.ctot_seg[0];
        if (j.nsplit > 1) {
            const bool s1 = m >= j.split_end[0], s2 = m >= j.split_end[1], s3 = m >= j.split_end[2];
            base = s3 ? j.y_seg[3] : s2 ? j.y_seg[2] : s1 ? j.y_seg[1] : j.y_seg[0];
            ct = s3 ? j.ctot_seg[3] : s2 ? j.ctot_seg[2] : s1 ? j.ctot_seg[1] : j.ctot_seg[0];
        }
        base[((size_t)img * ct + m) * j.PQ + pix] = v;
    }
}

SmallJobF small_job(const ConvSmall& c)
{
    const ConvGeom& g = c.g;
    SmallJobF j{};
    j.x = (const float*)c.x; j.w = (const float*)c.w; j.bias = c.bias; j.res = (const float*)c.res;
    j.res_ctot = g.res_ctot;
    j.C = g.C; j.H = g.H; j.W = g.W; j.K = g.K; j.S = g.S; j.sh = g.sh; j.sw = g.sw; j.ph = g.ph; j.pw = g.pw;
    j.Q = g.Q; j.PQ = g.P * g.Q; j.Kg = g.Kg; j.Ng = g.Ng; j.relu = g.relu;
    j.x_bytes = (int)((size_t)g.N * g.C * g.H * g.W * 4);
    j.w_bytes = (int)((size_t)g.K * g.Kg * 4);
    j.per_tap = g.C / BK;
    j.slices = g.R * g.S * j.per_tap;
    j.n_tiles = (g.Ng + 31) / 32;
    j.tiles = j.n_tiles * ((g.K + 31) / 32);
    for (int d = 0; d < 3; ++d) j.split_end[d] = 0x7FFFFFFF;
    if (c.split && c.split->n > 1) {
        j.nsplit = c.split->n;
        int start = 0;
        for (int d = 0; d < j.nsplit; ++d) {
            const ConvDest& s = c.split->dst[d];
            j.y_seg[d] = (float*)s.y + ((long)s.c_offset - start) * j.PQ;
            j.ctot_seg[d] = s.ctot;
            start += s.k;
            if (d + 1 < j.nsplit) j.split_end[d] = start;
        }
    } else {
        j.y_seg[0] = (float*)c.y + (size_t)g.y_coff * j.PQ;
        j.ctot_seg[0] = g.y_ctot;
    }
    return j;
}

template <int NW, int NS>
int launch_group(const ConvSmall* jobs, int n, hipStream_t st)
{
    SmallArgsF a{};
    a.n = n;
    int blocks = 0;
    for (int i = 0; i < n; ++i) {
        a.job[i] = small_job(jobs[i]);
        a.job[i].first = blocks;
        blocks += (a.job[i].tiles + 7) / 8 * 8;
    }
    hipLaunchKernelGGL((conv_f32_small_kernel<NW, NS>), dim3((unsigned)blocks), dim3(NW * 64), 0, st, a);
    return check_launch("conv_f32_small");
}

long small_tiles(const ConvGeom& g) { return ((long)g.Ng + 31) / 32 * ((g.K + 31) / 32); }

}  // namespace

// Measured in chains of dependent launches, us, kernel of conv_f32.hip (with scratch where it cuts the contraction) -> this one: 3x3 64 -> 192
// on one 56 x 56 map (588 tiles) 19.0 -> 14.2, at stride 2 (150) 11.6 -> 8.9; 1x1 480 -> 112 on 14 x 14 x 8 images (196)
// 11.4 -> 7.7; 3x3 192 -> 384 on 7 x 7 x 32 (588) 47 -> 31; 3x3 96 -> 208 on 14 x 14 x 32 (1372) 44 -> 34; 1x1 512 -> 320 on 14 x 14 x 20
// (1230) 24.7 -> 20.7; beyond that the larger tiles gain: 1x1 512 -> 512 on the same map (1968) 24.4 -> 30.0, 832 -> 2048 (7872) 119 -> 157.
// 1x1 filters: up to 4096 pixels.
// Long contractions are better off cut over workgroups, when the caller has scratch for that: here a round of tiles takes 0.085 us per
// slice of 16 whether it fills the device or not, there the time goes with tiles times slices.  Up to 64 tiles (1x1: 32) beyond
// 64 slices: 3x3 192 -> 384 on one 7 x 7 map (24 tiles, 108 slices) 10.2 cut against 13.5, 1x1 2048 -> 64 on the same map 8.9 and 13.0.
// Above that, by what a round leaves idle, counted from the three quarters of it that cost as much when cut: 14 x 14 maps, 3x3
// 512 -> 128 (76 tiles, 288 slices) 18.1 and 24.4, 352 -> 128 (100, 198) 18.6 and 18.4, 5x5 192 -> 160 (125, 300) 28.9 and 25.5, 352 -> 192
// (150, 550) 38.2 and 42.5; in a second round 3x3 352 -> 256 (296, 198) 30.0 and 34.1, 192 -> 224 (259, 108) 22.9 and 20.6, 352 -> 320 (490, 198)
// 41.4 and 37.4.  And where a strided layer's input, which every filter block reads for itself, is more than the L2 of a die holds:
// at stride 2 3x3 512 -> 192 on 6.4 MB (150, 288) 30.5 and 40.4, 352 -> 192 on 6.6 MB (222, 198) 27.8 and 31.7; 5x5 192 -> 256 on 2.4 MB
// (200, 300) 34.0 and 32.4.
// A strided row spreads the 32 pixels of a load over more lines, and every filter block reads them again: 5x5 96 -> 256 at stride 2 on 28 x 28
// takes 29.0 us tiled and 33.9 here on 6 images (296 tiles), 67 and 75 on 18, 98 and 113 on 28 (at stride 1 the same output: 95 and
// 74); contractions of up to 75 slices still gain or tie (5x5 32 -> 256 on 28 images 38 -> 35, 3x3 128 -> 128 34 -> 33).
// Filters are fetched 16 bytes at a time straight into LDS: they start on such a boundary.
bool conv_f32_small_takes(const ConvGeom& g, const void* w, bool scratch)
{
    const size_t xb = (size_t)g.N * g.C * g.H * g.W * 4, wb = (size_t)g.K * g.Kg * 4;
    if (g.nhwc || g.C % 16 != 0 || (!g.w_krsc && g.R * g.S != 1) || !aligned16(w) || xb >= (1ull << 31) || wb >= (1ull << 31)) return false;
    const long tiles = small_tiles(g), cus = device_cus();
    if (tiles > 11 * cus / 2 || conv_f32_pieces_takes(g) || conv_f32_direct_takes(g)) return false;
    if (g.R * g.S == 1 && g.Ng > 4096) return false;
    if (g.sw > 1 && g.Kg > 1200 && tiles > cus) return false;
    if (!scratch) return true;
    const long rounds = (tiles + cus - 1) / cus;
    if (tiles <= (g.R * g.S == 1 ? 32 : 64) && g.Kg > 1024) return false;
    if (g.sw > 1 && g.Kg > 2560 && xb > (4u << 20)) return false;
    return (3 * cus * rounds / 4 - tiles) * (g.Kg / BK) <= (rounds == 1 ? 85 : 60) * cus;
}

int launch_conv_f32_small(const ConvSmall* jobs, int n, hipStream_t st)
{
    // eight waves while there are at most two tiles per compute unit, else four (more workgroups side by side)
    long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += small_tiles(jobs[i].g);
    return tiles <= 2 * device_cus() ? launch_group<8, 2>(jobs, n, st) : launch_group<4, 2>(jobs, n, st);
}

}  // namespace dr
