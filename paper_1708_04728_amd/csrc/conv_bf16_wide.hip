// bf16 convolution of larger layers: one wide tile per compute unit, loading and multiplying waves apart.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (r, s, c)
//
// The streaming kernel (conv_bf16_dma.hip) gives every wave both jobs, and its tiles of 64 or 96 filters x 128 pixels ask more of the path
// into LDS (one 1 KiB load per 16 to 19 cycles and compute unit, whatever it fetches) than of the matrix cores: 24 loads, 460 cycles, for a
// slice of 64 x 128 that is 256 cycles of matrix work.  Here
//   * a tile is 32 TM filters x 32 TN pixels, as much as one workgroup's LDS (three slices of 64) and registers hold: 160 x 224 has 48
//     loads, 910 cycles, for 1120 of matrix work;
//   * four waves multiply (one per SIMD, 16 TM x 16 TN each), four send the loads.  A k-step's operands are read from LDS between the matrix
//     instructions of the one before it: a wave reads 16 bytes per lane in about 40 cycles, as long as two and a half instructions of 16 x 16 x 32
//     take.  (Eight multiplying waves read faster and gained nothing.)
//   * where a chunk of the contraction lies comes from a table in LDS, as in the kernel for small layers (conv_bf16_small.hip).
// Workgroups are persistent: the loading waves run on into the next tile while the others store.  The order of the sums is the streaming
// kernel's: the same bits.
//
// The layers of a module that do not depend on one another share a launch (conv_bf16_wide_group_kernel): each has a tile of its own and as many of the
// compute units as its work asks for, so that all of them are done at about the same time (wide_plan).  One by one each of them pays a start
// and an end of its own, about 6 us, and ends in a round that leaves compute units idle; 64 x 64 tiles, two to a compute unit, in the kernel for small
// layers ask twice as much of the path into LDS.  Modules of GoogLeNet, us, before and with it: 4a slim on 19 images 15.7 and 12.0, on 37 22.0 and 15.7, on 128 36.5 and
// 33.5; 3b fused on 12 27.3 and 22.3, on 64 79 and 68; 4e fused on 37 41.9 and 29.0; 5b fused on 100 38.8 and 28.3; 84 modules on 5 to 100 images
// 0.873 of the time, none slower by more than 1 %.
//
// What bounds it: the matrix cores at the clock that they reach on varying operands -- 0.70 us per slice of 160 x 224 on 224 compute
// units, 1.6 GHz -- and what a tile costs beside them: about 7 us for a layer of one round (a cold start, the store of the whole output at once),
// 3 us for each further round.  Measured, streaming kernel -> this one, batch 128: 3x3 144 -> 288 on 14 x 14 38.4 -> 24.6 us, 160 -> 320 39.8 -> 26.4,
// 128 -> 256 22.6 -> 18.3, 128 -> 192 on 28 x 28 57 -> 50, 192 -> 384 on 7 x 7 18.8 -> 13.1, 1x1 480 -> 304 on 14 x 14 21.3 -> 15.7; over 80 layers
// of GoogLeNet and of sizes drawn at random 0.83 of the time, 1.02 at worst.  GoogLeNet at batch 128: slim 722 -> 637 us, original 1584 -> 1499.
// It also runs beside other streams, where the streaming kernel keeps its larger tiles (SharedDeviceScope): modules that do not run by levels although
// their branches are wanted on streams (inception_levels.h), or while a trace of some layers runs.
#include <algorithm>
#include <utility>

#include "dr_internal.h"
#include "dr_store.h"
#include "conv_bf16_dev.h"
#include "conv_bf16_wide_plan.h"

namespace dr {
namespace {

constexpr int WIDE_TABLE = 1024;                         // chunks of 8 contraction elements that a layer may have (8 KB of LDS)
constexpr int WIDE_STAGES = 3;                           // slices in LDS

template <class F, int... I>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, const F& f) { (f(IC<I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void each(const F& f) { each_of(std::make_integer_sequence<int, N>{}, f); }

struct WideArgs {
    const uint16_t* x;
    const uint16_t* w;
    const float* bias;
    uint16_t* y_seg[4];                                  // destinations of the filter ranges (see ConvSplit), y_seg[0] alone otherwise
    int ctot_seg[4], split_end[3];
    int C, H, W, K, R, S, sh, sw, ph, pw, P, Q, Kg, Ng, relu;
    int x_bytes, w_bytes, pointwise;
    int c8, run_chunks, row_chunks, slices;              // see conv_bf16_small.hip
    unsigned magic_c8, magic_row;
    unsigned long long m_pq, m_q;
    int step_img, step_p, step_q;                        // 32 pixels as (images, rows, columns) of the output
    WalkArgs wk;
};

// A tile of 32 TM filters x 32 TN pixels: 2 x 2 multiplying waves with TM x TN blocks of 16 x 16 each, four loading waves
template <int TM, int TN>
__device__ __forceinline__ void wide_tiles(const WideArgs& a, const int block, unsigned char* const ring, u32x2* const table, float* const bias_lds)
{
    constexpr int NS = WIDE_STAGES, BM = TM * 32, BN = TN * 32, L = TM + TN, STAGE = (BM + BN) * 128;       // slices in LDS; loads of a wave per slice
    static_assert(BM <= 256 && (NS - 1) * L < 63, "loads in flight");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const TileWalk walk = tile_walk(a.wk, block);
    const int mt = walk.mt, slices = a.slices, total = walk.count * slices;

    if (wave >= 4) {
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, a.w_bytes, 0x00020000);
        const int lw = wave - 4, lrow = lw * 8 + (lane >> 3), lc = (lane & 7) ^ ((lrow >> 1) & 7);
        int a_voff[TM];
        unsigned b_base[TN], b_mask[TN];                 // windows of the pixels (conv_bf16_table.h)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = mt * BM + i * 32 + lrow;
            a_voff[i] = m < a.K ? (m * a.Kg + lc * 8) * 2 : OOB;
        }
        auto tile_setup = [&](int nt) __attribute__((always_inline)) {
            const int n0 = nt * BN + lrow;
            if (a.pointwise) {
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const int n = n0 + i * 32;
                    b_base[i] = window_offset(0, 0, n, 0, 0, a.C);
                    b_mask[i] = n < a.Ng ? CHUNK_NONE : WINDOW_NONE;
                }
                return;
            }
            const int nn = n0 < a.Ng ? n0 : 0;
            int img = div_small(nn, a.m_pq);
            const int pix = nn - img * a.P * a.Q;
            int p = div_small(pix, a.m_q), q = pix - p * a.Q;
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                const int ih0 = p * a.sh - a.ph, iw0 = q * a.sw - a.pw;
                b_base[i] = window_offset(img, ih0, iw0, a.H, a.W, a.C);
                b_mask[i] = window_mask(n0 + i * 32 < a.Ng, ih0, iw0, a.R, a.S, a.H, a.W);
                q += a.step_q;
                if (q >= a.Q) { q -= a.Q; ++p; }
                p += a.step_p;
                if (p >= a.P) { p -= a.P; ++img; }
                img += a.step_img;
            }
        };
        const int row_chunks = a.row_chunks, row_gap = (a.run_chunks - a.row_chunks) * 16;
        int ld_t = 0, ld_s = 0, ld_j0 = 0, soff_a = 0, stage = 0;        // tile, slice, chunk in the row, offset in a filter, LDS stage of the next slice
        tile_setup(walk.tile(0));
        const unsigned tab_rd = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)table + lc * 8;
        ring_barrier();
        for (int k = 1 - NS; k + NS - 1 < total; ++k) {
            u32x2 e = ds_read8(tab_rd + ld_s * 64);
            if (k >= 0) {
                wait_vmcnt<(NS - 2) * L>();
                ring_barrier();
            } else {
                wait_lgkm<0>();
            }
            touch(e);
            unsigned char* const sa = ring + stage * STAGE + lw * 1024;
            unsigned char* const sb = sa + BM * 128;
            const bool ok = chunk_exists(e[1]);
#pragma unroll
            for (int i = 0; i < TM; ++i) load_to_lds16(rw, sa + i * 4096, ok ? a_voff[i] : OOB, soff_a);
#pragma unroll
            for (int i = 0; i < TN; ++i) load_to_lds16(rx, sb + i * 4096, (b_mask[i] & e[1]) == 0 ? (int)(b_base[i] + e[0]) : OOB, 0);
            stage = stage + 1 == NS ? 0 : stage + 1;
            ld_j0 += 8;
            soff_a += 128;
            if (ld_j0 == row_chunks) { ld_j0 = 0; soff_a += row_gap; }
            if (++ld_s == slices) {
                ld_s = ld_j0 = soff_a = 0;
                if (++ld_t < walk.count) tile_setup(walk.tile(ld_t));
            }
        }
        if (total > 1) {
            wait_vmcnt<L>();
            ring_barrier();
        }
        wait_vmcnt<0>();
        ring_barrier();
        return;
    }

    for (int e = tid; e < slices * 8; e += 256) table[e] = chunk_entry(e, a.R, a.W, a.C, a.c8, a.run_chunks, a.row_chunks, a.magic_row, a.magic_c8);
    if (tid < BM) bias_lds[tid] = a.bias && mt * BM + tid < a.K ? a.bias[mt * BM + tid] : 0.f;
    ring_barrier();

    const int quad = lane >> 4, l16 = lane & 15, m0 = (wave & 1) * TM * 16, n0 = (wave >> 1) * TN * 16;
    const unsigned ring_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
    const unsigned lane_x = (quad << 4) ^ (((l16 >> 1) & 7) << 4);
    const unsigned a_rd = ring_lds + (m0 + l16) * 128 + lane_x, b_rd = ring_lds + BM * 128 + (n0 + l16) * 128 + lane_x;
    f32x4 acc[TM][TN];
    auto zero = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // A k-step of 32: TM TN matrix instructions on the operands of slot KS, and between them the TM + TN reads of the other slot
    u32x4 fa[2][TM], fb[2][TN];
    auto read = [&](auto slot_c, auto r_c, unsigned pa, unsigned pb) __attribute__((always_inline)) {
        constexpr int SLOT = decltype(slot_c)::value, R = decltype(r_c)::value;
        if constexpr (R < TM) fa[SLOT][R] = ds_read16<R * 2048>(pa);
        else fb[SLOT][R - TM] = ds_read16<(R - TM) * 2048>(pb);
    };
    auto fetch = [&](auto ks_c, int st) __attribute__((always_inline)) {
        constexpr int KS = decltype(ks_c)::value;
        const unsigned pa = (a_rd + st * STAGE) ^ (KS * 64), pb = (b_rd + st * STAGE) ^ (KS * 64);
        each<TM + TN>([&](auto r_c) __attribute__((always_inline)) { read(IC<KS>{}, r_c, pa, pb); });
    };
    auto step = [&](auto ks_c, auto first_c, int st) __attribute__((always_inline)) {     // multiplies slot KS, fetches k-step 1 - KS of stage st
        constexpr int KS = decltype(ks_c)::value, NEXT = 1 - KS, M = TM * TN, R = TM + TN;
        const unsigned pa = (a_rd + st * STAGE) ^ (NEXT * 64), pb = (b_rd + st * STAGE) ^ (NEXT * 64);
#pragma unroll
        for (int i = 0; i < TM; ++i) touch(fa[KS][i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) touch(fb[KS][j]);
        each<M>([&](auto x_c) __attribute__((always_inline)) {
            constexpr int X = decltype(x_c)::value, I = X / TN, J = X % TN;
            acc[I][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[KS][I]), __builtin_bit_cast(bf16x8, fb[KS][J]),
                                                                  decltype(first_c)::value ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[I][J], 0, 0, 0);
            each<R>([&](auto r_c) __attribute__((always_inline)) {
                if constexpr (decltype(r_c)::value * (M * 3 / 4) / R == X) {
                    __builtin_amdgcn_sched_barrier(0);
                    read(IC<NEXT>{}, r_c, pa, pb);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        });
    };
    // All values of a row of blocks first, without a branch, then its stores.  With a test for the ReLU and one for the edge between every two results and
    // the sums cleared by instructions of their own instead of by the first product, GoogLeNet at batch 128 took 563 us in slim form (now 558) and its 3b module
    // on 37 images 37.8 (36.4); 84 modules 0.8 % more, none less.  The rest of a store's time is memory's: nontemporal stores 596, whole lines 1 % faster at best.
    auto store_as = [&](auto relu_c, int nt) __attribute__((always_inline)) {
        constexpr bool RELU = decltype(relu_c)::value;
        int quad_ = quad, n_lane = nt * BN + n0 + l16;
        asm volatile("" : "+v"(quad_), "+v"(n_lane));    // (keeps what the store needs per lane out of the registers of the loop)
        const int mw = mt * BM + m0;
        uint16_t* const y0 = a.y_seg[0], * const y1 = a.y_seg[1], * const y2 = a.y_seg[2], * const y3 = a.y_seg[3];
        const int c0 = a.ctot_seg[0], c1 = a.ctot_seg[1], c2 = a.ctot_seg[2], c3 = a.ctot_seg[3];
#pragma unroll
        for (int i = 0; i < TM; i += 2) {
            const bool two = i + 1 < TM;
            const f32x4 b0 = *reinterpret_cast<const f32x4*>(&bias_lds[m0 + i * 16 + quad_ * 4]);
            const f32x4 b1 = two ? *reinterpret_cast<const f32x4*>(&bias_lds[m0 + i * 16 + 16 + quad_ * 4]) : f32x4{0.f, 0.f, 0.f, 0.f};
            // with two blocks, after the exchange: 8 filters of block i + (quad >> 1)
            const int mb = two ? mw + i * 16 + quad_ * 8 : mw + i * 16 + quad_ * 4;
            const bool s1 = mb >= a.split_end[0], s2 = mb >= a.split_end[1], s3 = mb >= a.split_end[2];
            const int ctot = s3 ? c3 : s2 ? c2 : s1 ? c1 : c0, left = mb < a.K ? a.Ng - n_lane : 0;
            uint16_t* dst = (s3 ? y3 : s2 ? y2 : s1 ? y1 : y0) + mb + (ptrdiff_t)n_lane * ctot;
            u32x4 v[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                unsigned p[2][2];
#pragma unroll
                for (int u = 0; u < (two ? 2 : 1); ++u) {
                    f32x4 o = acc[i + u][j] + (u ? b1 : b0);
                    if constexpr (RELU) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = fmaxf(o[e], 0.f);
                    }
                    p[u][0] = pack_bf16x2(o[0], o[1]);
                    p[u][1] = pack_bf16x2(o[2], o[3]);
                }
                if (two) {
                    // filters 4 quad .. + 3 of both blocks -> 8 consecutive ones of one block
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        const auto x32 = __builtin_amdgcn_permlane32_swap(p[0][d], p[1][d], false, false);
                        const auto x16 = __builtin_amdgcn_permlane16_swap(x32[0], x32[1], false, false);
                        v[j][d] = x16[0];
                        v[j][2 + d] = x16[1];
                    }
                } else {
                    v[j] = u32x4{p[0][0], p[0][1], 0u, 0u};
                }
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (j * 16 < left) {
                    if (two) *reinterpret_cast<u32x4*>(dst) = v[j];
                    else *reinterpret_cast<u32x2*>(dst) = u32x2{v[j][0], v[j][1]};
                }
                dst += (ptrdiff_t)ctot * 16;
            }
        }
    };
    auto store = [&](int nt) __attribute__((always_inline)) {
        if (a.relu) store_as(IC<1>{}, nt);
        else store_as(IC<0>{}, nt);
    };

    ring_barrier();                                      // slice 0
    fetch(IC<0>{}, 0);
    wait_lgkm<0>();
    int stage = 0, g = 0;
    for (int t = 0; t < walk.count; ++t) {
        auto slice = [&](auto first_c) __attribute__((always_inline)) {
            step(IC<0>{}, first_c, stage);
            stage = stage + 1 == NS ? 0 : stage + 1;
            wait_lgkm<0>();
            if (++g < total) ring_barrier();
            step(IC<1>{}, IC<0>{}, stage);      // (after the last slice: reads nobody uses)
            wait_lgkm<0>();
        };
        constexpr bool PEEL = TM * TN <= 30;    // (160 x 224: spills)
        if constexpr (PEEL) slice(IC<1>{});
        else zero();
        for (int s = PEEL; s < slices; ++s) slice(IC<0>{});
        store(walk.tile(t));
    }
}

template <int TM, int TN>
__global__ __launch_bounds__(512, 2) void conv_bf16_wide_kernel(const WideArgs a)
{
    __shared__ __attribute__((aligned(1024))) unsigned char ring[WIDE_STAGES * (TM + TN) * 4096];
    __shared__ __attribute__((aligned(16))) u32x2 table[WIDE_TABLE];
    __shared__ __attribute__((aligned(16))) float bias_lds[TM * 32];
    wide_tiles<TM, TN>(a, (int)blockIdx.x, ring, table, bias_lds);
}

// 3x3 max-pooling at stride 1 beside the layers: an item is a strip of POOL_ROWS rows of an output column and 8 channels, whose loads are all on their way
// before any is used; an image's items are dealt to the lanes in memory order, 512 at a time, and an eighth of them to every die.  Launched before or behind
// the layers it took 4 to 6 us in which the matrix cores stood still; its share of the compute units is as many as let it end with them, 2.2 us (loads of eight
// waves and their latency) for each 512 items.  Modules, us, before and with it: 4c fused on 37 images 22.1 and 20.3, on 19 19.8 and 15.7; 4e fused on 19 24.1 and
// 19.6; 5b fused on 64 26.7 and 22.3; fused GoogLeNet on 19 images 306 and 279.
constexpr int POOL_ROWS = 4, POOL_ITEMS = 512;
struct WidePool {
    const uint16_t* x;
    uint16_t* y;
    int C, H, W, P, Q, ph, pw, per_image, groups;        // items and groups of 512 of an image
    int blocks, per_die, share;                          // groups of 512 of all images; of a die; workgroups of this launch
    unsigned magic_cv, magic_qcv;
};
__device__ __forceinline__ void wide_pool(const WidePool& a, const int block)
{
    constexpr int NR = POOL_ROWS + 2;
    const int cv_n = a.C / 8, qcv = a.Q * cv_n;
    for (int i = block >> 3; i < a.per_die; i += a.share >> 3) {
        const int b = (block & 7) * a.per_die + i;
        if (b >= a.blocks) return;
        const int img = b / a.groups, item = (b - img * a.groups) * POOL_ITEMS + (int)threadIdx.x;
        if (item >= a.per_image) continue;
        const int strip = qcv == 1 ? item : (int)__umulhi((unsigned)item, a.magic_qcv), pair = item - strip * qcv;
        const int q = cv_n == 1 ? pair : (int)__umulhi((unsigned)pair, a.magic_cv), cv = pair - q * cv_n;
        const int p0 = strip * POOL_ROWS, h0 = p0 - a.ph, w0 = q - a.pw;
        const uint16_t* const xb = a.x + (size_t)img * a.H * a.W * a.C + cv * 8;
        u32x4 raw[NR][3];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                raw[r][c] = u32x4{0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u};      // -inf
                if ((unsigned)(h0 + r) < (unsigned)a.H && (unsigned)(w0 + c) < (unsigned)a.W)
                    raw[r][c] = *reinterpret_cast<const u32x4*>(xb + ((size_t)(h0 + r) * a.W + (w0 + c)) * a.C);
            }
        u32x4 o[POOL_ROWS];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float lo[NR], hi[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                lo[r] = fmaxf(fmaxf(__uint_as_float(raw[r][0][e] << 16), __uint_as_float(raw[r][1][e] << 16)), __uint_as_float(raw[r][2][e] << 16));
                hi[r] = fmaxf(fmaxf(__uint_as_float(raw[r][0][e] & 0xFFFF0000u), __uint_as_float(raw[r][1][e] & 0xFFFF0000u)), __uint_as_float(raw[r][2][e] & 0xFFFF0000u));
            }
#pragma unroll
            for (int r = 0; r < POOL_ROWS; ++r)
                o[r][e] = pack_bf16x2(fmaxf(fmaxf(lo[r], lo[r + 1]), lo[r + 2]), fmaxf(fmaxf(hi[r], hi[r + 1]), hi[r + 2]));
        }
#pragma unroll
        for (int r = 0; r < POOL_ROWS; ++r)
            if (p0 + r < a.P) *reinterpret_cast<u32x4*>(a.y + (((size_t)img * a.P + p0 + r) * a.Q + q) * a.C + cv * 8) = o[r];
    }
}

// Several layers side by side, each with a tile of its own and its share of the compute units.  (The job is copied, as in conv_bf16_small.hip.)
struct WideGroupArgs {
    int first_pool;                                      // first workgroup of the pooling layer; INT_MAX: none
    WidePool pool;
    int first[SMALL_GROUP_MAX];                          // first workgroup of each layer, a multiple of 8; beyond the last: INT_MAX
    int tile[SMALL_GROUP_MAX];                           // its place in WIDE_TILES
    WideArgs job[SMALL_GROUP_MAX];
};
__global__ __launch_bounds__(512, 2) void conv_bf16_wide_group_kernel(const WideGroupArgs args)
{
    __shared__ __attribute__((aligned(1024))) unsigned char ring[WIDE_STAGES * 12 * 4096];
    __shared__ __attribute__((aligned(16))) u32x2 table[WIDE_TABLE];
    __shared__ __attribute__((aligned(16))) float bias_lds[7 * 32];
    static_assert(SMALL_GROUP_MAX == 4, "jobs");
    if ((int)blockIdx.x >= args.first_pool) {
        const WidePool p = args.pool;
        wide_pool(p, (int)blockIdx.x - args.first_pool);
        return;
    }
    const int ji = ((int)blockIdx.x >= args.first[1]) + ((int)blockIdx.x >= args.first[2]) + ((int)blockIdx.x >= args.first[3]);
    const WideArgs a = args.job[ji];
    const int block = (int)blockIdx.x - args.first[ji];
    if (block >= a.wk.gn * a.wk.grid_m) return;
#define DR_TILE(T) case T: wide_tiles<WIDE_TILES[T][0], WIDE_TILES[T][1]>(a, block, ring, table, bias_lds); break
    switch (args.tile[ji]) {
    DR_TILE(0); DR_TILE(1); DR_TILE(2); DR_TILE(3); DR_TILE(4); DR_TILE(5); DR_TILE(6); DR_TILE(7); DR_TILE(8); DR_TILE(9); DR_TILE(10); DR_TILE(11); DR_TILE(12); DR_TILE(13);
    }
#undef DR_TILE
}

template <int TM, int TN>
int launch_tile(WideArgs a, hipStream_t st)
{
    constexpr int BM = TM * 32, BN = TN * 32;
    const int grid_m = (a.K + BM - 1) / BM, grid_n = (a.Ng + BN - 1) / BN, gn = std::min(std::max(device_cus() / grid_m, 1), grid_n);
    a.wk = make_walk(grid_m, gn, grid_n);
    hipLaunchKernelGGL((conv_bf16_wide_kernel<TM, TN>), dim3((unsigned)(gn * grid_m)), dim3(512), 0, st, a);
    return check_launch("conv_bf16_wide");
}

// The tile with the shortest time by the model (wide_tile_us).  Over these 10 tiles on 80 layers the time is the model's + 1.9 us, 6 % off on average, and
// the tile that it picks takes 1.01 times as long as the best one on average, 1.25 at worst (3x3 512 -> 40 on 43 x 40 x 103: 64 x 160 209 us, 128 x 128 167).
struct WideTile { int m, n, rounds; float us; };

WideTile wide_tile(int K, int Ng, int slices)
{
    WideTile best{0, 0, 0, 1e30f};
    const int cus = device_cus();
    for (int i = 0; i < WIDE_ALONE; ++i) {
        const int* const t = WIDE_TILES[i];
        const int bm = t[0] * 32, bn = t[1] * 32, grid_m = (K + bm - 1) / bm, grid_n = (Ng + bn - 1) / bn, gn = std::min(std::max(cus / grid_m, 1), grid_n);
        const int rounds = (grid_n + gn - 1) / gn * ((gn * grid_m + cus - 1) / cus);
        const float us = rounds * wide_tile_us(t[0], t[1], slices);
        if (us < best.us) best = WideTile{t[0], t[1], rounds, us};
    }
    return best;
}

}  // namespace

// Stores are 16 bytes, eight filters; the contraction has to fit the table.  Layers of up to 32 filters stay with the streaming kernel's tiles of
// 32, and so do contractions that end before the ring is filled: up to two slices, and where the tiles take more than one round up to three,
// 1x1 filters up to four (64 -> 64 on 56 x 56 x 128, one slice, 19.2 us there, 21.9 here; 104 -> 352 on 28 x 28 x 128, two, 26.0 and 28.1;
// 136 -> 392 on 28 x 56 x 24, three, 18.9 and 19.5; 240 -> 48 on 35 x 56 x 64, four, 15.2 and 16.5; in one round three slices of 1x1 160 -> 448 at
// stride 2 on 7 x 28 x 128 8.0 and 6.4; 3x3 24 -> 256 on 14 x 31 x 128, four slices in two rounds, 20.0 and 16.6).
bool conv_bf16_wide_takes(const ConvGeom& g, const void* x, const void* w, const void* residual, const void* y, const ConvSplit* split)
{
    int row_chunks;
    if (residual || !conv_bf16_dma_eligible(g, x, w) || g.K % 8 != 0 || g.K <= 32) return false;
    const int slices = chunk_slices(g.R, g.S, g.C, &row_chunks);
    if (slices < 3 || slices * 8 > WIDE_TABLE) return false;
    if (slices <= (g.R * g.S > 1 ? 3 : 4) && wide_tile(g.K, g.Ng, slices).rounds > 1) return false;
    if (split && split->n > 1) {
        for (int d = 0; d < split->n; ++d)
            if (split->dst[d].ctot % 8 != 0 || split->dst[d].c_offset % 8 != 0 || split->dst[d].k % 8 != 0 || !aligned16(split->dst[d].y)) return false;
        return true;
    }
    return g.y_ctot % 8 == 0 && g.y_coff % 8 == 0 && aligned16(y);
}

// Where the kernels that keep an input patch in LDS (conv_bf16_patch.hip, conv_bf16_rows.hip: 96 filters x 252 pixels a workgroup, two of them
// per compute unit) would have little more than a workgroup per compute unit, and this one has a single round: 5x5 48 -> 640 on 7 x 7 x 128
// (175 workgroups) 18.3 us there and 11.9 here, 64 -> 424 on 14 x 14 x 64 (250) 22.8 and 19.8, 3x3 48 -> 336 on
// 35 x 31 x 16 (276) 13.3 and 10.9; 64 -> 256 on 14 x 28 x 64 (300) 11.1 and 12.0, 5x5 16 -> 432 on 7 x 28 x 96 (375) 13.0 and 13.4.
// Layers of half a workgroup per compute unit and fewer are few (most are small layers) and stay where they were.
bool conv_bf16_wide_fills(const ConvGeom& g)
{
    int row_chunks;
    const long groups = (long)(g.K + 95) / 96 * ((g.Ng + 251) / 252), cus = device_cus();
    return 2 * groups > cus && 10 * groups <= 11 * cus && wide_tile(g.K, g.Ng, chunk_slices(g.R, g.S, g.C, &row_chunks)).rounds == 1;
}

static WideArgs wide_args(const ConvGeom& g, const uint16_t* x, const uint16_t* w, const float* bias, uint16_t* y, const ConvSplit* split)
{
    WideArgs a{};
    a.x = x; a.w = w; a.bias = bias;
    a.C = g.C; a.H = g.H; a.W = g.W; a.K = g.K; a.R = g.R; a.S = g.S; a.sh = g.sh; a.sw = g.sw; a.ph = g.ph; a.pw = g.pw;
    a.P = g.P; a.Q = g.Q; a.Kg = g.Kg; a.Ng = g.Ng; a.relu = g.relu;
    a.x_bytes = (int)((size_t)g.N * g.C * g.H * g.W * 2);
    a.w_bytes = (int)((size_t)g.K * g.Kg * 2);
    a.pointwise = g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    a.c8 = g.C / 8;
    a.run_chunks = g.S * a.c8;
    a.slices = chunk_slices(g.R, g.S, g.C, &a.row_chunks);
    a.magic_c8 = (unsigned)((0x100000000ull + a.c8 - 1) / a.c8);
    a.magic_row = (unsigned)((0x100000000ull + a.row_chunks - 1) / a.row_chunks);
    a.m_pq = ((1ull << 40) + (unsigned)(g.P * g.Q) - 1) / (unsigned)(g.P * g.Q);
    a.m_q = ((1ull << 40) + (unsigned)g.Q - 1) / (unsigned)g.Q;
    a.step_img = 32 / (g.P * g.Q);
    a.step_p = 32 % (g.P * g.Q) / g.Q;
    a.step_q = 32 % g.Q;
    set_destinations(a, split, y, g.y_ctot, g.y_coff);
    return a;
}

// A layer that may share a launch of wide tiles: what conv_bf16_wide_takes asks of the addresses, any filter count and contraction that fits the table
bool conv_bf16_wide_joins(const ConvGeom& g, const void* x, const void* w, const void* y, const ConvSplit* split)
{
    int row_chunks;
    if (!conv_bf16_dma_eligible(g, x, w) || g.K % 8 != 0 || g.Ng == 0 || chunk_slices(g.R, g.S, g.C, &row_chunks) * 8 > WIDE_TABLE) return false;
    if (split && split->n > 1) {
        for (int d = 0; d < split->n; ++d)
            if (split->dst[d].ctot % 8 != 0 || split->dst[d].c_offset % 8 != 0 || split->dst[d].k % 8 != 0 || !aligned16(split->dst[d].y)) return false;
        return true;
    }
    return g.y_ctot % 8 == 0 && g.y_coff % 8 == 0 && aligned16(y);
}

static int pool_groups(const ConvGeom& g) { return ((g.P + POOL_ROWS - 1) / POOL_ROWS * g.Q * (g.C / 8) + POOL_ITEMS - 1) / POOL_ITEMS; }

// Up to 7/4 groups of 512 items per compute unit: a larger pooling layer fills the device by itself and, bound by memory, takes longer on a share of it
// (module in original form: 512 channels of 14 x 14 on 64 images, 448 groups, 47.0 us with a launch of its own and 44.0; 28 x 28 x 256 on 37 images, 481, 67.5 and
// 69.4, on 100, 1300, 142 and 150; fused 3b on 19, 247, 28.3 and 25.5).  The kernel's divisions are exact where an image's items are that few.
bool conv_bf16_wide_pools(const ConvSmall& c)
{
    const ConvGeom& g = c.g;
    const double qcv = (double)g.Q * (g.C / 8);
    return !c.w && g.R == 3 && g.S == 3 && g.sh == 1 && g.sw == 1 && g.C % 8 == 0 && g.Ng > 0 && aligned16(c.x) && aligned16(c.y) &&
           qcv * qcv * (g.P + POOL_ROWS) < 4294967296.0 && 4l * g.N * pool_groups(g) <= 7l * device_cus();
}

static_assert(SMALL_GROUP_MAX <= WIDE_LAYERS, "layers of a plan");

int launch_conv_bf16_wide_group(const ConvSmall* jobs, int n, hipStream_t st, const ConvSmall* pool, bool* launched)
{
    WideGroupArgs a{};
    int blocks = 0;
    a.first_pool = 0x7FFFFFFF;
    if (pool) {
        const ConvGeom& g = pool->g;
        const int cv = g.C / 8, qcv = g.Q * cv, strips = (g.P + POOL_ROWS - 1) / POOL_ROWS, groups = pool_groups(g);
        a.pool = WidePool{(const uint16_t*)pool->x, (uint16_t*)pool->y, g.C, g.H, g.W, g.P, g.Q, g.ph, g.pw, strips * qcv, groups,
                          g.N * groups, (g.N * groups + 7) / 8, 0, (unsigned)((0x100000000ull + cv - 1) / cv), (unsigned)((0x100000000ull + qcv - 1) / qcv)};
    }
    WideLayer layers[SMALL_GROUP_MAX];
    WidePlan plan;
    for (int i = 0; i < n; ++i) {
        const ConvGeom& g = jobs[i].g;
        int row_chunks;
        layers[i] = WideLayer{g.K, g.Ng, chunk_slices(g.R, g.S, g.C, &row_chunks)};
    }
    *launched = wide_plan(layers, n, a.pool.blocks, device_cus(), &plan);
    if (!*launched) return DR_OK;
    a.pool.share = plan.pool_share;
    for (int i = 0; i < SMALL_GROUP_MAX; ++i) {
        a.first[i] = i < n ? blocks : 0x7FFFFFFF;
        if (i >= n) continue;
        const ConvSmall& c = jobs[i];
        const int bm = WIDE_TILES[plan.tile[i]][0] * 32, bn = WIDE_TILES[plan.tile[i]][1] * 32, grid_m = (c.g.K + bm - 1) / bm;
        a.tile[i] = plan.tile[i];
        a.job[i] = wide_args(c.g, (const uint16_t*)c.x, (const uint16_t*)c.w, c.bias, (uint16_t*)c.y, c.split);
        a.job[i].wk = make_walk(grid_m, plan.gn[i], (c.g.Ng + bn - 1) / bn);
        blocks += (plan.gn[i] * grid_m + 7) / 8 * 8;
    }
    if (pool) {
        a.first_pool = blocks;
        blocks += a.pool.share;
    }
    hipLaunchKernelGGL(conv_bf16_wide_group_kernel, dim3((unsigned)blocks), dim3(512), 0, st, a);
    return check_launch("conv_bf16_wide_group");
}

int launch_conv_bf16_wide(const ConvGeom& g, const uint16_t* x, const uint16_t* w, const float* bias, uint16_t* y, hipStream_t st, const ConvSplit* split)
{
    const WideArgs a = wide_args(g, x, w, bias, y, split);
    const WideTile t = wide_tile(g.K, g.Ng, a.slices);
    switch (t.m * 10 + t.n) {
    case 57: return launch_tile<5, 7>(a, st);
    case 47: return launch_tile<4, 7>(a, st);
    case 74: return launch_tile<7, 4>(a, st);
    case 65: return launch_tile<6, 5>(a, st);
    case 37: return launch_tile<3, 7>(a, st);
    case 64: return launch_tile<6, 4>(a, st);
    case 44: return launch_tile<4, 4>(a, st);
    case 27: return launch_tile<2, 7>(a, st);
    case 25: return launch_tile<2, 5>(a, st);
    default: return launch_tile<4, 3>(a, st);
    }
}

}  // namespace dr
