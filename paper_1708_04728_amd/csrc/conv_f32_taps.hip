// fp32 convolution of first layers: few channels, wide filters, no padding (NCHW, filters in KCRS order: AlexNet's 11x11 on the image).
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (pair of filter rows, tap s, row of the pair)
//
// conv_f32.hip runs such a layer over groups of 4 taps by a table: per slice of 16 and wave some 70 vector-ALU instructions (table reads, taps
// that the rounding of S to a multiple of 4 adds, zeroed on both sides, the tensor's last elements apart) beside 512 cycles of matrix work, and
// fp32 matrix instructions do not overlap with those.  Here nothing is left to compute in the loop:
//   * a slice is two filter rows (c, r), one for each half of the matrix instruction.  A row's taps are G groups of 4, 16 bytes per
//     pixel and per filter; the last group is the row's LAST four taps, so that it never reaches beyond the row, and its first D, which
//     the group before it holds, are skipped: R S taps cost R S / 2 instructions, none for padding;
//   * four waves load (a lane's offsets never change, the row's place is the load's scalar offset) and write LDS, four multiply.
// The store has the filter's place as scalar offset and no branch per element (1500 instructions before, 16 % of a tile's time).
// Measured, AlexNet's 11x11 3 -> 96 at stride 4 on 227 x 227 x 128 (27 GFLOP, 174 us at the 155 TFLOP/s that the matrix instructions reach on
// varying operands): 374 -> 235 us; without loads and stores it takes 185.
// LDS holds [row][group][pixel or filter][4 taps]: operand reads are 16 bytes per lane, neighbouring lanes side by side.
#include "dr_internal.h"
#include "dr_store.h"
#include "conv_bf16_dev.h"
#include "conv_f32_taps.h"

namespace dr {
namespace {

struct TapsArgs {
    const float *x, *w, *bias;
    float* y;
    int K, HW, W, C, R, S, rows, Kg, Ng, Q, PQ, sh, sw, y_ctot, relu;
    int x_bytes, w_bytes, grid_m;
};

template <int TM, int G, int D>
__global__ __launch_bounds__(512, 4) void conv_f32_taps_kernel(const TapsArgs a)
{
    constexpr int BM = TM * 32, BN = TAPS_BN, A_CHUNKS = 2 * G * BM, A_PER = (A_CHUNKS + 255) / 256, B_PER = G, STAGE = 2 * G * (BM + BN);
    __shared__ __attribute__((aligned(16))) f32x4 lds[2][STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // the filter blocks of a pixel tile, and neighbouring tiles, on one die
    const int nblk = (int)gridDim.x, die = (int)(blockIdx.x & 7), s = (int)(blockIdx.x >> 3), per = nblk >> 3, odd = nblk & 7;
    const int bid = die * per + min(die, odd) + s, m0 = bid % a.grid_m * BM, n0 = bid / a.grid_m * BN;
    const int slices = (a.rows + 1) / 2;

    if (wave >= 4) {
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, a.w_bytes, 0x00020000);
        const int lt = tid - 256;
        auto tap0 = [&](int g) { return g == G - 1 ? a.S - 4 : g * 4; };     // first tap of a group
        int va[A_PER], a_row[A_PER], vb[B_PER];
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int u = lt + i * 256, hg = u / BM, m = m0 + u - hg * BM;
            a_row[i] = hg / G;
            va[i] = u < A_CHUNKS && m < a.K ? (m * a.Kg + a_row[i] * a.S + tap0(hg - a_row[i] * G)) * 4 : OOB;
        }
        // B: pixel lt & 127; waves 4, 5 take rows and groups 0, 2, 4, .. , waves 6, 7 the others
        const int n = n0 + (lt & (BN - 1)), odd_hg = (wave - 4) >> 1;
        const int nn = n < a.Ng ? n : 0, img = nn / a.PQ, pix = nn - img * a.PQ, p = pix / a.Q, q = pix - p * a.Q;
        const int base = (img * a.C * a.HW + p * a.sh * a.W + q * a.sw) * 4;
#pragma unroll
        for (int i = 0; i < B_PER; ++i) {
            const int hg = 2 * i + odd_hg;
            vb[i] = n < a.Ng ? base + tap0(hg % G) * 4 : OOB;
        }
        f32x4 ra[A_PER], rb[B_PER];
        int r = 0, row = 0, soff_b = 0;                  // filter row within its channel, of all, and its offset in x
        auto advance = [&]() __attribute__((always_inline)) {
            ++row;
            soff_b += a.W * 4;
            if (++r == a.R) { r = 0; soff_b += (a.HW - a.R * a.W) * 4; }
        };
        auto load = [&]() __attribute__((always_inline)) {
            const int soff_a = row * a.S * 4, b0 = soff_b;
            if (row + 1 == a.rows) {                     // the last row has no partner: zeros in its place
#pragma unroll
                for (int i = 0; i < A_PER; ++i) va[i] = a_row[i] ? OOB : va[i];
#pragma unroll
                for (int i = 0; i < B_PER; ++i) vb[i] = 2 * i + odd_hg >= G ? OOB : vb[i];
            }
            advance();
            const int b1 = soff_b;
            advance();
#pragma unroll
            for (int i = 0; i < A_PER; ++i) ra[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, va[i], soff_a, 0));
#pragma unroll
            for (int i = 0; i < B_PER; ++i) rb[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, vb[i], 2 * i + odd_hg >= G ? b1 : b0, 0));
        };
        auto write = [&](int st) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < A_PER; ++i)
                if (A_CHUNKS % 256 == 0 || lt + i * 256 < A_CHUNKS) lds[st][lt + i * 256] = ra[i];
#pragma unroll
            for (int i = 0; i < B_PER; ++i) lds[st][A_CHUNKS + lt + i * 256] = rb[i];
        };
        load();
        write(0);
        if (slices > 1) load();
        ring_barrier();
        for (int k = 1; k < slices; ++k) {               // (buffer k & 1: slice k - 2 has been read)
            write(k & 1);
            if (k + 1 < slices) load();
            ring_barrier();
        }
        return;
    }

    const int half = lane >> 5, l32 = lane & 31;
    f32x16 acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    // The operands of a group are read while the group before it is multiplied; a slice's last group is multiplied behind the barrier
    f32x4 fa[2][TM], fb[2];
    auto read = [&](const f32x4* st, int g, int slot) __attribute__((always_inline)) {
        fb[slot] = st[A_CHUNKS + (half * G + g) * BN + wave * 32 + l32];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[slot][i] = st[(half * G + g) * BM + i * 32 + l32];
    };
    auto multiply = [&](int g, int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (g < G - 1 || t >= D)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[slot][i][t], fb[slot][t], acc[i], 0, 0, 0);
    };
    auto slice = [&](int k, auto st_c) __attribute__((always_inline)) {       // (two copies: LDS addresses are constants; G groups change the slots' roles from slice to slice)
        constexpr int ST = decltype(st_c)::value, FIRST = ST * G & 1;
#pragma unroll
        for (int g = 0; g < G - 1; ++g) {
            read(lds[ST], g + 1, (FIRST + g + 1) & 1);
            multiply(g, (FIRST + g) & 1);
        }
        if (k + 1 < slices) {
            ring_barrier();
            read(lds[1 - ST], 0, (FIRST + G) & 1);
        }
        multiply(G - 1, (FIRST + G - 1) & 1);
    };
    ring_barrier();
    read(lds[0], 0, 0);
    for (int k = 0; k < slices; k += 2) {
        slice(k, IC<0>{});
        if (k + 1 < slices) slice(k + 1, IC<1>{});
    }

    // ---- the store: a register is a filter of a pixel, 32 pixels side by side.  The filter's place is the store's scalar offset; lanes
    // without an output store out of range.
    const int n = n0 + wave * 32 + l32, img0 = n0 / a.PQ;
    const int img = n / a.PQ, pix = n - img * a.PQ;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)(a.y + (size_t)img0 * a.y_ctot * a.PQ), 0, 0x7FFFFFFF, 0x00020000);
    const __amdgpu_buffer_rsrc_t rbias = __builtin_amdgcn_make_buffer_rsrc((void*)a.bias, 0, a.bias ? a.K * 4 : 0, 0x00020000);
    const int mh = m0 + half * 4, vy = n < a.Ng ? (((img - img0) * a.y_ctot + mh) * a.PQ + pix) * 4 : OOB;
    const bool whole = m0 + BM <= a.K;                   // (wave-uniform)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            const int m4 = i * 32 + v4 * 8;
            const f32x4 bv = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rbias, (mh + m4) * 4, 0, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float o = acc[i][v4 * 4 + e] + bv[e];
                if (a.relu) o = fmaxf(o, 0.f);
                const int at = whole || mh + m4 + e < a.K ? vy : OOB;
#if defined(__HIP_DEVICE_COMPILE__)
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, o), ry, at, (m4 + e) * a.PQ * 4, 0);
#endif
            }
        }
}

template <int G, int D>
int launch_tm(const TapsArgs& a, int tm, unsigned blocks, hipStream_t st)
{
    if (tm == 1) hipLaunchKernelGGL((conv_f32_taps_kernel<1, G, D>), dim3(blocks), dim3(512), 0, st, a);
    else if (tm == 2) hipLaunchKernelGGL((conv_f32_taps_kernel<2, G, D>), dim3(blocks), dim3(512), 0, st, a);
    else hipLaunchKernelGGL((conv_f32_taps_kernel<3, G, D>), dim3(blocks), dim3(512), 0, st, a);
    return check_launch("conv_f32_taps");
}

long taps_blocks(const ConvGeom& g, int tm) { return ((long)g.K + tm * 32 - 1) / (tm * 32) * (((long)g.Ng + TAPS_BN - 1) / TAPS_BN); }

}  // namespace

// Filters 7, 8 or 10 to 12 taps wide (groups of 4 that overlap by at most a fifth), as conv_f32.hip's order over groups of 4 taps, which
// this kernel takes the place of.  Contractions of more than 64 filter rows on few pixels stay there, and with scratch memory shorter ones that are faster
// cut over workgroups (cut_beats_taps in conv_f32.hip).
bool conv_f32_taps_takes(const ConvGeom& g, const void* residual, const ConvSplit* split)
{
    const int G = (g.S + 3) / 4, D = 4 * G - g.S;
    if (g.nhwc || g.w_krsc || residual || (split && split->n > 1) || g.ph || g.pw || !((G == 2 && D <= 1) || (G == 3 && D <= 2))) return false;
    if (g.C * g.R > 64 && taps_blocks(g, 1) < device_cus()) return false;
    return taps_store_fits(g.K, g.y_ctot, g.P, g.Q);
}

int launch_conv_f32_taps(const ConvGeom& g, const float* x, const float* w, const float* bias, float* y, hipStream_t st)
{
    TapsArgs a;
    a.x = x; a.w = w; a.bias = bias;
    a.y = y + (size_t)g.y_coff * g.P * g.Q;
    a.K = g.K; a.HW = g.H * g.W; a.W = g.W; a.C = g.C; a.R = g.R; a.S = g.S; a.rows = g.C * g.R; a.Kg = g.Kg; a.Ng = g.Ng; a.Q = g.Q; a.PQ = g.P * g.Q;
    a.sh = g.sh; a.sw = g.sw; a.y_ctot = g.y_ctot; a.relu = g.relu;
    a.x_bytes = (int)((size_t)g.N * g.C * g.H * g.W * 4);
    a.w_bytes = (int)((size_t)g.K * g.Kg * 4);
    // few pixels: a filter block of 32 per workgroup, three times the workgroups (11x11 3 -> 96 at stride 4 on one image, AlexNet's first two
    // blocks 54.3 -> 42.4 us)
    int tm = taps_tm(g.K);
    if (taps_blocks(g, tm) < device_cus() / 2) tm = 1;
    a.grid_m = (g.K + tm * 32 - 1) / (tm * 32);
    const unsigned blocks = (unsigned)(a.grid_m * ((g.Ng + TAPS_BN - 1) / TAPS_BN));
    switch ((g.S + 3) / 4 * 10 + (4 - g.S % 4) % 4) {
    case 20: return launch_tm<2, 0>(a, tm, blocks, st);
    case 21: return launch_tm<2, 1>(a, tm, blocks, st);
    case 30: return launch_tm<3, 0>(a, tm, blocks, st);
    case 31: return launch_tm<3, 1>(a, tm, blocks, st);
    default: return launch_tm<3, 2>(a, tm, blocks, st);
    }
}

}  // namespace dr
