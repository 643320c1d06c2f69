// fp32 convolution on the bf16 matrix cores, strided layers (NCHW, filters in KRSC order, C % 16 == 0): the arithmetic and the structure of conv_f32_pieces.hip, with
// the activations cut for every tap.  (A patch of strided layers is four times as large per output and serves a quarter of the taps.)
// Bound by the loading waves: a slice of 32 k is four units of eight operands to load, cut and write for each of their lanes (128 x 128 tiles), 2700 cycles for
// 1536 of matrix work.  At stride 2 5x5 256 -> 96 on 20 x 23 x 112 651 us in the fp32 kernel, 256 here; 3x3 96 -> 208 on 56 x 56 x 99 750 and 243.
#include <algorithm>

#include "conv_f32_cut.h"
#include "conv_f32_direct_plan.h"

namespace dr {
namespace {

struct DirectArgs {
    KArgs k;
    unsigned long long by_pq, by_q;              // multipliers of div_small
};
// The kernel's arguments, read again from here on (as fresh_args in conv_f32_pieces.hip)
__device__ __forceinline__ const DirectArgs& fresh_direct()
{
    auto p = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const DirectArgs*)(const __attribute__((address_space(4))) DirectArgs*)p;
}

struct TileAt {
    int m0, n0, img0;
    __device__ __forceinline__ TileAt(const KArgs& a, int tile, int BM, int BN)
    {
        const int nt = tile / a.grid_m;
        m0 = (tile - nt * a.grid_m) * BM;
        n0 = nt * BN;
        img0 = n0 / (a.g.P * a.g.Q);
    }
};

template <int WGM, int WGN, int TM, int TN>
__device__ __forceinline__ void direct_tiles(const int tile0, const int count, unsigned char* const lds)
{
    constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, STEPS = 2;
    using LA = CutLayout<BM, STEPS>;
    using LB = CutLayout<BN, STEPS>;
    constexpr int STAGE = LA::BYTES + LB::BYTES, AU = (BM * 4 + 255) / 256;
    static_assert(WGM * WGN == 4 && BN == 128, "tile");
    const DirectArgs& da = fresh_direct();
    const KArgs& a = da.k;
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = g.R * g.S * (g.C >> 4), slices = (steps + 1) >> 1, end = tile0 + count;

    if (wave >= 4) {
        const int lt = tid - 256;
        int va[AU], a_ks[AU], a_lds[AU];
#pragma unroll
        for (int i = 0; i < AU; ++i) {
            const int U = i * 256 + lt, row = (U >> 1) % BM, c = U & 1;
            const int ks = __builtin_amdgcn_readfirstlane(U / (2 * BM));      // the same for a wave: 2 BM is a multiple of 64
            a_ks[i] = ks;
            va[i] = ks < 2 ? row * g.Kg * 4 + c * 32 : OOB;                   // (rows beyond the last filter lie behind the tensor)
            a_lds[i] = (ks * 2 + c) * LA::CHUNK + row * 16;
        }
        const int H = g.H, W = g.W, C = g.C, S = g.S, plane = H * W * 4, w_bytes = a.w_bytes, x_bytes = a.x_bytes, px = lt & (BN - 1);
        const int eight = __builtin_amdgcn_readfirstlane(lt / BN);            // which 8 of a k-step's channels
        const float *const w = a.w, *const x = a.x;
        float ra[2][AU][8], rb[2][2][8];
        // a walk over (tile, tap, 16 channels), two k-steps at a time
        int tile = tile0, step = 0, r = 0, t = 0, c0 = 0, a_m, ih0, iw0, xoff0;
        auto at_tile = [&]() __attribute__((always_inline)) {
            const DirectArgs& f = fresh_direct();
            const ConvGeom& g = f.k.g;
            const TileAt at(f.k, tile, BM, BN);
            const int PQ = g.P * g.Q, n = at.n0 + px, o = min(n, g.Ng - 1) - at.img0 * PQ, img = div_small(o, f.by_pq), pix = o - img * PQ, p = div_small(pix, f.by_q);
            a_m = at.m0 * g.Kg * 4;
            ih0 = n < g.Ng ? p * g.sh - g.ph : -(1 << 30);
            iw0 = (pix - p * g.Q) * g.sw - g.pw;
            xoff0 = (int)((unsigned)((at.img0 + img) * C) * (unsigned)(H * W) + (unsigned)(p * g.sh - g.ph) * (unsigned)W + (unsigned)iw0);
        };
        at_tile();
        auto load = [&](auto set_c) __attribute__((always_inline)) {
            constexpr int SET = decltype(set_c)::value;
#pragma unroll
            for (int i = 0; i < AU; ++i) {
                const bool in = step + a_ks[i] < steps && tile < end;
                const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, in ? w_bytes : 0, 0x00020000);
                const int so = in ? a_m + (step + a_ks[i]) * 64 : 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, va[i] + h * 16, so, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) ra[SET][i][h * 4 + e] = v[e];
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const bool in = step + u < steps && tile < end;
                const bool ok = in & ((unsigned)(ih0 + r) < (unsigned)H) & ((unsigned)(iw0 + t) < (unsigned)W);
                const int vo = ok ? (xoff0 + r * W + t) * 4 : OOB, cb = (c0 + eight * 8) * plane;
                const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((char*)x + cb, 0, x_bytes - cb, 0x00020000);
#pragma unroll
                for (int j = 0; j < 8; ++j) rb[SET][u][j] = buf_load(rx, vo, j * plane);
                if ((c0 += 16) == C) { c0 = 0; if (++t == S) { t = 0; ++r; } }
            }
            if ((step += 2) >= steps) {
                step = r = t = c0 = 0;
                if (++tile < end) at_tile();
            }
        };
        auto write = [&](auto set_c) __attribute__((always_inline)) {
            constexpr int SET = decltype(set_c)::value;
#pragma unroll
            for (int i = 0; i < AU; ++i)
                if (BM * 4 % 256 == 0 || a_ks[i] < 2) put_pieces(ra[SET][i], lds + SET * STAGE + a_lds[i], LA::PIECE);
#pragma unroll
            for (int u = 0; u < 2; ++u) put_pieces(rb[SET][u], lds + SET * STAGE + LA::BYTES + (u * 2 + eight) * LB::CHUNK + px * 16, LB::PIECE);
            __builtin_amdgcn_sched_barrier(0);       // (what is loaded goes to the registers that have just been read)
        };
        load(IC<0>{});
        load(IC<1>{});
        write(IC<0>{});
        load(IC<0>{});
        ring_barrier();
        auto iterate = [&](auto set_c) __attribute__((always_inline)) {
            write(set_c);
            load(set_c);
            ring_barrier();
        };
        for (int at = 0; at < count * slices; at += 2) {
            iterate(IC<1>{});
            iterate(IC<0>{});
        }
        return;
    }

    const int wm = wave / WGN, wn = wave % WGN;
    f32x16 acc[TM][TN], small[TM][TN];
    int stage = 0;
    ring_barrier();
    for (int tile = tile0; tile < end; ++tile) {
        multiply_tile<WGM, WGN, TM, TN, STEPS>(lds, slices, stage, acc, small);
        const DirectArgs& f = fresh_direct();
        const TileAt at(f.k, tile, BM, BN);
        finish_tile<TM, TN>(f.k, acc, small, at.m0 + wm * TM * 32, at.n0 + wn * TN * 32, at.n0, at.img0, f.by_pq);
    }
    if (count * slices & 1) ring_barrier();          // (the loading waves go in pairs of slices)
}

template <int TILE>
__global__ __launch_bounds__(512, 2) void conv_f32_direct_kernel(const DirectArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * cut_stage<direct_tile[TILE].bm, DIRECT_BN, 2>()];
    // consecutive workgroup ids are dealt to the 8 dies in turn: a range of tiles for each die
    const int G = (int)gridDim.x, id = (int)blockIdx.x, per = G >> 3, odd = G & 7, w = (id & 7) * per + min(id & 7, odd) + (id >> 3);
    const int tiles = a.k.grid_m * a.k.grid_n, whole = tiles / G, rest = tiles - whole * G, tile = w * whole + min(w, rest), count = whole + (w < rest);
    if constexpr (TILE == 0) direct_tiles<2, 2, 2, 2>(tile, count, lds);
    else if constexpr (TILE == 1) direct_tiles<1, 4, 3, 1>(tile, count, lds);
    else direct_tiles<2, 2, 1, 2>(tile, count, lds);
}

PiecesLayer layer_of(const ConvGeom& g) { return PiecesLayer{g.N, g.C, g.H, g.W, g.K, g.R, g.S, g.sh, g.sw, g.P, g.Q}; }

}  // namespace

bool conv_f32_direct_takes(const ConvGeom& g)
{
    const size_t xb = (size_t)g.N * g.C * g.H * g.W * 4, wb = (size_t)g.K * g.Kg * 4;
    return !g.nhwc && g.w_krsc && g.res_ctot == 0 && xb < (1ull << 31) && wb < (1ull << 31) && direct_pays(layer_of(g), device_cus());
}

int launch_conv_f32_direct(const ConvSmall& c, hipStream_t st)
{
    if (c.res || (c.split && c.split->n > 1)) return fail(DR_ERR_UNSUPPORTED, "conv_f32_direct: a residual or several destinations");
    double us;
    const int cus = device_cus(), tile = direct_best(layer_of(c.g), cus, &us), bm = direct_tile[tile].bm;
    DirectArgs a;
    a.k = conv_f32_args(c.g, (const float*)c.x, (const float*)c.w, c.bias, nullptr, (float*)c.y, nullptr);
    a.k.grid_m = (c.g.K + bm - 1) / bm;
    a.k.grid_n = (int)(((long)c.g.Ng + DIRECT_BN - 1) / DIRECT_BN);
    auto magic = [](int d) { return ((1ull << 40) + (unsigned)d - 1) / (unsigned)d; };
    a.by_pq = magic(c.g.P * c.g.Q); a.by_q = magic(c.g.Q);
    const dim3 grid((unsigned)std::min((long)cus, direct_count(layer_of(c.g), direct_tile[tile]))), block(512);
    if (tile == 0) hipLaunchKernelGGL(conv_f32_direct_kernel<0>, grid, block, 0, st, a);
    else if (tile == 1) hipLaunchKernelGGL(conv_f32_direct_kernel<1>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(conv_f32_direct_kernel<2>, grid, block, 0, st, a);
    return check_launch("conv_f32_direct");
}

}  // namespace dr
