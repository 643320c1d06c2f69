// fp32 convolution on the bf16 matrix cores (NCHW, filters in KRSC order, C % 16 == 0, stride 1): every operand as the sum of three bf16 pieces.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel, n = (image, p, q), k = (16 channels, r, s, channel)
//
// Arithmetic.  The fp32 matrix instructions reach 156 TFLOP/s here, those of bf16 1750.  An fp32 operand is the sum of three bf16 values, exactly (24 bits of
// significand, 8 each; Henry, Tang, Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations", 2019); of the nine products
// of two operands the six largest are taken, the three left out are together at most 2^-24 of the product, so the ceiling is 1750 / 6 = 290 TFLOP/s.  The largest product and the five small ones have sums of their own, added once at the end: the matrix instruction cuts what it adds to
// a sum at the sum's last bit, and with one sum for all of them the error of 9216 positive products grew to four times that of fp32 instructions.  Against 64 bits,
// relative 2-norm of 32 x 32 blocks over contractions of 144 / 576 / 2400 normal x normal: fp32 instructions 2.2e-7 / 4.3e-7 / 8.8e-7, here 0.7e-7 / 1.4e-7 / 3.0e-7
// (with one sum 1.9e-7 / 3.7e-7 / 7.7e-7); 8 layers with operands of normal, one-signed and uniform values 0.30 to 0.37 of fp32 instructions', strided ones 0.32 to 0.40.  Where one
// product outweighs all others (values spread log-normally over e^+-12) the products left out and the second sum show: 0.6e-7 to 1.1e-7, fp32 instructions 0.3e-7 to 0.7e-7.
// Operands are scaled by 2^24 where they are cut, sums by 2^-48 at the end: the lower pieces of small values, subnormal ones too, then stay above the smallest normal bf16.
// (Unscaled, channels of 2^-118 beside one of 1 whose filters are 0 had an error of 8.8e-6 in the place of 0.9e-7.  Looking for eights of small operands took six
// instructions where scaling takes eight; 15 layers 0.99 to 1.05 times as fast as with that.)  What is too large for pieces then shows among the sums: infinities, NaN, operands of 2^104 and more, sums of 2^80 and more leave an
// infinity or a NaN.  The blocks of 32 x 32 outputs concerned are computed again by fp32 instructions (exact_block): the values that those give, at about a third of their speed.
//
// Structure.  One workgroup per compute unit walks its share of the tiles (conv_f32_pieces_plan.h).  Four waves load, cut operands into pieces and write LDS, four multiply;
// vector instructions and bf16 matrix instructions of different waves overlap (six per matrix instruction cost 9 %, the clock that the power leaves).  A slice is 32
// k: the filters of two taps of 16 channels, double buffered.  The activations of 16 channels are cut ONCE per tile, not once per tap: LDS holds the tile's
// patch of input pixels, twice, and a tap reads it at a uniform offset (cutting them for every tap kept the loading waves busy 1.8 times as long: 5x5 96 -> 256
// on 27 x 27 x 128 637 us, with the patch 534).  The walk is one stream: the next tile's patch and filters are loaded and cut while the tile before it is
// multiplied and stored.  What matters in the loading waves: no wait for loads just sent (a register copy where two paths meet costs the full latency per slice:
// 540 -> 509), scalar registers that do not spill (fresh_args), biases loaded before the first store and stores without a branch each (21 000 -> 5 000 cycles a tile).
// Measured on rectified operands, fp32 kernels before -> here: 5x5 96 -> 256 on 27 x 27 x 128 (115 GFLOP) 870 -> 500 us, 229 TFLOP/s at the 1.75 GHz that the power leaves;
// 3x3 96 -> 128 on 28 x 28 x 32 59 -> 35, 64 -> 192 on 56 x 56 x 32 182 -> 141; 64 -> 128 5x5 on 29 x 25 x 120 280 -> 167.  In the loop the matrix cores are busy 75 to 85 %.
#include <algorithm>

#include "conv_f32_cut.h"
#include "conv_f32_pieces_plan.h"

namespace dr {
namespace {

// LDS: for each piece and each 8 of a slice's k a run of rows (filters or pixels), 16 bytes each
template <int ROWS> constexpr int chunk_stride() { return ROWS * 16 + 64; }
template <int ROWS> constexpr int piece_stride() { return 4 * chunk_stride<ROWS>(); }
// the bytes of a stage of filters and of a patch
constexpr int filter_bytes(const PiecesTile& t) { return 2 * 3 * 4 * (t.bm * 16 + 64); }
constexpr int patch_bytes(const PiecesTile& t) { return 3 * 2 * (t.patch + 1) * 16; }
constexpr int pieces_lds()
{
    int most = 0;
    for (const PiecesTile& t : pieces_tiles) most = std::max(most, filter_bytes(t) + 2 * patch_bytes(t) + t.patch * 8);
    return most;
}

struct PatchArgs {
    KArgs k;
    unsigned long long by_pw, by_rows, by_pq, by_q;      // multipliers of div_small
};

// The patch of a tile: for each image that it touches the input rows under its output rows, Q + S - 1 pixels each, one below the other
struct Patch {
    int m0, n0, img0, p0, first_rows;
    __device__ __forceinline__ Patch(const PatchArgs& a, int tile, int BM, int BN)
    {
        const ConvGeom& g = a.k.g;
        const int nt = tile / a.k.grid_m;
        m0 = (tile - nt * a.k.grid_m) * BM;
        n0 = nt * BN;
        img0 = n0 / (g.P * g.Q);
        p0 = (n0 - img0 * g.P * g.Q) / g.Q;
        first_rows = g.P - p0 + g.R - 1;
    }
    __device__ __forceinline__ int row(const ConvGeom& g, int img, int p) const       // first input row of the outputs in row p of image img0 + img
    {
        return img == 0 ? p - p0 : first_rows + (img - 1) * (g.P + g.R - 1) + p;
    }
};

// The kernel's arguments, read again from here on: what the hot loops do not use is not kept in scalar registers across them (with everything kept, 60 values a
// slice went through vector registers).
__device__ __forceinline__ const PatchArgs& fresh_args(int job)
{
    auto p = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr() + (unsigned)job * sizeof(PatchArgs);
    asm volatile("" : "+s"(p));
    return *(const PatchArgs*)(const __attribute__((address_space(4))) PatchArgs*)p;
}

// tiles [tile0, tile0 + count) of a layer, by one workgroup
template <int TILE, int WGM, int WGN, int TM, int TN>
__device__ __forceinline__ void patch_tiles(const int job, const int tile0, const int count, unsigned char* const lds)
{
    constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, PATCH = pieces_tiles[TILE].patch, PATCH_UNITS = PATCH * 2 / 256;
    static_assert(BM == pieces_tiles[TILE].bm && BN == pieces_tiles[TILE].bn, "tile");
    constexpr int PATCH_CHUNK = (PATCH + 1) * 16, PATCH_PIECE = 2 * PATCH_CHUNK, PATCH_BYTES = 3 * PATCH_PIECE;
    constexpr int CSA = chunk_stride<BM>(), PSA = piece_stride<BM>(), STAGE = 3 * PSA;
    constexpr int AU = (BM * 4 + 255) / 256;     // units of 8 k of a slice of 32 that a loading lane takes
    static_assert(WGM * WGN == 4 && BM % 32 == 0, "tile");
    const PatchArgs& pa = fresh_args(job);
    const KArgs& a = pa.k;
    const ConvGeom& g = a.g;
    unsigned char* const patch = lds + filter_bytes(pieces_tiles[TILE]);
    int* const table = reinterpret_cast<int*>(patch + 2 * PATCH_BYTES);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int HW = g.H * g.W, PW = g.Q + g.S - 1, T = g.R * g.S, blocks = g.C >> 4, steps = T * blocks, slices = (steps + 1) >> 1;

    if (wave >= 4) {
        const int lt = tid - 256;
        int va[AU], a_ks[AU], a_lds[AU];
#pragma unroll
        for (int i = 0; i < AU; ++i) {
            const int U = i * 256 + lt, row = (U >> 1) % BM, c = U & 1;
            const int ks = __builtin_amdgcn_readfirstlane(U / (2 * BM));      // the same for a wave: 2 BM is a multiple of 64
            a_ks[i] = ks;
            va[i] = ks < 2 ? row * g.Kg * 4 + c * 32 : OOB;                   // (rows beyond the last filter lie behind the tensor)
            a_lds[i] = (ks * 2 + c) * CSA + row * 16;
        }
        const int plane = HW * 4, C = g.C, w_bytes = a.w_bytes, x_bytes = a.x_bytes, grid_m = a.grid_m;
        const float *const w = a.w, *const x = a.x;
        float ra[2][AU][8], rb[8];
        // A: the filters, a walk over (tile, 16 channels, tap) that runs three slices ahead
        int a_tile = tile0, a_step = 0, a_tap = 0, a_blk = 0, a_m = Patch(pa, tile0, BM, BN).m0 * g.Kg * 4;
        const int a_end = tile0 + count;
        auto a_next = [&]() __attribute__((always_inline)) {
            const int o = a_m + (a_tap * C + a_blk * 16) * 4;
            if (++a_tap == T) { a_tap = 0; ++a_blk; }
            return o;
        };
        auto load_a = [&](auto set_c) __attribute__((always_inline)) {
            constexpr int SET = decltype(set_c)::value;
            const int o0 = a_next(), o1 = a_next();
#pragma unroll
            for (int i = 0; i < AU; ++i) {
                const bool in = a_step + a_ks[i] < steps && a_tile < a_end;
                const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, in ? w_bytes : 0, 0x00020000);
                const int so = in ? (a_ks[i] ? o1 : o0) : 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, va[i] + h * 16, so, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) ra[SET][i][h * 4 + e] = v[e];
                }
            }
            if ((a_step += 2) >= steps) {
                a_step = a_tap = a_blk = 0;
                ++a_tile;
                if (grid_m > 1) {
                    const PatchArgs& f = fresh_args(job);
                    a_m = Patch(f, a_tile, BM, BN).m0 * f.k.g.Kg * 4;
                }
            }
        };
        auto write_a = [&](auto set_c) __attribute__((always_inline)) {
            constexpr int SET = decltype(set_c)::value;
#pragma unroll
            for (int i = 0; i < AU; ++i)
                if (BM * 4 % 256 == 0 || a_ks[i] < 2) put_pieces(ra[SET][i], lds + SET * STAGE + a_lds[i], PSA);
        };

        // B: the patches, a walk over (tile, 16 channels, unit)
        int b_tile = tile0, b_blk = 0, b_unit = 0, b_units = 0, b_pixels = 0, b_serial = 0, b_at = 0;      // b_serial: blocks before the one that rb belongs to
        auto patch_of = [&](int tile) __attribute__((always_inline)) {
            const PatchArgs& pa = fresh_args(job);
            const ConvGeom& g = pa.k.g;
            const Patch t(pa, tile, BM, BN);
            const int HW = g.H * g.W, PQ = g.P * g.Q, PW = g.Q + g.S - 1;
            const int n_last = min(t.n0 + BN, g.Ng) - 1, o = n_last - t.img0 * PQ, img = div_small(o, pa.by_pq), p = div_small(o - img * PQ, pa.by_q);
            b_pixels = (t.row(g, img, p) + g.R) * PW;
            b_units = (2 * b_pixels + 255) >> 8;
#pragma unroll
            for (int i = 0; i < PATCH_UNITS; ++i) {
                const int U = i * 256 + lt, c = U >= b_pixels, px = U - (c ? b_pixels : 0);
                int row = div_small(px, pa.by_pw), image = t.img0, ih = t.p0 - g.ph + row;
                const int iw = px - row * PW - g.pw;
                const int below = row - t.first_rows, k = div_small(max(below, 0), pa.by_rows);
                image = below >= 0 ? t.img0 + 1 + k : image;
                ih = below >= 0 ? below - k * (g.P + g.R - 1) - g.ph : ih;
                const bool ok = (U < 2 * b_pixels) & ((unsigned)ih < (unsigned)g.H) & ((unsigned)iw < (unsigned)g.W);
                table[U] = ok ? ((image * g.C + c * 8) * HW + ih * g.W + iw) * 4 : OOB;
            }
        };
        auto load_b = [&](int unit, float (&v)[8]) __attribute__((always_inline)) {
            const int cb = b_blk * 16 * plane;                            // (behind the last tile: the last one's again, which nobody writes)
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((char*)x + cb, 0, x_bytes - cb, 0x00020000);
            const int o = table[unit * 256 + lt];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = buf_load(rx, o, j * plane);
        };
        auto place = [&](int unit) __attribute__((always_inline)) {      // (lanes beyond the patch: the place behind it)
            const int U = unit * 256 + lt, at = U * 16 + (U >= b_pixels ? PATCH_CHUNK - b_pixels * 16 : 0);
            return U < 2 * b_pixels ? at : PATCH * 16;
        };
        auto b_next = [&]() __attribute__((always_inline)) {             // the unit that is written next, into rb (behind the last tile: nothing)
            if (++b_unit == b_units) {
                b_unit = 0;
                ++b_serial;
                if (++b_blk == blocks) {
                    b_blk = 0;
                    if (++b_tile < a_end) patch_of(b_tile);
                }
            }
            b_at = place(b_unit);
            load_b(b_unit, rb);
        };
        load_a(IC<0>{});
        patch_of(tile0);
        {
            float first[PATCH_UNITS][8];
#pragma unroll
            for (int i = 0; i < PATCH_UNITS; ++i)
                if (i < b_units) load_b(i, first[i]);
            load_a(IC<1>{});
            write_a(IC<0>{});
            load_a(IC<0>{});
#pragma unroll
            for (int i = 0; i < PATCH_UNITS; ++i)
                if (i < b_units) put_pieces(first[i], patch + place(i), PATCH_PIECE);
            b_unit = b_units - 1;
            b_next();
        }
        ring_barrier();
        // Iteration (tile, k), between two barriers: the multiplying waves are in slice k, which starts in block (2 k) / T of the tile.  The next slice's
        // filters, and a unit of the next block's patch, from the first slice that lies in this block altogether.
        int k = 0, m_blk = 0, m_serial = 0, next_start = (T + 1) >> 1;
        const int total = count * slices;
        auto iterate = [&](auto set_c) __attribute__((always_inline)) {
            write_a(set_c);
            __builtin_amdgcn_sched_barrier(0);       // (what is loaded goes to the registers that have just been read, and is waited for when it is written)
            load_a(set_c);
            if (k >= next_start) { ++m_blk; ++m_serial; next_start = ((m_blk + 1) * T + 1) >> 1; }
            if (b_serial == m_serial + 1) {
                put_pieces(rb, patch + (b_serial & 1) * PATCH_BYTES + b_at, PATCH_PIECE);
                __builtin_amdgcn_sched_barrier(0);
                b_next();
            }
            if (++k == slices) { k = 0; m_blk = 0; ++m_serial; next_start = (T + 1) >> 1; }
            ring_barrier();
        };
        for (int at = 0; at < total; at += 2) {
            iterate(IC<1>{});
            iterate(IC<0>{});
        }
        return;
    }

    const int half = lane >> 5, l32 = lane & 31, wm = wave / WGN, wn = wave % WGN;
    f32x16 acc[TM][TN], small[TM][TN];
    u32x4 fa[2][TM][3], fb[2][TN][3];
    int a_rd = half * CSA + (wm * TM * 32 + l32) * 16;       // (and the stage)
    int b_px[TN];                                // byte of the first tap's pixel in a patch buffer
    // the k-step that is read next: tap and patch buffer
    int t_r, t_s, t_off, t_step, t_buf = 0;
    const int S = g.S, R = g.R, row_step = (PW - g.S) * 16;
    auto tap_next = [&]() __attribute__((always_inline)) {
        if (++t_step >= steps) return;           // (beside filters that are 0)
        t_off += 16;
        if (++t_s == S) {
            t_s = 0;
            t_off += row_step;
            if (++t_r == R) { t_r = 0; t_buf = PATCH_BYTES - t_buf; t_off = t_buf; }
        }
    };
    auto read = [&](auto ks_c, int e) __attribute__((always_inline)) {       // piece e of k-step KS of the stage
        constexpr int KS = decltype(ks_c)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[KS][i][e] = *reinterpret_cast<const u32x4*>(lds + a_rd + e * PSA + KS * 2 * CSA + i * 512);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[KS][j][e] = *reinterpret_cast<const u32x4*>(patch + b_px[j] + t_off + e * PATCH_PIECE);
    };
    auto multiply = [&](auto ks_c, int x, int y) __attribute__((always_inline)) {
        constexpr int KS = decltype(ks_c)::value;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (x + y) small[i][j] = mfma(fa[KS][i][x], fb[KS][j][y], small[i][j]);
                else acc[i][j] = mfma(fa[KS][i][0], fb[KS][j][0], acc[i][j]);
    };
    auto step = [&](auto ks_c) __attribute__((always_inline)) {              // the products of k-step KS, between them the other one's operands are read
        constexpr int KS = decltype(ks_c)::value;
        multiply(ks_c, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        read(IC<1 - KS>{}, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ks_c, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        read(IC<1 - KS>{}, 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ks_c, 1, 0);
        __builtin_amdgcn_sched_barrier(0);
        read(IC<1 - KS>{}, 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ks_c, 1, 1);
        multiply(ks_c, 0, 2);
        multiply(ks_c, 2, 0);
    };
    ring_barrier();
    int stage = 0;
    for (int tile = tile0; tile < tile0 + count; ++tile) {
        {
        const PatchArgs& pa = fresh_args(job);
        const ConvGeom& g = pa.k.g;
        const Patch t(pa, tile, BM, BN);
        const int n_last = min(t.n0 + BN, g.Ng) - 1, PQ = g.P * g.Q, PW = g.Q + g.S - 1;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int o = min(t.n0 + (wn * TN + j) * 32 + l32, n_last) - t.img0 * PQ, img = div_small(o, pa.by_pq), pix = o - img * PQ, p = div_small(pix, pa.by_q);
            b_px[j] = half * PATCH_CHUNK + (t.row(g, img, p) * PW + pix - p * g.Q) * 16;
        }
        }
        t_r = t_s = t_step = 0;
        t_off = t_buf;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = small[i][j][v] = 0.f;
#pragma unroll
        for (int e = 0; e < 3; ++e) read(IC<0>{}, e);
        for (int k = 0; k < slices; ++k) {
            tap_next();
            step(IC<0>{});
            tap_next();
            a_rd += stage ? -STAGE : STAGE;
            stage ^= 1;
            ring_barrier();
            step(IC<1>{});                       // (after the tile's last slice it reads what is read again)
        }
        const KArgs& a = fresh_args(job).k;
        const Patch t(fresh_args(job), tile, BM, BN);
        finish_tile<TM, TN>(a, acc, small, t.m0 + wm * TM * 32, t.n0 + wn * TN * 32, t.n0, t.img0, fresh_args(job).by_pq);
        t_buf = PATCH_BYTES - t_buf;
    }
    if (count * slices & 1) ring_barrier();      // (the loading waves go in pairs of slices)
}

struct PiecesArgs {
    PatchArgs job[PIECES_LAYERS];                // (first: fresh_args)
    int n, type[PIECES_LAYERS];
    PiecesShare share[PIECES_LAYERS];
};

// TILE: the tile of all layers; PIECES_TILES: each layer has its own (a kernel by itself: with all of them in one the compiler moves 30 registers through memory)
template <int TILE>
__global__ __launch_bounds__(512, 2) void conv_f32_pieces_kernel(const PiecesArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[pieces_lds()];
    // consecutive workgroup ids are dealt to the 8 dies in turn: a range of tiles for each die
    const int G = (int)gridDim.x, id = (int)blockIdx.x, per = G >> 3, odd = G & 7, w = (id & 7) * per + min(id & 7, odd) + (id >> 3);
    for (int j = 0; j < a.n; ++j) {
        const PiecesShare& s = a.share[j];
        int i = 0;
        while (i + 1 < s.n && w >= s.first[i + 1]) ++i;
        const int count = s.per[i], tile = s.tile[i] + (w - s.first[i]) * count, type = TILE < PIECES_TILES ? TILE : a.type[j];
        if (count == 0) continue;
        if (type == 0) patch_tiles<0, 2, 2, 2, 2>(j, tile, count, lds);
        else if (type == 1) patch_tiles<1, 1, 4, 3, 1>(j, tile, count, lds);
        else if (type == 2) patch_tiles<2, 2, 2, 1, 2>(j, tile, count, lds);
        else patch_tiles<3, 1, 4, 2, 2>(j, tile, count, lds);
    }
}

PiecesLayer layer_of(const ConvGeom& g) { return PiecesLayer{g.N, g.C, g.H, g.W, g.K, g.R, g.S, g.sh, g.sw, g.P, g.Q}; }

}  // namespace

bool conv_f32_pieces_takes(const ConvGeom& g)
{
    const size_t xb = (size_t)g.N * g.C * g.H * g.W * 4, wb = (size_t)g.K * g.Kg * 4;
    return !g.nhwc && g.w_krsc && g.res_ctot == 0 && xb < (1ull << 31) && wb < (1ull << 31) && pieces_pays(layer_of(g), device_cus());
}

int launch_conv_f32_pieces(const ConvSmall* jobs, int n, hipStream_t st)
{
    const int cus = device_cus();
    int order[PIECES_LAYERS], best_type[PIECES_LAYERS] = {};
    PiecesLayer layer[PIECES_LAYERS];
    for (int i = 0; i < n; ++i) {
        if (jobs[i].res || (jobs[i].split && jobs[i].split->n > 1)) return fail(DR_ERR_UNSUPPORTED, "conv_f32_pieces: a residual or several destinations");
        order[i] = i;
        layer[i] = layer_of(jobs[i].g);
    }
    std::sort(order, order + n, [&](int p, int q) { return pieces_slices(layer[p]) > pieces_slices(layer[q]); });      // the longest tiles first
    PiecesPlan best;
    PiecesLayer sorted[PIECES_LAYERS];
    for (int i = 0; i < n; ++i) sorted[i] = layer[order[i]];
    if (!pieces_choose(n, sorted, cus, best_type, &best)) return fail(DR_ERR_UNSUPPORTED, "conv_f32_pieces: no plan for %d layers", n);
    PiecesArgs a{};
    a.n = n;
    for (int i = 0; i < n; ++i) {
        const ConvSmall& c = jobs[order[i]];
        const PiecesTile& t = pieces_tiles[best_type[i]];
        PatchArgs& p = a.job[i];
        p.k = conv_f32_args(c.g, (const float*)c.x, (const float*)c.w, c.bias, nullptr, (float*)c.y, nullptr, t.bn);
        p.k.grid_m = (c.g.K + t.bm - 1) / t.bm;
        p.k.grid_n = (int)(((long)c.g.Ng + t.bn - 1) / t.bn);
        auto magic = [](int d) { return ((1ull << 40) + (unsigned)d - 1) / (unsigned)d; };
        p.by_pw = magic(c.g.Q + c.g.S - 1); p.by_rows = magic(c.g.P + c.g.R - 1); p.by_pq = magic(c.g.P * c.g.Q); p.by_q = magic(c.g.Q);
        a.type[i] = best_type[i];
        a.share[i] = best.layer[i];
    }
    bool mixed = false;
    for (int i = 1; i < n; ++i) mixed |= best_type[i] != best_type[0];
    const dim3 grid((unsigned)best.workgroups), block(512);
    if (mixed) hipLaunchKernelGGL(conv_f32_pieces_kernel<PIECES_TILES>, grid, block, 0, st, a);
    else if (best_type[0] == 0) hipLaunchKernelGGL(conv_f32_pieces_kernel<0>, grid, block, 0, st, a);
    else if (best_type[0] == 1) hipLaunchKernelGGL(conv_f32_pieces_kernel<1>, grid, block, 0, st, a);
    else if (best_type[0] == 2) hipLaunchKernelGGL(conv_f32_pieces_kernel<2>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(conv_f32_pieces_kernel<3>, grid, block, 0, st, a);
    return check_launch("conv_f32_pieces");
}

}  // namespace dr
