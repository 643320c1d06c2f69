// fp32 convolution forward (Eq. (7): Y_j = (W * X)_j + B_j) as an implicit GEMM on the gfx950
// matrix cores.
//
//   D[m][n] = sum_k A[m][k] * B[k][n]     m = output channel        (M  = K filters)
//                                         n = (image, p, q)         (Ng = N*P*Q)
//                                         k = (c, r, s)             (Kg = C*R*S)
//   A = the KCRS weight tensor viewed as an M x Kg matrix (no copy),
//   B = the im2col matrix, never materialised: each element is gathered from NCHW x on the fly.
//
// A workgroup of 256 threads (4 wave64) owns a BM x BN tile of D and walks Kg in slices of BK.
// Both operand slices are staged in LDS with the slice's k index contiguous per row (rows padded by
// 4 floats so that 128-bit LDS accesses of consecutive rows fall in distinct banks).
// v_mfma_f32_32x32x2_f32 consumes two k per instruction, one from lanes 0-31 and one from lanes
// 32-63; of every 16 k of a slice the kernel gives lane half g those in [8g, 8g + 8), so every lane
// fetches its A (or B) values of a slice with BK/8 128-bit LDS reads, and the products of an output are
// added in the same order whatever the depth of a slice (a layer's bits do not depend on whether it
// shares a launch, where slices are 16 deep).  Global loads run PF slices ahead of
// the MFMAs in registers (PF register sets), LDS is double buffered, one barrier per slice.  With
// lanes running along n, both the gather from x and the store to NCHW y are coalesced.  Bias, the
// optional residual sum and ReLU are applied in the store.
//
// On this GPU fp32 MFMA and ordinary vector-ALU instructions do not overlap (measured: their times
// add), so every address computation in the loop costs matrix throughput.  Two slice orders exist:
//   CF = true  ("channel fastest": filters given in KRSC order, C % BK == 0): a slice is BK
//        consecutive channels of one filter tap (r, s).  All per-lane offsets are loop invariants;
//        the slice only moves a wave-uniform scalar offset, which rides in the buffer instructions'
//        scalar operand, and the padding test is redone once per tap.  Almost no vector-ALU work
//        per slice, and the filter rows are read with 16-byte loads.
//   CF = false (filters in KCRS order, any shape): k runs in KCRS order.  The workgroup first writes a
//        table k -> (offset of x[0][c][r][s], r, s) to LDS (contractions of up to KTAB elements, which
//        covers the small-channel first layers this path is for); an element's k is the same for a
//        whole wave, so its table entry arrives by one broadcast LDS read and the lane adds its
//        pixel's base offset; with padding it also tests the (r, s) bits of two per-lane masks of
//        valid window rows and columns.  Filters of at most 31 taps use one word per entry (offset and tap) and one
//        per-lane mask of taps, for contractions of up to KTAB1 elements whose offsets fit the word (3x3 64 -> 192 at stride 2 on 56 x 56 x 32, which
//        decoded (c, r, s) element by element before: 81 -> 69 us).  Longer contractions decode (c, r, s) per element.
//        Without padding and with a filter width S that rounds up to a multiple of 4 cheaply (11 -> 12,
//        7 -> 8), k instead runs over (c, r, groups of 4 taps): the four activations of a group are
//        neighbours in memory and arrive by one 16-byte load per lane (consecutive pixels at stride 4
//        read consecutive 16-byte pieces), the taps added by the rounding count as zeros on both sides.
//        That quarter of the load instructions is what the first layer of AlexNet was limited by.
//
// A layer with fewer tiles than the device has compute units (one image, or a few) leaves most of the
// matrix cores idle while each workgroup walks the whole contraction alone.  Given scratch memory, the
// launcher then cuts the contraction into `splits` ranges of slices: blockIdx.y picks the range, the
// workgroup stores its raw partial sums to part[split][m][n], and conv_f32_reduce_kernel adds the
// ranges in a fixed order and applies bias, residual and ReLU.  No atomics: the result does not
// depend on the order in which workgroups finish.
#include <algorithm>
#include <type_traits>

#include "conv_f32_dev.h"
#include "conv_f32_kcrs33.h"
#include "conv_f32_table.h"

namespace dr {
namespace {

constexpr int NT = 256;       // threads per workgroup
constexpr int KTAB = 512;     // CF = false: contraction elements (or groups of 4 taps) whose two-word table entries are used
constexpr int KTAB1 = 2048;   // CF = false, at most 31 taps: elements whose one-word entries fit the LDS table (8 KB)

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding
// global load (its fence covers all address spaces), which would serialise the register prefetch
// with the MFMAs; global memory needs no ordering inside this kernel.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// BM x BN: workgroup tile; WGM x WGN: wave grid (4 waves); BK: k per LDS slice; PF: prefetch distance
// in slices; CF: slice order (see above); FR, FS: compile-time filter size for CF = false (0 = taken
// from the geometry at run time); TAB1: the table of one-word entries; SPLIT: the workgroup takes range blockIdx.y of the contraction and
// stores raw partial sums.
// The tile is computed by workgroup `block` of the layer's grid_m grid_n.  The LDS arrays (two buffers of BM resp. BN rows, the
// table of CF = false) are separate objects of the kernel: carved out of one array, the compiler orders every read of one
// operand behind the writes of the other (20 % slower).
template <int BM, int BN, int WGM, int WGN, int BK, int PF, bool CF, int FR, int FS, bool TAB1, bool SPLIT>
__device__ __forceinline__ void conv_f32_tile(const KArgs a, const int block, float (*const As)[BM * (BK + 4)], float (*const Bs)[BN * (BK + 4)], int* const ktab)
{
    constexpr int WM = BM / WGM, WN = BN / WGN;   // wave tile
    constexpr int TM = WM / 32, TN = WN / 32;     // 32x32 MFMA tiles per wave
    constexpr int LDT = BK + 4;                   // padded LDS row (floats)
    constexpr int KQ = BK / 4;                    // float4 groups per row
    constexpr int HK = BK / 2;                    // k per lane half
    static_assert(WGM * WGN == 4 && TM >= 1 && TN >= 1, "bad tiling");
    static_assert(BK == 16 || BK == 32, "BK");
    static_assert(PF == 1 || PF == 2, "PF");
    constexpr int A_F4 = BM * KQ;                 // float4 groups in an A slice
    constexpr int B_F4 = BN * KQ;
    constexpr int A_PER = (A_F4 + NT - 1) / NT;
    constexpr int B_PER = B_F4 / NT;
    static_assert(B_F4 % NT == 0, "BN * BK must be a multiple of 1024");
    static_assert(BN <= NT && NT % BN == 0, "one n per thread");

    const ConvGeom& g = a.g;
    const int R = FR ? FR : g.R, S = FS ? FS : g.S;
    const int RS = R * S;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    const int half = lane >> 5, l32 = lane & 31;

    // Workgroup -> tile.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs; the remap
    // gives each XCD a contiguous range of tiles (m fastest), so the tiles that share an input
    // region share an L2.
    int bid = block;
    const int nblk = a.grid_m * a.grid_n;
    if (nblk % 8 == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);
    const int m0 = (bid % a.grid_m) * BM;
    const int n0 = (bid / a.grid_m) * BN;

    const int HW = g.H * g.W, PQ = g.P * g.Q;

    // Global reads go through buffer descriptors: a lane whose element lies outside the tensor (zero
    // padding, ragged M / n / k tails) gets its offset moved beyond num_records and the hardware
    // returns 0 for it without touching memory, so the gather needs no branches.
    constexpr int OOB = (int)0x80000000;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, a.w_bytes, 0x00020000);

    // ---- per-thread gather state for B: one fixed n, B_PER groups of 4 consecutive k per slice
    constexpr int BKQ_STEP = NT / BN;             // k-groups covered by one pass of the workgroup
    const int bn = tid % BN;
    const int bkq0 = tid / BN;
    const int ng = n0 + bn;
    const bool n_ok = ng < g.Ng;
    int ih0 = -(1 << 30), iw0 = -(1 << 30);      // fails every bounds test when n is out of range
    int xoff0 = 0;                                // element offset of x[img][0][ih0][iw0]
    if (n_ok) {
        const int img = ng / PQ, pix = ng - img * PQ;
        const int p = pix / g.Q, q = pix - p * g.Q;
        ih0 = p * g.sh - g.ph;
        iw0 = q * g.sw - g.pw;
        // (a padded filter taller than a wide map: offsets of rows outside it may pass 2^31, their sum with the tap's does not)
        xoff0 = (int)((unsigned)(img * g.C * HW) + (unsigned)ih0 * (unsigned)g.W + (unsigned)iw0);
    }
    // ---- CF = false: the k table and this lane's masks of window rows / columns inside the image
    const bool rg = !CF && !TAB1 && a.row_groups;
    const int S4 = (S + 3) & ~3;
    const int kg_eff = rg ? g.C * R * S4 : g.Kg;     // contraction length including the taps added by rounding S up
    const int ktab_n = (kg_eff + BK - 1) / BK * BK;
    const bool use_tab = !CF && !TAB1 && !rg && ktab_n <= KTAB && R <= 31 && S <= 31;
    const bool nopad = g.ph == 0 && g.pw == 0;      // then every window lies inside the image
    unsigned rowmask = 0, colmask = 0;
    unsigned tap_out = 0xFFFFFFFFu;                  // (one-word table) bit r S + s: that tap lies outside the image; bits beyond: set
    if constexpr (!CF) {
        if constexpr (TAB1) {
            // one word per k: offset of x[0][c][r][s] in elements, and the tap
            for (int k = tid; k < ktab_n; k += NT) {
                int e = tab1_entry(0, TAB1_NO_TAP);
                if (k < g.Kg) {
                    const int c = k / RS, rs = k - c * RS, r = rs / S;
                    e = tab1_entry(c * HW + r * g.W + rs - r * S, rs);
                }
                ktab[k] = e;
            }
            if (n_ok)
                for (int r = 0, bit = 0; r < R; ++r)
                    for (int s_ = 0; s_ < S; ++s_, ++bit)
                        if ((unsigned)(ih0 + r) < (unsigned)g.H && (unsigned)(iw0 + s_) < (unsigned)g.W) tap_out &= ~(1u << bit);
            lds_barrier();                            // the table is complete before the first slice is gathered
        }
        if (use_tab) {
            for (int k = tid; k < ktab_n; k += NT) {
                int off = OOB, rs_bits = 31;          // beyond the contraction: the load returns 0 (mask bit 31 is never set)
                if (k < g.Kg) {
                    const int c = k / RS, rs = k - c * RS, r = rs / S, s_ = rs - r * S;
                    off = (int)(((unsigned)(c * HW) + (unsigned)r * (unsigned)g.W + (unsigned)s_) * 4u);
                    rs_bits = r | (s_ << 8);
                }
                ktab[2 * k] = off;
                ktab[2 * k + 1] = rs_bits;
            }
            if (n_ok) {
                for (int r = 0; r < R; ++r) rowmask |= ((unsigned)(ih0 + r) < (unsigned)g.H ? 1u : 0u) << r;
                for (int s_ = 0; s_ < S; ++s_) colmask |= ((unsigned)(iw0 + s_) < (unsigned)g.W ? 1u : 0u) << s_;
            }
            lds_barrier();                            // the table is complete before the first slice is gathered
        }
        if (rg) {
            // per group of 4 taps: {byte offset of x[0][c][r][s0], element offset of w[0][c][r][s0] | taps that exist << 24}
            for (int gq = tid; gq < ktab_n / 4; gq += NT) {
                int xo = OOB, meta = 0;
                const int kk = gq * 4;
                if (kk < kg_eff) {
                    const int c = kk / (R * S4), rem = kk - c * R * S4, r = rem / S4, s0 = rem - r * S4;
                    xo = (c * HW + r * g.W + s0) * 4;
                    meta = ((c * R + r) * S + s0) | (min(4, S - s0) << 24);
                }
                ktab[2 * gq] = xo;
                ktab[2 * gq + 1] = meta;
            }
            lds_barrier();
        }
    }
    const int bbase = n_ok ? (int)((unsigned)xoff0 * 4u) : OOB;        // (table paths) byte offset of this lane's window origin

    // ---- per-thread state for A: rows f / KQ of the slice, byte offset of the row start
    const bool vecA = (g.Kg & 3) == 0;
    int arow[A_PER];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
        const int f = tid + i * NT;
        const int gm = m0 + f / KQ;
        arow[i] = ((A_F4 % NT == 0 || f < A_F4) && gm < g.K) ? gm * g.Kg * 4 : OOB;
    }

    f32x4 ra[PF][A_PER], rb[PF][B_PER];

    // ---- CF = true: loader state.  Slices are visited tap by tap, BK channels at a time.
    int ld_c0 = 0, ld_r = 0, ld_s = 0;            // wave-uniform position of the next slice to load
    int vb[CF ? B_PER : 1][4];                    // per-lane byte offsets of the 4 channels of a group
    int va[CF ? A_PER : 1];                       // per-lane byte offset of a float4 of the filter row
    if constexpr (CF) {
#pragma unroll
        for (int i = 0; i < A_PER; ++i) va[i] = arow[i] + ((tid + i * NT) % KQ) * 16;
    }
    auto tap_offsets = [&]() {   // padding test of tap (ld_r, ld_s) for this lane's pixel
        const bool ok = ((unsigned)(ih0 + ld_r) < (unsigned)g.H) & ((unsigned)(iw0 + ld_s) < (unsigned)g.W);      // (no branch)
        const int base = ok ? (xoff0 + ld_r * g.W + ld_s) * 4 : OOB;
#pragma unroll
        for (int i = 0; i < B_PER; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) vb[CF ? i : 0][j] = base + ((bkq0 + i * BKQ_STEP) * 4 + j) * HW * 4;
    };

    // this workgroup's range of slices: [s_begin, s_begin + nslices)
    const int nslices_all = CF ? RS * (g.C / BK) : (kg_eff + BK - 1) / BK;
    const int s_begin = SPLIT ? (int)blockIdx.y * a.slices_per_split : 0;
    const int nslices = SPLIT ? min(a.slices_per_split, nslices_all - s_begin) : nslices_all;
    if constexpr (CF && SPLIT) {
        if (s_begin) {
            const int per_tap = g.C / BK, tap = s_begin / per_tap;
            ld_c0 = (s_begin - tap * per_tap) * BK;
            ld_r = tap / S;
            ld_s = tap - ld_r * S;
            if (ld_c0) tap_offsets();   // load_slice computes them itself at the first slice of a tap
        }
    }

    auto load_slice = [&](int it, auto set_c) {
        constexpr int SET = decltype(set_c)::value;
        if constexpr (CF) {
            if (ld_c0 == 0) tap_offsets();
            const int sa = ((ld_r * S + ld_s) * g.C + ld_c0) * 4;   // scalar parts of the addresses
            const int sb = ld_c0 * HW * 4;
#pragma unroll
            for (int i = 0; i < A_PER; ++i)
                ra[SET][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, va[i], sa, 0));
#pragma unroll
            for (int i = 0; i < B_PER; ++i) {
                f32x4 v;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = buf_load(rx, vb[i][j], sb);
                rb[SET][i] = v;
            }
            ld_c0 += BK;
            if (ld_c0 == g.C) { ld_c0 = 0; if (++ld_s == S) { ld_s = 0; ++ld_r; } }
        } else {
            const int k0 = (s_begin + it) * BK;
            if (rg) {
#pragma unroll
                for (int i = 0; i < A_PER; ++i) {
                    const int meta = ktab[2 * (k0 / 4 + (tid + i * NT) % KQ) + 1];
                    const int ao = meta & 0xFFFFFF, nt = meta >> 24;
                    f32x4 v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = buf_load(rw, j < nt ? arow[i] + (ao + j) * 4 : OOB, 0);
                    ra[SET][i] = v;
                }
#pragma unroll
                for (int i = 0; i < B_PER; ++i) {
                    const int gq = k0 / 4 + bkq0 + i * BKQ_STEP;              // the same for the whole wave
                    const int xo = ktab[2 * gq], nt = ktab[2 * gq + 1] >> 24;
                    const int vo = (int)((unsigned)bbase + (unsigned)xo);
                    f32x4 v;
                    if ((unsigned)vo < (unsigned)a.x_bytes && (unsigned)vo + 16u > (unsigned)a.x_bytes) {
                        // the tensor's last few elements: one by one, each checked against the end
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[j] = buf_load(rx, vo + 4 * j, 0);
                    } else {
                        v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, vo, 0, 0));
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = j < nt ? v[j] : 0.f;
                    rb[SET][i] = v;
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < A_PER; ++i) {
                const int gk = k0 + ((tid + i * NT) % KQ) * 4;
                const int off = arow[i] + gk * 4;
                if (vecA) {
                    ra[SET][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, gk < g.Kg ? off : OOB, 0, 0));
                } else {
                    f32x4 v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = buf_load(rw, gk + j < g.Kg ? off + 4 * j : OOB, 0);
                    ra[SET][i] = v;
                }
            }
            if constexpr (TAB1) {
                typedef int i32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
                for (int i = 0; i < B_PER; ++i) {
                    const i32x4 e = *reinterpret_cast<const i32x4*>(&ktab[k0 + (bkq0 + i * BKQ_STEP) * 4]);   // the same for the whole wave
                    f32x4 v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int vo = bbase + (tab1_offset(e[j]) << 2);
                        v[j] = buf_load(rx, (int)((tap_out >> tab1_tap(e[j])) << 31) | vo, 0);     // a tap outside: sign bit set, beyond the buffer
                    }
                    rb[SET][i] = v;
                }
            } else if (use_tab) {
#pragma unroll
                for (int i = 0; i < B_PER; ++i) {
                    const int gk = k0 + (bkq0 + i * BKQ_STEP) * 4;            // the same for the whole wave
                    typedef int i32x4 __attribute__((ext_vector_type(4)));
                    const i32x4 e01 = *reinterpret_cast<const i32x4*>(&ktab[2 * gk]);
                    const i32x4 e23 = *reinterpret_cast<const i32x4*>(&ktab[2 * gk + 4]);
                    const int off[4] = {e01[0], e01[2], e23[0], e23[2]}, rsb[4] = {e01[1], e01[3], e23[1], e23[3]};
                    f32x4 v;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        int vo = (int)((unsigned)bbase + (unsigned)off[j]);
                        if (!nopad) {
                            const bool ok = ((rowmask >> (rsb[j] & 255)) & (colmask >> (rsb[j] >> 8)) & 1u) != 0;
                            vo = ok ? vo : OOB;
                        }
                        v[j] = buf_load(rx, vo, 0);
                    }
                    rb[SET][i] = v;
                }
            } else {
#pragma unroll
            for (int i = 0; i < B_PER; ++i) {
                const int gk = k0 + (bkq0 + i * BKQ_STEP) * 4;
                int c = gk / RS;
                int rs = gk - c * RS;
                int r = rs / S;
                int s = rs - r * S;
                f32x4 v;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool ok = (gk + j < g.Kg) && (unsigned)(ih0 + r) < (unsigned)g.H && (unsigned)(iw0 + s) < (unsigned)g.W;
                    v[j] = buf_load(rx, ok ? (xoff0 + c * HW + r * g.W + s) * 4 : OOB, 0);
                    if (++s == S) { s = 0; if (++r == R) { r = 0; ++c; } }
                }
                rb[SET][i] = v;
            }
            }
        }
    };

    auto store_slice = [&](int buf, auto set_c) {
        constexpr int SET = decltype(set_c)::value;
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int f = tid + i * NT;
            if (A_F4 % NT == 0 || f < A_F4)
                *reinterpret_cast<f32x4*>(&As[buf][(f / KQ) * LDT + (f % KQ) * 4]) = ra[SET][i];
        }
#pragma unroll
        for (int i = 0; i < B_PER; ++i)
            *reinterpret_cast<f32x4*>(&Bs[buf][bn * LDT + (bkq0 + i * BKQ_STEP) * 4]) = rb[SET][i];
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // One slice: MFMAs on LDS buffer it&1; then register set SET (slice it+1, loaded PF slices ago)
    // moves to the other LDS buffer and is refilled with slice it+1+PF.
    auto slice_step = [&](int it, auto set_c) {
        const int buf = it & 1;
        f32x4 fa[TM][HK / 4], fb[TN][HK / 4];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const float* p = &As[buf][(wm * WM + i * 32 + l32) * LDT + half * 8];
#pragma unroll
            for (int h = 0; h < HK / 4; ++h) fa[i][h] = *reinterpret_cast<const f32x4*>(p + (h >> 1) * 16 + (h & 1) * 4);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const float* p = &Bs[buf][(wn * WN + j * 32 + l32) * LDT + half * 8];
#pragma unroll
            for (int h = 0; h < HK / 4; ++h) fb[j][h] = *reinterpret_cast<const f32x4*>(p + (h >> 1) * 16 + (h & 1) * 4);
        }
        auto products = [&](auto from_c, auto to_c) {
#pragma unroll
            for (int kk = decltype(from_c)::value; kk < decltype(to_c)::value; ++kk)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][kk >> 2][kk & 3], fb[j][kk >> 2][kk & 3],
                                                                         acc[i][j], 0, 0, 0);
        };
        // The next slice goes to LDS and the one behind it is asked for in the middle of the products: a matrix instruction takes 64 cycles and whatever
        // does not need the vector ALU is issued meanwhile.  (Behind the products it was a wave's own time: 3a slim on 64 images 165 us and 159,
        // 3x3 32 -> 256 on 30 x 45 x 9 52 and 48; loads that are always made, past the end from an empty buffer, so that the wait for a slice is not one
        // for the next slice too: 4 % slower, here and in the parameter gradient.)
        products(IC<0>{}, IC<4>{});
        __builtin_amdgcn_sched_barrier(0);
        if (it + 1 < nslices) {
            store_slice(buf ^ 1, set_c);
            if (it + 1 + PF < nslices) load_slice(it + 1 + PF, set_c);
        }
        __builtin_amdgcn_sched_barrier(0);
        products(IC<4>{}, IC<HK>{});
        lds_barrier();
    };

    load_slice(0, IC<0>{});
    store_slice(0, IC<0>{});
    if (1 < nslices) load_slice(1, IC<0>{});
    if (PF == 2 && 2 < nslices) load_slice(2, IC<PF - 1>{});
    lds_barrier();

    for (int it = 0; it < nslices; it += PF) {
        slice_step(it, IC<0>{});
        if (PF == 2 && it + 1 < nslices) slice_step(it + 1, IC<PF - 1>{});
    }

    store_tile<TM, TN, SPLIT>(a, acc, m0 + wm * WM, n0 + wn * WN, n0);
}

template <int BM, int BN, int WGM, int WGN, int BK, int PF, bool CF, int FR, int FS, bool TAB1, bool SPLIT>
__global__ __launch_bounds__(NT) void conv_f32_kernel(const KArgs a)
{
    __shared__ __attribute__((aligned(16))) float As[2][BM * (BK + 4)];
    __shared__ __attribute__((aligned(16))) float Bs[2][BN * (BK + 4)];
    // (the one-word table is an instantiation of its own: the longer table costs the other paths a workgroup per compute unit, which
    // AlexNet's first two convolutions at batch 128 show as 1465 us against 1518, and its code the element-by-element path 4 to 15 %)
    __shared__ __attribute__((aligned(16))) int ktab[CF ? 4 : TAB1 ? KTAB1 : 2 * KTAB];   // CF = false: {byte offset, r | s << 8} per k
    conv_f32_tile<BM, BN, WGM, WGN, BK, PF, CF, FR, FS, TAB1, SPLIT>(a, (int)blockIdx.x, As, Bs, ktab);
}

// 3x3 filters in KCRS order on a multiple of 16 channels: filters that change from call to call, as while a layer is being fitted, and are not worth
// packing.  In the order of the general path every activation costs a table entry, a shift, a mask and an add, 24 vector instructions a slice, which fp32
// matrix instructions do not overlap with.  Here the nine taps of 8 channels, 72 consecutive floats of a filter row, come to LDS as they are with 16-byte
// loads, and a slice is one filter row of those 8 channels: 24 k, of which lane half h takes channels 4 h .. 4 h + 3.  An activation's
// place is one of nine per-lane offsets (the padding is in them) and a channel, which is the load's scalar offset: no vector arithmetic in the loop.
// Filter rows lie 74 floats apart: two lanes to a bank both where a row is written, by 8 bytes, and where it is read (73, one lane to a bank in the reads
// and eight in the writes, 66 us instead of 63); an activation row is 24 floats, its 16-byte pieces in an order that bit 2 of the pixel turns
// round: 31 KB, five workgroups per compute unit (four: the same time).
// 3x3 64 -> 192 at stride 2 on 56 x 56 x 32, 1176 tiles in one round, 71 -> 60 us (92 TFLOP/s); on one image, with the parameter gradient and all that a
// step of the fitting takes, 44.7 -> 37.9.  What is left: the matrix cores are busy three quarters of the time, least when one or two workgroups
// remain on a compute unit.
template <int BM, int BN>
__global__ __launch_bounds__(NT, BM == 64 ? 5 : 4) void conv_f32_kcrs33_kernel(const KArgs a)
{
    constexpr int CB = KCRS33_CB, ROW = KCRS33_ROW, LDA = ROW + 2, WGN = BN / 32, OOB = (int)0x80000000;
    constexpr int A_F4 = BM * ROW / 4, A_PER = (A_F4 + NT - 1) / NT, CPT = CB * BN / NT;       // 16-byte loads of a block; channels of an activation a thread fetches
    static_assert(BM / 32 * WGN == 4 && (CPT == 2 || CPT == 4), "four waves");
    __shared__ __attribute__((aligned(16))) float As[BM * LDA];
    __shared__ __attribute__((aligned(16))) float Bs[2][BN * 24];
    const ConvGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const int wm = wave / WGN, wn = wave % WGN;
    int bid = (int)blockIdx.x;
    const int nblk = a.grid_m * a.grid_n;
    if (nblk % 8 == 0) bid = (bid & 7) * (nblk >> 3) + (bid >> 3);      // (a range of tiles per die, as above)
    const int m0 = (bid % a.grid_m) * BM, n0 = (bid / a.grid_m) * BN, HW = g.H * g.W, PQ = g.P * g.Q, blocks = g.C / CB;

    int va[A_PER], vb[3][3];
#pragma unroll
    for (int i = 0; i < A_PER; ++i) {
        const int f = tid + i * NT, row = f / (ROW / 4);
        va[i] = f < A_F4 && m0 + row < g.K ? ((m0 + row) * g.Kg + (f - row * (ROW / 4)) * 4) * 4 : OOB;
    }
    const int px = tid % BN, grp = tid / BN, n = n0 + px;
    {
        const int nn = n < g.Ng ? n : 0, img = nn / PQ, pix = nn - img * PQ, p = pix / g.Q, q = pix - p * g.Q, ih0 = p * g.sh - g.ph, iw0 = q * g.sw - g.pw;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const bool in = (n < g.Ng) & ((unsigned)(ih0 + r) < (unsigned)g.H) & ((unsigned)(iw0 + t) < (unsigned)g.W);
                vb[r][t] = in ? ((img * g.C + grp * CPT) * HW + (ih0 + r) * g.W + iw0 + t) * 4 : OOB;
            }
    }
    f32x4 ra[A_PER];
    float rb[3][CPT];
    auto load_a = [&](int blk) __attribute__((always_inline)) {
        const LoadRange l = kcrs33_filters(blk, blocks, a.w_bytes);
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, l.bytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < A_PER; ++i) ra[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, va[i], l.scalar, 0));
    };
    auto load_b = [&](int blk, auto r_c) __attribute__((always_inline)) {
        constexpr int R = decltype(r_c)::value;
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, kcrs33_plane(blk, blocks, 0, HW, a.x_bytes).bytes, 0x00020000);
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int j = 0; j < CPT; ++j) rb[t][j] = buf_load(rx, vb[R][t], kcrs33_plane(blk, blocks, j, HW, a.x_bytes).scalar);
    };
    auto put_a = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int f = tid + i * NT, row = f / (ROW / 4);
            if (A_F4 % NT == 0 || f < A_F4) {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                float* const d = As + f * 4 + 2 * row;
                *reinterpret_cast<f32x2*>(d) = f32x2{ra[i][0], ra[i][1]};
                *reinterpret_cast<f32x2*>(d + 2) = f32x2{ra[i][2], ra[i][3]};
            }
        }
    };
    auto put_b = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int h = CPT == 4 ? grp : grp >> 1;
            float* const d = &Bs[buf][px * 24 + (2 * t + (h ^ (px >> 2 & 1))) * 4 + (CPT == 4 ? 0 : (grp & 1) * 2)];
            if constexpr (CPT == 4) {
                *reinterpret_cast<f32x4*>(d) = f32x4{rb[t][0], rb[t][1], rb[t][2], rb[t][3]};
            } else {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                *reinterpret_cast<f32x2*>(d) = f32x2{rb[t][0], rb[t][1]};
            }
        }
    };
    f32x16 acc[1][1];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][0][v] = 0.f;
    const float* const a_rd = As + (wm * 32 + l32) * LDA + half * 36;
    const int b_px = wn * 32 + l32, b_rd = b_px * 24 + (half ^ (b_px >> 2 & 1)) * 4;
    auto multiply = [&](int buf, auto r_c, auto between) __attribute__((always_inline)) {
        constexpr int R = decltype(r_c)::value;
        float fa[3][4];
        f32x4 fb[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            fb[t] = *reinterpret_cast<const f32x4*>(&Bs[buf][b_rd + t * 8]);
#pragma unroll
            for (int j = 0; j < 4; ++j) fa[t][j] = a_rd[j * 9 + R * 3 + t];
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) {
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[t][j], fb[t][j], acc[0][0], 0, 0, 0);
            if (t == 1) {
                __builtin_amdgcn_sched_barrier(0);
                between();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // a block of 8 channels whose first slice is in buffer B0, its filters in LDS, its second slice and the next block's filters under way
    auto block = [&](int blk, auto b_c) __attribute__((always_inline)) {
        constexpr int B0 = decltype(b_c)::value;
        multiply(B0, IC<0>{}, [&]() __attribute__((always_inline)) { put_b(B0 ^ 1); load_b(blk, IC<2>{}); });
        lds_barrier();
        multiply(B0 ^ 1, IC<1>{}, [&]() __attribute__((always_inline)) { put_b(B0); load_b(blk + 1, IC<0>{}); });
        lds_barrier();
        multiply(B0, IC<2>{}, [&]() __attribute__((always_inline)) { put_b(B0 ^ 1); load_b(blk + 1, IC<1>{}); });
        lds_barrier();                                // every wave has read the filters
        put_a();
        load_a(blk + 2);
        lds_barrier();
    };
    load_a(0);
    load_b(0, IC<0>{});
    put_a();
    put_b(0);
    load_a(1);
    load_b(0, IC<1>{});
    lds_barrier();
    for (int blk = 0; blk < blocks; blk += 2) {
        block(blk, IC<0>{});
        block(blk + 1, IC<1>{});
    }
    store_tile<1, 1, false>(a, acc, m0 + wm * 32, n0 + wn * 32, n0);
}

// Several layers in one launch (KRSC filters or 1x1; each with the tile it would have by itself): the layers' tiles fill the device
// together, where each by itself ends in a round that leaves most compute units idle.
struct GroupArgs {
    int n;
    int first[SMALL_GROUP_MAX];                   // first workgroup of each layer
    int rows32[SMALL_GROUP_MAX];                  // 32 x 128 tiles instead of 64 x 64
    KArgs job[SMALL_GROUP_MAX];
};
__global__ __launch_bounds__(NT) void conv_f32_group_kernel(const GroupArgs args)
{
    __shared__ __attribute__((aligned(16))) float As[2 * 64 * 20];
    __shared__ __attribute__((aligned(16))) float Bs[2 * 128 * 20];
    int ji = 0;
    while (ji + 1 < args.n && (int)blockIdx.x >= args.first[ji + 1]) ++ji;
    const KArgs a = args.job[ji];
    const int block = (int)blockIdx.x - args.first[ji];
    if (args.rows32[ji]) conv_f32_tile<32, 128, 1, 4, 16, 2, true, 0, 0, false, false>(a, block, (float (*)[32 * 20])As, (float (*)[128 * 20])Bs, nullptr);
    else conv_f32_tile<64, 64, 2, 2, 16, 2, true, 0, 0, false, false>(a, block, (float (*)[64 * 20])As, (float (*)[64 * 20])Bs, nullptr);
}

// y = bias + residual + sum over the ranges of a split contraction, ReLU: one thread per output element,
// consecutive threads along n (these layers are small: what counts is the number of loads in flight).
__global__ __launch_bounds__(256) void conv_f32_reduce_kernel(const float* __restrict__ part, int splits, ConvGeom g,
                                                              const float* __restrict__ bias, const float* __restrict__ res,
                                                              float* __restrict__ y)
{
    const size_t total = (size_t)g.K * g.Ng;
    const int PQ = g.P * g.Q;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
        const int m = (int)(i / g.Ng), n = (int)(i - (size_t)m * g.Ng);
        float sum = 0.f;
#pragma unroll 4
        for (int s = 0; s < splits; ++s) sum += part[s * total + i];   // unrolled: four loads in flight, the order of the sum unchanged
        const int img = n / PQ, pix = n - img * PQ;
        float o = sum + (bias ? bias[m] : 0.f);
        if (res) o += res[((size_t)img * g.res_ctot + m) * PQ + pix];
        if (g.relu) o = fmaxf(o, 0.f);
        y[((size_t)img * g.y_ctot + g.y_coff + m) * PQ + pix] = o;
    }
}

// How a layer's contraction is cut when scratch memory is there: enough ranges to give the device about two
// workgroups per compute unit, each at least two slices long; 1 = not cut (the layer's tiles reach half
// of the compute units, or it is too shallow).
inline int split_plan(int tiles, int nslices, int* slices_per_split)
{
    const int cus = device_cus();
    *slices_per_split = nslices;
    if (2 * tiles > cus || nslices < 4) return 1;   // measured: no gain once half the compute units have a tile
    const int want = (2 * cus + tiles - 1) / tiles;
    int per = (nslices + want - 1) / want;
    if (per < 2) per = 2;
    *slices_per_split = per;
    return (nslices + per - 1) / per;
}

// Slices of the contraction, and whether a KCRS layer takes the groups-of-4-taps order (no padding, a filter width
// that rounding up to a multiple of 4 lengthens by at most a quarter, a table that fits LDS).
template <int BK>
int contraction_slices(const ConvGeom& g, int* row_groups)
{
    *row_groups = 0;
    if (g.C % BK == 0 && (g.w_krsc || g.R * g.S == 1)) return g.R * g.S * (g.C / BK);
    const int S4 = (g.S + 3) & ~3;
    const long kg4 = (long)g.C * g.R * S4;
    if (g.ph == 0 && g.pw == 0 && S4 * 4 <= g.S * 5 && (kg4 + BK - 1) / BK * BK <= 4 * KTAB) {
        *row_groups = 1;
        return (int)((kg4 + BK - 1) / BK);
    }
    return (g.Kg + BK - 1) / BK;
}

template <int BM, int BN, int BK>
size_t split_bytes(const ConvGeom& g)
{
    int rgm;
    const int nslices = contraction_slices<BK>(g, &rgm);
    int per;
    const int splits = split_plan(((g.K + BM - 1) / BM) * ((g.Ng + BN - 1) / BN), nslices, &per);
    return splits > 1 ? (size_t)splits * g.K * g.Ng * sizeof(float) : 0;
}

template <int BM, int BN, int WGM, int WGN, int BK, int PF>
int launch_tile(const KArgs& base, void* ws, size_t ws_bytes, hipStream_t st)
{
    KArgs a = base;
    a.grid_m = (a.g.K + BM - 1) / BM;
    a.grid_n = (a.g.Ng + BN - 1) / BN;
    a.part = nullptr;
    a.splits = 1;
    const int nslices = contraction_slices<BK>(a.g, &a.row_groups);
    a.slices_per_split = nslices;
    if (ws && a.nsplit <= 1) {
        int per;
        const int splits = split_plan(a.grid_m * a.grid_n, nslices, &per);
        if (splits > 1 && (size_t)splits * a.g.K * a.g.Ng * sizeof(float) <= ws_bytes && ((uintptr_t)ws & 15) == 0) {
            a.part = (float*)ws;
            a.splits = splits;
            a.slices_per_split = per;
        }
    }
    const dim3 grid((unsigned)(a.grid_m * a.grid_n), (unsigned)a.splits), block(NT);
    const int R = a.g.R, S = a.g.S;
#define DR_LAUNCH(CF, FR, FS, TAB1)                                                                                              \
    do {                                                                                                                   \
        if (a.part) hipLaunchKernelGGL((conv_f32_kernel<BM, BN, WGM, WGN, BK, PF, CF, FR, FS, TAB1, true>), grid, block, 0, st, a);   \
        else hipLaunchKernelGGL((conv_f32_kernel<BM, BN, WGM, WGN, BK, PF, CF, FR, FS, TAB1, false>), grid, block, 0, st, a);         \
    } while (0)
    if constexpr (BK == 32) {
        DR_LAUNCH(true, 0, 0, false);                // (see slices_of_32)
    } else {
        const bool tab1 = !a.row_groups && a.g.Kg <= KTAB1 && tab1_fits(a.g.C, a.g.H, a.g.W, R, S);
        if (a.g.C % BK == 0 && (a.w_krsc || R * S == 1)) DR_LAUNCH(true, 0, 0, false);      // (a 1x1 filter bank is the same array in both orders)
        else if (tab1 && R == 1 && S == 1) DR_LAUNCH(false, 1, 1, true);
        else if (tab1 && R == 3 && S == 3) DR_LAUNCH(false, 3, 3, true);
        else if (tab1 && R == 5 && S == 5) DR_LAUNCH(false, 5, 5, true);
        else if (tab1) DR_LAUNCH(false, 0, 0, true);
        else if (R == 1 && S == 1) DR_LAUNCH(false, 1, 1, false);
        else if (R == 3 && S == 3) DR_LAUNCH(false, 3, 3, false);
        else if (R == 5 && S == 5) DR_LAUNCH(false, 5, 5, false);
        else if (R == 7 && S == 7) DR_LAUNCH(false, 7, 7, false);
        else if (R == 11 && S == 11) DR_LAUNCH(false, 11, 11, false);
        else DR_LAUNCH(false, 0, 0, false);
    }
#undef DR_LAUNCH
    const int rc = check_launch("conv_f32");
    if (rc != DR_OK) return rc;
    if (a.part) {
        const ConvGeom& g = a.g;
        const size_t threads = (size_t)g.K * g.Ng;
        const unsigned blocks = (unsigned)std::min<size_t>((threads + 255) / 256, (size_t)device_cus() * 8);
        hipLaunchKernelGGL(conv_f32_reduce_kernel, dim3(blocks), dim3(256), 0, st, a.part, a.splits, g, a.bias, a.res, a.y);
        return check_launch("conv_f32 (sum of the split contraction)");
    }
    return DR_OK;
}

}  // namespace

// 32-row tiles when they pad the filter count less than 64-row tiles (16, 32, 96 filters ...), else 64 x 64 tiles
static bool rows_of_32(const ConvGeom& g) { return (g.K + 31) / 32 * 32 < (g.K + 63) / 64 * 64; }

// Depth of a slice: 32 channels where the count allows, which halves the barriers, and 16 for layers of more 64 x 64 tiles than the
// device holds at 32 (four workgroups per compute unit, seven at 16: 3x3 64 -> 192 on 28 x 28 x 32, 1176 tiles, 65 -> 56 us) unless
// they are few more than it holds at 16 (3x3 64 -> 320 on 14 x 14 x 128, 1960 tiles, 32 deep 89, 16 deep 97; 5x5 96 -> 256 on
// 27 x 27 x 48, 2188 tiles, 353 and 374; 3x3 64 -> 384 on 14 x 14 x 128, 2352 tiles, 109 and 103).  1x1 filters go by the same lines
// (512 -> 256 on 14 x 14 x 37, 456 tiles, 25.0 and 26.0; 512 -> 192 on 28 x 28 x 32, 1176, 58 and 49; 512 -> 2048 on 7 x 7 x 83, 2048,
// 82 and 91), with tiles of 32 x 128 by one per compute unit (64 -> 16 on 28 x 28 x 16, 98 tiles, 5.6 and 7.4; 192 -> 32 on 28 x 28 x 32,
// 196, 10.7 and 11.5; 512 -> 96 there, 588, 40 and 37).  The sums are in the same order either way.
static bool slices_of_32(const ConvGeom& g)
{
    const long cus = device_cus(), tiles = ((long)g.K + 63) / 64 * (((long)g.Ng + 63) / 64);
    if (!g.w_krsc || g.C % 32 != 0) return false;
    if (rows_of_32(g)) return g.R * g.S > 1 || ((long)g.K + 31) / 32 * (((long)g.Ng + 127) / 128) <= cus;
    return tiles <= 4 * cus || (g.C > 32 && tiles > 7 * cus && tiles <= 9 * cus);
}

// A layer for the kernel of conv_f32_taps.hip whose contraction scratch memory lets be cut over workgroups (see launch_tile): whether that is
// faster.  There a workgroup walks all pairs of filter rows, 0.34 us each; the cut takes a second launch, the partial sums' way through memory
// and the slices of a range.  Fitted to 200 layers of few pixels (5 and 7 % off), and within 9 % of the better one on each of them: 11x11 on 5 channels, two
// outputs, 6.8 us cut and 11.9 there, 12x12 on 5 channels 27 filters on 272 outputs 9.0 and 13.6; 11x11 on 3 channels 6 filters on 1575 outputs 7.5 and
// 8.7; 8x8 on 5 channels 13 filters on 12054 outputs 11.5 and 10.2, 10x10 on 3 channels 240 filters on 1740 outputs 17.3 and 8.1.
static bool cut_beats_taps(const ConvGeom& g, const void* ws, size_t ws_bytes)
{
    int row_groups, per;
    const int nslices = contraction_slices<16>(g, &row_groups);
    const int tiles = rows_of_32(g) ? ((g.K + 31) / 32) * ((g.Ng + 127) / 128) : ((g.K + 63) / 64) * ((g.Ng + 63) / 64);
    const int splits = split_plan(tiles, nslices, &per);
    const size_t bytes = (size_t)splits * g.K * g.Ng * sizeof(float);
    if (!ws || splits <= 1 || bytes > ws_bytes || ((uintptr_t)ws & 15) != 0) return false;
    const float taps_us = 3.0f + 0.34f * ((g.C * g.R + 1) / 2), cut_us = 6.4f + 0.84e-6f * bytes + 1.26f * (per - 2) + 0.071f * splits;
    return cut_us < 0.95f * taps_us;
}

// 3x3 filters in KCRS order that the general path does not cut over workgroups; they are read 16 bytes at a time.  No line on sizes: 88 layers drawn from 16 to
// 512 channels, 1 to 512 filters, maps of 3 to 112 and 1 to 64 images, strides 1 and 2, take 0.41 to 0.87 of the general path's time, 0.67 on average (the
// general order's 16-wide slices cost the same arithmetic on one tile as on a thousand: 32 -> 14 on 7 x 4, one image, 13.3 and 10.1 us; 64 -> 192 on
// 19 x 21 x 60 60.7 and 51.4; 272 -> 18 on 21 x 18 x 2 145 and 59).
static bool kcrs33_takes(const ConvGeom& g, const void* w, const void* ws, size_t ws_bytes, int nsplit)
{
    if (g.w_krsc || g.R != 3 || g.S != 3 || g.C % 16 != 0 || ((uintptr_t)w & 15) != 0) return false;
    const size_t cut = conv_f32_scratch_bytes(g);
    return !(ws && nsplit <= 1 && cut && cut <= ws_bytes && ((uintptr_t)ws & 15) == 0);
}

bool conv_f32_group_takes(const ConvGeom& g)
{
    const size_t xb = (size_t)g.N * g.C * g.H * g.W * 4, wb = (size_t)g.K * g.Kg * 4;
    return !g.nhwc && g.w_krsc && g.C % 16 == 0 && xb < (1ull << 31) && wb < (1ull << 31) && g.Ng > 0 && !conv_f32_direct_takes(g);
}

int launch_conv_f32_group(const ConvSmall* all, int n_all, hipStream_t st)
{
    ConvSmall jobs[SMALL_GROUP_MAX], pieces[SMALL_GROUP_MAX];
    int n = 0, n_pieces = 0;
    for (int i = 0; i < n_all; ++i) (conv_f32_pieces_takes(all[i].g) ? pieces[n_pieces++] : jobs[n++]) = all[i];
    if (n_pieces) {
        const int rc = launch_conv_f32_pieces(pieces, n_pieces, st);
        if (rc != DR_OK) return rc;
    }
    if (!n) return DR_OK;
    GroupArgs a{};
    a.n = n;
    int order[SMALL_GROUP_MAX], blocks = 0;
    for (int i = 0; i < n; ++i) order[i] = i;
    std::sort(order, order + n, [&](int p, int q) { return jobs[p].g.Kg > jobs[q].g.Kg; });      // the longest tiles first
    for (int i = 0; i < n; ++i) {
        const ConvSmall& c = jobs[order[i]];
        a.job[i] = conv_f32_args(c.g, (const float*)c.x, (const float*)c.w, c.bias, (const float*)c.res, (float*)c.y, c.split);
        a.rows32[i] = rows_of_32(c.g);
        a.job[i].grid_m = a.rows32[i] ? (c.g.K + 31) / 32 : (c.g.K + 63) / 64;
        a.job[i].grid_n = a.rows32[i] ? (c.g.Ng + 127) / 128 : (c.g.Ng + 63) / 64;
        a.first[i] = blocks;
        blocks += a.job[i].grid_m * a.job[i].grid_n;
    }
    hipLaunchKernelGGL(conv_f32_group_kernel, dim3((unsigned)blocks), dim3(NT), 0, st, a);
    return check_launch("conv_f32_group");
}

size_t conv_f32_scratch_bytes(const ConvGeom& g)
{
    if (conv_f32_pieces_takes(g) || conv_f32_direct_takes(g)) return 0;
    if (slices_of_32(g)) return rows_of_32(g) ? split_bytes<32, 128, 32>(g) : split_bytes<64, 64, 32>(g);
    return rows_of_32(g) ? split_bytes<32, 128, 16>(g) : split_bytes<64, 64, 16>(g);
}

int launch_conv_f32(const ConvGeom& g, const float* x, const float* w, const float* bias, const float* residual,
                    float* y, hipStream_t st, void* ws, size_t ws_bytes, const ConvSplit* split)
{
    TraceScope trace("conv_f32", &g, g.Ng, st);
    if (conv_f32_pieces_takes(g)) {
        const ConvSmall job{g, x, w, bias, residual, y, split};
        return launch_conv_f32_pieces(&job, 1, st);
    }
    if (conv_f32_direct_takes(g)) return launch_conv_f32_direct(ConvSmall{g, x, w, bias, residual, y, split}, st);
    if (conv_f32_small_takes(g, w, ws != nullptr)) {
        const ConvSmall job{g, x, w, bias, residual, y, split};
        return launch_conv_f32_small(&job, 1, st);
    }
    const size_t xb = (size_t)g.N * g.C * g.H * g.W * 4, wb = (size_t)g.K * g.Kg * 4;
    if (xb >= (1ull << 31) || wb >= (1ull << 31))
        return fail(DR_ERR_UNSUPPORTED, "conv_f32: input (%zu bytes) or filter tensor (%zu bytes) is 2 GiB or larger", xb, wb);
    // wide filters on few channels, no padding (conv_f32_taps.hip)
    if (conv_f32_taps_takes(g, residual, split) && !cut_beats_taps(g, ws, ws_bytes)) return launch_conv_f32_taps(g, x, w, bias, y, st);
    KArgs a = conv_f32_args(g, x, w, bias, residual, y, split);
    if (kcrs33_takes(g, w, ws, ws_bytes, a.nsplit)) {
        const bool rows32 = rows_of_32(g);
        a.grid_m = rows32 ? (g.K + 31) / 32 : (g.K + 63) / 64;
        a.grid_n = rows32 ? (g.Ng + 127) / 128 : (g.Ng + 63) / 64;
        const dim3 grid((unsigned)(a.grid_m * a.grid_n)), block(NT);
        if (rows32) hipLaunchKernelGGL((conv_f32_kcrs33_kernel<32, 128>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((conv_f32_kcrs33_kernel<64, 64>), grid, block, 0, st, a);
        return check_launch("conv_f32 (3x3, KCRS)");
    }
    // (32-deep slices with the groups-of-4-taps order: measured 10 % slower)
    if (slices_of_32(g))
        return rows_of_32(g) ? launch_tile<32, 128, 1, 4, 32, 2>(a, ws, ws_bytes, st) : launch_tile<64, 64, 2, 2, 32, 2>(a, ws, ws_bytes, st);
    return rows_of_32(g) ? launch_tile<32, 128, 1, 4, 16, 2>(a, ws, ws_bytes, st) : launch_tile<64, 64, 2, 2, 16, 2>(a, ws, ws_bytes, st);
}

}  // namespace dr
