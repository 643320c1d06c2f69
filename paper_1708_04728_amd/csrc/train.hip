// Layer-wise regression of a slim layer (Sec. 3.1: the optimisation goal below Eq. (4), Lemma 1): the slim
// layer f~(W, b; X) = max(conv(X; W, b), 0) is fitted to the feature map Y of the block it replaces by
// gradient descent on L(W, b) = sum || Y - f~(W, b; X) ||^2.  fp32, NCHW tensors, KCRS filters.
//
//   regression_loss_grad   dz = 2 (f - y) where f > 0 else 0,  L = sum (f - y)^2
//   conv_wgrad             dw[k][c,r,s] = sum_{n,p,q} dz[n,k,p,q] x[n,c,p*sh+r-ph,q*sw+s-pw],  db[k] = sum dz[n,k,p,q]
//                          (db: the row sums of the GEMM's first operand, kept by the first column tile's workgroups)
//   sgd_step               w -= lr * dw
//
// The weight gradient is a GEMM  D[m][n] = sum_l A[m][l] B[l][n]  with m = filter, n = (tap, channel) and the
// contraction over l = (image, p, q): A is dz (for one image and filter the (p, q) run is contiguous), B is
// gathered from x.  A workgroup owns a tile of 64, 128 or 192 x 64 of D for a range of slices of 32 l (each inside one image), stages
// a slice at a time in LDS (l contiguous per row, rows padded by 4 floats) and multiplies,
// each lane half taking 16 consecutive l of the slice so that an operand is four 128-bit LDS reads.  The ranges
// give enough workgroups to fill the device; their partial sums go to workspace and are added in a fixed
// order by a second kernel, so the result does not depend on scheduling.
#include <algorithm>
#include <type_traits>

#include "dr_internal.h"
#include "f32_pieces.h"

namespace dr {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr unsigned OOB = 0x80000000u;       // an offset beyond every buffer; offsets are unsigned, so that two of these may be added

// grid of a grid-stride kernel: at most 4096 workgroups (the loss kernel leaves one partial sum per workgroup)
inline unsigned blocks_for_train(size_t count)
{
    const size_t b = (count + 255) / 256;
    return (unsigned)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

// sum over the 256 threads of a workgroup, in a fixed order (wave shuffles, then the 4 wave sums through LDS)
__device__ __forceinline__ float block_sum(float v, float* red)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_down(v, d, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    const float s = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(256) void regression_loss_grad_kernel(const float* __restrict__ f, const float* __restrict__ y,
                                                                   float* __restrict__ dz, size_t nvec, size_t count, float* __restrict__ partial)
{
    __shared__ float red[4];
    float acc = 0.f;
    // 16-byte vectors where the three pointers allow it (nvec = 0 otherwise), then the scalar tail
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nvec; i += (size_t)gridDim.x * 256) {
        const f32x4 fv = reinterpret_cast<const f32x4*>(f)[i], yv = reinterpret_cast<const f32x4*>(y)[i];
        f32x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float d = fv[j] - yv[j];
            acc += d * d;
            o[j] = fv[j] > 0.f ? 2.f * d : 0.f;
        }
        reinterpret_cast<f32x4*>(dz)[i] = o;
    }
    for (size_t i = nvec * 4 + (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) {
        const float fi = f[i], d = fi - y[i];
        acc += d * d;
        dz[i] = fi > 0.f ? 2.f * d : 0.f;
    }
    const float s = block_sum(acc, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// out[0] = sum of partial[0..n): thread t adds the entries t, t + 256, ... in double, the 256 sums are then added
// in a fixed tree, so the value does not depend on scheduling
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ partial, int n, float* __restrict__ out)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += (double)partial[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int d = 128; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = (float)red[0];
}

struct WArgs {
    const float* x;
    const float* dz;
    float* out;            // the partial sums [splits][K][cols], then those of the bias gradient [splits][K] (splits > 1)
    float* dw;             // splits == 1: the results themselves
    float* db;             // (may be NULL)
    int N, C, H, W, K, R, S, sh, sw, ph, pw, P, Q;
    int CRS, grid_m, grid_n, splits, slices_per_img, slices;
    int cb_log2, cblocks, cols;                         // channels per column tile; channel blocks; columns of the partial sums (grid_n BN)
    int x_bytes, dz_bytes;
};

constexpr int BN = 64, BL = 32, LDT = BL + 4;

// dw[m][c R S + rs] of column `col`: tile col / BN holds 64 >> cb_log2 taps x (1 << cb_log2) channels; -1 for padding
__device__ __forceinline__ int wgrad_column(int col, int C, int RS, int cb_log2, int cblocks)
{
    const int nt = col / BN, l = col % BN, tg = nt / cblocks, cblk = nt - tg * cblocks;
    const int rs = tg * (BN >> cb_log2) + (l >> cb_log2), c = (cblk << cb_log2) + (l & ((1 << cb_log2) - 1));
    return rs < RS && c < C ? c * RS + rs : -1;
}

// Barrier that orders LDS traffic only (the global loads of the next slices stay in flight across it).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// TPT: taps per column tile (64 channels of one tap, 32 of two, 16 of four; 8 of eight or 4 of sixteen where a layer on the
// image would leave most of 16 channels empty: 11x11 3 -> 96 at stride 4 on 227 x 227 x 32 images 531 us with 16, 173 with 4; 7x7 3 -> 64 at
// stride 2 453 and 184; 5x5 8 -> 64 on 56 x 56 x 32 75 and 59).  A thread's eight columns
// belong to TPT taps, so the padding test is made TPT times per slice (with columns in (c, r, s) order it was made for every
// element and that arithmetic took longer than the multiplications), the rest of an address is a per-thread constant, and
// (p, q) advances by addition.  Two LDS buffers, one barrier per slice, loads one slice ahead; the next slice goes to LDS in the middle of the products.
// EIGHTS: channels come in eights, so that a column exists for all threads of its group of eight or for none: its offset is then the
// load's scalar offset, and a slice takes one address per tap instead of one per element.
//
// The products: operands cut into three bf16 pieces by the waves that read them, six products of 32 cycles for 16 k in the place of eight of 64, the five small
// ones in a sum of their own (as in conv_f32_pieces.hip).  Operands are scaled where they are written to LDS, once, so that no value is too small for its pieces
// (f32_pieces.h; with a look for small operands at every cut instead 57.9 us in the place of 55.7 for 64 -> 192 below, 44.1 and 42.4 for 64 -> 128).  Pieces alone gained nothing: fp32 matrix instructions
// hid the gathered loads, 16 of 4 bytes per thread and slice.  So dz comes 16 bytes at a time, and TM blocks of 64 filters share the columns: 24 + 8 loads' worth
// in 14 for three.  3x3 64 -> 192 at stride 2 on 56 x 56 x 32, the call with the sum of its ranges (5.7 us): 74.2 us with one block and fp32
// products, 75.6 with pieces, 72.8 with two blocks, 61.5 with three; 64 -> 128 54.6 and 48.6.  Vector instructions, most of them the cutting, now issue in half of the cycles, matrix instructions in
// a quarter; two waves per SIMD wait for LDS in the rest.  (Loads two slices ahead: three blocks spill, 84.1.)
// Ranges of fewer than ten slices (four with taller tiles) take fp32 products: they are start and end (32 -> 192 on 22 x 32, one image, 10.8 us before, 11.0 with
// pieces, 9.7 without; 64 -> 96 on 18 x 64 x 57, two blocks and nine slices, 35.1 and 38.2).  210 drawn layers 0.98 to 1.21, 1.076 on average.
template <int TPT, bool EIGHTS, int TM>
__global__ __launch_bounds__(256, TM == 1 ? 3 : 2) void conv_wgrad_f32_kernel(const WArgs a)
{
    constexpr int BM = TM * 64, AU = TM * 2;               // rows of a tile; of each thread
    __shared__ __attribute__((aligned(16))) float As[2][BM * LDT];
    __shared__ __attribute__((aligned(16))) float Bs[2][BN * LDT];
    __shared__ int redo;
    constexpr int CB = BN / TPT, NT = TPT < 8 ? TPT : 8, IPT = 8 / NT;     // channels per tile; taps of a thread's columns; columns per tap
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, half = lane >> 5, l32 = lane & 31;
    // workgroup b runs on die b & 7: a die takes a contiguous range of (split, column tile, row tile), so that the tiles of one
    // range of slices read x and dz through one L2
    const int die = blockIdx.x & 7, share = (int)gridDim.x >> 3, odd = gridDim.x & 7;
    int bid = die * share + min(die, odd) + (int)(blockIdx.x >> 3);
    const int mt = bid % a.grid_m; bid /= a.grid_m;
    const int nt = bid % a.grid_n, sp = bid / a.grid_n;
    const int m0 = mt * BM;
    const int lo = (int)((long)a.slices * sp / a.splits), total = (int)((long)a.slices * (sp + 1) / a.splits) - lo;
    const int PQ = a.P * a.Q, HW = a.H * a.W, RS = a.R * a.S;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc((void*)a.dz, 0, a.dz_bytes, 0x00020000);

    // loader: this thread fetches four elements of the slice, 4 (tid % 8) on, for rows tid / 8 + 32 i of dz, and element l = tid % 32 for
    // columns tid / 32 + 8 i.  A row or column that does not exist has the offset OOB; whatever is then read belongs to an output that is not stored.
    const int ll = tid & 31, row0 = tid >> 5;
    const int tg = nt / a.cblocks, c0 = (nt - tg * a.cblocks) * CB;
    // column row0 + 8 i: tap i / IPT and channel row0 + 8 (i % IPT) of the tile; with tiles of 4 channels tap 2 i + row0 / 4, channel row0 % 4
    auto tap_of = [&](int t) __attribute__((always_inline)) { return tg * TPT + (TPT > 8 ? 2 * t + (row0 >> 2) : t); };
    static_assert(!EIGHTS || TPT < 16, "a column tile of four channels");
    unsigned a_row[AU], b_row[EIGHTS ? 1 : 8];           // EIGHTS: of column row0; the others' distance from it is wave-uniform
    int b_off[8];                                        // (0: of an eight that does not exist, whose outputs are not stored)
    const int l4 = (tid & 7) * 4, row4 = tid >> 3;
#pragma unroll
    for (int i = 0; i < AU; ++i) a_row[i] = m0 + row4 + 32 * i < a.K ? (unsigned)((m0 + row4 + 32 * i) * PQ * 4) : OOB;
    int tap_r[NT], tap_s[NT];
    if constexpr (EIGHTS) {
        b_row[0] = (unsigned)((c0 + row0) * HW * 4);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            b_off[i] = c0 + 8 * (i % IPT) < a.C ? 8 * (i % IPT) * HW * 4 : 0;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = c0 + (TPT > 8 ? row0 & 3 : row0 + 8 * (i % IPT));
            b_row[i] = c < a.C && tap_of(i / IPT) < RS ? (unsigned)(c * HW * 4) : OOB;
            b_off[i] = 0;
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int rs = tap_of(t), r = rs / a.S;
        tap_r[t] = r - a.ph; tap_s[t] = rs - r * a.S - a.pw;
    }
    // the slice being fetched: image, first (p, q) run element and this thread's own
    int img, left, pq, p, q;                               // left: slices left in the image
    const int p_ll = ll / a.Q, q_ll = ll - p_ll * a.Q, step_p = BL / a.Q, step_q = BL - step_p * a.Q;
    auto start = [&]() __attribute__((always_inline)) {
        img = lo / a.slices_per_img;
        left = a.slices_per_img - (lo - img * a.slices_per_img);
        pq = (a.slices_per_img - left) * BL + ll;
        p = pq / a.Q;
        q = pq - p * a.Q;
    };
    f32x4 ra[AU];
    float rb[8];
    int rest;                                              // elements that are left of the image from this thread's four on
    auto fetch = [&]() __attribute__((always_inline)) {
        const bool on = pq < PQ;
        const int pq4 = pq - ll + l4;
        rest = PQ - pq4;
        const unsigned za = pq4 < PQ ? (unsigned)(pq4 * 4) : OOB;
        const int soff_a = img * a.K * PQ * 4, soff_b = img * a.C * HW * 4;
        const int ih0 = p * a.sh, iw0 = q * a.sw;
#pragma unroll
        for (int i = 0; i < AU; ++i) ra[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rz, a_row[i] + za, soff_a, 0));
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int ih = ih0 + tap_r[t], iw = iw0 + tap_s[t];
            const bool in = on & ((unsigned)ih < (unsigned)a.H) & ((unsigned)iw < (unsigned)a.W) & (!EIGHTS || tap_of(t) < RS);
            const unsigned xo = in ? (unsigned)((ih * a.W + iw) * 4) : OOB;
#pragma unroll
            for (int i = t * IPT; i < (t + 1) * IPT; ++i) rb[i] = buf_load(rx, b_row[EIGHTS ? 0 : i] + xo, soff_b + b_off[i]);
        }
        if (--left == 0) {
            ++img; left = a.slices_per_img;
            pq = ll; p = p_ll; q = q_ll;
        } else {
            pq += BL; p += step_p; q += step_q;
            if (q >= a.Q) { q -= a.Q; ++p; }
        }
    };
    float dbs[AU];                                         // this thread's share of the bias gradient (first column tile)
    auto put = [&](int buf, auto exact_c) __attribute__((always_inline)) {
        constexpr float scale = decltype(exact_c)::value ? 1.f : PIECES_SCALE;      // (here: a value is cut by up to 2 TM of the waves)
        if (PQ & 3) {                                      // (behind the image is the next filter's)
#pragma unroll
            for (int e = 1; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < AU; ++i) ra[i][e] = e < rest ? ra[i][e] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < AU; ++i) *reinterpret_cast<f32x4*>(&As[buf][(row4 + 32 * i) * LDT + l4]) = ra[i] * scale;
#pragma unroll
        for (int i = 0; i < 8; ++i) Bs[buf][(row0 + 8 * i) * LDT + ll] = rb[i] * scale;
        if (nt == 0) {
#pragma unroll
            for (int i = 0; i < AU; ++i) dbs[i] += (ra[i][0] + ra[i][1]) + (ra[i][2] + ra[i][3]);
        }
    };
    f32x16 acc[TM], small[TM];
    auto step = [&](int sl, auto exact_c) __attribute__((always_inline)) {
        constexpr bool EXACT = decltype(exact_c)::value;
        const int buf = sl & 1;
        const float* ap = As[buf] + (wm * TM * 32 + l32) * LDT + half * 16;
        const float* bp = Bs[buf] + (wn * 32 + l32) * LDT + half * 16;
        auto multiply = [&](int h) __attribute__((always_inline)) {      // eight of this lane's sixteen
            float fb[8];
            auto read = [&](const float* at, float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const f32x4 t = *reinterpret_cast<const f32x4*>(at + 8 * h + 4 * j);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[4 * j + e] = t[e];
                }
            };
            read(bp, fb);
            u32x4 pb[3];
            if constexpr (!EXACT) split8(fb, pb[0], pb[1], pb[2]);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                float fa[8];
                read(ap + i * 32 * LDT, fa);
                if constexpr (EXACT) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], acc[i], 0, 0, 0);
                } else {
                    u32x4 pa[3];
                    split8(fa, pa[0], pa[1], pa[2]);
                    acc[i] = mfma(pa[0], pb[0], acc[i]);
                    small[i] = mfma(pa[0], pb[1], small[i]);
                    small[i] = mfma(pa[1], pb[0], small[i]);
                    small[i] = mfma(pa[1], pb[1], small[i]);
                    small[i] = mfma(pa[0], pb[2], small[i]);
                    small[i] = mfma(pa[2], pb[0], small[i]);
                }
            }
        };
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);
        if (sl + 1 < total) {
            put(buf ^ 1, exact_c);
            if (sl + 2 < total) fetch();
        }
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        lds_barrier();
    };
    auto walk = [&](auto exact_c) __attribute__((always_inline)) {
        start();
#pragma unroll
        for (int i = 0; i < AU; ++i) dbs[i] = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = small[i][v] = 0.f;
        if (total > 0) {
            fetch();
            put(0, exact_c);
            if (1 < total) fetch();
        }
        lds_barrier();
        for (int sl = 0; sl < total; ++sl) step(sl, exact_c);
    };
    bool exact = a.slices < (TM == 1 ? 10 : 4) * a.splits;      // (uniform)
    if (!exact) {
        if (tid == 0) redo = 0;
        walk(std::false_type{});
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][v] += small[i][v];
                z = __builtin_fmaf(acc[i][v], 0.f, z);
                acc[i][v] *= PIECES_UNSCALE;
            }
        if (__any(z != 0.f)) redo = 1;                           // operands that pieces do not hold: the range again
        __syncthreads();
        exact = __builtin_amdgcn_readfirstlane(*(volatile int*)&redo) != 0;
    }
    if (exact) walk(std::true_type{});
    // register v holds row 8 (v / 4) + 4 half + v % 4 of column lane % 32
    const int col = nt * BN + wn * 32 + l32, n = wgrad_column(col, a.C, RS, __builtin_ctz(CB), a.cblocks);
#pragma unroll
    for (int v = 0; v < 16 * TM; ++v) {
        const int m = m0 + (wm * TM + v / 16) * 32 + 8 * (v % 16 >> 2) + 4 * half + (v & 3);
        if (m >= a.K) continue;
        if (a.splits > 1) a.out[((size_t)sp * a.K + m) * a.cols + col] = acc[v / 16][v % 16];
        else if (n >= 0) a.dw[(size_t)m * a.CRS + n] = acc[v / 16][v % 16];
    }
    if (nt == 0) {
        float* const db = a.splits > 1 ? a.out + (size_t)a.splits * a.K * a.cols + (size_t)sp * a.K : a.db;
#pragma unroll
        for (int i = 0; i < AU; ++i) {
            float t = dbs[i];
#pragma unroll
            for (int d = 4; d >= 1; d >>= 1) t += __shfl_down(t, d, 8);
            const int m = m0 + row4 + 32 * i;
            if ((tid & 7) == 0 && m < a.K && db) db[m] = t;
        }
    }
}

// The sum of the partial results over the splits, in split order: column by column of the [K][cols] sums, then the bias gradient.
// (Eight loads in flight per thread: a chain of single loads took 10 us for 14 MB.)  In double: up to 56 ranges one after the other in float were most of the error.  On a
// fitting step's own operands, relative to 64 bits, 64 -> 192 on 56 x 56 x 32: weights 1.08e-7 in float with 37 ranges of fp32 products, 1.12e-7 with 56 ranges of pieces, 0.28e-7 now; bias 0.92e-7, 1.08e-7
// and 0.29e-7.  Nine such layers 0.24 to 0.56 and 0.23 to 0.42 of the first; in the same time (memory's).
__global__ __launch_bounds__(256) void sum_splits_kernel(const float* __restrict__ part, int splits, int K, int C, int RS, int cb_log2, int cblocks, int cols,
                                                         float* __restrict__ dw, float* __restrict__ db)
{
    const size_t count = (size_t)K * cols, all = count + (size_t)K;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < all; i += (size_t)gridDim.x * 256) {
        const bool bias = i >= count;
        const size_t m = bias ? i - count : i / cols;
        const int n = bias ? 0 : wgrad_column((int)(i - m * cols), C, RS, cb_log2, cblocks);
        if (n < 0 || (bias && !db)) continue;
        const float* src = bias ? part + (size_t)splits * count + m : part + i;
        const size_t stride = bias ? (size_t)K : count;
        double s = 0.0;
#pragma unroll 8
        for (int sp = 0; sp < splits; ++sp) s += (double)src[(size_t)sp * stride];
        if (bias) db[m] = (float)s;
        else dw[m * ((size_t)C * RS) + n] = (float)s;
    }
}

__global__ __launch_bounds__(256) void sgd_step_kernel(float* __restrict__ w, const float* __restrict__ dw, float lr, size_t count)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256) w[i] = w[i] - lr * dw[i];
}

// How the gradient's GEMM is tiled and split: column tiles of 64 to 4 channels per tap (whichever gives the fewest, the most channels first:
// a tap costs a padding test), and as many ranges of slices as make up to three workgroups per compute unit (two with tiles of more than one block of filters; four instead of three: 1.071
// and 1.072 over 70 layers, with more partial sums), of at least four slices
// each, but from eight slices on a range per image up to 16 (3x3 8 -> 32 at stride 4 on 15 x 18 x 10 images, ten slices: 14.0 us in two
// ranges, 11.0 in ten); the sum of the ranges costs what more or shorter ones gain (7x7 128 -> 64 at stride 2 on 10 x 37 x 2, six
// slices: 12.9 in one range, 15.5 in two, 19.0 in six).
// Blocks of 64 filters of a tile: three or two where they divide the filters' blocks, padding none, and the tiles still fill the device (7x7 74 -> 192 on 48 x 36 x 2
// in two blocks, a fourth of them empty, 35.3 us before and 38.1; one 35.9).
struct WPlan { int tm, cb_log2, cblocks, grid_m, grid_n, slices_per_img, slices, splits; };
WPlan wgrad_plan(const ConvGeom& g)
{
    WPlan p{};
    const int RS = g.R * g.S;
    int best = 0;
    for (int l = 6; l >= 2; --l) {
        const int tpt = BN >> l, cblocks = (g.C + (1 << l) - 1) >> l, n = (RS + tpt - 1) / tpt * cblocks;
        if (best && n >= best) continue;
        best = n; p.cb_log2 = l; p.cblocks = cblocks; p.grid_n = n;
    }
    p.slices_per_img = std::max(1, (g.P * g.Q + BL - 1) / BL);
    p.slices = g.P * g.Q > 0 ? g.N * p.slices_per_img : 0;
    const int most = std::max(1, std::max(p.slices / 4, p.slices >= 8 ? std::min(g.N, 16) : 1));
    const int blocks = (g.K + 63) / 64;
    p.tm = 3;
    while (p.tm > 1 && (blocks % p.tm != 0 || (long)(blocks / p.tm) * p.grid_n * most < 2 * device_cus())) --p.tm;
    p.grid_m = blocks / p.tm;
    const int tiles = p.grid_m * p.grid_n;
    p.splits = std::max(1, std::min((p.tm == 1 ? 3 : 2) * device_cus() / tiles, most));
    return p;
}

}  // namespace

size_t regression_loss_workspace_bytes() { return 4096 * sizeof(float); }

int launch_regression_loss_grad(const float* f, const float* y, float* dz, size_t count, float* loss, void* ws, hipStream_t st)
{
    TraceScope trace("loss_grad", nullptr, (long long)count, st, 3ll * count * 4);
    const bool vec = (((uintptr_t)f | (uintptr_t)y | (uintptr_t)dz) & 15) == 0;
    const size_t nvec = vec ? count / 4 : 0;
    const unsigned grid = blocks_for_train(nvec ? nvec : count);
    hipLaunchKernelGGL(regression_loss_grad_kernel, dim3(grid), dim3(256), 0, st, f, y, dz, nvec, count, (float*)ws);
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, st, (const float*)ws, (int)grid, loss);
    return check_launch("regression_loss_grad");
}

size_t conv_wgrad_workspace_bytes(const ConvGeom& g)
{
    const WPlan p = wgrad_plan(g);
    return p.splits > 1 ? (size_t)p.splits * g.K * ((size_t)p.grid_n * BN + 1) * sizeof(float) : 0;
}

int launch_conv_wgrad_f32(const ConvGeom& g, const float* x, const float* dz, float* dw, float* db, void* ws, hipStream_t st)
{
    const WPlan p = wgrad_plan(g);
    WArgs a;
    a.x = x; a.dz = dz;
    a.N = g.N; a.C = g.C; a.H = g.H; a.W = g.W; a.K = g.K; a.R = g.R; a.S = g.S;
    a.sh = g.sh; a.sw = g.sw; a.ph = g.ph; a.pw = g.pw; a.P = g.P; a.Q = std::max(1, g.Q);
    a.CRS = g.Kg;
    a.grid_m = p.grid_m; a.grid_n = p.grid_n; a.splits = p.splits; a.slices_per_img = p.slices_per_img; a.slices = p.slices;
    a.cb_log2 = p.cb_log2; a.cblocks = p.cblocks; a.cols = p.grid_n * BN;
    a.x_bytes = (int)((size_t)g.N * g.C * g.H * g.W * 4);
    a.dz_bytes = (int)((size_t)g.N * g.K * g.P * g.Q * 4);
    a.out = (float*)ws; a.dw = dw; a.db = db;
    {
        ConvGeom t = g;
        TraceScope trace("conv_wgrad_f32", &t, g.Ng, st);
        const dim3 grid((unsigned)(a.grid_m * a.grid_n * a.splits)), block(256);
        auto launch = [&](auto taps, auto eights) {
            constexpr int T = decltype(taps)::value;
            constexpr bool E = decltype(eights)::value;
            if (p.tm == 3) hipLaunchKernelGGL((conv_wgrad_f32_kernel<T, E, 3>), grid, block, 0, st, a);
            else if (p.tm == 2) hipLaunchKernelGGL((conv_wgrad_f32_kernel<T, E, 2>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((conv_wgrad_f32_kernel<T, E, 1>), grid, block, 0, st, a);
        };
        using std::integral_constant;
        const bool eights = g.C % 8 == 0;
        if (p.cb_log2 == 6) eights ? launch(integral_constant<int, 1>{}, std::true_type{}) : launch(integral_constant<int, 1>{}, std::false_type{});
        else if (p.cb_log2 == 5) eights ? launch(integral_constant<int, 2>{}, std::true_type{}) : launch(integral_constant<int, 2>{}, std::false_type{});
        else if (p.cb_log2 == 4) eights ? launch(integral_constant<int, 4>{}, std::true_type{}) : launch(integral_constant<int, 4>{}, std::false_type{});
        else if (p.cb_log2 == 3) eights ? launch(integral_constant<int, 8>{}, std::true_type{}) : launch(integral_constant<int, 8>{}, std::false_type{});
        else launch(integral_constant<int, 16>{}, std::false_type{});
    }
    if (const int rc = check_launch("conv_wgrad")) return rc;
    if (a.splits > 1) {
        const size_t count = (size_t)g.K * (a.cols + 1);
        TraceScope trace("wgrad_sum", nullptr, (long long)count, st, (long long)((a.splits + 1) * count * 4));
        hipLaunchKernelGGL(sum_splits_kernel, dim3(blocks_for_train(count)), dim3(256), 0, st, (const float*)ws, a.splits, g.K, g.C, g.R * g.S, a.cb_log2, a.cblocks,
                           a.cols, dw, db);
    }
    return check_launch("conv_wgrad");
}

int launch_sgd_step(float* w, const float* dw, float lr, size_t count, hipStream_t st)
{
    if (count == 0) return DR_OK;
    TraceScope trace("sgd_step", nullptr, (long long)count, st, 3ll * count * 4);
    hipLaunchKernelGGL(sgd_step_kernel, dim3(blocks_for_train(count)), dim3(256), 0, st, w, dw, lr, count);
    return check_launch("sgd_step");
}

}  // namespace dr
