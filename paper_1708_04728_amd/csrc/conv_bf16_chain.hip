// The 1x1 convolutions around the residual sum of a folded ResNet bottleneck (Sec. 4.2) in one pass over the pixels:
//
//   y  = max(W3 m + b3 + s, 0)                 m: the 3x3 layer's output (or that layer here too), s: the block's input or Wp x + bp (projected shortcut)
//   m' = max(W1' y + b1', 0)                   the first layer of the bottleneck behind it, if there is one
//
// What bounds these layers is HBM: 64 -> 256 with its residual moves 1.2 KB per pixel for 33 KFLOP.  As layers of their own the
// projected shortcut is written and read once more, and y is read once more by the layer behind it.  Here both stay in registers.
// After the lane exchange of the store a lane holds 8 consecutive filters of its pixel, rounded to bf16: that is the matrix
// instruction's second operand for the next contraction over those filters (see pack_blocks), so m' takes y's registers as they are.
//
// A wave works alone: 32 pixels at a time, all filters, no barrier after the filters have reached LDS (each 1 KB fragment in the
// order the lanes read it, so reads are free of bank conflicts).  The next 32 pixels' operands and residuals are requested while the current
// ones are multiplied: 20 KB per wave in flight, eight waves per compute unit (one workgroup: the filters take up to 96 KB; ten or
// twelve waves: no faster).  A round's pixels lie next to one another across the whole device: a run of pixels per workgroup or
// per die took 7 % longer.
// What a lane holds of a tensor is 16 bytes of a pixel, half a line's quarter: an instruction that moves them as they are touches 32 lines for 1 KB,
// and the address path then takes longer than memory.  Where there are enough blocks to hide it every piece goes through LDS and an
// instruction moves eight whole lines: with the residual, 128 images of 56 x 56, 139 -> 101 us (117 -> 90 without a next layer); addresses that run on
// without a gap (in a working copy) 98 and 86.
// ResNet's conv2_x, three folded blocks on 56 x 56: 128 images 625 us as single layers, 402 in chains without and 380 with their 3x3 layers; 30 images
// 163, 122 and 106; one image 52, 42 and 39.
// What bounds the kernel that reads m: HBM, at 5.1 TB/s on the bytes left (360 MB in the first launch of that stage), as much as a copy reaches.
// The sums run in the order of the streaming kernel and every tensor it would store is rounded where it would be: the same bits.
#include "dr_internal.h"
#include "dr_store.h"
#include "conv_bf16_dev.h"

namespace dr {
namespace {

constexpr int CHAIN_WAVES = 8, CHAIN_KS = CHAIN_MID / 16, CHAIN_OB = CHAIN_OUT / 32, CHAIN_FRAGS = CHAIN_OB * CHAIN_KS;
constexpr int PART = 32 * 8;      // 16-byte chunks of 64 channels of 32 pixels: what moves between memory and LDS at a time

struct ChainArgs {
    ConvChain c;
    int m_bytes, y_bytes, x_bytes, next_bytes;
    unsigned long long magic_w, magic_h;     // for div_small (w_mid)
};

__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t r, int voff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
#else
    return u32x4{};
#endif
}
__device__ __forceinline__ void store16(u32x4 v, __amdgpu_buffer_rsrc_t r, int voff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, 0);
#endif
}
__device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// result registers 8 qp .. 8 qp + 7 of both halves of a pixel -> 8 consecutive filters
__device__ __forceinline__ void exchange(const f32x16& acc, int qp, float (&o)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[qp * 8 + e]), __float_as_uint(acc[qp * 8 + 4 + e]), false, false);
        o[e] = __uint_as_float(sw[0]);
        o[4 + e] = __uint_as_float(sw[1]);
    }
}
__device__ __forceinline__ void add_bias(const float* b, float (&o)[8])
{
    const f32x4 lo = *reinterpret_cast<const f32x4*>(b), hi = *reinterpret_cast<const f32x4*>(b + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { o[e] += lo[e]; o[4 + e] += hi[e]; }
}
__device__ __forceinline__ void relu8(float (&o)[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = fmaxf(o[e], 0.f);
}
__device__ __forceinline__ u32x4 pack8(const float (&o)[8])
{
    u32x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = pack_bf16x2(o[2 * e], o[2 * e + 1]);
    return pk;
}

// A value of which the compiler knows nothing.  Lanes read in `stage` what other lanes of their wave have written, and a wave's LDS instructions run in order:
// what has to be kept is the order of the program.  The compiler keeps it where one lane's write and read may be the same place, which with an index that
// comes from here they may, whatever it finds out about the others.  (A fence at wavefront scope in each place keeps more than that: one to eight images of
// 56 x 56 2 % longer in the kernel with the 3x3 layer, spills in the other.)
__device__ __forceinline__ int unknown(int v)
{
    asm("" : "+v"(v));
    return v;
}

// PROJ: the shortcut is Wp x; NEXT: m' is computed; LINES: memory is read and written by whole lines, through LDS
template <bool PROJ, bool NEXT, bool LINES>
__global__ __launch_bounds__(CHAIN_WAVES * 64) void conv_bf16_chain_kernel(const ChainArgs a)
{
    __shared__ u32x4 frag[(1 + PROJ + NEXT) * CHAIN_FRAGS * 64];
    __shared__ u32x4 stage_out[LINES ? CHAIN_WAVES * PART : 1], stage_res[LINES && !PROJ ? CHAIN_WAVES * PART : 1];
    u32x4* const stage_in = PROJ ? stage_out : stage_res;
    __shared__ __attribute__((aligned(16))) float bias[2 * CHAIN_OUT + CHAIN_MID];
    const ConvChain& c = a.c;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5, l32 = lane & 31;
    u32x4* const f_out = frag;
    u32x4* const f_proj = frag + (PROJ ? CHAIN_FRAGS * 64 : 0);
    u32x4* const f_next = frag + (1 + PROJ) * CHAIN_FRAGS * 64;

    // ---- filters and biases, zeros beyond the layers' own: fragment (i, ks) holds filters 32 i .., channels 16 ks .. of a bank
    auto bank = [&](u32x4* dst, const uint16_t* w, int rows, int cols, int ksteps) {
        for (int e = tid; e < CHAIN_FRAGS * 64; e += CHAIN_WAVES * 64) {
            const int f = e >> 6, i = f / ksteps, ks = f - i * ksteps;
            const int row = i * 32 + (e & 31), col = ks * 16 + ((e >> 5) & 1) * 8;
            dst[e] = row < rows && col < cols ? *reinterpret_cast<const u32x4*>(w + (size_t)row * cols + col) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    bank(f_out, c.w, c.out, c.mid, CHAIN_KS);
    if constexpr (PROJ) bank(f_proj, c.w_proj, c.out, c.c_in, CHAIN_KS);
    if constexpr (NEXT) bank(f_next, c.w_next, c.next, c.out, 2 * CHAIN_OB);
    for (int e = tid; e < CHAIN_OUT; e += CHAIN_WAVES * 64) {
        bias[e] = c.bias && e < c.out ? c.bias[e] : 0.f;
        if constexpr (PROJ) bias[CHAIN_OUT + e] = c.bias_proj && e < c.out ? c.bias_proj[e] : 0.f;
        if constexpr (NEXT)
            if (e < CHAIN_MID) bias[2 * CHAIN_OUT + e] = c.bias_next && e < c.next ? c.bias_next[e] : 0.f;
    }
    __syncthreads();

    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc((void*)c.m, 0, a.m_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)c.x, 0, a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)c.y, 0, a.y_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc((void*)c.m_next, 0, a.next_bytes, 0x00020000);
    const int blocks = (c.pixels + 31) >> 5, stride = (int)gridDim.x * CHAIN_WAVES;
    // The matrix instructions want chunk 2 q + half (8 channels) of pixel l & 31 of 64 channels.  LINES: a lane moves chunk l & 7 of pixel l >> 3 of
    // each eight instead, and `stage`, the wave's own, turns one into the other; chunk c of pixel p lies at c ^ (p & 7).
    const int line = wave * PART + (lane & 56) + ((lane & 7) ^ (lane >> 3)), op = unknown(wave * PART + l32 * 8), sw = l32 & 7;
    auto at = [&](int blk, int j, int C, int ch) __attribute__((always_inline)) {      // zeros are read, nothing written outside the tensor
        const int n = blk * 32 + (LINES ? j * 8 + (lane >> 3) : l32), c0 = ch + (LINES ? lane & 7 : 2 * j + half) * 8;
        return n < c.pixels && c0 < C ? (n * C + c0) * 2 : OOB;
    };
    auto fetch = [&](u32x4* v, __amdgpu_buffer_rsrc_t r, int blk, int C, int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = load16(r, at(blk, j, C, ch));
    };
    auto to_operands = [&](const u32x4* v, u32x4* o) __attribute__((always_inline)) {
        if constexpr (LINES) {
#pragma unroll
            for (int j = 0; j < 4; ++j) stage_in[line + j * 64] = v[j];
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = stage_in[op + ((2 * q + half) ^ sw)];
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = v[q];
        }
    };
    auto store = [&](const u32x4* o, __amdgpu_buffer_rsrc_t r, int blk, int C, int ch) __attribute__((always_inline)) {
        if constexpr (LINES) {
#pragma unroll
            for (int q = 0; q < 4; ++q) stage_out[op + ((2 * q + half) ^ sw)] = o[q];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) store16(LINES ? stage_out[line + j * 64] : o[j], r, at(blk, j, C, ch));
    };

    u32x4 mem_m[CHAIN_KS], mem_x[PROJ ? CHAIN_KS : 1], res[PROJ ? 1 : 2 * CHAIN_OB];      // as fetched
    int blk = (int)blockIdx.x + wave * (int)gridDim.x;
    fetch(mem_m, rm, blk, c.mid, 0);
    if constexpr (PROJ) {
        fetch(mem_x, rx, blk, c.c_in, 0);
    } else {
#pragma unroll
        for (int p = 0; p < CHAIN_OB / 2; ++p) fetch(res + 4 * p, rx, blk, c.out, 64 * p);
    }
    for (; blk < blocks; blk += stride) {
        u32x4 vm[CHAIN_KS], vx[PROJ ? CHAIN_KS : 1];
        to_operands(mem_m, vm);
        fetch(mem_m, rm, blk + stride, c.mid, 0);
        if constexpr (PROJ) {
            to_operands(mem_x, vx);
            fetch(mem_x, rx, blk + stride, c.c_in, 0);
        }
        // (the filters and biases read below are the same in every round: without this the compiler would fetch all of them ahead
        // of the loop, into registers it does not have)
        int fl = lane, bl = half * 8;
        asm volatile("" : "+v"(fl), "+v"(bl));
        u32x4 out[4], sc[2][4];
        auto next_res = [&](int p) __attribute__((always_inline)) {
            to_operands(res + 4 * p, sc[p & 1]);
            fetch(res + 4 * p, rx, blk + stride, c.out, p * 64);
        };
        f32x16 sum_next[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) sum_next[0][v] = sum_next[1][v] = 0.f;
#pragma unroll
        for (int i = 0; i < CHAIN_OB; ++i) {
            if constexpr (!PROJ) {
                if (i == 0) next_res(0);
                if (!(i & 1) && i + 2 < CHAIN_OB) next_res(i / 2 + 1);
            }
            f32x16 acc, accp;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = accp[v] = 0.f;
#pragma unroll
            for (int ks = 0; ks < CHAIN_KS; ++ks) {
                acc = mfma(f_out[(i * CHAIN_KS + ks) * 64 + fl], vm[ks], acc);
                if constexpr (PROJ) accp = mfma(f_proj[(i * CHAIN_KS + ks) * 64 + fl], vx[ks], accp);
            }
#pragma unroll
            for (int qp = 0; qp < 2; ++qp) {
                float o[8];
                exchange(acc, qp, o);
                add_bias(bias + i * 32 + qp * 16 + bl, o);
                u32x4 s;
                if constexpr (PROJ) {
                    float op[8];
                    exchange(accp, qp, op);
                    add_bias(bias + CHAIN_OUT + i * 32 + qp * 16 + bl, op);
                    s = pack8(op);
                } else {
                    s = sc[i >> 1 & 1][(i & 1) * 2 + qp];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[2 * e] += __uint_as_float(s[e] << 16);
                    o[2 * e + 1] += __uint_as_float(s[e] & 0xFFFF0000u);
                }
                relu8(o);
                const u32x4 pk = pack8(o);
                out[(i & 1) * 2 + qp] = pk;
                if constexpr (NEXT) {
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) sum_next[mb] = mfma(f_next[(mb * 2 * CHAIN_OB + 2 * i + qp) * 64 + fl], pk, sum_next[mb]);
                }
            }
            if (i & 1) store(out, ry, blk, c.out, (i - 1) * 32);
        }
        if constexpr (NEXT) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int qp = 0; qp < 2; ++qp) {
                    float o[8];
                    exchange(sum_next[mb], qp, o);
                    add_bias(bias + 2 * CHAIN_OUT + mb * 32 + qp * 16 + bl, o);
                    relu8(o);
                    out[2 * mb + qp] = pack8(o);
                }
            store(out, rn, blk, c.next, 0);
        }
    }
}

// The 3x3 layer in front of the expansion computed here too: its output m never leaves the compute unit.  Four waves multiply, 32 pixels each, and four
// load what the 3x3 layer needs into LDS: the tile's input patch -- the 128 pixels and a row and a pixel on either side of them, one run of memory, since
// pixels are numbered through rows and images; a tap outside the image reads a row of zeros -- and its filters by taps, through a ring of three.  Loads
// of the multiplying waves (residuals, a tile ahead) and of the loading ones are then waited for apart, which one memory counter for both would not
// allow.  The waves meet at every tap and once behind the last, from where on the loading waves bring the next tile's patch.
// What it is worth, layer and chain kernel -> this one, conv2_x of 1, 8, 30 and 128 images: 42 -> 39, 70 -> 57, 122 -> 106 and 402 -> 380 us; 90 maps of
// 33 x 51 186 -> 163.  W > 63 does not fit the patch, a projected block
// not the filters: those keep the layer of their own.
// What bounds it: a tile takes a multiplying wave about 24000 cycles, its bytes' share of HBM 17000; one such wave per SIMD, so that its LDS reads, stores
// and vector work (a lane exchange and a conversion for every result) are not hidden by another.  Tried: eight multiplying waves, which leaves
// registers for residuals half as far ahead, 415 us; four with that 392; no LDS for the 3x3 layer, its taps read from memory by every wave, 508.
constexpr int MID_PX = 128, MID_PATCH = 256, MID_RING = 3, TAPS = 9;      // pixels of a tile; pixels its patch may have (W <= 63); taps in LDS

template <bool NEXT>
__global__ __launch_bounds__(512, 2) void conv_bf16_chain_mid_kernel(const ChainArgs a)
{
    __shared__ u32x4 frag[(1 + NEXT) * CHAIN_FRAGS * 64];
    __shared__ __attribute__((aligned(1024))) unsigned char ring[MID_RING * CHAIN_MID * 128];
    __shared__ __attribute__((aligned(1024))) unsigned char patch[(MID_PATCH + 1) * 128];       // the last row: zeros
    __shared__ u32x4 stage_out[4 * PART], stage_in[4 * PART];
    __shared__ __attribute__((aligned(16))) float bias[CHAIN_OUT + 2 * CHAIN_MID];
    const ConvChain& c = a.c;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5, l32 = lane & 31;
    u32x4* const f_out = frag;
    u32x4* const f_next = frag + (NEXT ? CHAIN_FRAGS * 64 : 0);
    const int tiles = (c.pixels + MID_PX - 1) / MID_PX, G = (int)gridDim.x, W = c.w_map;
    // a round's tiles lie next to one another across the device, a die's (workgroup id & 7) next to one another: they share their patches' rows
    const int b = (int)blockIdx.x, first = G % 8 == 0 ? (b & 7) * (G >> 3) + (b >> 3) : b;

    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc((void*)c.m, 0, a.m_bytes, 0x00020000);
    const int lw = wave & 3, lrow = lw * 8 + (lane >> 3), lc = (lane & 7) ^ ((lrow >> 1) & 7);      // (loading: row of 32, chunk of the row; chunk j of row r lies at j ^ ((r >> 1) & 7))
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)c.w_mid, 0, CHAIN_MID * TAPS * CHAIN_MID * 2, 0x00020000);
    auto load_patch = [&](int tile) __attribute__((always_inline)) {
        const int n0 = tile * MID_PX - W - 1 + lrow;
#pragma unroll
        for (int i = 0; i < MID_PATCH / 32; ++i) {
            const int n = n0 + i * 32;
            load_to_lds16(rm, patch + i * 4096 + lw * 1024, n >= 0 && n < c.pixels ? n * (CHAIN_MID * 2) + lc * 16 : OOB, 0);
        }
    };
    auto load_tap = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            load_to_lds16(rw, ring + t % MID_RING * (CHAIN_MID * 128) + i * 4096 + lw * 1024, ((i * 32 + lrow) * (TAPS * CHAIN_MID) + lc * 8) * 2, t * (CHAIN_MID * 2));
    };
    if (wave >= 4 && first < tiles) {
        load_patch(first);
        load_tap(0);
        load_tap(1);
    }
    auto bank = [&](u32x4* dst, const uint16_t* w, int rows, int cols, int ksteps) {
        for (int e = tid; e < CHAIN_FRAGS * 64; e += 512) {
            const int f = e >> 6, i = f / ksteps, ks = f - i * ksteps;
            const int row = i * 32 + (e & 31), col = ks * 16 + ((e >> 5) & 1) * 8;
            dst[e] = row < rows && col < cols ? *reinterpret_cast<const u32x4*>(w + (size_t)row * cols + col) : u32x4{0u, 0u, 0u, 0u};
        }
    };
    bank(f_out, c.w, c.out, CHAIN_MID, CHAIN_KS);
    if constexpr (NEXT) bank(f_next, c.w_next, c.next, c.out, 2 * CHAIN_OB);
    for (int e = tid; e < CHAIN_OUT; e += 512) {
        bias[e] = c.bias && e < c.out ? c.bias[e] : 0.f;
        if (e < CHAIN_MID) {
            bias[CHAIN_OUT + e] = c.bias_mid ? c.bias_mid[e] : 0.f;
            bias[CHAIN_OUT + CHAIN_MID + e] = NEXT && c.bias_next && e < c.next ? c.bias_next[e] : 0.f;
        }
    }
    if (tid < 32) reinterpret_cast<unsigned*>(patch + MID_PATCH * 128)[tid] = 0u;

    if (wave >= 4) {
        for (int tile = first; tile < tiles; tile += G) {
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
                if (t + 1 < TAPS) wait_vmcnt<2>();
                else wait_vmcnt<0>();
                ring_barrier();                       // tap t has landed, tap t - 1 has been read
                if (t + 2 < TAPS) load_tap(t + 2);
            }
            ring_barrier();                           // the last tap and the patch have been read
            if (tile + G < tiles) {
                load_patch(tile + G);
                load_tap(0);
                load_tap(1);
            }
        }
        return;
    }

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)c.x, 0, a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void*)c.y, 0, a.y_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rn = __builtin_amdgcn_make_buffer_rsrc((void*)c.m_next, 0, a.next_bytes, 0x00020000);
    // memory by whole lines, as in the kernel above
    const int line = wave * PART + (lane & 56) + ((lane & 7) ^ (lane >> 3)), op = unknown(wave * PART + l32 * 8), sw = l32 & 7;
    auto at = [&](int n0, int j, int C, int ch) __attribute__((always_inline)) {
        const int n = n0 + j * 8 + (lane >> 3), c0 = ch + (lane & 7) * 8;
        return n < c.pixels && c0 < C ? (n * C + c0) * 2 : OOB;
    };
    u32x4 res[2 * CHAIN_OB];
    auto fetch_res = [&](int n0, int p) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) res[4 * p + j] = load16(rx, at(n0, j, c.out, 64 * p));
    };
    auto to_operands = [&](const u32x4* v, u32x4* o) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) stage_in[line + j * 64] = v[j];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = stage_in[op + ((2 * q + half) ^ sw)];
    };
    auto store = [&](const u32x4* o, __amdgpu_buffer_rsrc_t r, int n0, int C, int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) stage_out[op + ((2 * q + half) ^ sw)] = o[q];
#pragma unroll
        for (int j = 0; j < 4; ++j) store16(stage_out[line + j * 64], r, at(n0, j, C, ch));
    };
    const unsigned char* const a_rd = ring + l32 * 128;
    const int a_sw = half ^ ((l32 >> 1) & 7);
#pragma unroll
    for (int p = 0; p < CHAIN_OB / 2; ++p) fetch_res(first * MID_PX + wave * 32, p);

    for (int tile = first; tile < tiles; tile += G) {
        const int n0 = tile * MID_PX + wave * 32, n = n0 + l32, next0 = n0 + G * MID_PX;      // this wave's pixels now and in the next round
        unsigned taps = 0u;                               // a bit for each tap inside the image
        if (n < c.pixels) {
            const int row = div_small(n, a.magic_w), q = n - row * W, p = row - div_small(row, a.magic_h) * c.h_map;
            const unsigned cols = (q > 0 ? 1u : 0u) | 2u | (q < W - 1 ? 4u : 0u);
            taps = (p > 0 ? cols : 0u) | cols << 3 | (p < c.h_map - 1 ? cols << 6 : 0u);
        }
        // ---- the 3x3 layer.  Behind the barrier of a tap its operands are read while the tap before it is multiplied.
        f32x16 sum[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[0][v] = sum[1][v] = 0.f;
        u32x4 fa[2][2][CHAIN_KS], fb[2][CHAIN_KS];
        auto multiply = [&](int s) __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < CHAIN_KS; ++ks)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) sum[mb] = mfma(fa[s][mb][ks], fb[s][ks], sum[mb]);
        };
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            const int row = taps >> t & 1u ? wave * 32 + l32 + t / 3 * W + t % 3 : MID_PATCH, b_sw = half ^ ((row >> 1) & 7);
            const unsigned char* const b_rd = patch + row * 128;
            ring_barrier();
#pragma unroll
            for (int ks = 0; ks < CHAIN_KS; ++ks) {
                fb[t & 1][ks] = *reinterpret_cast<const u32x4*>(b_rd + ((b_sw ^ (2 * ks)) << 4));
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
                    fa[t & 1][mb][ks] = *reinterpret_cast<const u32x4*>(a_rd + t % MID_RING * (CHAIN_MID * 128) + mb * 4096 + ((a_sw ^ (2 * ks)) << 4));
            }
            if (t) multiply((t + 1) & 1);
        }
        ring_barrier();
        multiply((TAPS - 1) & 1);
        u32x4 vm[CHAIN_KS], out[4], sc[2][4];
        int fl = lane, bl = half * 8;                     // (see the kernel above)
        asm volatile("" : "+v"(fl), "+v"(bl));
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int qp = 0; qp < 2; ++qp) {
                float o[8];
                exchange(sum[mb], qp, o);
                add_bias(bias + CHAIN_OUT + mb * 32 + qp * 16 + bl, o);
                relu8(o);
                vm[2 * mb + qp] = pack8(o);
            }
        // ---- the expansion, the residual sum and the next block's first layer
        auto next_res = [&](int p) __attribute__((always_inline)) {
            to_operands(res + 4 * p, sc[p & 1]);
            fetch_res(next0, p);
        };
        f32x16 sum_next[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) sum_next[0][v] = sum_next[1][v] = 0.f;
#pragma unroll
        for (int i = 0; i < CHAIN_OB; ++i) {
            if (i == 0) next_res(0);
            if (!(i & 1) && i + 2 < CHAIN_OB) next_res(i / 2 + 1);
            f32x16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
            for (int ks = 0; ks < CHAIN_KS; ++ks) acc = mfma(f_out[(i * CHAIN_KS + ks) * 64 + fl], vm[ks], acc);
#pragma unroll
            for (int qp = 0; qp < 2; ++qp) {
                float o[8];
                exchange(acc, qp, o);
                add_bias(bias + i * 32 + qp * 16 + bl, o);
                const u32x4 s = sc[i >> 1 & 1][(i & 1) * 2 + qp];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[2 * e] += __uint_as_float(s[e] << 16);
                    o[2 * e + 1] += __uint_as_float(s[e] & 0xFFFF0000u);
                }
                relu8(o);
                const u32x4 pk = pack8(o);
                out[(i & 1) * 2 + qp] = pk;
                if constexpr (NEXT) {
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) sum_next[mb] = mfma(f_next[(mb * 2 * CHAIN_OB + 2 * i + qp) * 64 + fl], pk, sum_next[mb]);
                }
            }
            if (i & 1) store(out, ry, n0, c.out, (i - 1) * 32);
        }
        if constexpr (NEXT) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int qp = 0; qp < 2; ++qp) {
                    float o[8];
                    exchange(sum_next[mb], qp, o);
                    add_bias(bias + CHAIN_OUT + CHAIN_MID + mb * 32 + qp * 16 + bl, o);
                    relu8(o);
                    out[2 * mb + qp] = pack8(o);
                }
            store(out, rn, n0, c.next, 0);
        }
    }
}

// Lines from 1024 blocks of 32 pixels on, half of what the waves hold at a time: 16 images of 56 x 56 (1568) 93.2 us without, 90.9 with, eight (784)
// 69.7 and 69.7.  With fewer a wave has one block and the way through LDS only adds to its latency: four images 52.1 and 52.7, one 41.9 and 43.2.
template <bool PROJ, bool NEXT>
int launch_chain(const ChainArgs& a, hipStream_t st)
{
    const int blocks = (a.c.pixels + 31) / 32, cus = device_cus();
    const dim3 grid((unsigned)(blocks < cus ? blocks : cus)), block(CHAIN_WAVES * 64);
    if (blocks >= 4 * cus)
        hipLaunchKernelGGL((conv_bf16_chain_kernel<PROJ, NEXT, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((conv_bf16_chain_kernel<PROJ, NEXT, false>), grid, block, 0, st, a);
    return check_launch("conv_bf16_chain");
}

}  // namespace

// Whole 16-byte channel groups, widths the kernel's registers hold, 32-bit offsets (also for the pixels a wave asks for past the end).
bool conv_bf16_chain_eligible(const ConvChain& c)
{
    const auto width = [](int v, int most) { return v >= 8 && v % 8 == 0 && v <= most; };
    if (!width(c.mid, CHAIN_MID) || !width(c.out, CHAIN_OUT) || !width(c.c_in, c.w_proj ? CHAIN_MID : CHAIN_OUT) || (!c.w_proj && c.c_in != c.out)) return false;
    if (c.w_next && !width(c.next, CHAIN_MID)) return false;
    if (c.w_mid && (c.w_proj || c.mid != CHAIN_MID || MID_PX + 2 * c.w_map + 2 > MID_PATCH || c.h_map > (1 << 16) || !aligned16(c.w_mid))) return false;
    if (!aligned16(c.m) || !aligned16(c.x) || !aligned16(c.y) || !aligned16(c.m_next) || !aligned16(c.w) || !aligned16(c.w_proj) || !aligned16(c.w_next)) return false;
    return c.pixels > 0 && c.pixels < (1 << 24) && (double)c.pixels * c.out * 2.0 < 2147483648.0;
}

int launch_conv_bf16_chain(const ConvChain& c, hipStream_t st)
{
    ChainArgs a;
    a.c = c;
    a.m_bytes = c.pixels * c.mid * 2;
    a.x_bytes = c.pixels * c.c_in * 2;
    a.y_bytes = c.pixels * c.out * 2;
    a.next_bytes = c.w_next ? c.pixels * c.next * 2 : 0;
    a.magic_w = a.magic_h = 0;
    if (c.w_mid) {
        a.magic_w = ((1ull << 40) + (unsigned)c.w_map - 1) / (unsigned)c.w_map;
        a.magic_h = ((1ull << 40) + (unsigned)c.h_map - 1) / (unsigned)c.h_map;
        const int tiles = (c.pixels + MID_PX - 1) / MID_PX, cus = device_cus();
        const dim3 grid((unsigned)(tiles < cus ? tiles : cus)), block(512);
        if (c.w_next) hipLaunchKernelGGL(conv_bf16_chain_mid_kernel<true>, grid, block, 0, st, a);
        else hipLaunchKernelGGL(conv_bf16_chain_mid_kernel<false>, grid, block, 0, st, a);
        return check_launch("conv_bf16_chain");
    }
    if (c.w_proj) return c.w_next ? launch_chain<true, true>(a, st) : launch_chain<true, false>(a, st);
    return c.w_next ? launch_chain<false, true>(a, st) : launch_chain<false, false>(a, st);
}

}  // namespace dr
