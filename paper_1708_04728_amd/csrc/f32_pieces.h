// fp32 operands as three bf16 pieces: cutting and multiplying (conv_f32_pieces.hip has the arithmetic).
#pragma once
#include "dr_store.h"

namespace dr {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// What operands are multiplied by before they are cut, and their sums of products after.  Every fp32 value is a multiple of 2^-149, so that the pieces of a scaled one
// are multiples of 2^-125: none falls below the smallest normal bf16, 2^-126, whatever lies beside it.  Values of 2^104 and more, and sums of 2^80 and more, become
// infinities or NaN among the sums, as infinite operands do, and are then computed without pieces.
constexpr float PIECES_SCALE = 0x1p24f, PIECES_UNSCALE = 0x1p-48f;

// Eight operands as three vectors of bf16: high + middle + low == v, exactly (8 bits of the significand each, the lower ones with a sign of their own).
__device__ __forceinline__ void split8(const float (&v)[8], u32x4& high, u32x4& middle, u32x4& low)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned h = pack_bf16x2(v[2 * i], v[2 * i + 1]);
        const float ra = v[2 * i] - __uint_as_float(h << 16), rb = v[2 * i + 1] - __uint_as_float(h & 0xFFFF0000u);
        const unsigned m = pack_bf16x2(ra, rb);
        const float la = ra - __uint_as_float(m << 16), lb = rb - __uint_as_float(m & 0xFFFF0000u);
        high[i] = h;
        middle[i] = m;
        low[i] = __builtin_amdgcn_perm(__float_as_uint(lb), __float_as_uint(la), 0x07060302u);
    }
}

__device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

}  // namespace
}  // namespace dr
