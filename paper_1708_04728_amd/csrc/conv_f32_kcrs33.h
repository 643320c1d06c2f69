// The buffers and scalar offsets of the loads of conv_f32_kcrs33_kernel (conv_f32.hip).  Plain constant expressions, so that the same lines run in the kernel
// and on the host.
#pragma once

namespace dr {

constexpr int KCRS33_CB = 8, KCRS33_ROW = KCRS33_CB * 9;       // channels of a block; consecutive floats of a filter row in it

// The bytes that a load's descriptor spans and its scalar offset.  The loads run ahead of the last block, and there nothing is to be read: an empty buffer,
// beside which the scalar offset has to be 0 too, since the hardware compares a lane's offset with the bytes that are left behind the scalar part.
struct LoadRange { int bytes, scalar; };
constexpr LoadRange kcrs33_filters(int blk, int blocks, int w_bytes)
{
    return blk < blocks ? LoadRange{w_bytes, blk * KCRS33_ROW * 4} : LoadRange{0, 0};
}
// channel j of a thread's in the block; HW: elements of a plane
constexpr LoadRange kcrs33_plane(int blk, int blocks, int j, int HW, int x_bytes)
{
    return blk < blocks ? LoadRange{x_bytes, (blk * KCRS33_CB + j) * HW * 4} : LoadRange{0, 0};
}

}  // namespace dr
