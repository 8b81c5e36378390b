// Sums over lanes by data-parallel moves (DPP), without LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace bemtx {

template <int CTRL, int RM = 0xF> __device__ inline float dpp_mov(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, RM, 0xF, true));
}
template <int CTRL, int RM = 0xF> __device__ inline double dpp_mov(double v)
{
    int2 q = __builtin_bit_cast(int2, v);
    q.x = __builtin_amdgcn_update_dpp(0, q.x, CTRL, RM, 0xF, true);
    q.y = __builtin_amdgcn_update_dpp(0, q.y, CTRL, RM, 0xF, true);
    return __builtin_bit_cast(double, q);
}
// sum over the 16 lanes of a DPP row, in lane 15 of the row
template <class R> __device__ inline R rsum15(R v)
{
    v += dpp_mov<0x111>(v);        // row_shr:1
    v += dpp_mov<0x112>(v);        // row_shr:2
    v += dpp_mov<0x114>(v);        // row_shr:4
    v += dpp_mov<0x118>(v);        // row_shr:8
    return v;
}
// sum over the 64 lanes of a wave, in lane 63
template <class R> __device__ inline R wsum63(R v)
{
    v = rsum15(v);
    v += dpp_mov<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_mov<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

}  // namespace bemtx
