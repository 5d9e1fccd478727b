// What the quantisers of rows share (quantize.hip, quantize_weight.hip).
#pragma once
#include "paro_internal.h"

namespace paro {

// v of another lane of the same 16 (DPP control word CTRL)
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

// 1 / s of an fp16 value s >= 2^-14, correctly rounded: the hardware's estimate and one Newton step (compared with the division
// on all of them)
__device__ __forceinline__ float quant_rcp(float s)
{
    const float r = __builtin_amdgcn_rcpf(s);
    return fmaf(fmaf(-s, r, 1.0f), r, r);
}

}  // namespace paro
