// What the quantisers of rows share (quantize.hip, quantize_weight.hip).
#pragma once
#include "rotate_lane.h"

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

// rotate_layers with the order of the two products of every sum written out (the one that is there first is rounded, the
// later one joins it in a fused multiply-add): a code on a rounding tie must not depend on how the compiler schedules.
template <int K, int U>
__device__ __forceinline__ void quant_rotate(const LanePlan<K> &P, float (&a)[U], float (&b)[U])
{
#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float na = l == 0 ? fmaf(P.m00[l], a[u], P.m01[l] * b[u]) : fmaf(P.m01[l], b[u], P.m00[l] * a[u]);
            const float nb = l == 0 ? fmaf(P.m10[l], a[u], P.m11[l] * b[u]) : fmaf(P.m11[l], b[u], P.m10[l] * a[u]);
            a[u] = na;
            b[u] = (l + 1 < K) ? __int_as_float(__builtin_amdgcn_ds_bpermute(P.src[l], __float_as_int(nb))) : nb;
        }
}

}  // namespace paro
