// INT4 quantiser of Eq. 1 (formats and decisions: quantize.hip) for large weights that are not transformed.
//
// quantize_kernel holds two values of a row per lane and reduces over the wave, 28672 x 4096 84 us; here a wave has 32 rows of one
// group and lanes r and r + 32 the two halves of row r: a row's extrema are one exchange between the two, its scale and zero point
// are computed once for the 32 rows, and eight codes of consecutive channels are in one lane.  63 us (295 MB read and written: 60 at
// the rate of a large copy; 50 where the weight is still in the last-level cache).  The same bits: no result of a row depends on other rows.
//
// A transform stays with quantize_kernel.  One matrix per group through the matrix cores, kept as two fp16 parts (22 bits), was built: 139 -> 101
// us, but it is further off from 64 bits than fp32 coefficients where layers or pairs are few (one layer of 8 pairs 1.4 times), and a
// row's codes then depend on how many rows the call has, since small calls are slower that way.
#include "paro_internal.h"
#include "quantize_common.h"
#include <type_traits>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x4 u32x4_any __attribute__((aligned(4)));

struct PlainQuantArgs {
    const _Float16 *W; int64_t ldw;
    int N, C;
    uint32_t *codes;                         // [N][C/8]
    _Float16 *scales;                        // [C/128][N]
    uint32_t *qzeros;                        // [C/128][N/8]
};

constexpr int kPlainWaves = 4;               // waves per block, 32 rows each (two runs of 32 per wave are 7 % slower)
constexpr int kTileRows = 32;
constexpr int kStageBytes = kTileRows * kGroup * 2;

template <int N, class F, int I = 0>
__device__ __forceinline__ void wq_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        wq_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}

// max of v and of the lane 32 further (both lanes get it)
__device__ __forceinline__ float max_halves(float v)
{
    const u32x2 t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}

__global__ __launch_bounds__(kPlainWaves * 64, 4) void quantize_plain_kernel(PlainQuantArgs a)
{
    __shared__ __attribute__((aligned(16))) char s_rows[kPlainWaves][kStageBytes];
    const int g = blockIdx.x;
    const int lane = threadIdx.x & 63, half = lane >> 5, trow = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.y * kPlainWaves + wave;
    if (tile * kTileRows >= a.N) return;
    char *stage = s_rows[wave];

    // 16 bytes of row 4 i + lane / 16; rows beyond the last repeat it and are not written
    const _Float16 *w0 = a.W + (size_t)g * kGroup + (lane & 15) * 8;
    u32x4 in[8];
    wq_for<8>([&](auto I) { in[I] = *(const u32x4_any *)(w0 + (int64_t)min(tile * kTileRows + 4 * I + (lane >> 4), a.N - 1) * a.ldw); });
    wq_for<8>([&](auto I) {
        const int r = 4 * I + (lane >> 4);
        *(u32x4 *)(stage + r * 256 + (((lane & 15) ^ (r & 15)) << 4)) = in[I];
    });
    __builtin_amdgcn_wave_barrier();
    const int row = tile * kTileRows + trow;             // the row this lane has half of: channels 64 half + 8 k .. + 7
    const bool live = row < a.N;
    half8 x[8];
    wq_for<8>([&](auto K) { x[K] = *(const half8 *)(stage + trow * 256 + (((8 * half + K) ^ (trow & 15)) << 4)); });
    __builtin_amdgcn_wave_barrier();

    half2v hx = {x[0][0], x[0][1]}, hn = hx;
#pragma unroll
    for (int i = 2; i < 64; i += 2) {
        const half2v h = {x[i / 8][i % 8], x[i / 8][i % 8 + 1]};
        hx = __builtin_elementwise_max(hx, h); hn = __builtin_elementwise_min(hn, h);
    }
    const float mxv = max_halves((float)__builtin_elementwise_max(hx[0], hx[1]));
    const float mnv = -max_halves(-(float)__builtin_elementwise_min(hn[0], hn[1]));
    // scale, reciprocal and zero point as in quantize_kernel
    const float range = mxv - mnv;
    constexpr float kR15 = 1.0f / 15.0f;
    const float s15 = range * kR15;
    float s32 = range < __builtin_inff() ? fmaf(fmaf(-15.0f, s15, range), kR15, s15) : range;
    if (!(s32 >= 6.103515625e-05f)) s32 = 6.103515625e-05f;
    const _Float16 s16 = (_Float16)s32;
    const float s = (float)s16, rs = range < __builtin_inff() && s < __builtin_inff() ? quant_rcp(s) : 0.f;
    // without a reciprocal the scale is infinite or, the range being NaN, the floor: then the product with `by` is the quotient
    const bool plain = rs > 0.f;
    const float by = plain ? rs : s < __builtin_inff() ? 16384.f : 0.f;
    float zq = mnv * by;
    zq = plain ? fmaf(fmaf(-s, zq, mnv), by, zq) : zq;
    const float zf = __builtin_amdgcn_fmed3f(-rintf(zq), 0.0f, 15.0f);
    // rint(v / s) + z between 0 and 15 (a NaN: 0), as the low bits of v / s, held between -z and 15 - z, plus 1.5 * 2^23;
    // four of these shifted together, less what the four constants come to, are the half-word of four codes
    const float lo = -zf, hi = 15.f - zf;
    const uint32_t base = (0x4B400000u - (uint32_t)zf) * 0x1111u;
    uint32_t c4[16];
    auto code4 = [&](auto K, auto quotient) {
        uint32_t c = 0;
        wq_for<4>([&](auto U) {
            constexpr int i = 4 * K + U;
            const float q = __builtin_amdgcn_fmed3f(quotient((float)x[i / 8][i % 8]), lo, hi) + 12582912.f;
            c = U == 0 ? __float_as_uint(q) - base : (__float_as_uint(q) << (4 * U)) + c;
            asm("" : "+v"(c));                           // (or the sums are regrouped into separate shifts)
        });
        c4[K] = c;
        if constexpr (K % 2) __builtin_amdgcn_sched_barrier(0);          // (or all 64 values are live at once)
    };
    const bool all_plain = __all(plain);
    wq_for<8>([&](auto PART) {                           // (in parts: what the two branches share would be live for all of them)
        if (all_plain)
            wq_for<2>([&](auto K) {
                code4(std::integral_constant<int, PART * 2 + K>{}, [&](float f) { const float q0 = f * by; return fmaf(fmaf(-s, q0, f), by, q0); });
            });
        else
            wq_for<2>([&](auto K) {
                code4(std::integral_constant<int, PART * 2 + K>{},
                      [&](float f) { const float q0 = f * by, q = fmaf(fmaf(-s, q0, f), by, q0); return plain ? q : q0; });
            });
    });
    if (half == 0 && live) a.scales[(size_t)g * a.N + row] = s16;
    uint32_t z = (uint32_t)zf << (4 * (lane & 7));       // 8 rows to a word; N is a multiple of 8
    auto other = [&](auto CTRL) { z |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)z, decltype(CTRL)::value, 0xf, 0xf, true); };
    other(std::integral_constant<int, kQuadXor1>{}); other(std::integral_constant<int, kQuadXor2>{});
    other(std::integral_constant<int, kHalfMirror>{});
    if (half == 0 && (lane & 7) == 0 && live) a.qzeros[(size_t)g * (a.N / 8) + row / 8] = z;
    if (live) {
        uint32_t words[8];
        wq_for<8>([&](auto K) { words[K] = __builtin_amdgcn_perm(c4[2 * K + 1], c4[2 * K], 0x05040100u); });
        u32x4_any *out = (u32x4_any *)(a.codes + (size_t)row * (a.C / 8) + (size_t)g * (kGroup / 8) + 8 * half);
        const u32x4 c0 = {words[0], words[1], words[2], words[3]}, c1 = {words[4], words[5], words[6], words[7]};
        __builtin_nontemporal_store(c0, out);
        __builtin_nontemporal_store(c1, out + 1);
    }
}

// Back-to-back calls over 400 MB of weights, us, quantize_kernel / this one: 20736 (row, group) pairs 4.4 / 4.4, 35520 6.4 / 6.2,
// 4096 x 4096 (131072) 18.6 / 11.0, 28672 x 4096 84 / 63.  (MXFP4 is memory-bound on either.)
bool quantize_plain_pays(int N, int C) { return (int64_t)N * (C / kGroup) >= 24576; }

hipError_t launch_quantize_plain(const paro_half_t *W, int64_t ldw, int N, int C, uint32_t *codes, paro_half_t *scales, uint32_t *qzeros, hipStream_t s)
{
    const PlainQuantArgs a{(const _Float16 *)W, ldw, N, C, codes, (_Float16 *)scales, qzeros};
    const int tiles = (N + kTileRows - 1) / kTileRows;
    hipLaunchKernelGGL(quantize_plain_kernel, dim3(C / kGroup, (tiles + kPlainWaves - 1) / kPlainWaves), dim3(kPlainWaves * 64), 0, s, a);
    return hipGetLastError();
}

}  // namespace paro
