// Quantisers of transformed rows: the weight side of the method, offline (the equivalent transform of Eq. 8 applied to every
// output row of a dense fp16 weight, then the round-to-nearest INT4 quantiser of Eq. 1 with one (scale, zero) per 128
// input channels, Section 2.1), the activation side of the W4A4 extension (App. A.3: Y' = Q(X T^-1) . Q(T W) + b: the
// transformed activations quantised while they are still in the wave's registers), and both with a microscaling FP4
// quantiser (MXFP4 of the OCP Microscaling Formats specification, the 4-bit type the matrix cores of this chip take).
//
//   weight       w'_n = R_K ... R_1 . diag(1 / ch_scale) . w_n      (scale_order 0; the plan's multipliers are reciprocated)
//   activations  x'   = R_K ... R_1 . diag(ch_scale) . x
//   INT4         s = (max - min) / 15,  z = -round(min / s),  q = clamp(round(v / s) + z, 0, 15) per row and group; the
//                decisions in fp32 with the fp16-rounded scale that is stored (IEEE division, round-half-to-even), scale
//                floor 2^-14, zero point clamped to 0..15.  The paper names no activation quantiser of its own: the
//                same decisions per token and group.
//   MXFP4        32 consecutive channels share 2^e, e = floor(log2(max |v|)) - 2 (>= -127), stored as e + 127; every value
//                becomes the E2M1 code of v / 2^e, to nearest, ties to the even code, saturated at 6.  A block that is
//                NaN throughout has e = 126 and codes +-6: what is multiplied with it overflows.
// so that  sum_c (q - z) s . x'_c  ~  w_n . x  for the activations x' that paro_rotate_scale produces (Eq. 2).
//
// One wavefront owns a channel group and a run of rows, four rows at a time (few rows: one each, kQuantFewRows), with the
// lane plan and layer loop of the activation kernel (rotate_lane.h): the plan (7.4 KB at K = 8, 29 times a row's group) is
// read once per run, the four rows' chains of multiply-adds and permutes are independent, and rows go through a
// wave-private LDS area as [channel][4 rows].  No single unit bounds it: the vector pipes (INT4 weights: some 88
// instructions per (row, group), 38 of them rotation; taking 13 of 101 out gave 4 % with a rotation and 13 % without), the
// permutes' LDS time, and 6 waves per SIMD (77 registers) to overlap the two -
//   - INT4: minimum and maximum of the four rows are reduced together, each swap of half waves merging two rows, so that
//     every 16 lanes end up with one row's and the scale, its reciprocal and the zero point are computed once for all
//     four; v / s is the correctly rounded quotient from the correctly rounded reciprocal and one residual (Markstein's
//     theorem), which holds for finite v and s: rows with an infinite scale, and rows of infinities (whose range is NaN
//     and whose scale is the floor), divide; range / 15 and the zero point the same way; codes leave past the L2;
//   - MXFP4: the rotated values are read back in channel order, 8 per lane, so that a block's maximum is two steps within
//     four lanes and the codes are four instructions of the FP4 converter (equal to the thresholds of the format on every
//     tie and its neighbours, probed over all exponents; the tests pin those that fp16 inputs and scales reach).
// Measured over back-to-back calls (before: one row of INT4 weights per wave, plan re-read for each; MXFP4 one row at a
// time, 14 instructions of thresholds per value): INT4 weight 28672 x 4096 414 -> 146 us (137 with reciprocals in place of the
// three divisions, bytes picked by permutes and the factor of one left out; without a rotation 97 -> 84, large
// ones now in quantize_weight.hip), MXFP4 activations 2048 x 4096
// 21.0 -> 12.2, 2048 x 14336 55.8 -> 35.2 us (11.8 and 35.5 with codes past the L2, as INT4 codes leave it: weights 1 to 7 % faster
// alone, a GEMM behind as fast over 36 shapes), INT4 activations 24.7 -> 14.3 and 78.3 -> 39.6 us (now 13.9 on the former); 1 x 4096
// MXFP4 3.0 -> 2.6, INT4 2.9 -> 2.8; the same bits throughout.
#include "paro_internal.h"
#include "quantize_common.h"
#include "rotate_lane.h"
#include <type_traits>

namespace paro {

constexpr int kQuantWaves = 4;       // waves per block
constexpr int kQuantRows = 4;        // rows side by side
constexpr int kQuantBatches = 8;     // most batches of kQuantRows rows per wave (unrolled, see rotate.hip)
constexpr int kQuantPad = kGroup + 4;
// (row, group) pairs below which rows go one to a wave.  Replayed graph, one row / four rows side by side, us: MXFP4 activations
// 1 x 4096 2.62 / 3.0, 112 x 4096 (3584 pairs) 3.63 / 3.5; INT4 activations 1 x 4096 2.80 / 3.47, 78 x 896 3.0 / 3.82.
constexpr int64_t kQuantFewRows = 3072;

enum QuantKind { kW4Weight, kA4Act, kMxAct, kMxWeight };

struct QuantArgs {
    const uint32_t *plan;
    const _Float16 *X; int64_t ldx;
    int T, C, rows_per_wave;         // rows; rows_per_wave: a multiple of the kernel's U
    uint32_t *codes;                 // [T][C/8]
    _Float16 *scales;                // kW4Weight: [C/128][T], kA4Act: [T][C/128]
    uint16_t *qzeros;                // kW4Weight: [C/128][T/8] words, as halves
    uint8_t *bytes;                  // kA4Act: zero points [T][C/128]; MXFP4: scales [T][C/32]
};

template <int N, class F, int I = 0>
__device__ __forceinline__ void quant_while(F &&f)
{
    if constexpr (I < N) {
        if (f(std::integral_constant<int, I>{})) quant_while<N, F, I + 1>(static_cast<F &&>(f));
    }
}

// Maximum over the wave of four values per lane; lanes 0-15 return that of v[0], 16-31 of v[2], 32-47 of v[1], 48-63 of v[3].
__device__ __forceinline__ float wave_max4(const float (&v)[4])
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    auto merge32 = [](float a, float b) {
        const u32x2 t = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
    };
    const u32x2 t = __builtin_amdgcn_permlane16_swap(__float_as_uint(merge32(v[0], v[1])), __float_as_uint(merge32(v[2], v[3])), false, false);
    float m = fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
    m = fmaxf(m, dpp<kQuadXor1>(m));
    m = fmaxf(m, dpp<kQuadXor2>(m));
    m = fmaxf(m, dpp<kHalfMirror>(m));
    return fmaxf(m, dpp<kMirror>(m));
}
constexpr int kRowLane[4] = {0, 32, 16, 48};         // a lane that holds row u's maximum
__device__ __forceinline__ int row_of_lane(int lane) { return ((lane >> 5) & 1) | ((lane >> 3) & 2); }
__device__ __forceinline__ float from_lane(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

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

// K < 0: no transform (rows quantised as they are).  U: rows side by side, kQuantRows, or one where the rows do not fill the
// chip: four rows then only lengthen the chain of one wave.
template <int K, int KIND, int U>
__global__ __launch_bounds__(kQuantWaves * 64) void quantize_kernel(QuantArgs a)
{
    constexpr bool WSIDE = KIND == kW4Weight || KIND == kMxWeight, INT4 = KIND == kW4Weight || KIND == kA4Act;
    static_assert(U == kQuantRows || (U == 1 && KIND != kW4Weight && K >= 0), "");
    __shared__ __attribute__((aligned(16))) uint32_t s_stage[kQuantWaves][kGroup * U / 2];               // [channel][U rows] fp16
    __shared__ __attribute__((aligned(16))) uint32_t s_out[kQuantWaves][INT4 ? kGroup : U * kQuantPad];  // codes [channel][4 rows], or values [U rows][channel]
    const int g = blockIdx.x, G = a.C / kGroup;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t0 = ((int64_t)blockIdx.y * kQuantWaves + wave) * a.rows_per_wave;
    if (t0 >= a.T) return;
    const int n_rows = (int)(a.T - t0 < a.rows_per_wave ? a.T - t0 : a.rows_per_wave);

    // the wave's rows from one uniform address each (row strides of weights are not limited); rows beyond the run repeat
    // its last one and are not written
    const _Float16 *x0 = a.X + t0 * a.ldx + (size_t)g * kGroup;
    auto load_row = [&](int r) { return *((const uint32_t *)(x0 + (int64_t)(r < n_rows ? r : n_rows - 1) * a.ldx) + lane); };
    uint32_t cur[U], nxt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = load_row(u);

    LanePlan<(K > 0 ? K : 0)> P;
    float ia = 1.f, ib = 1.f, oa = 1.f, ob = 1.f;
    int ch_a = 2 * lane, ch_b = 2 * lane + 1;
    if constexpr (K >= 0) {
        load_lane_plan<K>(a.plan + (size_t)g * plan_group_dwords(K), lane, P);
        // the plan carries the activation-side multipliers; the weights take their reciprocals
        ia = WSIDE ? 1.0f / P.sia : P.sia; ib = WSIDE ? 1.0f / P.sib : P.sib;
        oa = WSIDE ? 1.0f / P.soa : P.soa; ob = WSIDE ? 1.0f / P.sob : P.sob;
        ch_a = P.out_a; ch_b = P.out_b;
    }
    typedef _Float16 half4v __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
    char *sp = (char *)s_stage[wave];
    auto lo_pair = [](uint32_t x, uint32_t y) { return (x & 0xffffu) | (y << 16); };
    auto hi_pair = [](uint32_t x, uint32_t y) { return (x >> 16) | (y & 0xffff0000u); };
    const int orow = lane >> 4, oword = lane & 15;       // the row of a batch and its 8 channels this lane writes out
    const uint32_t pick_row = 0x0400u + 0x0101u * orow;  // byte orow of two dwords
    bool scales_out = false;                             // multiplying by one is left out

    quant_while<U == 1 ? 1 : kQuantBatches>([&](auto I) {
        constexpr int t = I * U;
        if (t >= n_rows) return false;
        if constexpr (U > 1)
#pragma unroll
            for (int u = 0; u < U; ++u) nxt[u] = load_row(t + U + u);
        float va[U], vb[U];
        if constexpr (K >= 0 && U == 1) {
            typedef uint32_t __attribute__((may_alias)) u32_halves;
            *(u32_halves *)(sp + lane * 4) = cur[0];
            __builtin_amdgcn_wave_barrier();
            va[0] = (float)*(const _Float16 *)(sp + P.in_a * 2) * ia;
            vb[0] = (float)*(const _Float16 *)(sp + P.in_b * 2) * ib;
            quant_rotate<K, U>(P, va, vb);
            va[0] *= oa; vb[0] *= ob;
        } else if constexpr (K >= 0) {
            const u32x4v in = {lo_pair(cur[0], cur[1]), lo_pair(cur[2], cur[3]), hi_pair(cur[0], cur[1]), hi_pair(cur[2], cur[3])};
            *(u32x4v *)(sp + lane * 16) = in;
            __builtin_amdgcn_wave_barrier();
            const half4v ha = *(const half4v *)(sp + P.in_a * 8), hb = *(const half4v *)(sp + P.in_b * 8);
#pragma unroll
            for (int u = 0; u < U; ++u) { va[u] = (float)ha[u] * ia; vb[u] = (float)hb[u] * ib; }
            quant_rotate<K, U>(P, va, vb);
            // (asked here and not above, where it would hold up the first rows' requests: 0.1 to 0.2 us of a launch of few rows)
            if constexpr (t == 0) scales_out = __any(oa != 1.f || ob != 1.f);
            if (scales_out)
#pragma unroll
                for (int u = 0; u < U; ++u) { va[u] *= oa; vb[u] *= ob; }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                union { uint32_t u; _Float16 h[2]; } c; c.u = cur[u];
                va[u] = (float)c.h[0]; vb[u] = (float)c.h[1];
            }
        }
        const int64_t row = t0 + t + orow;               // the row this lane writes out
        const bool live = orow < U && t + orow < n_rows;
        if constexpr (INT4) {
            float mx[U], nmn[U], mxv, mnv;
#pragma unroll
            for (int u = 0; u < U; ++u) { mx[u] = fmaxf(va[u], vb[u]); nmn[u] = fmaxf(-va[u], -vb[u]); }
            if constexpr (U == 1) {
                const float m = wave_max4({mx[0], nmn[0], mx[0], nmn[0]});
                mxv = from_lane(m, kRowLane[0]); mnv = -from_lane(m, kRowLane[1]);
            } else {
                mxv = wave_max4(mx); mnv = -wave_max4(nmn);
            }
            const float range = mxv - mnv;
            // correctly rounded quotients by reciprocal and residual, as for the codes: range / 15 where the range is finite
            constexpr float kR15 = 1.0f / 15.0f;
            const float s15 = range * kR15;
            float s32 = range < __builtin_inff() ? fmaf(fmaf(-15.0f, s15, range), kR15, s15) : range;
            if (!(s32 >= 6.103515625e-05f)) s32 = 6.103515625e-05f;
            const _Float16 s16 = (_Float16)s32;
            const float s = (float)s16, rs = range < __builtin_inff() && s < __builtin_inff() ? quant_rcp(s) : 0.f;  // 0: infinite scale, or a group of infinities
            float zq = mnv * rs;
            zq = fmaf(fmaf(-s, zq, mnv), rs, zq);
            if (__any(!(rs > 0.f))) zq = rs > 0.f ? zq : mnv / s;
            const float zf = __builtin_amdgcn_fmed3f(-rintf(zq), 0.0f, 15.0f);
            uint32_t ca = 0, cb = 0, zhalf = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float su = from_lane(s, kRowLane[u]), ru = from_lane(rs, kRowLane[u]), zu = from_lane(zf, kRowLane[u]);
                float qa, qb;
                if (ru > 0.f) {                          // (uniform)
                    const float a0 = va[u] * ru, b0 = vb[u] * ru;
                    qa = fmaf(fmaf(-su, a0, va[u]), ru, a0);
                    qb = fmaf(fmaf(-su, b0, vb[u]), ru, b0);
                } else {
                    qa = va[u] / su; qb = vb[u] / su;
                }
                ca = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(rintf(qa) + zu, 0.0f, 15.0f), u, ca);   // NaN: 0
                cb = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(rintf(qb) + zu, 0.0f, 15.0f), u, cb);
                if constexpr (KIND == kW4Weight) zhalf |= (uint32_t)zu << (4 * u);
            }
            s_out[wave][ch_a] = ca;
            s_out[wave][ch_b] = cb;
            __builtin_amdgcn_wave_barrier();
            uint32_t d[8];
            *(u32x4v *)&d[0] = *(const u32x4v *)&s_out[wave][oword * 8];
            *(u32x4v *)&d[4] = *(const u32x4v *)&s_out[wave][oword * 8 + 4];
            // byte orow of every dword, two to a half, four to a dword, then the nibbles together
            auto pick = [&](int k) { return __builtin_amdgcn_perm(d[k + 1], d[k], pick_row); };
            const uint32_t c03 = __builtin_amdgcn_perm(pick(2), pick(0), 0x05040100u), c47 = __builtin_amdgcn_perm(pick(6), pick(4), 0x05040100u);
            const uint32_t word = __builtin_amdgcn_perm(c47 | (c47 >> 4), c03 | (c03 >> 4), 0x06040200u);
            if (live) __builtin_nontemporal_store(word, &a.codes[(size_t)row * (a.C / 8) + (size_t)g * (kGroup / 8) + oword]);
            const int64_t prow = t0 + t + row_of_lane(lane);         // the row whose scale this lane holds
            if (oword == 0 && row_of_lane(lane) < U && t + row_of_lane(lane) < n_rows) {
                if constexpr (KIND == kW4Weight) a.scales[(size_t)g * a.T + prow] = s16;
                else { a.scales[(size_t)prow * G + g] = s16; a.bytes[(size_t)prow * G + g] = (uint8_t)zf; }
            }
            if constexpr (KIND == kW4Weight)             // T is a multiple of 8, t0 + t of 4: half a word
                if (lane == 0) a.qzeros[(size_t)g * (a.T / 4) + (t0 + t) / 4] = (uint16_t)zhalf;
        } else {
            float v[8];
            if constexpr (K >= 0) {
                float *so = (float *)s_out[wave];
#pragma unroll
                for (int u = 0; u < U; ++u) { so[u * kQuantPad + ch_a] = va[u]; so[u * kQuantPad + ch_b] = vb[u]; }
                __builtin_amdgcn_wave_barrier();
                const float *row_v = so + (U == 1 ? 0 : orow) * kQuantPad + oword * 8;
                *(float4 *)&v[0] = *(const float4 *)row_v;
                *(float4 *)&v[4] = *(const float4 *)(row_v + 4);
            } else {
                uint32_t *so = s_out[wave];
#pragma unroll
                for (int u = 0; u < U; ++u) so[u * kQuantPad + lane] = cur[u];
                __builtin_amdgcn_wave_barrier();
                union { u32x4v u; _Float16 h[8]; } c; c.u = *(const u32x4v *)(so + orow * kQuantPad + oword * 4);
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = (float)c.h[k];
            }
            float amax = fabsf(v[0]);                    // NaN where all 32 are
#pragma unroll
            for (int k = 1; k < 8; ++k) amax = fmaxf(amax, fabsf(v[k]));
            amax = fmaxf(amax, dpp<kQuadXor1>(amax));
            amax = fmaxf(amax, dpp<kQuadXor2>(amax));
            int e = (int)(__float_as_uint(amax) >> 23) - 127 - 2;
            if (e < -127) e = -127;
            const float sc = __uint_as_float(e > -127 ? (uint32_t)(e + 127) << 23 : 0x00400000u);       // 2^e
            uint32_t word = 0;
            word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, v[0], v[1], sc, 0);
            word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, v[2], v[3], sc, 1);
            word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, v[4], v[5], sc, 2);
            word = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(word, v[6], v[7], sc, 3);
            if (live) {
                __builtin_nontemporal_store(word, &a.codes[(size_t)row * (a.C / 8) + (size_t)g * (kGroup / 8) + oword]);
                if ((lane & 3) == 0) a.bytes[(size_t)row * (a.C / 32) + (size_t)g * (kGroup / 32) + (oword >> 2)] = (uint8_t)(e + 127);
            }
        }
        __builtin_amdgcn_wave_barrier();
        if constexpr (U > 1)
#pragma unroll
            for (int u = 0; u < U; ++u) cur[u] = nxt[u];
        return true;
    });
}

template <int K, int KIND>
static hipError_t launch_quant_k(QuantArgs &a, hipStream_t s)
{
    // runs of up to 32 rows per wave, shorter while that leaves fewer than ~4096 waves
    const int G = a.C / kGroup;
    int rpw = kQuantBatches * kQuantRows;
    while (rpw > kQuantRows && (int64_t)G * ((a.T + rpw - 1) / rpw) < 4096) rpw >>= 1;
    constexpr bool ONE = KIND != kW4Weight && K >= 0;
    if (ONE && (int64_t)G * a.T < kQuantFewRows) rpw = 1;
    a.rows_per_wave = rpw;
    const int waves_t = (a.T + rpw - 1) / rpw;
    const dim3 grid(G, (waves_t + kQuantWaves - 1) / kQuantWaves), block(kQuantWaves * 64);
    if constexpr (ONE)
        if (rpw == 1) {
            hipLaunchKernelGGL((quantize_kernel<K, KIND, 1>), grid, block, 0, s, a);
            return hipGetLastError();
        }
    hipLaunchKernelGGL((quantize_kernel<K, KIND, kQuantRows>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <int KIND>
static hipError_t launch_quant(const paro_rotation *rot, QuantArgs &a, hipStream_t s)
{
    if (!rot) {
        if constexpr (KIND == kW4Weight || KIND == kMxWeight) return launch_quant_k<-1, KIND>(a, s);
        return hipErrorInvalidValue;
    }
    a.plan = (const uint32_t *)rot->plan;
    switch (rot->n_layers) {
    case 0: return launch_quant_k<0, KIND>(a, s);
    case 1: return launch_quant_k<1, KIND>(a, s);
    case 2: return launch_quant_k<2, KIND>(a, s);
    case 3: return launch_quant_k<3, KIND>(a, s);
    case 4: return launch_quant_k<4, KIND>(a, s);
    case 5: return launch_quant_k<5, KIND>(a, s);
    case 6: return launch_quant_k<6, KIND>(a, s);
    case 7: return launch_quant_k<7, KIND>(a, s);
    default: return launch_quant_k<8, KIND>(a, s);
    }
}

hipError_t launch_quantize(const paro_rotation *rot, const paro_half_t *W, int64_t ldw, int N, int C, uint32_t *qweight,
                           paro_half_t *scales, uint32_t *qzeros, hipStream_t s)
{
    if (!rot && quantize_plain_pays(N, C)) return launch_quantize_plain(W, ldw, N, C, qweight, scales, qzeros, s);
    QuantArgs a{nullptr, (const _Float16 *)W, ldw, N, C, 0, qweight, (_Float16 *)scales, (uint16_t *)qzeros, nullptr};
    return launch_quant<kW4Weight>(rot, a, s);
}

hipError_t launch_quantize_act(const paro_rotation &rot, const paro_half_t *X, int64_t ldx, int T, uint32_t *codes,
                               paro_half_t *scales, uint8_t *zeros, hipStream_t s)
{
    QuantArgs a{nullptr, (const _Float16 *)X, ldx, T, rot.c_in, 0, codes, (_Float16 *)scales, nullptr, zeros};
    return launch_quant<kA4Act>(&rot, a, s);
}

hipError_t launch_quantize_act_mxfp4(const paro_rotation &rot, const paro_half_t *X, int64_t ldx, int T, uint32_t *codes,
                                     uint8_t *scales, hipStream_t s)
{
    QuantArgs a{nullptr, (const _Float16 *)X, ldx, T, rot.c_in, 0, codes, nullptr, nullptr, scales};
    return launch_quant<kMxAct>(&rot, a, s);
}

// rows of a dense weight [N][ldw]; rot == nullptr: no transform
hipError_t launch_quantize_weight_mxfp4(const paro_rotation *rot, const paro_half_t *W, int64_t ldw, int N, int C,
                                        uint32_t *codes, uint8_t *scales, hipStream_t s)
{
    QuantArgs a{nullptr, (const _Float16 *)W, ldw, N, C, 0, codes, nullptr, nullptr, scales};
    return launch_quant<kMxWeight>(rot, a, s);
}

}  // namespace paro
