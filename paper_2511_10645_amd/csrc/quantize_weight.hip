// Weight side, offline, for large weights: the equivalent transform of Eq. 8 applied to every output row of a dense fp16
// weight, then the INT4 quantiser of Eq. 1 or the MXFP4 conversion (formats and decisions: quantize.hip).
//
// One transform serves all rows of a weight, so the K layers of a channel group are multiplied out once per block, into the
// group's 128 x 128 matrix R_K ... R_1 diag(1 / ch_scale) (scale_order 1: the factors on the left), and the rows go through
// the matrix cores.  Pair by pair (quantize.hip) the rotation alone is 38 vector instructions and 7 permutes per (row, group),
// and two values per lane need wave reductions for the quantiser: 88 instructions, 131 us of issue at 28672 x 4096, of the
// 139 us that it takes; here 18 instructions and 64 cycles of matrix instructions, 88 us, 12 of them until the matrix stands.
//
// The matrix is formed by rotating the 128 unit vectors with the lane plan in fp64, times a power of two that brings the
// largest factor to 2^13, and kept as the sum of two fp16 numbers (22 bits, at least that many for every column down to 2^-10
// of the largest): a product with an fp16 weight is exact, the sums are fp32, the low parts of all channels first.  The
// transformed values are off from 64 bits by 1.10e-7 of a group's root mean square (rms; pair by pair 1.11e-7; with the vectors
// rotated in fp32 1.35e-7, and low and high parts in turn 1.51e-7).
//
// A block is one group and a run of rows, 8 waves; a wave takes 32 rows at a time, whose results stand as 64 of the 128
// channels in lane r and the others in lane r + 32 (v_mfma_f32_32x32x16_f16 with the matrix as the left operand): a row's
// extrema are one exchange between the two, its scale and zero point are computed once for the 32 rows, and eight codes of
// consecutive channels meet by exchanging half words.  Rows are read 256 bytes at a time, two tiles ahead (one ahead: 82 us
// where two take 74).
//
// A row with an infinity or a NaN in it (0 x inf) and every row of a group whose factors are not finite or differ by more
// than 2^10 are transformed pair by pair instead, four at a time: no result of a row depends on other rows.
//
// Without a transform the same division of rows among lanes, without a matrix.
#include "paro_internal.h"
#include "quantize_common.h"
#include <type_traits>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x4 u32x4_any __attribute__((aligned(4)));

struct WeightQuantArgs {
    const uint32_t *plan;
    const _Float16 *W; int64_t ldw;
    int N, C, n_layers, tiles_per_block;     // a tile: 32 rows
    uint32_t *codes;                         // [N][C/8]
    _Float16 *scales;                        // INT4: [C/128][N]
    uint32_t *qzeros;                        // INT4: [C/128][N/8]
    uint8_t *bytes;                          // MXFP4: scales [N][C/32]
};

constexpr int kTileRows = 32;
constexpr int kMatrixBytes = kGroup * kGroup * 2;       // one of the two parts
constexpr int kStageBytes = kTileRows * kGroup * 2;     // a wave's rows
constexpr int kPairBytes = 4 * kGroup * 4;              // a wave's rows on the way back from the pairwise transform

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

__device__ __forceinline__ double from_lane64(int addr, double v)
{
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(addr, __double2hiint(v)), __builtin_amdgcn_ds_bpermute(addr, __double2loint(v)));
}

// The lane plan with layers beyond n_layers as identities, and the multipliers of the weight side.
__device__ __forceinline__ void load_weight_plan(const uint32_t *gplan, int n_layers, int lane, LanePlan<kMaxLayers> &P)
{
    const uint32_t io = gplan[lane];
    P.in_a = io & 0xff; P.in_b = (io >> 8) & 0xff; P.out_a = (io >> 16) & 0xff; P.out_b = io >> 24;
    P.sia = 1.0f / __uint_as_float(gplan[1 * 64 + lane]); P.sib = 1.0f / __uint_as_float(gplan[2 * 64 + lane]);
    P.soa = 1.0f / __uint_as_float(gplan[3 * 64 + lane]); P.sob = 1.0f / __uint_as_float(gplan[4 * 64 + lane]);
    float c[kMaxLayers], sn[kMaxLayers];
    uint32_t meta[kMaxLayers];
#pragma unroll
    for (int l = 0; l < kMaxLayers; ++l) {           // (all rows requested before the first is used)
        const uint32_t *row = gplan + (size_t)(kPlanHeadRows + kPlanRowsPerLayer * (l < n_layers ? l : 0)) * 64;
        c[l] = __uint_as_float(row[lane]); sn[l] = __uint_as_float(row[64 + lane]); meta[l] = row[128 + lane];
    }
#pragma unroll
    for (int l = 0; l < kMaxLayers; ++l) {
        const bool real = l < n_layers;
        const uint32_t m = real ? meta[l] : (uint32_t)lane * 4 | kMetaAIsI | kMetaKeepI;
        expand_coeffs(real ? c[l] : 1.f, real ? sn[l] : 0.f, m, P.m00[l], P.m01[l], P.m10[l], P.m11[l]);
        P.src[l] = (int)(m & 0xff);
    }
}

template <bool MX, bool ROT, int WAVES>
__global__ __launch_bounds__(WAVES * 64, ROT ? 2 : 4) void quantize_weight_kernel(WeightQuantArgs a)
{
    static_assert(ROT || !MX, "");
    extern __shared__ __attribute__((aligned(16))) char s_mem[];       // ROT: matrix, then per wave rows and pairwise rows
    const int g = blockIdx.x;
    const int lane = threadIdx.x & 63, half = lane >> 5, trow = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char *stage = s_mem + (ROT ? 2 * kMatrixBytes : 0) + wave * kStageBytes;
    const int tiles = (a.N + kTileRows - 1) / kTileRows;
    const int tile_end = min(tiles, (int)(blockIdx.y + 1) * a.tiles_per_block);
    int tile = blockIdx.y * a.tiles_per_block + wave;

    // rows: 16 bytes of row 4 i + lane / 16, two tiles ahead; rows beyond the block's last repeat it and are not written
    const _Float16 *w0 = a.W + (size_t)g * kGroup + (lane & 15) * 8;
    const int last = min(a.N, tile_end * kTileRows) - 1;
    u32x4 next[2][8];
    auto load_rows = [&](int t, auto SET) {
        wq_for<8>([&](auto I) {
            const int row = min(t * kTileRows + 4 * I + (lane >> 4), last);
            next[SET][I] = *(const u32x4_any *)(w0 + (int64_t)row * a.ldw);
        });
    };
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;

    float up = 1.f, unscale = 1.f;           // INT4: v below is the value times up
    bool pairwise = false;                   // no row of this group goes through the matrix
    const uint32_t *gplan = ROT ? a.plan + (size_t)g * plan_group_dwords(a.n_layers) : nullptr;
    if constexpr (ROT) {
        LanePlan<kMaxLayers> P;
        load_weight_plan(gplan, a.n_layers, lane, P);
        load_rows(tile, even);
        load_rows(tile + WAVES, odd);
        // the largest factor of the group to 2^13 .. 2^14; factors of zero (a multiplier that is infinite) count as none
        float hi = 0.f, lo = 0.f;            // of exponents: largest, and largest of the negated
        bool finite = true;
        auto factor = [&](float s) {
            const int e = (int)(__float_as_uint(s) >> 23) & 0xff;
            finite = finite && e != 0xff;
            if (s != 0.f) { hi = fmaxf(hi, (float)e); lo = fmaxf(lo, (float)(256 - e)); }
        };
        factor(P.sia * P.soa); factor(P.sib * P.sob);      // one side's are all ones
        auto wave_max = [&](float v) {
            v = fmaxf(v, dpp<kQuadXor1>(v)); v = fmaxf(v, dpp<kQuadXor2>(v));
            v = fmaxf(v, dpp<kHalfMirror>(v)); v = fmaxf(v, dpp<kMirror>(v));
            v = fmaxf(v, __shfl_xor(v, 16));
            return max_halves(v);
        };
        hi = wave_max(hi); lo = 256.f - wave_max(lo);
        const int e_hi = __builtin_amdgcn_readfirstlane((int)hi), e_lo = __builtin_amdgcn_readfirstlane((int)lo);
        pairwise = __any(!finite) || e_hi - e_lo > 10 || e_hi < 40 || e_hi > 200;
        up = pairwise ? 1.f : __uint_as_float((uint32_t)(127 + 13 + 127 - e_hi) << 23);
        unscale = pairwise ? 1.f : __uint_as_float((uint32_t)(e_hi - 13) << 23);
        // 128 / WAVES unit vectors, four at a time
        char *m_hi = s_mem, *m_lo = s_mem + kMatrixBytes;
        for (int j0 = wave * (kGroup / WAVES); j0 < (wave + 1) * (kGroup / WAVES); j0 += 4) {
            double va[4], vb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                va[u] = P.in_a == j0 + u ? P.sia * up : 0.f;
                vb[u] = P.in_b == j0 + u ? P.sib * up : 0.f;
            }
#pragma unroll
            for (int l = 0; l < kMaxLayers; ++l)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double na = fma((double)P.m00[l], va[u], P.m01[l] * vb[u]), nb = fma((double)P.m10[l], va[u], P.m11[l] * vb[u]);
                    va[u] = na;
                    vb[u] = l + 1 < kMaxLayers ? from_lane64(P.src[l], nb) : nb;
                }
            auto put = [&](int ch, const double (&v)[4], float s) {
                half4 h, l;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double m = v[u] * s;
                    h[u] = (_Float16)(float)m;
                    l[u] = (_Float16)(float)(m - (double)h[u]);
                }
                // operand order: [32 channels out][16 channels in][lane: channel out % 32, in / 8 % 2][8 channels in]
                const int off = ((((ch >> 5) * 8 + (j0 >> 4)) * 64 + (ch & 31) + 32 * ((j0 >> 3) & 1)) << 4) + (j0 & 7) * 2;
                *(half4 *)(m_hi + off) = h;
                *(half4 *)(m_lo + off) = l;
            };
            put(P.out_a, va, P.soa);
            put(P.out_b, vb, P.sob);
        }
        __syncthreads();
    } else {
        load_rows(tile, even);               // one tile per wave
    }

    // The next rows take the place of the present ones ahead of the stores: at the head of the loop, their wait would be one for
    // the stores as well.
    auto stage_rows = [&](auto SET) {
        wq_for<8>([&](auto I) {
            const int r = 4 * I + (lane >> 4);
            *(u32x4 *)(stage + r * 256 + (((lane & 15) ^ (r & 15)) << 4)) = next[SET][I];
        });
        __builtin_amdgcn_wave_barrier();
    };
    if (tile >= tile_end) return;
    stage_rows(even);
    auto one_tile = [&](auto SET) {
        const int row = tile * kTileRows + trow;         // the row this lane has half of
        const bool live = row < a.N;
        // ROT: channels 16 k + 8 half .. + 7, the operand of step k; else channels 64 half + 8 k .. + 7
        half8 x[8];
        wq_for<8>([&](auto K) { x[K] = *(const half8 *)(stage + trow * 256 + (((ROT ? 2 * K + half : 8 * half + K) ^ (trow & 15)) << 4)); });
        if constexpr (ROT) load_rows(tile + 2 * WAVES, SET);

        // v(i): ROT: channels 32 (i / 16) + 8 (i / 4 % 4) + 4 half + i % 4, else 64 half + i
        float16v acc[4];
        if constexpr (ROT) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
            // the low parts of all channels, then the high ones (fewer roundings of large sums): steps of 16 channels in, 4 x 32
            // channels out; operands are requested kAhead steps ahead
            constexpr int kAhead = 4;
            half8 m[kAhead];
            auto load_m = [&](auto I) { m[I % kAhead] = *(const half8 *)(s_mem + (1 - I / 32) * kMatrixBytes + ((I % 4 * 8 + I / 4 % 8) * 64 + lane) * 16); };
            wq_for<kAhead>([&](auto I) { load_m(I); });
            wq_for<64>([&](auto I) {
                acc[I % 4] = __builtin_amdgcn_mfma_f32_32x32x16_f16(m[I % kAhead], x[I / 4 % 8], acc[I % 4], 0, 0, 0);
                if constexpr (I + kAhead < 64) load_m(std::integral_constant<int, I + kAhead>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (MX)
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[t][i] *= unscale;
            // every output of a row with an infinity or a NaN is one
            const uint64_t bad = __ballot(live && (pairwise || !(fabsf(acc[0][0]) < __builtin_inff())));
            if (bad) {
                LanePlan<kMaxLayers> P;
                load_weight_plan(gplan, a.n_layers, lane, P);
                float *back = (float *)(s_mem + 2 * kMatrixBytes + WAVES * kStageBytes + wave * kPairBytes);
#pragma unroll 1
                for (int r0 = 0; r0 < kTileRows; r0 += 4) {
                    if (!((bad >> r0) & 15)) continue;
                    float va[4], vb[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const char *rp = stage + (r0 + u) * 256;
                        auto at = [&](int ch) { return (float)*(const _Float16 *)(rp + (((ch >> 3) ^ ((r0 + u) & 15)) << 4) + (ch & 7) * 2); };
                        va[u] = at(P.in_a) * P.sia;
                        vb[u] = at(P.in_b) * P.sib;
                    }
                    quant_rotate<kMaxLayers, 4>(P, va, vb);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        back[u * kGroup + P.out_a] = va[u] * P.soa * (MX ? 1.f : up);
                        back[u * kGroup + P.out_b] = vb[u] * P.sob * (MX ? 1.f : up);
                    }
                    __builtin_amdgcn_wave_barrier();
                    if ((trow & ~3) == r0 && ((bad >> trow) & 1)) {
#pragma unroll
                        for (int t = 0; t < 4; ++t)
#pragma unroll
                            for (int i = 0; i < 16; ++i) acc[t][i] = back[(trow & 3) * kGroup + 32 * t + 8 * (i / 4) + 4 * half + i % 4];
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        auto v = [&](int i) -> float { if constexpr (ROT) return acc[i / 16][i % 16]; else return (float)x[i / 8][i % 8]; };
        // Words of 8 codes: ROT: 4 half-words per tile of 32 channels, exchanged so that lane r has the words of channels 0..63
        // and lane r + 32 the others, as without a transform.
        uint32_t words[8];
        auto join = [&](int k, uint32_t low, uint32_t high) {      // half-words of word k of tiles t and t + 2
            const u32x2 t = __builtin_amdgcn_permlane32_swap(low, high, false, false);
            words[k] = __builtin_amdgcn_perm(t[1], t[0], 0x05040100u);
        };
        if constexpr (!MX) {
            float mxv, mnv;
            if constexpr (ROT) {
                mxv = mnv = v(0);
#pragma unroll
                for (int i = 1; i < 64; ++i) { mxv = fmaxf(mxv, v(i)); mnv = fminf(mnv, v(i)); }
            } else {
                half2v hx = {x[0][0], x[0][1]}, hn = hx;
#pragma unroll
                for (int i = 2; i < 64; i += 2) {
                    const half2v h = {x[i / 8][i % 8], x[i / 8][i % 8 + 1]};
                    hx = __builtin_elementwise_max(hx, h); hn = __builtin_elementwise_min(hn, h);
                }
                mxv = (float)__builtin_elementwise_max(hx[0], hx[1]); mnv = (float)__builtin_elementwise_min(hn[0], hn[1]);
            }
            mxv = max_halves(mxv) * unscale; mnv = -max_halves(-mnv) * unscale;
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
            const float lo = -zf, hi = 15.f - zf, s_up = s * up, by_up = by * unscale;
            const uint32_t base = (0x4B400000u - (uint32_t)zf) * 0x1111u;
            uint32_t c4[16];
            auto code4 = [&](auto K, auto quotient) {
                uint32_t c = 0;
                wq_for<4>([&](auto U) {
                    const float q = __builtin_amdgcn_fmed3f(quotient(v(4 * K + U)), lo, hi) + 12582912.f;
                    c = U == 0 ? __float_as_uint(q) - base : (__float_as_uint(q) << (4 * U)) + c;
                    asm("" : "+v"(c));                   // (or the sums are regrouped into separate shifts)
                });
                c4[K] = c;
                if constexpr (K % 2) __builtin_amdgcn_sched_barrier(0);          // (or all 64 values are live at once)
            };
            const bool all_plain = __all(plain);
            wq_for<ROT ? 1 : 8>([&](auto PART) {         // (in parts: what the two branches share would be live for all of them)
                constexpr int per = ROT ? 16 : 2;
                if (all_plain)
                    wq_for<per>([&](auto K) {
                        code4(std::integral_constant<int, PART * per + K>{},
                              [&](float f) { const float q0 = f * by_up; return fmaf(fmaf(-s_up, q0, f), by_up, q0); });
                    });
                else
                    wq_for<per>([&](auto K) {
                        code4(std::integral_constant<int, PART * per + K>{},
                              [&](float f) { const float q0 = f * by_up, q = fmaf(fmaf(-s_up, q0, f), by_up, q0); return plain ? q : q0; });
                    });
            });
            if constexpr (ROT) wq_for<8>([&](auto K) { join(K, c4[K], c4[8 + K]); });
            else wq_for<8>([&](auto K) { words[K] = __builtin_amdgcn_perm(c4[2 * K + 1], c4[2 * K], 0x05040100u); });
            __builtin_amdgcn_sched_barrier(0);           // the requests for the next rows have until here to return
            if constexpr (ROT) stage_rows(std::integral_constant<int, 1 - SET>{});
            if (half == 0 && live) a.scales[(size_t)g * a.N + row] = s16;
            uint32_t z = (uint32_t)zf << (4 * (lane & 7));       // 8 rows to a word; N is a multiple of 8
            auto other = [&](auto CTRL) { z |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)z, decltype(CTRL)::value, 0xf, 0xf, true); };
            other(std::integral_constant<int, kQuadXor1>{}); other(std::integral_constant<int, kQuadXor2>{});
            other(std::integral_constant<int, kHalfMirror>{});
            if (half == 0 && (lane & 7) == 0 && live) a.qzeros[(size_t)g * (a.N / 8) + row / 8] = z;
        } else {
            // blocks of 32 channels: one per tile, half of each in this lane
            uint32_t sbytes = 0, c4[16];
            wq_for<4>([&](auto B) {
                float amax = fabsf(v(B * 16));                   // NaN where all 32 are
#pragma unroll
                for (int i = 1; i < 16; ++i) amax = fmaxf(amax, fabsf(v(B * 16 + i)));
                amax = max_halves(amax);
                int e = (int)(__float_as_uint(amax) >> 23) - 127 - 2;
                if (e < -127) e = -127;
                const float sc = __uint_as_float(e > -127 ? (uint32_t)(e + 127) << 23 : 0x00400000u);       // 2^e
                sbytes |= (uint32_t)(e + 127) << (8 * B);
                wq_for<4>([&](auto Q) {
                    constexpr int i0 = B * 16 + 4 * Q;
                    uint32_t c = 0;
                    c = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, v(i0), v(i0 + 1), sc, 0);
                    c4[i0 / 4] = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(c, v(i0 + 2), v(i0 + 3), sc, 1);
                });
            });
            wq_for<8>([&](auto K) { join(K, c4[K], c4[8 + K]); });
            __builtin_amdgcn_sched_barrier(0);
            stage_rows(std::integral_constant<int, 1 - SET>{});
            if (live && half == 0) {
                uint8_t *out = a.bytes + (size_t)row * (a.C / 32) + (size_t)g * (kGroup / 32);
                if (((uintptr_t)a.bytes & 3) == 0) *(uint32_t *)out = sbytes;
                else for (int k = 0; k < 4; ++k) out[k] = (uint8_t)(sbytes >> (8 * k));
            }
        }
        if (live) {
            u32x4_any *out = (u32x4_any *)(a.codes + (size_t)row * (a.C / 8) + (size_t)g * (kGroup / 8) + 8 * half);
            const u32x4 c0 = {words[0], words[1], words[2], words[3]}, c1 = {words[4], words[5], words[6], words[7]};
            __builtin_nontemporal_store(c0, out);
            __builtin_nontemporal_store(c1, out + 1);
        }
        tile += WAVES;
    };
    while (true) {
        one_tile(even);
        if (!ROT || tile >= tile_end) break;
        one_tile(odd);
        if (tile >= tile_end) break;
    }
}

template <bool MX, bool ROT, int WAVES>
static hipError_t launch_weight(WeightQuantArgs &a, hipStream_t s)
{
    const int G = a.C / kGroup, tiles = (a.N + kTileRows - 1) / kTileRows;
    constexpr int lds = ROT ? 2 * kMatrixBytes + WAVES * (kStageBytes + kPairBytes) : WAVES * kStageBytes;
    if constexpr (ROT) {
        // One block per compute unit; forming the matrix takes about as long as two rounds of 8 tiles, so the runs of a group
        // are as many as leave the fewest rounds and matrices in a row.
        int best = 1;
        int64_t cost = INT64_MAX;
        const int most = (tiles + WAVES - 1) / WAVES;
        for (int nb = 1; nb <= most && (nb == 1 || (int64_t)G * nb <= 2048); ++nb) {
            const int per = (tiles + nb - 1) / nb;
            const int64_t c = (((int64_t)G * nb + 255) / 256) * (2 + (per + WAVES - 1) / WAVES);
            if (c < cost) { cost = c; best = nb; }
        }
        a.tiles_per_block = (tiles + best - 1) / best;
        static std::atomic<uint64_t> done{0};
        const int dev = once_pending(done);
        if (dev >= 0) {
            hipError_t e = hipFuncSetAttribute((const void *)&quantize_weight_kernel<MX, ROT, WAVES>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            once_done(done, dev);
        }
    } else {
        a.tiles_per_block = WAVES;               // (two tiles per wave are 7 % slower)
    }
    const dim3 grid(G, (tiles + a.tiles_per_block - 1) / a.tiles_per_block);
    hipLaunchKernelGGL((quantize_weight_kernel<MX, ROT, WAVES>), grid, dim3(WAVES * 64), lds, s, a);
    return hipGetLastError();
}

// Back-to-back calls over 400 MB of weights, us, quantize_kernel / this one.  INT4 with a transform: 4096 x 4096 (131072 (row,
// group) pairs) 26.9 / 26.5, 5120 x 5120 42.3 / 37.5, 28672 x 4096 139 / 88, 5120 x 27648 176 / 108; MXFP4 204800 pairs 36.8 / 35.9,
// 28672 x 4096 131 / 91; a launch that forms matrices does not end before 17 us.  INT4 without a transform: 20736 pairs 5.1 / 5.0,
// 37312 7.1 / 6.6, 4096 x 4096 17.3 / 10.0, 28672 x 4096 78.5 / 49.3; MXFP4 without is memory-bound on either (50.5 / 55.4).
bool quantize_tiles_pay(const paro_rotation *rot, bool mx, int N, int C)
{
    const int64_t pairs = (int64_t)N * (C / kGroup);
    if (!rot) return !mx && pairs >= 24576;
    return rot->n_layers > 0 && pairs >= (mx ? 240000 : 160000);
}

hipError_t launch_quantize_tiles(const paro_rotation *rot, bool mx, const paro_half_t *W, int64_t ldw, int N, int C, uint32_t *codes,
                                 paro_half_t *scales, uint32_t *qzeros, uint8_t *bytes, hipStream_t s)
{
    WeightQuantArgs a{nullptr, (const _Float16 *)W, ldw, N, C, 0, 0, codes, (_Float16 *)scales, qzeros, bytes};
    if (!rot) return mx ? hipErrorInvalidValue : launch_weight<false, false, 4>(a, s);
    a.plan = (const uint32_t *)rot->plan;
    a.n_layers = rot->n_layers;
    return mx ? launch_weight<true, true, 8>(a, s) : launch_weight<false, true, 8>(a, s);
}

}  // namespace paro
