// W4A16 linear on weights in the interchange layout, up to 32 tokens (Eq. 2): what a call runs on when the weight was not
// repacked, or has no repacked form because its input width is no multiple of 512 channels.  More tokens take
// linear_tile.hip.
//
// A wave is independent of every other wave until its sums are complete.  A block is 4 waves and owns all tokens of 64
// outputs; its waves take the channel groups in turn (wave w: groups w, w + 4, ...), so that every weight and every
// activation enters the compute unit once and the loop has no LDS, no barrier and no hand-over:
//   - weights: a lane's 16 bytes of a row's group are 32 channels of that row, which is the B operand of four
//     v_mfma_f32_16x16x32_f16 once the codes stand in fp16 registers as q - z (exact; 14 vector instructions per 8
//     weights in the natural code order, 9 in the repacked one); the group's scale multiplies the fp32 sums;
//   - registers are a ring of two groups: a register is refilled for the group after next right after its last use.
// The loop is written as slots, one MFMA each, with a piece of the next tile's dequantisation, a piece of the previous
// tile's scaling and at most two loads in its shadow, pinned by scheduling barriers.  The 4 waves' sums meet in LDS once;
// K is also split between blocks where the outputs alone are too few of them and the call has a scratch part.
//
// Bound by the weight stream and, at few groups per wave, by the chain load -> dequantise -> multiply -> sum.  The
// kernel before it read the activations in 2-byte pieces for every output row: 11008 -> 4096 at 24 tokens 939 us.
#include "paro_internal.h"
#include <type_traits>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowsWaves = 4, kRowsTiles = 4;       // waves per block (K in turn); 16-output tiles per block
constexpr uint32_t kOobR = 0x80000000u;             // beyond every buffer: reads as zero

__device__ inline __amdgpu_buffer_rsrc_t rows_rsrc(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}
__device__ inline half2v rows_h2(uint32_t u) { union { uint32_t u; half2v h; } c; c.u = u; return c.h; }
__device__ inline uint32_t rows_u32(half2v h) { union { uint32_t u; half2v h; } c; c.h = h; return c.u; }
__device__ inline uint32_t rows_uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

template <int N, class F, int I = 0>
__device__ __forceinline__ void rows_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        rows_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}

struct RowsArgs {
    const char *qweight;
    const _Float16 *scales;
    const uint32_t *qzeros;
    const _Float16 *X; int64_t ldx;
    _Float16 *Y; int64_t ldy;
    const _Float16 *bias;
    float *partial;                                  // [k slices][T][N] where K is split between blocks, else NULL
    int T, C, N, G, groups_per_split;
    uint32_t m_lo, k_lo;                             // 0x000F000F, 0x64006400: arguments, so that (u & m) | k is one instruction
};

// TB: blocks of 16 tokens, 1 or 2
template <int TB>
__global__ __launch_bounds__(kRowsWaves * 64, 2) void linear_rows_kernel(RowsArgs a)
{
    constexpr int NT = kRowsTiles, R = 2;            // tiles of 16 outputs; ring of groups
    constexpr int S = 4 * TB;                        // slots (MFMAs) per tile
    constexpr int P = 16 / S;                        // dequantisation pieces per slot
    static_assert(NT % 2 == 0 && (TB == 1 || TB == 2), "");
    __shared__ __attribute__((aligned(16))) float s_sum[kRowsWaves * TB * NT * 256];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * 16 * NT;
    const int n_rows = min(a.N - n0, 16 * NT);       // multiple of 16
    const int g_end = min(a.G, (int)(blockIdx.y + 1) * a.groups_per_split);
    const int g_first = blockIdx.y * a.groups_per_split + wave;
    const int n_grp = g_first < g_end ? (g_end - g_first + kRowsWaves - 1) / kRowsWaves : 0;   // of this wave
    const int ft = lane & 15, fkb = lane >> 4;

    // ---- addresses: a per-lane offset that is fixed (or out of range) plus a wave-uniform one -----------------------
    const __amdgpu_buffer_rsrc_t xr = rows_rsrc(a.X, ((size_t)(a.T - 1) * a.ldx + a.C) * 2);
    const __amdgpu_buffer_rsrc_t wr = rows_rsrc(a.qweight + (size_t)n0 * (a.C / 2), (size_t)n_rows * (a.C / 2));
    const __amdgpu_buffer_rsrc_t sr = rows_rsrc(a.scales, (size_t)a.G * a.N * 2);
    const __amdgpu_buffer_rsrc_t zr = rows_rsrc(a.qzeros, (size_t)a.G * a.N / 2);
    uint32_t xv[TB];
    rows_for<TB>([&](auto B) { xv[B] = B * 16 + ft < a.T ? (uint32_t)(((size_t)(B * 16 + ft) * a.ldx + fkb * 32) * 2) : kOobR; });
    const uint32_t wv = (uint32_t)ft * (uint32_t)(a.C / 2) + fkb * 16;
    // whole dwords, shifted where they are used: a 16-bit load's extension would be waited for where it is loaded
    const uint32_t sv = (ft & 14) * 2u, zv = (ft >> 3) * 4u;
    uint32_t n_tile[NT];                             // tiles beyond N read the last one again: their sums are not stored
    rows_for<NT>([&](auto N_) { n_tile[N_] = rows_uniform(min((int)N_, n_rows / kTileN - 1) * kTileN); });

    half8 xa[R][TB][4];
    u32x4 wq[R][NT];
    uint32_t wsc[R][NT], wz[R][NT];
    // the group that is being requested; beyond the wave's last one the per-lane offsets are out of range (nothing is fetched)
    uint32_t l_xv[TB], l_wv = kOobR, l_sv = kOobR, l_zv = kOobR, l_g = 0;
    auto request = [&](int i) {
        const bool ok = i < n_grp;
        rows_for<TB>([&](auto B) { l_xv[B] = ok ? xv[B] : kOobR; });
        l_wv = ok ? wv : kOobR; l_sv = ok ? sv : kOobR; l_zv = ok ? zv : kOobR;
        l_g = rows_uniform(g_first + i * kRowsWaves);
    };
    auto load_x = [&](int ring, int tb, int j) {
        union { u32x4 u; half8 h; } v;
        v.u = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(l_xv[tb] + j * 16), (int)(l_g * kGroup * 2), 0);
        xa[ring][tb][j] = v.h;
    };
    auto load_w = [&](int ring, int n) {
        const uint32_t first = l_g * (uint32_t)a.N + n0 + n_tile[n];
        wq[ring][n] = __builtin_amdgcn_raw_buffer_load_b128(wr, (int)l_wv, (int)(n_tile[n] * (uint32_t)(a.C / 2) + l_g * 64), 2);
        wsc[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(sr, (int)l_sv, (int)(first * 2u), 0);
        wz[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(zr, (int)l_zv, (int)(first / 2u), 0);
    };

    auto to_vgpr = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_ds_bpermute(lane << 2, (int)v); };
    const uint32_t c_mlo = to_vgpr(a.m_lo), c_klo = to_vgpr(a.k_lo);

    float4v tot[TB][NT], gacc[2][TB];
    union BFrag { u32x4 u; half8 h; } bf[2][4];
    float sc[2] = {0.f, 0.f};
    half2v nz = rows_h2(0);
    uint32_t sp = 0;                                 // codes 0, 2 (then 1, 3 eight bits higher) of a half word, spread
    rows_for<TB>([&](auto B) {
        rows_for<NT>([&](auto N_) { tot[B][N_] = float4v{0.f, 0.f, 0.f, 0.f}; });
        gacc[1][B] = float4v{0.f, 0.f, 0.f, 0.f};
    });
    // piece p (0..15) of the dequantisation of tile n in ring slot `ring` into bf[par]; the last piece also takes the
    // scale and refills the tile's registers (tile 0's are refilled in the next group's second slot)
    auto deq_piece = [&](auto PC, auto RING, auto N_, auto PAR) {
        constexpr int p = PC, w4 = p / 4, part = p % 4, ring = RING, n = N_, par = PAR;
        if constexpr (p == 0) nz = rows_h2((0xE400u + ((wz[ring][n] >> (4 * (ft & 7))) & 15u)) * 0x00010001u);   // -(1024 + z), twice
        const uint32_t u = wq[ring][n][w4];
        // codes 2 part and 2 part + 1 into the low nibbles of the two halves
        if constexpr (part == 0) { const uint32_t x = u & 0xffffu; sp = x | (x << 12); }
        if constexpr (part == 2) { const uint32_t x = u >> 16; sp = x | (x << 12); }
        bf[par][w4].u[part] = rows_u32(rows_h2(((part & 1 ? sp >> 8 : sp) & c_mlo) | c_klo) + nz);
        if constexpr (p == 15) {
            union { uint16_t u; _Float16 h; } c; c.u = (uint16_t)(wsc[ring][n] >> (16 * (ft & 1)));
            sc[par] = (float)c.h;
            if constexpr (n > 0) load_w(ring, n);
        }
    };

    // ---- prologue: the first R groups in the order in which the loop refills them, pinned (a load that the scheduler
    // moves behind the others would be waited for together with all of them) ----
    rows_for<R>([&](auto I) {
        request(I);
        rows_for<NT>([&](auto N_) { load_w(I, N_); __builtin_amdgcn_sched_barrier(0); });
        rows_for<4>([&](auto J) { rows_for<TB>([&](auto B) { load_x(I, B, J); __builtin_amdgcn_sched_barrier(0); }); });
    });
    using I0 = std::integral_constant<int, 0>;
    rows_for<16>([&](auto PC) { deq_piece(PC, I0{}, I0{}, I0{}); });

    // Whole rounds of the ring: groups beyond the wave's last read as zeros (an early end inside the loop would make the
    // compiler count the requests in flight for the shortest path).
    for (int i = 0; i < n_grp; i += R)
        rows_for<R>([&](auto U) {
            constexpr int ring = U;
            rows_for<NT>([&](auto N_) {
                constexpr int n = N_, par = n & 1;
                constexpr int nn = n + 1 < NT ? n + 1 : 0;                   // next tile: the following group's first after the last
                constexpr int nring = n + 1 < NT ? ring : (ring + 1) % R;
                rows_for<S>([&](auto SL) {
                    constexpr int s = SL, j = s / TB, tb = s % TB;
                    const float4v zero = {0.f, 0.f, 0.f, 0.f};
                    gacc[par][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[ring][tb][j], bf[par][j].h, j == 0 ? zero : gacc[par][tb], 0, 0, 0);
                    if constexpr (n == 0 && s == 1) { request(i + ring + R); load_w(ring, 0); }
                    if constexpr (n == NT - 1) load_x(ring, tb, j);
                    rows_for<P>([&](auto Q) {
                        deq_piece(std::integral_constant<int, s * P + Q>{}, std::integral_constant<int, nring>{},
                                  std::integral_constant<int, nn>{}, std::integral_constant<int, (par ^ 1)>{});
                    });
                    // the previous tile's sums of token block t, two slots or more after their last MFMA
                    constexpr int t = TB == 1 ? (s == 2 ? 0 : -1) : (s >= 2 && s < 2 + TB ? s - 2 : -1);
                    if constexpr (t >= 0) tot[t][(n + NT - 1) % NT] += sc[par ^ 1] * gacc[par ^ 1][t];
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        });
    rows_for<TB>([&](auto B) { tot[B][NT - 1] += sc[1] * gacc[1][B]; });     // the last tile of the last group

    // ---- the 4 waves' sums; lane l of a 16 x 16 tile holds output l % 16 of tokens 4 (l / 16) .. + 3 ----------------
    rows_for<TB>([&](auto B) {
        rows_for<NT>([&](auto N_) { *(float4v *)(s_sum + ((wave * TB + B) * NT + N_) * 256 + lane * 4) = tot[B][N_]; });
    });
    __syncthreads();
    for (int u = threadIdx.x; u < TB * NT * 64; u += kRowsWaves * 64) {
        const int tile = u >> 6, l = u & 63;
        const int n = tile % NT, t0 = tile / NT * 16 + (l >> 4) * 4;
        if (n * 16 >= n_rows) continue;
        float4v sum = *(const float4v *)(s_sum + u * 4);
#pragma unroll
        for (int w = 1; w < kRowsWaves; ++w) sum += *(const float4v *)(s_sum + w * TB * NT * 256 + u * 4);
        const int col = n0 + n * 16 + (l & 15);
        if (a.partial) {
            float *dst = a.partial + ((size_t)blockIdx.y * a.T + t0) * a.N + col;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + r < a.T) dst[(size_t)r * a.N] = sum[r];
        } else {
            const float bv = a.bias ? (float)a.bias[col] : 0.f;
            _Float16 *dst = a.Y + (size_t)t0 * a.ldy + col;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + r < a.T) dst[(size_t)r * a.ldy] = (_Float16)(sum[r] + bv);
        }
    }
}

// Slices of K so that there is about one block per compute unit, each of whole rounds of the block's 4 waves and of at
// least two groups per wave.  (11008 -> 4096, 64 blocks per slice, at 24 tokens: 1 / 2 / 4 / 8 slices 30 / 18 / 13 / 15 us
// before the summing launch of about 2 us.)
static void rows_split(int c_in, int c_out, int &k_split, int &groups_per_split)
{
    const int G = c_in / kGroup, blocks = (c_out + 16 * kRowsTiles - 1) / (16 * kRowsTiles);
    int ks = blocks >= 192 ? 1 : 256 / blocks;
    while (ks > 1 && G < ks * 2 * kRowsWaves) --ks;
    groups_per_split = (G + ks - 1) / ks;
    groups_per_split = (groups_per_split + kRowsWaves - 1) / kRowsWaves * kRowsWaves;
    k_split = (G + groups_per_split - 1) / groups_per_split;
}

size_t linear_rows_scratch_bytes(const paro_w4_weight &w, int T)
{
    int ks, gps;
    rows_split(w.c_in, w.c_out, ks, gps);
    return ks > 1 ? (size_t)ks * T * w.c_out * sizeof(float) : 0;
}

// scales as dwords; row offsets of a block and the whole code array in 31 bits; up to 32 tokens
bool linear_rows_supported(const paro_w4_weight &w, int64_t ldx, int T)
{
    return w.qweight && w.scales && w.qzeros && ((uintptr_t)w.scales % 4) == 0 && T <= 32 && (size_t)T * ldx * 2 < (1ull << 31) &&
           (size_t)w.c_out * (w.c_in / 2) < (1ull << 31);
}

hipError_t launch_linear_rows(const paro_w4_weight &w, const paro_half_t *X, int64_t ldx, paro_half_t *Y, int64_t ldy, int T,
                              void *scratch, size_t scratch_bytes, hipStream_t s)
{
    RowsArgs a;
    a.qweight = (const char *)w.qweight; a.scales = (const _Float16 *)w.scales; a.qzeros = w.qzeros;
    a.X = (const _Float16 *)X; a.ldx = ldx; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.G = w.c_in / kGroup;
    a.m_lo = 0x000F000Fu; a.k_lo = 0x64006400u;
    int ks;
    rows_split(w.c_in, w.c_out, ks, a.groups_per_split);
    const bool split = ks > 1 && scratch && scratch_bytes >= (size_t)ks * T * w.c_out * sizeof(float) && ((uintptr_t)scratch % 16) == 0;
    if (!split) { ks = 1; a.groups_per_split = a.G; }
    a.partial = split ? (float *)scratch : nullptr;
    const dim3 grid((w.c_out + 16 * kRowsTiles - 1) / (16 * kRowsTiles), ks), block(kRowsWaves * 64);
    if (T <= 16) hipLaunchKernelGGL(linear_rows_kernel<1>, grid, block, 0, s, a);
    else         hipLaunchKernelGGL(linear_rows_kernel<2>, grid, block, 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !split) return e;
    return launch_splitk_reduce(a.partial, ks, T, 0, w.c_out, w.bias, Y, ldy, s);
}

}  // namespace paro
