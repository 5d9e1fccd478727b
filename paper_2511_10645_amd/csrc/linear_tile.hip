// W4A16 linear, tiled, with the weights straight in registers (Eq. 2): from 33 tokens to some hundreds (a thousand on the
// narrower outputs), and weights in the interchange layout above 32 tokens.
//
// At these sizes neither of the other kernels fits.  The streaming kernel keeps a K-slice of activations in registers (32
// tokens fill half the register file) and re-reads the weights for every further 32 tokens.  The GEMM's 128 x 256 tiles are
// few, pay for rows that do not exist and carry every weight through LDS as fp16.  Here a block is 8 waves, each with 64
// tokens x 32 outputs of 64 (or 128) tokens x 128 outputs:
//   - activations (32 KB per step: 64 tokens x 2 groups, or 128 tokens x 1 group) go through LDS, whole 256-byte rows per
//     request, the 16-byte chunk index XOR-ed with the row so that both directions are conflict-free; requested two
//     steps ahead, written one step ahead, re-read into the fragment registers slot by slot as these fall free;
//   - weights never touch LDS: a lane's 16 bytes of a 16 x 128 tile are its operand of four v_mfma_f32_16x16x32_f16 once
//     the codes stand in registers as q - z (exact in fp16); the group's scale multiplies the fp32 sums of the group;
//   - with 64 tokens the waves split the step's two groups and add their sums through LDS at the end.
// The step is written as slots, one MFMA each, with a piece of the next tile's dequantisation, a piece of the previous
// tile's scaling and one load, LDS read or write in its shadow, pinned by scheduling barriers; one block barrier per step.
// K is split between blocks where the tiles alone are too few (fp32 partial tiles, summed by the GEMM's second kernel).
//
// What bounds it: no single unit.  Taking out a part of the step (timing only, 1024 tokens, 1.38 us per step) gives
// 1.01 without dequantisation, 1.15 without the scaling, 1.16 without LDS reads, 1.04 without staging: the parts add up, as
// in the GEMM, because the chip's clock pays for every instruction.  That is 0.35 us per 64 x 64 x 128 of work against
// the GEMM's 0.24 on full tiles, hence the line between the two (linear_tile_estimate_us).  Bare calls in a replayed graph
// over 350 MB of weights, summing launch included, us, before (the cheaper of the other two) -> now: 64 tokens 4096 -> 28672
// 37.8 -> 25.7, 14336 -> 4096 28.1 -> 20.9; 128 tokens 4096 -> 6144 22.9 -> 19.3, 4096 -> 4096 23.6 -> 16.9, 4096 -> 28672
// 49.3 -> 43.6; 201 tokens 4096 -> 6144 27.5 -> 22.4, 4096 -> 4096 22.9 -> 18.1.  Interchange layout, 11008 -> 4096 at 48
// tokens: rotated call 1874 -> 23.5 (K over 8 blocks); the bare call, which has no workspace and is not split, 1872 -> 52.3.
#include "paro_internal.h"
#include <type_traits>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kOobT = 0x80000000u;             // beyond every buffer: reads as zero, is not written
__device__ inline __amdgpu_buffer_rsrc_t tile_rsrc(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}
__device__ inline half2v tile_h2(uint32_t u) { union { uint32_t u; half2v h; } c; c.u = u; return c.h; }
__device__ inline uint32_t tile_u32(half2v h) { union { uint32_t u; half2v h; } c; c.h = h; return c.u; }
__device__ inline uint32_t tile_uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

template <int N, class F, int I = 0>
__device__ __forceinline__ void tile_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        tile_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}

struct TileArgs {
    const char *w;                                   // repacked blob, or qweight of the interchange layout
    uint32_t scales_off, zeros_off;                  // of the blob
    const _Float16 *scales; const uint32_t *qzeros;  // interchange layout
    const _Float16 *X; int64_t ldx;
    _Float16 *Y; int64_t ldy;
    const _Float16 *bias;
    float *partial;                                  // [k_split][T][N] where K is split between blocks
    int T, C, N, G, m_tiles, n_tiles, k_split, groups_per_split;
    uint32_t m_lo, m_hi, k_lo, k_hi;                 // 0x000F000F, 0x00F000F0, 0x64006400, 0x54005400 (see gemm.hip)
};

constexpr int kTileThreads = 512, kTileBuf = 32768;

// What the 16-byte chunk index of a row is XOR-ed with: the row, bit 3 flipped by bit 2.  A 16-byte LDS read serves lanes
// 0-3, 12-15 and 20-27 together (then 4-11, 16-19 and 28-31): rows 0-3 and 12-15 of one quarter of the channels and rows
// 4-11 of the next.  With the row itself the two sets of chunks coincide: 2.01 M conflict cycles over the chip at 64 tokens
// 4096 -> 28672 (of 1.25 M instruction cycles of LDS), now 57 k; 1 to 4 % faster (LDS is not what bounds the kernel).
__device__ inline int chunk_xor(int row) { return (row & 15) ^ ((row & 4) << 1); }

template <int MW, int NW, int KW, bool IC>
__global__ __launch_bounds__(kTileThreads, 2) void linear_tile_kernel(TileArgs a)
{
    static_assert(MW * NW * KW == 8 && MW * KW == 2 && NW == 4, "");
    constexpr int TB = 4, NT = 2, S = 16, TM = 64 * MW, TN = 32 * NW;
    extern __shared__ __attribute__((aligned(16))) char s_x[];            // [2][KW][TM][256 B]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = wave % NW, mw = wave / NW % MW, kw = wave / (NW * MW);

    // Consecutive tiles - token tiles first, then output tiles, then slices of K - on one XCD: its L2 serves a tile's
    // weights to the further token tiles and a slice's activations to the further output tiles, and every XCD has the
    // same number of blocks (to one) whatever the counts are.  (The GEMM's patches of powers of two leave XCDs idle at 5
    // token tiles: 8192 -> 16384 at 640 tokens 300 us against 212.)
    const int tiles = a.m_tiles * a.n_tiles, all = tiles * a.k_split, per_xcd = (all + 7) / 8;
    const int idx = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (idx >= all) return;
    const int kslice = idx / tiles, tile = idx % tiles, mt = tile % a.m_tiles, ntile = tile / a.m_tiles;
    const int m0 = (int)tile_uniform(mt * TM), n0 = (int)tile_uniform(ntile * TN + nw * 32);
    const int rows = min(a.T - m0, TM);
    const int g0 = (int)tile_uniform(kslice * a.groups_per_split), g_end = min(a.G, g0 + a.groups_per_split);
    const int n_steps = (g_end - g0 + KW - 1) / KW;
    const int ft = lane & 15, fkb = lane >> 4;

    // ---- activations: thread -> 16-byte chunk tid % 16 of rows tid / 16 + 32 i of the step's [KW][TM] rows ----------
    const __amdgpu_buffer_rsrc_t xr = tile_rsrc(a.X + (size_t)m0 * a.ldx, ((size_t)(rows - 1) * a.ldx + a.C) * 2);
    const int sc16 = tid & 15, srow = tid >> 4;
    uint32_t xg[4];
    tile_for<4>([&](auto I) {
        const int row = srow + 32 * I, t = row % TM;
        xg[I] = t < rows ? (uint32_t)(((size_t)t * a.ldx) * 2 + sc16 * 16) : kOobT;
    });
    const int xw = srow * 256 + ((sc16 ^ chunk_xor(srow)) << 4);           // + 8192 i
    u32x4 xs[4];
    auto load_x = [&](int step, auto I) {
        const int g = g0 + step * KW + (KW == 1 ? 0 : (int)I / 2);        // rows 0..63 of KW = 2: the step's first group
        xs[I] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(g < g_end ? xg[I] : kOobT), (int)tile_uniform(g * 256), 0);
    };
    auto store_x = [&](int buf, auto I) { *(u32x4 *)(s_x + buf * kTileBuf + xw + I * 8192) = xs[I]; };
    int xa_off[4];
    tile_for<4>([&](auto J) { xa_off[J] = (kw * TM + mw * 64 + ft) * 256 + (((fkb * 4 + J) ^ chunk_xor(ft)) << 4); });
    half8 xa[TB][4];
    auto read_x = [&](int buf, auto B, auto J) { xa[B][J] = *(const half8 *)(s_x + buf * kTileBuf + xa_off[J] + B * 4096); };

    // ---- weights of the wave: two 16-row tiles ----------------------------------------------------------------------
    const int n_rows = min(a.N - n0, 32);            // multiple of 16; <= 0: this wave's outputs do not exist
    const int tile0 = n0 / kTileN;
    const __amdgpu_buffer_rsrc_t wr = IC ? tile_rsrc(a.w, n_rows > 0 ? (size_t)a.N * (a.C / 2) : 0)
                                         : tile_rsrc(a.w, a.zeros_off + packed_zeros_bytes(a.C, a.N));
    const __amdgpu_buffer_rsrc_t sr = tile_rsrc(a.scales, IC ? (size_t)a.G * a.N * 2 : 0);
    const __amdgpu_buffer_rsrc_t zr = tile_rsrc(a.qzeros, IC ? (size_t)a.G * a.N / 2 : 0);
    constexpr uint32_t kWGroup = IC ? 64 : 1024;
    const uint32_t wv = IC ? (uint32_t)ft * (uint32_t)(a.C / 2) + fkb * 16 : lane * 16u;
    const uint32_t sv = IC ? (ft & 14) * 2u : ft * 8u, zv = IC ? (ft >> 3) * 4u : (ft & 14) * 2u;
    const uint32_t z_sh = IC ? 4 * (ft & 7) : 16 * (ft & 1);
    uint32_t w_tile[NT], s_tile[NT];
    tile_for<NT>([&](auto N_) {
        const int n = N_ * kTileN < n_rows ? (int)N_ : 0;
        w_tile[N_] = tile_uniform(IC ? (uint32_t)(n0 + n * 16) * (uint32_t)(a.C / 2) : (uint32_t)(tile0 + n) * (uint32_t)a.G * 1024u);
        s_tile[N_] = tile_uniform(IC ? (uint32_t)(n0 + n * kTileN) : (uint32_t)(tile0 + n) * (uint32_t)(a.G / kSliceGroups));
    });
    u32x4 wq[2][NT];
    uint32_t wsc[2][NT], wz[2][NT];
    auto load_w = [&](int step, auto RING, auto N_) {
        constexpr int ring = RING, n = N_;
        const int g = g0 + step * KW + kw;
        const bool ok = g < g_end && n_rows > 0;
        const uint32_t gu = tile_uniform(g);
        wq[ring][n] = __builtin_amdgcn_raw_buffer_load_b128(wr, (int)(ok ? wv : kOobT), (int)(w_tile[n] + gu * kWGroup), 0);
        if constexpr (IC) {
            wsc[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(sr, (int)(ok ? sv : kOobT), (int)((gu * (uint32_t)a.N + s_tile[n]) * 2u), 0);
            wz[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(zr, (int)(ok ? zv : kOobT), (int)((gu * (uint32_t)a.N + s_tile[n]) / 2u), 0);
        } else {
            const uint32_t sl = s_tile[n] + (gu >> 2);
            wsc[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(wr, (int)(ok ? sv : kOobT), (int)(a.scales_off + sl * 128u + (gu & 2) * 2), 0);
            wz[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(wr, (int)(ok ? zv : kOobT), (int)(a.zeros_off + sl * 32u), 0);
        }
    };
    auto to_vgpr = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_ds_bpermute(lane << 2, (int)v); };
    const uint32_t c_mlo = to_vgpr(a.m_lo), c_mhi = to_vgpr(a.m_hi), c_klo = to_vgpr(a.k_lo), c_khi = to_vgpr(a.k_hi);

    float4v tot[TB][NT], gacc[2][TB];
    union BFrag { u32x4 u; half8 h; } bf[2][4];
    float sc[2] = {0.f, 0.f};
    half2v nlo = tile_h2(0), nhi = tile_h2(0);
    uint32_t sp = 0;
    tile_for<TB>([&](auto B) {
        tile_for<NT>([&](auto N_) { tot[B][N_] = float4v{0.f, 0.f, 0.f, 0.f}; });
        gacc[1][B] = float4v{0.f, 0.f, 0.f, 0.f};
    });
    auto deq_piece = [&](auto PC, int step, auto RING, auto N_) {
        constexpr int p = PC, w4 = p / 4, part = p % 4, ring = RING, n = N_;
        const uint32_t g = tile_uniform(g0 + step * KW + kw);
        if constexpr (p == 0) {
            const uint32_t z = (wz[ring][n] >> (IC ? z_sh : z_sh + 4 * (g & 3))) & 15u;
            nlo = tile_h2((0xE400u + z) * 0x00010001u);              // -(1024 + z), twice
            if constexpr (!IC) nhi = tile_h2((0xD400u + (z << 4)) * 0x00010001u);    // -(64 + z), twice
        }
        const uint32_t u = wq[ring][n][w4];
        if constexpr (IC) {
            if constexpr (part == 0) { const uint32_t x = u & 0xffffu; sp = x | (x << 12); }
            if constexpr (part == 2) { const uint32_t x = u >> 16; sp = x | (x << 12); }
            bf[n][w4].u[part] = tile_u32(tile_h2(((part & 1 ? sp >> 8 : sp) & c_mlo) | c_klo) + nlo);
        } else {
            const uint32_t v = part < 2 ? u : u >> 8;
            if constexpr (part & 1) bf[n][w4].u[part] = tile_u32(tile_h2((v & c_mhi) | c_khi) + nhi);
            else bf[n][w4].u[part] = tile_u32(tile_h2((v & c_mlo) | c_klo) + nlo);
        }
        if constexpr (p == 15) {
            union { uint16_t u; _Float16 h; } c; c.u = (uint16_t)(wsc[ring][n] >> (IC ? 16 * (ft & 1) : 16 * (g & 1)));
            sc[n] = (float)c.h;
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    // ---- prologue ----
    tile_for<4>([&](auto I) { load_x(0, I); __builtin_amdgcn_sched_barrier(0); });
    tile_for<2>([&](auto U) { tile_for<NT>([&](auto N_) { load_w(U, U, N_); __builtin_amdgcn_sched_barrier(0); }); });
    tile_for<4>([&](auto I) { store_x(0, I); });
    tile_for<4>([&](auto I) { load_x(1, I); __builtin_amdgcn_sched_barrier(0); });
    __syncthreads();
    tile_for<TB>([&](auto B) { tile_for<4>([&](auto J) { read_x(0, B, J); }); });
    tile_for<16>([&](auto PC) { deq_piece(PC, 0, I0{}, I0{}); });

    for (int s0 = 0; s0 < n_steps; s0 += 2) {
        tile_for<2>([&](auto U) {
            constexpr int ring = U;
            const int step = s0 + ring;
            tile_for<NT>([&](auto N_) {
                constexpr int n = N_;
                tile_for<S>([&](auto SL) {
                    constexpr int s = SL, j = s / TB, tb = s % TB;
                    const float4v zero = {0.f, 0.f, 0.f, 0.f};
                    gacc[n][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[tb][j], bf[n][j].h, j == 0 ? zero : gacc[n][tb], 0, 0, 0);
                    if constexpr (n == 0) deq_piece(SL, step, U, I1{});
                    else deq_piece(SL, step + 1, std::integral_constant<int, (ring ^ 1)>{}, I0{});
                    if constexpr (s >= 2 && s < 2 + TB) tot[s - 2][n ^ 1] += sc[n ^ 1] * gacc[n ^ 1][s - 2];
                    if constexpr (n == 0) {
                        if constexpr (s == 1) load_w(step + 2, U, I0{});
                        // the next step's rows into the other buffer (last read before the previous barrier)
                        if constexpr (s >= 6 && s < 14 && s % 2 == 0) store_x(ring ^ 1, std::integral_constant<int, (s - 6) / 2>{});
                        if constexpr (s >= 6 && s < 14 && s % 2 == 1) load_x(step + 2, std::integral_constant<int, (s - 6) / 2>{});
                    } else {
                        if constexpr (s == 1) load_w(step + 2, U, I1{});
                        read_x(ring ^ 1, std::integral_constant<int, tb>{}, std::integral_constant<int, j>{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (n == 0) __syncthreads();
            });
        });
    }
    tile_for<TB>([&](auto B) { tot[B][1] += sc[1] * gacc[1][B]; });

    // ---- epilogue: lane holds output ft of tokens 4 fkb .. + 3 of a 16 x 16 tile ------------------------------------
    __syncthreads();
    if constexpr (KW == 2) {                         // the second half of K through LDS (the loop's buffers are free)
        float4v *sum = (float4v *)s_x + (size_t)(wave % 4) * TB * NT * 64;
        if (kw == 1) tile_for<TB>([&](auto B) { tile_for<NT>([&](auto N_) { sum[(B * NT + N_) * 64 + lane] = tot[B][N_]; }); });
        __syncthreads();
        if (kw == 1) return;
        tile_for<TB>([&](auto B) { tile_for<NT>([&](auto N_) { tot[B][N_] += sum[(B * NT + N_) * 64 + lane]; }); });
    }
    if (n_rows <= 0) return;
    const int mrow0 = m0 + mw * 64;
    if (a.partial) {
        float *dst = a.partial + ((size_t)kslice * a.T + mrow0 + fkb * 4) * a.N + n0 + ft;
        tile_for<TB>([&](auto B) {
            tile_for<NT>([&](auto N_) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (mrow0 + B * 16 + fkb * 4 + r < a.T && N_ * 16 < n_rows) dst[(size_t)(B * 16 + r) * a.N + N_ * 16] = tot[B][N_][r];
            });
        });
        return;
    }
    // a 16 x 32 strip through a wave-private kilobyte of LDS, out as one 16-byte store per lane
    _Float16 *strip = (_Float16 *)(s_x + 2 * kTileBuf - 8192 + wave * 1024);
    float bv[NT];
    tile_for<NT>([&](auto N_) { bv[N_] = (a.bias && N_ * 16 < n_rows) ? (float)a.bias[n0 + N_ * 16 + ft] : 0.f; });
    const int orow = lane >> 2, ocol = (lane & 3) * 8;
    tile_for<TB>([&](auto B) {
        tile_for<NT>([&](auto N_) {
#pragma unroll
            for (int r = 0; r < 4; ++r) strip[(fkb * 4 + r) * 32 + N_ * 16 + ft] = (_Float16)(tot[B][N_][r] + bv[N_]);
        });
        __builtin_amdgcn_wave_barrier();
        const u32x4 v = *(const u32x4 *)(strip + orow * 32 + ocol);
        if (ocol < n_rows && mrow0 + B * 16 + orow < a.T)
            *(u32x4 *)(a.Y + (size_t)(mrow0 + B * 16 + orow) * a.ldy + n0 + ocol) = v;
        __builtin_amdgcn_wave_barrier();
    });
}

template <int MW, int NW, int KW, bool IC>
static hipError_t launch_tile_cfg(TileArgs &a, hipStream_t s)
{
    a.m_tiles = (a.T + 64 * MW - 1) / (64 * MW); a.n_tiles = (a.N + 32 * NW - 1) / (32 * NW);
    const unsigned blocks = (unsigned)(((size_t)a.m_tiles * a.n_tiles * a.k_split + 7) / 8 * 8);
    static std::atomic<uint64_t> attr_done{0};
    if (const int dev = once_pending(attr_done); dev >= 0) {
        hipError_t e = hipFuncSetAttribute((const void *)linear_tile_kernel<MW, NW, KW, IC>, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * kTileBuf);
        if (e != hipSuccess) return e;
        once_done(attr_done, dev);
    }
    hipLaunchKernelGGL((linear_tile_kernel<MW, NW, KW, IC>), dim3(blocks), dim3(kTileThreads), 2 * kTileBuf, s, a);
    return hipGetLastError();
}


// Which tile, and how many slices of K: the least of a cost model fitted to 4700 timings (58 shapes from 512 to 27648
// channels and 512 to 55296 outputs, 33 to 2048 tokens; 7 % off in the mean): 1.6 us, per round of 256 blocks 3.5 us (first
// requests, stores) and 0.96 us per step, 1.09 us where the blocks fill the chip, and for split K 1.7 us (the summing
// launch's share of a graph; begin to end in a trace it is 4), 0.23 us per slice and the partial tiles at 6.9 TB/s.
struct TilePlan { bool two_m; int k_split, groups_per_split; double est_us; };
static TilePlan plan_tile(int c_in, int c_out, int T)
{
    TilePlan best{false, 1, 0, 1e30};
    const int G = c_in / kGroup, n_tiles = (c_out + 127) / 128;
    for (int two = 0; two <= (T > 64 ? 1 : 0); ++two) {
        const int m_tiles = (T + (two ? 127 : 63)) / (two ? 128 : 64);
        for (int ks = 1; ks <= 16 && (ks == 1 || (ks * 4 <= G && (long)m_tiles * n_tiles * ks <= 512)); ++ks) {
            const int gps = ((G + ks - 1) / ks + 3) / 4 * 4;             // whole steps of either tile, an even number of them
            if ((G + gps - 1) / gps != ks) continue;
            const long blocks = (long)m_tiles * n_tiles * ks, rounds = ((blocks + 7) / 8 + 31) / 32;
            const double step_us = (blocks >= 160 ? 1.09 : 0.96) - (two ? 0.04 : 0.0);
            double us = 1.6 + (double)rounds * (3.5 + (two ? gps : gps / 2) * step_us);
            if (ks > 1) us += 1.7 + 0.23 * ks + (double)ks * T * c_out * 8.0 / 6.9e6;
            if (us < best.est_us) best = TilePlan{two != 0, ks, gps, us};
        }
    }
    return best;
}

double linear_tile_estimate_us(const paro_w4_weight &w, int T) { return plan_tile(w.c_in, w.c_out, T).est_us; }

size_t linear_tile_scratch_bytes(const paro_w4_weight &w, int T)
{
    const TilePlan p = plan_tile(w.c_in, w.c_out, T);
    return p.k_split > 1 ? (size_t)p.k_split * T * w.c_out * sizeof(float) : 0;
}

void linear_tile_plan(const paro_w4_weight &w, int T, int &tokens, int &k_slices)
{
    const TilePlan p = plan_tile(w.c_in, w.c_out, T);
    tokens = p.two_m ? 128 : 64; k_slices = p.k_split;
}

// the weights are addressed with 31-bit byte offsets, the scales of the interchange layout as dwords
bool linear_tile_supported(const paro_w4_weight &w, bool interchange)
{
    if (!interchange) return w.packed && packed_blob_bytes(w.c_in, w.c_out) < (1ull << 31);
    return w.qweight && w.scales && w.qzeros && ((uintptr_t)w.scales % 4) == 0 && (size_t)w.c_out * (w.c_in / 2) < (1ull << 31);
}

hipError_t launch_linear_tile(const paro_w4_weight &w, bool interchange, const paro_half_t *X, int64_t ldx, paro_half_t *Y,
                              int64_t ldy, int T, void *scratch, size_t scratch_bytes, const void *least, hipStream_t s)
{
    TilePlan p = plan_tile(w.c_in, w.c_out, T);
    TileArgs a;
    a.w = interchange ? (const char *)w.qweight : (const char *)w.packed;
    a.scales_off = (uint32_t)packed_tiles_bytes(w.c_in, w.c_out);
    a.zeros_off = a.scales_off + (uint32_t)packed_scales_bytes(w.c_in, w.c_out);
    a.scales = (const _Float16 *)w.scales; a.qzeros = w.qzeros;
    a.X = (const _Float16 *)X; a.ldx = ldx; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.G = w.c_in / kGroup;
    a.m_lo = 0x000F000Fu; a.m_hi = 0x00F000F0u; a.k_lo = 0x64006400u; a.k_hi = 0x54005400u;
    if (p.k_split > 1 && !(scratch && scratch_bytes >= (size_t)p.k_split * T * w.c_out * sizeof(float) && ((uintptr_t)scratch % 16) == 0)) {
        if (!interchange) return hipErrorInvalidValue;                   // the caller takes another kernel then
        p.k_split = 1; p.groups_per_split = (a.G + 3) / 4 * 4;           // no room for partial tiles
    }
    a.k_split = p.k_split; a.groups_per_split = p.groups_per_split;
    a.partial = p.k_split > 1 ? (float *)scratch : nullptr;
    hipError_t e = interchange ? (p.two_m ? launch_tile_cfg<2, 4, 1, true>(a, s) : launch_tile_cfg<1, 4, 2, true>(a, s))
                               : (p.two_m ? launch_tile_cfg<2, 4, 1, false>(a, s) : launch_tile_cfg<1, 4, 2, false>(a, s));
    if (e != hipSuccess || p.k_split == 1) return e;
    return launch_splitk_reduce(a.partial, p.k_split, T, 0, w.c_out, w.bias, Y, ldy, least, s);
}

}  // namespace paro
