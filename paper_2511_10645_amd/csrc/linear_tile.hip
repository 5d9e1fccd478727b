// W4A16 linear, tiled, with the weights straight in registers (Eq. 2): from 33 tokens to some hundreds (thousands where
// the outputs are few), and weights in the interchange layout above 32 tokens where linear_ic.hip is not the faster.
//
// At these sizes neither of the other kernels fits.  The streaming kernel keeps a K-slice of activations in registers (32
// tokens fill half the register file) and re-reads the weights for every further 32 tokens.  The GEMM's 128 x 256 tiles are
// few, pay for rows that do not exist and carry every weight through LDS as fp16.  Here a block is 8 waves and 64 or 128
// tokens x 128 outputs.  Every wave has 64 tokens x 32 outputs, with 64 tokens of one of a step's two groups (128 tokens of
// more groups: below):
//   - activations (32 KB per step) go through LDS, whole 256-byte rows per request, the 16-byte chunk index XOR-ed with the row
//     so that both directions are conflict-free; requested two steps ahead, written one step ahead, re-read into the fragment
//     registers slot by slot as these fall free;
//   - weights never touch LDS: a lane's 16 bytes of a 16 x 128 tile are its operand of four v_mfma_f32_16x16x32_f16 once
//     the codes stand in registers as q - z (exact in fp16); the group's scale multiplies the fp32 sums of the group;
//   - the two halves of K are added through LDS at the end.
// The step is written as slots, one MFMA each, with a piece of the next tile's dequantisation, a piece of the previous
// tile's scaling and one load, LDS read or write in its shadow, pinned by scheduling barriers; one block barrier per step.
// K is split between blocks where the tiles alone are too few (fp32 partial tiles, summed by the GEMM's second kernel).
//
// What bounds it: no single unit.  Taking out a part of the step (timing only) takes off what the part issues: the parts add
// up, as in the GEMM, because the chip's clock pays for every instruction; at 64 tokens the weight stream is next (4096 -> 28672
// without multiplication and scaling 18 of 25 us).  Bare calls in a replayed graph over 350 MB of weights, summing launch included,
// us, the cheaper of the other two kernels -> this one: 64 tokens 4096 -> 28672 37.8 -> 25.4, 14336 -> 4096 28.1 -> 19.5;
// 128 tokens 4096 -> 6144 22.9 -> 18.9, 4096 -> 4096 23.6 -> 15.7, 4096 -> 28672 49.3 -> 38.6; 201 tokens 4096 -> 6144 27.5 -> 21.2,
// 4096 -> 4096 22.9 -> 17.9.  Interchange layout, 11008 -> 4096 at 48 tokens: rotated call 1874 -> 23.5 (K over 8 blocks); the
// bare call, which has no workspace and is not split, 1872 -> 52.3.
#include "paro_internal.h"
#include <algorithm>
#include <type_traits>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void tile_lds_t;

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

// Results leave the L2 as they are written (sc1) instead of all at once at the end of the launch; rows beyond a tile's are
// beyond the buffer.  us, plain stores / these: 4096 -> 28672 at 128 tokens 38.8 / 37.6, 14336 -> 4096 at 64 (partial tiles)
// 24.0 / 23.4 rotated.  Not outputs whose rows do not begin on a cache line: two tiles share the line there, and each would write
// its piece (512 -> 32656 at 128 tokens 10.7 / 11.8, 640 -> 8208 at 1000 31.2 / 32.2); partial tiles gain even so (8192 -> 1552 at
// 129 tokens 16.3 / 15.6).
constexpr int kAuxThrough = 16;
__device__ __forceinline__ void tile_store(bool through, u32x4 v, __amdgpu_buffer_rsrc_t r, int off)
{
    if (through) __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, kAuxThrough);
    else __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
}
__device__ inline __amdgpu_buffer_rsrc_t tile_outputs(const TileArgs &a, int m0, int rows)
{
    return tile_rsrc(a.Y + (size_t)m0 * a.ldy, ((size_t)(rows - 1) * a.ldy + a.N) * 2);
}
__device__ inline __amdgpu_buffer_rsrc_t tile_partials(const TileArgs &a, int kslice, int m0, int rows)
{
    return tile_rsrc(a.partial ? a.partial + ((size_t)kslice * a.T + m0) * a.N : nullptr, a.partial ? (size_t)rows * a.N * 4 : 0);
}

// What the 16-byte chunk index of a row is XOR-ed with: the row, bit 3 flipped by bit 2.  A 16-byte LDS read serves lanes
// 0-3, 12-15 and 20-27 together (then 4-11, 16-19 and 28-31): rows 0-3 and 12-15 of one quarter of the channels and rows
// 4-11 of the next.  With the row itself the two sets of chunks coincide: 2.01 M conflict cycles over the chip at 64 tokens
// 4096 -> 28672 (of 1.25 M instruction cycles of LDS), now 57 k; 1 to 4 % faster (LDS is not what bounds the kernel).
__device__ inline int chunk_xor(int row) { return (row & 15) ^ ((row & 4) << 1); }

// MW: 64-token parts of the block's tile; one: the waves split a step's two groups, two: a step is one group
template <int MW, bool IC>
__global__ __launch_bounds__(kTileThreads, 2) void linear_tile_kernel(TileArgs a)
{
    constexpr int NW = 4, KW = 2 / MW, TB = 4, NT = 2, S = 16, TM = 64 * MW, TN = 32 * NW;
    extern __shared__ __attribute__((aligned(16))) char s_x[];            // [2][KW][TM][256 B]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = wave % NW, mw = wave / NW % MW, kw = wave / (NW * MW);

    // Consecutive tiles - token tiles first, then output tiles, then slices of K - on one XCD: its L2 serves a tile's
    // weights to the further token tiles and a slice's activations to the further output tiles, and every XCD has the
    // same number of blocks (to one) whatever the counts are.  (Patches of powers of two leave XCDs idle at 5 token tiles:
    // 8192 -> 16384 at 640 tokens 300 us against 212.)
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
        const int g = g0 + step * KW + (KW == 1 ? 0 : (int)I / 2);         // rows 0..63 of KW = 2: the step's first group
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
    if (a.partial) {
        const __amdgpu_buffer_rsrc_t pr = tile_partials(a, kslice, m0, rows);
        tile_for<TB>([&](auto B) {
            tile_for<NT>([&](auto N_) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (N_ * 16 < n_rows)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(tot[B][N_][r]), pr, ((mw * 64 + B * 16 + fkb * 4 + r) * a.N + n0 + ft + N_ * 16) * 4, 0, kAuxThrough);
            });
        });
        return;
    }
    const __amdgpu_buffer_rsrc_t yr = tile_outputs(a, m0, rows);
    const bool through = (((uintptr_t)a.Y | (uintptr_t)(a.ldy * 2)) & 127) == 0;
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
        if (ocol < n_rows) tile_store(through, v, yr, ((mw * 64 + B * 16 + orow) * (int)a.ldy + n0 + ocol) * 2);
        __builtin_amdgcn_wave_barrier();
    });
}

constexpr int kTile2Stage = 65536, kTile2Lds = 2 * kTile2Stage;

// 128 tokens x 128 outputs.  A wave has 64 x 64 of them and one of a step's two groups, so that an operand read from LDS serves
// two tiles of v_mfma_f32_32x32x16_f16 (half the LDS reads and half the matrix instructions per product of the 64 x 32 tile above,
// which bounded it: read, dequantised and scaled in phases that every wave went through together, the units took turns).
// Activations go to LDS directly, 64 KB per step in a ring of two: behind the barrier that ends a step its buffer is requested
// anew at once.  Weights are two groups ahead in registers; what is multiplied next is read and dequantised while this is.
// The matrix pipes are busy 0.47 of a block's cycles (30 % of the launch at 4096 -> 28672, 128 tokens), issue the rest; without
// activations' requests (timing only) 35 us of 39.8.  A launch begins and ends in 9 us, 2 of them the first requests, 2 to 4 the sums and the
// stores (an empty kernel takes 1.7 us whatever its LDS and threads): not for few groups (kTileWideGroups).
// us, that -> this: 4096 -> 28672 at 128 tokens 44.3 -> 37.6, rotated 49.2 -> 43.5; 14336 -> 4096 at 201 42.2 -> 38.5;
// 512 -> 32656 at 289 rotated 27.4 -> 23.0; 75 random shapes of 65 to 1100 tokens 0.976 of the time (other kernels' among them).

template <int N> __device__ __forceinline__ void tile_wait_vm() { __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14)); }

template <bool IC>
__global__ __launch_bounds__(kTileThreads, 2) void linear_tile2_kernel(TileArgs a)
{
    constexpr int MW = 2, KW = 2, NW = 2, TB = 2, NT = 2, TM = 64 * MW, TN = 128, KK = 8;
    extern __shared__ __attribute__((aligned(16))) char s_x[];            // [2][KW][TM][256 B]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = wave % NW, mw = wave / NW % MW, kw = wave / (NW * MW);

    // Consecutive tiles - token tiles first, then output tiles, then slices of K - on one XCD: its L2 serves a tile's
    // weights to the further token tiles and a slice's activations to the further output tiles, and every XCD has the
    // same number of blocks (to one) whatever the counts are.  (Patches of powers of two leave XCDs idle at 5 token tiles:
    // 8192 -> 16384 at 640 tokens 300 us against 212.)
    const int tiles = a.m_tiles * a.n_tiles, all = tiles * a.k_split, per_xcd = (all + 7) / 8;
    const int idx = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (idx >= all) return;
    const int kslice = idx / tiles, tile = idx % tiles, mt = tile % a.m_tiles, ntile = tile / a.m_tiles;
    const int m0 = (int)tile_uniform(mt * TM), n0 = (int)tile_uniform(ntile * TN + nw * 64);
    const int rows = min(a.T - m0, TM);
    const int g0 = (int)tile_uniform(kslice * a.groups_per_split), g_end = min(a.G, g0 + a.groups_per_split);
    const int n_steps = (g_end - g0 + KW - 1) / KW, n_own = (int)tile_uniform((g_end - g0 - kw + KW - 1) / KW);   // groups of this wave
    const int r32 = lane & 31, half = lane >> 5, ft = lane & 15;

    // ---- activations: this wave requests 32 rows of one group of a step, 4 whole rows per request -------------------
    const __amdgpu_buffer_rsrc_t xr = tile_rsrc(a.X + (size_t)m0 * a.ldx, ((size_t)(rows - 1) * a.ldx + a.C) * 2);
    const int x_group = wave / (TM / 32), x_row = wave % (TM / 32) * 32;
    uint32_t xg[4];                                  // rows beyond T are beyond the buffer; the last four are 16 rows on
    tile_for<4>([&](auto I) {
        const int t = x_row + 4 * I + (lane >> 4);
        xg[I] = (uint32_t)((size_t)t * a.ldx * 2) + (((lane & 15) ^ (t & 15)) << 4);
    });
    const uint32_t x_next = tile_uniform((uint32_t)(a.ldx * 32));
    auto request_x = [&](int step, int buf, auto I) {
        const int g = g0 + step * KW + x_group;
        char *dst = s_x + buf * kTile2Stage + wave * 8192 + I * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (tile_lds_t *)dst, 16, (int)((g < g_end ? xg[I % 4] : kOobT) + (I / 4) * x_next), (int)tile_uniform(g * 256), 0, 0);
    };
    // operand kk = 4 i + j of a group: channels 64 i + 32 half + 8 j .. + 7, chunk 8 i + 4 half + j
    const int x_off = (kw * TM + mw * 64 + r32) * 256 + (((half * 4) ^ ft) << 4);
    half8 xa[2][TB];
    auto read_x = [&](int buf, auto B, auto KK_) {
        constexpr int kk = KK_;
        xa[kk & 1][B] = *(const half8 *)(s_x + (x_off ^ (((kk / 4) * 8 + kk % 4) << 4)) + buf * kTile2Stage + B * 8192);
    };

    // ---- weights of the wave: two tiles of 32 rows, lane: row lane % 32, channels 32 half .. + 31 and 64 + 32 half .. + 31
    const int n_rows = min(a.N - n0, 64);            // multiple of 16; <= 0: this wave's outputs do not exist
    const __amdgpu_buffer_rsrc_t wr = IC ? tile_rsrc(a.w, n_rows > 0 ? (size_t)a.N * (a.C / 2) : 0)
                                         : tile_rsrc(a.w, a.zeros_off + packed_zeros_bytes(a.C, a.N));
    const __amdgpu_buffer_rsrc_t sr = tile_rsrc(a.scales, IC ? (size_t)a.G * a.N * 2 : 0);
    const __amdgpu_buffer_rsrc_t zr = tile_rsrc(a.qzeros, IC ? (size_t)a.G * a.N / 2 : 0);
    constexpr uint32_t kWGroup = IC ? 64 : 1024, kWHalf = IC ? 32 : 512;
    const uint32_t z_sh = IC ? 4 * (ft & 7) : 16 * (ft & 1);
    uint32_t wv[NT], sv[NT], zv[NT];
    tile_for<NT>([&](auto N_) {
        const int c = N_ * 32 + (lane & 16) < n_rows ? N_ * 32 + (lane & 16) : 0;      // rows beyond N read others: not stored
        const uint32_t row = (uint32_t)max(n0 + c, 0), t16 = row / kTileN;
        wv[N_] = IC ? (row + ft) * (uint32_t)(a.C / 2) + half * 16 : t16 * (uint32_t)a.G * 1024u + half * 256 + ft * 16;
        sv[N_] = IC ? (row + (ft & 14)) * 2u : t16 * (uint32_t)(a.G / kSliceGroups) * 128u + ft * 8;
        zv[N_] = IC ? row / 2 + (ft >> 3) * 4 : t16 * (uint32_t)(a.G / kSliceGroups) * 32u + (ft & 14) * 2;
        if (n_rows <= 0) wv[N_] = sv[N_] = zv[N_] = kOobT;
    });
    u32x4 wq[2][NT][2];
    uint32_t wsc[2][NT], wz[2][NT];
    auto load_w = [&](int step, auto RING, auto N_, auto H) {
        const int g = g0 + step * KW + kw;
        wq[RING][N_][H] = __builtin_amdgcn_raw_buffer_load_b128(wr, (int)((g < g_end ? wv[N_] : kOobT) + H * kWHalf), (int)tile_uniform(g * kWGroup), 0);
    };
    auto load_sz = [&](int step, auto RING, auto N_) {
        const int g = g0 + step * KW + kw;
        const uint32_t gu = tile_uniform(g), so = g < g_end ? sv[N_] : kOobT, zo = g < g_end ? zv[N_] : kOobT;
        if constexpr (IC) {
            wsc[RING][N_] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(sr, (int)so, (int)(gu * (uint32_t)a.N * 2u), 0);
            wz[RING][N_] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(zr, (int)zo, (int)(gu * (uint32_t)a.N / 2u), 0);
        } else {
            wsc[RING][N_] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(wr, (int)so, (int)(a.scales_off + (gu >> 2) * 128u + (gu & 2) * 2), 0);
            wz[RING][N_] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(wr, (int)zo, (int)(a.zeros_off + (gu >> 2) * 32u), 0);
        }
    };
    auto to_vgpr = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_ds_bpermute(lane << 2, (int)v); };
    const uint32_t c_mlo = to_vgpr(a.m_lo), c_mhi = to_vgpr(a.m_hi), c_klo = to_vgpr(a.k_lo), c_khi = to_vgpr(a.k_hi);

    const float16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float16v tot[NT][TB], gacc[NT][TB];
    union BFrag { u32x4 u; half8 h; } bf[2][NT];
    float sc[NT];
    half2v nlo[NT], nhi[NT];
    uint32_t sp[NT];
    tile_for<NT>([&](auto N_) {
        sc[N_] = 0.f;
        tile_for<TB>([&](auto B) { tot[N_][B] = gacc[N_][B] = zero; });
    });
    // two channels of operand kk of tile n: part 0..3
    auto deq_piece = [&](int step, auto RING, auto N_, auto KK_, auto PART) {
        constexpr int ring = RING, n = N_, kk = KK_, part = PART;
        if constexpr (kk == 0 && part == 0) {
            const uint32_t g = tile_uniform(g0 + step * KW + kw);
            const uint32_t z = (wz[ring][n] >> (IC ? z_sh : z_sh + 4 * (g & 3))) & 15u;
            nlo[n] = tile_h2((0xE400u + z) * 0x00010001u);              // -(1024 + z), twice
            if constexpr (!IC) nhi[n] = tile_h2((0xD400u + (z << 4)) * 0x00010001u);    // -(64 + z), twice
        }
        const uint32_t u = wq[ring][n][kk / 4][kk % 4];
        if constexpr (IC) {
            if constexpr (part == 0) { const uint32_t x = u & 0xffffu; sp[n] = x | (x << 12); }
            if constexpr (part == 2) { const uint32_t x = u >> 16; sp[n] = x | (x << 12); }
            bf[kk & 1][n].u[part] = tile_u32(tile_h2(((part & 1 ? sp[n] >> 8 : sp[n]) & c_mlo) | c_klo) + nlo[n]);
        } else {
            const uint32_t v = part < 2 ? u : u >> 8;
            if constexpr (part & 1) bf[kk & 1][n].u[part] = tile_u32(tile_h2((v & c_mhi) | c_khi) + nhi[n]);
            else bf[kk & 1][n].u[part] = tile_u32(tile_h2((v & c_mlo) | c_klo) + nlo[n]);
        }
    };
    auto take_scale = [&](int step, auto RING, auto N_) {
        const uint32_t g = tile_uniform(g0 + step * KW + kw);
        union { uint16_t u; _Float16 h; } c; c.u = (uint16_t)(wsc[RING][N_] >> (IC ? 16 * (ft & 1) : 16 * (g & 1)));
        sc[N_] = (float)c.h;
    };
    using I0 = std::integral_constant<int, 0>;

    // ---- prologue ----
    tile_for<8>([&](auto I) { request_x(0, 0, I); __builtin_amdgcn_sched_barrier(0); });
    tile_for<2>([&](auto U) {
        tile_for<NT>([&](auto N_) { load_w(U, U, N_, I0{}); __builtin_amdgcn_sched_barrier(0); });
        tile_for<NT>([&](auto N_) { load_w(U, U, N_, std::integral_constant<int, 1>{}); load_sz(U, U, N_); __builtin_amdgcn_sched_barrier(0); });
    });
    tile_wait_vm<8>();                               // the first step's
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    tile_for<3>([&](auto I) { request_x(1, 1, I); });
    tile_for<TB>([&](auto B) { read_x(0, B, I0{}); });
    tile_for<NT>([&](auto N_) { tile_for<4>([&](auto P) { deq_piece(0, I0{}, N_, I0{}, P); }); });

    auto multiply = [&](int step, auto U) {
        constexpr int ring = U;
        tile_for<KK>([&](auto KK_) {
            constexpr int kk = KK_, nk = (kk + 1) % KK, nring = kk == KK - 1 ? ring ^ 1 : ring;
            using NK = std::integral_constant<int, nk>; using NRing = std::integral_constant<int, nring>;
            tile_for<4>([&](auto SL) {
                constexpr int s = SL, n = s / TB, tb = s % TB;
                if constexpr (kk == 0)
                    if (step <= n_own) tot[n][tb] += sc[n] * gacc[n][tb];      // of the group before
                gacc[n][tb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[kk & 1][tb], bf[kk & 1][n].h, kk == 0 ? zero : gacc[n][tb], 0, 0, 0);
                if constexpr (kk == KK - 1 && s == 1) {
                    // the next step's rows are in LDS, this wave's by the count (two weight requests are younger),
                    // the others' by the barrier, behind which this step's buffer is free, too
                    __builtin_amdgcn_s_waitcnt(0xc07f);
                    tile_wait_vm<2>();
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                }
                constexpr int rs = kk == KK - 1 ? s - 1 : s;
                if constexpr (rs >= 0 && rs < TB) read_x(nring, std::integral_constant<int, (rs >= 0 && rs < TB ? rs : 0)>{}, NK{});
                tile_for<2>([&](auto P) { deq_piece(nk ? step : step + 1, NRing{}, std::integral_constant<int, s / 2>{}, NK{}, std::integral_constant<int, s % 2 * 2 + P>{}); });
                constexpr int xi = kk == KK - 1 ? s - 1 : kk == 0 ? s + 3 : kk == 1 && s == 0 ? 7 : -1;      // the first three behind the barrier of the step before
                if constexpr (xi >= 0) request_x(kk == KK - 1 ? step + 2 : step + 1, kk == KK - 1 ? ring : ring ^ 1, std::integral_constant<int, (xi >= 0 ? xi : 0)>{});
                if constexpr (kk == 3 && s < NT) load_w(step + 2, U, std::integral_constant<int, s % NT>{}, I0{});
                if constexpr (kk == KK - 2 && s < NT) take_scale(step, U, std::integral_constant<int, s % NT>{});
                if constexpr (kk == KK - 1 && s >= 2) {
                    load_w(step + 2, U, std::integral_constant<int, s % NT>{}, std::integral_constant<int, 1>{});
                    load_sz(step + 2, U, std::integral_constant<int, s % NT>{});
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    // Whole pairs of steps (an exit inside the loop would join the requests of two histories at its head).  Requests beyond the
    // last group or token are out of range and fetch nothing.  What then stands in LDS is multiplied but reaches no stored sum:
    // tokens are rows of the product, and the sums of a group that does not exist are not added.
    int steps_run = 0;
    for (int step = 0; step < n_steps; step += 2) {
        multiply(step, I0{});
        multiply(step + 1, std::integral_constant<int, 1>{});
        steps_run = step + 2;
    }
    if (steps_run <= n_own)
        tile_for<NT>([&](auto N_) { tile_for<TB>([&](auto B) { tot[N_][B] += sc[N_] * gacc[N_][B]; }); });

    // ---- epilogue: of the two waves of a 64 x 64 tile each gives away 32 tokens and finishes the others.  A lane holds output
    // lane % 32 of tokens 8 (r / 4) + 4 half + r % 4 ------------------------------------------------------------------
    tile_wait_vm<0>();                               // nothing is on its way into the ring any more
    __syncthreads();
    float16v own[NT];
    float4v *const sums = (float4v *)s_x;
    auto exchange = [&](auto OWN) {
        tile_for<NT>([&](auto N_) {
            own[N_] = tot[N_][OWN];
            const float16v &v = tot[N_][1 - OWN];
            tile_for<4>([&](auto R) { sums[((wave * NT + N_) * 4 + R) * 64 + lane] = float4v{v[(int)R * 4], v[(int)R * 4 + 1], v[(int)R * 4 + 2], v[(int)R * 4 + 3]}; });
        });
    };
    if (kw == 0) exchange(I0{});
    else exchange(std::integral_constant<int, 1>{});
    __syncthreads();
    if (n_rows <= 0) return;
    const int r0 = mw * 64 + kw * 32, other = wave ^ (NW * MW);
    tile_for<NT>([&](auto N_) {
        tile_for<4>([&](auto R) {
            const float4v v = sums[((other * NT + N_) * 4 + R) * 64 + lane];
            tile_for<4>([&](auto E) { own[N_][(int)R * 4 + E] += v[(int)E]; });
        });
    });
    if (a.partial) {
        const __amdgpu_buffer_rsrc_t pr = tile_partials(a, kslice, m0, rows);
        tile_for<NT>([&](auto N_) {
            if (N_ * 32 + r32 < n_rows)
                tile_for<16>([&](auto E) {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(own[N_][(int)E]), pr, ((r0 + half * 4 + E / 4 * 8 + E % 4) * a.N + n0 + N_ * 32 + r32) * 4, 0, kAuxThrough);
                });
        });
        return;
    }
    // 32 x 64 through a wave-private part of LDS (rows padded by 16 bytes), out as 16-byte stores, eight of them a line
    constexpr int kRow = 72;
    _Float16 *const strip = (_Float16 *)(s_x + kTile2Stage) + wave * (32 * kRow);
    const __amdgpu_buffer_rsrc_t yr = tile_outputs(a, m0, rows);
    const bool through = (((uintptr_t)a.Y | (uintptr_t)(a.ldy * 2)) & 127) == 0;
    tile_for<NT>([&](auto N_) {
        const float bv = a.bias && N_ * 32 + r32 < n_rows ? (float)a.bias[n0 + N_ * 32 + r32] : 0.f;
        tile_for<16>([&](auto E) { strip[(half * 4 + E / 4 * 8 + E % 4) * kRow + N_ * 32 + r32] = (_Float16)(own[N_][(int)E] + bv); });
    });
    __builtin_amdgcn_wave_barrier();
    const int ocol = (lane & 7) * 8;
    tile_for<4>([&](auto H) {
        const int orow = H * 8 + (lane >> 3);
        const u32x4 o = *(const u32x4 *)(strip + orow * kRow + ocol);
        if (ocol < n_rows) tile_store(through, o, yr, ((r0 + orow) * (int)a.ldy + n0 + ocol) * 2);
    });
}

// MW: 64-token parts of the tile; WIDE: 64 x 64 per wave (two parts)
template <int MW, bool WIDE, bool IC>
static hipError_t launch_tile_cfg(TileArgs &a, hipStream_t s)
{
    constexpr auto kernel = WIDE ? linear_tile2_kernel<IC> : linear_tile_kernel<MW, IC>;
    constexpr int tm = 64 * MW, lds = WIDE ? kTile2Lds : 2 * kTileBuf;
    a.m_tiles = (a.T + tm - 1) / tm; a.n_tiles = (a.N + 127) / 128;
    const unsigned blocks = (unsigned)(((size_t)a.m_tiles * a.n_tiles * a.k_split + 7) / 8 * 8);
    static std::atomic<uint64_t> attr_done{0};
    if (const int dev = once_pending(attr_done); dev >= 0) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        once_done(attr_done, dev);
    }
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kTileThreads), lds, s, a);
    return hipGetLastError();
}

// 128-token tiles with fewer groups per block than this keep 64 x 32 per wave: a block of the wide kernel begins slower and takes
// groups in fours.  us, narrow / wide: 512 channels 9.1 / 10.2 (-> 16384 at 200 tokens), 1024 13.3 / 13.7, 1536 17.5 / 17.7 (but
// 17.2 / 16.9 -> 17424 at 105, a tie over 12 shapes), 2048 21.9 / 21.6 (and 1 to 5 % on 7 of 8 others); interchange layout,
// 256 -> 16400 at 300 tokens 13.3 / 18.7, 640 -> 16384 at 512 21.9 / 25.8, 1152 -> 12304 at 129 15.8 / 16.9, 1408 -> 17424 a tie.
constexpr int kTileWideGroups = 12;

// Which tile, and how many slices of K: the least of a cost model fitted to 521 timings with either forced (13 shapes, 80 to 900
// tokens; 4 and 5 % off in the mean, the choice costs 0.2 % over the best, 5 % at most): a fixed time, per round of 256 blocks
// the first requests and the stores, and the steps, longer where the blocks fill the chip; for split K the summing launch and
// the partial tiles.  128-token tiles take 0.8 of the time per token, but their blocks are longer and begin slower: 4096 -> 28672
// at 128 tokens 39 us against 47, 4096 -> 4096 at 201 tokens 21.5 against 18.8.  128-token tiles of few groups: 24 shapes of the
// interchange layout in one to five rounds, 2 % off.
struct TilePlan { bool two_m; int k_split, groups_per_split; double est_us, fit_us; };
static size_t tile_partial_bytes(int k_split, int T, int c_out) { return k_split > 1 ? (size_t)k_split * T * c_out * sizeof(float) : 0; }

// room: bytes for partial tiles; what needs more is not planned.  (Bare calls on interchange weights have none: unsplit with the
// tile that was best for the split, 13696 -> 1936 at 757 tokens takes 106 us, with the one that is best unsplit 63; 18 such
// calls 0.54 to 0.70 of the time.)
static TilePlan plan_tile(int c_in, int c_out, int T, bool interchange, size_t room)
{
    struct Fit { double call, round, step, step_full, sum, slice, mb; };
    // est_us stays the model that the lines to the other kernels were fitted with (low by up to 2 us on few steps, high by up to a
    // fifth on 128-token tiles): the GEMM rounds the weights to fp16, and no call is to lose precision.  Where neither model's choice
    // has room, the kernel with fewer slices is as slow as the others, and they stay.
    double lines_us = 1e30, least_us = 1e30;
    bool line_fits = false, least_fits = false;
    // The interchange layout costs 14 instead of 9 instructions per 8 weights, more of a step of the wide kernel (80 shapes with either
    // forced, 3 % off; priced as repacked weights 5888 -> 16944 at 464 tokens took 162 us in 128-token tiles instead of 157).
    static const Fit fits[2][2] = {{{1.7, 3.8, 0.94, 1.04, 1.3, 0.27, 0.151}, {3.0, 4.2, 1.49, 1.71, 0.5, 0.245, 0.189}},
                                   {{2.0, 3.36, 1.04, 1.12, 1.3, 0.27, 0.151}, {0.5, 4.9, 1.88, 1.96, 0.5, 0.245, 0.189}}};
    TilePlan best{false, 1, 0, 1e30, 1e30};
    const int G = c_in / kGroup, n_tiles = (c_out + 127) / 128;
    for (int two = 0; two <= (T > 64 ? 1 : 0); ++two) {
        const Fit &f = fits[interchange][two];
        const int m_tiles = (T + (two ? 127 : 63)) / (two ? 128 : 64);
        for (int ks = 1; ks <= 16 && (ks == 1 || (ks * 4 <= G && (long)m_tiles * n_tiles * ks <= 512)); ++ks) {
            const int gps = ((G + ks - 1) / ks + 3) / 4 * 4;             // whole steps, an even number of them
            if ((G + gps - 1) / gps != ks) continue;
            // Not the 8 groups of 1024 channels, which are two pairs of steps: the model takes both for equal, but in two slices
            // they take 8.4 us instead of 8.1 (69 to 126 tokens, 128 to 208 outputs); up to 64 outputs 7.0 to 7.9 instead of 7.8 to 8.0.
            if (ks > 1 && G == 8 && c_out > 64) continue;
            const bool fits_room = tile_partial_bytes(ks, T, c_out) <= room;
            const long blocks = (long)m_tiles * n_tiles * ks, rounds = ((blocks + 7) / 8 + 31) / 32;
            const int groups = std::min(G, gps);
            double us = two && groups < kTileWideGroups
                            ? 1.6 + (double)rounds * (3.5 + (groups + 1) / 2 * 2 * (blocks >= 160 ? 1.08 : 0.97))
                            : f.call + (double)rounds * (f.round + gps / 2 * (blocks >= 160 ? f.step_full : f.step));
            if (ks > 1) us += f.sum + f.slice * ks + (double)ks * T * c_out * 8.0e-6 * f.mb;
            if (us < least_us) { least_us = us; least_fits = fits_room; }
            if (fits_room && us < best.fit_us) best = TilePlan{two != 0, ks, gps, us, us};
            double line = 1.6 + (double)rounds * (3.5 + (two ? gps : gps / 2) * ((blocks >= 160 ? 1.09 : 0.96) - (two ? 0.04 : 0.0)));
            if (ks > 1) line += 1.7 + 0.23 * ks + (double)ks * T * c_out * 8.0 / 6.9e6;
            if (line < lines_us) { lines_us = line; line_fits = fits_room; }
        }
    }
    best.est_us = line_fits || least_fits ? lines_us : 1e30;
    return best;
}

double linear_tile_estimate_us(const paro_w4_weight &w, int T, size_t room) { return plan_tile(w.c_in, w.c_out, T, false, room).est_us; }
// whether a call on interchange weights that takes `us` elsewhere is faster there, by more than the two models are off
bool linear_tile_loses(const paro_w4_weight &w, int T, size_t room, double us)
{
    const TilePlan p = plan_tile(w.c_in, w.c_out, T, true, room);
    return us < (p.k_split > 1 ? 0.85 : 0.95) * p.fit_us;
}

size_t linear_tile_scratch_bytes(const paro_w4_weight &w, int T, bool interchange, size_t room)
{
    return tile_partial_bytes(plan_tile(w.c_in, w.c_out, T, interchange, room).k_split, T, w.c_out);
}

void linear_tile_plan(const paro_w4_weight &w, int T, bool interchange, size_t room, int &tokens, int &k_slices)
{
    const TilePlan p = plan_tile(w.c_in, w.c_out, T, interchange, room);
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
    const TilePlan p = plan_tile(w.c_in, w.c_out, T, interchange, scratch && ((uintptr_t)scratch % 16) == 0 ? scratch_bytes : 0);
    TileArgs a;
    a.w = interchange ? (const char *)w.qweight : (const char *)w.packed;
    a.scales_off = (uint32_t)packed_tiles_bytes(w.c_in, w.c_out);
    a.zeros_off = a.scales_off + (uint32_t)packed_scales_bytes(w.c_in, w.c_out);
    a.scales = (const _Float16 *)w.scales; a.qzeros = w.qzeros;
    a.X = (const _Float16 *)X; a.ldx = ldx; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.G = w.c_in / kGroup;
    a.m_lo = 0x000F000Fu; a.m_hi = 0x00F000F0u; a.k_lo = 0x64006400u; a.k_hi = 0x54005400u;
    a.k_split = p.k_split; a.groups_per_split = p.groups_per_split;
    a.partial = p.k_split > 1 ? (float *)scratch : nullptr;
    const bool wide = p.two_m && std::min(a.G, p.groups_per_split) >= kTileWideGroups;
    const hipError_t e = interchange ? (wide      ? launch_tile_cfg<2, true, true>(a, s)
                                        : p.two_m ? launch_tile_cfg<2, false, true>(a, s)
                                                  : launch_tile_cfg<1, false, true>(a, s))
                                     : (wide      ? launch_tile_cfg<2, true, false>(a, s)
                                        : p.two_m ? launch_tile_cfg<2, false, false>(a, s)
                                                  : launch_tile_cfg<1, false, false>(a, s));
    if (e != hipSuccess || p.k_split == 1) return e;
    return launch_splitk_reduce(a.partial, p.k_split, T, 0, w.c_out, w.bias, Y, ldy, least, s);
}

}  // namespace paro
