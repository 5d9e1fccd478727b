// W4A16 linear in which every wave is on its own until its sums are complete (Eq. 2), in two forms:
//   - repacked weights with activations in operand order, 33 to 256 tokens, where the outputs are few: a rotation pass can
//     write its result in any order, and writes it in this one (rotate.hip) where this kernel follows;
//   - weights in the interchange layout on row-major activations, up to 32 tokens, where the outputs are many and the channels few
//     (the others: linear_ic.hip, which chooses).
//
// A block is 4 waves and owns (16 TB tokens) x (16 NT outputs); its waves take the channel groups in turn (wave w: groups
// w, w + 4, ...), so that every weight and every activation enters the compute unit once and the loop has no LDS, no
// barrier and no hand-over:
//   - weights: a lane's 16 bytes of a row's group are 32 channels of that row, which is the B operand of four
//     v_mfma_f32_16x16x32_f16 once the codes stand in fp16 registers as q - z (exact; 14 vector instructions per 8
//     weights in the natural code order, 9 in the repacked one); the group's scale multiplies the fp32 sums;
//   - activations straight into fragment registers: in operand order a fragment is one contiguous kilobyte, of row-major
//     rows it is 16-byte pieces of 32 cache lines, each a request of its own, which matters less the fewer the tokens are;
//   - registers are a ring of two groups: a register is refilled for the group after next right after its last use.
// The loop is written as slots, one MFMA each, with a piece of the next tile's dequantisation, a piece of the previous
// tile's scaling and at most two loads in its shadow, pinned by scheduling barriers.  The 4 waves' sums meet in LDS once;
// K is also split between blocks where the outputs alone are too few of them (operand order).
//
// Bound by the weight stream and, at few groups per wave, by the chain load -> dequantise -> multiply -> sum; at more
// tokens by what a compute unit takes in (a block reads all channels of its 32 tokens, 256 KB at 4096), hence
// only where the outputs are few and K is not long (14336 -> 4096 at 64 tokens: 27.0 against 24.5 us in linear_tile.hip).
// Whole rotated calls in a replayed graph over 350 MB of weights, us (before: row-major activations into linear_tile.hip, mostly
// with split K and its summing launch), 64 tokens: 4096 -> 4096 16.8, now 10.7; 4096 -> 6144 18.6, now 14.1; 128 tokens:
// 19.7, now 14.9; 23.3, now 20.5.
#include "paro_internal.h"
#include <type_traits>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRowsWaves = 4, kRowsTiles = 4;       // waves per block (K in turn); 16-output tiles per block (interchange layout)
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
    const char *w;                                   // qweight, or the repacked blob
    uint32_t scales_off, zeros_off;                  // of the blob
    const _Float16 *scales;                          // interchange layout
    const uint32_t *qzeros;
    const _Float16 *X; int64_t ldx;                  // row-major, or (OPERAND) blocks of 16 tokens x 128 channels
    _Float16 *Y; int64_t ldy;
    const _Float16 *bias;
    float *partial;                                  // [k slices][T][N] where K is split between blocks, else NULL
    int T, C, N, G, m_tiles, n_tiles, k_split, groups_per_split;
    uint32_t m_lo, m_hi, k_lo, k_hi;                 // 0x000F000F, 0x00F000F0, 0x64006400, 0x54005400: arguments, so that
};                                                   // (u & m) | k is one instruction

// TB: blocks of 16 tokens per block; NT: tiles of 16 outputs; OPERAND: the second form above.  Activations in operand order:
// a block of r = 16 tokens (the last one: of those that are left) x one group is [4 fragments j][4 kb][r tokens][16 B],
// channels 32 kb + 8 j .. + 7.
// WHOLE: every block of 16 tokens of this tile is whole, so that its strides are constants (with strides in registers, as a
// ragged last tile has them, 4096 -> 4096 at 64 tokens takes 0.1 to 0.2 us more).
template <int TB, int NT, bool OPERAND, bool WHOLE>
__device__ __forceinline__ void linear_rows_tile(const RowsArgs &a, float *s_sum, int kslice, int mt, int ntile)
{
    constexpr int R = 2;                             // ring of groups
    constexpr int S = 4 * TB;                        // slots (MFMAs) per tile
    constexpr int P = 16 / S;                        // dequantisation pieces per slot
    static_assert(NT % 2 == 0 && (TB == 1 || TB == 2), "");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = (int)rows_uniform(mt * 16 * TB), n0 = (int)rows_uniform(ntile * 16 * NT);
    const int m_rows = min(a.T - m0, 16 * TB);
    const int n_rows = min(a.N - n0, 16 * NT);       // multiple of 16
    const int g_end = min(a.G, (int)rows_uniform((kslice + 1) * a.groups_per_split));
    const int g_first = (int)rows_uniform(kslice * a.groups_per_split) + wave;
    const int n_grp = g_first < g_end ? (g_end - g_first + kRowsWaves - 1) / kRowsWaves : 0;   // of this wave
    const int ft = lane & 15, fkb = lane >> 4;

    // ---- addresses: a per-lane offset that is fixed (or out of range) plus a wave-uniform one -----------------------
    const int n_tb = (m_rows + 15) / 16;
    const __amdgpu_buffer_rsrc_t xr = OPERAND ? rows_rsrc((const char *)a.X + (size_t)m0 * a.C * 2, (size_t)m_rows * 2 * a.C)
                                              : rows_rsrc(a.X, ((size_t)(a.T - 1) * a.ldx + a.C) * 2);
    const __amdgpu_buffer_rsrc_t wr = OPERAND ? rows_rsrc(a.w, a.zeros_off + packed_zeros_bytes(a.C, a.N))
                                              : rows_rsrc(a.w + (size_t)n0 * (a.C / 2), (size_t)n_rows * (a.C / 2));
    const __amdgpu_buffer_rsrc_t sr = rows_rsrc(a.scales, OPERAND ? 0 : (size_t)a.G * a.N * 2);
    const __amdgpu_buffer_rsrc_t zr = rows_rsrc(a.qzeros, OPERAND ? 0 : (size_t)a.G * a.N / 2);
    uint32_t xv[TB], x_base[TB], x_rows[TB];         // per lane, and per block of 16 tokens (surplus blocks repeat the first)
    rows_for<TB>([&](auto B) {
        x_base[B] = OPERAND ? rows_uniform(B < n_tb ? B * 32u * (uint32_t)a.C : 0u) : 0u;
        x_rows[B] = !OPERAND ? 1u : WHOLE ? 16u : rows_uniform((uint32_t)min(16, B < n_tb ? m_rows - B * 16 : m_rows));
        if constexpr (!OPERAND) xv[B] = B * 16 + ft < a.T ? (uint32_t)(((size_t)(B * 16 + ft) * a.ldx + fkb * 32) * 2) : kOobR;
        else if constexpr (WHOLE) xv[B] = lane * 16u;
        else xv[B] = (uint32_t)ft < x_rows[B] ? __umul24(fkb * 16u, x_rows[B]) + ft * 16u : kOobR;
    });
    constexpr uint32_t kXGroup = kGroup * 2, kXFrag = OPERAND ? 64 : 16;             // per row of the block, or of the input
    const uint32_t wv = OPERAND ? lane * 16u : (uint32_t)ft * (uint32_t)(a.C / 2) + fkb * 16;
    // Whole dwords, shifted where they are used: a 16-bit load's extension would be waited for where it is loaded.  (The
    // wave's groups share g % 4 in the blob: they are kRowsWaves = 4 apart, and a split begins at a multiple of 4.)
    static_assert(kRowsWaves == kSliceGroups, "");
    const int g4 = g_first & 3;
    const uint32_t sv = OPERAND ? ft * 8u + (g4 & 2) * 2 : (ft & 14) * 2u, zv = OPERAND ? (ft & 14) * 2u : (ft >> 3) * 4u;
    const uint32_t s_shift = OPERAND ? 16 * (g4 & 1) : 16 * (ft & 1), z_shift = OPERAND ? 16 * (ft & 1) + 4 * g4 : 4 * (ft & 7);
    // tiles beyond N read the last one again: their sums are not stored
    uint32_t w_tile[NT], s_tile[NT];
    rows_for<NT>([&](auto N_) {
        const int n = min((int)N_, n_rows / kTileN - 1), tile = n0 / kTileN + n;
        w_tile[N_] = rows_uniform(OPERAND ? (uint32_t)tile * (uint32_t)a.G * 1024u : (uint32_t)n * 16u * (uint32_t)(a.C / 2));
        s_tile[N_] = rows_uniform(OPERAND ? (uint32_t)tile * (uint32_t)(a.G / kSliceGroups) : (uint32_t)(n0 + n * kTileN));
    });

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
        const uint32_t group = x_base[tb] + l_g * kXGroup * x_rows[tb], frag = j * kXFrag * x_rows[tb];
        if constexpr (OPERAND && !WHOLE) v.u = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)l_xv[tb], (int)(group + frag), 0);
        else v.u = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(l_xv[tb] + frag), (int)group, 0);
        xa[ring][tb][j] = v.h;
    };
    auto load_w = [&](int ring, int n) {
        if constexpr (OPERAND) {
            const uint32_t sl = s_tile[n] + (l_g >> 2);
            wq[ring][n] = __builtin_amdgcn_raw_buffer_load_b128(wr, (int)l_wv, (int)(w_tile[n] + l_g * 1024u), 0);
            wsc[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(wr, (int)l_sv, (int)(a.scales_off + sl * 128u), 0);
            wz[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(wr, (int)l_zv, (int)(a.zeros_off + sl * 32u), 0);
        } else {
            const uint32_t first = l_g * (uint32_t)a.N + s_tile[n];
            wq[ring][n] = __builtin_amdgcn_raw_buffer_load_b128(wr, (int)l_wv, (int)(w_tile[n] + l_g * 64u), 2);
            wsc[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(sr, (int)l_sv, (int)(first * 2u), 0);
            wz[ring][n] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(zr, (int)l_zv, (int)(first / 2u), 0);
        }
    };

    auto to_vgpr = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_ds_bpermute(lane << 2, (int)v); };
    const uint32_t c_mlo = to_vgpr(a.m_lo), c_mhi = to_vgpr(a.m_hi), c_klo = to_vgpr(a.k_lo), c_khi = to_vgpr(a.k_hi);

    float4v tot[TB][NT], gacc[2][TB];
    union BFrag { u32x4 u; half8 h; } bf[2][4];
    float sc[2] = {0.f, 0.f};
    half2v nlo = rows_h2(0), nhi = rows_h2(0);
    uint32_t sp = 0;                                 // codes 0, 2 (then 1, 3 eight bits higher) of a half word, spread
    rows_for<TB>([&](auto B) {
        rows_for<NT>([&](auto N_) { tot[B][N_] = float4v{0.f, 0.f, 0.f, 0.f}; });
        gacc[1][B] = float4v{0.f, 0.f, 0.f, 0.f};
    });
    // piece p (0..15) of the dequantisation of tile n in ring slot `ring` into bf[par]; the last piece also takes the
    // scale and refills the tile's registers (tile 0's are refilled in the next group's second slot)
    auto deq_piece = [&](auto PC, auto RING, auto N_, auto PAR) {
        constexpr int p = PC, w4 = p / 4, part = p % 4, ring = RING, n = N_, par = PAR;
        if constexpr (p == 0) {
            const uint32_t z = (wz[ring][n] >> z_shift) & 15u;
            nlo = rows_h2((0xE400u + z) * 0x00010001u);                      // -(1024 + z), twice
            if constexpr (OPERAND) nhi = rows_h2((0xD400u + (z << 4)) * 0x00010001u);    // -(64 + z), twice
        }
        const uint32_t u = wq[ring][n][w4];
        if constexpr (OPERAND) {
            const uint32_t v = part < 2 ? u : u >> 8;
            if constexpr (part & 1) bf[par][w4].u[part] = rows_u32(rows_h2((v & c_mhi) | c_khi) + nhi);
            else bf[par][w4].u[part] = rows_u32(rows_h2((v & c_mlo) | c_klo) + nlo);
        } else {
            // codes 2 part and 2 part + 1 into the low nibbles of the two halves
            if constexpr (part == 0) { const uint32_t x = u & 0xffffu; sp = x | (x << 12); }
            if constexpr (part == 2) { const uint32_t x = u >> 16; sp = x | (x << 12); }
            bf[par][w4].u[part] = rows_u32(rows_h2(((part & 1 ? sp >> 8 : sp) & c_mlo) | c_klo) + nlo);
        }
        if constexpr (p == 15) {
            union { uint16_t u; _Float16 h; } c; c.u = (uint16_t)(wsc[ring][n] >> s_shift);
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
            float *dst = a.partial + ((size_t)kslice * a.T + m0 + t0) * a.N + col;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + r < m_rows) dst[(size_t)r * a.N] = sum[r];
        } else {
            const float bv = a.bias ? (float)a.bias[col] : 0.f;
            _Float16 *dst = a.Y + (size_t)(m0 + t0) * a.ldy + col;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + r < m_rows) dst[(size_t)r * a.ldy] = (_Float16)(sum[r] + bv);
        }
    }
}

template <int TB, int NT, bool OPERAND>
__global__ __launch_bounds__(kRowsWaves * 64, 2) void linear_rows_kernel(RowsArgs a)
{
    __shared__ __attribute__((aligned(16))) float s_sum[kRowsWaves * TB * NT * 256];
    if constexpr (OPERAND) {
        // an XCD's blocks are a run of (K-slice, output tile, token tile), the last running fastest: its L2 serves a
        // weight tile to the further token tiles, and every XCD gets the same number of blocks
        const int tiles = a.m_tiles * a.n_tiles, all = tiles * a.k_split, per_xcd = (all + 7) / 8;
        const int idx = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
        if (idx >= all) return;
        const int mt = idx % tiles % a.m_tiles, ntile = idx % tiles / a.m_tiles;
        if (a.T % 16 == 0 || mt + 1 < a.m_tiles) linear_rows_tile<TB, NT, true, true>(a, s_sum, idx / tiles, mt, ntile);
        else linear_rows_tile<TB, NT, true, false>(a, s_sum, idx / tiles, mt, ntile);
    } else {
        linear_rows_tile<TB, NT, false, false>(a, s_sum, (int)blockIdx.y, 0, (int)blockIdx.x);
    }
}

// ---- interchange layout ------------------------------------------------------------------------------------------------
hipError_t launch_linear_direct(const paro_w4_weight &w, const paro_half_t *X, int64_t ldx, paro_half_t *Y, int64_t ldy, int T, hipStream_t s)
{
    RowsArgs a;
    a.w = (const char *)w.qweight; a.scales_off = a.zeros_off = 0; a.m_tiles = a.n_tiles = a.k_split = 0; a.scales = (const _Float16 *)w.scales; a.qzeros = w.qzeros;
    a.X = (const _Float16 *)X; a.ldx = ldx; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.G = w.c_in / kGroup; a.groups_per_split = a.G; a.partial = nullptr;
    a.m_lo = 0x000F000Fu; a.m_hi = 0x00F000F0u; a.k_lo = 0x64006400u; a.k_hi = 0x54005400u;
    const dim3 grid((w.c_out + 16 * kRowsTiles - 1) / (16 * kRowsTiles)), block(kRowsWaves * 64);
    if (T <= 16) hipLaunchKernelGGL((linear_rows_kernel<1, kRowsTiles, false>), grid, block, 0, s, a);
    else         hipLaunchKernelGGL((linear_rows_kernel<2, kRowsTiles, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

// ---- repacked weights, activations in operand order ---------------------------------------------------------------------
// Outputs per block and K split from a cost model fitted to 4226 timings (140 shapes, 33 to 256 tokens, activations already in
// operand order), 4 to 6 % off: per round of blocks over the chip a chain of steps (a group per wave each), the weight
// stream, what further blocks of the same compute unit add, and for split K the summing launch and the partial tiles.
// 32 outputs per block where they then fit one round (4096 -> 4096 at 64 tokens, linear alone: 6.9 us, 64 outputs 9.4); 64 beyond it, for
// every block reads all of its activations (4096 -> 28672: 33.4 against 40.3 us).
struct OperandPlan { int nt, k_split, groups_per_split; double est_us; };
static OperandPlan plan_operand(int c_in, int c_out, int T)
{
    OperandPlan best{4, 1, 0, 1e30};
    const int G = c_in / kGroup, m_tiles = (T + 31) / 32;
    const double mb = (double)c_in * c_out / 2.0e6;
    for (int nt = 2; nt <= 4; nt += 2) {
        const int n_tiles = (c_out + 16 * nt - 1) / (16 * nt);
        for (int ks = 1; ks <= 4 && (ks == 1 || (G >= ks * 8 && (long)m_tiles * n_tiles * ks <= 512)); ++ks) {
            const int gps = ((G + ks - 1) / ks + kRowsWaves - 1) / kRowsWaves * kRowsWaves;
            if ((G + gps - 1) / gps != ks) continue;
            const long blocks = (long)m_tiles * n_tiles * ks;
            const double rounds = (double)((blocks + 255) / 256), steps = (gps / kRowsWaves + 1) / 2 * 2;
            const double more = blocks > 256 ? (double)blocks / 256.0 - 1.0 : 0.0, part_mb = (double)ks * T * c_out * 8.0 / 1.0e6;
            double us = nt == 2 ? 2.74 + rounds * (0.21 + 0.40 * steps) + more * (0.28 + 0.057 * steps) + 0.108 * mb
                                : 3.82 + rounds * 0.637 * steps + more * (1.03 + 0.019 * steps) + 0.085 * mb;
            if (ks > 1) us += 2.0 + (nt == 2 ? 0.227 : 0.175) * part_mb;
            if (us < best.est_us) best = OperandPlan{nt, ks, gps, us};
        }
    }
    return best;
}

// 33 to 256 tokens (measured range; below, the streaming kernel hosts or follows the rotation), 31-bit byte offsets
bool linear_operand_supported(const paro_w4_weight &w, int T)
{
    return T > 32 && T <= 256 && linear_tile_supported(w, false) && (size_t)T * w.c_in * 2 < (1ull << 31);
}

// The time behind a rotation pass, where activations come from another compute unit's stores: the same model fitted to 3833
// rotated calls (649 shapes), 5 % off.  (plan_operand's ranks its own choices, but is 4 to 9 % low there.)
double linear_operand_estimate_us(const paro_w4_weight &w, int T)
{
    const OperandPlan p = plan_operand(w.c_in, w.c_out, T);
    const long blocks = (long)((T + 31) / 32) * ((w.c_out + 16 * p.nt - 1) / (16 * p.nt)) * p.k_split;
    const double rounds = (double)((blocks + 255) / 256), steps = (p.groups_per_split / kRowsWaves + 1) / 2 * 2;
    const double more = blocks > 256 ? (double)blocks / 256.0 - 1.0 : 0.0, mb = (double)w.c_in * w.c_out / 2.0e6;
    const double part_mb = p.k_split > 1 ? (double)p.k_split * T * w.c_out * 8.0 / 1.0e6 : 0.0;
    if (p.nt == 2) return 2.76 + rounds * (0.297 + 0.454 * steps) + 0.463 * more + 0.07 * mb + (p.k_split > 1 ? 2.34 + 0.345 * part_mb : 0.0);
    return 4.35 + 0.639 * rounds * steps + 1.09 * more + 0.076 * mb + (p.k_split > 1 ? 2.88 + 0.152 * part_mb : 0.0);
}

size_t linear_operand_scratch_bytes(const paro_w4_weight &w, int T)
{
    const OperandPlan p = plan_operand(w.c_in, w.c_out, T);
    return p.k_split > 1 ? (size_t)p.k_split * T * w.c_out * sizeof(float) : 0;
}

void linear_operand_plan(const paro_w4_weight &w, int T, int &outputs, int &k_slices)
{
    const OperandPlan p = plan_operand(w.c_in, w.c_out, T);
    outputs = 16 * p.nt; k_slices = p.k_split;
}

template <int NT>
static hipError_t launch_operand_nt(RowsArgs &a, hipStream_t s)
{
    a.m_tiles = (a.T + 31) / 32; a.n_tiles = (a.N + 16 * NT - 1) / (16 * NT);
    hipLaunchKernelGGL((linear_rows_kernel<2, NT, true>), dim3((unsigned)(a.m_tiles * a.n_tiles * a.k_split + 7) / 8 * 8),
                       dim3(kRowsWaves * 64), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_linear_operand(const paro_w4_weight &w, const paro_half_t *Xop, paro_half_t *Y, int64_t ldy, int T, void *scratch,
                                 size_t scratch_bytes, const void *least, hipStream_t s)
{
    const OperandPlan p = plan_operand(w.c_in, w.c_out, T);
    RowsArgs a;
    a.w = (const char *)w.packed;
    a.scales_off = (uint32_t)packed_tiles_bytes(w.c_in, w.c_out);
    a.zeros_off = a.scales_off + (uint32_t)packed_scales_bytes(w.c_in, w.c_out);
    a.scales = nullptr; a.qzeros = nullptr;
    a.X = (const _Float16 *)Xop; a.ldx = 0; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.G = w.c_in / kGroup;
    a.m_lo = 0x000F000Fu; a.m_hi = 0x00F000F0u; a.k_lo = 0x64006400u; a.k_hi = 0x54005400u;
    // the caller takes this kernel only where its partial tiles have room
    if (p.k_split > 1 && !(scratch && scratch_bytes >= (size_t)p.k_split * T * w.c_out * sizeof(float) && ((uintptr_t)scratch % 16) == 0)) return hipErrorInvalidValue;
    a.k_split = p.k_split; a.groups_per_split = p.groups_per_split;
    a.partial = p.k_split > 1 ? (float *)scratch : nullptr;
    const hipError_t e = p.nt == 2 ? launch_operand_nt<2>(a, s) : launch_operand_nt<4>(a, s);
    if (e != hipSuccess || p.k_split == 1) return e;
    return launch_splitk_reduce(a.partial, p.k_split, T, 0, w.c_out, w.bias, Y, ldy, least, s);
}

}  // namespace paro
