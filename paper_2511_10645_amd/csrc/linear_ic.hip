// W4A16 linear on weights in the interchange layout, up to 32 tokens, and up to 256 where that is the faster (Eq. 2): what a call
// runs on when the weight was not repacked, or has no repacked form because its input width is no multiple of 512 channels.
// (More: linear_tile.hip.)
//
// A block owns 16 NT outputs and all tokens (more than 32: up to 32 of them, as many blocks as it takes, all at once).  It walks its channels in stages of KG groups; KG consumer waves (times NCOL columns
// of NTW output tiles) take one group each, and their sums meet in LDS once at the end.  Everything goes from memory to LDS
// without passing through registers, and who requests what is split by latency, because a wave's requests complete in order:
// the producer wave requests only what comes from memory (codes, scales and zero points, RW stages deep), the consumers the
// activations, which every block reads and the L2 holds (XR stages deep).  One barrier per stage, behind which the operands of
// the next stage are read from LDS while this one is multiplied.
//
// A request of 64 lanes x 16 bytes covers whole rows of a stage (256 or 512 bytes of a weight row, 1 or 2 KB of a token), so that
// every four lanes ask for 64 consecutive bytes.  (Read straight into operand registers, where lane % 16 is the row, each lane is
// a request of its own: a quarter of the compute unit's rate, which bounded the kernel before.)  The 16-byte chunk index is
// XOR-ed with the row where it is requested, so that the operand reads are conflict-free.  The codes become q - z in fp16, exact;
// the group's scale multiplies the fp32 sums.
//
// Bound now by the instructions of a stage: 1 us per 8 groups of one tile, of which the codes' 14 instructions per 8 weights and
// the 8 operand reads are most; more waves or deeper rings change nothing (11 groups per consumer and no barrier, each with a
// ring of its own: 15.8 us for 11008 -> 4096 at 24 tokens against 14.6; requests two ahead instead of ten: the same).
// Measured, us, before -> now (graph replay over 350 MB of weights): 11008 -> 4096 at 24 tokens bare 36.8 -> 14.0, rotated
// 20.4 -> 17.4 (four slices of K), one token bare 19.3 -> 9.0; 2176 -> 4112 at 24 tokens bare 11.0 -> 6.3; 4224 -> 22016 32.3 -> 23;
// 106 random shapes: bare 0.60 of the time, rotated 0.80 in the geometric mean; many outputs on few channels: ic_few_channels.
// 33 tokens and more, tiled kernel -> this one: 9600 -> 2272 at 48 bare 45.9 -> 15.5, 11008 -> 4096 at 48 bare 53.0 -> 18.1, 4096 -> 4096 at 64
// bare 22.8 -> 9.2, rotated 18.2 -> 13.1, 1024 -> 208 at 128 bare 9.4 -> 4.3, 2816 -> 3440 at 256 bare 18.8 -> 18.3: linear_rows_pay.
#include "paro_internal.h"
#include <algorithm>
#include <cmath>
#include <iterator>
#include <type_traits>
#include <utility>

namespace paro {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void ic_lds_t;

constexpr uint32_t kOobI = 0x80000000u;             // beyond every buffer: nothing is fetched
template <int N> __device__ __forceinline__ void ic_wait_vm() { __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14)); }

__device__ inline __amdgpu_buffer_rsrc_t ic_rsrc(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}
__device__ inline half2v ic_h2(uint32_t u) { union { uint32_t u; half2v h; } c; c.u = u; return c.h; }
__device__ inline uint32_t ic_u32(half2v h) { union { uint32_t u; half2v h; } c; c.h = h; return c.u; }
__device__ inline uint32_t ic_uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

template <int N, class F, int I = 0>
__device__ __forceinline__ void ic_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        ic_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}

// until the requests of at most N stages, P each, are outstanding, or of the `left` stages that were requested at all
template <int P, int N> __device__ __forceinline__ void ic_wait_stages(int left)
{
    if constexpr (N == 0) ic_wait_vm<0>();
    else if (left >= N) ic_wait_vm<(N * P < 63 ? N * P : 63)>();
    else ic_wait_stages<P, N - 1>(left);
}

struct IcArgs {
    const char *w;                                   // qweight
    const _Float16 *scales;
    const uint32_t *qzeros;
    const _Float16 *X; int64_t ldx;
    _Float16 *Y; int64_t ldy;
    const _Float16 *bias;
    float *partial;                                  // [k slices][T][N] where K is split between blocks, else NULL
    int T, C, N, G, groups_per_split;
    uint32_t m_lo, k_lo;                             // 0x000F000F, 0x64006400: arguments, so that (u & m) | k is one instruction
    int pass_tokens;                                 // of a block where there are more than 32
};

constexpr int ic_wstage(int kg, int nt) { return kg * nt * 1024 + (kg * nt * 32 + 255) / 256 * 256 + 256; }  // codes | scales | zero points
constexpr int ic_lds(int kg, int consumers, int rpw, int nt, int xr, int rw) { return xr * consumers * rpw * (kg * 256) + rw * ic_wstage(kg, nt); }

// TB: blocks of 16 tokens; RPW: token rows that a consumer wave requests per stage; NCOL, NTW: see above; XR, RW: stages in the
// rings of activations and weights
// PASSES: more than 32 tokens, blockIdx.z has pass_tokens of them each (as a condition at run time it costs the others 0.1 us).
template <int TB, int RPW, int KG, int NCOL, int NTW, int XR, int RW, bool PASSES>
__global__ __launch_bounds__((KG * NCOL + 1) * 64) void linear_ic_kernel(IcArgs a)
{
    constexpr int NC = KG * NCOL, NT = NCOL * NTW, kXRow = KG * 256, kXStage = NC * RPW * kXRow, kWTile = KG * 1024, kWStage = ic_wstage(KG, NT);
    constexpr int kXReq = RPW * (KG / 4);            // requests of a consumer per stage
    constexpr int kScaleReq = (KG * NT + 7) / 8, kPer = KG * NT + kScaleReq + 1;         // requests of a stage of weights
    static_assert((KG == 4 || KG == 8) && (XR - 1) * kXReq < 64 && (RW - 2) * kPer < 64 && KG * TB * NT * 1024 <= XR * kXStage + RW * kWStage, "");
    static_assert((XR - 1) * kXStage + TB * 16 * kXRow <= XR * kXStage + RW * kWStage, "operand reads of rows beyond a stage stay in LDS");
    extern __shared__ __attribute__((aligned(16))) char s_ic[];
    char *const s_w = s_ic + XR * kXStage;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * 16 * NT, n_rows = min(a.N - n0, 16 * NT);          // multiple of 16
    const int g_lo = (int)blockIdx.y * a.groups_per_split, g_hi = min(a.G, g_lo + a.groups_per_split);
    const int t_lo = PASSES ? (int)blockIdx.z * a.pass_tokens : 0, T = PASSES ? min(a.T - t_lo, a.pass_tokens) : a.T;      // tokens of this block
    // Stage st is groups g_lo + KG st .. + KG - 1; a last stage of fewer is moved back to the last KG (those that were there
    // already are not multiplied again).
    const int n_grp = g_hi - g_lo, n_st = (n_grp + KG - 1) / KG, g_last = n_grp < KG ? 0 : n_grp - KG;
    auto stage_group = [&](int st) { return (uint32_t)min(KG * st, g_last); };     // from g_lo
    // chunk (16 bytes) c of row r lies at c ^ swz(r): a 16-byte read serves rows 0-3 and 12-15 of one quarter of a group and rows
    // 4-11 of the next together, then the others
    auto swz = [](int row) { return (row & 15) ^ ((row & 4) << 1); };
    const int ft = lane & 15, fkb = lane >> 4;
    const int kg = wave % KG, col = wave / KG;                                     // of a consumer
    float4v tot[TB][NTW];
    ic_for<TB>([&](auto B) { ic_for<NTW>([&](auto N_) { tot[B][N_] = float4v{0.f, 0.f, 0.f, 0.f}; }); });

    // Tokens beyond T and groups beyond a split of fewer than four are not fetched.  What stands in their place in LDS reaches no
    // stored sum: tokens are rows of the product, and such groups are not multiplied.
    if (wave == NC) {
        const __amdgpu_buffer_rsrc_t wr = ic_rsrc(a.w + (size_t)n0 * (a.C / 2), (size_t)n_rows * (a.C / 2));
        const __amdgpu_buffer_rsrc_t sr = ic_rsrc(a.scales, (size_t)a.G * a.N * 2);
        const __amdgpu_buffer_rsrc_t zr = ic_rsrc(a.qzeros, (size_t)a.G * a.N / 2);
        uint32_t wv[NT][KG], sv[kScaleReq], zv;
        ic_for<NT>([&](auto N_) {
            ic_for<KG>([&](auto I) {
                const int row = 16 / KG * I + lane / (4 * KG), c = lane % (4 * KG) ^ swz(row);
                wv[N_][I] = c < 4 * n_grp ? (uint32_t)((N_ * 16 < n_rows ? N_ * 16 : 0) + row) * (uint32_t)(a.C / 2) + g_lo * 64 + (c << 4) : kOobI;
            });
        });
        ic_for<kScaleReq>([&](auto I) {
            const uint32_t d = I * 64 + lane, gi = d / (8 * NT), r = d % (8 * NT);
            sv[I] = gi < (uint32_t)KG && (int)gi < n_grp ? ((g_lo + gi) * (uint32_t)a.N + n0) * 2 + r * 4 : kOobI;
        });
        zv = lane < 2 * KG * NT && lane / (2 * NT) < n_grp ? ((g_lo + lane / (2 * NT)) * (uint32_t)a.N + n0) / 2 + lane % (2 * NT) * 4 : kOobI;
        uint32_t slot = 0;
        auto request = [&](int st) {
            const uint32_t g = ic_uniform(stage_group(st));
            char *dst = s_w + slot;
            slot = slot == (RW - 1) * kWStage ? 0 : slot + kWStage;
            ic_for<NT>([&](auto N_) {
                ic_for<KG>([&](auto I) {
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (ic_lds_t *)(dst + N_ * kWTile + I * 1024), 16, (int)wv[N_][I], (int)(g * 64), 0, 0);
                });
            });
            ic_for<kScaleReq>([&](auto I) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, (ic_lds_t *)(dst + NT * kWTile + I * 256), 4, (int)sv[I], (int)(g * (uint32_t)a.N * 2), 0, 0);
            });
            __builtin_amdgcn_raw_ptr_buffer_load_lds(zr, (ic_lds_t *)(dst + kWStage - 256), 4, (int)zv, (int)(g * (uint32_t)a.N / 2), 0, 0);
        };
        for (int st = 0; st < RW && st < n_st; ++st) request(st);
        ic_wait_stages<kPer, RW - 1>(n_st - 1);
        __builtin_amdgcn_s_barrier();
        for (int st = 0; st < n_st; ++st) {
            ic_wait_stages<kPer, RW - 2>(n_st - 2 - st);     // stage st + 1 is in LDS
            __builtin_amdgcn_s_barrier();
            if (st + RW < n_st) request(st + RW);            // into the slot of stage st, which every wave has read
        }
    } else {
        const __amdgpu_buffer_rsrc_t xr = ic_rsrc(a.X + (size_t)t_lo * a.ldx, ((size_t)(T - 1) * a.ldx + a.C) * 2);
        uint32_t xv[kXReq];
        ic_for<kXReq>([&](auto I) {
            const int row = wave * RPW + I / (KG / 4), c = (I % (KG / 4) * 64 + lane) ^ swz(row);
            xv[I] = row < T && c < 16 * n_grp ? (uint32_t)(((size_t)row * a.ldx) * 2) + g_lo * 256 + (c << 4) : kOobI;
        });
        uint32_t slot = 0;
        auto request = [&](int st) {
            const uint32_t g = ic_uniform(stage_group(st));
            char *dst = s_ic + slot + wave * (kXReq * 1024);
            slot = slot == (XR - 1) * kXStage ? 0 : slot + kXStage;
            ic_for<kXReq>([&](auto I) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (ic_lds_t *)(dst + I * 1024), 16, (int)xv[I], (int)(g * 256), 0, 0);
            });
        };
        auto to_vgpr = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_ds_bpermute(lane << 2, (int)v); };
        const uint32_t c_m = to_vgpr(a.m_lo), c_k = to_vgpr(a.k_lo);
        int x_off[4];
        ic_for<4>([&](auto J) { x_off[J] = ft * kXRow + kg * 256 + (((fkb * 4 + J) ^ swz(ft)) << 4); });
        const int w_off = col * (NTW * kWTile) + ft * (KG * 64) + (((kg * 4 + fkb) ^ swz(ft)) << 4);
        const int s_off = NT * kWTile + kg * (NT * 32) + col * (NTW * 32) + ft * 2;
        const int z_off = kWStage - 256 + kg * (NT * 8) + col * (NTW * 8) + (ft >> 3) * 4, z_shift = 4 * (ft & 7);
        // the operands of a stage are read while the stage before it is multiplied
        struct Operands { half8 x[TB][4]; u32x4 w[NTW]; uint32_t z[NTW]; _Float16 s[NTW]; } op[2];
        uint32_t xslot = 0, wslot = 0;
        auto read = [&](Operands &o) {
            const char *xs = s_ic + xslot, *ws = s_w + wslot;
            xslot = xslot == (XR - 1) * kXStage ? 0 : xslot + kXStage;
            wslot = wslot == (RW - 1) * kWStage ? 0 : wslot + kWStage;
            ic_for<NTW>([&](auto N_) {
                o.w[N_] = *(const u32x4 *)(ws + w_off + N_ * kWTile);
                o.z[N_] = *(const uint32_t *)(ws + z_off + N_ * 8);
                o.s[N_] = *(const _Float16 *)(ws + s_off + N_ * 32);
            });
            ic_for<4>([&](auto J) { ic_for<TB>([&](auto B) { o.x[B][J] = *(const half8 *)(xs + x_off[J] + B * (16 * kXRow)); }); });
        };
        for (int st = 0; st < XR && st < n_st; ++st) request(st);
        ic_wait_stages<kXReq, XR - 1>(n_st - 1);
        __builtin_amdgcn_s_barrier();
        read(op[0]);
        for (int s0 = 0; s0 < n_st; s0 += 2)
            ic_for<2>([&](auto U) {
                const int st = s0 + U;
                if (st >= n_st) return;                      // (uniform; the last pass)
                ic_wait_stages<kXReq, XR - 2>(n_st - 2 - st);  // this wave's part of stage st + 1 is in LDS
                __builtin_amdgcn_s_waitcnt(0xc07f);          // stage st's operands have been read
                __builtin_amdgcn_s_barrier();
                if (st + XR < n_st) request(st + XR);        // into the slot of stage st
                read(op[1 - U]);
                __builtin_amdgcn_sched_barrier(0);
                const Operands &o = op[U];
                if ((int)stage_group(st) + kg >= KG * st && kg < n_grp)     // (uniform)
                    ic_for<NTW>([&](auto N_) {
                        const half2v nz = ic_h2((0xE400u + ((o.z[N_] >> z_shift) & 15u)) * 0x00010001u);  // -(1024 + z), twice
                        float4v acc[TB];
                        ic_for<4>([&](auto J) {
                            const uint32_t u = o.w[N_][(int)J], lo = u & 0xffffu, hi = u >> 16, a0 = lo | (lo << 12), a1 = hi | (hi << 12);
                            union { u32x4 u; half8 h; } b;   // codes 2 k and 2 k + 1 into the low nibbles of two halves
                            b.u[0] = ic_u32(ic_h2((a0 & c_m) | c_k) + nz);
                            b.u[1] = ic_u32(ic_h2(((a0 >> 8) & c_m) | c_k) + nz);
                            b.u[2] = ic_u32(ic_h2((a1 & c_m) | c_k) + nz);
                            b.u[3] = ic_u32(ic_h2(((a1 >> 8) & c_m) | c_k) + nz);
                            ic_for<TB>([&](auto B) {
                                const float4v zero = {0.f, 0.f, 0.f, 0.f};
                                acc[B] = __builtin_amdgcn_mfma_f32_16x16x32_f16(o.x[B][J], b.h, J == 0 ? zero : acc[B], 0, 0, 0);
                            });
                        });
                        ic_for<TB>([&](auto B) { tot[B][N_] += (float)o.s[N_] * acc[B]; });
                    });
                __builtin_amdgcn_sched_barrier(0);
            });
    }

    // ---- the consumers' sums; lane l of a 16 x 16 tile holds output l % 16 of tokens 4 (l / 16) .. + 3 ----------------
    __builtin_amdgcn_s_waitcnt(0x0070);              // no request is outstanding: the rings become [group][TB][NT][256] sums
    __syncthreads();
    float *s_sum = (float *)s_ic;
    if (wave < NC)
        ic_for<TB>([&](auto B) {
            ic_for<NTW>([&](auto N_) { *(float4v *)(s_sum + ((kg * TB + B) * NT + col * NTW + N_) * 256 + lane * 4) = tot[B][N_]; });
        });
    __syncthreads();
    for (int u = threadIdx.x; u < TB * NT * 64; u += (NC + 1) * 64) {
        const int tile = u >> 6, l = u & 63;
        const int n = tile % NT, t0 = tile / NT * 16 + (l >> 4) * 4;
        if (n * 16 >= n_rows) continue;
        float4v sum = *(const float4v *)(s_sum + u * 4);
#pragma unroll
        for (int w = 1; w < KG; ++w) sum += *(const float4v *)(s_sum + w * TB * NT * 256 + u * 4);
        const int o = n0 + n * 16 + (l & 15);
        if (a.partial) {
            float *dst = a.partial + ((size_t)blockIdx.y * a.T + t_lo + t0) * a.N + o;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + r < T) dst[(size_t)r * a.N] = sum[r];
        } else {
            const float bv = a.bias ? (float)a.bias[o] : 0.f;
            _Float16 *dst = a.Y + (size_t)(t_lo + t0) * a.ldy + o;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (t0 + r < T) dst[(size_t)r * a.ldy] = (_Float16)(sum[r] + bv);
        }
    }
}

// Tiles per block and slices of K by a model fitted to 106 random shapes (2 % off; the choice costs 0.3 % over the best): a block
// per compute unit and round, a fixed time and one per stage, which grows with the blocks that share the memory.  At 24 tokens,
// 4096 outputs, a stage of 8 groups of one tile takes 1.0 us, of 4 groups of two tiles 0.7, of four tiles 1.1.
struct IcPlan { int nt, k_split, groups_per_split; double us; };
constexpr int kIcMaxTokens = 256;
static int ic_passes(int T) { return (T + 31) / 32; }
static int ic_pass_tokens(int T) { return T <= 32 ? T : ((T + ic_passes(T) - 1) / ic_passes(T) + 7) / 8 * 8; }
static IcPlan ic_plan(int c_in, int c_out, int T, bool may_split)
{
    const int pass = ic_pass_tokens(T);
    struct Fit { int nt; double first, round, stage, busy; };
    static const Fit fits[3][4] = {                          // up to 8, 16, 32 tokens
        {{1, 1.13, 1.76, 0.476, 0.115}, {2, 1.84, 1.06, 0.480, -0.008}, {4, 0.65, 2.41, 0.721, 0.130}, {8, 1.94, 1.74, 1.249, 0.454}},
        {{1, 1.44, 1.51, 0.496, 0.318}, {2, 0.88, 2.11, 0.473, 0.163}, {4, 0.25, 2.97, 0.744, 0.356}, {0, 0, 0, 0, 0}},
        {{1, 1.71, 1.44, 0.604, 0.418}, {2, 1.33, 2.01, 0.525, 0.192}, {4, 1.17, 2.42, 0.809, 0.258}, {0, 0, 0, 0, 0}},
    };
    const int G = c_in / kGroup;
    IcPlan best{1, 1, G, 1e30};
    for (const Fit &f : fits[pass <= 8 ? 0 : pass <= 16 ? 1 : 2])
        for (int ks = 1; f.nt && ks <= (may_split ? 4 : 1); ++ks) {
            const int gps = (G + ks - 1) / ks, kg = f.nt == 1 ? 8 : 4, stages = (gps + kg - 1) / kg;
            if ((G + gps - 1) / gps != ks) continue;
            const double blocks = (double)((c_out + 16 * f.nt - 1) / (16 * f.nt)) * ks * ic_passes(T);
            double us = f.first + std::ceil(blocks / 256) * (f.round + stages * (f.stage + f.busy * std::min(blocks, 256.0) / 256));
            if (ks > 1) us += 2.0 + 0.14e-6 * 8.0 * ks * T * c_out;          // the summing launch; partial tiles written and read
            if (us < best.us) best = IcPlan{f.nt, ks, gps, us};
        }
    return best;
}

size_t linear_rows_scratch_bytes(const paro_w4_weight &w, int T)
{
    const IcPlan p = ic_plan(w.c_in, w.c_out, T, true);
    return p.k_split > 1 ? (size_t)p.k_split * T * w.c_out * sizeof(float) : 0;
}

// scales as dwords; row offsets of a block and the whole code array in 31 bits
bool linear_rows_supported(const paro_w4_weight &w, int64_t ldx, int T)
{
    return w.qweight && w.scales && w.qzeros && ((uintptr_t)w.scales % 4) == 0 && T <= kIcMaxTokens && (size_t)T * ldx * 2 < (1ull << 31) &&
           (size_t)w.c_out * (w.c_in / 2) < (1ull << 31);
}

// Where the kernel of linear_rows.hip, whose small blocks share a compute unit, is the faster one: few channels and more outputs than
// one round of blocks has, or two stages of which one is nearly empty.  us, it / this kernel, bare, 301 shapes: 512 -> 39280 at 2 tokens
// 8.2 / 9.7, 1024 -> 43280 at 4 9.7 / 14.2, 128 -> 49216 at 10 6.8 / 11.8, 640 -> 19072 at 16 7.1 / 8.8, 768 -> 18240 at 4 6.7 / 7.3,
// 384 -> 51168 at 25 13.7 / 15.1; but 256 -> 31184 at 3 (one round) 6.0 / 5.4, 1152 -> 26784 at 24 12.6 / 12.6; the choice costs 0.6 %
// over the better one (at most 13 %: 1152 -> 24672 at 2 tokens 8.5 / 9.6, 3200 -> 24112 at 10 17.9 / 20.2).
static bool ic_few_channels(const IcPlan &p, int c_in, int c_out, int T)
{
    const int G = c_in / kGroup;
    const bool rounds = c_out > 256 * 16 * p.nt;
    if (p.k_split > 1) return false;
    if (T > 16) return G <= 3 && rounds;
    return G <= 20 && (rounds || (T <= 8 && G > 4 && G <= 8 && c_out >= 8192));
}

// 16, 32, 64 outputs per block x up to 8, 16, 24, 32 tokens, and 128 outputs up to 8 tokens: the template's arguments
struct IcConfig { int tb, rpw, kg, ncol, ntw, xr, rw; };
constexpr IcConfig kIcConfigs[] = {
    {1, 1, 8, 1, 1, 3, 7}, {1, 2, 8, 1, 1, 3, 6}, {2, 3, 8, 1, 1, 2, 6}, {2, 4, 8, 1, 1, 2, 3},
    {1, 1, 4, 2, 1, 3, 6}, {1, 2, 4, 2, 1, 4, 7}, {2, 3, 4, 2, 1, 4, 6}, {2, 4, 4, 2, 1, 3, 6},
    {1, 1, 4, 2, 2, 3, 3}, {1, 2, 4, 2, 2, 4, 5}, {2, 3, 4, 2, 2, 3, 4}, {2, 4, 4, 2, 2, 3, 3},
    {1, 1, 4, 2, 4, 3, 3},
};
static int ic_config(int nt, int T) { return nt == 8 ? 12 : (nt == 4 ? 8 : nt == 2 ? 4 : 0) + (T - 1) / 8; }

template <int I, bool PASSES>
static hipError_t launch_ic_cfg(const IcArgs &a, dim3 grid, hipStream_t s)
{
    constexpr IcConfig c = kIcConfigs[I];
    constexpr auto kernel = linear_ic_kernel<c.tb, c.rpw, c.kg, c.ncol, c.ntw, c.xr, c.rw, PASSES>;
    constexpr int lds = ic_lds(c.kg, c.kg * c.ncol, c.rpw, c.ncol * c.ntw, c.xr, c.rw);
    static_assert(lds <= 160 * 1024, "");
    static std::atomic<uint64_t> attr_done{0};
    if (const int dev = once_pending(attr_done); dev >= 0) {
        hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        once_done(attr_done, dev);
    }
    hipLaunchKernelGGL(kernel, grid, dim3((c.kg * c.ncol + 1) * 64), lds, s, a);
    return hipGetLastError();
}
template <size_t... I>
static hipError_t launch_ic(int config, const IcArgs &a, dim3 grid, hipStream_t s, std::index_sequence<I...>)
{
    static constexpr hipError_t (*launch[])(const IcArgs &, dim3, hipStream_t) = {launch_ic_cfg<I, false>...};
    static constexpr hipError_t (*passes[])(const IcArgs &, dim3, hipStream_t) = {launch_ic_cfg<I, kIcConfigs[I].tb == 2>...};      // 17..32 tokens each
    return a.T > 32 ? passes[config](a, grid, s) : launch[config](a, grid, s);
}

// the plan of a call with this much room for partial tiles
static IcPlan ic_plan_in(const paro_w4_weight &w, int T, size_t room)
{
    const IcPlan p = ic_plan(w.c_in, w.c_out, T, true);
    return p.k_split == 1 || (size_t)p.k_split * T * w.c_out * sizeof(float) <= room ? p : ic_plan(w.c_in, w.c_out, T, false);
}

// More than 32 tokens: where blocks of up to 32 tokens, all at once, take less than the tiled kernel in the room there is for partial tiles.
// That one's blocks are 64 tokens x 128 outputs, few where the outputs are, and walk all of K one after the other; here every 32 tokens read the
// weights once more and the codes are unpacked again, which loses where the blocks fill several rounds: 256 -> 5840 at 256 tokens bare
// 7.6 / 11.3 us, 4224 -> 9408 at 200 42 / 56.  Both by their models, with a margin of 5 % (15 % where the tiled kernel splits K): 309 calls of
// 33 to 256 tokens, 256 to 15000 channels, 16 to 24000 outputs take 0.64 of the time, within 1 % of the better of the two in the mean; none slower.
bool linear_rows_pay(const paro_w4_weight &w, int64_t ldx, int T, size_t room)
{
    return linear_rows_supported(w, ldx, T) && (T <= 32 || !linear_tile_supported(w, true) || linear_tile_loses(w, T, room, ic_plan_in(w, T, room).us));
}

void linear_rows_plan(const paro_w4_weight &w, int T, size_t room, int &outputs, int &k_slices, int &config, int &stages, int &ring)
{
    const IcPlan p = ic_plan_in(w, T, room);
    k_slices = p.k_split; outputs = 0; config = -1; stages = ring = 0;
    if (T <= 32 && ic_few_channels(p, w.c_in, w.c_out, T)) return;
    outputs = 16 * p.nt; config = ic_config(p.nt, ic_pass_tokens(T));
    const IcConfig c = kIcConfigs[config];
    stages = (p.groups_per_split + c.kg - 1) / c.kg; ring = std::max(c.xr, c.rw);
}

hipError_t launch_linear_rows(const paro_w4_weight &w, const paro_half_t *X, int64_t ldx, paro_half_t *Y, int64_t ldy, int T,
                              void *scratch, size_t scratch_bytes, const void *least, hipStream_t s)
{
    const IcPlan p = ic_plan_in(w, T, scratch && ((uintptr_t)scratch % 16) == 0 ? scratch_bytes : 0);
    const bool split = p.k_split > 1;
    if (T <= 32 && ic_few_channels(p, w.c_in, w.c_out, T)) return launch_linear_direct(w, X, ldx, Y, ldy, T, s);
    IcArgs a;
    a.w = (const char *)w.qweight; a.scales = (const _Float16 *)w.scales; a.qzeros = w.qzeros;
    a.X = (const _Float16 *)X; a.ldx = ldx; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.partial = split ? (float *)scratch : nullptr;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.G = w.c_in / kGroup; a.groups_per_split = p.groups_per_split;
    a.pass_tokens = ic_pass_tokens(T);
    a.m_lo = 0x000F000Fu; a.k_lo = 0x64006400u;
    const dim3 grid((w.c_out + 16 * p.nt - 1) / (16 * p.nt), p.k_split, ic_passes(T));
    const hipError_t e = launch_ic(ic_config(p.nt, a.pass_tokens), a, grid, s, std::make_index_sequence<std::size(kIcConfigs)>{});
    if (e != hipSuccess || !split) return e;
    return launch_splitk_reduce(a.partial, p.k_split, T, 0, w.c_out, w.bias, Y, ldy, least, s);
}

}  // namespace paro
