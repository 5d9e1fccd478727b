// Weight-activation form of the linear layer with both operands in MXFP4 (App. A.3, first equation):
//      Y' = Q(X T^-1) . Q(T W) + b
// on the block-scaled FP4 matrix instruction of this chip, which takes E2M1 codes and one E8M0 scale per
// 32 elements of each operand directly: nothing is dequantised, the codes go from memory to the matrix
// core as they are and the products are accumulated in fp32.
//
// v_mfma_scale_f32_16x16x128_f8f6f4 (FP4 x FP4): lane l of the A operand holds row l % 16, elements
// 32 (l / 16) .. + 31 of the 128-wide K-step as 16 bytes (element k in nibble k % 8 of dword k / 8), and
// ONE scale byte for those 32 elements - an MX block is exactly a lane's share; B likewise with column
// l % 16; D as for the other 16x16 shapes (lane: column l % 16, rows 4 (l / 16) + r).  The scale operand
// is a dword of which an immediate picks the byte, so one register serves four K-steps.
//
// Weights are repacked once into that operand order ("tiles" of 16 rows x 128 channels = 1 KB, then
// per 16 rows x 512 channels one dword per lane with the four K-steps' scale bytes), so a wave's load of
// a tile is one contiguous kilobyte.  Activations stay in the plain row order their quantiser writes:
// a lane's 32 elements are 16 contiguous bytes of its token's row.
//
// Two kernels.  Up to 64 tokens per pass: HBM-bound stream of the weight tiles (0.53 B per weight), one
// 512-channel slice per wave and pass, all slices of K inside one block (a wave takes SPW slices when
// there are more than 12), partial tiles summed through LDS; no exchange between blocks.  More tokens:
// a tiled GEMM (see below).
#include "paro_internal.h"
#include "tile_order.h"
#include <algorithm>
#include <type_traits>

namespace paro {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr uint32_t kOobM = 0x80000000u;
__device__ inline __amdgpu_buffer_rsrc_t mx_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
__device__ inline v8i as_operand(u32x4 v) { return v8i{(int)v[0], (int)v[1], (int)v[2], (int)v[3], 0, 0, 0, 0}; }

template <int N, class F, int I = 0>
__device__ __forceinline__ void mx_static_while(F &&f)
{
    if constexpr (I < N) {
        if (f(std::integral_constant<int, I>{})) mx_static_while<N, F, I + 1>(static_cast<F &&>(f));
    }
}
template <int N, class F, int I = 0>
__device__ __forceinline__ void mx_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        mx_for<N, F, I + 1>(static_cast<F &&>(f));
    }
}
// until at most N vector-memory requests of this wave are outstanding (LDS and scalar counts unrestricted)
template <int N> __device__ __forceinline__ void mx_wait_vm() { __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14)); }

// ------------------------------------------------------------------------------------------
// Layout: plain [N][C/8] words + [N][C/32] bytes  <->  blob = tiles | scale dwords
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mxfp4_repack_kernel(const uint32_t *__restrict__ codes,
                                                           const uint8_t *__restrict__ scales, int N, int C,
                                                           u32x4 *__restrict__ tiles, uint32_t *__restrict__ sdw)
{
    const int K128 = C / 128, KS = C / 512;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t n_tiles16 = (size_t)(N / 16) * K128 * 64;
    if (idx < n_tiles16) {
        const int lane = (int)(idx & 63);
        const size_t tk = idx >> 6;
        const int k128 = (int)(tk % K128);
        const size_t nt = tk / K128;
        const size_t row = nt * 16 + (lane & 15);
        tiles[idx] = *(const u32x4 *)(codes + row * (C / 8) + (size_t)k128 * 16 + (lane >> 4) * 4);
    }
    const size_t n_sdw = (size_t)(N / 16) * KS * 64;
    if (idx < n_sdw) {
        const int lane = (int)(idx & 63);
        const size_t ts = idx >> 6;
        const int ks = (int)(ts % KS);
        const size_t nt = ts / KS;
        const uint8_t *sr = scales + (nt * 16 + (lane & 15)) * (size_t)(C / 32) + (size_t)ks * 16 + (lane >> 4);
        sdw[idx] = (uint32_t)sr[0] | ((uint32_t)sr[4] << 8) | ((uint32_t)sr[8] << 16) | ((uint32_t)sr[12] << 24);
    }
}

// one thread per (row, 32-channel block): 32 code bytes and the scale byte, from either layout
__global__ __launch_bounds__(256) void mxfp4_unpack_kernel(const uint32_t *__restrict__ codes,
                                                           const uint8_t *__restrict__ scales,
                                                           const u32x4 *__restrict__ tiles,
                                                           const uint32_t *__restrict__ sdw, int N, int C,
                                                           uint8_t *__restrict__ out_codes, uint8_t *__restrict__ out_scales)
{
    const int B = C / 32;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)N * B) return;
    const size_t row = idx / B;
    const int b = (int)(idx % B);
    u32x4 v;
    uint32_t sc;
    if (tiles) {
        const int lane = (int)(row & 15) + 16 * (b & 3);
        v = tiles[((row / 16) * (C / 128) + b / 4) * 64 + lane];
        sc = (sdw[((row / 16) * (C / 512) + b / 16) * 64 + lane] >> (8 * ((b / 4) & 3))) & 0xffu;
    } else {
        v = *(const u32x4 *)(codes + row * (C / 8) + (size_t)b * 4);
        sc = scales[row * B + b];
    }
    uint8_t *o = out_codes + row * C + (size_t)b * 32;
#pragma unroll
    for (int j = 0; j < 32; ++j) o[j] = (uint8_t)((v[j / 8] >> (4 * (j % 8))) & 15u);
    out_scales[idx] = (uint8_t)sc;
}

hipError_t launch_mxfp4_repack(const paro_mxfp4_weight &w, void *packed_out, hipStream_t s)
{
    const size_t n = (size_t)w.c_out * w.c_in / 32;                   // 16-byte chunks of codes
    hipLaunchKernelGGL(mxfp4_repack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w.codes, w.scales,
                       w.c_out, w.c_in, (u32x4 *)packed_out,
                       (uint32_t *)((char *)packed_out + (size_t)w.c_out * w.c_in / 2));
    return hipGetLastError();
}

hipError_t launch_mxfp4_unpack(const paro_mxfp4_weight &w, uint8_t *codes, uint8_t *scales, hipStream_t s)
{
    const size_t n = (size_t)w.c_out * w.c_in / 32;
    const u32x4 *tiles = (const u32x4 *)w.packed;
    const uint32_t *sdw = w.packed ? (const uint32_t *)((const char *)w.packed + (size_t)w.c_out * w.c_in / 2) : nullptr;
    hipLaunchKernelGGL(mxfp4_unpack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w.codes, w.scales, tiles,
                       sdw, w.c_out, w.c_in, codes, scales);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Up to 64 tokens per pass
// ------------------------------------------------------------------------------------------
struct MxArgs {
    const void *blob; uint32_t blob_bytes, scales_off;
    const uint32_t *xc; const uint8_t *xs;          // activations of this pass: [T][C/8] words, [T][C/32] bytes
    _Float16 *Y; int64_t ldy;
    const _Float16 *bias;
    int T, C, N, NT, KS, tiles_per_block;
};

constexpr int kMxStages = 3;
constexpr int kMxMaxUnits = 16;                      // (tile, slice) units per wave: the stream is unrolled
constexpr int kMxMaxWaves = 12;                      // 3 waves per SIMD: 170 registers each

struct MxStage { u32x4 w[4]; uint32_t sc; };

// SPW: 512-channel slices per wave (wave w takes slices w, w + waves, ...).  TB: blocks of 16 tokens per wave
// (the weight tile of a unit is multiplied with each; the 4 MFMAs per token block are a small part of a unit's
// time, so up to 64 tokens cost little more than 16).  SPW * TB sets of activation fragments live in registers:
// up to 5 with 12 waves per block, up to 8 with 8.
template <int SPW, int TB>
__global__ __launch_bounds__((SPW * TB <= 5 ? kMxMaxWaves : 8) * 64) void mxfp4_decode_kernel(MxArgs a)
{
    constexpr int NS = kMxStages;
    extern __shared__ __attribute__((aligned(16))) float s_part[];       // [tiles per block][waves][TB][256]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int tile_lo = blockIdx.x * a.tiles_per_block;
    const int tile_hi = min(a.NT, tile_lo + a.tiles_per_block);
    const int n_iter = tile_hi - tile_lo;
    const int K128 = a.C / 128;
    const __amdgpu_buffer_rsrc_t blob = mx_rsrc(a.blob, a.blob_bytes);

    // ---- activations of the wave's slices as A operands: lane = (token l % 16 of its block, 32-channel block l / 16) ----
    const int ft = lane & 15, fkb = lane >> 4;
    u32x4 xf[SPW][TB][4];
    uint32_t xsc[SPW][TB];
    {
        const __amdgpu_buffer_rsrc_t xr = mx_rsrc(a.xc, (uint32_t)((size_t)a.T * a.C / 2));
        const __amdgpu_buffer_rsrc_t sr = mx_rsrc(a.xs, (uint32_t)((size_t)a.T * a.C / 32));
#pragma unroll
        for (int q = 0; q < SPW; ++q)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
                const int ks = wave + q * nw, t = tb * 16 + ft;
                const bool ok = ks < a.KS && t < a.T;
                const uint32_t xo = ok ? (uint32_t)((size_t)t * (a.C / 2) + (size_t)ks * 256 + fkb * 16) : kOobM;
#pragma unroll
                for (int m = 0; m < 4; ++m) xf[q][tb][m] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(xo + m * 64), 0, 0);
                // the slice's 16 scale bytes: dword m = K-step m, byte kb = the lane's block
                const u32x4 sc = __builtin_amdgcn_raw_buffer_load_b128(sr, ok ? (int)((size_t)t * (a.C / 32) + (size_t)ks * 16) : (int)kOobM, 0, 0);
                const int sh = 8 * fkb;
                xsc[q][tb] = ((sc[0] >> sh) & 0xffu) | (((sc[1] >> sh) & 0xffu) << 8) | (((sc[2] >> sh) & 0xffu) << 16) |
                             (((sc[3] >> sh) & 0xffu) << 24);
            }
    }
    // unit i = (tile tile_lo + i / SPW, slice wave + (i % SPW) waves); nothing to load beyond the range: zeros
    MxStage st[NS];
    auto load_unit = [&](int i, MxStage &s) {
        const int ti = i / SPW, ks = wave + (i % SPW) * nw;
        const bool ok = ti < n_iter && ks < a.KS;
        const uint32_t tile = (uint32_t)(tile_lo + ti);
        const uint32_t off = ok ? ((tile * K128 + ks * 4) * 64u + lane) * 16u : kOobM;
#pragma unroll
        for (int m = 0; m < 4; ++m) s.w[m] = __builtin_amdgcn_raw_buffer_load_b128(blob, (int)(off + m * 1024u), 0, 2);
        s.sc = __builtin_amdgcn_raw_buffer_load_b32(blob, ok ? (int)(a.scales_off + ((tile * a.KS + ks) * 64u + lane) * 4u) : (int)kOobM, 0, 0);
    };
#pragma unroll
    for (int i = 0; i + 1 < NS; ++i) load_unit(i, st[i]);

    float4v acc[TB];
    mx_static_while<kMxMaxUnits>([&](auto I) {
        constexpr int i = I;
        constexpr int q = i % SPW;
        if (i / SPW >= n_iter) return false;
        load_unit(i + NS - 1, st[(i + NS - 1) % NS]);
        const MxStage &s = st[i % NS];
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            if constexpr (q == 0) acc[tb] = float4v{0.f, 0.f, 0.f, 0.f};
            acc[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_operand(xf[q][tb][0]), as_operand(s.w[0]), acc[tb], 4, 4, 0, (int)xsc[q][tb], 0, (int)s.sc);
            acc[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_operand(xf[q][tb][1]), as_operand(s.w[1]), acc[tb], 4, 4, 1, (int)xsc[q][tb], 1, (int)s.sc);
            acc[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_operand(xf[q][tb][2]), as_operand(s.w[2]), acc[tb], 4, 4, 2, (int)xsc[q][tb], 2, (int)s.sc);
            acc[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(as_operand(xf[q][tb][3]), as_operand(s.w[3]), acc[tb], 4, 4, 3, (int)xsc[q][tb], 3, (int)s.sc);
            if constexpr (q == SPW - 1) *(float4v *)(s_part + (((size_t)(i / SPW) * nw + wave) * TB + tb) * 256 + lane * 4) = acc[tb];
        }
        return true;
    });
    __syncthreads();
    // ---- sum the waves' partial tiles: element lane * 4 + r <-> token 4 (lane / 16) + r of its block, row lane % 16 ----
    const int per_tile = a.T * kTileN;
    for (int idx = threadIdx.x; idx < n_iter * per_tile; idx += blockDim.x) {
        const int i = idx / per_tile, rem = idx % per_tile;
        const int t = rem / kTileN, nn = rem % kTileN;
        const int e = (t >> 4) * 256 + (((t & 15) >> 2) * 16 + nn) * 4 + (t & 3);
        float sum = 0.f;
        for (int w = 0; w < nw; ++w) sum += s_part[((size_t)i * nw + w) * (TB * 256) + e];
        const size_t n = (size_t)(tile_lo + i) * kTileN + nn;
        if (a.bias) sum += (float)a.bias[n];
        a.Y[(size_t)t * a.ldy + n] = (_Float16)sum;
    }
}

// Geometry of a pass of T tokens: TB token blocks per wave, as many as the registers allow for this K.
struct MxGeometry { int spw, tb, waves, tiles_per_block, blocks; size_t lds; };
static bool mx_geometry(int c_in, int c_out, int T, MxGeometry &g)
{
    const int KS = c_in / 512, NT = c_out / kTileN;
    const int want = T > 32 ? 4 : T > 16 ? 2 : 1;
    g.tb = 0;
    for (int tb = want; tb >= 1 && !g.tb; tb >>= 1) {
        // sets of fragments = SPW * TB: up to 5 with 12 waves per block, up to 8 with 8 waves
        const int spw12 = (KS + kMxMaxWaves - 1) / kMxMaxWaves, spw8 = (KS + 7) / 8;
        if (spw12 * tb <= 5) { g.tb = tb; g.spw = spw12; }
        else if (spw8 * tb <= 8) { g.tb = tb; g.spw = spw8; }
    }
    if (!g.tb || g.spw > 5) return false;
    g.waves = (KS + g.spw - 1) / g.spw;
    int tpb = (NT + 255) / 256;                               // one block per compute unit
    if (tpb > kMxMaxUnits / g.spw) tpb = kMxMaxUnits / g.spw;
    if (tpb * g.waves * g.tb > 144) tpb = 144 / (g.waves * g.tb);   // TB KB of LDS per (tile, wave)
    if (tpb < 1) return false;
    g.tiles_per_block = tpb;
    g.blocks = (NT + tpb - 1) / tpb;
    g.lds = (size_t)tpb * g.waves * g.tb * 1024;
    return true;
}

bool mxfp4_linear_supported(const paro_mxfp4_weight &w)
{
    MxGeometry g;
    return w.packed && w.c_in % 512 == 0 && w.c_out % 16 == 0 && mx_geometry(w.c_in, w.c_out, 1, g) &&
           (size_t)w.c_out * w.c_in / 2 + (size_t)w.c_out * w.c_in / 32 < (1ull << 31);
}

// tokens one pass of the streaming kernel takes for this K (64, 32 or 16)
static int mxfp4_pass_tokens(const paro_mxfp4_weight &w, int T)
{
    MxGeometry g;
    return mx_geometry(w.c_in, w.c_out, T, g) ? 16 * g.tb : 16;
}

template <int SPW, int TB>
static hipError_t launch_mxfp4_decode_cfg(const MxArgs &a, const MxGeometry &g, hipStream_t s)
{
    static std::atomic<uint64_t> attr_done{0};
    if (const int dev = once_pending(attr_done); dev >= 0) {
        hipError_t e = hipFuncSetAttribute((const void *)mxfp4_decode_kernel<SPW, TB>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        once_done(attr_done, dev);
    }
    hipLaunchKernelGGL((mxfp4_decode_kernel<SPW, TB>), dim3(g.blocks), dim3(g.waves * 64), g.lds, s, a);
    return hipGetLastError();
}

// one pass of up to mxfp4_pass_tokens() tokens
static hipError_t launch_mxfp4_decode(const paro_mxfp4_weight &w, const uint32_t *xc, const uint8_t *xs, int T,
                                      paro_half_t *Y, int64_t ldy, hipStream_t s)
{
    MxGeometry g;
    if (!mx_geometry(w.c_in, w.c_out, T, g) || T > 16 * g.tb) return hipErrorInvalidValue;
    MxArgs a;
    a.blob = w.packed;
    a.scales_off = (uint32_t)((size_t)w.c_out * w.c_in / 2);
    a.blob_bytes = a.scales_off + (uint32_t)((size_t)w.c_out * w.c_in / 32);
    a.xc = xc; a.xs = xs; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.NT = w.c_out / kTileN; a.KS = w.c_in / 512;
    a.tiles_per_block = g.tiles_per_block;
    switch (g.tb * 8 + g.spw) {
    case 1 * 8 + 1: return launch_mxfp4_decode_cfg<1, 1>(a, g, s);
    case 1 * 8 + 2: return launch_mxfp4_decode_cfg<2, 1>(a, g, s);
    case 1 * 8 + 3: return launch_mxfp4_decode_cfg<3, 1>(a, g, s);
    case 1 * 8 + 4: return launch_mxfp4_decode_cfg<4, 1>(a, g, s);
    case 1 * 8 + 5: return launch_mxfp4_decode_cfg<5, 1>(a, g, s);
    case 2 * 8 + 1: return launch_mxfp4_decode_cfg<1, 2>(a, g, s);
    case 2 * 8 + 2: return launch_mxfp4_decode_cfg<2, 2>(a, g, s);
    case 2 * 8 + 3: return launch_mxfp4_decode_cfg<3, 2>(a, g, s);
    case 2 * 8 + 4: return launch_mxfp4_decode_cfg<4, 2>(a, g, s);
    case 4 * 8 + 1: return launch_mxfp4_decode_cfg<1, 4>(a, g, s);
    case 4 * 8 + 2: return launch_mxfp4_decode_cfg<2, 4>(a, g, s);
    default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------------------------------
// More tokens: tiled GEMM on v_mfma_scale_f32_32x32x64_f8f6f4 (lane l of an operand: row l % 32, elements 32 (l / 32) .. + 31 of
// the 64-wide step, one scale byte; D: lane = column l % 32, rows 8 (r / 4) + 4 (l / 32) + r % 4).  The weight is the A operand
// and the activations are the B operand, so that a lane's sums are consecutive outputs of one token.
//
// A block is 4 waves side by side along the outputs and owns 128 tokens x 128 NTW outputs; two blocks share a compute unit, so
// that one multiplies while the other waits at a barrier, fills its pipeline or stores its tile.
//   - Weights never touch LDS: every weight of a tile is needed by exactly one wave, which fetches it from the repacked blob
//     (contiguous 512-byte runs) into a register ring of three K-steps (128 channels each).
//   - Activations go from memory to LDS without passing through registers, 256 channels (whole 128-byte lines) of 8 rows per
//     wave request, into a ring of four such steps: one barrier and one wait per 256 channels, for requests made 768 channels
//     earlier.  The 16-byte chunk index of a row is XOR-ed with bits 1..3 of the row: a 16-byte read serves lanes 0-3, 12-15 and
//     20-27 together (then 4-11, 16-19 and 28-31), which are then 16 bank groups, and every four lanes of a request still ask for
//     64 consecutive bytes (in the order [chunk][row], conflict-free as well, each lane is a request of its own).
//   - Scale bytes: the weight's as one dword per lane and 512 channels from the blob; the activations' through LDS as
//     [K-step][row] dwords, two slices of 512 channels deep.
//   - Outputs leave past the L2 (non-temporal): a round's tiles finish together, and their 33 MB would push the operands out of
//     the L2s (4096 tokens 5120 -> 55296: 636 us with plain stores, 581).  A ragged last tile does the same (in 2-byte stores
//     it alone took 2 to 4 us: 168 tokens 1536 -> 19040 15.2 us with the quantiser, now 12.7).
// What bounds it (counters, 4096 tokens 5120 -> 55296): the chip's power - 1.6 GHz with the matrix cores busy 61 % of the cycles -
// and the operand traffic out of L2 (9 GB; with all-zero operands, which cost no switching, 431 us).  2048 tokens 4096 -> 28672: 2.3
// GHz, busy 44 %.  NTW = 2 takes all 256 registers and spills one, in the prologue and back behind the loop.
// Measured, us, before (256 x 256 tiles of 8 waves, activations through registers, 16x16x128 instruction, one block per
// compute unit) -> now: 2048 tokens 4096 -> 6144 42.3 -> 36.0, 4096 -> 4096 26.9 -> 21.1, 4096 -> 28672 168.7 -> 143.1 (3.4
// PFLOP/s), 14336 -> 4096 74.6 -> 65.9; 4096 tokens 5120 -> 55296 698 -> 579 (4.0); 256 tokens 14336 -> 4096 53.8 -> 27.9;
// with the quantiser, 111 random shapes of 33 to 2048 tokens: 0.77 of the time in the geometric mean, none more than 1.5 % slower.
// ------------------------------------------------------------------------------------------
struct MxGemmArgs {
    const void *blob; uint32_t blob_bytes, scales_off;
    const uint32_t *xc; const uint8_t *xs;
    _Float16 *Y; int64_t ldy;
    const _Float16 *bias;
    int T, C, N, K128, KS;
    int m_tiles, n_tiles;
};

typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void mx_lds;

constexpr int kMxBM = 128;                               // tokens per block
constexpr int kMxRing = 4, kMxPair = kMxBM * 128;        // activation ring: bytes of 256 channels of all rows
constexpr int kMxScaleSlice = 4 * kMxBM * 4;             // [K-step][row] scale dwords of 512 channels
constexpr int kMxGemmLds = kMxRing * kMxPair + 2 * kMxScaleSlice;
constexpr int kMxChunk = 12;                             // K-steps written out in the loop body: three periods of 4, four of 3

template <int NTW>
__global__ __launch_bounds__(256, 2) void mxfp4_gemm_kernel(MxGemmArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char smem_mx[];
    constexpr int BN = 128 * NTW, MT = kMxBM / 32, XR = 4;   // XR: activation requests of a wave per 256 channels
    int idx, mt0, ntile;
    if (!tile_index(a.m_tiles * a.n_tiles, idx)) return;
    tile_place(idx, a.m_tiles, a.n_tiles, mt0, ntile);
    const int m0 = mt0 * kMxBM;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 31, lh = lane >> 5;
    const int n0 = ntile * BN + wave * 32 * NTW;             // the wave's outputs
    const __amdgpu_buffer_rsrc_t xr = mx_rsrc(a.xc, (uint32_t)((size_t)a.T * a.C / 2));
    const __amdgpu_buffer_rsrc_t sr = mx_rsrc(a.xs, (uint32_t)((size_t)a.T * a.C / 32));
    const __amdgpu_buffer_rsrc_t br = mx_rsrc(a.blob, a.blob_bytes);
    const int n_ks = a.K128, n_pairs = n_ks / 2;

    // ---- activations: wave w, request i: rows 8 (XR w + i) .. + 7.  Rows beyond T read row T - 1 (their sums are not stored) ----
    uint32_t gx[XR];
#pragma unroll
    for (int i = 0; i < XR; ++i) {
        const int row = min(m0 + (wave * XR + i) * 8 + (lane >> 3), a.T - 1);
        gx[i] = (uint32_t)((size_t)row * (a.C / 2)) + (((lane & 7) ^ (lane >> 4) ^ (4 * (i & 1))) << 4);
    }
    auto load_x = [&](int pair) {
        const bool ok = pair < n_pairs;                      // beyond the row's end: out of range, nothing is fetched
        char *dst = smem_mx + (pair & (kMxRing - 1)) * kMxPair + wave * (XR * 1024);
#pragma unroll
        for (int i = 0; i < XR; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (mx_lds *)(dst + i * 1024), 16, (int)(ok ? gx[i] : kOobM), pair * 128, 0, 0);
    };
    // scale bytes: thread -> row tid / 2, K-steps 2 (tid % 2), + 1 of the slice
    const uint32_t gs = (uint32_t)((size_t)min(m0 + (tid >> 1), a.T - 1) * (a.C / 32)) + (tid & 1) * 8;
    char *const scales = smem_mx + kMxRing * kMxPair;
    u32x2 xs_next;
    auto load_xs = [&](int slice) { xs_next = __builtin_amdgcn_raw_buffer_load_b64(sr, (int)(slice < a.KS ? gs : kOobM), slice * 16, 0); };
    auto store_xs = [&](int slice) {
        char *dst = scales + (slice & 1) * kMxScaleSlice + (tid & 1) * (8 * kMxBM) + (tid >> 1) * 4;
        *(uint32_t *)dst = xs_next[0];
        *(uint32_t *)(dst + 4 * kMxBM) = xs_next[1];
    };
    // ---- weights: n-tile nt of the wave = two 16-row tiles of the blob; lane: row lr, 32-channel block 2 h + lh ----
    uint32_t gb[NTW], gw[NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
        const int n = n0 + nt * 32 + lr;
        const uint32_t t16 = (uint32_t)(n >> 4), slot = (uint32_t)(lh * 16 + (lr & 15));
        gb[nt] = n < a.N ? (t16 * (uint32_t)a.K128 * 64u + slot) * 16u : kOobM;
        gw[nt] = n < a.N ? a.scales_off + (t16 * (uint32_t)a.KS * 64u + slot) * 4u : kOobM;
    }
    u32x4 wb[3][NTW][2];
    auto load_w = [&](int ks, auto R, auto NT, auto H) {
        wb[R][NT][H] = __builtin_amdgcn_raw_buffer_load_b128(br, (int)(ks < n_ks ? gb[NT] + H * 512 : kOobM), ks * 1024, 0);
    };
    uint32_t wsc[3][NTW][2];                                 // scale dwords: ring of three slices (a copy would wait for the load)
    auto load_ws = [&](int slice, auto R) {
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                wsc[R][nt][h] = __builtin_amdgcn_raw_buffer_load_b32(br, (int)(slice < a.KS ? gw[nt] + h * 128 : kOobM), slice * 256, 0);
    };

    float16v acc[NTW][MT];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nt][mt][r] = 0.f;

    // fragment of token tile mt, 64-channel step kh = 2 kp + h of a pair: chunk 2 kh + lh of the row
    int fx[4];
#pragma unroll
    for (int kh = 0; kh < 4; ++kh) fx[kh] = lr * 128 + (((2 * kh + lh) ^ ((lr >> 1) & 7)) << 4);
    constexpr int kAhead = 3, kRegs = kAhead + 1;            // fragments are requested this many token tiles ahead
    u32x4 xf[kRegs];
    uint32_t xsd[MT];
    auto read_x = [&](const char *pair, auto Q) {            // Q: (kp * 2 + h) * MT + mt within the pair
        constexpr int q = Q, mt = q % MT, kh = q / MT;
        xf[q % kRegs] = *(const u32x4 *)(pair + mt * 4096 + fx[kh]);
    };
    const int fs = lr * 4;
    const uint32_t s_shift = 8 * lh;

    // ---- prologue ----
    using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>; using I2 = std::integral_constant<int, 2>;
    // Requests leave in the order written, which the wait below counts on (the compiler moved the weights of K-steps 1 and 2 behind
    // everything else, which was safe; in front of pair 0 they would not be).
    auto in_order = [] { __builtin_amdgcn_sched_barrier(0); };
    load_xs(0);
    load_ws(0, I0{});
    in_order();
    load_x(0);
    in_order();
    mx_for<NTW>([&](auto NT) { load_w(0, I0{}, NT, I0{}); load_w(0, I0{}, NT, I1{}); });
    in_order();
    load_x(1);
    in_order();
    mx_for<NTW>([&](auto NT) { load_w(1, I1{}, NT, I0{}); load_w(1, I1{}, NT, I1{}); });
    in_order();
    load_x(2);
    in_order();
    mx_for<NTW>([&](auto NT) { load_w(2, I2{}, NT, I0{}); load_w(2, I2{}, NT, I1{}); });
    in_order();
    store_xs(0);
    in_order();
    load_xs(1);
    load_ws(1, I1{});
    in_order();
    // activations of pair 0 are in LDS when at most the requests made after them are outstanding (8 NTW + 9)
    mx_wait_vm<8 * NTW>();
    __builtin_amdgcn_s_waitcnt(0xc07f);                      // LDS writes done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    mx_for<kAhead>([&](auto Q) { read_x(smem_mx, Q); });
    mx_for<MT>([&](auto M) { xsd[M] = *(const uint32_t *)(scales + fs + M * 128); });

    for (int ks0 = 0; ks0 < n_ks; ks0 += kMxChunk) {
        mx_static_while<kMxChunk / 4>([&](auto S) {
            const int slice = (ks0 >> 2) + S;
            if (slice >= a.KS) return false;
            mx_for<4>([&](auto U) {
                constexpr int u = U, kp = u & 1, r3 = (S * 4 + u) % 3;
                const int ks = slice * 4 + u, pair = ks >> 1;
                const char *cur = smem_mx + (pair & (kMxRing - 1)) * kMxPair;
                const char *nxt = smem_mx + ((pair + 1) & (kMxRing - 1)) * kMxPair;
                const char *snx = scales + ((u == 3 ? slice + 1 : slice) & 1) * kMxScaleSlice + ((u + 1) & 3) * 512 + fs;
                using R3 = std::integral_constant<int, r3>;
                mx_for<2 * MT>([&](auto Q) {
                    constexpr int q = Q, h = q / MT, mt = q % MT, qa = kp * 2 * MT + q;   // position within the pair
                    if constexpr (kp == 1 && q == 2 * MT - kAhead) {
                        // every wave's part of the next pair has arrived (requested two pairs ago, older than the weights
                        // of this K-step) and every wave has read the previous pair for the last time
                        mx_wait_vm<8 * NTW>();
                        __builtin_amdgcn_s_waitcnt(0xc07f);
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                        load_x(pair + 3);
                    }
                    if constexpr (qa + kAhead < 4 * MT) read_x(cur, std::integral_constant<int, qa + kAhead>{});
                    else read_x(nxt, std::integral_constant<int, qa + kAhead - 4 * MT>{});
                    if constexpr (h == 0) xsd[mt] >>= s_shift;
                    mx_for<NTW>([&](auto NT) {
                        acc[NT][mt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(as_operand(wb[R3{}][NT][h]), as_operand(xf[qa % kRegs]), acc[NT][mt], 4, 4,
                                                                                       u, (int)wsc[S][NT][h], 2 * h, (int)xsd[mt]);
                    });
                    if constexpr (h == 1) xsd[mt] = *(const uint32_t *)(snx + mt * 128);
                    if constexpr (h == 1 && mt == 0) mx_for<NTW>([&](auto NT) { load_w(ks + 3, R3{}, NT, I0{}); });
                    if constexpr (h == 1 && mt == MT - 1) mx_for<NTW>([&](auto NT) { load_w(ks + 3, R3{}, NT, I1{}); });
                    if constexpr (u == 0 && q == 1) { store_xs(slice + 1); load_xs(slice + 2); load_ws(slice + 2, std::integral_constant<int, (S + 2) % 3>{}); }   // the slice before: last read before the latest barrier
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            return true;
        });
    }

    // ---- epilogue.  A wave's 32 tokens x 32 NTW outputs at a time go through a wave-private strip of LDS (the ring is free once
    // every wave is here and no request is outstanding) and leave as 16 bytes per lane, whole rows of the strip. ----
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    constexpr int kStrip = 64 * NTW + 16;                                            // bytes of a strip's row
    char *strip = smem_mx + wave * 32 * kStrip;
    const __amdgpu_buffer_rsrc_t yr = mx_rsrc(a.Y, (uint32_t)(((size_t)(a.T - 1) * a.ldy + a.N) * 2));
    const bool row_wide = a.ldy % 8 == 0 && ((uintptr_t)a.Y % 16) == 0;             // 8 outputs are all there or none is
    if (a.bias) {
        const __amdgpu_buffer_rsrc_t bias = mx_rsrc(a.bias, (uint32_t)a.N * 2);      // outputs beyond N read as zero
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                union { uint16_t u; _Float16 h; } b;
                b.u = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(bias, (n0 + nt * 32 + (r >> 2) * 8 + lh * 4 + (r & 3)) * 2, 0, 0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) acc[nt][mt][r] += (float)b.h;
            }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int o = nt * 32 + g * 8 + lh * 4;                              // 4 consecutive outputs
                union { _Float16 h[4]; u32x2 u; } v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v.h[r] = (_Float16)acc[nt][mt][g * 4 + r];
                *(u32x2 *)(strip + lr * kStrip + o * 2) = v.u;
            }
        __builtin_amdgcn_wave_barrier();
        if (row_wide) {
            constexpr int kLanes = 4 * NTW, kRows = 64 / kLanes;                     // lanes per row, rows per access
#pragma unroll
            for (int i = 0; i < 32 / kRows; ++i) {
                const int row = i * kRows + lane / kLanes, col = (lane % kLanes) * 8, m = m0 + mt * 32 + row;
                const u32x4 v = *(const u32x4 *)(strip + row * kStrip + col * 2);
                const uint32_t off = m < a.T && n0 + col < a.N ? (uint32_t)(((size_t)m * a.ldy + n0 + col) * 2) : kOobM;
                __builtin_amdgcn_raw_buffer_store_b128(v, yr, (int)off, 0, 2);
            }
        } else {
            for (int e = lane; e < 32 * 32 * NTW; e += 64) {
                const int row = e / (32 * NTW), col = e % (32 * NTW), m = m0 + mt * 32 + row, n = n0 + col;
                const uint16_t v = *(const uint16_t *)(strip + row * kStrip + col * 2);
                const uint32_t off = m < a.T && n < a.N ? (uint32_t)(((size_t)m * a.ldy + n) * 2) : kOobM;
                __builtin_amdgcn_raw_buffer_store_b16(v, yr, (int)off, 0, 0);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int NTW>
static hipError_t launch_mxfp4_gemm_cfg(MxGemmArgs &a, hipStream_t s)
{
    a.m_tiles = (a.T + kMxBM - 1) / kMxBM; a.n_tiles = (a.N + 128 * NTW - 1) / (128 * NTW);
    const unsigned blocks = (unsigned)(((size_t)a.m_tiles * a.n_tiles + 7) / 8 * 8);
    static std::atomic<uint64_t> attr_done{0};
    if (const int dev = once_pending(attr_done); dev >= 0) {
        hipError_t e = hipFuncSetAttribute((const void *)mxfp4_gemm_kernel<NTW>, hipFuncAttributeMaxDynamicSharedMemorySize, kMxGemmLds);
        if (e != hipSuccess) return e;
        once_done(attr_done, dev);
    }
    hipLaunchKernelGGL(mxfp4_gemm_kernel<NTW>, dim3(blocks), dim3(256), kMxGemmLds, s, a);
    return hipGetLastError();
}

// 128 outputs per block while 256 would fill at most half of the compute units.  Both widths forced on 322 shapes, us with the
// quantiser, 128 / 256 outputs: 4608 -> 13984 at 152 tokens (110 tiles of 256) 13.9 / 18.0 without it, 3072 -> 34736 at 67 (136)
// 19.9 / 18.1, 2048 -> 18416 at 185 (144) 15.4 / 14.5; the choice costs 0.1 % over the better one, with the line at 192 tiles 0.3 %.
static bool mxfp4_gemm_small_tiles(const paro_mxfp4_weight &w, int T)
{
    return (long)((T + kMxBM - 1) / kMxBM) * ((w.c_out + 255) / 256) <= 128;
}

// Time of the GEMM behind the quantiser, up to 260 tokens and a round of blocks (512 = two per compute unit): a fixed part and a
// time per K-step that grow with the blocks; 272 shapes, 4 % off.
static double mxfp4_gemm_us(const paro_mxfp4_weight &w, int T)
{
    const bool small = mxfp4_gemm_small_tiles(w, T);
    const int bn = small ? 128 : 256;
    const double k = w.c_in / 128, f = (double)((T + kMxBM - 1) / kMxBM) * ((w.c_out + bn - 1) / bn) / 512.0;
    return small ? 3.55 + k * (0.257 + 0.104 * f) + 3.3 * f : 4.38 + k * (0.356 + 0.248 * f) + 3.8 * f;
}

// Time of the streaming kernel: per pass and round of blocks the fragments of the activations, the waves' start, the sums of the
// partial tiles and the units of the stream, and what the matrix cores take; 250 shapes of up to 5 passes, 4 % off.
static double mxfp4_stream_us(const paro_mxfp4_weight &w, int T)
{
    const double mb = ((double)w.c_out * w.c_in / 2 + (double)w.c_out * w.c_in / 32) / 1.0e6;
    double us = 0;
    MxGeometry g;
    for (int t0 = 0; t0 < T && mx_geometry(w.c_in, w.c_out, T - t0, g); t0 += 16 * g.tb) {
        const double rows = std::min(T - t0, 16 * g.tb), rounds = (g.blocks + 255) / 256;
        us += rounds * (0.48 * g.spw * g.tb + 0.464 * g.waves + 0.037 * g.tiles_per_block * rows / g.waves + 0.722 * g.tiles_per_block * g.spw) + 0.026 * mb * g.tb;
    }
    return us;
}

static hipError_t launch_mxfp4_gemm(const paro_mxfp4_weight &w, const uint32_t *xc, const uint8_t *xs, int T, paro_half_t *Y,
                                    int64_t ldy, hipStream_t s)
{
    MxGemmArgs a;
    a.blob = w.packed;
    a.scales_off = (uint32_t)((size_t)w.c_out * w.c_in / 2);
    a.blob_bytes = a.scales_off + (uint32_t)((size_t)w.c_out * w.c_in / 32);
    a.xc = xc; a.xs = xs; a.Y = (_Float16 *)Y; a.ldy = ldy; a.bias = (const _Float16 *)w.bias;
    a.T = T; a.C = w.c_in; a.N = w.c_out; a.K128 = w.c_in / 128; a.KS = w.c_in / 512;
    return mxfp4_gemm_small_tiles(w, T) ? launch_mxfp4_gemm_cfg<1>(a, s) : launch_mxfp4_gemm_cfg<2>(a, s);
}

// Which kernel: the streaming kernel reads the whole weight once per 64 tokens (32 or 16 where K is deep), the GEMM once per
// 128 but works on whole tiles whatever T is.  Up to 32 tokens a single pass is always taken (30 x 10240 -> 21392: 21.7 us against
// 25.8).  Both kernels forced on 272 shapes of 33 to 420 tokens: the choice costs 0.3 % over the better one (the streaming kernel
// stays where the models tie within 5 %; 48 tokens 19456 -> 3536: 34.0 us, the GEMM 45.8; 79 tokens 3584 -> 1088: 11.2 against 9.7).
static bool mxfp4_gemm_route(const paro_mxfp4_weight &w, int T, int64_t ldy)
{
    // the GEMM addresses the activations and the outputs with 32-bit offsets
    return T > std::min(mxfp4_pass_tokens(w, T), 32) && (size_t)T * w.c_in / 2 < (1ull << 31) && ((size_t)(T - 1) * ldy + w.c_out) * 2 < (1ull << 31) &&
           1.05 * mxfp4_gemm_us(w, T) < mxfp4_stream_us(w, T);
}

int mxfp4_linear_plan(const paro_mxfp4_weight &w, int T)
{
    return !mxfp4_gemm_route(w, T, w.c_out) ? 0 : mxfp4_gemm_small_tiles(w, T) ? 128 : 256;
}

hipError_t launch_mxfp4_linear(const paro_mxfp4_weight &w, const uint32_t *x_codes, const uint8_t *x_scales, int T,
                               paro_half_t *Y, int64_t ldy, hipStream_t s)
{
    if (mxfp4_gemm_route(w, T, ldy)) return launch_mxfp4_gemm(w, x_codes, x_scales, T, Y, ldy, s);
    for (int t0 = 0; t0 < T;) {
        const int pass = mxfp4_pass_tokens(w, T - t0);
        const int tp = T - t0 < pass ? T - t0 : pass;
        hipError_t e = launch_mxfp4_decode(w, x_codes + (size_t)t0 * (w.c_in / 8), x_scales + (size_t)t0 * (w.c_in / 32), tp,
                                           Y + (size_t)t0 * ldy, ldy, s);
        if (e != hipSuccess) return e;
        t0 += tp;
    }
    return hipSuccess;
}

}  // namespace paro
