// gfx950 kernels of the learned warm start: a 3-D convolutional
// encoder-decoder that maps A^T y to a starting volume for the solver.
//
// Activations are channels-last BF16 [D][H][W][C]; weights keep an FP32
// master copy [Cout][K] with K = tap * Cin + ci (tap = dz*9 + dy*3 + dx for
// 3x3x3, offsets -1..1, zero padding), packed to BF16 for the MFMA kernels.
//
// Convolution = implicit GEMM on v_mfma_f32_16x16x32_bf16 (FP32 accumulate):
// K runs over (tap, ci).  The staged 3x3x3 kernels take the weights as the first
// operand (rows are output channels, columns voxels), the general ones the voxels.
// Operand lane layout of the 16x16x32 instruction: lane l supplies
// A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j][l % 16], j = 0..7, and
// holds D[4 (l / 16) + i][l % 16], i = 0..3.
#include <algorithm>

#include "ltm_internal.h"
#include "ltm_nn.h"

namespace ltm {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

__device__ __forceinline__ float bf2f(u16 v) { return __uint_as_float((unsigned)v << 16); }

__device__ __forceinline__ u16 f2bf(float f)
{
    // round to nearest even (finite inputs); NaN stays NaN
    unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}

// Where the 8-channel group g of voxel v of a staged halo lies: at v * (CIN / 8) +
// (g ^ conv_swizzle<CIN>(v)), in units of 16 bytes.  One clock of a 16-byte read
// serves lanes 0..3 and 20..23 (and so on): four voxels' group g and the next
// four's group g + 1.  They fall on different banks as they are for 32-byte
// voxels, and with this exchange of groups for 64-byte ones and multiples.
template <int CIN>
__device__ __forceinline__ int conv_swizzle(int v)
{
    return CIN % 64 == 0 ? (v & 3) << 1 : CIN % 32 == 0 ? v & 2 : 0;
}

// Kernels that end in a global atomic per workgroup on the same few addresses: one
// workgroup of 16 waves per compute unit, as the atomics of one address take
// about 12 (maxima) to 28 ns (sums) each, one after the other.  With 1024
// workgroups of 4 waves the maximum of 128^3 values took 51 us, the masked
// gradient with its bias sums 29 us however small; now 3 and 15 us.
constexpr unsigned kSumBlock = 1024;

unsigned sum_blocks(size_t n)
{
    const size_t b = (n + kSumBlock - 1) / kSumBlock;
    return (unsigned)(b > 256 ? 256 : (b ? b : 1));
}

union Frag {
    bf16x8 v;
    uint4 q;
    unsigned int w[4];
    u16 h[8];
};

// ---------------------------------------------------------------- conv forward
// One workgroup: 4 waves x MT tiles of 16 output voxels (flattened index),
// all NT x 16 output channels.  Input channels come from in0 (c0 channels)
// then in1 (c1 channels, the concatenated skip); the input grid is the
// output grid >> up (nearest upsampling fused into the read).
template <int KS, bool CIN1, int NT, int MT>
__global__ __launch_bounds__(256) void k_conv_fwd(ConvFwd a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int V = a.D * a.H * a.W;
    const int Din = a.D >> a.up, Hin = a.H >> a.up, Win = a.W >> a.up;
    const int cin = a.c0 + a.c1;
    const int taps = KS * KS * KS;
    const int vbase = (blockIdx.x * 4 + wave) * (16 * MT);
    // this workgroup's output channels: tiles [blockIdx.y NT, blockIdx.y NT + NT)
    const int c16 = blockIdx.y * NT * 16;

    int vz[MT], vy[MT], vx[MT];
    bool vin[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int v = vbase + m * 16 + r;
        vin[m] = v < V;
        const int vv = vin[m] ? v : 0;
        vx[m] = vv % a.W;
        vy[m] = (vv / a.W) % a.H;
        vz[m] = vv / (a.W * a.H);
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (CIN1) {
        for (int k0 = 0; k0 < a.Kp; k0 += 32) {
            const int kk = k0 + 8 * kg;
            Frag A[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                A[m].q = uint4{0u, 0u, 0u, 0u};
                if (!vin[m]) continue;
                // one input channel: the 8 K values are 8 taps
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int tap = kk + j;
                    if (tap >= taps) continue;
                    const int dz = KS == 3 ? tap / 9 - 1 : 0, dy = KS == 3 ? (tap / 3) % 3 - 1 : 0,
                              dx = KS == 3 ? tap % 3 - 1 : 0;
                    const int z = vz[m] + dz, y = vy[m] + dy, x = vx[m] + dx;
                    if (z < 0 || z >= a.D || y < 0 || y >= a.H || x < 0 || x >= a.W) continue;
                    const size_t src = ((size_t)(z >> a.up) * Hin + (y >> a.up)) * Win + (x >> a.up);
                    A[m].h[j] = a.in0[src];
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                Frag B;
                B.q = *reinterpret_cast<const uint4*>(a.wt + (size_t)(c16 + t * 16 + r) * a.Kp + kk);
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[m].v, B.v, acc[m][t], 0, 0, 0);
            }
        }
    } else {
        // U K-steps at a time: all their operand loads are issued before
        // their MFMAs.  Loads are branch-free: an out-of-range tap or voxel
        // reads a valid address and selects zero; a K-step past Kp repeats
        // step k0 and is skipped.
        constexpr int U = 2;
        for (int k0 = 0; k0 < a.Kp; k0 += 32 * U) {
            Frag A[U][MT], B[U][NT];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int kk = (k0 + 32 * u < a.Kp ? k0 + 32 * u : k0) + 8 * kg;
                const int tap = kk / cin, ci = kk - tap * cin;
                const bool tapok = tap < taps;
                const int dz = KS == 3 ? tap / 9 - 1 : 0, dy = KS == 3 ? (tap / 3) % 3 - 1 : 0,
                          dx = KS == 3 ? tap % 3 - 1 : 0;
                // the 8 channels [ci, ci + 8) lie in one input (c0 % 8 == 0)
                const bool first = ci < a.c0;
                const u16* src_base = first ? a.in0 + ci : a.in1 + (ci - a.c0);
                const int cst = first ? a.c0 : a.c1;
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const int z = vz[m] + dz, y = vy[m] + dy, x = vx[m] + dx;
                    const bool ok = vin[m] && tapok && (unsigned)z < (unsigned)a.D &&
                                    (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;
                    const size_t src =
                        ok ? ((size_t)(z >> a.up) * Hin + (y >> a.up)) * Win + (x >> a.up) : 0;
                    const uint4 q = *reinterpret_cast<const uint4*>(src_base + src * cst);
                    A[u][m].q = ok ? q : uint4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    B[u][t].q = *reinterpret_cast<const uint4*>(a.wt + (size_t)(c16 + t * 16 + r) * a.Kp + kk);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (k0 + 32 * u >= a.Kp) break;
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int m = 0; m < MT; ++m)
                        acc[m][t] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[u][m].v, B[u][t].v, acc[m][t], 0, 0, 0);
            }
        }
    }
    // epilogue: bias, ReLU, store (BF16 or FP32, optionally split in two
    // channel ranges for the input gradient of a concatenation)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int co = c16 + t * 16 + r;
            if (co >= a.cout) continue;
            const float b = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int v = vbase + m * 16 + 4 * kg + i;
                if (v >= V) continue;
                float val = acc[m][t][i] + b;
                if (a.relu) val = fmaxf(val, 0.0f);
                if (co < a.split) {
                    const size_t o = (size_t)v * a.split + co;
                    if (a.out_f32) reinterpret_cast<float*>(a.out)[o] = val;
                    else reinterpret_cast<u16*>(a.out)[o] = f2bf(val);
                } else {
                    const int c2 = a.cout - a.split;
                    const size_t o = (size_t)v * c2 + (co - a.split);
                    if (a.out_f32) reinterpret_cast<float*>(a.out2)[o] = val;
                    else reinterpret_cast<u16*>(a.out2)[o] = f2bf(val);
                }
            }
        }
}

// The block of a 3-D grid that this workgroup takes.  Workgroups go to the
// eight XCDs in turn, each with an L2 of its own: each XCD takes one contiguous
// range of the blocks, so that neighbours read their common halo through one L2.
__device__ __forceinline__ int3 xcd_block()
{
    const unsigned id = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned n = gridDim.x * gridDim.y * gridDim.z, x = id & 7;
    const unsigned b = x * (n >> 3) + min(x, n & 7) + (id >> 3);
    const unsigned r = b / gridDim.x;
    return int3{(int)(b - r * gridDim.x), (int)(r % gridDim.y), (int)(r / gridDim.y)};
}

constexpr int kTX = 16, kTY = 4;
constexpr int kHX = kTX + 2, kHY = kTY + 2;

// What a tap outside the grid reads: selecting the address rather than the loaded
// value keeps a thread's loads in flight together.
__device__ __attribute__((aligned(16))) unsigned kZeroVoxel[4];

__device__ __forceinline__ uint4 load_or_zero(const u16* p, bool ok)
{
    // both addresses in the global address space: a generic load would also wait
    // for LDS
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) u32x4* GlobalPtr;
    const u32x4 q = *(ok ? (GlobalPtr)p : (GlobalPtr)kZeroVoxel);
    return uint4{q.x, q.y, q.z, q.w};
}

__device__ __forceinline__ u16 load_or_zero16(const u16* p, bool ok)
{
    typedef const __attribute__((address_space(1))) u16* GlobalPtr;
    return *(ok ? (GlobalPtr)p : (GlobalPtr)kZeroVoxel);
}

// The 8 channels [ci, ci + 8) of input voxel (x, y, z) on the output grid (the
// upsampled and the concatenated inputs resolved), zero outside the grid.
__device__ __forceinline__ uint4 conv_input(const ConvFwd& a, int x, int y, int z, int ci)
{
    const bool ok = (unsigned)x < (unsigned)a.W && (unsigned)y < (unsigned)a.H && (unsigned)z < (unsigned)a.D;
    const int xc = ok ? x : 0, yc = ok ? y : 0, zc = ok ? z : 0;
    const u16* src = ci < a.c0
        ? a.in0 + (((size_t)(zc >> a.up) * (a.H >> a.up) + (yc >> a.up)) * (a.W >> a.up) + (xc >> a.up)) * a.c0 + ci
        : a.in1 + (((size_t)zc * a.H + yc) * a.W + xc) * a.c1 + (ci - a.c0);
    return load_or_zero(src, ok);
}

// Whether four channels of an output voxel can be stored at once.
__device__ __forceinline__ bool conv_vec(const ConvFwd& a)
{
    return ((a.split | (a.cout - a.split)) & 3) == 0 &&
           ((reinterpret_cast<uintptr_t>(a.out) | reinterpret_cast<uintptr_t>(a.out2)) & 15) == 0;
}

// Two floats rounded to nearest even BF16 (NaN stays NaN).
__device__ __forceinline__ unsigned f2bf2(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v{(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(unsigned, v);
}

// Bias, ReLU and store (BF16 or FP32, split in two channel ranges for the input
// gradient of a concatenation) of a wave's M x NW accumulators: vox(m) is the lane's
// voxel of row m (negative: none), [c16 + 16 t + 4 kg, + 4) its channels.
template <int M, int NW, class Vox>
__device__ __forceinline__ void conv_epilogue(const ConvFwd& a, const f32x4 (&acc)[M][NW], int c16, int kg, Vox vox)
{
    const bool vec = conv_vec(a);
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        const int co = c16 + t * 16 + 4 * kg;
        if (co >= a.cout) continue;
        float b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = a.bias && co + i < a.cout ? a.bias[co + i] : 0.0f;
        auto value = [&](int m, int i) {
            const float v = acc[m][t][i] + b[i];
            return a.relu ? fmaxf(v, 0.0f) : v;
        };
        if (vec) {
            const bool first = co < a.split;
            const int st = first ? a.split : a.cout - a.split, c = first ? co : co - a.split;
            void* out = first ? a.out : a.out2;
            if (a.out_f32) {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const int v = vox(m);
                    if (v >= 0)
                        *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + (size_t)(unsigned)v * (unsigned)st + c) =
                            float4{value(m, 0), value(m, 1), value(m, 2), value(m, 3)};
                }
            } else {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const int v = vox(m);
                    if (v >= 0)
                        *reinterpret_cast<uint2*>(reinterpret_cast<u16*>(out) + (size_t)(unsigned)v * (unsigned)st + c) =
                            uint2{f2bf2(value(m, 0), value(m, 1)), f2bf2(value(m, 2), value(m, 3))};
                }
            }
            continue;
        }
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int v = vox(m);
            if (v < 0) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (co + i >= a.cout) continue;
                const bool first = co + i < a.split;
                const size_t o = first ? (size_t)v * a.split + co + i
                                       : (size_t)v * (a.cout - a.split) + (co + i - a.split);
                void* out = first ? a.out : a.out2;
                if (a.out_f32) reinterpret_cast<float*>(out)[o] = value(m, i);
                else reinterpret_cast<u16*>(out)[o] = (u16)f2bf2(value(m, i), 0.0f);
            }
        }
    }
}

// 3x3x3 convolution of CIN = 16, 32 or 64 input channels, its input tile staged in
// LDS: a workgroup computes a 16 x 4 x TZ (x, y, z) block of output voxels and
// stages the block's input halo (18 x 6 x (TZ + 2) voxels, all channels) once,
// so each voxel fragment is one 16-byte LDS read instead of a global gather.  K
// runs over (tap, channel) as in the packed weights.  WN waves share a row of
// voxels and split the output channels, so a wave has WN rows x TZ planes of 16
// voxels and NT / WN channel tiles.  The weights are the matrix instruction's
// first operand: a lane then holds four consecutive channels of one voxel and
// stores them at once.
//
// What bounds it: the issue of vector instructions around the matrix ones, and the
// wait for the halo.  So a thread stages one (x, channel group) of many rows, all
// their loads in flight; the steps are unrolled, their LDS offsets immediates from
// a few lane bases; the weights' addresses are scalar.  WN is what reads the
// weights seldom enough: 64 -> 32 channels at 64^3, WN 1 112 us, WN 2 70 us.  With
// eight channel tiles that is 4 (WN 1, 2, 4 at 64^3: 16 -> 128 channels 89, 65,
// 57 us, 32 -> 128 97, 73, 70 us, 64 -> 128 429, 238, 150 us; 32^3 and 128^3 alike).
// Of the kernel with one staging load in flight, scattered stores and table offsets
// to this one: 16 -> 16 channels at 128^3 82 -> 61 us, 32 -> 16 163 -> 104, 64 -> 32
// at 64^3 137 -> 70 (418 TFLOP/s), 32 -> 32 at 64^3 46 -> 24 us.
template <int CIN, int NT, int TZ, int WN>
__global__ __launch_bounds__(256) void k_conv_fwd_tile(ConvFwd a)
{
    constexpr int kHZ = TZ + 2, NW = NT / WN, G = CIN / 8, kSteps = (27 * CIN + 31) / 32;
    extern __shared__ uint4 hs4[];                         // [kHZ][kHY][kHX][G], swizzled
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, kg = lane >> 4;
    const int3 blk = xcd_block();
    const int x0 = blk.x * kTX, y0 = blk.y * kTY, z0 = blk.z * TZ;
    {
        constexpr int kRow = kHX * G, kRows = kHY * kHZ;   // 16-byte items of a halo row, rows
        constexpr int kPass = 256 / kRow, kTrips = (kRows + kPass - 1) / kPass;
        constexpr int kBatch = kTrips <= 12 ? kTrips : (kTrips + 1) / 2;
        const int row0 = threadIdx.x / kRow, it = threadIdx.x % kRow, hx = it / G, g = it % G;
        const bool first = g * 8 < a.c0;
        const int sh = first ? a.up : 0, cst = first ? a.c0 : a.c1;
        const u16* src = first ? a.in0 + g * 8 : a.in1 + (g * 8 - a.c0);
        const int x = x0 + hx - 1, Wl = a.W >> sh, Hl = a.H >> sh;
        const bool okx = (unsigned)x < (unsigned)a.W;
        if (row0 < kPass)
#pragma unroll
            for (int b0 = 0; b0 < kTrips; b0 += kBatch) {
                uint4 q[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const int row = row0 + (b0 + j) * kPass, hz = row / kHY, hy = row - hz * kHY;
                    const int y = y0 + hy - 1, z = z0 + hz - 1;
                    const bool ok = okx && (unsigned)y < (unsigned)a.H && (unsigned)z < (unsigned)a.D;
                    const int vox = ok ? ((z >> sh) * Hl + (y >> sh)) * Wl + (x >> sh) : 0;
                    q[j] = load_or_zero(src + (size_t)(unsigned)vox * (unsigned)cst, ok);
                }
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const int row = row0 + (b0 + j) * kPass, vox = row * kHX + hx;
                    if (row < kRows) hs4[vox * G + (g ^ conv_swizzle<CIN>(vox))] = q[j];
                }
            }
    }
    const int wy = wave / WN * WN, c16 = wave % WN * NW * 16;
    // the fragment at tap (dz, dy, dx) of the lane's voxel (x0 + r, y0 + wy + j,
    // z0 + m) starts at halo voxel vb + c, c = (m + dz) 108 + (j + dy) 18 + dx (taps
    // counted from 0); the swizzle repeats with c mod 4
    const int vb = wy * kHX + r;
    constexpr int kBases = CIN == 16 ? 4 : 4 * (CIN / 32);
    int base[kBases];
    if constexpr (CIN == 16) {
        // a step's taps t and t + 1 are 1, 16 (next row) or 70 (next plane) voxels
        // apart; the last step has tap 26 alone
        base[0] = (vb + (kg >> 1)) * G + (kg & 1);
        base[1] = (vb + (kg >> 1) * 16) * G + (kg & 1);
        base[2] = (vb + (kg >> 1) * 70) * G + (kg & 1);
        base[3] = vb * G + (kg & 1);
    } else {
#pragma unroll
        for (int i = 0; i < kBases; ++i)
            base[i] = vb * G + ((kg + i / 4 * 4) ^ conv_swizzle<CIN>(vb + i % 4));
    }
    f32x4 acc[WN * TZ][NW];
#pragma unroll
    for (int m = 0; m < WN * TZ; ++m)
#pragma unroll
        for (int t = 0; t < NW; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the weight fragments of the next P steps are in flight
    constexpr int P = NW == 1 ? 6 : NW == 2 ? (TZ == 8 ? 3 : 4) : 2;
    const unsigned boff = (unsigned)(r * a.Kp + 8 * kg);
    Frag Bq[P][NW];
    auto loadB = [&](Frag (&b)[NW], int ks) {
#pragma unroll
        for (int t = 0; t < NW; ++t)
            b[t].q = *reinterpret_cast<const uint4*>(a.wt + (size_t)(c16 + t * 16) * a.Kp + ks * 32 + boff);
    };
#pragma unroll
    for (int p = 0; p < P; ++p) loadB(Bq[p], p);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        const int tap = s * 32 / CIN;
        const int tv = (tap / 9 * kHY + tap / 3 % 3) * kHX + tap % 3;
        const bool pad = CIN == 16 && s == kSteps - 1;
        Frag A[WN * TZ];
#pragma unroll
        for (int m = 0; m < WN * TZ; ++m) {
            const int c = tv + m / WN * (kHY * kHX) + m % WN * kHX;
            const int bi = CIN == 16 ? (pad ? 3 : tap % 3 != 2 ? 0 : tap % 9 != 8 ? 1 : 2)
                                     : c % 4 + s % (CIN / 32 + (CIN == 16)) * 4;
            A[m].q = hs4[base[bi] + c * G];
            if (pad && kg >= 2) A[m].q = uint4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int m = 0; m < WN * TZ; ++m)
#pragma unroll
            for (int t = 0; t < NW; ++t)
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bq[s % P][t].v, A[m].v, acc[m][t], 0, 0, 0);
        if (s + P < kSteps) loadB(Bq[s % P], s + P);
    }
    // epilogue: rows 4 kg .. 4 kg + 3 of column r are four channels of voxel x0 + r
    conv_epilogue(a, acc, c16, kg, [&](int m) {
        const int z = z0 + m / WN, y = y0 + wy + m % WN;
        return x0 + r < a.W && y < a.H && z < a.D ? (z * a.H + y) * a.W + x0 + r : -1;
    });
}

// The same for any other multiple of 8 input channels up to 64: halo offsets from
// a table in LDS, a wave has one row of voxels and all channel tiles.
template <int NT, int TZ>
__global__ __launch_bounds__(256) void k_conv_fwd_lds(ConvFwd a)
{
    constexpr int kHZ = TZ + 2, NW = NT, M = TZ;
    extern __shared__ uint4 hs4[];
    u16* hs = reinterpret_cast<u16*>(hs4);                 // [kHZ][kHY][kHX][cin]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int cin = a.c0 + a.c1;
    const int3 blk = xcd_block();
    const int x0 = blk.x * kTX, y0 = blk.y * kTY, z0 = blk.z * TZ;
    // stage the halo in 8-channel groups (16 bytes; c0 and c1 are multiples of 8),
    // kStage of them in flight per thread: one trip at the most channels that this
    // TZ is chosen for
    constexpr int kStage = TZ == 8 ? 9 : TZ == 4 ? 11 : 14;
    const int groups = cin >> 3;
    // groups is a power of two for 8, 16, 32 and 64 channels: split i by shifts
    const bool gpow2 = (groups & (groups - 1)) == 0;
    const int lg = __ffs(groups) - 1;
    const int items = kHX * kHY * kHZ * groups;
    for (int i0 = threadIdx.x; i0 < items; i0 += 256 * kStage) {
        uint4 q[kStage];
        int dst[kStage];
#pragma unroll
        for (int j = 0; j < kStage; ++j) {
            const int i = min(i0 + 256 * j, items - 1);
            const int g = gpow2 ? (i & (groups - 1)) : i % groups;
            const int vox = gpow2 ? (i >> lg) : i / groups;
            const int hx = vox % kHX, hy = (vox / kHX) % kHY, hz = vox / (kHX * kHY);
            dst[j] = vox * cin + g * 8;
            q[j] = conv_input(a, x0 + hx - 1, y0 + hy - 1, z0 + hz - 1, g * 8);
        }
        // an index past the last repeats the last: the same value again
#pragma unroll
        for (int j = 0; j < kStage; ++j) *reinterpret_cast<uint4*>(hs + dst[j]) = q[j];
    }
    // per K-step and lane group: the halo offset (in u16) of the 8 channels
    // [ci, ci + 8) of tap (dz, dy, dx), relative to the lane's output voxel;
    // steps past the 27 taps (K padding, zero weights) point at offset 0 and
    // their voxel fragment is zeroed below
    const int nsteps = a.Kp >> 5;
    int* koff = reinterpret_cast<int*>(hs + (size_t)kHX * kHY * kHZ * cin);
    for (int i = threadIdx.x; i < nsteps * 4; i += 256) {
        const int k = (i >> 2) * 32 + 8 * (i & 3);
        const int tap = k / cin, ci = k - tap * cin;
        int off = 0;
        if (tap < 27) {
            const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
            off = ((dz * kHY + dy) * kHX + dx) * cin + ci;
        }
        koff[i] = off;
    }
    __syncthreads();
    f32x4 acc[M][NW];
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int t = 0; t < NW; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the lane's output voxel (x0 + r, y0 + wave, z0 + m) sits at halo
    // (1 + r, 1 + wave, 1 + m)
    const u16* abase = hs + (size_t)(((1 * kHY + 1 + wave) * kHX) + 1 + r) * cin;
    const int zstride = kHY * kHX * cin;
    const u16* bbase = a.wt + (size_t)r * a.Kp + 8 * kg;
    auto loadB = [&](Frag (&b)[NW], int ks) {
#pragma unroll
        for (int t = 0; t < NW; ++t)
            b[t].q = *reinterpret_cast<const uint4*>(bbase + (size_t)t * 16 * a.Kp + ks * 32);
    };
    // only the last step can hold K padding
    auto mma = [&](const Frag (&b)[NW], int off, bool pad_step, int ks) {
        const bool ok = !pad_step || (ks * 32 + 8 * kg) < 27 * cin;
        Frag A[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            A[m].q = *reinterpret_cast<const uint4*>(abase + m * zstride + off);
            if (pad_step) A[m].q = ok ? A[m].q : uint4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int t = 0; t < NW; ++t)
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[t].v, A[m].v, acc[m][t], 0, 0, 0);
    };
    // the weight fragments and halo offsets of the next P steps are in flight
    // while a step runs its MFMAs
    constexpr int P = NW == 2 ? 3 : 2;
    Frag Bq[P][NW];
    int offq[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        offq[p] = p < nsteps ? koff[p * 4 + kg] : 0;
        if (p < nsteps) loadB(Bq[p], p);
    }
    int ks0 = 0;
    for (; ks0 + 2 * P < nsteps; ks0 += P) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            mma(Bq[p], offq[p], false, ks0 + p);
            loadB(Bq[p], ks0 + p + P);
            offq[p] = koff[(ks0 + p + P) * 4 + kg];
        }
    }
    for (; ks0 < nsteps; ks0 += P) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int ks = ks0 + p;
            if (ks < nsteps) {
                mma(Bq[p], offq[p], ks == nsteps - 1, ks);
                if (ks + P < nsteps) {
                    loadB(Bq[p], ks + P);
                    offq[p] = koff[(ks + P) * 4 + kg];
                }
            }
        }
    }
    // epilogue: rows 4 kg .. 4 kg + 3 of column r are four channels of voxel x0 + r
    conv_epilogue(a, acc, 0, kg, [&](int m) {
        const int z = z0 + m, y = y0 + wave;
        return x0 + r < a.W && y < a.H && z < a.D ? (z * a.H + y) * a.W + x0 + r : -1;
    });
}

// 3x3x3 convolution of CIN = 32, 64, 96 or 128 input channels, one plane of the
// halo at a time: the taps run plane by plane (dz = -1, 0, 1), so a workgroup that
// computes 16 x 4 x 1 output voxels and NT tiles of 16 channels needs one
// 18 x 6 x 1 plane in LDS, and loads the next one into registers while it works.
// For many channels (a whole halo does not fit) and for small grids (where the
// whole-halo kernel's blocks leave compute units idle).  K order, waves and
// operands as in k_conv_fwd_tile.  What bounds it: the weights' reads through L1.
// 128 -> 64 channels at 32^3: gathered from global memory 99 us, here 51; 128 ->
// 128 at 16^3 60 -> 29 us; 64 -> 64 at 32^3 26 us with whole halos, 20 here.
template <int NT, int WN, int CIN>
__global__ __launch_bounds__(256) void k_conv_fwd_planes(ConvFwd a, int ncb)
{
    constexpr int NW = NT / WN, CC = CIN / 32, S = 9 * CC, G = CIN / 8;
    constexpr int kItems = kHX * kHY * G, kStage = (kItems + 255) / 256;
    __shared__ uint4 hs4[kHX * kHY * G];                   // [kHY][kHX][G], swizzled
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, kg = lane >> 4;
    const int3 blk = xcd_block();
    const int x0 = blk.x / ncb * kTX, y0 = blk.y * kTY, z = blk.z;
    const int wy = wave / WN * WN;
    const int c16 = (blk.x % ncb * NT + wave % WN * NW) * 16;
    uint4 q[kStage];
    auto fetch = [&](int dz) {
#pragma unroll
        for (int j = 0; j < kStage; ++j) {
            const int i = min((int)threadIdx.x + 256 * j, kItems - 1), vox = i / G;
            q[j] = conv_input(a, x0 + vox % kHX - 1, y0 + vox / kHX - 1, z + dz, i % G * 8);
        }
    };
    f32x4 acc[WN][NW];
#pragma unroll
    for (int m = 0; m < WN; ++m)
#pragma unroll
        for (int t = 0; t < NW; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // lane bases of the fragments, as in k_conv_fwd_tile
    const int vb = wy * kHX + r;
    constexpr int kBases = CIN % 64 ? 4 : 8;
    int base[kBases];
#pragma unroll
    for (int i = 0; i < kBases; ++i) base[i] = vb * G + ((kg + i / 4 * 4) ^ conv_swizzle<CIN>(vb + i % 4));
    const unsigned boff = (unsigned)(r * a.Kp + 8 * kg);
    constexpr int P = 3;                                   // divides S
    Frag Bq[P][NW];
    auto loadB = [&](Frag (&b)[NW], int ks) {
#pragma unroll
        for (int t = 0; t < NW; ++t)
            b[t].q = *reinterpret_cast<const uint4*>(a.wt + (size_t)(c16 + t * 16) * a.Kp + ks * 32 + boff);
    };
    fetch(-1);
#pragma unroll
    for (int p = 0; p < P; ++p) loadB(Bq[p], p);
    for (int dz = 0; dz < 3; ++dz) {
        if (dz) __syncthreads();                           // the plane before is consumed
#pragma unroll
        for (int j = 0; j < kStage; ++j) {
            const int i = min((int)threadIdx.x + 256 * j, kItems - 1);
            hs4[i / G * G + (i % G ^ conv_swizzle<CIN>(i / G))] = q[j];
        }
        __syncthreads();
        if (dz < 2) fetch(dz);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int tv = s / CC / 3 * kHX + s / CC % 3, ck = s % CC;
            Frag A[WN];
#pragma unroll
            for (int m = 0; m < WN; ++m) {
                const int c = tv + m * kHX;
                A[m].q = hs4[base[c % 4 + (kBases == 8 ? ck % 2 * 4 : 0)] + c * G + (kBases == 8 ? ck / 2 * 8 : ck * 4)];
            }
#pragma unroll
            for (int m = 0; m < WN; ++m)
#pragma unroll
                for (int t = 0; t < NW; ++t)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bq[s % P][t].v, A[m].v, acc[m][t], 0, 0, 0);
            loadB(Bq[s % P], min(dz * S + s + P, 3 * S - 1));
        }
    }
    conv_epilogue(a, acc, c16, kg, [&](int m) {
        const int y = y0 + wy + m;
        return x0 + r < a.W && y < a.H ? (z * a.H + y) * a.W + x0 + r : -1;
    });
}

// 3x3x3 convolution of a single input channel (the network's input layer),
// up to 16 output channels: 27 MACs per output channel, so FP32 FMAs on the
// BF16 values (their products are exact in FP32) instead of MFMAs whose K
// values would each be a separately gathered tap.  A workgroup stages the
// input halo of a 16 x 4 x 4 VZ output block in LDS; each thread computes the
// channels of VZ output voxels along z.
//
// What bounds it: the FMAs, and the weights' loads and conversions to FP32, which
// VZ voxels share: 16 channels of 128^3 voxels 68 -> 50 us with VZ = 4.
template <int VZ>
__global__ __launch_bounds__(256) void k_conv_fwd_c1(ConvFwd a)
{
    constexpr int kHZ = 4 * VZ + 2;
    __shared__ float halo[kHZ][6][18];
    const int x0 = blockIdx.x * 16, y0 = blockIdx.y * 4, z0 = blockIdx.z * 4 * VZ;
    const int Hin = a.H >> a.up, Win = a.W >> a.up;
#pragma unroll 4
    for (int i = threadIdx.x; i < 18 * 6 * kHZ; i += 256) {
        const int hx = i % 18, hy = (i / 18) % 6, hz = i / 108;
        const int x = x0 + hx - 1, y = y0 + hy - 1, z = z0 + hz - 1;
        const bool ok = (unsigned)x < (unsigned)a.W && (unsigned)y < (unsigned)a.H && (unsigned)z < (unsigned)a.D;
        const size_t src = ((size_t)(z >> a.up) * Hin + (y >> a.up)) * Win + (x >> a.up);
        const u16 v = a.in0[ok ? src : 0];
        halo[hz][hy][hx] = ok ? bf2f(v) : 0.0f;
    }
    __syncthreads();
    const int tx = threadIdx.x & 15, ty = (threadIdx.x >> 4) & 3, tz = (threadIdx.x >> 6) * VZ;
    const int x = x0 + tx, y = y0 + ty;
    if (x >= a.W || y >= a.H) return;
    float v[VZ + 2][9];
#pragma unroll
    for (int p = 0; p < VZ + 2; ++p)
#pragma unroll
        for (int t = 0; t < 9; ++t) v[p][t] = halo[tz + p][ty + t / 3][tx + t % 3];
    const size_t vox = ((size_t)(z0 + tz) * a.H + y) * a.W + x, plane = (size_t)a.H * a.W;
    // one voxel's 16 BF16 channels leave as two 16-byte stores
    const bool whole = !a.out_f32 && a.split == 16 && a.cout == 16 && (reinterpret_cast<uintptr_t>(a.out) & 15) == 0;
    unsigned packed[VZ][8];
#pragma unroll
    for (int c2 = 0; c2 < 8; ++c2) {
        float out[2][VZ];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int co = min(2 * c2 + h, a.cout - 1);    // past the last: repeated, not stored
            const u16* wr = a.wt + (size_t)co * a.Kp;
#pragma unroll
            for (int j = 0; j < VZ; ++j) out[h][j] = 0.0f;
#pragma unroll
            for (int t = 0; t < 27; ++t) {
                const float w = bf2f(wr[t]);
#pragma unroll
                for (int j = 0; j < VZ; ++j) out[h][j] = fmaf(w, v[j + t / 9][t % 9], out[h][j]);
            }
            const float b = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
            for (int j = 0; j < VZ; ++j) {
                out[h][j] += b;
                if (a.relu) out[h][j] = fmaxf(out[h][j], 0.0f);
            }
            if (!whole && 2 * c2 + h < a.cout) {
                const bool first = co < a.split;
                const int st = first ? a.split : a.cout - a.split, c = first ? co : co - a.split;
                void* dst = first ? a.out : a.out2;
#pragma unroll
                for (int j = 0; j < VZ; ++j) {
                    if (z0 + tz + j >= a.D) continue;
                    const size_t o = (vox + j * plane) * st + c;
                    if (a.out_f32) reinterpret_cast<float*>(dst)[o] = out[h][j];
                    else reinterpret_cast<u16*>(dst)[o] = (u16)f2bf2(out[h][j], 0.0f);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < VZ; ++j) packed[j][c2] = f2bf2(out[0][j], out[1][j]);
    }
    if (!whole) return;
#pragma unroll
    for (int j = 0; j < VZ; ++j) {
        if (z0 + tz + j >= a.D) continue;
        uint4* dst = reinterpret_cast<uint4*>(reinterpret_cast<u16*>(a.out) + (vox + j * plane) * 16);
        dst[0] = uint4{packed[j][0], packed[j][1], packed[j][2], packed[j][3]};
        dst[1] = uint4{packed[j][4], packed[j][5], packed[j][6], packed[j][7]};
    }
}

// ---------------------------------------------------------------- wgrad
// dW[co][k] += sum_v dY[v][co] X_k[v], k = tap * Cin + ci, X_k the input
// shifted by the tap (and upsampled when up = 1).  MFMA rows are output
// channels, columns are k, the reduction runs over 32 voxels of one output
// z-slice at a time.  A workgroup's 4 waves own 4 (co, k) tiles of one share
// of one slice (gridDim.z shares of its 32-voxel groups) and add them into
// the FP32 gradient with atomics.
template <int KS>
__global__ __launch_bounds__(256) void k_conv_wgrad(ConvWgrad a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int n_co = (a.cout + 15) / 16;
    const int n_k = (a.K + 15) / 16;
    const int tile = blockIdx.x * 4 + wave;
    if (tile >= n_co * n_k) return;
    const int cot = tile % n_co, kt = tile / n_co;
    const int z = blockIdx.y;
    const int HW = a.H * a.W;
    const int Hin = a.H >> a.up, Win = a.W >> a.up;
    const int cin = a.c0 + a.c1;
    const int co = cot * 16 + r;           // A row of this lane
    const int k = kt * 16 + r;             // B column of this lane
    const bool kvalid = k < a.K;
    const int tap = kvalid ? k / cin : 0, ci = kvalid ? k - tap * cin : 0;
    const int dz = KS == 3 ? tap / 9 - 1 : 0, dy = KS == 3 ? (tap / 3) % 3 - 1 : 0,
              dx = KS == 3 ? tap % 3 - 1 : 0;
    const int zz = z + dz;
    const bool zin = kvalid && zz >= 0 && zz < a.D;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    // this workgroup's share of the slice (gridDim.z shares of 32-voxel groups)
    const int ngroups = (HW + 31) / 32;
    const int g0 = (int)(((long long)ngroups * blockIdx.z) / gridDim.z);
    const int g1 = (int)(((long long)ngroups * (blockIdx.z + 1)) / gridDim.z);
    for (int v0 = g0 * 32; v0 < g1 * 32; v0 += 32) {
        Frag A, B;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int v = v0 + 8 * kg + j;
            u16 av = 0, bv = 0;
            if (v < HW) {
                if (co < a.cout) av = a.dy[((size_t)z * HW + v) * a.cout + co];
                const int y = v / a.W + dy, x = v % a.W + dx;
                if (zin && y >= 0 && y < a.H && x >= 0 && x < a.W) {
                    const size_t src = ((size_t)(zz >> a.up) * Hin + (y >> a.up)) * Win + (x >> a.up);
                    bv = ci < a.c0 ? a.in0[src * a.c0 + ci] : a.in1[src * a.c1 + (ci - a.c0)];
                }
            }
            A.h[j] = av;
            B.h[j] = bv;
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.v, B.v, acc, 0, 0, 0);
    }
    // D[row = 4 kg + i][col = r]: row is the output channel, col is k
    const int kc = kt * 16 + r;
    if (kc >= a.K) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = cot * 16 + 4 * kg + i;
        if (c < a.cout && acc[i] != 0.0f) unsafeAtomicAdd(&a.dw[(size_t)c * a.K + kc], acc[i]);
    }
}

// k_conv_wgrad for grids whose H and W are powers of two (H W a multiple of
// 32) and cout a multiple of 16: voxel coordinates by shifts, no branches in
// the operand loads (an out-of-range tap reads a valid address and selects
// zero), the input base pointer and channel stride of each lane hoisted, and
// each wave owning NK k-tiles of one output-channel tile, so one dY fragment
// feeds NK MFMAs.
template <int KS, int NK>
__global__ __launch_bounds__(256) void k_conv_wgrad_pow2(ConvWgrad a, int lw, int lh)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int n_co = a.cout >> 4;
    const int n_kg = ((a.K + 15) / 16 + NK - 1) / NK;
    const int tile = blockIdx.x * 4 + wave;
    if (tile >= n_co * n_kg) return;
    const int cot = tile % n_co, kgi = tile / n_co;
    const int z = blockIdx.y;
    const int W = 1 << lw, H = 1 << lh, HW = W * H;
    const int Hin = H >> a.up, Win = W >> a.up;
    const int cin = a.c0 + a.c1;
    const u16* dyz = a.dy + (size_t)z * HW * a.cout + cot * 16 + r;
    // per k-tile: this lane's B column k = tap * cin + ci
    const u16* base[NK];
    int cst[NK], ddy[NK], ddx[NK], zoff[NK];
    bool live[NK];
#pragma unroll
    for (int t = 0; t < NK; ++t) {
        const int k = (kgi * NK + t) * 16 + r;
        const bool kv = k < a.K;
        const int tap = kv ? k / cin : 0, ci = kv ? k - tap * cin : 0;
        const int dz = KS == 3 ? tap / 9 - 1 : 0;
        ddy[t] = KS == 3 ? (tap / 3) % 3 - 1 : 0;
        ddx[t] = KS == 3 ? tap % 3 - 1 : 0;
        const int zz = z + dz;
        live[t] = kv && zz >= 0 && zz < a.D;
        zoff[t] = live[t] ? (zz >> a.up) * Hin * Win : 0;
        base[t] = ci < a.c0 ? a.in0 + ci : a.in1 + (ci - a.c0);
        cst[t] = ci < a.c0 ? a.c0 : a.c1;
    }
    f32x4 acc[NK];
#pragma unroll
    for (int t = 0; t < NK; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // a wave walks a whole slice, U voxel groups at a time: all their loads
    // are issued before their MFMAs (a group past the slice loads group 0
    // and is skipped)
    constexpr int U = 4;
    // this workgroup's share of the slice's voxel groups (gridDim.z shares)
    const int ngroups = HW >> 5;
    const int sb = (int)(((long long)ngroups * blockIdx.z) / gridDim.z);
    const int nsteps = (int)(((long long)ngroups * (blockIdx.z + 1)) / gridDim.z);
    for (int s0 = sb; s0 < nsteps; s0 += U) {
        Frag A[U], B[U][NK];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int vb = (s0 + u < nsteps ? s0 + u : sb) * 32 + 8 * kg;
#pragma unroll
            for (int j = 0; j < 8; ++j) A[u].h[j] = dyz[(size_t)(vb + j) * a.cout];
            const int y0 = vb >> lw, x0 = vb & (W - 1);   // the 8 voxels share a row (W >= 8)
#pragma unroll
            for (int t = 0; t < NK; ++t) {
                const int y = y0 + ddy[t];
                const bool rowok = live[t] && (unsigned)y < (unsigned)H;
                const int rowoff = zoff[t] + (rowok ? (y >> a.up) : 0) * Win;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int x = x0 + j + ddx[t];
                    const bool ok = rowok && (unsigned)x < (unsigned)W;
                    const u16 val = base[t][(size_t)(rowoff + (ok ? (x >> a.up) : 0)) * cst[t]];
                    B[u][t].h[j] = ok ? val : (u16)0;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u >= nsteps) break;
#pragma unroll
            for (int t = 0; t < NK; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[u].v, B[u][t].v, acc[t], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < NK; ++t) {
        const int kc = (kgi * NK + t) * 16 + r;
        if (kc >= a.K) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = cot * 16 + 4 * kg + i;
            if (acc[t][i] != 0.0f) unsafeAtomicAdd(&a.dw[(size_t)c * a.K + kc], acc[t][i]);
        }
    }
}

// Weight gradient of a 3x3x3 convolution in chunks of XC (32, 64 or 128) voxels
// of a row (the last one zero past the row's end), Cin and Cout multiples of 16.  A tap's x shift
// is moved from the input onto dY: sum_x dY[x] X[x + dx] = sum_x' dY[x' - dx]
// X[x'], each input position x' paired by the unit that holds it.  A unit is
// XC voxels (chunk) of one output row (z, y).  Per unit a workgroup holds in
// LDS the 9 input rows (z + dz, y + dy) the taps reach, at the unit's own x
// range and for one 16-channel input tile, and the unit's dY for one
// 16-channel output tile in three copies shifted by dx = -1, 0, 1 (zeros
// outside the grid; upsampling and concatenation resolved while staging).
// Both are stored transposed, [channel][x], so every MFMA operand (8
// consecutive voxels of one channel) is one aligned 16-byte LDS read, and one
// input fragment feeds the three taps that differ only in dx.  Units run over
// (z, chunk, y) with y fastest: the input rows sit in a ring of 3 x 3 slots
// (slot (dz, y' mod 3)), so a unit after its y - 1 neighbour loads only the 3
// rows y + 1; and the next unit's loads are issued into registers before the
// current unit's MFMAs.  A workgroup owns (output tile, input tile, a
// contiguous share of the units); wave w holds the 9 k-tiles of dy = w - 1 in
// registers over its share and adds them into dw once.
//
// Rows of no whole chunk: an FP32 run ends after kRunUnits units and is added to the
// share's sum, as the kernels that gather voxel by voxel, which such rows came from,
// end one with each slice at the latest.  The second set of accumulators has to leave
// three waves per SIMD their registers: 64 -> 32 channels at 64 x 64 x 60 101 us, with two
// waves 132.  (Whole chunks keep to one run per share; a second set there, at rows of
// 128, costs the network's training step 9%.)
constexpr int kRunUnits = 8;

template <int XC>
struct WgradStage {
    static constexpr int NX8 = XC / 8;
    static constexpr int NIT = (9 * 2 * NX8 + 191) / 192;     // input items per thread (a full stage)
    static constexpr int NDI = (2 * (XC + 2) + 191) / 192;    // dY items per thread
    Frag q[NIT][8];
    Frag f[NDI];
};

template <int XC, bool kRagged>
__device__ __forceinline__ void wgrad_load(const ConvWgrad& a, int cit, int cot, int z, int y, int x0, bool full,
                                           WgradStage<XC>& st)
{
    constexpr int NX8 = XC / 8;
    const int nitems = (full ? 9 : 3) * 2 * NX8;
    const int Hin = a.H >> a.up, Win = a.W >> a.up;
#pragma unroll
    for (int it = 0; it < WgradStage<XC>::NIT; ++it) {
        const int i = (int)threadIdx.x + 192 * it;
        const int x8 = i % NX8, g = (i / NX8) & 1, rs = i / (2 * NX8);
        const int dzi = full ? rs / 3 : rs, k = full ? rs % 3 : 2;
        const int zz = z + dzi - 1, yy = y + k - 1;
        const int ci = cit * 16 + g * 8;
        const int xb = x0 + x8 * 8;
        auto voxel = [&](const u16* p, int x) {
            return !kRagged ? *reinterpret_cast<const uint4*>(p) : load_or_zero(p, x < a.W);
        };
        if (i < nitems && (unsigned)zz < (unsigned)a.D && (unsigned)yy < (unsigned)a.H) {
            if (ci < a.c0) {
                const u16* src = a.in0 + ((size_t)(zz >> a.up) * Hin + (yy >> a.up)) * Win * a.c0 + ci;
#pragma unroll
                for (int jx = 0; jx < 8; ++jx)
                    st.q[it][jx].q = voxel(src + (size_t)((xb + jx) >> a.up) * a.c0, xb + jx);
            } else {
                const u16* src = a.in1 + ((size_t)zz * a.H + yy) * a.W * a.c1 + (ci - a.c0);
#pragma unroll
                for (int jx = 0; jx < 8; ++jx)
                    st.q[it][jx].q = voxel(src + (size_t)(xb + jx) * a.c1, xb + jx);
            }
        } else {
#pragma unroll
            for (int jx = 0; jx < 8; ++jx) st.q[it][jx].q = uint4{0u, 0u, 0u, 0u};
        }
    }
    const size_t rowbase = ((size_t)z * a.H + y) * a.W;
#pragma unroll
    for (int it = 0; it < WgradStage<XC>::NDI; ++it) {
        const int i = (int)threadIdx.x + 192 * it;
        const int h = i >> 1, half = i & 1;
        const int x = x0 - 1 + h;
        st.f[it].q = (i < 2 * (XC + 2) && (unsigned)x < (unsigned)a.W)
            ? *reinterpret_cast<const uint4*>(a.dy + (rowbase + x) * a.cout + cot * 16 + half * 8)
            : uint4{0u, 0u, 0u, 0u};
    }
}

template <int XC>
__device__ __forceinline__ void wgrad_store(int y, bool full, const WgradStage<XC>& st, u16* xs, u16* dys)
{
    constexpr int NX8 = XC / 8, XS = XC + 8;
    const int nitems = (full ? 9 : 3) * 2 * NX8;
#pragma unroll
    for (int it = 0; it < WgradStage<XC>::NIT; ++it) {
        const int i = (int)threadIdx.x + 192 * it;
        if (i >= nitems) continue;
        const int x8 = i % NX8, g = (i / NX8) & 1, rs = i / (2 * NX8);
        const int dzi = full ? rs / 3 : rs, k = full ? rs % 3 : 2;
        const int slot = dzi * 3 + (y + k + 2) % 3;               // input row y + k - 1 -> slot (dz, y' mod 3)
        u16* dst = xs + (slot * 16 + g * 8) * XS + x8 * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            // channel j of voxels 2m, 2m + 1 -> one dword (low, high half)
            const unsigned sel = (j & 1) ? 0x07060302u : 0x05040100u;
            uint4 o;
            o.x = __builtin_amdgcn_perm(st.q[it][1].w[j >> 1], st.q[it][0].w[j >> 1], sel);
            o.y = __builtin_amdgcn_perm(st.q[it][3].w[j >> 1], st.q[it][2].w[j >> 1], sel);
            o.z = __builtin_amdgcn_perm(st.q[it][5].w[j >> 1], st.q[it][4].w[j >> 1], sel);
            o.w = __builtin_amdgcn_perm(st.q[it][7].w[j >> 1], st.q[it][6].w[j >> 1], sel);
            *reinterpret_cast<uint4*>(dst + j * XS) = o;
        }
    }
    // dY halo x0 - 1 + h: copy d (dx = d - 1) holds dY[x0 + i - dx] at i = h + d - 2
#pragma unroll
    for (int it = 0; it < WgradStage<XC>::NDI; ++it) {
        const int i = (int)threadIdx.x + 192 * it;
        if (i >= 2 * (XC + 2)) continue;
        const int h = i >> 1, half = i & 1;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int ix = h + d - 2;
            if ((unsigned)ix < (unsigned)XC) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    dys[(d * 16 + half * 8 + j) * XS + ix] = st.f[it].h[j];
            }
        }
    }
}

template <int XC, bool kRagged>
__global__ __launch_bounds__(192, kRagged && XC < 128 ? 3 : 1) void k_conv_wgrad_rows(ConvWgrad a, int nshare)
{
    constexpr int XS = XC + 8;                   // LDS row stride (elements), padded against bank conflicts
    extern __shared__ uint4 sm4[];
    u16* xs = reinterpret_cast<u16*>(sm4);       // [9 slots][16 channels][XS]
    u16* dys = xs + 9 * 16 * XS;                 // [3 shifts][16 channels][XS]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int n_co = a.cout >> 4;
    const int cot = blockIdx.x % n_co, cit = blockIdx.x / n_co;
    const int cin = a.c0 + a.c1;
    const int chunks = kRagged ? (a.W + XC - 1) / XC : a.W / XC;
    const int nunits = a.D * chunks * a.H;
    const int u0 = (int)(((long long)nunits * blockIdx.y) / nshare);
    const int u1 = (int)(((long long)nunits * (blockIdx.y + 1)) / nshare);
    f32x4 acc[3][3], runs[kRagged ? 3 : 1][kRagged ? 3 : 1];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            acc[s][d] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (kRagged) runs[s][d] = acc[s][d];
        }
    // unit -> (z, chunk, y), y fastest
    auto coords = [&](int unit, int& z, int& y, int& x0) {
        const int zc = unit / a.H;
        y = unit - zc * a.H;
        z = zc / chunks;
        x0 = (zc - z * chunks) * XC;
    };
    WgradStage<XC> st;
    int z, y, x0;
    if (u0 < u1) {
        coords(u0, z, y, x0);
        wgrad_load<XC, kRagged>(a, cit, cot, z, y, x0, true, st);
    }
    for (int unit = u0; unit < u1; ++unit) {
        const bool full = unit == u0 || y == 0;
        const int ycur = y;
        __syncthreads();   // the previous unit's fragments are read
        wgrad_store<XC>(ycur, full, st, xs, dys);
        __syncthreads();
        if (unit + 1 < u1) {
            coords(unit + 1, z, y, x0);
            wgrad_load<XC, kRagged>(a, cit, cot, z, y, x0, y == 0, st);
        }
        // wave w: dy = w - 1, input row y' = ycur + w - 1 in slot (s, y' mod 3)
        const int ks = (ycur + wave + 2) % 3;
#pragma unroll
        for (int gv = 0; gv < XC; gv += 32) {
            Frag A[3];
#pragma unroll
            for (int d = 0; d < 3; ++d)
                A[d].q = *reinterpret_cast<const uint4*>(dys + (d * 16 + r) * XS + gv + 8 * kg);
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                Frag B;
                B.q = *reinterpret_cast<const uint4*>(xs + ((s * 3 + ks) * 16 + r) * XS + gv + 8 * kg);
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    acc[s][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[d].v, B.v, acc[s][d], 0, 0, 0);
            }
        }
        if constexpr (kRagged)
            if ((unit - u0) % kRunUnits == kRunUnits - 1 || unit + 1 == u1) {
#pragma unroll
                for (int s = 0; s < 3; ++s)
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        runs[s][d] += acc[s][d];
                        acc[s][d] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
    }
    // D[4 kg + i][r]: output channel cot 16 + 4 kg + i, input channel
    // cit 16 + r of tap (dz = s - 1, dy = wave - 1, dx = d - 1)
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int k = ((s * 3 + wave) * 3 + d) * cin + cit * 16 + r;
            if constexpr (kRagged) acc[s][d] = runs[s][d];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = cot * 16 + 4 * kg + i;
                if (acc[s][d][i] != 0.0f) unsafeAtomicAdd(&a.dw[(size_t)c * a.K + k], acc[s][d][i]);
            }
        }
}

template <int XC>
hipError_t wgrad_rows(const ConvWgrad& a, hipStream_t s)
{
    const int tiles = (a.cout / 16) * ((a.c0 + a.c1) / 16);
    const int units = a.D * a.H * ((a.W + XC - 1) / XC);
    // shares of the units per (output tile, input tile) until two (rows of 128) or
    // three workgroups per compute unit run; each share adds its partial sums into
    // dw.  2, 3 and 5 of them: 16 -> 16 channels at 128^3 80, 114 (2.5) and 110 us (3),
    // 64 -> 64 at 32^3 82, 68 and 65, 32 -> 64 at 32^3 52, 44 and 48, 64 -> 32 at 64^3 95,
    // 78 and 95 us: beyond three the adds to one address, one after the other, cost more
    // (four, in a training step: 60 us more over its ten layers of 64^3 and 32^3 voxels,
    // though called over and over on one input they are faster)
    const size_t lds = (size_t)12 * 16 * (XC + 8) * sizeof(u16);
    const int shares = std::max(1, std::min(units, (XC == 128 ? 512 : 768) / tiles));
    if (a.W % XC)
        hipLaunchKernelGGL((k_conv_wgrad_rows<XC, true>), dim3(tiles, shares), dim3(192), lds, s, a, shares);
    else
        hipLaunchKernelGGL((k_conv_wgrad_rows<XC, false>), dim3(tiles, shares), dim3(192), lds, s, a, shares);
    return hipGetLastError();
}

// Weight gradient of a 3x3x3 convolution with one input channel (the input
// layer) on rows of XC (32, 64 or 128) voxels.  With one channel, the 9 input
// rows (z + dz, y + dy) a unit's taps reach are the columns of one MFMA B
// operand (9 of 16 used), staged in three copies shifted by dx = -1, 0, 1
// (zeros outside the grid); the unit's dY of one 16-channel output tile is
// staged transposed, [co][x].  Each 32 voxels take 3 MFMAs (one per x shift)
// into D[co][row], tap = row * 3 + d; a wave takes every fourth group of 32
// voxels, and the workgroup sums its waves in LDS and adds into dw once.
template <int XC>
__global__ __launch_bounds__(256) void k_conv_wgrad_c1(ConvWgrad a, int nshare)
{
    constexpr int XS = XC + 8;
    __shared__ __align__(16) u16 xs[3 * 16 * XS];   // [shift][row][x]; rows 9..15 stay zero
    __shared__ __align__(16) u16 dys[16 * XS];      // [co][x]
    __shared__ float red[27 * 16];                  // [tap][co]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int cot = blockIdx.x;
    const int chunks = (a.W + XC - 1) / XC;
    const int nunits = a.D * a.H * chunks;
    const int u0 = (int)(((long long)nunits * blockIdx.y) / nshare);
    const int u1 = (int)(((long long)nunits * (blockIdx.y + 1)) / nshare);
    for (int i = threadIdx.x; i < 3 * 16 * XS; i += 256) xs[i] = 0;
    for (int i = threadIdx.x; i < 27 * 16; i += 256) red[i] = 0.0f;
    f32x4 acc[3], runs[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) acc[d] = runs[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    // a unit's loads are in flight while the one before is multiplied
    constexpr int NI = (9 * (XC + 2) + 255) / 256;
    u16 q[NI];
    Frag f{};
    auto load = [&](int unit) {
        const int row = unit / chunks, x0 = (unit - row * chunks) * XC;
        const int z = row / a.H, y = row - z * a.H;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int i = threadIdx.x + 256 * j, rr = i / (XC + 2), h = i - rr * (XC + 2);
            const int zz = z + rr / 3 - 1, yy = y + rr % 3 - 1, x = x0 - 1 + h;
            const bool ok = rr < 9 && (unsigned)zz < (unsigned)a.D && (unsigned)yy < (unsigned)a.H &&
                            (unsigned)x < (unsigned)a.W;
            q[j] = load_or_zero16(a.in0 + (ok ? ((size_t)zz * a.H + yy) * a.W + x : 0), ok);
        }
        const int x = threadIdx.x >> 1;
        if (threadIdx.x < XC * 2)
            f.q = load_or_zero(a.dy + ((size_t)row * a.W + min(x0 + x, a.W - 1)) * a.cout + cot * 16 +
                                   (threadIdx.x & 1) * 8, x0 + x < a.W);
    };
    if (u0 < u1) load(u0);
    auto run = [&](int ua, int ub) {
        for (int unit = ua; unit < ub; ++unit) {
            __syncthreads();   // the previous unit's fragments are read (and the clears done)
            // input halo x0 - 1 + h: copy d (dx = d - 1) holds X[x0 + i + dx] at i = h - d
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int i = threadIdx.x + 256 * j, rr = i / (XC + 2), h = i - rr * (XC + 2);
                if (rr >= 9) continue;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const int ix = h - d;
                    if ((unsigned)ix < (unsigned)XC) xs[(d * 16 + rr) * XS + ix] = q[j];
                }
            }
            if (threadIdx.x < XC * 2) {
#pragma unroll
                for (int j = 0; j < 8; ++j) dys[((threadIdx.x & 1) * 8 + j) * XS + (threadIdx.x >> 1)] = f.h[j];
            }
            __syncthreads();
            if (unit + 1 < u1) load(unit + 1);
            for (int gv = wave * 32; gv < XC; gv += 128) {
                Frag A;
                A.q = *reinterpret_cast<const uint4*>(dys + r * XS + gv + 8 * kg);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    Frag B;
                    B.q = *reinterpret_cast<const uint4*>(xs + (d * 16 + r) * XS + gv + 8 * kg);
                    acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A.v, B.v, acc[d], 0, 0, 0);
                }
            }
        }
    };
    for (int ua = u0; ua < u1; ua += kRunUnits) {
        run(ua, min(ua + kRunUnits, u1));
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            runs[d] += acc[d];
            acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // D[4 kg + i][r]: output channel cot 16 + 4 kg + i, input row r (< 9),
    // x shift d -> tap r * 3 + d
    if (r < 9) {
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (runs[d][i] != 0.0f) atomicAdd(&red[(r * 3 + d) * 16 + 4 * kg + i], runs[d][i]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 27 * 16; i += 256) {
        const int tap = i >> 4, co = i & 15;
        if (red[i] != 0.0f) unsafeAtomicAdd(&a.dw[(size_t)(cot * 16 + co) * a.K + tap], red[i]);
    }
}

template <int XC>
hipError_t wgrad_c1(const ConvWgrad& a, hipStream_t s)
{
    const int cot = a.cout / 16;
    const int units = a.D * a.H * ((a.W + XC - 1) / XC);
    // shares of the units until 512 workgroups run; each adds 16 x 27 sums, one after
    // the other at each address (128^3: 256 shares 120 us, 512 107, 1024 146).  The FP32
    // runs end within a share (kRunUnits), so that fewer shares do not lengthen them
    const int shares = std::max(1, std::min(units, 512 / cot));
    hipLaunchKernelGGL((k_conv_wgrad_c1<XC>), dim3(cot, shares), dim3(256), 0, s, a, shares);
    return hipGetLastError();
}

// Weight gradient of a 1x1x1 convolution to one output channel (the output
// layer): dw[ci] += sum_v dY[v] X[v][ci].  Each thread sums its voxels' CIN
// channels in registers (16-byte loads), then waves and the workgroup combine
// them, one atomic per channel and workgroup.
template <int CIN>
__global__ __launch_bounds__(kSumBlock) void k_wgrad_1x1_out1(ConvWgrad a, size_t nvox)
{
    __shared__ float red[CIN];
    if (threadIdx.x < CIN) red[threadIdx.x] = 0.0f;
    __syncthreads();
    float sum[CIN];
#pragma unroll
    for (int c = 0; c < CIN; ++c) sum[c] = 0.0f;
    for (size_t v = (size_t)blockIdx.x * kSumBlock + threadIdx.x; v < nvox; v += (size_t)gridDim.x * kSumBlock) {
        const float g = bf2f(a.dy[v]);
        const u16* x = a.in0 + v * CIN;
#pragma unroll
        for (int c8 = 0; c8 < CIN; c8 += 8) {
            Frag q;
            q.q = *reinterpret_cast<const uint4*>(x + c8);
#pragma unroll
            for (int j = 0; j < 8; ++j) sum[c8 + j] = fmaf(g, bf2f(q.h[j]), sum[c8 + j]);
        }
    }
#pragma unroll
    for (int c = 0; c < CIN; ++c) {
        float t = sum[c];
        for (int o = 32; o >= 1; o >>= 1) t += __shfl_xor(t, o);
        if ((threadIdx.x & 63) == 0 && t != 0.0f) atomicAdd(&red[c], t);
    }
    __syncthreads();
    if (threadIdx.x < CIN && red[threadIdx.x] != 0.0f) unsafeAtomicAdd(&a.dw[threadIdx.x], red[threadIdx.x]);
}

// 1x1x1 convolution to one output channel (the output layer): each voxel's
// CIN channels (16-byte loads) dotted with the weight row, plus bias, ReLU if
// asked.
template <int CIN>
__global__ __launch_bounds__(256) void k_conv1x1_out1(ConvFwd a, size_t nvox)
{
    float w[CIN];
#pragma unroll
    for (int c8 = 0; c8 < CIN; c8 += 8) {
        Frag q;
        q.q = *reinterpret_cast<const uint4*>(a.wt + c8);
#pragma unroll
        for (int j = 0; j < 8; ++j) w[c8 + j] = bf2f(q.h[j]);
    }
    const float b = a.bias ? a.bias[0] : 0.0f;
    for (size_t v = (size_t)blockIdx.x * 256 + threadIdx.x; v < nvox; v += (size_t)gridDim.x * 256) {
        const u16* x = a.in0 + v * CIN;
        float acc = 0.0f;
#pragma unroll
        for (int c8 = 0; c8 < CIN; c8 += 8) {
            Frag q;
            q.q = *reinterpret_cast<const uint4*>(x + c8);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = fmaf(bf2f(q.h[j]), w[c8 + j], acc);
        }
        acc += b;
        if (a.relu) acc = fmaxf(acc, 0.0f);
        if (a.out_f32) reinterpret_cast<float*>(a.out)[v] = acc;
        else reinterpret_cast<u16*>(a.out)[v] = f2bf(acc);
    }
}

// ---------------------------------------------------------------- elementwise
// Pack FP32 master weights [Cout][K] into the BF16 forward layout
// [NT*16][Kp] and the input-gradient layout [Cin_pad][Kp'] (flipped taps,
// in/out channels swapped), zero padded.
__global__ void k_pack(const float* __restrict__ w, int cout, int cin, int taps, u16* __restrict__ wf,
                       int rows_f, int kp_f, u16* __restrict__ wb, int rows_b, int kp_b)
{
    const int K = taps * cin;
    const size_t nf = (size_t)rows_f * kp_f, nb = wb ? (size_t)rows_b * kp_b : 0;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nf + nb;
         i += (size_t)gridDim.x * blockDim.x) {
        if (i < nf) {
            const int row = (int)(i / kp_f), k = (int)(i % kp_f);
            wf[i] = (row < cout && k < K) ? f2bf(w[(size_t)row * K + k]) : (u16)0;
        } else {
            const size_t j = i - nf;
            const int c = (int)(j / kp_b), kb = (int)(j % kp_b);   // c: input channel
            u16 v = 0;
            if (c < cin && kb < taps * cout) {
                const int tb = kb / cout, o = kb - tb * cout;
                const int t = taps - 1 - tb;                        // flipped tap
                v = f2bf(w[(size_t)o * K + t * cin + c]);
            }
            wb[j] = v;
        }
    }
}

// y = 2x2x2 max of x (BF16, channels-last), arg = winning child 0..7.
__global__ void k_maxpool(const u16* __restrict__ x, u16* __restrict__ y, unsigned char* __restrict__ arg,
                          int D, int H, int W, int C)
{
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    const size_t n = (size_t)Do * Ho * Wo * C;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t v = i / C;
        const int xo = (int)(v % Wo), yo = (int)((v / Wo) % Ho), zo = (int)(v / ((size_t)Wo * Ho));
        float best = -INFINITY;
        int bi = 0;
        for (int q = 0; q < 8; ++q) {
            const int z = 2 * zo + (q >> 2), yy = 2 * yo + ((q >> 1) & 1), xx = 2 * xo + (q & 1);
            const float val = bf2f(x[(((size_t)z * H + yy) * W + xx) * C + c]);
            if (val > best) {
                best = val;
                bi = q;
            }
        }
        y[i] = f2bf(best);
        arg[i] = (unsigned char)bi;
    }
}

// dx[child] += dy at the winning child (FP32 accumulate into dx).
__global__ void k_maxpool_bwd(const float* __restrict__ dy, const unsigned char* __restrict__ arg,
                              float* __restrict__ dx, int D, int H, int W, int C)
{
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    const size_t n = (size_t)Do * Ho * Wo * C;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t v = i / C;
        const int xo = (int)(v % Wo), yo = (int)((v / Wo) % Ho), zo = (int)(v / ((size_t)Wo * Ho));
        const int q = arg[i];
        const int z = 2 * zo + (q >> 2), yy = 2 * yo + ((q >> 1) & 1), xx = 2 * xo + (q & 1);
        dx[(((size_t)z * H + yy) * W + xx) * C + c] += dy[i];
    }
}

// dlow = sum of the 8 children of dhigh (backward of nearest 2x upsampling).
__global__ void k_sumpool(const float* __restrict__ dh, float* __restrict__ dl, int D, int H, int W, int C,
                          int accumulate)
{
    const int Do = D / 2, Ho = H / 2, Wo = W / 2;
    const size_t n = (size_t)Do * Ho * Wo * C;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t v = i / C;
        const int xo = (int)(v % Wo), yo = (int)((v / Wo) % Ho), zo = (int)(v / ((size_t)Wo * Ho));
        float s = 0.0f;
        for (int q = 0; q < 8; ++q) {
            const int z = 2 * zo + (q >> 2), yy = 2 * yo + ((q >> 1) & 1), xx = 2 * xo + (q & 1);
            s += dh[(((size_t)z * H + yy) * W + xx) * C + c];
        }
        dl[i] = accumulate ? dl[i] + s : s;
    }
}

// g = dOut * (out > 0) as BF16 (the MFMA operand) and its per-channel sum.
// When C divides the grid stride (C a power of two up to 256) every thread
// keeps one channel: its sum stays in a register, lanes of one channel are
// combined with wave shuffles and each wave adds C values into LDS.
__global__ void k_relu_mask_pc(const float* __restrict__ dout, const u16* __restrict__ out, int relu,
                               u16* __restrict__ g, float* __restrict__ dbias, size_t n, int C)
{
    extern __shared__ float sb[];
    for (int c = threadIdx.x; c < C; c += blockDim.x) sb[c] = 0.0f;
    __syncthreads();
    float part = 0.0f;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        float v = dout[i];
        if (relu && !(bf2f(out[i]) > 0.0f)) v = 0.0f;
        const u16 b = f2bf(v);
        g[i] = b;
        part += bf2f(b);
    }
    // lanes l and l + C (C < 64) hold the same channel
    for (int o = 32; o >= C && o > 0; o >>= 1) part += __shfl_xor(part, o);
    const int lane = threadIdx.x & 63;
    if (lane < C && part != 0.0f) atomicAdd(&sb[threadIdx.x % C], part);
    __syncthreads();
    if (dbias)
        for (int c = threadIdx.x; c < C; c += blockDim.x)
            if (sb[c] != 0.0f) unsafeAtomicAdd(&dbias[c], sb[c]);
}

// k_relu_mask_pc over 8 consecutive elements per thread and step (16-byte
// loads and stores).  C divides 2048, so a thread's 8 elements keep their
// channels (8 t + j) mod C through the grid-stride loop: the 8 sums stay in
// registers, lanes holding the same channels are combined with wave
// shuffles, and the rest reach LDS once per wave.
__global__ __launch_bounds__(kSumBlock) void k_relu_mask_v8(const float* __restrict__ dout, const u16* __restrict__ out,
                                                      int relu, u16* __restrict__ g, float* __restrict__ dbias,
                                                      size_t n8, int C)
{
    extern __shared__ float sb[];
    for (int c = threadIdx.x; c < C; c += blockDim.x) sb[c] = 0.0f;
    __syncthreads();
    float part[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = t0; i < n8; i += (size_t)gridDim.x * blockDim.x) {
        const float4 d0 = reinterpret_cast<const float4*>(dout)[2 * i];
        const float4 d1 = reinterpret_cast<const float4*>(dout)[2 * i + 1];
        float v[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
        if (relu) {
            Frag o;
            o.q = reinterpret_cast<const uint4*>(out)[i];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (!(bf2f(o.h[j]) > 0.0f)) v[j] = 0.0f;
        }
        Frag b;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            b.h[j] = f2bf(v[j]);
            part[j] += bf2f(b.h[j]);
        }
        reinterpret_cast<uint4*>(g)[i] = b.q;
    }
    // C < 8: element j of a thread has channel j mod C
    if (C <= 4)
#pragma unroll
        for (int j = 0; j < 4; ++j) part[j] += part[j + 4];
    if (C <= 2)
#pragma unroll
        for (int j = 0; j < 2; ++j) part[j] += part[j + 2];
    if (C == 1) part[0] += part[1];
    // lanes l and l ^ o hold the same channels when C divides 8 o
    for (int o = 32; o >= 1 && 8 * o >= C; o >>= 1)
#pragma unroll
        for (int j = 0; j < 8; ++j) part[j] += __shfl_xor(part[j], o);
    const int lane = threadIdx.x & 63;
    if (lane < (C >= 8 ? C / 8 : 1))
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < C && part[j] != 0.0f) atomicAdd(&sb[(int)((8 * t0 + j) % (size_t)C)], part[j]);
    __syncthreads();
    if (dbias)
        for (int c = threadIdx.x; c < C; c += blockDim.x)
            if (sb[c] != 0.0f) unsafeAtomicAdd(&dbias[c], sb[c]);
}

__global__ void k_relu_mask(const float* __restrict__ dout, const u16* __restrict__ out, int relu,
                            u16* __restrict__ g, float* __restrict__ dbias, size_t n, int C)
{
    extern __shared__ float sb[];
    for (int c = threadIdx.x; c < C; c += blockDim.x) sb[c] = 0.0f;
    __syncthreads();
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        float v = dout[i];
        if (relu && !(bf2f(out[i]) > 0.0f)) v = 0.0f;
        const u16 b = f2bf(v);
        g[i] = b;
        if (v != 0.0f) atomicAdd(&sb[i % C], bf2f(b));
    }
    __syncthreads();
    if (dbias)
        for (int c = threadIdx.x; c < C; c += blockDim.x)
            if (sb[c] != 0.0f) unsafeAtomicAdd(&dbias[c], sb[c]);
}

// Loss 1/V sum (x - t)^2 of the network output (FP32) against the target,
// and its gradient through the final ReLU.
__global__ __launch_bounds__(kSumBlock) void k_mse(const float* __restrict__ x, const float* __restrict__ t, float* __restrict__ g,
                      double* __restrict__ loss, size_t n)
{
    __shared__ double red[kSumBlock / 64];
    double s = 0.0;
    const float inv = 1.0f / (float)n;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const double dd = (double)x[i] - (double)t[i];   // exact for FP32 inputs
        s += dd * dd;
        const float d = x[i] - t[i];
        g[i] = 2.0f * d * inv;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s = 0.0;
        for (unsigned w = 0; w < blockDim.x / 64; ++w) s += red[w];
        unsafeAtomicAdd(loss, s / (double)n);
    }
}

// Adam on FP32 master weights (bias-corrected), gradients cleared after use.
__global__ void k_adam(float* __restrict__ w, float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, size_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        g[i] = 0.0f;
    }
}

// Network input: A^T y scaled by 1 / max (max over the volume), as BF16.
__global__ __launch_bounds__(kSumBlock) void k_absmax(const float* __restrict__ x, size_t n,
                                                      unsigned int* __restrict__ out)
{
    __shared__ float red[kSumBlock / 64];
    float mval = 0.0f;
#pragma unroll 4
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        mval = fmaxf(mval, fabsf(x[i]));
    for (int o = 32; o > 0; o >>= 1) mval = fmaxf(mval, __shfl_xor(mval, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mval;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned w = 1; w < blockDim.x / 64; ++w) mval = fmaxf(mval, red[w]);
        atomicMax(out, __float_as_uint(mval));
    }
}

__global__ void k_scale_to_bf16(const float* __restrict__ x, const unsigned int* __restrict__ mx,
                                u16* __restrict__ y, size_t n)
{
    const float m = __uint_as_float(*mx);
    const float s = m > 0.0f ? 1.0f / m : 0.0f;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i] * s);
}

__global__ void k_add(float* __restrict__ a, const float* __restrict__ b, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        a[i] += b[i];
}

__global__ void k_fill_u32(unsigned int* p, size_t n, unsigned int v)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

unsigned nblocks(size_t n)
{
    size_t b = (n + 255) / 256;
    return (unsigned)(b > 16384 ? 16384 : (b ? b : 1));
}

template <int KS, bool CIN1, int NT, int MT>
hipError_t conv_launch(const ConvFwd& a, int groups, hipStream_t s)
{
    const int V = a.D * a.H * a.W;
    const int per_block = 4 * 16 * MT;
    hipLaunchKernelGGL((k_conv_fwd<KS, CIN1, NT, MT>), dim3((V + per_block - 1) / per_block, groups), dim3(256),
                       0, s, a);
    return hipGetLastError();
}

template <int KS, bool CIN1, int NT>
hipError_t conv_mt(const ConvFwd& a, hipStream_t s)
{
    constexpr int MT = NT >= 8 ? 1 : (NT >= 4 ? 2 : 4);
    const int V = a.D * a.H * a.W;
    // small grids (16^3, 32^3): one 16-channel tile and 16 voxels per wave, the
    // channel tiles spread over blockIdx.y, so enough waves run to hide latency
    if (NT > 1 && (long long)(V + 4 * 16 * MT - 1) / (4 * 16 * MT) < 256)
        return conv_launch<KS, CIN1, 1, 1>(a, NT, s);
    return conv_launch<KS, CIN1, NT, MT>(a, 1, s);
}

template <int KS, bool CIN1>
hipError_t conv_nt(const ConvFwd& a, int nt, hipStream_t s)
{
    switch (nt) {
        case 1: return conv_mt<KS, CIN1, 1>(a, s);
        case 2: return conv_mt<KS, CIN1, 2>(a, s);
        case 4: return conv_mt<KS, CIN1, 4>(a, s);
        case 8: return conv_mt<KS, CIN1, 8>(a, s);
        default: return hipErrorInvalidValue;
    }
}

template <int CIN>
hipError_t conv_planes(const ConvFwd& a, int nt, int ncb, dim3 g, hipStream_t s)
{
    switch (nt) {
    case 1: hipLaunchKernelGGL((k_conv_fwd_planes<1, 1, CIN>), g, dim3(256), 0, s, a, ncb); break;
    case 2: hipLaunchKernelGGL((k_conv_fwd_planes<2, 2, CIN>), g, dim3(256), 0, s, a, ncb); break;
    default: hipLaunchKernelGGL((k_conv_fwd_planes<4, 4, CIN>), g, dim3(256), 0, s, a, ncb); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t nn_conv_fwd(const ConvFwd& a, int ks, hipStream_t s)
{
    const int nt = (a.cout + 15) / 16;
    const int ntp = nt <= 1 ? 1 : (nt <= 2 ? 2 : (nt <= 4 ? 4 : 8));
    const int cin = a.c0 + a.c1;
    const bool cin1 = cin == 1;
    if (ks == 3 && cin % 32 == 0 && cin <= 128 && a.D < 65536) {
        const int tz = cin <= 32 ? 4 : 2;
        const size_t plane = (size_t)((a.W + kTX - 1) / kTX) * ((a.H + kTY - 1) / kTY);
        // fewer than two whole-halo workgroups per compute unit (with eight channel
        // tiles, fewer than one: 64 -> 128 channels at 32^3 are 35 us by planes, 33
        // with whole halos)
        const size_t blocks = plane * ((a.D + tz - 1) / tz);
        if (cin > 64 || blocks < 256 || (blocks < 512 && ntp <= 4)) {
            // channel tiles per workgroup: as many as leave two workgroups per
            // compute unit
            int nt = std::min(ntp, 4);
            while (nt > 1 && plane * a.D * (ntp / nt) < 512) nt /= 2;
            const dim3 g((a.W + kTX - 1) / kTX * (ntp / nt), (a.H + kTY - 1) / kTY, a.D);
            return cin == 32   ? conv_planes<32>(a, nt, ntp / nt, g, s)
                   : cin == 64 ? conv_planes<64>(a, nt, ntp / nt, g, s)
                   : cin == 96 ? conv_planes<96>(a, nt, ntp / nt, g, s)
                               : conv_planes<128>(a, nt, ntp / nt, g, s);
        }
    }
    if (ks == 3 && cin >= 8 && cin <= 64 && cin % 8 == 0) {
        // 8 output planes per workgroup up to 16 channels (35 KiB halo), 4 up to 32
        // (41 KiB), 2 up to 64 (55 KiB)
        const int tz = (cin <= 16 && ntp <= 4) ? 8 : (cin <= 32 ? 4 : 2);
        const dim3 g((a.W + kTX - 1) / kTX, (a.H + kTY - 1) / kTY, (a.D + tz - 1) / tz);
        const size_t halo = (size_t)kHX * kHY * (tz + 2) * cin * sizeof(unsigned short);
#define LTM_TILE(CIN, NT, TZ, WN) \
    hipLaunchKernelGGL((k_conv_fwd_tile<CIN, NT, TZ, WN>), g, dim3(256), halo, s, a); break
        switch (cin * 16 + ntp) {
        case 16 * 16 + 1: LTM_TILE(16, 1, 8, 1);
        case 16 * 16 + 2: LTM_TILE(16, 2, 8, 1);
        case 16 * 16 + 4: LTM_TILE(16, 4, 8, 1);
        case 16 * 16 + 8: LTM_TILE(16, 8, 4, 4);
        case 32 * 16 + 1: LTM_TILE(32, 1, 4, 1);
        case 32 * 16 + 2: LTM_TILE(32, 2, 4, 2);
        case 32 * 16 + 4: LTM_TILE(32, 4, 4, 4);
        case 32 * 16 + 8: LTM_TILE(32, 8, 4, 4);
        case 64 * 16 + 1: LTM_TILE(64, 1, 2, 1);
        case 64 * 16 + 2: LTM_TILE(64, 2, 2, 2);
        case 64 * 16 + 4: LTM_TILE(64, 4, 2, 2);
        case 64 * 16 + 8: LTM_TILE(64, 8, 2, 4);
        default: {
            // the halo, then the per-step offset table (nsteps x 4 ints)
            const size_t lds = halo + (size_t)(a.Kp / 32) * 4 * sizeof(int);
#define LTM_CONV(NT, TZ) hipLaunchKernelGGL((k_conv_fwd_lds<NT, TZ>), g, dim3(256), lds, s, a); break
            switch (tz * 16 + ntp) {
            case 8 * 16 + 1: LTM_CONV(1, 8);
            case 8 * 16 + 2: LTM_CONV(2, 8);
            case 8 * 16 + 4: LTM_CONV(4, 8);
            case 4 * 16 + 1: LTM_CONV(1, 4);
            case 4 * 16 + 2: LTM_CONV(2, 4);
            case 4 * 16 + 4: LTM_CONV(4, 4);
            case 4 * 16 + 8: LTM_CONV(8, 4);
            case 2 * 16 + 1: LTM_CONV(1, 2);
            case 2 * 16 + 2: LTM_CONV(2, 2);
            case 2 * 16 + 4: LTM_CONV(4, 2);
            default: LTM_CONV(8, 2);
            }
        }
        }
#undef LTM_TILE
#undef LTM_CONV
        return hipGetLastError();
    }
    if (ks == 1 && a.cout == 1 && a.c1 == 0 && !a.up && (cin == 8 || cin == 16 || cin == 32)) {
        const size_t nvox = (size_t)a.D * a.H * a.W;
        const dim3 g(std::min(nblocks(nvox), 4096u));
        if (cin == 8) hipLaunchKernelGGL((k_conv1x1_out1<8>), g, dim3(256), 0, s, a, nvox);
        else if (cin == 16) hipLaunchKernelGGL((k_conv1x1_out1<16>), g, dim3(256), 0, s, a, nvox);
        else hipLaunchKernelGGL((k_conv1x1_out1<32>), g, dim3(256), 0, s, a, nvox);
        return hipGetLastError();
    }
    if (ks == 3 && cin1 && a.c1 == 0 && a.cout <= 16) {
        // four voxels per thread while that leaves two workgroups per compute unit
        const dim3 g((a.W + 15) / 16, (a.H + 3) / 4, (a.D + 15) / 16);
        if ((size_t)g.x * g.y * g.z >= 512)
            hipLaunchKernelGGL(k_conv_fwd_c1<4>, g, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL(k_conv_fwd_c1<1>, dim3(g.x, g.y, (a.D + 3) / 4), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    if (ks == 3) return cin1 ? conv_nt<3, true>(a, ntp, s) : conv_nt<3, false>(a, ntp, s);
    return cin1 ? conv_nt<1, true>(a, ntp, s) : conv_nt<1, false>(a, ntp, s);
}

hipError_t nn_conv_wgrad(const ConvWgrad& a, int ks, hipStream_t s)
{
    const int cin = a.c0 + a.c1;
    auto lg2 = [](int n) { int l = 0; while ((1 << l) < n) ++l; return (1 << l) == n ? l : -1; };
    const int lw = lg2(a.W), lh = lg2(a.H);
    const bool pow2 = lw >= 3 && lh >= 0 && (a.W * a.H) % 32 == 0;
    // the chunk that pads the rows least, the longest of those.  Padding pays: 64 ->
    // 64 channels at 48 x 48 x 40 gathered voxel by voxel take 823 us, padded 92; only rows of 8 (a
    // quarter of a chunk) stay with the shift-indexed kernel (rows of 16: 52 us there,
    // 44 padded, 128 -> 128 channels at 16^3)
    int xc = 32;
    for (int c : {64, 128})
        if ((a.W + c - 1) / c * c <= (a.W + xc - 1) / xc * xc) xc = c;
    // (rows of no whole chunk may come from buffers that the gathering kernels accept,
    // aligned to an element only)
    const bool whole = a.W % 32 == 0;
    const bool aligned = ((reinterpret_cast<uintptr_t>(a.in0) | reinterpret_cast<uintptr_t>(a.in1) |
                           reinterpret_cast<uintptr_t>(a.dy)) & 15) == 0;
    if (ks == 3 && (whole || ((a.W >= 16 || !pow2) && aligned)) && cin % 16 == 0 && a.c0 % 8 == 0 && a.cout % 16 == 0 && a.K == 27 * cin &&
        (!a.up || (a.W % 2 == 0 && a.H % 2 == 0 && a.D % 2 == 0))) {
        if (xc == 128) return wgrad_rows<128>(a, s);
        if (xc == 64) return wgrad_rows<64>(a, s);
        return wgrad_rows<32>(a, s);
    }
    if (ks == 3 && cin == 1 && a.c1 == 0 && !a.up && (whole || aligned) && a.cout % 16 == 0 && a.K == 27) {
        if (xc == 128) return wgrad_c1<128>(a, s);
        if (xc == 64) return wgrad_c1<64>(a, s);
        return wgrad_c1<32>(a, s);
    }
    if (ks == 1 && a.cout == 1 && a.c1 == 0 && !a.up && a.K == cin && (cin == 8 || cin == 16 || cin == 32)) {
        const size_t nvox = (size_t)a.D * a.H * a.W;
        const dim3 g(sum_blocks(nvox));
        if (cin == 8) hipLaunchKernelGGL((k_wgrad_1x1_out1<8>), g, dim3(kSumBlock), 0, s, a, nvox);
        else if (cin == 16) hipLaunchKernelGGL((k_wgrad_1x1_out1<16>), g, dim3(kSumBlock), 0, s, a, nvox);
        else hipLaunchKernelGGL((k_wgrad_1x1_out1<32>), g, dim3(kSumBlock), 0, s, a, nvox);
        return hipGetLastError();
    }
    if (ks == 3 && pow2 && a.cout % 16 == 0 &&
        (!a.up || (a.W % 2 == 0 && a.H % 2 == 0))) {
        constexpr int NK = 2;
        const int tiles = (a.cout / 16) * (((a.K + 15) / 16 + NK - 1) / NK);
        // split each slice's voxel groups over workgroups until ~8192 waves
        // run (one per tile, slice and share); each share adds its own
        // partial sums into dw
        const int blocks = (tiles + 3) / 4 * a.D;
        const int groups = a.W * a.H / 32;
        const int shares = std::max(1, std::min(groups, 2048 / std::max(1, blocks)));
        hipLaunchKernelGGL((k_conv_wgrad_pow2<3, NK>), dim3((tiles + 3) / 4, a.D, shares), dim3(256), 0, s, a,
                           lw, lh);
        return hipGetLastError();
    }
    const int tiles = ((a.cout + 15) / 16) * ((a.K + 15) / 16);
    const int blocks = (tiles + 3) / 4 * a.D;
    const int shares = std::max(1, std::min((a.W * a.H + 31) / 32, 2048 / std::max(1, blocks)));
    dim3 grid((tiles + 3) / 4, a.D, shares);
    if (ks == 3)
        hipLaunchKernelGGL(k_conv_wgrad<3>, grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(k_conv_wgrad<1>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t nn_pack(const float* w, int cout, int cin, int taps, unsigned short* wf, int rows_f, int kp_f,
                   unsigned short* wb, int rows_b, int kp_b, hipStream_t s)
{
    const size_t n = (size_t)rows_f * kp_f + (wb ? (size_t)rows_b * kp_b : 0);
    hipLaunchKernelGGL(k_pack, dim3(nblocks(n)), dim3(256), 0, s, w, cout, cin, taps, wf, rows_f, kp_f, wb,
                       rows_b, kp_b);
    return hipGetLastError();
}

hipError_t nn_maxpool(const unsigned short* x, unsigned short* y, unsigned char* arg, int D, int H, int W, int C,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_maxpool, dim3(nblocks((size_t)D * H * W * C / 8)), dim3(256), 0, s, x, y, arg, D, H, W, C);
    return hipGetLastError();
}

hipError_t nn_maxpool_bwd(const float* dy, const unsigned char* arg, float* dx, int D, int H, int W, int C,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_maxpool_bwd, dim3(nblocks((size_t)D * H * W * C / 8)), dim3(256), 0, s, dy, arg, dx, D,
                       H, W, C);
    return hipGetLastError();
}

hipError_t nn_sumpool(const float* dh, float* dl, int D, int H, int W, int C, int accumulate, hipStream_t s)
{
    hipLaunchKernelGGL(k_sumpool, dim3(nblocks((size_t)D * H * W * C / 8)), dim3(256), 0, s, dh, dl, D, H, W, C,
                       accumulate);
    return hipGetLastError();
}

hipError_t nn_relu_mask(const float* dout, const unsigned short* out, int relu, unsigned short* g,
                        float* dbias, size_t n, int C, hipStream_t s)
{
    // at most one workgroup per compute unit: each adds C partial sums into dbias
    // with global atomics, which contend on the C addresses
    const bool pow2 = C >= 1 && (C & (C - 1)) == 0;
    const bool aligned = ((reinterpret_cast<uintptr_t>(dout) | reinterpret_cast<uintptr_t>(out) |
                           reinterpret_cast<uintptr_t>(g)) & 15) == 0;
    if (pow2 && C <= 2048 && n % 8 == 0 && aligned) {   // C divides the grid stride in elements (2048 k)
        hipLaunchKernelGGL(k_relu_mask_v8, dim3(sum_blocks(n / 8)), dim3(kSumBlock), C * sizeof(float), s,
                           dout, out, relu, g, dbias, n / 8, C);
        return hipGetLastError();
    }
    const dim3 grid(std::min(nblocks(n), 1024u));
    if (pow2 && C <= 256)   // C divides the grid stride (a multiple of 256)
        hipLaunchKernelGGL(k_relu_mask_pc, grid, dim3(256), C * sizeof(float), s, dout, out, relu, g, dbias, n, C);
    else
        hipLaunchKernelGGL(k_relu_mask, grid, dim3(256), C * sizeof(float), s, dout, out, relu, g, dbias, n, C);
    return hipGetLastError();
}

hipError_t nn_mse(const float* x, const float* t, float* g, double* loss, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_mse, dim3(sum_blocks(n)), dim3(kSumBlock), 0, s, x, t, g, loss, n);
    return hipGetLastError();
}

hipError_t nn_adam(float* w, float* g, float* m, float* v, size_t n, float lr, float b1, float b2, float eps,
                   int step, hipStream_t s)
{
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(nblocks(n)), dim3(256), 0, s, w, g, m, v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t nn_prep_input(const float* x, unsigned short* y, unsigned int* scratch, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, scratch, (size_t)1, 0u);
    hipLaunchKernelGGL(k_absmax, dim3(sum_blocks(n)), dim3(kSumBlock), 0, s, x, n, scratch);
    hipLaunchKernelGGL(k_scale_to_bf16, dim3(nblocks(n)), dim3(256), 0, s, x, scratch, y, n);
    return hipGetLastError();
}

hipError_t nn_add(float* a, const float* b, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_add, dim3(nblocks(n)), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

}  // namespace ltm
