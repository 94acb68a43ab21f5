// k_fused_tile.hip -- several fused blocks per sweep on the matrix cores.
//
// A workgroup holds a tile of 2^13 amplitudes (qubits 0..3, whole lines of 128
// bytes, and nine more) in LDS and applies, one after the other, every block of
// its list: blocks of at most five qubits, all of them the tile's. A block is
// the product of k_fused.hip, Y = M X with X[r][j] of 32 rows (the block's
// qubits); the tile has 256 columns, 8 parts of 32 for 4 waves. A wave reads a
// part's right operands from LDS, and writes its products back in their place: nothing
// but the barrier after each block ties the waves together. The left operand is
// read per block from memory (16 KB, cache resident) into registers.
//
// LDS: amplitude i sits at i ^ S(i), S linear over the bits above the fifth, so
// that 5 of a block's 8 column bits can be chosen which spread 32 lanes over
// all 64 banks for 97 % of the target sets.
//
// Bound: FP32 by the matrix cores (64 clocks per product: 8192 of a CU per block
// and tile, 224 us per block at 27 qubits, where a sweep of its own takes 370 to
// 400, bound by memory), which two workgroups per CU keep 66 % busy at 2.2 GHz
// (median of the sweeps); BF16x3 by memory. The planned 20-layer brickwork: FP32 at
// 27 qubits 45 blocks in 19 sweeps, 18.0 -> 15.1 ms; BF16x3 at 26 qubits 45 blocks in
// 26 sweeps (18 of two or three blocks at 0.23 ms, 8 of one at 0.19), 8.5 -> 5.5 ms.
// What the pause between the products is was not found: both parts' operands read
// at once, priorities or a delay that let one workgroup run ahead, tiles of 2^12
// with three workgroups per CU (335 us a block as now), and a persistent grid with
// the next tile's loads in flight (869 us a sweep instead of 820) gained nothing.
#include "sv_device.h"
#include "sv_internal.h"
#include "tile_device.h"

namespace sv {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int T = kFusedTileBits;
constexpr int kThreads = 256;
constexpr int kIter = (1 << T) / (2 * kThreads);      // float4 per thread

__device__ __forceinline__ bf16x8 to_bf16(const float (&x)[8])
{
    bf16x8 r;
#pragma unroll
    for (int q = 0; q < 8; ++q) r[q] = (__bf16)x[q];
    return r;
}

// the left operand of a block: fragments as k_fused.hip lays them out
template <int MODE>
struct Left;
template <>
struct Left<0> {
    float a[2][32];
    __device__ __forceinline__ void load(const float* m, int lane)
    {
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float4 t = reinterpret_cast<const float4*>(m)[(b * 8 + q) * 64 + lane];
                a[b][4 * q] = t.x;
                a[b][4 * q + 1] = t.y;
                a[b][4 * q + 2] = t.z;
                a[b][4 * q + 3] = t.w;
            }
    }
    __device__ __forceinline__ void mul(const float2 (&x)[16], f32x16& c0, f32x16& c1) const
    {
#pragma unroll
        for (int s = 0; s < 32; ++s) {
            const float v = s < 16 ? x[s].x : x[s - 16].y;
            c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][s], v, c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1][s], v, c1, 0, 0, 0);
        }
    }
};
template <>
struct Left<1> {
    bf16x8 hi[2][4], lo[2][4];
    __device__ __forceinline__ void load(const float* m, int lane)
    {
        const u32x4* f = reinterpret_cast<const u32x4*>(m);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                hi[b][s] = __builtin_bit_cast(bf16x8, f[((b * 4 + s) * 2 + 0) * 64 + lane]);
                lo[b][s] = __builtin_bit_cast(bf16x8, f[((b * 4 + s) * 2 + 1) * 64 + lane]);
            }
    }
    __device__ __forceinline__ void mul(const float2 (&x)[16], f32x16& c0, f32x16& c1) const
    {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            float xh[8], xl[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float2 v = (s & 1) ? x[8 + q] : x[q];
                xh[q] = s < 2 ? v.x : v.y;
            }
            const bf16x8 bh = to_bf16(xh);
#pragma unroll
            for (int q = 0; q < 8; ++q) xl[q] = xh[q] - (float)bh[q];
            const bf16x8 bl = to_bf16(xl);
            c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo[0][s], bh, c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo[1][s], bh, c1, 0, 0, 0);
            c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[0][s], bl, c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[1][s], bl, c1, 0, 0, 0);
            c0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[0][s], bh, c0, 0, 0, 0);
            c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[1][s], bh, c1, 0, 0, 0);
        }
    }
};

template <int MODE>
__global__ __launch_bounds__(kThreads, 2) void k_fused_tile(FusedTileArgs a)
{
    __shared__ float2 lds[1 << T];
    char* const mem = reinterpret_cast<char*>(lds);
    cword* W = (cword*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                        offsetof(FusedTileArgs, blocks));
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63, wave = (int)(tid >> 6), h = lane >> 5, c32 = lane & 31;
    float2* psi = a.psi + (uint64_t)blockIdx.y * a.N;
    uint64_t base = xcd_block(blockIdx.x, gridDim.x);
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int p = a.pos[i];
        base = ((base >> p) << (p + 1)) | (base & ((1ull << p) - 1ull));
    }
    // amplitudes 2 (tid + 256 i), + 1
    uint64_t off = base;
    uint32_t at = 0;                                  // byte address in LDS
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        off |= (uint64_t)((tid >> b) & 1u) << a.pos[b + 1];
        at ^= (0u - ((tid >> b) & 1u)) & (8u * fused_tile_place(2u << b));
    }
    float4 v[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        uint64_t o = off;
#pragma unroll
        for (int b = 0; b < T - 9; ++b)
            if ((i >> b) & 1) o |= 1ull << a.pos[9 + b];
        v[i] = ld4(psi + o);
    }
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const uint32_t p = at ^ (8u * fused_tile_place((uint32_t)i << 9));
        *reinterpret_cast<float2*>(mem + p) = make_float2(v[i].x, v[i].y);
        *reinterpret_cast<float2*>(mem + (p ^ 8u)) = make_float2(v[i].z, v[i].w);
    }
    for (int n = 0; n < a.nblocks; ++n, W += kFusedTileWords) {
        Left<MODE> left;
        left.load(a.amat + (size_t)blockIdx.y * a.amat_stride + 4 * (size_t)W[7], lane);
        // byte addresses of the row, column and part bits
        const uint32_t w0 = W[0], w1 = W[1], w2 = W[2], w3 = W[3], w4 = W[4], w5 = W[5], w6 = W[6];
        const uint32_t row[5] = {w0 & 0xffffu, w0 >> 16, w1 & 0xffffu, w1 >> 16, w2 & 0xffffu};
        const uint32_t col[5] = {w2 >> 16, w3 & 0xffffu, w3 >> 16, w4 & 0xffffu, w4 >> 16};
        const uint32_t part[3] = {w5 & 0xffffu, w5 >> 16, w6 & 0xffffu};
        uint32_t lo = ((wave & 1) ? part[1] : 0u) ^ ((wave & 2) ? part[2] : 0u);
#pragma unroll
        for (int k = 0; k < 5; ++k) lo ^= (0u - (uint32_t)((c32 >> k) & 1)) & col[k];
        // row r of the operand: 2 s + h (FP32), 8 h + s % 8 + 16 (s / 8) (BF16x3); of
        // the result 8 (q / 4) + 4 h + q % 4. Row bit j is row[4 - j].
        const uint32_t in = lo ^ ((0u - (uint32_t)h) & (MODE == 0 ? row[4] : row[1]));
        const uint32_t out = lo ^ ((0u - (uint32_t)h) & row[2]);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float2 x[16];
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const int r = MODE == 0 ? 2 * s : (s & 7) + 16 * (s >> 3);
                uint32_t o = u ? part[0] : 0u;
#pragma unroll
                for (int j = 0; j < 5; ++j)
                    if ((r >> j) & 1) o ^= row[4 - j];
                x[s] = *reinterpret_cast<const float2*>(mem + (in ^ o));
            }
            f32x16 c0 = {0}, c1 = {0};
            left.mul(x, c0, c1);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int r = 8 * (q >> 2) + (q & 3);
                uint32_t o = u ? part[0] : 0u;
#pragma unroll
                for (int j = 0; j < 5; ++j)
                    if ((r >> j) & 1) o ^= row[4 - j];
                *reinterpret_cast<float2*>(mem + (out ^ o)) = make_float2(c0[q], c1[q]);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const uint32_t p = at ^ (8u * fused_tile_place((uint32_t)i << 9));
        const float2 x = *reinterpret_cast<const float2*>(mem + p), y = *reinterpret_cast<const float2*>(mem + (p ^ 8u));
        uint64_t o = off;
#pragma unroll
        for (int b = 0; b < T - 9; ++b)
            if ((i >> b) & 1) o |= 1ull << a.pos[9 + b];
        st4(psi + o, make_float4(x.x, x.y, y.x, y.y));
    }
}

}  // namespace

void launch_fused_tile(const FusedTileArgs& a, int nrows, int mode, hipStream_t st)
{
    const dim3 grid((unsigned)(a.N >> T), (unsigned)nrows);
    if (mode == SV_FUSED_FP32_MFMA)
        hipLaunchKernelGGL(k_fused_tile<0>, grid, dim3(kThreads), 0, st, a);
    else
        hipLaunchKernelGGL(k_fused_tile<1>, grid, dim3(kThreads), 0, st, a);
    SV_HIP(hipGetLastError());
}

}  // namespace sv
