// k_pauli.hip -- many Pauli strings per sweep of the state.
//
// <P> = sum_b conj(psi[b ^ x]) i^{|x & z|} (-1)^{|b & z|} psi[b]. A workgroup
// holds a tile (2^T amplitudes that differ in T chosen qubits) in LDS; a
// string whose x bits are among them finds both amplitudes there, whatever
// its z bits. b and b ^ x give the same term, so the pairs are taken once, split
// by x's top bit: per distinct x and part (real, imaginary) a thread forms the
// products conj(psi[b ^ x]) psi[b] of its 8 pairs (x = 0: 16 amplitudes) in FP64
// once, per string it sums them with the signs of z, and the waves' sums go
// through a fixed tree into one LDS slot per string and wave.
//
// Bound: vector instructions (0.052 of the 0.082 ms of a sweep at 24 qubits with
// 24 strings; its read takes 0.021): a string costs a thread 8 sign products and
// the 30 instructions of the wave's sum, an x 85. The 69 strings X X, Y Y, Z Z
// of a 24-qubit chain are 3 sweeps instead of 26: 0.83 -> 0.27 ms. With the 16
// products of both halves of each pair a sweep took 0.120.
#include <type_traits>

#include "tile_device.h"

namespace sv {

namespace {

constexpr int kOwn = 16;                              // amplitudes per thread

// c summed with the signs of one string into the wave's slot.
template <int K>
__device__ __forceinline__ void add_string(const double (&c)[K], uint32_t h, uint32_t zouter, uint32_t tid,
                                           uint32_t tile, bool act, double* slot)
{
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int j = 0; j < K; j += 2) {
        s0 = fma(c[j], (h >> j) & 1u ? -1.0 : 1.0, s0);
        s1 = fma(c[j + 1], (h >> (j + 1)) & 1u ? -1.0 : 1.0, s1);
    }
    double s = s0 + s1;
    if (K < kOwn) s += s;                             // the pair's other half
    const uint32_t minus = (uint32_t)__popc(tid & ((h >> 16) & 255u)) + (uint32_t)__popc(tile & zouter) + ((h >> 29) & 1u);
    s = wave_sum(act ? minus & 1u ? -s : s : 0.0);
    if ((tid & 63) == 63) *slot += s;
}

__global__ __launch_bounds__(256) void k_pauli_tile(PauliTileArgs a)
{
    __shared__ float2 lds[1 << kTileMaxBits];
    __shared__ double acc[kPauliTerms * 4];           // [term][wave]
    cword* W = (cword*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                        offsetof(PauliTileArgs, words));
    const uint32_t tid = threadIdx.x;
    const int T = a.T, waves = (int)blockDim.x >> 6, wave = (int)(tid >> 6);
    const uint32_t threads = 1u << (T - 4);           // that own amplitudes
    const bool act = tid < threads;
    const uint32_t me = act ? tid : 0u;               // the others' sums are left out
    const int row = (int)blockIdx.y;
    const float2* psi = row < a.nrow0 ? a.p0 + (uint64_t)row * a.N : a.p1 + (uint64_t)(row - a.nrow0) * a.N;
    for (int i = (int)tid; i < a.nterms * waves; i += (int)blockDim.x) acc[i] = 0.0;
    uint64_t off = 0;
    each<0, kTileMaxBits - 4>([&](auto B) SV_INLINE { off |= (uint64_t)((tid >> B) & 1u) << a.pos[B]; });
    uint64_t step[4];                                 // of a thread's amplitudes
#pragma unroll
    for (int k = 0; k < 4; ++k) step[k] = 1ull << (int)__builtin_amdgcn_readfirstlane(a.pos[T - 4 + k]);
    const uint32_t ntiles = (uint32_t)(a.N >> T);
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        uint64_t base = tile;
        each<0, kTileMaxBits>([&](auto B) SV_INLINE {
            const int p = a.pos[B];
            if (B < T) base = ((base >> p) << (p + 1)) | (base & ((1ull << p) - 1ull));
        });
        __syncthreads();                              // the tile before has been read
        if (act) {
            float2 v[kOwn];
#pragma unroll
            for (int j = 0; j < kOwn; ++j) {
                uint64_t o = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if ((j >> k) & 1) o |= step[k];
                v[j] = psi[base + off + o];
            }
#pragma unroll
            for (int j = 0; j < kOwn; ++j) lds[j * threads + tid] = v[j];
        }
        __syncthreads();
        cword* pc = W;
        int term = 0;
        for (int g = 0; g < a.ngroups; ++g) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readfirstlane((int)(pc[0] & 0xfffu));
            const bool imag = (pc[0] >> 12) & 1u;
            const int nt = (int)(pc[0] >> 16);
            pc += 1;
            if (x == 0) {
                double c[kOwn];
#pragma unroll
                for (int j = 0; j < kOwn; ++j) {
                    const float2 w = lds[j * threads + me];
                    c[j] = fma((double)w.x, (double)w.x, (double)w.y * w.y);
                }
                for (int t = 0; t < nt; ++t, ++term, pc += 2)
                    add_string<kOwn>(c, pc[0], pc[1], tid, tile, act, acc + term * waves + wave);
                continue;
            }
            const uint32_t p = 31u - (uint32_t)__builtin_clz(x), low = (uint32_t)T - 4u;
            const uint32_t in = p < low, up = in ? 0u : p - low, lmask = (1u << (in ? p : low)) - 1u, umask = (1u << up) - 1u;
            const uint32_t i0 = (me & lmask) | (me & ~lmask) << in, i1 = i0 ^ (x & ((1u << (low + in)) - 1u));
            const uint32_t xh = x >> (low + in) << (low + in);
            double c[kOwn / 2];
            auto pairs = [&](auto Imag) SV_INLINE {
#pragma unroll
                for (uint32_t k = 0; k < kOwn / 2; ++k) {
                    const uint32_t hi = ((k & ~umask) << (1u - in) | (k & umask)) << (low + in);
                    const float2 v = lds[i0 + hi], w = lds[i1 + (hi ^ xh)];
                    c[k] = Imag ? fma((double)w.x, (double)v.y, (double)-w.y * (double)v.x)
                                : fma((double)w.x, (double)v.x, (double)w.y * (double)v.y);
                }
            };
            if (imag)
                pairs(std::integral_constant<bool, true>());
            else
                pairs(std::integral_constant<bool, false>());
            for (int t = 0; t < nt; ++t, ++term, pc += 2)
                add_string<kOwn / 2>(c, pc[0], pc[1], tid, tile, act, acc + term * waves + wave);
        }
    }
    __syncthreads();
    for (int t = (int)tid; t < a.nterms; t += (int)blockDim.x) {
        double s = acc[t * waves];
        for (int w = 1; w < waves; ++w) s += acc[t * waves + w];
        a.part[((uint64_t)row * a.nterms + t) * gridDim.x + blockIdx.x] = s;
    }
}

}  // namespace

// Workgroups per row: four per compute unit over all rows.
int pauli_tile_grid(int n, int T, int rows)
{
    const uint64_t most = std::max<uint64_t>(1, (uint64_t)device_info().cu_count * 4 / rows);
    return (int)std::min<uint64_t>(1ull << (n - T), most);
}

void launch_pauli_tile(const PauliTileArgs& a, int rows, double* out, hipStream_t st)
{
    const int n = __builtin_ctzll(a.N), grid = pauli_tile_grid(n, a.T, rows);
    hipLaunchKernelGGL(k_pauli_tile, dim3((unsigned)grid, (unsigned)rows), dim3((unsigned)std::max(64, 1 << (a.T - 4))), 0,
                       st, a);
    SV_HIP(hipGetLastError());
    launch_sum_slots(a.part, grid, rows * a.nterms, out, st);
}

}  // namespace sv
