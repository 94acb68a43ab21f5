// k_tile_adj.hip -- the per-gate adjoint backward in tiles of state and
// co-state: of a state that fits one workgroup's LDS twice (4..12 qubits) the
// whole gate list in one launch, of a larger one a list of gates per sweep.
//
// The program (tile.h) holds the circuit's gates from last to first, as their
// U^*. Every step un-applies its gates from psi and from lambda; before that,
// a gate with a derivative adds its inner products over the threads' register
// amplitudes in FP64 (products of two FP32 values are exact there):
//   rotation exp(-i theta P / 2): Im <lambda|P|psi>, which is the derivative;
//   any other one-target gate: the correlation S_ij = sum conj(lambda_i) psi_j
//   over the pairs it acts on, from which the host forms 2 Re sum G_ij S_ij.
// Wave sums go through a fixed tree of lane moves into one LDS slot per value
// and wave (the rotations of a step share one tree), a workgroup's slots sum
// over its tiles, and a second kernel sums the workgroups' values, so results
// are bitwise reproducible.
//
// Bound, one tile per row: the latency of a step (branches, the sums' lane
// moves). Eight rows of 10 qubits, 70 gates: one launch where one launch per
// gate made 180 of 2-3.5 us each. Larger states: the vector unit; a rotation
// costs 64 instructions for both vectors, 48 for its products and 20 for its
// share of the sum per 512 amplitudes. 25-qubit ring of 10 RX, RY and CNOT
// layers: 29 sweeps at 0.46 ms, 13.2 ms in all (84 matrix-core blocks: 18.4; with
// a tree per value and all four products of a pair 17); 16 rows of 18 qubits,
// 3 ladder blocks: 6 sweeps, 0.34 ms (18 matrix-core blocks: 0.63 and 1 ms of
// host work on their matrices).
#include <cstddef>

#include "tile_device.h"

namespace sv {

namespace {

constexpr int kR = kTileRegBits - 1;                  // 8 amplitudes of each vector per thread
constexpr int kM = 1 << kR;
constexpr int kTBits = kTileMaxBits - kR;

// Re and Im of conj(l) x added to (re, im)
__device__ __forceinline__ void corr(float lr, float li, float xr, float xi, double& re, double& im)
{
    re = fma((double)lr, (double)xr, fma((double)li, (double)xi, re));
    im = fma((double)lr, (double)xi, fma(-(double)li, (double)xr, im));
}

// Derivative values of a gate on register bit TB: `kind` as TileDeriv.
// Written by lane 63 to slot[0..] (stride `waves`; TILES: added to it).
template <bool TILES, int TB>
__device__ __forceinline__ void derivative(const Amps<kM>& x, const Amps<kM>& l, uint32_t kind, const Where& at,
                                           double* slot, int waves)
{
    double r00 = 0, i00 = 0, r01 = 0, i01 = 0, r10 = 0, i10 = 0, r11 = 0, i11 = 0;
    const bool off = kind & (TD_X | TD_Y | TD_GENERAL), diag = kind & (TD_Z | TD_GENERAL);
    each<0, kM>([&](auto J) SV_INLINE {
        constexpr int j = J, o = j | (1 << TB);
        if constexpr (!((j >> TB) & 1)) {
            const bool on = at(j);
            const float l0r = on ? l.re[j] : 0.f, l0i = on ? l.im[j] : 0.f;
            const float l1r = on ? l.re[o] : 0.f, l1i = on ? l.im[o] : 0.f;
            if (off) {
                corr(l0r, l0i, x.re[o], x.im[o], r01, i01);
                corr(l1r, l1i, x.re[j], x.im[j], r10, i10);
            }
            if (diag) {
                corr(l0r, l0i, x.re[j], x.im[j], r00, i00);
                corr(l1r, l1i, x.re[o], x.im[o], r11, i11);
            }
        }
    });
    const bool writer = (threadIdx.x & 63) == 63;
    double v = i00 - i11;                             // Im <l|Z|x>
    if (kind & TD_X) v = i01 + i10;
    if (kind & TD_Y) v = r10 - r01;
    auto put = [&](int i, double w) SV_INLINE {
        w = wave_sum(w);
        if (writer) slot[i * waves] = TILES ? slot[i * waves] + w : w;
    };
    if (!(kind & TD_GENERAL)) {
        put(0, v);
    } else {
        const double all[8] = {r00, i00, r01, i01, r10, i10, r11, i11};
#pragma unroll
        for (int i = 0; i < 8; ++i) put(i, all[i]);
    }
}

// This thread's part of a rotation's derivative: Im <l|P|x> on register bit TB.
template <int TB>
__device__ __forceinline__ double rotation(const Amps<kM>& x, const Amps<kM>& l, uint32_t kind)
{
    double s = 0.0;
    auto add = [&](float a, float b) SV_INLINE { s = fma((double)a, (double)b, s); };
    auto pair = [&](auto F) SV_INLINE {
        each<0, kM>([&](auto J) SV_INLINE {
            constexpr int j = J, o = j | (1 << TB);
            if constexpr (!((j >> TB) & 1)) F(l.re[j], l.im[j], l.re[o], l.im[o], x.re[j], x.im[j], x.re[o], x.im[o]);
        });
    };
    if (kind & TD_X)
        pair([&](float l0r, float l0i, float l1r, float l1i, float x0r, float x0i, float x1r, float x1i) SV_INLINE {
            add(l0r, x1i), add(-l0i, x1r), add(l1r, x0i), add(-l1i, x0r);
        });
    if (kind & TD_Y)
        pair([&](float l0r, float l0i, float l1r, float l1i, float x0r, float x0i, float x1r, float x1i) SV_INLINE {
            add(l1r, x0r), add(l1i, x0i), add(-l0r, x1r), add(-l0i, x1i);
        });
    if (kind & TD_Z)
        pair([&](float l0r, float l0i, float l1r, float l1i, float x0r, float x0i, float x1r, float x1i) SV_INLINE {
            add(l0r, x0i), add(-l0i, x0r), add(-l1r, x1i), add(l1i, x1r);
        });
    return s;
}

// The wave's sums of three values, in lanes 0, 1 and 2 (mod 4): the first two
// exchanges halve the values a lane carries.
__device__ __forceinline__ double wave_sum3(double a, double b, double c)
{
    const bool odd = threadIdx.x & 1u, high = threadIdx.x & 2u;
    const double ab = (odd ? b : a) + lane_move<0xb1>(odd ? a : b);       // lane ^ 1
    const double cc = c + lane_move<0xb1>(c);
    double v = (high ? cc : ab) + lane_move<0x4e>(high ? ab : cc);        // lane ^ 2
    v += lane_move<0x124>(v);                                             // by 4 and 8 within sixteen
    v += lane_move<0x128>(v);
    v = add_swapped<16>(v);
    return add_swapped<32>(v);
}

template <bool TILES>
__global__ __launch_bounds__(1 << kTBits, TILES ? 4 : 2) void k_tile_adj(TileAdjArgs a)
{
    extern __shared__ float2 dyn[];
    cword* W = (cword*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                        offsetof(TileAdjArgs, words));
    const uint32_t tid = threadIdx.x;
    const int T = a.T, waves = (int)blockDim.x >> 6;
    float2* lx = dyn;
    float2* ll = dyn + (1 << T);
    double* part = reinterpret_cast<double*>(dyn + (2 << T));     // [values][waves], then loss, drift
    touch_program(W, a.nwords);
    const bool act = tid < (1u << (T - kR));
    const int rel_row = (int)blockIdx.y, row = a.row0 + rel_row;
    float2* psi = a.psi + (uint64_t)row * a.N;
    float2* lam = a.lam + (uint64_t)row * a.N;
    const int wave = (int)(tid >> 6);

    // float4 e = 2 (tid + 2^(T-3) i): tile bits are the qubits themselves
    auto element = [&](uint32_t e) SV_INLINE {
        uint32_t v = e & 15u;
        each<4, kTileMaxBits>([&](auto B) SV_INLINE { v ^= (0u - ((e >> B) & 1u)) & swz_col(B); });
        return v;
    };
    double loss = 0.0, drift = 0.0;
    if constexpr (TILES)
        for (int i = (int)tid; i < a.nvalues * waves; i += (int)blockDim.x) part[i] = 0.0;
    uint32_t tile = TILES ? blockIdx.x : 0u;
    do {
        // TILES: place in memory of the thread's float4 i, relative to the row
        uint64_t base = 0;
        auto memory = [&](int i) SV_INLINE {
            uint64_t o = base;
            each<0, kR - 1>([&](auto K) SV_INLINE {
                if ((i >> K) & 1) o |= 1ull << a.pos[kTileMaxBits - kR + 1 + K];
            });
            return o;
        };
        if constexpr (TILES) {
            base = tile;
            each<0, kTileMaxBits>([&](auto B) SV_INLINE {
                const int p = a.pos[B];
                base = ((base >> p) << (p + 1)) | (base & ((1ull << p) - 1ull));
            });
            each<1, kTBits + 1>([&](auto B) SV_INLINE { base |= (uint64_t)((tid >> (B - 1)) & 1u) << a.pos[B]; });
            __syncthreads();                              // the tile before has been read
            float4 v[kM / 2], g[kM / 2];
            each<0, kM / 2>([&](auto I) SV_INLINE {
                v[I] = ld4(psi + memory(I));
                g[I] = ld4(lam + memory(I));
            });
            each<0, kM / 2>([&](auto I) SV_INLINE {
                const uint32_t at = element(2 * tid + ((uint32_t)I << (kTBits + 1)));
                lx[at] = lo2(v[I]);
                lx[at ^ 1] = hi2(v[I]);
                ll[at] = lo2(g[I]);
                ll[at ^ 1] = hi2(g[I]);
            });
        } else if (act) {
            for (int i = 0; i < kM / 2; ++i) {
                const uint32_t e = 2 * tid + ((uint32_t)i << (T - kR + 1)), at = element(e);
                const float4 v = ld4<false>(psi + e);
                float4 g;
                if (a.coeff) {
                    // lambda = sum_q c_q Z_q psi
                    const double* c = a.coeff + (uint64_t)row * a.coeff_stride;
                    double f0 = 0.0, f1 = 0.0;
                    for (int q = 0; q < T; ++q) {
                        const double cq = c[q];
                        f0 += (e >> q) & 1u ? -cq : cq;
                        f1 += ((e | 1u) >> q) & 1u ? -cq : cq;
                    }
                    g = make_float4((float)(f0 * v.x), (float)(f0 * v.y), (float)(f1 * v.z), (float)(f1 * v.w));
                } else {
                    g = ld4<false>(lam + e);
                }
                loss += (double)v.x * g.x + (double)v.y * g.y + (double)v.z * g.z + (double)v.w * g.w;
                lx[at] = lo2(v);
                lx[at ^ 1] = hi2(v);
                ll[at] = lo2(g);
                ll[at ^ 1] = hi2(g);
            }
        }

        cword* pc = W;
        int value = 0;
        for (int r = 0; r < a.nrounds; ++r) {
            const uint32_t r0 = pc[0];
            const int nsteps = (int)(r0 & 255u), nouter = (int)((r0 >> 8) & 255u);
            uint32_t at = thread_columns<kTBits>(pc, tid, 1, 8);
            const uint32_t tix = thread_index<kTBits>(pc, tid);
            uint32_t sign = 0;
            Cx phase{1.f, 0.f};
            cword* ps = pc + kTileRoundWords;
            const bool mapped = (r0 >> 18) & 1u;
            if (mapped) ps += kTileMapWords + ((nouter + 3) & ~3);
            u32x4 next = ld_head(ps);
            thread_steps(W, ps, next, (int)(r0 >> 24), tix, tile, rel_row, sign, phase);
            uint32_t rel[kM];
            reg_columns<kR>(pc, 5, rel);
            __syncthreads();
            Amps<kM> x, l;
            each<0, kM>([&](auto J) SV_INLINE {
                const float2 v = act ? lx[at ^ rel[J]] : make_float2(0.f, 0.f);
                const float2 g = act ? ll[at ^ rel[J]] : make_float2(0.f, 0.f);
                x.re[J] = v.x;
                x.im[J] = v.y;
                l.re[J] = g.x;
                l.im[J] = g.y;
            });
            uint32_t flips = 0;
            for (int g = 0; g < nsteps; ++g) {
                const u32x4 h = next;
                ps += kTileHeadWords;
                next = ld_head(ps);
                // derivatives of the step's gates: they act on different register bits
                const uint32_t tctl = h.x & TF_OTHER ? (h.x >> 16) & 0xfffu : 0u;
                const bool outer = !TILES || !(h.x & TF_OTHER) || (tile & h.y) == h.y;
                const Where where{outer && (tix & tctl) == tctl, h.x & TF_OTHER ? (int)((h.x >> 8) & 15) : 0};
                if ((h.x & (TF_DERIV | TF_LAYER)) == (TF_DERIV | TF_LAYER) && !(h.w & 0x88800u)) {
                    const uint32_t k0 = (h.w >> 8) & 15u, k1 = (h.w >> 12) & 15u, k2 = (h.w >> 16) & 15u;
                    double v0 = 0.0, v1 = 0.0, v2 = 0.0;
                    if (k0) v0 = rotation<0>(x, l, k0);
                    if (k1) v1 = rotation<1>(x, l, k1);
                    if (k2) v2 = rotation<2>(x, l, k2);
                    const double v = wave_sum3(v0, v1, v2);
                    const int n0 = k0 ? 1 : 0, n1 = n0 + (k1 ? 1 : 0), n2 = n1 + (k2 ? 1 : 0);
                    const uint32_t lane = tid & 63u;
                    const bool mine = lane == 0 ? k0 != 0 : lane == 1 ? k1 != 0 : lane == 2 && k2 != 0;
                    double* slot = part + (value + (lane == 0 ? 0 : lane == 1 ? n0 : n1)) * waves + wave;
                    if (mine) *slot = TILES ? *slot + v : v;
                    value += n2;
                } else if (h.x & TF_DERIV) {
#define SV_DERIVATIVE(TB)                                                                        \
        {                                                                                        \
            const uint32_t kind = (h.w >> (8 + 4 * (TB))) & 15u;                                 \
            if (kind) {                                                                          \
                derivative<TILES, TB>(x, l, kind, where, part + value * waves + wave, waves);    \
                value += kind & TD_GENERAL ? 8 : 1;                                              \
            }                                                                                    \
        }
                    SV_DERIVATIVE(0)
                    SV_DERIVATIVE(1)
                    SV_DERIVATIVE(2)
#undef SV_DERIVATIVE
                }
                if (h.x & TF_LAYER) {
                    cword* w = W + h.z * rel_row;
                    f32x8 m[kR];
                    each<0, kR>([&](auto B) SV_INLINE { m[B] = ld_mat(w + 4 * ((h.y >> (8 * B)) & 255u)); });
                    const uint32_t on_bits = h.x >> 8;
                    constexpr int R = kR;
                    constexpr int M = kM;
                    if (h.x & TF_DENSE) SV_BITS(on_bits, pairs<M, TB>(x, Dense{m[TB]}); pairs<M, TB>(l, Dense{m[TB]});)
                    if (h.x & TF_REAL) SV_BITS(on_bits, pairs<M, TB>(x, Real{m[TB]}); pairs<M, TB>(l, Real{m[TB]});)
                    if (h.x & TF_IMOFF) SV_BITS(on_bits, pairs<M, TB>(x, ImOff{m[TB]}); pairs<M, TB>(l, ImOff{m[TB]});)
                    if (h.x & TF_DIAG) SV_BITS(on_bits, pairs<M, TB>(x, Diag{m[TB]}); pairs<M, TB>(l, Diag{m[TB]});)
                }
                if (h.x & TF_OTHER) {
                    cword* w = W + (h.z & 0xffffu) + (h.z >> 16) * rel_row;
                    constexpr int R = kR;
                    constexpr int M = kM;
                    if (h.x & TF_SIGN) flips ^= outer ? h.w : 0u;
                    if (h.x & TF_APPLY) {
                        each<0, M>([&](auto J) SV_INLINE {
                            const uint32_t f = (flips << (31 - J)) & 0x80000000u;
                            flip(x.re[J], x.im[J], f);
                            flip(l.re[J], l.im[J], f);
                        });
                        flips = 0;
                    }
                    if (h.x & TF_LANE_SIGN) {
                        const uint32_t mine = where.on ? h.w : 0u;
                        each<0, M>([&](auto J) SV_INLINE {
                            const uint32_t f = (mine << (31 - J)) & 0x80000000u;
                            flip_v(x.re[J], x.im[J], f);
                            flip_v(l.re[J], l.im[J], f);
                        });
                    }
                    if (h.x & TF_PHASE) {
                        const RegPhase p = reg_phase(h, w, tix, tile);
                        phases<M>(x, where, p);
                        phases<M>(l, where, p);
                    }
                    if (h.x & TF_CTRL)
                        SV_BITS(h.w, pairs_where<M, TB>(x, where, ld_mat(w)); pairs_where<M, TB>(l, where, ld_mat(w));)
                    if (h.x & TF_DENSE2) SV_PAIRS(h.w, dense2<M, A, B>(x, where, w); dense2<M, A, B>(l, where, w);)
                }
            }
            if ((r0 >> 16) & 1u)
                each<0, kM>([&](auto J) SV_INLINE {
                    flip_v(x.re[J], x.im[J], sign);
                    flip_v(l.re[J], l.im[J], sign);
                });
            if ((r0 >> 17) & 1u)
                each<0, kM>([&](auto J) SV_INLINE {
                    times(x.re[J], x.im[J], phase);
                    times(l.re[J], l.im[J], phase);
                });
            if (mapped) {
                at = thread_columns<kTBits>(pc, tid, 12, 16) ^ pc[19];
                reg_columns<kR>(pc, 17, rel);
                for (int i = 0; i < nouter; ++i) {
                    const uint32_t o = pc[20 + i];
                    if ((tile >> (o & 31u)) & 1u) at ^= o >> 16;
                }
                __syncthreads();
            }
            if (act)
                each<0, kM>([&](auto J) SV_INLINE {
                    lx[at ^ rel[J]] = make_float2(x.re[J], x.im[J]);
                    ll[at ^ rel[J]] = make_float2(l.re[J], l.im[J]);
                });
            pc = ps;
        }
        __syncthreads();
        if constexpr (TILES) {
            each<0, kM / 2>([&](auto I) SV_INLINE {
                const uint32_t at = element(2 * tid + ((uint32_t)I << (kTBits + 1)));
                st4(psi + memory(I), pack4(lx[at], lx[at ^ 1]));
                st4(lam + memory(I), pack4(ll[at], ll[at ^ 1]));
            });
        } else if (act) {
            for (int i = 0; i < kM / 2; ++i) {
                const uint32_t e = 2 * tid + ((uint32_t)i << (T - kR + 1)), at = element(e);
                const float4 v = pack4(lx[at], lx[at ^ 1]);
                st4<false>(psi + e, v);
                st4<false>(lam + e, pack4(ll[at], ll[at ^ 1]));
                const double re = e == 0 ? (double)v.x - 1.0 : (double)v.x;
                drift += re * re + (double)v.y * v.y + (double)v.z * v.z + (double)v.w * v.w;   // || psi - e_0 ||^2
            }
        }
        tile += gridDim.x;
    } while (TILES && tile < (uint32_t)(a.N >> T));
    if constexpr (TILES) {
        __syncthreads();
        for (int v = (int)tid; v < a.nvalues; v += (int)blockDim.x) {
            double s = part[v * waves];
            for (int w = 1; w < waves; ++w) s += part[v * waves + w];
            a.out[((uint64_t)rel_row * a.nvalues + v) * gridDim.x + blockIdx.x] = s;
        }
        return;
    }
    loss = wave_sum(loss);
    drift = wave_sum(drift);
    if ((tid & 63) == 63) {
        part[a.nvalues * waves + wave] = loss;
        part[(a.nvalues + 1) * waves + wave] = drift;
    }
    __syncthreads();
    // a segment's values, then the loss (first segment) and the drift (last)
    double* out = a.out + (uint64_t)row * a.out_stride;
    for (int v = (int)tid; v < a.nvalues + 2; v += (int)blockDim.x) {
        double s = part[v * waves];
        for (int w = 1; w < waves; ++w) s += part[v * waves + w];
        if (v < a.nvalues) out[a.value0 + v] = s;
        else if (v == a.nvalues) {
            if (a.first) out[a.out_stride - 2] = s;
        } else if (a.last) {
            out[a.out_stride - 1] = s;
        }
    }
}

}  // namespace

void launch_tile_adj(const TileAdjArgs& a, int grid, int rows, hipStream_t st)
{
    const int threads = std::max(64, 1 << (a.T - kR));
    auto lds_bytes = [](int T, int values, int waves) {
        return ((size_t)2 << T) * sizeof(float2) + (size_t)(values + 2) * waves * sizeof(double);
    };
    const size_t lds = lds_bytes(a.T, a.nvalues, threads / 64);
    const bool tiles = (a.N >> a.T) > 1;
    const void* f = tiles ? reinterpret_cast<const void*>(&k_tile_adj<true>) : reinterpret_cast<const void*>(&k_tile_adj<false>);
    // Two tiles of 2^12 and the values are more than the 64 KiB a launch has by
    // default. The limit is the function's, not the launch's: always the largest
    // launch's, so that no thread lowers it between another's call and launch.
    if (lds > 65536)
        SV_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds_bytes(kTileMaxBits, tiles ? kAdjTileValues : kAdjValues, 1 << (kTBits - 6))));
    if (tiles)
        hipLaunchKernelGGL(k_tile_adj<true>, dim3((unsigned)grid, (unsigned)rows), dim3((unsigned)threads), lds, st, a);
    else
        hipLaunchKernelGGL(k_tile_adj<false>, dim3(1, (unsigned)rows), dim3((unsigned)threads), lds, st, a);
    SV_HIP(hipGetLastError());
}

}  // namespace sv
