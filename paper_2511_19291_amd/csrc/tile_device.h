// tile_device.h -- device pieces shared by the kernels that run tile programs
// (k_tile.hip, k_tile_adj.hip): reading the program, and the gates on a
// thread's register amplitudes.
#pragma once

#include <type_traits>

#include "sv_device.h"
#include "tile.h"

namespace sv {

typedef const __attribute__((address_space(4))) uint32_t cword;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ u32x4 ld_head(cword* p)
{
    return *(const __attribute__((address_space(4))) u32x4*)p;
}

// (16-byte aligned; the words of the smaller kinds lie in the first four)
__device__ __forceinline__ f32x8 ld_mat(cword* p)
{
    typedef f32x8 __attribute__((aligned(16))) f32x8_16;
    return *(const __attribute__((address_space(4))) f32x8_16*)p;
}

// (a lambda not inlined before the first scalar replacement keeps the
// amplitudes it captures in scratch memory)
#define SV_INLINE __attribute__((always_inline))

// f(0), ..., f(N - 1) with the index a constant: the thread's amplitudes are
// only ever named by constants, so they stay in registers
template <int I, int N, class F>
__device__ __forceinline__ void each(const F& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each<I + 1, N>(f);
    }
}

__host__ __device__ constexpr uint32_t swz_col(int b)
{
    return (1u << b) ^ (b >= 4 ? kTileSwz[b - 4] : 0u);
}

// The thread's amplitudes, real and imaginary parts apart (plain floats named
// by constants only).
template <int M>
struct Amps {
    float re[M], im[M];
};

struct Cx {
    float re, im;
};

__device__ __forceinline__ float sel(bool c, float a, float b) { return c ? a : b; }
__device__ __forceinline__ Cx sel(bool c, Cx a, Cx b) { return Cx{c ? a.re : b.re, c ? a.im : b.im}; }
// a b, and c + a b, in the order of cmul and cfma
__device__ __forceinline__ Cx mul(Cx a, Cx b) { return Cx{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ Cx mad(Cx a, Cx b, Cx c)
{
    return Cx{fmaf(a.re, b.re, fmaf(-a.im, b.im, c.re)), fmaf(a.re, b.im, fmaf(a.im, b.re, c.im))};
}

// One-target matrices on a pair, in place: y0 = m00 x0 + m01 x1,
// y1 = m10 x0 + m11 x1, sums in that order. Written as instructions because
// each result has to land in its own amplitude's register: from plain
// arithmetic the compiler leaves the results elsewhere and moves every
// amplitude at every join of the kernel's branches (2.2 vector instructions
// for every one of arithmetic). The products of x0 come first, and an
// instruction needs no result of the one or two before it.
struct Dense {
    f32x8 m;
    __device__ __forceinline__ void operator()(float& r0, float& i0, float& r1, float& i1) const
    {
        float t, u, a, b;
        asm("v_mul_f32 %4, %13, %1\n\t"
            "v_mul_f32 %5, %13, %0\n\t"
            "v_mul_f32 %6, %9, %1\n\t"
            "v_mul_f32 %7, %9, %0\n\t"
            "v_fma_f32 %4, %12, %0, -%4\n\t"
            "v_fma_f32 %5, %12, %1, %5\n\t"
            "v_fma_f32 %0, %8, %0, -%6\n\t"
            "v_fma_f32 %1, %8, %1, %7\n\t"
            "v_fma_f32 %4, -%15, %3, %4\n\t"
            "v_fma_f32 %5, %15, %2, %5\n\t"
            "v_fma_f32 %0, -%11, %3, %0\n\t"
            "v_fma_f32 %1, %11, %2, %1\n\t"
            "v_fma_f32 %0, %10, %2, %0\n\t"
            "v_fma_f32 %1, %10, %3, %1\n\t"
            "v_fma_f32 %2, %14, %2, %4\n\t"
            "v_fma_f32 %3, %14, %3, %5"
            : "+v"(r0), "+v"(i0), "+v"(r1), "+v"(i1), "=&v"(t), "=&v"(u), "=&v"(a), "=&v"(b)
            : "s"(m[0]), "s"(m[1]), "s"(m[2]), "s"(m[3]), "s"(m[4]), "s"(m[5]), "s"(m[6]), "s"(m[7]));
    }
};

// A real matrix, and one with a real diagonal and imaginary off-diagonal
// entries: the general product without the terms that are products with an
// exact zero (equal for finite amplitudes), half the operations.
struct Real {
    f32x8 m;
    __device__ __forceinline__ void operator()(float& r0, float& i0, float& r1, float& i1) const
    {
        float t, u;
        asm("v_mul_f32 %4, %8, %0\n\t"
            "v_mul_f32 %5, %8, %1\n\t"
            "v_mul_f32 %0, %6, %0\n\t"
            "v_mul_f32 %1, %6, %1\n\t"
            "v_fma_f32 %0, %7, %2, %0\n\t"
            "v_fma_f32 %1, %7, %3, %1\n\t"
            "v_fma_f32 %2, %9, %2, %4\n\t"
            "v_fma_f32 %3, %9, %3, %5"
            : "+v"(r0), "+v"(i0), "+v"(r1), "+v"(i1), "=&v"(t), "=&v"(u)
            : "s"(m[0]), "s"(m[1]), "s"(m[2]), "s"(m[3]));
    }
};

struct ImOff {
    f32x8 m;
    __device__ __forceinline__ void operator()(float& r0, float& i0, float& r1, float& i1) const
    {
        float t, u;
        asm("v_mul_f32 %4, -%8, %1\n\t"
            "v_mul_f32 %5, %8, %0\n\t"
            "v_mul_f32 %0, %6, %0\n\t"
            "v_mul_f32 %1, %6, %1\n\t"
            "v_fma_f32 %0, -%7, %3, %0\n\t"
            "v_fma_f32 %1, %7, %2, %1\n\t"
            "v_fma_f32 %2, %9, %2, %4\n\t"
            "v_fma_f32 %3, %9, %3, %5"
            : "+v"(r0), "+v"(i0), "+v"(r1), "+v"(i1), "=&v"(t), "=&v"(u)
            : "s"(m[0]), "s"(m[1]), "s"(m[2]), "s"(m[3]));
    }
};

struct Diag {
    f32x8 m;
    __device__ __forceinline__ void operator()(float& r0, float& i0, float& r1, float& i1) const
    {
        float t, u, a, b;
        asm("v_mul_f32 %4, %9, %1\n\t"
            "v_mul_f32 %5, %9, %0\n\t"
            "v_mul_f32 %6, %11, %3\n\t"
            "v_mul_f32 %7, %11, %2\n\t"
            "v_fma_f32 %0, %8, %0, -%4\n\t"
            "v_fma_f32 %1, %8, %1, %5\n\t"
            "v_fma_f32 %2, %10, %2, -%6\n\t"
            "v_fma_f32 %3, %10, %3, %7"
            : "+v"(r0), "+v"(i0), "+v"(r1), "+v"(i1), "=&v"(t), "=&v"(u), "=&v"(a), "=&v"(b)
            : "s"(m[0]), "s"(m[1]), "s"(m[2]), "s"(m[3]));
    }
};

// f on every pair (j, j | 1 << TB)
template <int M, int TB, class F>
__device__ __forceinline__ void pairs(Amps<M>& x, const F& f)
{
    each<0, M>([&](auto J) SV_INLINE {
        constexpr int j = J, o = j | (1 << TB);
        if constexpr (!((j >> TB) & 1)) f(x.re[j], x.im[j], x.re[o], x.im[o]);
    });
}

// Where a controlled gate acts: lanes whose thread controls hold, register
// amplitudes whose control bits are all set. Kept by selects, not branches.
struct Where {
    bool on;
    int rcm;
    __device__ __forceinline__ bool operator()(int j) const { return on & ((j & rcm) == rcm); }
};

template <int M, int TB>
__device__ __forceinline__ void pairs_where(Amps<M>& x, const Where& at, const f32x8& m)
{
    each<0, M>([&](auto J) SV_INLINE {
        constexpr int j = J, o = j | (1 << TB);
        if constexpr (!((j >> TB) & 1)) {
            float r0 = x.re[j], i0 = x.im[j], r1 = x.re[o], i1 = x.im[o];
            Dense{m}(r0, i0, r1, i1);
            const bool on = at(j);
            x.re[j] = sel(on, r0, x.re[j]);
            x.im[j] = sel(on, i0, x.im[j]);
            x.re[o] = sel(on, r1, x.re[o]);
            x.im[o] = sel(on, i1, x.im[o]);
        }
    });
}

// 4 x 4 on bits A > B, A the most significant bit of the matrix index
template <int M, int A, int B>
__device__ __forceinline__ void dense2(Amps<M>& x, const Where& at, cword* w)
{
    each<0, M>([&](auto J) SV_INLINE {
        constexpr int j = J;
        if constexpr (!((j >> A) & 1) && !((j >> B) & 1)) {
            constexpr int j1 = j | (1 << B), j2 = j | (1 << A), j3 = j1 | j2;
            const bool on = at(j);
            const Cx v0{x.re[j], x.im[j]}, v1{x.re[j1], x.im[j1]}, v2{x.re[j2], x.im[j2]}, v3{x.re[j3], x.im[j3]};
            auto row = [&](int i, Cx old) SV_INLINE {
                const f32x8 m = ld_mat(w + 8 * i);
                const Cx y = mad(Cx{m[6], m[7]}, v3, mad(Cx{m[4], m[5]}, v2, mad(Cx{m[2], m[3]}, v1, mul(Cx{m[0], m[1]}, v0))));
                return sel(on, y, old);
            };
            const Cx y0 = row(0, v0), y1 = row(1, v1), y2 = row(2, v2), y3 = row(3, v3);
            x.re[j] = y0.re;
            x.im[j] = y0.im;
            x.re[j1] = y1.re;
            x.im[j1] = y1.im;
            x.re[j2] = y2.re;
            x.im[j2] = y2.im;
            x.re[j3] = y3.re;
            x.im[j3] = y3.im;
        }
    });
}

// (r, i) times p, in place
__device__ __forceinline__ void times(float& r, float& i, Cx p)
{
    float t, u;
    asm("v_mul_f32 %2, %5, %1\n\t"
        "v_mul_f32 %3, %5, %0\n\t"
        "v_fma_f32 %0, %4, %0, -%2\n\t"
        "v_fma_f32 %1, %4, %1, %3"
        : "+v"(r), "+v"(i), "=&v"(t), "=&v"(u)
        : "v"(p.re), "v"(p.im));
}

// the sign bits of (r, i) flipped where f has its own set, in place: f the
// same for all lanes, and each lane's own
__device__ __forceinline__ void flip(float& r, float& i, uint32_t f)
{
    asm("v_xor_b32 %0, %2, %0\n\t"
        "v_xor_b32 %1, %2, %1"
        : "+v"(r), "+v"(i)
        : "s"(f));
}
__device__ __forceinline__ void flip_v(float& r, float& i, uint32_t f)
{
    asm("v_xor_b32 %0, %2, %0\n\t"
        "v_xor_b32 %1, %2, %1"
        : "+v"(r), "+v"(i)
        : "v"(f));
}

// every amplitude j times phase(j) where `at` says
template <int M, class F>
__device__ __forceinline__ void phases(Amps<M>& x, const Where& at, const F& phase)
{
    each<0, M>([&](auto J) SV_INLINE {
        const Cx p = phase((int)J);
        float r = x.re[J], i = x.im[J];
        times(r, i, p);
        const bool on = at(J);
        x.re[J] = sel(on, r, x.re[J]);
        x.im[J] = sel(on, i, x.im[J]);
    });
}

// The branches on a step's kind and target bits stand in the kernel itself, not
// in a function that takes the amplitudes by reference: the compiler would
// merge such a function's branches while the amplitudes are still memory to
// it, and then cannot bring them into registers. A step's kinds and bits are
// flags, each tested by an `if` of its own with nothing in an `else`: the
// branches are made one sequence anyway, and wherever the compiler knows two
// of them to exclude each other it keeps a second copy of the amplitudes for
// the later one (up to a hundred moves a step).
#define SV_BITS(flags, ...)                                                                  \
    {                                                                                        \
        if ((flags) & 1u) { constexpr int TB = 0; __VA_ARGS__ }                              \
        if constexpr (R > 1) if ((flags) & 2u) { constexpr int TB = R > 1 ? 1 : 0; __VA_ARGS__ } \
        if constexpr (R > 2) if ((flags) & 4u) { constexpr int TB = R > 2 ? 2 : 0; __VA_ARGS__ } \
        if constexpr (R > 3) if ((flags) & 8u) { constexpr int TB = R > 3 ? 3 : 0; __VA_ARGS__ } \
    }
#define SV_PAIR(flags, idx, HI, LO, ...)                                                     \
    if constexpr (R > (HI))                                                                  \
        if ((flags) & (1u << (idx))) { constexpr int A = R > (HI) ? (HI) : 1, B = R > (HI) ? (LO) : 0; __VA_ARGS__ }
#define SV_PAIRS(flags, ...)                                                                 \
    {                                                                                        \
        SV_PAIR(flags, 0, 1, 0, __VA_ARGS__) SV_PAIR(flags, 1, 2, 0, __VA_ARGS__)            \
        SV_PAIR(flags, 2, 2, 1, __VA_ARGS__) SV_PAIR(flags, 3, 3, 0, __VA_ARGS__)            \
        SV_PAIR(flags, 4, 3, 1, __VA_ARGS__) SV_PAIR(flags, 5, 3, 2, __VA_ARGS__)            \
    }

// The round's columns: XOR of the columns of the thread's set bits (the first
// eight packed from word c, the others from c2), and of every register index.
template <int TBITS>
__device__ __forceinline__ uint32_t thread_columns(cword* pc, uint32_t tid, int c, int c2)
{
    uint32_t v = 0;
    each<0, TBITS>([&](auto K) SV_INLINE {
        const uint32_t w = K < 8 ? pc[c + K / 2] : pc[c2 + (K - 8) / 2];
        v ^= (0u - ((tid >> K) & 1u)) & ((w >> (16 * (K & 1))) & 0xffffu);
    });
    return v;
}

template <int R>
__device__ __forceinline__ void reg_columns(cword* pc, int c, uint32_t (&v)[1 << R])
{
    each<0, (1 << R)>([&](auto J) SV_INLINE {
        v[J] = 0;
        each<0, R>([&](auto K) SV_INLINE {
            if constexpr ((J >> K) & 1) v[J] ^= (pc[c + K / 2] >> (16 * (K & 1))) & 0xffffu;
        });
    });
}

// tile index of the thread's first amplitude
template <int TBITS>
__device__ __forceinline__ uint32_t thread_index(cword* pc, uint32_t tid)
{
    uint32_t tix = 0;
    each<0, TBITS>([&](auto K) SV_INLINE {
        const uint32_t bits = K < 8 ? pc[7] : pc[9];
        tix |= (0u - ((tid >> K) & 1u)) & (1u << ((bits >> (4 * (K & 7))) & 15u));
    });
    return tix;
}

// The thread steps of a round (headers from ps on, `next` the first): the sign
// and the phase that all of the thread's amplitudes take.
__device__ __forceinline__ void thread_steps(cword* W, cword*& ps, u32x4& next, int count, uint32_t tix, uint32_t tile,
                                             uint32_t row, uint32_t& sign, Cx& phase)
{
    for (int g = count; g > 0; --g) {
        const u32x4 h = next;
        ps += kTileHeadWords;
        next = ld_head(ps);
        const uint32_t tctl = (h.x >> 16) & 0xfffu;
        const bool on = ((tile & h.y) == h.y) & ((tix & tctl) == tctl);
        if (h.x & TF_SIGN) {
            sign ^= on ? 0x80000000u : 0u;
            continue;
        }
        // no, one or two free bits
        const f32x8 m = ld_mat(W + (h.z & 0xffffu) + (h.z >> 16) * row);
        const bool b0 = ((((h.w >> 20) & 3u) == kPlaceThread ? tix : tile) >> (h.w & 255u)) & 1u;
        const bool b1 = ((((h.w >> 22) & 3u) == kPlaceThread ? tix : tile) >> ((h.w >> 8) & 255u)) & 1u;
        const int nfree = (h.w >> 16) & 3;
        const Cx one = sel(b0, Cx{m[2], m[3]}, Cx{m[0], m[1]});
        const Cx two = sel(b0, sel(b1, Cx{m[6], m[7]}, Cx{m[4], m[5]}), sel(b1, Cx{m[2], m[3]}, Cx{m[0], m[1]}));
        const Cx p = nfree == 0 ? Cx{m[0], m[1]} : nfree == 1 ? one : two;
        phase = sel(on, mul(p, phase), phase);
    }
}

// A PHASE step's phases by (register bit 0 set, register bit 1 set), and which
// register bits these are (0: none).
struct RegPhase {
    Cx q[4];
    int f0, f1;
    __device__ __forceinline__ Cx operator()(int j) const
    {
        const bool s0 = (j & f0) != 0, s1 = (j & f1) != 0;
        return sel(s0, sel(s1, q[3], q[2]), sel(s1, q[1], q[0]));
    }
};

__device__ __forceinline__ RegPhase reg_phase(const u32x4& h, cword* w, uint32_t tix, uint32_t tile)
{
    const f32x8 m = ld_mat(w);
    const int pl0 = (h.w >> 20) & 3, pl1 = (h.w >> 22) & 3, at0 = h.w & 255, at1 = (h.w >> 8) & 255;
    const bool b0 = (pl0 != kPlaceReg) & (bool)(((pl0 == kPlaceThread ? tix : tile) >> at0) & 1);
    const bool b1 = (pl1 != kPlaceReg) & (bool)(((pl1 == kPlaceThread ? tix : tile) >> at1) & 1);
    const int nfree = (h.w >> 16) & 3;
    const Cx e0{m[0], m[1]}, e1{m[2], m[3]}, e2{m[4], m[5]}, e3{m[6], m[7]};
    auto entry = [&](bool s0, bool s1) SV_INLINE {
        const Cx one = sel(s0, e1, e0);
        const Cx two = sel(s0, sel(s1, e3, e2), sel(s1, e1, e0));
        return nfree == 0 ? e0 : nfree == 1 ? one : two;
    };
    RegPhase r;
    r.f0 = pl0 == kPlaceReg && nfree > 0 ? 1 << at0 : 0;
    r.f1 = pl1 == kPlaceReg && nfree > 1 ? 1 << at1 : 0;
    r.q[0] = entry(b0, b1);
    r.q[1] = entry(b0, true);
    r.q[2] = entry(true, b1);
    r.q[3] = entry(true, true);
    return r;
}

// v plus the value of another lane (0 where the mask leaves the lane out)
template <int CTRL, int ROWS>
__device__ __forceinline__ double plus_lane(double v)
{
    const uint64_t b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROWS, 0xf, false);
    return v + __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// v of another lane (a DPP move without masks)
template <int CTRL>
__device__ __forceinline__ double lane_move(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// v plus v of lane ^ D, D = 16 or 32: the swap exchanges the odd groups of D
// lanes of one register with the even ones of the other.
template <int D>
__device__ __forceinline__ double add_swapped(double v)
{
    auto swap = [](int w) SV_INLINE {
        if constexpr (D == 16) return __builtin_amdgcn_permlane16_swap((uint32_t)w, (uint32_t)w, false, false);
        else return __builtin_amdgcn_permlane32_swap((uint32_t)w, (uint32_t)w, false, false);
    };
    const auto lo = swap(__double2loint(v)), hi = swap(__double2hiint(v));
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// the wave's sum, in lane 63
__device__ __forceinline__ double wave_sum(double v)
{
    v = plus_lane<0xb1, 0xf>(v);      // lane ^ 1
    v = plus_lane<0x4e, 0xf>(v);      // lane ^ 2
    v = plus_lane<0x141, 0xf>(v);     // mirrored within eight
    v = plus_lane<0x140, 0xf>(v);     // mirrored within sixteen
    v = plus_lane<0x142, 0xa>(v);     // lane 15 of a row to the next
    return plus_lane<0x143, 0xc>(v);  // lane 31 to the upper half
}

// The lines of a program of nw words brought into the scalar cache all at
// once: met one after the other, each would be a wait for memory.
__device__ __forceinline__ void touch_program(cword* W, int nw)
{
    uint32_t touch = 0;
    for (int i = 0; i < nw; i += 64) touch |= W[i] | W[i + 16] | W[i + 32] | W[i + 48];
    asm volatile("" ::"s"(touch));
}

}  // namespace sv
