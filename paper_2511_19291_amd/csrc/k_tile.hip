// k_tile.hip -- a list of gates per sweep of the state.
//
// One workgroup loads a tile (tile.h) with 16-byte accesses, keeps it in LDS
// (8-byte elements, swizzled), runs the program's rounds and writes it back.
// Within a round a thread's 2^R amplitudes stay in registers; between rounds
// every thread writes the elements it read back to where it read them, so a
// single barrier separates two rounds. A run of CNOTs, X and SWAPs at a
// round's end is an affine map of the tile's index: it only changes the
// addresses written to.
//
// Bound: far beyond the caches, the vector unit. 27-qubit brickwork (540 U3 +
// 260 CZ): 23 launches at 0.92 ms, 21.8 ms in all (one sweep per gate:
// 213 ms); 16 instructions a pair and general gate are 2880 of the 4000
// vector instructions of a wave and launch, issued at 97 % of one every four
// cycles; HBM traffic (16 B per amplitude and launch) would take 0.33 ms of
// each 0.92. The matrix cores (v_mfma_f32_4x4x1, one pair per lane) halve the
// instructions of the gates but not the time (0.92 ms a launch): their
// results need moving back to the amplitudes' registers. Small states: the
// latency of a step, about 0.4 us, half of it branches; a 12-qubit,
// 140-gate circuit takes 39 us (140 launches: 370 us).
//
// The program travels in the kernel arguments (read through the scalar
// cache), so a launch needs no upload, keeps no buffer and can be captured.
#include <cstddef>

#include "tile_device.h"

namespace sv {

namespace {

template <int R>
__global__ __launch_bounds__(1 << (kTileMaxBits - R), 4) void k_tile(TileArgs a)
{
    constexpr int M = 1 << R, TBITS = kTileMaxBits - R;    // register amplitudes; thread bits of a full tile
    __shared__ float2 lds[1 << kTileMaxBits];
    cword* W = (cword*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                        offsetof(TileArgs, words));
    const uint32_t tid = threadIdx.x;
    const int T = a.T;
    touch_program(W, a.nwords);
    const bool act = tid < (1u << (T - R));
    const int row = a.row0 + (int)blockIdx.y;
    const uint32_t tile = (uint32_t)xcd_block(blockIdx.x, gridDim.x);
    float2* psi = row < a.nrow0 ? a.p0 + (uint64_t)row * a.N : a.p1 + (uint64_t)(row - a.nrow0) * a.N;
    uint64_t base = tile;
    for (int i = 0; i < T; ++i) {
        const int p = a.pos[i];
        base = ((base >> p) << (p + 1)) | (base & ((1ull << p) - 1ull));
    }
    psi += base;

    // memory side: float4 e = 2 tid + 2^(T-R+1) i, i < M / 2: its place in
    // memory and its LDS element. Formed for the loads and again for the
    // stores rather than held in registers across the gates.
    auto place = [&](uint32_t t, uint64_t& off, uint32_t& el) SV_INLINE {
        off = 0;
        el = 0;
        each<1, TBITS + 1>([&](auto B) SV_INLINE {
            const uint32_t on = (t >> (B - 1)) & 1u;
            off |= (uint64_t)on << a.pos[B];
            el ^= (0u - on) & swz_col(B);
        });
    };
    auto part = [&](int i, uint64_t& ioff, uint32_t& iel) SV_INLINE {
        ioff = 0;
        iel = 0;
        each<0, R - 1>([&](auto K) SV_INLINE {
            if ((i >> K) & 1) {
                const int b = T - R + 1 + K;
                ioff |= 1ull << a.pos[b];
                iel ^= (1u << b) ^ (b >= 4 ? kTileSwz[b - 4] : 0u);
            }
        });
    };
    if (act) {
        uint64_t off, ioff;
        uint32_t el, iel;
        place(tid, off, el);
        float4 v[M / 2];
        each<0, M / 2>([&](auto I) SV_INLINE {
            part(I, ioff, iel);
            v[I] = ld4(psi + off + ioff);
        });
        each<0, M / 2>([&](auto I) SV_INLINE {
            part(I, ioff, iel);
            lds[el ^ iel] = lo2(v[I]);
            lds[el ^ iel ^ 1] = hi2(v[I]);
        });
    }

    cword* pc = W;
    for (int r = 0; r < a.nrounds; ++r) {
        const uint32_t r0 = pc[0];
        const int nsteps = (int)(r0 & 255u), nouter = (int)((r0 >> 8) & 255u);
        uint32_t at = thread_columns<TBITS>(pc, tid, 1, 8);
        const uint32_t tix = thread_index<TBITS>(pc, tid);
        // Phases that all of the thread's amplitudes take: they commute with
        // everything else in the round, so they are collected first and
        // applied once.
        uint32_t sign = 0;
        Cx phase{1.f, 0.f};
        cword* ps = pc + kTileRoundWords;
        const bool mapped = (r0 >> 18) & 1u;
        if (mapped) ps += kTileMapWords + ((nouter + 3) & ~3);
        u32x4 next = ld_head(ps);                 // one step ahead (the array has room behind the last)
        thread_steps(W, ps, next, (int)(r0 >> 24), tix, tile, blockIdx.y, sign, phase);
        uint32_t rel[M];
        reg_columns<R>(pc, 5, rel);
        __syncthreads();
        Amps<M> x;
        each<0, M>([&](auto J) SV_INLINE {
            const float2 v = act ? lds[at ^ rel[J]] : make_float2(0.f, 0.f);
            x.re[J] = v.x;
            x.im[J] = v.y;
        });
        uint32_t flips = 0;
        for (int g = 0; g < nsteps; ++g) {
            const u32x4 h = next;
            ps += kTileHeadWords;
            next = ld_head(ps);
            if (h.x & TF_LAYER) {
                // up to one uncontrolled gate of one kind on each register bit
                cword* w = W + h.z * blockIdx.y;
                f32x8 m[4];
                each<0, R>([&](auto B) SV_INLINE { m[B] = ld_mat(w + 4 * ((h.y >> (8 * B)) & 255u)); });
                const uint32_t on_bits = h.x >> 8;
                if (h.x & TF_DENSE) SV_BITS(on_bits, pairs<M, TB>(x, Dense{m[TB]});)
                if (h.x & TF_REAL) SV_BITS(on_bits, pairs<M, TB>(x, Real{m[TB]});)
                if (h.x & TF_IMOFF) SV_BITS(on_bits, pairs<M, TB>(x, ImOff{m[TB]});)
                if (h.x & TF_DIAG) SV_BITS(on_bits, pairs<M, TB>(x, Diag{m[TB]});)
            }
            if (h.x & TF_OTHER) {
                const uint32_t tctl = (h.x >> 16) & 0xfffu;
                const bool on = ((tile & h.y) == h.y) & ((tix & tctl) == tctl);
                const Where where{on, (int)((h.x >> 8) & 15)};
                cword* w = W + (h.z & 0xffffu) + (h.z >> 16) * blockIdx.y;
                // sign flips: those without thread controls are collected
                // while they follow each other, one bit per register amplitude
                if (h.x & TF_SIGN) flips ^= (tile & h.y) == h.y ? h.w : 0u;
                if (h.x & TF_APPLY) {
                    each<0, M>([&](auto J) SV_INLINE { flip(x.re[J], x.im[J], (flips << (31 - J)) & 0x80000000u); });
                    flips = 0;
                }
                if (h.x & TF_LANE_SIGN) {
                    const uint32_t mine = on ? h.w : 0u;
                    each<0, M>([&](auto J) SV_INLINE { flip_v(x.re[J], x.im[J], (mine << (31 - J)) & 0x80000000u); });
                }
                if (h.x & TF_PHASE) phases<M>(x, where, reg_phase(h, w, tix, tile));
                if (h.x & TF_CTRL) SV_BITS(h.w, pairs_where<M, TB>(x, where, ld_mat(w));)
                if (h.x & TF_DENSE2) SV_PAIRS(h.w, dense2<M, A, B>(x, where, w);)
            }
        }
        if ((r0 >> 16) & 1u)
            each<0, M>([&](auto J) SV_INLINE {
                flip_v(x.re[J], x.im[J], sign);
            });
        if ((r0 >> 17) & 1u)
            each<0, M>([&](auto J) SV_INLINE { times(x.re[J], x.im[J], phase); });
        if (mapped) {
            // the index map costs nothing but other addresses (and a barrier:
            // they are other threads' elements)
            at = thread_columns<TBITS>(pc, tid, 12, 16);
            reg_columns<R>(pc, 17, rel);
            at ^= pc[19];
            for (int i = 0; i < nouter; ++i) {
                const uint32_t o = pc[20 + i];
                if ((tile >> (o & 31u)) & 1u) at ^= o >> 16;
            }
            __syncthreads();
        }
        if (act)
            each<0, M>([&](auto J) SV_INLINE { lds[at ^ rel[J]] = make_float2(x.re[J], x.im[J]); });
        pc = ps;
    }
    __syncthreads();
    if (act) {
        uint32_t t = tid;
        asm volatile("" : "+v"(t));
        uint64_t off, ioff;
        uint32_t el, iel;
        place(t, off, el);
        each<0, M / 2>([&](auto I) SV_INLINE {
            part(I, ioff, iel);
            st4(psi + off + ioff, pack4(lds[el ^ iel], lds[el ^ iel ^ 1]));
        });
    }
}

}  // namespace

void launch_tile(const TileArgs& a, int rows, int reg_bits, hipStream_t st)
{
    const int n = __builtin_ctzll(a.N);
    const dim3 grid((unsigned)(1ull << (n - a.T)), (unsigned)rows);
    const dim3 block((unsigned)std::max(64, 1 << (a.T - reg_bits)));
    if (reg_bits == kTileRegBits - 1) hipLaunchKernelGGL(k_tile<kTileRegBits - 1>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(k_tile<kTileRegBits>, grid, block, 0, st, a);
    SV_HIP(hipGetLastError());
}

}  // namespace sv
