// What the kernels that keep a tile of the state in LDS and apply gates one by
// one in registers share (gate passes, adjoint sweeps): index arithmetic,
// the register ops, and the host's choice of a pass's tile and gates.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "internal.hpp"
#include "tile.hpp"

namespace qvm {
namespace {

constexpr int kSlots = 4;                        // slots of a round, at most

template <typename R> struct GT;
template <> struct GT<float> {
    using T = float2;
    using V16 = float __attribute__((ext_vector_type(4)));
    static constexpr int EP = 2, C = 4, LMAX = 13;
};
template <> struct GT<double> {
    using T = double2;
    using V16 = double __attribute__((ext_vector_type(2)));
    static constexpr int EP = 1, C = 3, LMAX = 12;
};

// Bits of x placed on the set bits of mask, ascending, a run at a time.
__device__ __forceinline__ uint64_t place(uint64_t x, uint64_t mask) {
    uint64_t r = 0;
    while (mask) {
        const uint64_t low = mask & (~mask + 1);
        const uint64_t run = ((mask + low) & ~mask) - low;       // the lowest run of ones
        const int len = __builtin_popcountll(run);
        r |= (x * low) & run;
        x = len < 64 ? x >> len : 0;
        mask &= ~run;
    }
    return r;
}

// XOR (for disjoint bits: OR) of the entries at the bits set in j.
template <int N, typename U>
__device__ __forceinline__ U subset(const U (&v)[N], int j) {
    U r = 0;
#pragma unroll
    for (int k = 0; k < N; ++k)
        if ((j >> k) & 1) r ^= v[k];
    return r;
}

template <typename T>
__device__ __forceinline__ T gld(uint32_t off) {
    return *(const __attribute__((address_space(3))) T*)(size_t)off;
}
template <typename T>
__device__ __forceinline__ void gst(uint32_t off, T v) {
    *(__attribute__((address_space(3))) T*)(size_t)off = v;
}
template <typename R> struct Vec2;
template <> struct Vec2<float> { using V = float __attribute__((ext_vector_type(2))); };
template <> struct Vec2<double> { using V = double __attribute__((ext_vector_type(2))); };

// ------------------------------------------------- ops on the 16 registers
__device__ __forceinline__ float flip_sign(float x, uint32_t f) { return __uint_as_float(__float_as_uint(x) ^ f); }
__device__ __forceinline__ double flip_sign(double x, uint32_t f) {
    return __hiloint2double(__double2hiint(x) ^ (int)f, __double2loint(x));
}

// Ops in place.  A loop over ops keeps a thread's amplitudes where they are
// only if every op can end in the registers it began in; one that cannot
// makes each op, also the others, copy all amplitudes (32 moves after the 48
// multiply-adds of a rotation of 16 complex128 amplitudes).  So
// - an op that needs its inputs until its last result is done takes the
//   results back by moves that the compiler does not see through (move_to);
// - ops are chosen by one test after the other, each without an else, on
//   copies of the code that the compiler cannot relate (is): control flow is
//   structured into such tests anyway, and an op behind an else would keep the
//   amplitudes of before the tested op alive through it.
__device__ __forceinline__ bool is(uint32_t code, uint32_t c) {
    asm volatile("" : "+s"(code));
    return code == c;
}
__device__ __forceinline__ bool below(uint32_t code, uint32_t c) {
    asm volatile("" : "+s"(code));
    return code < c;
}
__device__ __forceinline__ float move_to(float x) {
    float d;
    asm volatile("v_mov_b32 %0, %1" : "=v"(d) : "v"(x));
    return d;
}
__device__ __forceinline__ double move_to(double x) {
    double d;
    asm volatile("v_mov_b64 %0, %1" : "=v"(d) : "v"(x));
    return d;
}

template <typename R, typename T>
__device__ __forceinline__ void pair2(const R* m, T& v0, T& v1) {
    T o0, o1;
    o0.x = m[0] * v0.x - m[1] * v0.y + m[2] * v1.x - m[3] * v1.y;
    o0.y = m[0] * v0.y + m[1] * v0.x + m[2] * v1.y + m[3] * v1.x;
    o1.x = m[4] * v0.x - m[5] * v0.y + m[6] * v1.x - m[7] * v1.y;
    o1.y = m[4] * v0.y + m[5] * v0.x + m[6] * v1.y + m[7] * v1.x;
    asm volatile("" : "+v"(o0.x), "+v"(o0.y), "+v"(o1.x), "+v"(o1.y));
    v0 = {move_to(o0.x), move_to(o0.y)};
    v1 = {move_to(o1.x), move_to(o1.y)};
}

// v times p, in place.
template <typename R, typename T>
__device__ __forceinline__ void phase1(R pr, R pi, T& v) {
    const R t = pi * v.y, u = pr * v.y;
    v.y = u + pi * v.x;
    v.x = pr * v.x - t;
}

template <typename R, int S, typename T, int NA>
__device__ __forceinline__ void op_d1(T (&a)[NA], const R* m, uint32_t jbits) {
    constexpr uint32_t ALL = (S == 0 ? 0x5555u : S == 1 ? 0x3333u : S == 2 ? 0x0f0fu : 0x00ffu) & ((1u << NA) - 1u);
    if (is(jbits, ALL)) {
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (!(j & (1 << S))) pair2<R>(m, a[j], a[j | (1 << S)]);
        jbits = 0;
    }
    if (!is(jbits, 0)) {
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (!(j & (1 << S)) && ((jbits >> j) & 1)) pair2<R>(m, a[j], a[j | (1 << S)]);
    }
}

// Amplitudes j and j ^ X exchanged, in place (no select of both).
__device__ __forceinline__ void exchange(float& x, float& y, uint32_t m) {
    const uint32_t a = __float_as_uint(x), b = __float_as_uint(y), d = (a ^ b) & m;
    x = __uint_as_float(a ^ d);
    y = __uint_as_float(b ^ d);
}
__device__ __forceinline__ void exchange(double& x, double& y, uint32_t m) {
    const uint32_t al = __double2loint(x), ah = __double2hiint(x), bl = __double2loint(y), bh = __double2hiint(y);
    const uint32_t dl = (al ^ bl) & m, dh = (ah ^ bh) & m;
    x = __hiloint2double(ah ^ dh, al ^ dl);
    y = __hiloint2double(bh ^ dh, bl ^ dl);
}
template <int X, typename T, int NA>
__device__ __forceinline__ void op_move(T (&a)[NA], uint32_t jbits) {
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        if (j & (X & -X)) continue;                            // the lowest moved bit is 0 in the first of a pair
        const uint32_t m = 0u - ((jbits >> j) & 1u);
        exchange(a[j].x, a[j ^ X].x, m);
        exchange(a[j].y, a[j ^ X].y, m);
    }
}

// =============================================================== scheduling
inline int pc(uint64_t v) { return __builtin_popcountll(v); }

// A gate acts non-diagonally on the bits xq and diagonally on the bits zq.
struct Sched {
    uint64_t bx = 0, bz = 0;                     // bits held by gates passed over
    template <typename G> bool free(const G& g) const { return !(g.xq & (bx | bz)) && !(g.zq & bx); }
    template <typename G> void hold(const G& g) {
        bx |= g.xq;
        bz |= g.zq;
    }
};

inline uint32_t local_bits(uint64_t phys, uint64_t qmask) {            // phys bits (all in qmask) as tile-local bits
    uint32_t r = 0;
    for (uint64_t m = phys; m; m &= m - 1)
        r |= 1u << pc(qmask & ((m & (~m + 1)) - 1));
    return r;
}
inline uint32_t tile_index_bits(uint64_t phys, uint64_t qmask) {       // phys bits outside qmask as bits of the tile index
    uint32_t r = 0;
    for (uint64_t m = phys & ~qmask; m; m &= m - 1) r |= 1u << pc(~qmask & ((m & (~m + 1)) - 1));
    return r;
}

// Bits of the tile for the next pass and the gates it takes: gates in list
// order, a gate passed over when a gate before it that was passed over
// holds one of its bits (two gates that both act diagonally on the bits
// they share commute) or when its bits do not fit in the tile.
template <typename GATE>
uint64_t take_pass(const std::vector<GATE>& G, const std::vector<char>& done, size_t first, int n, int L, int c,
                   uint64_t need, std::vector<int>& ops) {
    const uint64_t all = n >= 64 ? ~0ull : (1ull << n) - 1;
    uint64_t T = ((1ull << std::min(c, n)) - 1) | need;
    if (L >= n) T = all;
    Sched s;
    ops.clear();
    for (size_t i = first; i < G.size() && (s.bx & all) != all; ++i) {
        if (done[i]) continue;
        const GATE& g = G[i];
        if (s.free(g) && pc(T | g.xq) <= L) {
            T |= g.xq;
            ops.push_back((int)i);
        } else {
            s.hold(g);
        }
    }
    for (int q = 0; q < n && pc(T) < L; ++q) T |= 1ull << q;     // long runs: the lowest bits left
    return T;
}

}  // namespace
}  // namespace qvm
