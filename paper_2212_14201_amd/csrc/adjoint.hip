// Batched adjoint (reverse-sweep) gradient of f(theta) = <psi(theta)|H|psi(theta)>
// for circuits of one-target gates (any controls) whose trainable gates are
// RX/RY/RZ rotations U = exp(-i theta G / 2), G in {X, Y, Z} (the paper's
// variational circuits, "Variational quantum circuit"; the method is the
// published reverse sweep of Jones & Gacon, arXiv:2009.02823):
//   psi_L = U_L ... U_1 |0>,  lambda_L = H psi_L,  f = Re <psi_L|lambda_L>,
//   for l = L .. 1:  df/dtheta_l = Im <lambda_l| G_l |psi_l>   (trainable l),
//                    psi <- U_l^dagger psi,  lambda <- U_l^dagger lambda.
// A controlled rotation's generator acts only where its controls are 1.
//
// All batch elements advance together: one launch per pass covers the whole
// batch (blockIdx.y = batch element).  A pass keeps a tile of psi (and, in
// the reverse sweep, the same tile of lambda) in LDS and runs every gate of
// the list that can run on the tile's qubits, in rounds of a few slot qubits
// whose amplitudes a thread holds in registers (the gate passes of qvm_run,
// with a matrix per batch element); the reverse sweep undoes the passes in
// the opposite order.
//
// complex128: consecutive uncontrolled one-target gates on a qubit, U = U_m
// ... U_1, are applied as one matrix, and all their gradients come from three
// numbers of the qubit after the run, S_P = Im <lambda| P |psi> for P = X, Y,
// Z: with V = U_m ... U_{l+1}, Im <lambda_l| G |psi_l> = Im <lambda| V G
// V^dagger |psi> = sum_P R_PG S_P, R the rotation of V.
//
// complex64: gate by gate, in the order of the groups below, each product
// rounded in a fixed way (adj_apply), as merged or reordered gates would round
// the states (and so the gradients) otherwise.
//
// Before, both sweeps in both types launched a kernel per group of four (three)
// target qubits, and the host computed every matrix.  20 qubits, complex64, 944
// gates (640 trainable), batch 64: 92 groups each way, forward 23.6 ms, reverse
// 58.4, a call 85.9 ms; now 41 passes each way, 13.2 and 44 ms, a call 60.9.
// The passes' traffic takes 7 and 14 ms; in the reverse sweep vector
// instructions take 61% of the cycles (half of them the gradient terms, which
// are formed and summed in double precision), with two waves per SIMD.  11
// qubits, complex128, batch 8, a state one tile: a call 568 us, now 265 (8
// blocks: a chain of rounds, bound by latency).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "gatepass.hpp"

namespace qvm {

template <typename R> struct AC2;
template <> struct AC2<float> { using T = float2; };
template <> struct AC2<double> { using T = double2; };

constexpr int kAdjBlocks = 64;        // reduction partials per row, at most
constexpr int kAdjMaxSums = 192;      // gradient sums per pass (they stay in LDS)
constexpr int kAdjMaxTrain = 64;      // trainable gates per group
constexpr int kAdjMaxOps = 512;       // gates per group, steps per pass
constexpr int kAdjSlots = 4;          // slots of a round, at most
constexpr int kAdjThreads = 256;
template <typename R> constexpr int adj_slots() { return sizeof(R) == 4 ? 4 : 3; }
template <typename R> constexpr int adj_width() { return sizeof(R) == 4 ? 12 : 11; }   // 32 KiB of a state

__device__ double adj_block_sum(double v, double* sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// A record applies to the register pairs in jbits of thread t in tile w when
// (t & tm) == tv and (w & om) == ov (as in gatepass.hip).  Codes, + s for
// slot s: AD_MAT the matrix of run `mat`; AD_RE the same without its imaginary
// part (RY, H: all zero), AD_DG without its off-diagonal entries (RZ); AD_MOVE
// the pair's amplitudes exchanged; AD_SIGN a factor of -1.
enum : uint32_t { AD_MAT = 0, AD_RE = 4, AD_DG = 8, AD_MOVE = 12, AD_SIGN = 16, AD_RX = 20 };
struct AdjOp {
    uint32_t code, jbits;
    uint32_t tm, tv, om, ov;
    uint32_t mat;
    uint32_t grad;           // 0, or (first of its sums in the pass + 1) << 3 | the Paulis needed (1 X, 2 Y, 4 Z)
};
struct AdjRound {
    uint32_t bit[kAdjSlots]; // tile-local bit of each slot, ascending
    uint32_t lds[kAdjSlots]; // its LDS byte address
    uint32_t nops, pad[7];
};
static_assert(sizeof(AdjOp) == 32 && sizeof(AdjRound) == 64, "whole scalar loads");

struct AdjPass {
    uint64_t qmask;          // tile bits
    uint64_t state_len;
    uint32_t L, nrounds;
    uint32_t words;          // offset of the pass's records
    uint32_t ntiles;
    uint32_t nsum, row0;     // gradient sums; partial row of the first one
    uint32_t init;           // forward, first pass: the state is |0..0>, not what memory holds
    uint32_t top[kAdjSlots]; // positions of the highest tile bits, ascending
};

// A value widened where it is used: left to itself the compiler widens all of
// a thread's amplitudes ahead of the branches that use some (256 registers).
__device__ __forceinline__ double widen(float x) {
    double d;
    asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(d) : "v"(x));
    return d;
}
__device__ __forceinline__ double widen(double x) { return x; }

// S_X, S_Y or S_Z (V = 1, 2, 3) of one pair (the qubit's 0 and 1 amplitudes).
template <int V, typename T>
__device__ __forceinline__ double pauli_term(const T& a0, const T& a1, const T& l0, const T& l1) {
    const double p0r = widen(a0.x), p0i = widen(a0.y), p1r = widen(a1.x), p1i = widen(a1.y);
    const double q0r = widen(l0.x), q0i = widen(l0.y), q1r = widen(l1.x), q1i = widen(l1.y);
    if (V == 1) return (q0r * p1i - q0i * p1r) + (q1r * p0i - q1i * p0r);        // X: (p1, p0)
    if (V == 2) return (q1r * p0r + q1i * p0i) - (q0r * p1r + q0i * p1i);        // Y: (-i p1, i p0)
    return (q0r * p0i - q0i * p0r) - (q1r * p1i - q1i * p1r);                    // Z: (p0, -p1)
}

// The wave's sum, in lane 63: register-to-register moves, rows of 16 lanes
// first (exchanges through LDS held the wave up for every gate).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)u, CTRL, ROWS, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
    return v + __longlong_as_double((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double wave_total(double v) {
    v = dpp_add<0x111, 0xf>(v);      // row_shr:1
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
}

// The sum of one Pauli on slot S, added to the wave's in LDS at `at`.
template <int V, int S, int NA, typename T>
__device__ __forceinline__ void adj_sum(const T (&a)[NA], const T (&l)[NA], uint32_t jb, bool act, uint32_t at,
                                        uint32_t lane) {
    double g = 0;
    constexpr uint32_t ALL = (S == 0 ? 0x5555u : S == 1 ? 0x3333u : S == 2 ? 0x0f0fu : 0x00ffu) & ((1u << NA) - 1u);
    if (act && jb == ALL) {
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (!(j & (1 << S))) {
                g += pauli_term<V>(a[j], a[j | (1 << S)], l[j], l[j | (1 << S)]);
                __builtin_amdgcn_sched_barrier(0);
            }
    } else if (act) {
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (!(j & (1 << S)) && ((jb >> j) & 1)) {
                g += pauli_term<V>(a[j], a[j | (1 << S)], l[j], l[j | (1 << S)]);
                // (pairs one after the other: eight pairs' widened values
                // at once would take 128 registers)
                __builtin_amdgcn_sched_barrier(0);
            }
    }
    g = wave_total(g);
    if (lane == 63) gst<double>(at, gld<double>(at) + g);
}

// One product rounded, the other fused.
__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// A step on slot S of one state's registers, in place (gatepass.hpp).  Every
// product is written as it rounds: the first of a row's four rounded, the
// others fused in order; in the real part the second comes first.  SWAP: in
// the imaginary part too, except in the first pair.  complex64 states are
// rounded so, psi without and lambda with SWAP, as the sweep's first kernels
// were compiled; other orders change the gradients by 1e-7 of their size.
// The forms without the zero entries round alike.  (As dense products with an
// else for every kind the reverse sweep took 55 ms, these forms with all
// amplitudes copied for every gate 57, in place 47, without a branch for
// every pair 44.)
template <typename R, int S, bool ADJ, bool SWAP, int NA, typename T>
__device__ __forceinline__ void adj_apply(T (&a)[NA], const R* m, uint32_t kind, uint32_t jb) {
    // the matrix m or its adjoint, negated where it is used (a transposed copy
    // made ahead of the branches costs all ops their place again)
    struct {
        const R* m;
        __device__ __forceinline__ R operator[](int i) const {
            if (!ADJ) return m[i];
            const int j = i == 2 || i == 3 ? i + 2 : i == 4 || i == 5 ? i - 2 : i;
            return (i & 1) ? -m[j] : m[j];
        }
    } const u{m};
    constexpr uint32_t ALL = (S == 0 ? 0x5555u : S == 1 ? 0x3333u : S == 2 ? 0x0f0fu : 0x00ffu) & ((1u << NA) - 1u);
    auto each = [&](auto f) {
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (!(j & (1 << S)) && ((jb >> j) & 1)) f(a[j], a[j | (1 << S)], SWAP && j != 0);
    };
    // (all pairs without a branch for each)
    auto most = [&](auto f) {
        if (is(jb, ALL)) {
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if (!(j & (1 << S))) f(a[j], a[j | (1 << S)], SWAP && j != 0);
        }
        if (!is(jb, ALL)) each(f);
    };
    if (is(kind, AD_RE))
        most([&](T& v0, T& v1, bool) {
            const R x = u[4] * v0.x, y = u[4] * v0.y;
            v0.x = mad(u[2], v1.x, u[0] * v0.x);
            v0.y = mad(u[2], v1.y, u[0] * v0.y);
            v1.x = mad(u[6], v1.x, x);
            v1.y = mad(u[6], v1.y, y);
        });
    if (is(kind, AD_RX))
        most([&](T& v0, T& v1, bool) {
            const R x = u[5] * v0.y, y = u[5] * v0.x;
            v0.x = mad(-u[3], v1.y, u[0] * v0.x);
            v0.y = mad(u[3], v1.x, u[0] * v0.y);
            v1.x = mad(u[6], v1.x, -x);
            v1.y = mad(u[6], v1.y, y);
        });
    if (is(kind, AD_DG))
        most([&](T& v0, T& v1, bool sw) {
            const R t = u[1] * v0.y, x = v0.x;
            v0.y = sw ? mad(u[0], v0.y, u[1] * x) : mad(u[1], x, u[0] * v0.y);
            v0.x = mad(u[0], x, -t);
            const R r = mad(-u[7], v1.y, u[6] * v1.x);
            v1.y = mad(u[7], v1.x, u[6] * v1.y);
            asm volatile("" : "+v"(v1.y));
            v1.x = move_to(r);
        });
    if (is(kind, AD_MOVE)) op_move<(1 << S)>(a, jb);
    if (is(kind, AD_MAT))
        each([&](T& v0, T& v1, bool sw) {
            auto re = [&](int i) {
                return mad(-u[i + 3], v1.y, mad(u[i + 2], v1.x, mad(u[i], v0.x, -(u[i + 1] * v0.y))));
            };
            auto im = [&](int i) {
                const R t = sw ? mad(u[i], v0.y, u[i + 1] * v0.x) : mad(u[i + 1], v0.x, u[i] * v0.y);
                return mad(u[i + 3], v1.x, mad(u[i + 2], v1.y, t));
            };
            T o0{re(0), im(0)}, o1{re(4), im(4)};
            asm volatile("" : "+v"(o0.x), "+v"(o0.y), "+v"(o1.x), "+v"(o1.y));
            v0 = T{move_to(o0.x), move_to(o0.y)};
            v1 = T{move_to(o1.x), move_to(o1.y)};
        });
}

// A step on one state.
template <typename R, int RS, bool ADJ, bool SWAP, int NA, typename T>
__device__ __forceinline__ void adj_step(T (&a)[NA], const R* u, uint32_t kind, uint32_t slot, uint32_t jb, bool act) {
    uint32_t on = act;
    asm volatile("" : "+v"(on));
    if (on) {
        if (is(kind, AD_SIGN)) {
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                const uint32_t f = (jb << (31 - j)) & 0x80000000u;
                a[j].x = flip_sign(a[j].x, f);
                a[j].y = flip_sign(a[j].y, f);
            }
        }
        if (is(slot, 0)) adj_apply<R, 0, ADJ, SWAP, NA>(a, u, kind, jb);
        if constexpr (RS > 1)
            if (is(slot, 1)) adj_apply<R, 1, ADJ, SWAP, NA>(a, u, kind, jb);
        if constexpr (RS > 2)
            if (is(slot, 2)) adj_apply<R, 2, ADJ, SWAP, NA>(a, u, kind, jb);
        if constexpr (RS > 3)
            if (is(slot, 3)) adj_apply<R, 3, ADJ, SWAP, NA>(a, u, kind, jb);
    }
}

template <typename R, int RS, bool REV>
__global__ __launch_bounds__(256, REV ? 2 : 4) void k_adj_pass(typename AC2<R>::T* __restrict__ psi,
                                                     typename AC2<R>::T* __restrict__ lam, AdjPass A,
                                                     const uint32_t* __restrict__ table,
                                                     const R* __restrict__ mats, uint32_t batch, uint32_t nblk,
                                                     double* __restrict__ part) {
    using T = typename AC2<R>::T;
    using V16 = typename GT<R>::V16;
    using V2 = typename Vec2<R>::V;
    // (constant address space: the stores to the states do not touch these)
    typedef uint32_t U8 __attribute__((ext_vector_type(8), aligned(4)));
    typedef const __attribute__((address_space(4))) uint32_t* CW;
    typedef const __attribute__((address_space(4))) U8* C8;
    typedef const __attribute__((address_space(4))) R* CR;
    constexpr int EP = GT<R>::EP, NA = 1 << RS;
    constexpr int NIT = NA >= EP ? NA / EP : 1;                // 16-byte pieces per thread
    constexpr int PB = NIT == 1 ? 0 : EP == 2 ? RS - 1 : RS;   // bits of the piece index
    constexpr uint32_t ES = sizeof(T);
    constexpr int NS = REV ? 2 : 1;                            // states
    const uint32_t nt = 1u << (A.L - RS);                      // working threads
    const uint32_t tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t b = blockIdx.y;
    const bool live = tid < nt;
    const uint32_t lam0 = ES << A.L;                           // LDS: psi tile, lambda tile, sums
    const uint32_t acc0 = lam0 * NS;
    T* P[2] = {psi + (size_t)b * A.state_len, lam + (size_t)b * A.state_len};
    if constexpr (REV) {
        for (uint32_t i = tid; i < A.nsum * nw; i += blockDim.x) gst<double>(acc0 + 8 * i, 0.0);
    }
    uint64_t gtop[PB ? PB : 1];
    uint32_t stop[PB ? PB : 1];
#pragma unroll
    for (int k = 0; k < PB; ++k) {
        gtop[k] = 1ull << A.top[kAdjSlots - PB + k];
        stop[k] = tile_swizzle(1u << (A.L - PB + k));
    }
    auto goff = [&](int i) -> uint64_t { if constexpr (PB > 0) return subset<PB>(gtop, i); else return 0; };
    auto soff = [&](int i) -> uint32_t { if constexpr (PB > 0) return subset<PB>(stop, i); else return 0; };
    const uint64_t gt = place(EP * tid, A.qmask);
    const uint32_t st0 = tile_swizzle(EP * tid);
    for (uint32_t w = blockIdx.x; w < A.ntiles; w += gridDim.x) {
        const uint64_t g0 = place(w, ~A.qmask) + gt;
        if (live) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                V16 v[NIT];
#pragma unroll
                for (int i = 0; i < NIT; ++i) {
                    if (!REV && A.init) {
                        v[i] = V16{};
                        if (g0 + goff(i) == 0) v[i][0] = 1;
                    } else {
                        v[i] = __builtin_nontemporal_load((const V16*)(P[s] + g0 + goff(i)));
                    }
                }
#pragma unroll
                for (int i = 0; i < NIT; ++i) {
                    const uint32_t q = st0 ^ soff(i);
                    if constexpr (EP == 2) {
                        const V16 x = (q & 1) ? V16{v[i][2], v[i][3], v[i][0], v[i][1]} : v[i];
                        gst<V16>(s * lam0 + (q & ~1u) * ES, x);
                    } else {
                        gst<V16>(s * lam0 + q * ES, v[i]);
                    }
                }
            }
        }
        __syncthreads();
        CW p = (CW)table + A.words;
        for (uint32_t r = 0; r < A.nrounds; ++r) {
            const U8 hd = *(C8)p;
            const uint32_t nops = p[8];
            p += sizeof(AdjRound) / 4;
            // the head one record ahead, the matrix of the record at hand
            // while the head after it is on its way
            U8 h = *(C8)p;
            uint32_t le = tid;                                 // a zero inserted at every slot
#pragma unroll
            for (int k = 0; k < RS; ++k) le = ((le & ~(hd[k] - 1)) << 1) | (le & (hd[k] - 1));
            const uint32_t sl = tile_swizzle(le) * ES;
            uint32_t so[RS];
#pragma unroll
            for (int k = 0; k < RS; ++k) so[k] = hd[kAdjSlots + k];
            T a[NA], l[NA];
            if (live) {
#pragma unroll
                for (int j = 0; j < NA; ++j) {
                    const uint32_t at = sl ^ subset<RS>(so, j);
                    const V2 x = gld<V2>(at);
                    a[j].x = x[0];
                    a[j].y = x[1];
                    if constexpr (REV) {
                        const V2 y = gld<V2>(lam0 + at);
                        l[j].x = y[0];
                        l[j].y = y[1];
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < NA; ++j) a[j] = l[j] = T{0, 0};
            }
            R m[8];
            auto matrix = [&](uint32_t idx) {
                CR q = (CR)mats + ((size_t)idx * batch + b) * 8;
#pragma unroll
                for (int i = 0; i < 8; ++i) m[i] = q[i];
            };
            matrix(h[6]);
            for (uint32_t oi = 0; oi < nops; ++oi) {
                const U8 cur = h;
                R u[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) u[i] = m[i];
                p += sizeof(AdjOp) / 4;
                h = *(C8)p;                                    // (after the last record: in bounds, not used)
                if ((w & cur[4]) == cur[5]) {
                    const bool act = live && (le & cur[2]) == cur[3];
                    const uint32_t jb = cur[1], kind = cur[0] & ~3u, slot = cur[0] & 3u, need = cur[7] & 7u;
                    const uint32_t at = acc0 + 8 * (wave * A.nsum + (cur[7] >> 3) - 1);
                    // (the sums first, by themselves: what changes the
                    // amplitudes is one region of its own)
                    if constexpr (REV) {
                        if (need) {
#define QVM_ADJ_SUM(SL)                                                                           \
    if constexpr (SL < RS)                                                                        \
        if (is(slot, SL)) {                                                                       \
            if (need & 1) adj_sum<1, SL, NA>(a, l, jb, act, at, lane);                            \
            if (need & 2) adj_sum<2, SL, NA>(a, l, jb, act, at + 8 * (need & 1), lane);           \
            if (need & 4) adj_sum<3, SL, NA>(a, l, jb, act, at + 8 * __popc(need & 3), lane);     \
        }
                            QVM_ADJ_SUM(0) QVM_ADJ_SUM(1) QVM_ADJ_SUM(2) QVM_ADJ_SUM(3)
#undef QVM_ADJ_SUM
                        }
                    }
                    adj_step<R, RS, REV, false, NA>(a, u, kind, slot, jb, act);
                    if constexpr (REV) adj_step<R, RS, true, sizeof(R) == 4, NA>(l, u, kind, slot, jb, act);
                }
                matrix(oi + 1 < nops ? h[6] : 0);
            }
            if (live) {
#pragma unroll
                for (int j = 0; j < NA; ++j) {
                    const uint32_t at = sl ^ subset<RS>(so, j);
                    gst<V2>(at, V2{a[j].x, a[j].y});
                    if constexpr (REV) gst<V2>(lam0 + at, V2{l[j].x, l[j].y});
                }
            }
            __syncthreads();
        }
        if (live) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int i = 0; i < NIT; ++i) {
                    const uint32_t q = st0 ^ soff(i);
                    V16 x;
                    if constexpr (EP == 2) {
                        x = gld<V16>(s * lam0 + (q & ~1u) * ES);
                        if (q & 1) x = V16{x[2], x[3], x[0], x[1]};
                    } else {
                        x = gld<V16>(s * lam0 + q * ES);
                    }
                    __builtin_nontemporal_store(x, (V16*)(P[s] + g0 + goff(i)));
                }
        }
        __syncthreads();                                       // the tile has been read: the next may come in
    }
    if constexpr (REV) {
        for (uint32_t i = tid; i < A.nsum; i += blockDim.x) {
            double s = 0;
            for (uint32_t v = 0; v < nw; ++v) s += gld<double>(acc0 + 8 * (v * A.nsum + i));
            part[((size_t)(A.row0 + i) * nblk + blockIdx.x) * batch + b] = s;
        }
    }
}

// Gates of the runs, as the kernels below read them.
struct AdjGateDev {
    uint32_t gen;            // 1/2/3: RX/RY/RZ with angle theta[occ][b]; 0: the matrix m
    uint32_t occ;
    double m[8];
};
struct AdjRunDev {
    uint32_t first;          // its gates: [first, next run's first)
    uint32_t grow;           // (first row of its sums + 1) << 3 | the Paulis they are of, 0: none
};
static_assert(sizeof(AdjGateDev) == 72 && sizeof(AdjRunDev) == 8, "table layout");

__device__ __forceinline__ void gate_mat(const AdjGateDev& g, const double* __restrict__ theta, uint32_t batch,
                                         uint32_t b, double (&m)[8]) {
    if (!g.gen) {
        for (int i = 0; i < 8; ++i) m[i] = g.m[i];
        return;
    }
    double s, c;
    sincos(theta[(size_t)g.occ * batch + b] / 2, &s, &c);
    for (int i = 0; i < 8; ++i) m[i] = 0;
    if (g.gen == 3) {
        m[0] = c; m[1] = -s; m[6] = c; m[7] = s;
    } else {
        m[0] = c; m[6] = c;
        if (g.gen == 1) { m[3] = -s; m[5] = -s; }
        else { m[2] = -s; m[4] = s; }
    }
}

// c = a b for 2 x 2 complex matrices.
__device__ __forceinline__ void mul22(const double (&a)[8], const double (&b)[8], double (&c)[8]) {
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            double re = 0, im = 0;
            for (int k = 0; k < 2; ++k) {
                const double ar = a[4 * i + 2 * k], ai = a[4 * i + 2 * k + 1];
                const double br = b[4 * k + 2 * j], bi = b[4 * k + 2 * j + 1];
                re += ar * br - ai * bi;
                im += ar * bi + ai * br;
            }
            c[4 * i + 2 * j] = re;
            c[4 * i + 2 * j + 1] = im;
        }
}

// The matrices of the runs for every batch element (double precision, then
// rounded to R): on the device, as the host took longer over 944 x 64
// angles than the sweeps do.
template <typename R>
__global__ __launch_bounds__(256) void k_adj_mats(const AdjRunDev* __restrict__ runs, uint32_t nruns,
                                                  const AdjGateDev* __restrict__ gates,
                                                  const double* __restrict__ theta, uint32_t batch,
                                                  R* __restrict__ mats) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (uint64_t)nruns * batch) return;
    const uint32_t r = (uint32_t)(i / batch), b = (uint32_t)(i % batch);
    double u[8], m[8], t[8];
    gate_mat(gates[runs[r].first], theta, batch, b, u);
    for (uint32_t g = runs[r].first + 1; g < runs[r + 1].first; ++g) {
        gate_mat(gates[g], theta, batch, b, m);
        mul22(m, u, t);
        for (int k = 0; k < 8; ++k) u[k] = t[k];
    }
    for (int k = 0; k < 8; ++k) mats[i * 8 + k] = (R)u[k];
}

// The gradients of a run's gates from its three sums: last gate first, with
// rot the rotation of the gates after it (column G: V G V^dagger in X, Y, Z).
__global__ __launch_bounds__(256) void k_adj_grads(const AdjRunDev* __restrict__ runs, uint32_t nruns,
                                                   const AdjGateDev* __restrict__ gates,
                                                   const double* __restrict__ theta, uint32_t batch, uint32_t nblk,
                                                   const double* __restrict__ part, double* __restrict__ out) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (uint64_t)nruns * batch) return;
    const uint32_t r = (uint32_t)(i / batch), b = (uint32_t)(i % batch);
    if (!runs[r].grow) return;
    uint32_t row = (runs[r].grow >> 3) - 1;
    double S[3] = {0, 0, 0};
    for (int v = 0; v < 3; ++v) {
        if (!((runs[r].grow >> v) & 1)) continue;
        double s = 0;
        for (uint32_t k = 0; k < nblk; ++k) s += part[((size_t)row * nblk + k) * batch + b];
        S[v] = s;
        ++row;
    }
    double rot[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
    for (uint32_t g = runs[r + 1].first; g-- > runs[r].first;) {
        const AdjGateDev& G = gates[g];
        if (G.gen) {
            const int c = (int)G.gen - 1;
            out[(size_t)G.occ * batch + b] = rot[c] * S[0] + rot[3 + c] * S[1] + rot[6 + c] * S[2];
        }
        if (g == runs[r].first) break;
        double u[8];
        gate_mat(G, theta, batch, b, u);
        // the gate's rotation: column Q from M = U Q U^dagger = x X + y Y + z Z
        double q[9];
        for (int c = 0; c < 3; ++c) {
            double t[8], ud[8], m[8];
            const double Q[3][8] = {{0, 0, 1, 0, 1, 0, 0, 0}, {0, 0, 0, -1, 0, 1, 0, 0}, {1, 0, 0, 0, 0, 0, -1, 0}};
            ud[0] = u[0]; ud[1] = -u[1]; ud[2] = u[4]; ud[3] = -u[5];
            ud[4] = u[2]; ud[5] = -u[3]; ud[6] = u[6]; ud[7] = -u[7];
            double qq[8];
            for (int k = 0; k < 8; ++k) qq[k] = Q[c][k];
            mul22(u, qq, t);
            mul22(t, ud, m);
            q[c] = m[2];
            q[3 + c] = -m[3];
            q[6 + c] = 0.5 * (m[0] - m[6]);
        }
        double n[9];
        for (int x = 0; x < 3; ++x)
            for (int y = 0; y < 3; ++y) n[3 * x + y] = rot[3 * x] * q[y] + rot[3 * x + 1] * q[3 + y] + rot[3 * x + 2] * q[6 + y];
        for (int k = 0; k < 9; ++k) rot[k] = n[k];
    }
}

// |0..0> in every batch element.
template <typename R>
__global__ __launch_bounds__(256) void k_bzero(typename AC2<R>::T* __restrict__ psi, uint64_t total,
                                               uint64_t state_len) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        typename AC2<R>::T v;
        v.x = (i % state_len) == 0 ? (R)1 : (R)0;
        v.y = 0;
        psi[i] = v;
    }
}

struct PauliTerms {
    int nt;
    uint64_t x[48], z[48];
    double c[48];
};

// lam = sum_t c_t P_t psi, with (P psi)_i = i^{|x&z|} (-1)^{|z&(i^x)|} psi_{i^x}.
template <typename R>
__global__ __launch_bounds__(256) void k_bpauli(const typename AC2<R>::T* __restrict__ psi,
                                                typename AC2<R>::T* __restrict__ lam,
                                                uint64_t state_len, PauliTerms T, int accumulate) {
    const int b = blockIdx.y;
    const auto* P = psi + (size_t)b * state_len;
    auto* Lm = lam + (size_t)b * state_len;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < state_len; i += stride) {
        R sr = 0, si = 0;
        if (accumulate) {
            sr = Lm[i].x;
            si = Lm[i].y;
        }
        for (int t = 0; t < T.nt; ++t) {
            const uint64_t j = i ^ T.x[t];
            const auto v = P[j];
            R vr = v.x, vi = v.y;
            if (__popcll(T.z[t] & j) & 1) { vr = -vr; vi = -vi; }
            R wr = vr, wi = vi;
            switch (__popcll(T.x[t] & T.z[t]) & 3) {
                case 1: wr = -vi; wi = vr; break;
                case 2: wr = -vr; wi = -vi; break;
                case 3: wr = vi; wi = -vr; break;
                default: break;
            }
            sr += (R)T.c[t] * wr;
            si += (R)T.c[t] * wi;
        }
        typename AC2<R>::T o;
        o.x = sr;
        o.y = si;
        Lm[i] = o;
    }
}

// part[b][blk] = partial Re <psi|lam> of batch element b.
template <typename R>
__global__ __launch_bounds__(256) void k_bdot(const typename AC2<R>::T* __restrict__ psi,
                                              const typename AC2<R>::T* __restrict__ lam,
                                              uint64_t state_len, double* __restrict__ part) {
    __shared__ double sh[4];
    const int b = blockIdx.y;
    const auto* P = psi + (size_t)b * state_len;
    const auto* Lm = lam + (size_t)b * state_len;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    double s = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < state_len; i += stride)
        s += (double)P[i].x * (double)Lm[i].x + (double)P[i].y * (double)Lm[i].y;
    const double r = adj_block_sum(s, sh);
    if (threadIdx.x == 0) part[(size_t)b * kAdjBlocks + blockIdx.x] = r;
}

// out[r] = sum over kAdjBlocks partials of row r, in order.
__global__ __launch_bounds__(256) void k_rows(const double* __restrict__ part, uint64_t rows,
                                              double* __restrict__ out) {
    const uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    double s = 0;
    for (int k = 0; k < kAdjBlocks; ++k) s += part[r * kAdjBlocks + k];
    out[r] = s;
}

namespace {

struct AdjGate {
    int target;
    uint64_t cmask;
    int pidx;          // -1: fixed
    int gen;           // 1/2/3 for trainable X/Y/Z rotations
    bool named;        // fixed and not an explicit matrix: unitary
    std::vector<cd> u; // fixed gates: 2x2
};

struct AdjLayout {
    size_t mats_off, mats_bytes;     // the runs' 2x2 matrices, per batch element
    size_t aux_off, aux_bytes;       // angles, gate and run tables
    size_t part_off, part_bytes;     // reduction partials: kAdjBlocks per (trainable gate + 1, batch element)
    size_t res_off, res_bytes;       // reduced rows
    size_t need;                     // bytes the problem is charged (the static workspace holds 64 MiB of them)
    size_t tab_off, tab_bytes;       // op records of the passes
    size_t total;
};

constexpr size_t kAdjTab = 128 << 10;

AdjLayout adj_layout(int batch, size_t n_gates, size_t n_occ) {
    auto al = [](size_t v) { return (v + 255) & ~size_t(255); };
    AdjLayout L{};
    size_t off = 0;
    L.mats_off = off;
    L.mats_bytes = n_gates * (size_t)batch * 8 * sizeof(double);
    off += L.mats_bytes;
    L.aux_off = off;                 // (with the matrices: 2 x n_gates x batch x 64 bytes and 32 per gate)
    L.aux_bytes = al(2 * L.mats_bytes) - L.mats_bytes + al((n_gates + 1) * 32);
    off += L.aux_bytes;
    L.part_off = off;
    L.part_bytes = al((n_occ + 1) * (size_t)batch * kAdjBlocks * sizeof(double));
    off += L.part_bytes;
    L.res_off = off;
    L.res_bytes = al((n_occ + 1) * (size_t)batch * sizeof(double));
    off += L.res_bytes;
    L.need = off;
    L.tab_off = off;
    L.tab_bytes = kAdjTab;
    L.total = off + L.tab_bytes;
    return L;
}

qvm_status adj_fail(qvm_status st, const std::string& m) { return fail(st, "adjoint: " + m); }

// A step of the sweep: a run of uncontrolled gates on one qubit, or one gate.
struct AdjStep {
    std::vector<int> gates;          // in program order
    int target;
    uint64_t cmask;
    uint64_t xq, zq;                 // bits it does not / does act diagonally on
    uint32_t kind;                   // AD_MAT, AD_RE, AD_DG, AD_MOVE or AD_SIGN
    uint32_t need;                   // Paulis its gradients take (0: nothing trainable)
    int run;                         // row of the matrix table (AD_MAT, AD_RE, AD_DG)
    int row;                         // first row of its gradient sums, -1: none
    bool fence = false;              // not unitary: no other step passes it
    bool matrix() const { return kind != AD_MOVE && kind != AD_SIGN; }
};

// Unitary to the rounding of the states' type.  The sums of two gates that
// commute may be taken in either order because undoing a unitary leaves them
// as they are; undoing any other matrix, by its adjoint, changes them.
bool adj_unitary(const std::vector<cd>& u, qvm_dtype dt) {
    const double tol = dt == QVM_C64 ? 1e-6 : 1e-13;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const cd d = std::conj(u[a]) * u[b] + std::conj(u[2 + a]) * u[2 + b];
            if (!(std::abs(d - (a == b ? 1.0 : 0.0)) < tol)) return false;
        }
    return true;
}

// merge: consecutive uncontrolled gates on a qubit as one step (complex128).
std::vector<AdjStep> adj_steps(const std::vector<AdjGate>& G, bool merge, qvm_dtype dt) {
    std::vector<AdjStep> out;
    int open[QVM_MAX_QUBITS];
    std::fill(open, open + QVM_MAX_QUBITS, -1);
    const cd one(1.0, 0.0), zero(0.0, 0.0);
    for (size_t i = 0; i < G.size(); ++i) {
        const AdjGate& g = G[i];
        // an explicit matrix need not be unitary: the rotation of a run is
        // not defined for it, so it stands alone
        const bool joins = merge && g.cmask == 0 && (g.pidx >= 0 || g.named);
        if (joins && open[g.target] >= 0) {
            AdjStep& s = out[open[g.target]];
            s.gates.push_back((int)i);
            s.kind = AD_MAT;
            continue;
        }
        AdjStep s{{(int)i}, g.target, g.cmask, 1ull << g.target, g.cmask, AD_MAT, 0, -1, -1};
        s.fence = g.pidx < 0 && !g.named && !adj_unitary(g.u, dt);
        for (uint64_t m = s.fence ? ~0ull : g.cmask | s.xq; m; m &= m - 1)
            if (__builtin_ctzll(m) < QVM_MAX_QUBITS) open[__builtin_ctzll(m)] = -1;
        if (joins) open[g.target] = (int)out.size();
        if (g.pidx >= 0) {
            s.kind = g.gen == 1 ? AD_RX : g.gen == 2 ? AD_RE : AD_DG;
        } else {
            const bool diag = g.u[1] == zero && g.u[2] == zero, off = g.u[0] == zero && g.u[3] == zero;
            bool re = true;
            for (const cd& x : g.u) re = re && x.imag() == 0.0;
            if (!joins && diag && g.u[0] == one && g.u[3] == -one) {
                s.kind = AD_SIGN;
                s.zq |= s.xq;
                s.xq = 0;
            } else if (!joins && off && g.u[1] == one && g.u[2] == one) {
                s.kind = AD_MOVE;
            } else {
                s.kind = diag ? AD_DG : re ? AD_RE : AD_MAT;
            }
        }
        out.push_back(std::move(s));
    }
    for (AdjStep& s : out) {
        // a run whose only trainable gate is its last needs that gate's
        // generator alone
        size_t trainable = 0;
        for (int gi : s.gates) trainable += G[gi].pidx >= 0;
        if (!trainable) continue;
        s.need = trainable == 1 && G[s.gates.back()].pidx >= 0 ? 1u << (G[s.gates.back()].gen - 1) : 7u;
    }
    return out;
}

// One pass: its tile's bits and its rounds, each with its slot bits and its
// steps in order.
struct AdjPassPlan {
    uint64_t qmask;
    std::vector<std::vector<int>> rounds;
    std::vector<uint64_t> slots;
    std::vector<int> steps;          // complex128: the pass's steps, before they are put into rounds
};

// Slots left free: the highest tile bits.
uint64_t adj_fill(uint64_t sm, uint64_t qmask, int rs) {
    for (int b = 63; b >= 0 && pc(sm) < rs; --b)
        if ((qmask >> b) & 1) sm |= 1ull << b;
    return sm;
}

// Groups of at most r target qubits.  Each group scans the gates not yet
// placed, in program order, and takes a gate when none of its qubits is held
// by a gate the scan has passed over (so the order of gates that share a
// qubit is kept: gates that share no qubit commute) and its target is a slot
// or a slot is free.
struct AdjGroup {
    std::vector<int> steps;          // in program order
    uint64_t slots;                  // targets, and the highest other qubits if they are fewer than r
    int train;
};

std::vector<AdjGroup> adj_groups(const std::vector<AdjStep>& S, int n, int r) {
    std::vector<AdjGroup> out;
    std::vector<char> done(S.size(), 0);
    size_t left = S.size(), first = 0;
    while (left) {
        AdjGroup g{};
        uint64_t blocked = 0, t = 0;
        for (size_t i = first; i < S.size(); ++i) {
            if (done[i]) continue;
            const uint64_t tb = 1ull << S[i].target, q = tb | S[i].cmask;
            bool ok = !(q & blocked);
            if (ok && !(t & tb) && pc(t) == r) ok = false;
            if (ok && S[i].need && g.train == kAdjMaxTrain) ok = false;
            if (ok && (int)g.steps.size() == kAdjMaxOps) ok = false;
            if (!ok) {
                blocked |= q;
                continue;
            }
            t |= tb;
            g.steps.push_back((int)i);
            done[i] = 1;
            --left;
            g.train += S[i].need != 0;
        }
        while (first < S.size() && done[first]) ++first;
        g.slots = adj_fill(t, (1ull << n) - 1, r);
        out.push_back(std::move(g));
    }
    return out;
}

void adj_shift(AdjGroup& g, int by) {
    for (int& i : g.steps) i += by;
}
void adj_shift(AdjPassPlan& P, int by) {
    for (int& i : P.steps) i += by;
    for (auto& r : P.rounds)
        for (int& i : r) i += by;
}

// make (groups or passes of a list of steps) of each part between fences and
// of each fence, one after the other.
template <typename F>
auto adj_fenced(const std::vector<AdjStep>& S, F make) -> decltype(make(S)) {
    auto fence = [](const AdjStep& s) { return s.fence; };
    if (std::none_of(S.begin(), S.end(), fence)) return make(S);
    decltype(make(S)) out;
    for (auto a = S.begin(); a != S.end();) {
        const auto b = a->fence ? a + 1 : std::find_if(a, S.end(), fence);
        for (auto& x : make(std::vector<AdjStep>(a, b))) {
            adj_shift(x, (int)(a - S.begin()));
            out.push_back(std::move(x));
        }
        a = b;
    }
    return out;
}

// complex64: a group is a round, and consecutive groups share a pass while
// their slots and the low bits fit in the tile.
std::vector<AdjPassPlan> adj_passes_ordered(const std::vector<AdjGroup>& groups, int n, int L, int c) {
    std::vector<AdjPassPlan> out;
    size_t ops = 0, sums = 0;
    for (const AdjGroup& g : groups) {
        if (out.empty() || pc(out.back().qmask | g.slots) > L || ops + g.steps.size() > (size_t)kAdjMaxOps ||
            sums + g.train > (size_t)kAdjMaxSums) {
            out.push_back(AdjPassPlan{(1ull << std::min(c, n)) - 1, {}, {}, {}});
            ops = sums = 0;
        }
        out.back().qmask |= g.slots;
        out.back().rounds.push_back(g.steps);
        out.back().slots.push_back(g.slots);
        ops += g.steps.size();
        sums += g.train;
    }
    for (AdjPassPlan& P : out)
        for (int q = 0; q < n && pc(P.qmask) < std::min(L, n); ++q) P.qmask |= 1ull << q;
    return out;
}

// complex128: the passes of a gate list (gatepass.hip), gates in any order
// that keeps those of every shared qubit.
std::vector<AdjPassPlan> adj_passes_free(const std::vector<AdjStep>& S, int n, int L, int c) {
    std::vector<AdjPassPlan> out;
    std::vector<char> done(S.size(), 0);
    std::vector<int> ops;
    size_t left = S.size(), first = 0;
    while (left) {
        while (done[first]) ++first;
        const uint64_t qmask = take_pass(S, done, first, n, L, c, 0, ops);
        // the first of the list as far as the limits go (a prefix of a valid order)
        size_t keep = 0, sums = 0;
        for (; keep < ops.size() && keep < (size_t)kAdjMaxOps; ++keep) {
            const size_t k = pc(S[ops[keep]].need);
            if (sums + k > (size_t)kAdjMaxSums) break;
            sums += k;
        }
        ops.resize(keep);
        for (int i : ops) done[i] = 1;
        left -= ops.size();
        out.push_back(AdjPassPlan{qmask, {}, {}, ops});
    }
    return out;
}

// The rounds of a pass, forward or undone.
AdjPassPlan adj_rounds(const std::vector<AdjStep>& S, AdjPassPlan P, bool rev, int rs) {
    if (P.steps.empty()) {           // complex64 has them already
        if (rev) {
            std::reverse(P.rounds.begin(), P.rounds.end());
            std::reverse(P.slots.begin(), P.slots.end());
            for (auto& r : P.rounds) std::reverse(r.begin(), r.end());
        }
        return P;
    }
    std::vector<int> left = P.steps, next;
    if (rev) std::reverse(left.begin(), left.end());
    while (!left.empty()) {
        Sched sc;
        uint64_t sm = 0;
        std::vector<int> now;
        next.clear();
        for (int i : left) {
            if (sc.free(S[i]) && pc(sm | S[i].xq) <= rs) {
                sm |= S[i].xq;
                now.push_back(i);
            } else {
                sc.hold(S[i]);
                next.push_back(i);
            }
        }
        P.rounds.push_back(std::move(now));
        P.slots.push_back(adj_fill(sm, P.qmask, rs));
        left.swap(next);
    }
    return P;
}

std::vector<AdjPassPlan> adj_passes(const std::vector<AdjStep>& S, int n, qvm_dtype dt) {
    return adj_fenced(S, [&](const std::vector<AdjStep>& part) {
        if (dt == QVM_C64)
            return adj_passes_ordered(adj_groups(part, n, std::min(n, adj_slots<float>())), n, std::min(n, adj_width<float>()), GT<float>::C);
        return adj_passes_free(part, n, std::min(n, adj_width<double>()), GT<double>::C);
    });
}

// Records of one pass; row0: the first row of its sums.
void adj_records(const std::vector<AdjStep>& S, const AdjPassPlan& P, int rs, size_t elem, uint32_t row0,
                 std::vector<uint32_t>& tab) {
    auto put = [&](const void* p, size_t bytes) {
        const size_t at = tab.size();
        tab.resize(at + bytes / 4);
        memcpy(&tab[at], p, bytes);
    };
    for (size_t r = 0; r < P.rounds.size(); ++r) {
        const uint64_t sm = P.slots[r];
        AdjRound rh{};
        uint64_t phys[kAdjSlots] = {0, 0, 0, 0};
        int k = 0;
        for (uint64_t m = sm; m; m &= m - 1, ++k) {
            phys[k] = m & (~m + 1);
            rh.bit[k] = local_bits(phys[k], P.qmask);
            rh.lds[k] = tile_swizzle(rh.bit[k]) * (uint32_t)elem;
        }
        rh.nops = (uint32_t)P.rounds[r].size();
        put(&rh, sizeof(rh));
        for (int i : P.rounds[r]) {
            const AdjStep& s = S[i];
            AdjOp o{};
            const uint64_t tbit = 1ull << s.target;
            uint64_t cond = s.cmask;                        // bits that must be 1
            int slot = 0;
            for (int q = 0; q < rs; ++q)
                if (phys[q] == tbit) slot = q;
            o.code = s.kind;
            if (s.kind == AD_SIGN) cond |= tbit;
            else o.code += (uint32_t)slot;
            uint32_t cj = 0;
            for (int q = 0; q < rs; ++q)
                if (cond & phys[q]) cj |= 1u << q;
            for (uint32_t j = 0; j < 1u << rs; ++j)
                if ((j & cj) == cj && (s.kind == AD_SIGN || !(j & (1u << slot)))) o.jbits |= 1u << j;
            o.tm = o.tv = local_bits(cond & P.qmask & ~sm, P.qmask);
            o.om = o.ov = tile_index_bits(cond, P.qmask);
            o.mat = s.matrix() ? (uint32_t)s.run : 0;
            o.grad = s.need ? ((uint32_t)s.row - row0 + 1) << 3 | s.need : 0;
            put(&o, sizeof(o));
        }
    }
}

}  // namespace

template <typename R>
static qvm_status adjoint_t(int n, int batch, const std::vector<AdjGate>& G, int n_params,
                            const double* params, const PauliTerms* terms, int n_term_chunks,
                            void* psi_dev, void* lam_dev, char* work, const AdjLayout& L,
                            hipStream_t stream, bool want_grad, double* f_out, double* grad_out) {
    using T = typename AC2<R>::T;
    T* psi = (T*)psi_dev;
    T* lam = (T*)lam_dev;
    const uint64_t N = 1ull << n;
    qvm_sv dummy{};
    qvm_sv* sv = &dummy;      // for the error macros only
    std::vector<AdjStep> S = adj_steps(G, sizeof(R) == 8, sizeof(R) == 4 ? QVM_C64 : QVM_C128);
    const int rs = std::min(n, adj_slots<R>());
    const std::vector<AdjPassPlan> passes = adj_passes(S, n, sizeof(R) == 4 ? QVM_C64 : QVM_C128);
    // run and gradient rows in pass order; a pass's gradient rows are consecutive
    std::vector<AdjRunDev> runs;
    std::vector<AdjGateDev> gates;
    size_t nsum = 0;
    std::vector<int> occ_gate;                    // trainable occurrence -> gate
    auto steps_of = [](const AdjPassPlan& P) {
        std::vector<int> v = P.steps;
        for (const auto& r : P.rounds) v.insert(v.end(), r.begin(), r.end());
        return v;
    };
    for (const AdjPassPlan& P : passes)
        for (int i : steps_of(P)) {
            AdjStep& s = S[i];
            if (!s.matrix()) continue;
            s.run = (int)runs.size();
            AdjRunDev rd{(uint32_t)gates.size(), 0};
            if (s.need) {
                s.row = (int)nsum;
                rd.grow = ((uint32_t)s.row + 1) << 3 | s.need;
                nsum += pc(s.need);
            }
            runs.push_back(rd);
            for (int gi : s.gates) {
                AdjGateDev g{};
                if (G[gi].pidx >= 0) {
                    g.gen = (uint32_t)G[gi].gen;
                    g.occ = (uint32_t)occ_gate.size();
                    occ_gate.push_back(gi);
                } else {
                    for (int e = 0; e < 4; ++e) {
                        g.m[2 * e] = G[gi].u[e].real();
                        g.m[2 * e + 1] = G[gi].u[e].imag();
                    }
                }
                gates.push_back(g);
            }
        }
    const size_t nocc = occ_gate.size(), nrun = runs.size();
    runs.push_back(AdjRunDev{(uint32_t)gates.size(), 0});
    // one upload: angles per (occurrence, batch element), gates, runs
    const size_t o_gate = nocc * batch * sizeof(double), o_run = o_gate + gates.size() * sizeof(AdjGateDev);
    const size_t aux_used = o_run + runs.size() * sizeof(AdjRunDev);
    std::vector<char> aux(aux_used);
    for (size_t o = 0; o < nocc; ++o) {
        double* t = (double*)aux.data() + o * batch;
        const int p = G[occ_gate[o]].pidx;
        for (int b = 0; b < batch; ++b) t[b] = params[(size_t)b * n_params + p];
    }
    if (!gates.empty()) memcpy(aux.data() + o_gate, gates.data(), gates.size() * sizeof(AdjGateDev));
    memcpy(aux.data() + o_run, runs.data(), runs.size() * sizeof(AdjRunDev));
    char* daux = work + L.aux_off;
    if (aux_used > L.aux_bytes) return adj_fail(QVM_ENOMEM, "internal: gate tables exceed their share of the workspace");
    const double* dtheta = (const double*)daux;
    const AdjGateDev* dgates = (const AdjGateDev*)(daux + o_gate);
    const AdjRunDev* druns = (const AdjRunDev*)(daux + o_run);
    R* mats = (R*)(work + L.mats_off);
    double* part = (double*)(work + L.part_off);
    double* res = (double*)(work + L.res_off);
    uint32_t* dtab = (uint32_t*)(work + L.tab_off);
    QVM_HIP(sv, hipMemcpyAsync(daux, aux.data(), aux_used, hipMemcpyHostToDevice, stream));
    const unsigned rb = (unsigned)((nrun * (size_t)batch + 255) / 256);
    if (nrun) {
        hipLaunchKernelGGL((k_adj_mats<R>), dim3(rb), dim3(256), 0, stream, druns, (uint32_t)nrun, dgates, dtheta,
                           (uint32_t)batch, mats);
        QVM_LAUNCH_CHECK(sv);
    }
    // the passes' records, forward then undone, uploaded as far as they fit at once
    const size_t cap = L.tab_bytes / 4, pad = 32;
    struct Rec { size_t at; uint64_t qmask; uint32_t rounds, row0, nsum; };
    std::vector<std::vector<uint32_t>> tabs;      // alive until the stream is waited for
    std::vector<Rec> recs;
    const size_t total = (want_grad ? 2 : 1) * passes.size();
    auto prepare = [&](size_t from) -> qvm_status {
        std::vector<uint32_t> t, one;
        for (size_t q = recs.size(); q < total; ++q) {
            const bool rev = q >= passes.size();
            const AdjPassPlan P = adj_rounds(S, passes[rev ? total - 1 - q : q], rev, rs);
            Rec r{0, P.qmask, (uint32_t)P.rounds.size(), ~0u, 0};
            for (const auto& rd : P.rounds)
                for (int i : rd)
                    if (S[i].need) {
                        r.row0 = std::min(r.row0, (uint32_t)S[i].row);
                        r.nsum += (uint32_t)pc(S[i].need);
                    }
            one.clear();
            adj_records(S, P, rs, sizeof(T), r.row0, one);
            if (t.size() + one.size() + pad > cap) break;
            r.at = t.size();
            t.insert(t.end(), one.begin(), one.end());
            recs.push_back(r);
        }
        if (recs.size() == from) return adj_fail(QVM_ENOMEM, "internal: a pass's records exceed their space");
        t.resize(t.size() + pad);
        tabs.push_back(std::move(t));
        QVM_HIP(sv, hipMemcpyAsync(dtab, tabs.back().data(), tabs.back().size() * 4, hipMemcpyHostToDevice, stream));
        return QVM_OK;
    };
    // the tiles of both states and the sums may take more than 64 KiB of LDS
    auto lds_limit = [&](const void* fn) -> qvm_status {
        static std::atomic<bool> set[64];
        int dev = 0;
        QVM_HIP(sv, hipGetDevice(&dev));
        if (dev < 0 || dev >= 64) return adj_fail(QVM_EUNSUPPORTED, "device index above 63");
        if (!set[dev].load()) {
            QVM_HIP(sv, hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLdsMax));
            set[dev].store(true);
        }
        return QVM_OK;
    };
    const dim3 blk(256);
    double* gpart = part + (size_t)batch * kAdjBlocks;           // (the f partials first)
    uint32_t nblk = 1;
    auto launch_pass = [&](size_t q) -> qvm_status {
        if (q >= recs.size()) {
            qvm_status st = prepare(q);
            if (st) return st;
        }
        const bool rev = q >= passes.size();
        const uint64_t qmask = recs[q].qmask;
        AdjPass A{};
        A.qmask = qmask;
        A.state_len = N;
        A.L = (uint32_t)pc(qmask);
        A.nrounds = recs[q].rounds;
        A.words = (uint32_t)recs[q].at;
        A.ntiles = (uint32_t)(N >> A.L);
        A.nsum = rev ? recs[q].nsum : 0;
        A.row0 = recs[q].row0;
        A.init = q == 0;
        int k = kAdjSlots;
        for (int b = n - 1; b >= 0 && k > 0; --b)
            if ((qmask >> b) & 1) A.top[--k] = (uint32_t)b;
        const unsigned threads = std::max(64u, 1u << (A.L - rs));
        const size_t lds = (sizeof(T) << A.L) * (rev ? 2 : 1) + (size_t)A.nsum * (threads / 64) * sizeof(double);
        const dim3 grid(rev ? std::min(nblk, A.ntiles) : A.ntiles, (unsigned)batch);
#define QVM_ADJ_LAUNCH(RR, REV)                                                                            \
    {                                                                                                      \
        hipLaunchKernelGGL((k_adj_pass<R, RR, REV>), grid, dim3(threads), lds, stream, psi, lam, A, dtab,  \
                           mats, (uint32_t)batch, nblk, gpart);                                            \
    }
        if (rev && rs == adj_slots<R>()) {       // (fewer slots: tiny states)
            const qvm_status st = lds_limit((const void*)k_adj_pass<R, adj_slots<R>(), true>);
            if (st) return st;
        }
#define QVM_ADJ_CASE(RR)                                  \
    case RR:                                              \
        if constexpr (RR <= adj_slots<R>()) {             \
            if (rev) QVM_ADJ_LAUNCH(RR, true) else QVM_ADJ_LAUNCH(RR, false) \
        }                                                 \
        break;
        switch (rs) { QVM_ADJ_CASE(1) QVM_ADJ_CASE(2) QVM_ADJ_CASE(3) QVM_ADJ_CASE(4) }
#undef QVM_ADJ_CASE
#undef QVM_ADJ_LAUNCH
        QVM_LAUNCH_CHECK(sv);
        return QVM_OK;
    };
    // forward
    if (passes.empty()) {
        hipLaunchKernelGGL((k_bzero<R>), dim3(1024), blk, 0, stream, psi, N * (uint64_t)batch, N);
        QVM_LAUNCH_CHECK(sv);
    }
    for (size_t q = 0; q < passes.size(); ++q) {
        qvm_status st = launch_pass(q);
        if (st) return st;
    }
    // lambda = H psi, f = Re <psi|lambda>
    for (int ch = 0; ch < n_term_chunks; ++ch) {
        hipLaunchKernelGGL((k_bpauli<R>), dim3((unsigned)std::min<uint64_t>((N + 255) / 256, 4096), batch),
                           blk, 0, stream, psi, lam, N, terms[ch], ch > 0 ? 1 : 0);
        QVM_LAUNCH_CHECK(sv);
    }
    hipLaunchKernelGGL((k_bdot<R>), dim3(kAdjBlocks, batch), blk, 0, stream, psi, lam, N, part);
    QVM_LAUNCH_CHECK(sv);
    hipLaunchKernelGGL(k_rows, dim3((batch + 255) / 256), blk, 0, stream, part, (uint64_t)batch, res);
    QVM_LAUNCH_CHECK(sv);
    if (!want_grad) {
        QVM_HIP(sv, hipMemcpyAsync(f_out, res, batch * sizeof(double), hipMemcpyDeviceToHost, stream));
        QVM_HIP(sv, hipStreamSynchronize(stream));
        return QVM_OK;
    }
    // reverse sweep; blocks per element: as many partials as there is room for
    if (nsum) {
        const size_t room = std::min<size_t>(kAdjBlocks, nocc * kAdjBlocks / nsum);
        while (2 * nblk <= room) nblk *= 2;
        // (fewer than nblk tiles: every block still has its partial)
        nblk = (uint32_t)std::min<uint64_t>(nblk, std::max<uint64_t>(1, N >> std::min(n, adj_width<R>())));
    }
    for (size_t q = passes.size(); q < total; ++q) {
        qvm_status st = launch_pass(q);
        if (st) return st;
    }
    if (nsum) {
        hipLaunchKernelGGL(k_adj_grads, dim3(rb), blk, 0, stream, druns, (uint32_t)nrun, dgates, dtheta,
                           (uint32_t)batch, nblk, gpart, res + batch);
        QVM_LAUNCH_CHECK(sv);
    }
    std::vector<double> rv((nocc + 1) * (size_t)batch);
    QVM_HIP(sv, hipMemcpyAsync(rv.data(), res, rv.size() * sizeof(double), hipMemcpyDeviceToHost, stream));
    QVM_HIP(sv, hipStreamSynchronize(stream));
    std::copy(rv.begin(), rv.begin() + batch, f_out);
    std::fill(grad_out, grad_out + (size_t)batch * n_params, 0.0);
    for (size_t o = 0; o < nocc; ++o)
        for (int b = 0; b < batch; ++b)
            grad_out[(size_t)b * n_params + G[occ_gate[o]].pidx] += rv[(o + 1) * batch + b];
    return QVM_OK;
}

static qvm_status adj_prepare(int n, int batch, const qvm_gate* gates, size_t n_gates,
                              const int32_t* param_index, int n_params, size_t n_terms,
                              const uint64_t* x, const uint64_t* z, const double* c,
                              std::vector<AdjGate>& G, std::vector<PauliTerms>& terms) {
    if (n < 1 || n > QVM_MAX_QUBITS) return adj_fail(QVM_EARG, "n_qubits outside 1..34");
    if (batch < 1 || batch > 65535) return adj_fail(QVM_EARG, "batch outside 1..65535");
    if (n_gates && (!gates || !param_index)) return adj_fail(QVM_EARG, "NULL gate list");
    if (n_params < 0) return adj_fail(QVM_EARG, "negative n_params");
    if (n_terms < 1 || !x || !z || !c) return adj_fail(QVM_EARG, "empty or NULL observable");
    const uint64_t lim = (n >= 64) ? ~0ull : ((1ull << n) - 1);
    for (size_t t = 0; t < n_terms; ++t)
        if ((x[t] & ~lim) || (z[t] & ~lim)) return adj_fail(QVM_ERANGE, "Pauli mask names a qubit >= n");
    G.clear();
    for (size_t i = 0; i < n_gates; ++i) {
        qvm_status st = validate_gate(gates[i], n, true);
        if (st) return fail(st, "adjoint gate " + std::to_string(i) + ": " + qvm_last_error());
        if (gates[i].k != 1) return adj_fail(QVM_EUNSUPPORTED, "gate " + std::to_string(i) + " has k != 1");
        AdjGate a{};
        a.target = gates[i].targets[0];
        a.cmask = gates[i].ctrl_mask;
        a.pidx = param_index[i];
        if (a.pidx >= n_params) return adj_fail(QVM_ERANGE, "parameter index >= n_params");
        if (a.pidx >= 0) {
            switch (gates[i].kind) {
                case QVM_G_RX: a.gen = 1; break;
                case QVM_G_RY: a.gen = 2; break;
                case QVM_G_RZ: a.gen = 3; break;
                default: return adj_fail(QVM_EARG, "trainable gate " + std::to_string(i) + " is not RX/RY/RZ");
            }
        } else {
            a.pidx = -1;
            a.named = gates[i].kind != QVM_G_MATRIX;
            st = gate_matrix(gates[i], a.u);
            if (st) return st;
        }
        G.push_back(std::move(a));
    }
    terms.clear();
    for (size_t t0 = 0; t0 < n_terms; t0 += 48) {
        PauliTerms T{};
        T.nt = (int)std::min<size_t>(48, n_terms - t0);
        for (int t = 0; t < T.nt; ++t) {
            T.x[t] = x[t0 + t];
            T.z[t] = z[t0 + t];
            T.c[t] = c[t0 + t];
        }
        terms.push_back(T);
    }
    return QVM_OK;
}

// Trainable gates: the gradient rows the sweep fills (plus row 0, f).
size_t adj_trainable(const std::vector<AdjGate>& G) {
    size_t t = 0;
    for (const AdjGate& g : G) t += g.pidx >= 0;
    return t;
}

qvm_status adj_dispatch(int n, qvm_dtype dt, int batch, const std::vector<AdjGate>& G, int n_params,
                        const double* params_host, const std::vector<PauliTerms>& terms, void* psi_dev,
                        void* lam_dev, char* work, const AdjLayout& L, void* hip_stream, double* f_out,
                        double* grad_out);

// Workspace of qvm_adjoint_expect_grad_static: one array per device, held
// until the process ends.  Host code never passes the array's name to a
// kernel or a copy (on the host it is only a stand-in for the symbol): its
// device address is looked up once per device, with that device current,
// and kept below.  Every entry a call reads is written earlier in the same
// call (matrices and op table copied in, each reduction partial stored by
// its block), so nothing needs clearing between calls.
static __device__ __align__(256) char scratch[QVM_ADJ_SCRATCH_BYTES + kAdjTab];

constexpr int kMaxDevices = 64;
static char* g_scratch_dev[kMaxDevices] = {};
static std::mutex g_scratch_mu;

qvm_status adj_scratch(char** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(QVM_EDEVICE, std::string("adjoint: hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return adj_fail(QVM_EUNSUPPORTED, "device index above 63");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(QVM_EDEVICE, std::string("adjoint: hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_dev[dev] = (char*)p;
    }
    *out = g_scratch_dev[dev];
    return QVM_OK;
}

}  // namespace qvm

using namespace qvm;

extern "C" {

qvm_status qvm_adjoint_group_count(int n, qvm_dtype dt, const qvm_gate* gates, size_t n_gates,
                                   const int32_t* param_index, int n_params, int32_t* n_groups) {
    if (dt != QVM_C64 && dt != QVM_C128) return adj_fail(QVM_EARG, "unknown dtype");
    if (!n_groups) return adj_fail(QVM_EARG, "NULL output");
    std::vector<AdjGate> G;
    std::vector<PauliTerms> terms;
    const uint64_t z = 0;
    const double c = 0;
    qvm_status st = adj_prepare(n, 1, gates, n_gates, param_index, n_params, 1, &z, &z, &c, G, terms);
    if (st) return st;
    const int r = std::min(n, dt == QVM_C64 ? adj_slots<float>() : adj_slots<double>());
    *n_groups = (int32_t)adj_fenced(adj_steps(G, false, dt), [&](const std::vector<AdjStep>& part) {
                    return adj_groups(part, n, r);
                }).size();
    return QVM_OK;
}

qvm_status qvm_adjoint_pass_count(int n, qvm_dtype dt, const qvm_gate* gates, size_t n_gates,
                                  const int32_t* param_index, int n_params, int32_t* n_passes) {
    if (dt != QVM_C64 && dt != QVM_C128) return adj_fail(QVM_EARG, "unknown dtype");
    if (!n_passes) return adj_fail(QVM_EARG, "NULL output");
    std::vector<AdjGate> G;
    std::vector<PauliTerms> terms;
    const uint64_t z = 0;
    const double c = 0;
    qvm_status st = adj_prepare(n, 1, gates, n_gates, param_index, n_params, 1, &z, &z, &c, G, terms);
    if (st) return st;
    *n_passes = (int32_t)adj_passes(adj_steps(G, dt == QVM_C128, dt), n, dt).size();
    return QVM_OK;
}

size_t qvm_adjoint_workspace_bytes(int n_qubits, int batch, size_t n_gates) {
    (void)n_qubits;
    return adj_layout(batch, n_gates, n_gates).total;
}

qvm_status qvm_adjoint_expect_grad(int n, qvm_dtype dt, int batch, const qvm_gate* gates,
                                   size_t n_gates, const int32_t* param_index, int n_params,
                                   const double* params_host, size_t n_terms, const uint64_t* x_mask,
                                   const uint64_t* z_mask, const double* coeff, void* psi_dev,
                                   void* lam_dev, void* work_dev, size_t work_bytes, void* hip_stream,
                                   double* f_out, double* grad_out) {
    if (dt != QVM_C64 && dt != QVM_C128) return adj_fail(QVM_EARG, "unknown dtype");
    if (!psi_dev || !lam_dev || !work_dev || !f_out) return adj_fail(QVM_EARG, "NULL buffer");
    if (n_params > 0 && !params_host) return adj_fail(QVM_EARG, "NULL parameters");
    if (psi_dev == lam_dev) return adj_fail(QVM_EARG, "psi and lambda must not alias");
    std::vector<AdjGate> G;
    std::vector<PauliTerms> terms;
    qvm_status st = adj_prepare(n, batch, gates, n_gates, param_index, n_params, n_terms, x_mask,
                                z_mask, coeff, G, terms);
    if (st) return st;
    const AdjLayout L = adj_layout(batch, G.size(), adj_trainable(G));
    if (work_bytes < L.total) return adj_fail(QVM_ENOMEM, "workspace too small");
    return adj_dispatch(n, dt, batch, G, n_params, params_host, terms, psi_dev, lam_dev, (char*)work_dev, L,
                        hip_stream, f_out, grad_out);
}

qvm_status qvm_adjoint_expect_grad_static(int n, qvm_dtype dt, int batch, const qvm_gate* gates,
                                          size_t n_gates, const int32_t* param_index, int n_params,
                                          const double* params_host, size_t n_terms,
                                          const uint64_t* x_mask, const uint64_t* z_mask,
                                          const double* coeff, void* psi_dev, void* lam_dev,
                                          void* hip_stream, double* f_out, double* grad_out) {
    if (dt != QVM_C64 && dt != QVM_C128) return adj_fail(QVM_EARG, "unknown dtype");
    if (!psi_dev || !lam_dev || !f_out) return adj_fail(QVM_EARG, "NULL buffer");
    if (n_params > 0 && !params_host) return adj_fail(QVM_EARG, "NULL parameters");
    if (psi_dev == lam_dev) return adj_fail(QVM_EARG, "psi and lambda must not alias");
    std::vector<AdjGate> G;
    std::vector<PauliTerms> terms;
    qvm_status st = adj_prepare(n, batch, gates, n_gates, param_index, n_params, n_terms, x_mask,
                                z_mask, coeff, G, terms);
    if (st) return st;
    const AdjLayout L = adj_layout(batch, G.size(), adj_trainable(G));
    if (L.need > QVM_ADJ_SCRATCH_BYTES)
        return adj_fail(QVM_ENOMEM, "needs " + std::to_string(L.need) + " bytes of workspace, the static "
                        "scratch holds " + std::to_string((size_t)QVM_ADJ_SCRATCH_BYTES));
    char* work = nullptr;
    st = adj_scratch(&work);
    if (st) return st;
    return adj_dispatch(n, dt, batch, G, n_params, params_host, terms, psi_dev, lam_dev, work, L, hip_stream,
                        f_out, grad_out);
}

}  // extern "C"

namespace qvm {

qvm_status adj_dispatch(int n, qvm_dtype dt, int batch, const std::vector<AdjGate>& G, int n_params,
                        const double* params_host, const std::vector<PauliTerms>& terms, void* psi_dev,
                        void* lam_dev, char* work, const AdjLayout& L, void* hip_stream, double* f_out,
                        double* grad_out) {
    const bool want = grad_out != nullptr;
    if (dt == QVM_C64)
        return adjoint_t<float>(n, batch, G, n_params, params_host, terms.data(), (int)terms.size(),
                                psi_dev, lam_dev, work, L, (hipStream_t)hip_stream, want, f_out, grad_out);
    return adjoint_t<double>(n, batch, G, n_params, params_host, terms.data(), (int)terms.size(),
                             psi_dev, lam_dev, work, L, (hipStream_t)hip_stream, want, f_out, grad_out);
}

}  // namespace qvm
