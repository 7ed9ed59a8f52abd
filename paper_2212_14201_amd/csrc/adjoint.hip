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
// complex64: gate by gate, in the order of the groups below, as merged or
// reordered gates would round the states (and so the gradients) otherwise.
// The forward sweep puts the groups into passes, the reverse sweep launches
// one kernel per group (k_adj_group).
//
// Before, both sweeps in both types launched a kernel per group, and the host
// computed every matrix.  20 qubits, complex64, 944 gates (640 trainable),
// batch 64: forward 92 groups in 23.6 ms, now 41 passes in 14.5; reverse 58.4
// ms, now 55.6; a call 86.4 ms, now 72.7.  11 qubits, complex128, batch
// 8, a state one tile: a call 568 us, now 282 (the two sweeps 55 and 120 us on
// 8 blocks: a chain of rounds, bound by latency).
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
enum : uint32_t { AD_MAT = 0, AD_RE = 4, AD_DG = 8, AD_MOVE = 12, AD_SIGN = 16 };
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

// S_X, S_Y, S_Z of one pair (the qubit's 0 and 1 amplitudes), added to g.
template <typename T>
__device__ __forceinline__ void pauli_terms(double (&g)[3], uint32_t need, const T& a0, const T& a1, const T& l0,
                                            const T& l1) {
    const double p0r = a0.x, p0i = a0.y, p1r = a1.x, p1i = a1.y;
    const double q0r = l0.x, q0i = l0.y, q1r = l1.x, q1i = l1.y;
    if (need & 1) g[0] += (q0r * p1i - q0i * p1r) + (q1r * p0i - q1i * p0r);    // X: (p1, p0)
    if (need & 2) g[1] += (q1r * p0r + q1i * p0i) - (q0r * p1r + q0i * p1i);    // Y: (-i p1, i p0)
    if (need & 4) g[2] += (q0r * p0i - q0i * p0r) - (q1r * p1i - q1i * p1r);    // Z: (p0, -p1)
}

template <int S, int NA, typename T>
__device__ __forceinline__ void adj_grad(double (&g)[3], uint32_t need, const T (&a)[NA], const T (&l)[NA],
                                         uint32_t jbits) {
#pragma unroll
    for (int j = 0; j < NA; ++j)
        if (!(j & (1 << S)) && ((jbits >> j) & 1)) pauli_terms(g, need, a[j], a[j | (1 << S)], l[j], l[j | (1 << S)]);
}

// The wave's sums of three values: X in lanes 0-15, Y in 16-31, Z in 32-47
// (seven exchanges where three separate sums take eighteen).
__device__ __forceinline__ double wave_sum3(const double (&g)[3], uint32_t lane) {
    const bool hi = (lane & 32) != 0, up = (lane & 16) != 0;
    double a0 = hi ? g[2] : g[0], a1 = hi ? 0.0 : g[1];
    a0 += __shfl_xor(hi ? g[0] : g[2], 32, 64);
    a1 += __shfl_xor(hi ? g[1] : 0.0, 32, 64);
    double b = up ? a1 : a0;
    b += __shfl_xor(up ? a0 : a1, 16, 64);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) b += __shfl_xor(b, o, 64);
    return b;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// A step's gradient sums on slot S, added to the wave's in LDS at `at`.
template <int S, int NA, typename T>
__device__ __forceinline__ void adj_sums(const T (&a)[NA], const T (&l)[NA], uint32_t need, uint32_t jb, bool act,
                                         uint32_t at, uint32_t lane) {
    double g[3] = {0, 0, 0};
    if (need == 7) {
        if (act) adj_grad<S, NA>(g, 7, a, l, jb);
        const double s = wave_sum3(g, lane);
        if ((lane & 15) == 0 && lane < 48) gst<double>(at + lane / 2, gld<double>(at + lane / 2) + s);
        return;
    }
    if (act) {
        if (need == 1) adj_grad<S, NA>(g, 1, a, l, jb);
        else if (need == 2) adj_grad<S, NA>(g, 2, a, l, jb);
        else adj_grad<S, NA>(g, 4, a, l, jb);
    }
    const double s = wave_sum(g[0] + g[1] + g[2]);             // (two of them are 0)
    if (lane == 0) gst<double>(at, gld<double>(at) + s);
}

// One product rounded, the other fused.
__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }

// A step on slot S of one state's registers.  The forms without the zero
// entries round as the full product does (which rounds its first or, where
// it subtracts, its second product and fuses the others in order).
template <typename R, int S, int NA, typename T>
__device__ __forceinline__ void adj_apply(T (&a)[NA], const R* u, uint32_t kind, uint32_t jb) {
    constexpr uint32_t ALL = (S == 0 ? 0x5555u : S == 1 ? 0x3333u : S == 2 ? 0x0f0fu : 0x00ffu) & ((1u << NA) - 1u);
    if (kind == AD_MAT) {
        op_d1<R, S>(a, u, jb);
    } else if (kind == AD_MOVE) {
        op_move<(1 << S)>(a, jb);
    } else {
        auto re = [&](int j) {
            T &v0 = a[j], &v1 = a[j | (1 << S)];
            T o0, o1;
            o0.x = mad(u[2], v1.x, u[0] * v0.x);
            o0.y = mad(u[2], v1.y, u[0] * v0.y);
            o1.x = mad(u[6], v1.x, u[4] * v0.x);
            o1.y = mad(u[6], v1.y, u[4] * v0.y);
            v0 = o0;
            v1 = o1;
        };
        auto dg = [&](int j) {
            T &v0 = a[j], &v1 = a[j | (1 << S)];
            T o0, o1;
            o0.x = mad(u[0], v0.x, -(u[1] * v0.y));
            o0.y = mad(u[1], v0.x, u[0] * v0.y);
            o1.x = mad(-u[7], v1.y, u[6] * v1.x);
            o1.y = mad(u[7], v1.x, u[6] * v1.y);
            v0 = o0;
            v1 = o1;
        };
        if (kind == AD_RE) {
            if (jb == ALL) {
#pragma unroll
                for (int j = 0; j < NA; ++j)
                    if (!(j & (1 << S))) re(j);
            } else {
#pragma unroll
                for (int j = 0; j < NA; ++j)
                    if (!(j & (1 << S)) && ((jb >> j) & 1)) re(j);
            }
        } else {
            if (jb == ALL) {
#pragma unroll
                for (int j = 0; j < NA; ++j)
                    if (!(j & (1 << S))) dg(j);
            } else {
#pragma unroll
                for (int j = 0; j < NA; ++j)
                    if (!(j & (1 << S)) && ((jb >> j) & 1)) dg(j);
            }
        }
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
    typedef uint32_t U8 __attribute__((ext_vector_type(8), aligned(4)));
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
        const uint32_t* __restrict__ p = table + A.words;
        for (uint32_t r = 0; r < A.nrounds; ++r) {
            const U8 hd = *(const U8*)p;
            const uint32_t nops = p[8];
            p += sizeof(AdjRound) / 4;
            // the head one record ahead, the matrix of the record at hand
            // while the head after it is on its way
            U8 h = *(const U8*)p;
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
                const R* __restrict__ q = mats + ((size_t)idx * batch + b) * 8;
#pragma unroll
                for (int i = 0; i < 8; ++i) m[i] = q[i];
            };
            matrix(h[6]);
            for (uint32_t oi = 0; oi < nops; ++oi) {
                const U8 cur = h;
                R u[8];
                if constexpr (REV) {                           // the adjoint
                    u[0] = m[0]; u[1] = -m[1]; u[2] = m[4]; u[3] = -m[5];
                    u[4] = m[2]; u[5] = -m[3]; u[6] = m[6]; u[7] = -m[7];
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) u[i] = m[i];
                }
                p += sizeof(AdjOp) / 4;
                h = *(const U8*)p;                             // (after the last record: in bounds, not used)
                if ((w & cur[4]) == cur[5]) {
                    const bool act = live && (le & cur[2]) == cur[3];
                    const uint32_t jb = cur[1], kind = cur[0] & ~3u, slot = cur[0] & 3u, need = cur[7] & 7u;
                    const uint32_t at = acc0 + 8 * (wave * A.nsum + (cur[7] >> 3) - 1);
                    if (kind == AD_SIGN) {
                        if (act) {
#pragma unroll
                            for (int j = 0; j < NA; ++j) {
                                const uint32_t f = (jb << (31 - j)) & 0x80000000u;
                                a[j].x = flip_sign(a[j].x, f);
                                a[j].y = flip_sign(a[j].y, f);
                                if constexpr (REV) {
                                    l[j].x = flip_sign(l[j].x, f);
                                    l[j].y = flip_sign(l[j].y, f);
                                }
                            }
                        }
                    }
#define QVM_ADJ_SLOT(SL)                                                                      \
    else if (RS == SL + 1 || slot == SL) {                                                    \
        constexpr int S = SL < RS ? SL : 0;                                                   \
        if constexpr (REV)                                                                    \
            if (need) adj_sums<S, NA>(a, l, need, jb, act, at, lane);                         \
        if (act) {                                                                            \
            adj_apply<R, S, NA>(a, u, kind, jb);                                              \
            if constexpr (REV) adj_apply<R, S, NA>(l, u, kind, jb);                           \
        }                                                                                     \
    }
                    QVM_ADJ_SLOT(0) QVM_ADJ_SLOT(1) QVM_ADJ_SLOT(2) QVM_ADJ_SLOT(3)
#undef QVM_ADJ_SLOT
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

// The reverse sweep in complex64: one launch per group.  A thread owns one
// item, the 16 amplitudes of psi and of lambda that differ only in the
// group's slot bits (at most four target qubits; controls may sit on any
// qubit), held in registers for the whole group: one read and one write of
// each state.  Controls on slot bits are tests of the register index, others
// one test of the item's base index.  Bound by arithmetic (the gradient terms
// in double precision): at 20 qubits, batch 64 a group of ten gates takes 605
// us for 2 GiB read and written, which alone take 335.  635 us before the
// wave's sum left LDS and records were read ahead.  Tiles of both states in
// LDS (k_adj_pass) took 600, and shorter forms for matrices with zeros 585,
// but what the compiler contracts into fused multiply-adds differs from one
// pair of registers to the next here, so other code rounds lambda otherwise
// (gradients off by 1e-7 of their size): the products stay as they are.
struct AdjOpDev {
    uint64_t cout;     // control bits outside the slots
    int32_t slot;      // target slot
    int32_t cj;        // control bits among the slots, as a mask over slots
    int32_t gate;      // row of the matrix table
    int32_t gen;       // 1/2/3 = X/Y/Z generator of a trainable gate, 0 fixed
    int32_t tix;       // index among the group's trainable gates
    int32_t pad;
};

struct AdjGroupArgs {
    uint64_t tbit[kAdjSlots];  // slot s <-> bit tbit[s] of the amplitude index
    uint64_t tmask;    // OR of the slot bits
    int32_t count, pad;
    int32_t n_train, row0;   // trainable gates; gradient row of the first one
};

// Im( conj(l0) (G p)_0 + conj(l1) (G p)_1 ) in double for G = X, Y, Z.
__device__ __forceinline__ double gen_term(int gen, const float2& a0, const float2& a1, const float2& l0,
                                           const float2& l1) {
    const double p0r = a0.x, p0i = a0.y, p1r = a1.x, p1i = a1.y;
    const double q0r = l0.x, q0i = l0.y, q1r = l1.x, q1i = l1.y;
    if (gen == 1) return (q0r * p1i - q0i * p1r) + (q1r * p0i - q1i * p0r);   // X: (p1, p0)
    if (gen == 2) return -(q0r * p1r + q0i * p1i) + (q1r * p0r + q1i * p0i);  // Y: (-i p1, i p0)
    return (q0r * p0i - q0i * p0r) - (q1r * p1i - q1i * p1r);                  // Z: (p0, -p1)
}

__device__ __forceinline__ void mul2(const float* m, float2& v0, float2& v1) {
    float2 o0, o1;
    o0.x = m[0] * v0.x - m[1] * v0.y + m[2] * v1.x - m[3] * v1.y;
    o0.y = m[0] * v0.y + m[1] * v0.x + m[2] * v1.y + m[3] * v1.x;
    o1.x = m[4] * v0.x - m[5] * v0.y + m[6] * v1.x - m[7] * v1.y;
    o1.y = m[4] * v0.y + m[5] * v0.x + m[6] * v1.y + m[7] * v1.x;
    v0 = o0;
    v1 = o1;
}

// The wave's sum, in lane 63: register-to-register moves, rows of 16 lanes
// first, as six exchanges through LDS held up the wave for every gate.
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

// One gate on target slot S of the registers (pairs j0, j0 | 2^S).  Returns
// the thread's gradient term (trainable gate) before the update.
template <int NA, int S>
__device__ __forceinline__ double adj_slot(float2 (&a)[NA], float2 (&l)[NA], const float* m, int cj, bool cok, int gen) {
    double g = 0;
#pragma unroll
    for (int j0 = 0; j0 < NA; ++j0) {
        if (j0 & (1 << S)) continue;
        const int j1 = j0 | (1 << S);
        if (!(cok && (j0 & cj) == cj)) continue;
        if (gen) g += gen_term(gen, a[j0], a[j1], l[j0], l[j1]);
        mul2(m, l[j0], l[j1]);
        mul2(m, a[j0], a[j1]);
    }
    return g;
}

template <int r>
__global__ __launch_bounds__(kAdjThreads) void k_adj_group(float2* __restrict__ psi, float2* __restrict__ lam,
                                                           uint64_t state_len, uint64_t items, AdjGroupArgs A,
                                                           const AdjOpDev* __restrict__ ops,
                                                           const float* __restrict__ mats, int batch,
                                                           double* __restrict__ part) {
    constexpr int NA = 1 << r;
    __shared__ double acc[kAdjMaxTrain * (kAdjThreads / 64)];
    const int b = blockIdx.y;
    float2* P = psi + (size_t)b * state_len;
    float2* Lm = lam + (size_t)b * state_len;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < A.n_train * (kAdjThreads / 64); i += kAdjThreads) acc[i] = 0;
    __syncthreads();
    uint64_t off[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        uint64_t o = 0;
#pragma unroll
        for (int s = 0; s < r; ++s)
            if (j & (1 << s)) o |= A.tbit[s];
        off[j] = o;
    }
    const uint64_t stride = (uint64_t)gridDim.x * kAdjThreads;
    // the loop bound is uniform over the wave, so every lane takes part in
    // the wave reductions; lanes past the end hold zeros and store nothing
    for (uint64_t w0 = (uint64_t)blockIdx.x * kAdjThreads + wave * 64; w0 < items; w0 += stride) {
        const uint64_t w = w0 + lane;
        const bool act = w < items;
        const uint64_t base = act ? place(w, ~A.tmask) : 0;
        float2 a[NA], l[NA];
#pragma unroll
        for (int j = 0; j < NA; ++j) {
            a[j] = act ? P[base | off[j]] : float2{0, 0};
            l[j] = act ? Lm[base | off[j]] : float2{0, 0};
        }
        // the record two gates ahead, the matrix one ahead
        AdjOpDev next = ops[A.count - 1], after = ops[max(A.count - 2, 0)];
        float mn[8];
        auto matrix = [&](int gate) {
            const float* md = mats + ((size_t)gate * batch + b) * 8;
#pragma unroll
            for (int i = 0; i < 8; ++i) mn[i] = md[i];
        };
        matrix(next.gate);
        for (int oi = 0; oi < A.count; ++oi) {
            const AdjOpDev op = next;
            float m[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) m[i] = mn[i];
            next = after;
            matrix(next.gate);
            after = ops[max(A.count - 3 - oi, 0)];
            const bool cok = act && (base & op.cout) == op.cout;
            const int gen = op.gen;
            double g = 0;
            switch (op.slot) {
                case 0: g = adj_slot<NA, 0>(a, l, m, op.cj, cok, gen); break;
                case 1: if constexpr (r > 1) g = adj_slot<NA, (r > 1 ? 1 : 0)>(a, l, m, op.cj, cok, gen); break;
                case 2: if constexpr (r > 2) g = adj_slot<NA, (r > 2 ? 2 : 0)>(a, l, m, op.cj, cok, gen); break;
                default: if constexpr (r > 3) g = adj_slot<NA, (r > 3 ? 3 : 0)>(a, l, m, op.cj, cok, gen); break;
            }
            if (gen) {
                g = wave_total(g);
                if (lane == 63) acc[op.tix * (kAdjThreads / 64) + wave] += g;
            }
        }
        if (act) {
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                P[base | off[j]] = a[j];
                Lm[base | off[j]] = l[j];
            }
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < A.n_train; t += kAdjThreads) {
        const double* v = acc + t * (kAdjThreads / 64);
        part[((size_t)(A.row0 + t) * kAdjBlocks + blockIdx.x) * batch + b] = (v[0] + v[1]) + (v[2] + v[3]);
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
    if constexpr (sizeof(R) == 4) {                            // and their adjoints
        R* d = mats + ((size_t)nruns * batch + i) * 8;
        d[0] = (R)u[0]; d[1] = (R)-u[1]; d[2] = (R)u[4]; d[3] = (R)-u[5];
        d[4] = (R)u[2]; d[5] = (R)-u[3]; d[6] = (R)u[6]; d[7] = (R)-u[7];
    }
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
    bool matrix() const { return kind < AD_MOVE; }
};

// merge: consecutive uncontrolled gates on a qubit as one step (complex128).
std::vector<AdjStep> adj_steps(const std::vector<AdjGate>& G, bool merge) {
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
        for (uint64_t m = g.cmask | s.xq; m; m &= m - 1) open[__builtin_ctzll(m)] = -1;
        if (joins) open[g.target] = (int)out.size();
        if (g.pidx >= 0) {
            s.kind = g.gen == 2 ? AD_RE : g.gen == 3 ? AD_DG : AD_MAT;
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
    std::vector<int> slots;          // target qubits, as they came
    int train;
};

std::vector<AdjGroup> adj_groups(const std::vector<AdjStep>& S, int r) {
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
            if (!(t & tb)) g.slots.push_back(S[i].target);
            t |= tb;
            g.steps.push_back((int)i);
            done[i] = 1;
            --left;
            g.train += S[i].need != 0;
        }
        while (first < S.size() && done[first]) ++first;
        out.push_back(std::move(g));
    }
    return out;
}

// complex64, forward: a group is a round, and consecutive groups share a pass
// while their targets and the low bits fit in the tile.
std::vector<AdjPassPlan> adj_passes_ordered(const std::vector<AdjGroup>& groups, int n, int L, int c, int r) {
    std::vector<AdjPassPlan> out;
    size_t ops = 0;
    for (const AdjGroup& g : groups) {
        uint64_t t = 0;
        for (int q : g.slots) t |= 1ull << q;
        if (out.empty() || pc(out.back().qmask | t) > L || ops + g.steps.size() > (size_t)kAdjMaxOps) {
            out.push_back(AdjPassPlan{(1ull << std::min(c, n)) - 1, {}, {}, {}});
            ops = 0;
        }
        out.back().qmask |= t;
        out.back().rounds.push_back(g.steps);
        out.back().slots.push_back(t);
        ops += g.steps.size();
    }
    for (AdjPassPlan& P : out) {
        for (int q = 0; q < n && pc(P.qmask) < std::min(L, n); ++q) P.qmask |= 1ull << q;
        for (uint64_t& t : P.slots) t = adj_fill(t, P.qmask, r);
    }
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
    if (P.steps.empty()) return P;   // (complex64 has them already)
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

std::vector<AdjPassPlan> adj_passes(const std::vector<AdjStep>& S, const std::vector<AdjGroup>& groups, int n,
                                    qvm_dtype dt) {
    if (dt == QVM_C64)
        return adj_passes_ordered(groups, n, std::min(n, adj_width<float>()), GT<float>::C, std::min(n, adj_slots<float>()));
    return adj_passes_free(S, n, std::min(n, adj_width<double>()), GT<double>::C);
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

// Slots of a group in k_adj_group: its targets as they came, then the highest
// other qubits, so that the item index runs over the low bits and a wave's
// loads stay contiguous.
std::vector<int> adj_slot_bits(const AdjGroup& g, int n, int r) {
    std::vector<int> bits = g.slots;
    uint64_t t = 0;
    for (int q : bits) t |= 1ull << q;
    for (int q = n - 1; (int)bits.size() < r && q >= 0; --q)
        if (!((t >> q) & 1)) bits.push_back(q);
    return bits;
}

void adj_group_ops(const std::vector<AdjStep>& S, const std::vector<AdjGate>& G, const AdjGroup& g,
                   const std::vector<int>& bits, uint32_t row0, std::vector<uint32_t>& tab) {
    for (int i : g.steps) {
        const AdjStep& s = S[i];
        const AdjGate& gate = G[s.gates[0]];
        AdjOpDev o{};
        o.gate = s.run;
        o.cout = s.cmask;
        for (size_t k = 0; k < bits.size(); ++k) {
            if (bits[k] == s.target) o.slot = (int)k;
            if ((s.cmask >> bits[k]) & 1) {
                o.cj |= 1 << k;
                o.cout &= ~(1ull << bits[k]);
            }
        }
        o.gen = gate.pidx >= 0 ? gate.gen : 0;
        o.tix = s.need ? s.row - (int)row0 : -1;
        const size_t at = tab.size();
        tab.resize(at + sizeof(o) / 4);
        memcpy(&tab[at], &o, sizeof(o));
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
    std::vector<AdjStep> S = adj_steps(G, sizeof(R) == 8);
    const int rs = std::min(n, adj_slots<R>());
    std::vector<AdjGroup> groups;
    if (sizeof(R) == 4) groups = adj_groups(S, rs);
    const std::vector<AdjPassPlan> passes = adj_passes(S, groups, n, sizeof(R) == 4 ? QVM_C64 : QVM_C128);
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
    const size_t total = passes.size() + (!want_grad ? 0 : sizeof(R) == 4 ? groups.size() : passes.size());
    auto prepare = [&](size_t from) -> qvm_status {
        std::vector<uint32_t> t, one;
        for (size_t q = recs.size(); q < total; ++q) {
            const bool rev = q >= passes.size();
            Rec r{0, 0, 0, ~0u, 0};
            auto sums = [&](const std::vector<int>& steps) {
                for (int i : steps)
                    if (S[i].need) {
                        r.row0 = std::min(r.row0, (uint32_t)S[i].row);
                        r.nsum += (uint32_t)pc(S[i].need);
                    }
            };
            one.clear();
            if (rev && sizeof(R) == 4) {
                const AdjGroup& g = groups[total - 1 - q];
                sums(g.steps);
                adj_group_ops(S, G, g, adj_slot_bits(g, n, rs), r.row0, one);
            } else {
                const AdjPassPlan P = adj_rounds(S, passes[rev ? total - 1 - q : q], rev, rs);
                r.qmask = P.qmask;
                r.rounds = (uint32_t)P.rounds.size();
                for (const auto& rd : P.rounds) sums(rd);
                adj_records(S, P, rs, sizeof(T), r.row0, one);
            }
            one.resize((one.size() + 1) & ~size_t(1));
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
    hipLaunchKernelGGL((k_adj_pass<R, RR, REV>), grid, dim3(threads), lds, stream, psi, lam, A, dtab, mats, \
                       (uint32_t)batch, nblk, gpart);
        if (!rev) {
            switch (rs) {
                case 1: QVM_ADJ_LAUNCH(1, false) break;
                case 2: QVM_ADJ_LAUNCH(2, false) break;
                case 3: QVM_ADJ_LAUNCH(3, false) break;
                default: if constexpr (sizeof(R) == 4) { QVM_ADJ_LAUNCH(4, false) } break;
            }
        } else if constexpr (sizeof(R) == 8) {
            const qvm_status st = rs == 3 ? lds_limit((const void*)k_adj_pass<R, 3, true>) : QVM_OK;
            if (st) return st;
            switch (rs) {
                case 1: QVM_ADJ_LAUNCH(1, true) break;
                case 2: QVM_ADJ_LAUNCH(2, true) break;
                default: QVM_ADJ_LAUNCH(3, true) break;
            }
        }
#undef QVM_ADJ_LAUNCH
        QVM_LAUNCH_CHECK(sv);
        return QVM_OK;
    };
    auto launch_group = [&](size_t q) -> qvm_status {
        if (q >= recs.size()) {
            qvm_status st = prepare(q);
            if (st) return st;
        }
        const AdjGroup& g = groups[total - 1 - q];
        AdjGroupArgs A{};
        const std::vector<int> bits = adj_slot_bits(g, n, rs);
        for (int k = 0; k < rs; ++k) A.tmask |= A.tbit[k] = 1ull << bits[k];
        A.count = (int32_t)g.steps.size();
        A.n_train = g.train;
        A.row0 = g.train ? (int32_t)recs[q].row0 : 0;
        const AdjOpDev* ops = (const AdjOpDev*)(dtab + recs[q].at);
        const R* adj = mats + nrun * (size_t)batch * 8;
        const dim3 grid(kAdjBlocks, (unsigned)batch);
#define QVM_ADJ_LAUNCH(RR)                                                                              \
    hipLaunchKernelGGL((k_adj_group<RR>), grid, blk, 0, stream, psi, lam, N, N >> RR, A, ops, adj, batch, gpart);
        if constexpr (sizeof(R) == 4) {
            switch (rs) {
                case 1: QVM_ADJ_LAUNCH(1) break;
                case 2: QVM_ADJ_LAUNCH(2) break;
                case 3: QVM_ADJ_LAUNCH(3) break;
                default: QVM_ADJ_LAUNCH(4) break;
            }
        }
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
    if (sizeof(R) == 4) {
        nblk = kAdjBlocks;
    } else if (nsum) {
        const size_t room = std::min<size_t>(kAdjBlocks, nocc * kAdjBlocks / nsum);
        while (2 * nblk <= room) nblk *= 2;
        // (fewer than nblk tiles: every block still has its partial)
        nblk = (uint32_t)std::min<uint64_t>(nblk, std::max<uint64_t>(1, N >> std::min(n, adj_width<R>())));
    }
    for (size_t q = passes.size(); q < total; ++q) {
        qvm_status st = sizeof(R) == 4 ? launch_group(q) : launch_pass(q);
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
    *n_groups = (int32_t)adj_groups(adj_steps(G, false), r).size();
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
    const std::vector<AdjStep> S = adj_steps(G, dt == QVM_C128);
    std::vector<AdjGroup> groups;
    if (dt == QVM_C64) groups = adj_groups(S, std::min(n, adj_slots<float>()));
    *n_passes = (int32_t)adj_passes(S, groups, n, dt).size();
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
