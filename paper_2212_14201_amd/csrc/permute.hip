// Back to the identity layout: the physical bits of the state permuted in few
// passes (qvm_reset_layout).
//
// A pass keeps tiles of the lowest c bits (128-byte runs) and up to nine more
// in LDS and writes them back with the tile's bits in another order, so every
// qubit whose bit and place are both among the tile's bits arrives.  The next
// pass takes other bits.  A swap of two bits moves half of the state, and so
// half as much as a pass, but a layout is many swaps away from the identity,
// and a swap with one of the lowest bits moves pieces shorter than a 128-byte
// line.
//
// What bounds it: HBM.  26 qubits, complex128 (1 GiB), the layout after a
// random circuit, 13 swaps away: 2.83 ms as swaps (160 to 580 us each), now
// 0.81 in two passes of 5.3 TB/s.  30 qubits, complex64 (8 GiB), 15 swaps away:
// 51 ms, now 13.6 in four.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "gatepass.hpp"

namespace qvm {

namespace {

constexpr int kPermThreads = 512;
constexpr int kPermPieces = 8;                   // 16-byte pieces per thread

struct PermArgs {
    uint64_t qmask;                              // tile bits
    uint32_t L, pad;
    uint32_t top[3];                             // positions of the three highest tile bits, ascending
    uint32_t src[13];                            // LDS byte address of the tile bit that output bit b comes from
};

template <typename R>
__global__ __launch_bounds__(kPermThreads) void k_permute(typename GT<R>::T* __restrict__ psi, PermArgs A) {
    using V16 = typename GT<R>::V16;
    using V2 = typename Vec2<R>::V;
    constexpr int EP = GT<R>::EP, LB = EP == 2 ? 1 : 0;
    constexpr uint32_t ES = sizeof(typename GT<R>::T);
    const uint32_t tid = threadIdx.x, nt = 1u << (A.L - LB - 3);
    const bool live = tid < nt;
    const uint64_t g0 = place(blockIdx.x, ~A.qmask) + place(EP * tid, A.qmask);
    uint64_t gtop[3];
    uint32_t stop[3], otop[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        gtop[k] = 1ull << A.top[k];
        stop[k] = tile_swizzle(1u << (A.L - 3 + k));
        otop[k] = A.src[A.L - 3 + k];
    }
    if (live) {
        const uint32_t s0 = tile_swizzle(EP * tid);
        V16 v[kPermPieces];
#pragma unroll
        for (int i = 0; i < kPermPieces; ++i)
            v[i] = __builtin_nontemporal_load((const V16*)(psi + g0 + subset<3>(gtop, i)));
#pragma unroll
        for (int i = 0; i < kPermPieces; ++i) {
            const uint32_t s = s0 ^ subset<3>(stop, i);
            if constexpr (EP == 2) {
                const V16 x = (s & 1) ? V16{v[i][2], v[i][3], v[i][0], v[i][1]} : v[i];
                gst<V16>((s & ~1u) * ES, x);
            } else {
                gst<V16>(s * ES, v[i]);
            }
        }
    }
    __syncthreads();
    if (live) {
        uint32_t o0 = 0;                         // the thread's bits, from where they are
        for (uint32_t b = 0; b + 3 + LB < A.L; ++b) o0 ^= ((tid >> b) & 1u) ? A.src[LB + b] : 0u;
#pragma unroll
        for (int i = 0; i < kPermPieces; ++i) {
            const uint32_t o = o0 ^ subset<3>(otop, i);
            V16 x;
            if constexpr (EP == 2) {
                const V2 a = gld<V2>(o), b = gld<V2>(o ^ A.src[0]);
                x = V16{a[0], a[1], b[0], b[1]};
            } else {
                x = gld<V16>(o);
            }
            __builtin_nontemporal_store(x, (V16*)(psi + g0 + subset<3>(gtop, i)));
        }
    }
}

// cur[p]: the bit that the amplitudes' bit p is to become.  The bits of the
// next pass: the lowest c, then, one at a time, the one that lets most bits
// of the tile arrive.
uint64_t next_tile(const int* cur, int n, int L, int c) {
    uint64_t Q = (1ull << std::min(c, n)) - 1;
    int home[QVM_MAX_QUBITS];                    // where bit b is now
    for (int p = 0; p < n; ++p) home[cur[p]] = p;
    while (pc(Q) < L) {
        int best = -1, gain = -1;
        for (int p = 0; p < n; ++p) {
            if ((Q >> p) & 1) continue;
            const uint64_t with = Q | 1ull << p;
            int g = 0;
            if (cur[p] != p) g = 1 + 2 * (int)((with >> cur[p]) & 1) + 2 * (int)((with >> home[p]) & 1);
            if (g > gain) {
                gain = g;
                best = p;
            }
        }
        Q |= 1ull << best;
    }
    return Q;
}

// cur after a pass over Q; from[p]: the bit whose amplitudes' bit goes to p.
void arrange(int* cur, int n, uint64_t Q, int* from) {
    int old[QVM_MAX_QUBITS];
    std::copy(cur, cur + n, old);
    uint64_t placed = 0, taken = 0;              // bits that have their content; contents that have a bit
    auto put = [&](int p, int q) {
        from[p] = q;
        cur[p] = old[q];
        placed |= 1ull << p;
        taken |= 1ull << q;
    };
    for (int q = 0; q < n; ++q)
        if (((Q >> q) & 1) && ((Q >> old[q]) & 1)) put(old[q], q);
    for (int q = 0; q < n; ++q)                  // the rest stay where they are, as far as there is room
        if (((Q >> q) & 1) && !((taken >> q) & 1) && !((placed >> q) & 1)) put(q, q);
    int p = 0;
    for (int q = 0; q < n; ++q) {
        if (!((Q >> q) & 1) || ((taken >> q) & 1)) continue;
        while (!((Q >> p) & 1) || ((placed >> p) & 1)) ++p;
        put(p, q);
    }
}

template <typename R>
qvm_status permute_pass(qvm_sv* sv, uint64_t Q, const int* from) {
    using T = typename GT<R>::T;
    const int n = sv->n, L = pc(Q);
    PermArgs A{};
    A.qmask = Q;
    A.L = (uint32_t)L;
    int k = 3, e = 0;
    for (int b = n - 1; k > 0; --b)
        if ((Q >> b) & 1) A.top[--k] = (uint32_t)b;
    for (int b = 0; b < n; ++b)
        if ((Q >> b) & 1) A.src[e++] = tile_swizzle(local_bits(1ull << from[b], Q)) * (uint32_t)sizeof(T);
    const unsigned threads = std::max(64u, 1u << (L - 3 - (GT<R>::EP == 2 ? 1 : 0)));
    const int tok = prof_begin(sv);
    hipLaunchKernelGGL((k_permute<R>), dim3(1u << (n - L)), dim3(threads), sizeof(T) << L, sv->stream, (T*)sv->amps, A);
    QVM_LAUNCH_CHECK(sv);
    prof_end(sv, tok, PK_SWAP, 2.0 * (double)(1ull << n) * sizeof(T), 0.0);
    return QVM_OK;
}

}  // namespace

// Swaps where they are cheaper, in units of a swap of two bits above the lowest
// c (26 qubits: complex64 96 us, complex128 170 to 190): with the highest of
// those c the swap moves half lines (155; 345), with a lower one shorter pieces
// (285 to 420; 550 to 580); a pass takes 190; 375 to 400.  Below 2^8 amplitudes
// a tile would not fill the threads' pieces.
qvm_status reset_layout(qvm_sv* sv) {
    const int n = sv->n, c = sv->dt == QVM_C64 ? GT<float>::C : GT<double>::C;
    const int L = std::min(n, sv->dt == QVM_C64 ? GT<float>::LMAX : GT<double>::LMAX);
    int cur[QVM_MAX_QUBITS], from[QVM_MAX_QUBITS], sim[QVM_MAX_QUBITS];
    for (int q = 0; q < n; ++q) cur[sv->perm[q]] = q;
    auto home = [&](const int* at) {
        for (int p = 0; p < n; ++p)
            if (at[p] != p) return false;
        return true;
    };
    double swaps = 0, passes = 0;
    std::copy(cur, cur + n, sim);
    for (int q = 0; q < n; ++q)
        if (sim[q] != q) {
            const int p = (int)(std::find(sim, sim + n, q) - sim);
            swaps += std::min(p, q) >= c ? 1.0 : std::min(p, q) == c - 1 ? 1.9 : 3.0;
            std::swap(sim[p], sim[q]);
        }
    if (n >= 8) {
        std::copy(cur, cur + n, sim);
        while (!home(sim)) {
            arrange(sim, n, next_tile(sim, n, L, c), from);
            passes += 2.2;
        }
    }
    if (n < 8 || swaps <= passes) {
        for (int q = 0; q < n; ++q) {
            if (cur[q] == q) continue;
            const int p = (int)(std::find(cur, cur + n, q) - cur);
            const qvm_status st = launch_swap_bits(sv, p, q);
            if (st) return st;
            std::swap(cur[p], cur[q]);
            sv->perm[cur[p]] = p;
            sv->perm[cur[q]] = q;
        }
        return QVM_OK;
    }
    while (!home(cur)) {
        const uint64_t Q = next_tile(cur, n, L, c);
        arrange(cur, n, Q, from);
        const qvm_status st = sv->dt == QVM_C64 ? permute_pass<float>(sv, Q, from) : permute_pass<double>(sv, Q, from);
        if (st) return st;
        for (int p = 0; p < n; ++p) sv->perm[cur[p]] = p;
    }
    return QVM_OK;
}

}  // namespace qvm
