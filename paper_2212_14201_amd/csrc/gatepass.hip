// Gate passes: a gate list applied gate by gate, many gates per pass over the
// state (qvm_run).
//
// A gate on its own reads and writes the state for at most 16 multiply-adds
// per amplitude pair, so one kernel per gate is bound by HBM (measured 5.6 ms
// per 30-qubit complex128 gate) and, below about 20 qubits, by its launch
// (2.7-4 us).  A gate pass keeps tiles of up to 2^13 (complex64) / 2^12
// (complex128) amplitudes in LDS and applies every gate of the list that can
// run on the tile's qubits, each gate by itself: unlike a fused plan no
// matrices of different qubits are multiplied together.
//
//   pass   one workgroup per tile: the 2^L amplitudes that share all
//          non-tile physical bits; the tile always holds the c lowest bits
//          (128-byte runs).  Targets of non-diagonal gates must be tile
//          bits; controls and diagonal gates may sit anywhere.
//   round  a thread holds the 16 (8 in passes of few tiles) amplitudes that
//          differ in four (three) of the tile bits, the slots, in registers
//          and applies, in order, the gates whose targets are slots; then the
//          amplitudes go back to LDS and the next round takes other slots.
//          16 amplitudes (32 or 64 VGPRs) keep four waves per SIMD in
//          complex64 and two in complex128 (of 64 KiB tiles).
//   record what a round applies at once: one gate, the signs that are due, or
//          a LAYER, the factors and the one-target gates that are due
//          (pass_gates): in complex64 as rotations and phases, in complex128
//          as the matrices they are.
//
// What bounds it: 28 qubits, complex128, 8 layers of U3 + CZ (332 gates):
// 361 ms with one kernel per gate; 31.6 ms in 6 passes with a dense 2 x 2
// product and a record per gate, 27.5 with LAYER and SIGNS records (a dozen
// branches to choose a record's op): vector instructions in 69% of the cycles.
// The FP64 multiply-adds alone take 12 ms, the passes' traffic 8.  (As
// rotations and phases, a third of the multiply-adds, 21.6 ms, but further
// from the gates: pass_gates.)
// 25 qubits, complex64, 4 layers of rotations + CNOTs (400 gates): 35.3 ms
// with one kernel per gate, 1.92 with dense products, now 1.75 (11 passes,
// whose traffic takes 0.92).  12 qubits, complex128, 20 layers (350 gates, one
// workgroup): 1.38 ms, 0.187, now 0.156.
//
// The list's records are written to the workspace by k_put kernels, which
// carry them as kernel arguments: no copy from host memory that the caller
// or this call would have to keep alive, and a captured graph holds them.
// A k_put takes 2 to 5 us (its argument block is read from host memory), so
// it carries up to 16,000 bytes (3,840: 165 -> 155 us for 200 mixed gates on
// 12 qubits).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <vector>

#include "gatepass.hpp"

namespace qvm {

namespace {

// Op codes.  D1 + s: dense gate on slot s; D2 + pair: on the slot pair (0,1),
// (0,2), (0,3), (1,2), (1,3), (2,3); D3 + s: on the three slots other than s;
// PHASE: one factor; SIGN: a factor of -1; DIAG: two factors chosen by the
// parity of some index bits (RZ, RZZ); MOVE + x: amplitudes j and j ^ x
// exchanged (x = 1..15 over the slots); SIGNS: factors of -1, each on its own
// condition; LAYER: a factor of its own for every register, then a real
// rotation on each of some slots.
enum : uint32_t { GP_D1 = 0, GP_D2 = 4, GP_D3 = 10, GP_PHASE = 14, GP_DIAG = 15, GP_MOVE = 16, GP_SIGNS = 32, GP_LAYER = 33 };

// One op: 8 words, then its values (R).  A record applies to register j of
// thread (local index) t in tile w when bit j of jbits is set, (t & tm) ==
// tv and (w & om) == ov.  t is the tile element with the slot bits at zero.
struct OpHead {
    uint32_t code;          // op code | words to the next record << 8
    uint32_t jbits;         // registers it applies to (D1..D3: by the first of each group) |
                            // DIAG: registers with odd slot parity << 16 |
                            // LAYER: the slots rotated, and kTable if there are factors |
                            // SIGNS: how many conditions follow (SignCond)
    uint32_t tm, tv;
    uint32_t om, ov;
    uint32_t pt, po;        // DIAG: parity masks over t and w
};
static_assert(sizeof(OpHead) == 32, "eight words");
constexpr uint32_t kTable = 16;
// Values of a LAYER record before its factors: complex64 two per slot (a
// rotation), complex128 a 2 x 2 matrix for every slot in the mask.
template <typename R>
__host__ __device__ constexpr int layer_vals(uint32_t mask) {
    return sizeof(R) == 4 ? 2 * kSlots : 8 * __builtin_popcount(mask);
}
struct SignCond {
    uint32_t jbits, tm, tv, om, ov, pad[3];
};
static_assert(sizeof(SignCond) == 32, "eight words");

// A round: 16 words.  The slots' addresses are worked out on the host: the
// same uniform arithmetic in every wave cost more scalar instructions per
// round (about 1,250) than the round's gates take vector ones.
struct RoundHead {
    uint32_t bit[kSlots];   // tile-local bit of each slot, ascending
    uint32_t lds[kSlots];   // its LDS byte address (linear over GF(2))
    uint32_t nops;
    uint32_t phys[kSlots];  // its physical bit's position, for a direct round
    uint32_t pad[3];
};
static_assert(sizeof(RoundHead) == 64, "sixteen words");
constexpr uint32_t RND_WORDS = 16;

struct PassArgs {
    uint64_t qmask;         // physical tile bits
    uint32_t L;
    uint32_t nrounds;
    uint32_t words;         // offset of the pass's records in the table
    uint32_t direct;        // bit 0: the first round loads from memory, bit 1: the last one stores there
    uint32_t top[kSlots];   // positions of the four highest tile bits (a thread's pieces), ascending
    uint32_t lines;         // 128-byte lines of the records
};

// A pass that also measures: the reduced density matrix of four tile bits
// (k_gate_pass with RDM), after the pass's gates.
struct RdmArgs {
    uint32_t ntiles;        // the workgroups loop over the tiles: one partial each
    uint32_t store;         // 0: no gates ran, the tile is as it was
    uint32_t slot[kSlots];  // LDS byte addresses of the measured bits, ascending
    uint32_t col[9];        // LDS byte addresses of the other tile bits, ascending
    uint32_t pad;
};

constexpr uint32_t kWarmGroups = 512;            // workgroups that read the records ahead: two per CU
constexpr uint32_t kPutWords = 4000;              // 16,000 bytes of records per k_put launch
struct PutArgs {
    uint32_t* dst;
    uint32_t n, pad;
    uint32_t w[kPutWords];
};

__global__ __launch_bounds__(256) void k_put(PutArgs a) {
    // the records straight from the argument block (a dynamic index into the
    // by-value struct would copy it to scratch first)
    const uint32_t* arg = (const uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t* dst = a.dst;
    for (uint32_t i = threadIdx.x; i < a.n; i += 256) dst[i] = arg[4 + i];
}

// Dense gate on K of the slots (slot mask SM); mv: 2^K x 2^K complex.
template <typename R, int K, int SM, typename T, int NA>
__device__ __forceinline__ void op_dk(T (&a)[NA], const R* __restrict__ mv, uint32_t jbits) {
    constexpr int D = 1 << K;
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        if (j & SM) continue;
        if (!((jbits >> j) & 1)) continue;
        T o[D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
            R re = 0, im = 0;
            int sub = 0;                                       // register offset of column c
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const R mr = mv[2 * (i * D + c)], mi = mv[2 * (i * D + c) + 1];
                const T v = a[j | sub];
                re += mr * v.x - mi * v.y;
                im += mr * v.y + mi * v.x;
                sub = (sub - SM) & SM;
            }
            o[i].x = re;
            o[i].y = im;
        }
        // all of the results, then back (move_to)
#pragma unroll
        for (int i = 0; i < D; i += 4)
            asm volatile("" : "+v"(o[i].x), "+v"(o[i].y), "+v"(o[i + 1].x), "+v"(o[i + 1].y), "+v"(o[i + 2].x),
                         "+v"(o[i + 2].y), "+v"(o[i + 3].x), "+v"(o[i + 3].y));
        int sub = 0;
#pragma unroll
        for (int i = 0; i < D; ++i) {
            a[j | sub] = T{move_to(o[i].x), move_to(o[i].y)};
            sub = (sub - SM) & SM;
        }
    }
}

// The rotation [c -s; s c] on slot S as three shears: v0 += a v1, v1 += b v0,
// v0 += a v1 with a = -tan(angle / 2) and b = s, angle in [0, pi/2].  Six
// multiply-adds per pair, all in place, where a dense gate takes sixteen and
// three register moves.
template <typename R, int S, typename T, int NA>
__device__ __forceinline__ void op_turn(T (&a)[NA], R ta, R tb) {
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        if (j & (1 << S)) continue;
        T &v0 = a[j], &v1 = a[j | (1 << S)];
        v0.x += ta * v1.x;
        v0.y += ta * v1.y;
        v1.x += tb * v0.x;
        v1.y += tb * v0.y;
        v0.x += ta * v1.x;
        v0.y += ta * v1.y;
    }
}

// A LAYER's matrix m on slot S, if S is in the mask jb, and the values of the
// next one (after the last: in bounds, not used), loaded while it is applied.
template <typename R, int S, typename T, int NA>
__device__ __forceinline__ void op_next(T (&a)[NA], R (&m)[8], const R* __restrict__& mv, uint32_t jb) {
    if (!(jb & (1u << S))) return;
    R next[8];
    mv += 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) next[i] = mv[i];
#pragma unroll
    for (int j = 0; j < NA; ++j)
        if (!(j & (1 << S))) pair2<R>(m, a[j], a[j | (1 << S)]);
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = next[i];
}

// A record's head and its first 8 values, in scalar registers: the next
// record is loaded while the current one is applied (a wave otherwise waits
// for two dependent scalar loads per gate, 1,500 cycles of a 2,000-cycle
// gate where one workgroup holds the whole state).
template <typename R> struct Rec {
    static constexpr int NW = 8 + 8 * (int)sizeof(R) / 4;      // 16 or 24 words (a round's head is 16)
    uint32_t w[NW];
    __device__ __forceinline__ void load(const uint32_t* __restrict__ p) {
        typedef uint32_t U8 __attribute__((ext_vector_type(8), aligned(4)));
#pragma unroll
        for (int i = 0; i < NW; i += 8) {
            const U8 x = *(const U8*)(p + i);
#pragma unroll
            for (int k = 0; k < 8; ++k) w[i + k] = x[k];
        }
    }
    __device__ __forceinline__ R val(int i) const {
        if constexpr (sizeof(R) == 4) return __uint_as_float(w[8 + i]);
        else return __longlong_as_double((long long)((uint64_t)w[8 + 2 * i] | (uint64_t)w[9 + 2 * i] << 32));
    }
};

template <typename R, typename T, int NA>
__device__ __forceinline__ void apply_op(T (&a)[NA], const OpHead& h, const Rec<R>& rec,
                                         const R* __restrict__ mv, uint32_t le, uint32_t w) {
    const uint32_t code = h.code & 0xffu;
    const uint32_t jb = h.jbits & 0xffffu;
    if (!below(code, GP_SIGNS)) {
        if (is(code, GP_LAYER)) {
            if (jb & kTable) {
                const R* __restrict__ f = mv + layer_vals<R>(jb & (kTable - 1));
#pragma unroll
                for (int j = 0; j < NA; ++j) phase1<R>(f[2 * j], f[2 * j + 1], a[j]);
            }
            if constexpr (sizeof(R) == 4) {
                if (jb & 1) op_turn<R, 0>(a, rec.val(0), rec.val(1));
                if (jb & 2) op_turn<R, 1>(a, rec.val(2), rec.val(3));
                if (jb & 4) op_turn<R, 2>(a, rec.val(4), rec.val(5));
                if constexpr (NA == 16)
                    if (jb & 8) op_turn<R, 3>(a, rec.val(6), rec.val(7));
            } else {
                R m[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) m[i] = rec.val(i);
                op_next<R, 0>(a, m, mv, jb);
                op_next<R, 1>(a, m, mv, jb);
                op_next<R, 2>(a, m, mv, jb);
                if constexpr (NA == 16) op_next<R, 3>(a, m, mv, jb);
            }
        }
        if (is(code, GP_SIGNS)) {
            // each register's sign: the parity of the conditions the thread meets
            uint32_t odd = 0;
            typedef uint32_t U8 __attribute__((ext_vector_type(8), aligned(4)));
            const U8* __restrict__ c = (const U8*)mv;
            for (uint32_t i = 0; i < jb; ++i) {
                const U8 x = c[i];
                odd ^= (((w & x[3]) ^ x[4]) | ((le & x[1]) ^ x[2])) == 0 ? x[0] : 0u;
            }
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                const uint32_t f = (odd << (31 - j)) & 0x80000000u;
                a[j].x = flip_sign(a[j].x, f);
                a[j].y = flip_sign(a[j].y, f);
            }
        }
    }
    if (below(code, GP_D2)) {
        R m[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) m[i] = rec.val(i);
        if (is(code, GP_D1)) op_d1<R, 0>(a, m, jb);
        if (is(code, GP_D1 + 1)) op_d1<R, 1>(a, m, jb);
        if (is(code, GP_D1 + 2)) op_d1<R, 2>(a, m, jb);
        if constexpr (NA == 16)
            if (is(code, GP_D1 + 3)) op_d1<R, 3>(a, m, jb);
    }
    if (below(code - GP_PHASE, GP_SIGNS - GP_PHASE)) {
        if (is(code, GP_PHASE)) {
            const R pr = rec.val(0), pi = rec.val(1);
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if ((jb >> j) & 1) phase1(pr, pi, a[j]);
        }
        if (is(code, GP_DIAG)) {
            const bool odd = ((__popc(le & h.pt) + __popc(w & h.po)) & 1) != 0;
            const R er = odd ? rec.val(2) : rec.val(0), ei = odd ? rec.val(3) : rec.val(1);     // registers of even slot parity
            const R qr = odd ? rec.val(0) : rec.val(2), qi = odd ? rec.val(1) : rec.val(3);
#pragma unroll
            for (int j = 0; j < NA; ++j)
                if ((jb >> j) & 1) {
                    const bool o = (h.jbits >> (16 + j)) & 1;
                    phase1<R>(o ? qr : er, o ? qi : ei, a[j]);
                }
        }
#define QVM_GP_MV(X) if constexpr (X < NA) if (is(code, GP_MOVE + X)) op_move<X>(a, jb);
        QVM_GP_MV(1) QVM_GP_MV(2) QVM_GP_MV(4) QVM_GP_MV(8)
        if (!below(code, GP_MOVE + 3) && __popc(code - GP_MOVE) > 1) {
            QVM_GP_MV(3) QVM_GP_MV(5) QVM_GP_MV(6) QVM_GP_MV(7) QVM_GP_MV(9) QVM_GP_MV(10) QVM_GP_MV(11) QVM_GP_MV(12)
            QVM_GP_MV(13) QVM_GP_MV(14) QVM_GP_MV(15)
        }
#undef QVM_GP_MV
    }
    if (below(code - GP_D2, GP_PHASE - GP_D2)) {
#define QVM_GP_DK(C, K, SM) if constexpr (SM < NA) if (is(code, C)) op_dk<R, K, SM>(a, mv, jb);
        QVM_GP_DK(GP_D2 + 0, 2, 3) QVM_GP_DK(GP_D2 + 1, 2, 5) QVM_GP_DK(GP_D2 + 2, 2, 9) QVM_GP_DK(GP_D2 + 3, 2, 6)
        QVM_GP_DK(GP_D2 + 4, 2, 10) QVM_GP_DK(GP_D2 + 5, 2, 12) QVM_GP_DK(GP_D3 + 0, 3, 14) QVM_GP_DK(GP_D3 + 1, 3, 13)
        QVM_GP_DK(GP_D3 + 2, 3, 11) QVM_GP_DK(GP_D3 + 3, 3, 7)
#undef QVM_GP_DK
    }
}

// ------------------------------------------------------------------ kernel
// 2^(L-RS) threads work (at least a wave is launched); thread t's item in a
// round is the tile element with t spread around the RS slots.  LDS addresses
// use the tile kernel's swizzle: linear over GF(2), so register j's address
// is the thread's XOR a uniform word, and four lane bits rarely collide.
typedef double D4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kRdmVals = 512;               // values of a partial: 8 per lane
constexpr uint32_t kRdmBlocks = 512;             // workgroups of a measuring pass, at most: two per CU (2,048: 15.2 against 14.2 ms a run below)

// rho_ij = sum over the tile's columns of psi_i conj(psi_j), i and j over the
// 16 values of the measured bits: a product of the 16 x 2^(L-4) matrix of
// the tile's amplitudes with its adjoint, on FP64 MFMA 16x16x4.  Lane l reads
// amplitude l % 16 of column l / 16 of four; the same registers are both
// operands: re re + im im is rho's real part, im re minus its transpose the
// imaginary part (the host subtracts).  Three instructions per 64
// amplitudes: about half the time their traffic takes.
template <typename R>
__device__ __forceinline__ void rdm_tile(D4& rr, D4& ri, const RdmArgs& M, uint32_t L) {
    using V2 = typename Vec2<R>::V;
    const uint32_t lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ncol = 1u << (L - kSlots);
    uint32_t at = 0;                                           // the lane's amplitude and column of four
#pragma unroll
    for (int b = 0; b < kSlots; ++b) at ^= ((lane >> b) & 1) ? M.slot[b] : 0u;
    at ^= ((lane >> 4) & 1) ? M.col[0] : 0u;
    at ^= ((lane >> 5) & 1) ? M.col[1] : 0u;
    for (uint32_t c = 4 * wv; c < ncol; c += 4 * nw) {
        uint32_t u = 0;
#pragma unroll
        for (int b = 2; b < 9; ++b) u ^= ((c >> b) & 1) ? M.col[b] : 0u;
        V2 v = {0, 0};
        if (c + (lane >> 4) < ncol) v = gld<V2>(at ^ u);
        const double x = v[0], y = v[1];
        rr = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, rr, 0, 0, 0);
        rr = __builtin_amdgcn_mfma_f64_16x16x4f64(y, y, rr, 0, 0, 0);
        ri = __builtin_amdgcn_mfma_f64_16x16x4f64(y, x, ri, 0, 0, 0);
    }
}

template <typename R, int RS, bool RDM>
__global__ __launch_bounds__(RS == 4 && sizeof(R) == 8 ? 256 : 512, RS == 4 && sizeof(R) == 8 ? 2 : 4) void k_gate_pass(
    typename GT<R>::T* __restrict__ psi, PassArgs A, const uint32_t* __restrict__ table, RdmArgs M,
    double* __restrict__ part) {
    using T = typename GT<R>::T;
    using V16 = typename GT<R>::V16;
    using V2 = typename Vec2<R>::V;
    constexpr int EP = GT<R>::EP;
    constexpr int kAmps = 1 << RS;                             // amplitudes per thread
    constexpr int NIT = kAmps / EP;                            // 16-byte pieces per thread
    constexpr uint32_t ES = sizeof(T);
    const uint32_t nt = 1u << (A.L - RS);                  // working threads
    const uint32_t tid = threadIdx.x;
    const bool live = tid < nt;
    T a[kAmps];
    D4 rr = {0, 0, 0, 0}, ri = {0, 0, 0, 0};                   // RDM: sums of the workgroup's tiles
    if (blockIdx.x < kWarmGroups) {
        // the records into L2 while the tile is on its way: they were
        // written on another die (200 mixed gates, 17 qubits, complex64, ten
        // passes of 64 workgroups: 179 -> 165 us)
        uint32_t x = 0;
        for (uint32_t i = tid; i < A.lines; i += blockDim.x) x ^= table[A.words + 32 * i];
        asm volatile("" ::"v"(x));
    }
    for (uint32_t w = blockIdx.x;;) {
    const uint64_t base = place(w, ~A.qmask);
    // stream in: pieces tid + nt i of the tile, all in flight, then to LDS.
    // The index's high bits i are the tile's highest bits: a piece's offset
    // and LDS slot are the thread's plus (XOR) those of the bits set in i.
    constexpr int PB = EP == 2 ? RS - 1 : RS;                        // bits of i
    uint64_t gtop[PB];
    uint32_t stop[PB];
#pragma unroll
    for (int k = 0; k < PB; ++k) {
        gtop[k] = 1ull << A.top[kSlots - PB + k];
        stop[k] = tile_swizzle(1u << (A.L - PB + k));
    }
    if (!(A.direct & 1)) {
        if (live) {
            const uint64_t g0 = base + place(EP * tid, A.qmask);
            const uint32_t s0 = tile_swizzle(EP * tid);
            V16 v[NIT];
#pragma unroll
            for (int i = 0; i < NIT; ++i)
                v[i] = __builtin_nontemporal_load((const V16*)(psi + g0 + subset<PB>(gtop, i)));
#pragma unroll
            for (int i = 0; i < NIT; ++i) {
                const uint32_t s = s0 ^ (uint32_t)subset<PB>(stop, i);
                if constexpr (EP == 2) {
                    const V16 x = (s & 1) ? V16{v[i][2], v[i][3], v[i][0], v[i][1]} : v[i];
                    gst<V16>((s & ~1u) * ES, x);
                } else {
                    gst<V16>(s * ES, v[i]);
                }
            }
        }
        __syncthreads();
    }
    const uint32_t* __restrict__ p = table + A.words;
    Rec<R> cur, nxt;
    cur.load(p);
    for (uint32_t r = 0; r < A.nrounds; ++r) {
        uint32_t hd[RND_WORDS];
#pragma unroll
        for (int i = 0; i < (int)RND_WORDS; ++i) hd[i] = cur.w[i];
        const uint32_t nops = hd[8];
        p += RND_WORDS;
        nxt.load(p);
        uint32_t le = tid;                                     // a zero inserted at every slot
#pragma unroll
        for (int k = 0; k < RS; ++k) le = ((le & ~(hd[k] - 1)) << 1) | (le & (hd[k] - 1));
        uint32_t sl = tile_swizzle(le) * ES;
        uint32_t so[RS];
#pragma unroll
        for (int k = 0; k < RS; ++k) so[k] = hd[4 + k];
        uint64_t go[RS];
#pragma unroll
        for (int k = 0; k < RS; ++k) go[k] = 1ull << hd[9 + k];
        if (live) {
            if (r == 0 && (A.direct & 1)) {
                const uint64_t gb = base + place(le, A.qmask);
#pragma unroll
                for (int j = 0; j < kAmps; ++j) {
                    const V2 x = __builtin_nontemporal_load((const V2*)(psi + gb + subset<RS>(go, j)));
                    a[j].x = x[0];
                    a[j].y = x[1];
                }
            } else {
#pragma unroll
                for (int j = 0; j < kAmps; ++j) {
                    const V2 x = gld<V2>(sl ^ subset<RS>(so, j));
                    a[j].x = x[0];
                    a[j].y = x[1];
                }
            }
        }
        cur = nxt;
        for (uint32_t q = 0; q < nops; ++q) {
            const OpHead h{cur.w[0], cur.w[1], cur.w[2], cur.w[3], cur.w[4], cur.w[5], cur.w[6], cur.w[7]};
            const R* mv = (const R*)(p + sizeof(OpHead) / 4);
            p += h.code >> 8;
            nxt.load(p);
            if ((w & h.om) == h.ov && (le & h.tm) == h.tv) apply_op<R>(a, h, cur, mv, le, w);
            cur = nxt;
        }
        const bool last = r + 1 == A.nrounds;
        if (live) {
            if (last && (A.direct & 2)) {
                const uint64_t gb = base + place(le, A.qmask);
#pragma unroll
                for (int j = 0; j < kAmps; ++j)
                    __builtin_nontemporal_store(V2{a[j].x, a[j].y}, (V2*)(psi + gb + subset<RS>(go, j)));
            } else {
#pragma unroll
                for (int j = 0; j < kAmps; ++j) gst<V2>(sl ^ subset<RS>(so, j), V2{a[j].x, a[j].y});
            }
        }
        if (!(last && (A.direct & 2))) __syncthreads();
    }
    if constexpr (RDM) rdm_tile<R>(rr, ri, M, A.L);
    if (!(A.direct & 2) && live && (!RDM || M.store)) {
        const uint64_t g0 = base + place(EP * tid, A.qmask);
        const uint32_t s0 = tile_swizzle(EP * tid);
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const uint32_t s = s0 ^ subset<PB>(stop, i);
            V16 x;
            if constexpr (EP == 2) {
                x = gld<V16>((s & ~1u) * ES);
                if (s & 1) x = V16{x[2], x[3], x[0], x[1]};
            } else {
                x = gld<V16>(s * ES);
            }
            __builtin_nontemporal_store(x, (V16*)(psi + g0 + subset<PB>(gtop, i)));
        }
    }
    if constexpr (!RDM) break;
    w += gridDim.x;
    if (w >= M.ntiles) break;
    __syncthreads();                                           // the tile has been read: the next may come in
    }
    if constexpr (RDM) {
        // the waves' sums through LDS, in order
        __syncthreads();
        const uint32_t lane = tid & 63, wv = tid >> 6;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            gst<double>(8 * (512 * wv + 64 * q + lane), rr[q]);
            gst<double>(8 * (512 * wv + 64 * (q + 4) + lane), ri[q]);
        }
        __syncthreads();
        for (uint32_t e = tid; e < kRdmVals; e += blockDim.x) {
            double s = 0;
            for (uint32_t v = 0; v < blockDim.x / 64; ++v) s += gld<double>(8 * (512 * v + e));
            part[(size_t)blockIdx.x * kRdmVals + e] = s;
        }
    }
}

// The partials of nb workgroups, in order: 16 values per block.
__global__ __launch_bounds__(256) void k_rdm_final(const double* __restrict__ part, uint32_t nb,
                                                   double* __restrict__ out) {
    __shared__ double sh[16][17];
    const uint32_t v = threadIdx.x & 15, g = threadIdx.x >> 4;
    double s = 0;
    for (uint32_t b = g; b < nb; b += 16) s += part[(size_t)b * kRdmVals + 16 * blockIdx.x + v];
    sh[g][v] = s;
    __syncthreads();
    if (g == 0) {
        double r = 0;
        for (int i = 0; i < 16; ++i) r += sh[i][v];
        out[16 * blockIdx.x + v] = r;
    }
}

// =============================================================== scheduling
// A gate (or a merged run of uncontrolled one-target gates on one qubit) on
// physical bits.
struct GGate {
    LOp op;
    uint64_t xq;            // bits it does not act diagonally on (dense targets, moved bits)
    uint64_t zq;            // bits it acts diagonally on (controls, diagonal targets)
    double frac;            // share of the amplitudes its own kernel would touch
};

// A gate as its pass applies it (pass_gates).
struct PGate {
    const LOp* op;
    uint64_t xq, zq;
    double frac;
    bool lone;              // one-target, uncontrolled: a LAYER's, after pre
    double a, b;            // complex64: its rotation
    int npre;
    int bit[4];
    cd pre[4];
};

template <typename R>
struct Emit {
    std::vector<uint32_t>& tab;
    uint64_t qmask;
    uint64_t slots_phys;
    int rs;                                      // slots
    uint64_t slot_phys[kSlots];                  // ascending

    uint32_t slot_bits(uint64_t phys) const {
        uint32_t r = 0;
        for (int s = 0; s < rs; ++s)
            if (phys & slot_phys[s]) r |= 1u << s;
        return r;
    }
    // registers j whose slot bits match (mask, val) and with no bit of `zero`
    uint32_t regs(uint32_t mask, uint32_t val, uint32_t zero) const {
        uint32_t b = 0;
        for (uint32_t j = 0; j < 1u << rs; ++j)
            if ((j & mask) == val && !(j & zero)) b |= 1u << j;
        return b;
    }
    void record(OpHead h, const double* v, int nv) {
        const int words = (int)(sizeof(OpHead) / 4) + (int)(nv * sizeof(R) / 4);
        h.code |= (uint32_t)words << 8;
        const size_t at = tab.size();
        tab.resize(at + words);
        memcpy(&tab[at], &h, sizeof(h));
        for (int i = 0; i < nv; ++i) {
            const R x = (R)v[i];
            memcpy((char*)&tab[at + sizeof(OpHead) / 4] + i * sizeof(R), &x, sizeof(R));
        }
    }
    OpHead head(uint32_t code, uint64_t cmask, uint64_t cval, uint32_t zero) const {
        OpHead h{};
        h.code = code;
        h.jbits = regs(slot_bits(cmask), slot_bits(cval), zero);
        const uint64_t in = cmask & qmask & ~slots_phys;
        h.tm = local_bits(in, qmask);
        h.tv = local_bits(in & cval, qmask);
        h.om = tile_index_bits(cmask, qmask);
        h.ov = tile_index_bits(cval, qmask);
        return h;
    }
    // A diagonal op on slots alone: its factors per register multiplied into
    // f, or false.
    bool slot_factors(const LOp& o, cd* f) const {
        uint64_t bits = o.cls == OP_PHASE ? o.cond_mask : o.cmask;
        if (o.cls == OP_DIAG)
            for (int r = 0; r < o.k; ++r) bits |= 1ull << o.t[r];
        if ((o.cls != OP_PHASE && o.cls != OP_DIAG) || (bits & ~slots_phys)) return false;
        if (!f) return true;
        for (uint32_t j = 0; j < 1u << rs; ++j) {
            uint64_t at = 0;
            for (int s = 0; s < rs; ++s)
                if ((j >> s) & 1) at |= slot_phys[s];
            if (o.cls == OP_PHASE) {
                if ((at & o.cond_mask) == o.cond_val) f[j] *= o.phase;
            } else if ((at & o.cmask) == o.cmask) {
                int e = 0;
                for (int r = 0; r < o.k; ++r) e |= (int)((at >> o.t[r]) & 1) << r;
                f[j] *= o.m[e];
            }
        }
        return true;
    }
    // factors f (or none) and the gates (rotations or matrices) of the slots in mask
    void layer(const cd* f, uint32_t mask, const PGate* const* at) {
        double v[8 * kSlots + (2 << kSlots)] = {};
        int nv = 0;
        for (int k = 0; k < kSlots; ++k) {
            if (!((mask >> k) & 1)) continue;
            if constexpr (sizeof(R) == 4) {
                v[2 * k] = at[k]->a;
                v[2 * k + 1] = at[k]->b;
            } else {
                for (int e = 0; e < 4; ++e) {
                    v[nv++] = at[k]->op->m[e].real();
                    v[nv++] = at[k]->op->m[e].imag();
                }
            }
        }
        nv = layer_vals<R>(mask);
        if (f)
            for (uint32_t j = 0; j < 1u << rs; ++j) {
                v[nv++] = f[j].real();
                v[nv++] = f[j].imag();
            }
        OpHead h{};
        h.code = GP_LAYER;
        h.jbits = mask | (f ? kTable : 0);
        record(h, v, nv);
    }
    void signs(const std::vector<SignCond>& c) {
        OpHead h{};
        const size_t words = sizeof(OpHead) / 4 + c.size() * sizeof(SignCond) / 4;
        h.code = GP_SIGNS | (uint32_t)words << 8;
        h.jbits = (uint32_t)c.size();
        const size_t at = tab.size();
        tab.resize(at + words);
        memcpy(&tab[at], &h, sizeof(h));
        memcpy(&tab[at + sizeof(h) / 4], c.data(), c.size() * sizeof(SignCond));
    }
    // records it writes for one gate
    int gate(const LOp& o) {
        double v[128];
        switch (o.cls) {
            case OP_PHASE: {
                v[0] = o.phase.real();
                v[1] = o.phase.imag();
                record(head(GP_PHASE, o.cond_mask, o.cond_val, 0), v, 2);
                return 1;
            }
            case OP_DIAG: {
                const int D = 1 << o.k;
                auto bits = [&](int j) {
                    uint64_t b = 0;
                    for (int r = 0; r < o.k; ++r)
                        if ((j >> r) & 1) b |= 1ull << o.t[r];
                    return b;
                };
                bool par = true;
                for (int j = 0; j < D; ++j)
                    if (o.m[j] != o.m[pc((uint64_t)j) & 1]) par = false;
                if (par) {
                    const uint64_t tm = bits(D - 1);
                    OpHead h = head(GP_DIAG, o.cmask, o.cmask, 0);
                    const uint32_t ps = slot_bits(tm);
                    for (uint32_t j = 0; j < 1u << rs; ++j)
                        if (__builtin_popcount(j & ps) & 1) h.jbits |= 1u << (16 + j);
                    h.pt = local_bits(tm & qmask & ~slots_phys, qmask);
                    h.po = tile_index_bits(tm, qmask);
                    for (int i = 0; i < 2; ++i) {
                        v[2 * i] = o.m[i].real();
                        v[2 * i + 1] = o.m[i].imag();
                    }
                    record(h, v, 4);
                    return 1;
                }
                for (int j = 0; j < D; ++j) {                   // one factor per entry, each on its own amplitudes
                    v[0] = o.m[j].real();
                    v[1] = o.m[j].imag();
                    record(head(GP_PHASE, o.cmask | bits(D - 1), o.cmask | bits(j), 0), v, 2);
                }
                return D;
            }
            case OP_SWAPPAIR: {
                // the condition on the amplitude of a pair whose lowest
                // moved bit is 0 (the lowered op names the one with hbit 0)
                const uint64_t cm = o.cond_mask | o.hbit;
                uint64_t cv = o.cond_val & ~o.hbit;
                if (cm & cv & o.xmask & (~o.xmask + 1)) cv ^= cm & o.xmask;
                record(head(GP_MOVE + slot_bits(o.xmask), cm, cv, 0), v, 0);
                return 1;
            }
            default: break;
        }
        // dense: matrix rows and columns reordered to ascending slots
        const int D = 1 << o.k;
        uint64_t tm = 0;
        for (int r = 0; r < o.k; ++r) tm |= 1ull << o.t[r];
        int at[3] = {0, 0, 0};                                  // matrix bit of the s-th lowest target
        {
            int s = 0;
            for (uint64_t m = tm; m; m &= m - 1, ++s)
                for (int r = 0; r < o.k; ++r)
                    if (o.t[r] == __builtin_ctzll(m)) at[s] = r;
        }
        auto src = [&](int j) {
            int q = 0;
            for (int s = 0; s < o.k; ++s)
                if ((j >> s) & 1) q |= 1 << at[s];
            return q;
        };
        for (int i = 0; i < D; ++i)
            for (int j = 0; j < D; ++j) {
                const cd x = o.m[(size_t)src(i) * D + src(j)];
                v[2 * (i * D + j)] = x.real();
                v[2 * (i * D + j) + 1] = x.imag();
            }
        const uint32_t sm = slot_bits(tm);
        uint32_t code;
        if (o.k == 1) code = GP_D1 + __builtin_ctz(sm);
        else if (o.k == 3) code = GP_D3 + __builtin_ctz(~sm);      // (three slots: the code without slot 3)
        else code = GP_D2 + (sm == 3 ? 0 : sm == 5 ? 1 : sm == 9 ? 2 : sm == 6 ? 3 : sm == 10 ? 4 : 5);
        record(head(code, o.cmask, o.cmask, sm), v, 2 * D * D);
        return 1;
    }
};

// A pass's gates as its records take them.  Phases (diagonal one-target gates)
// wait on their bit, through gates that act diagonally on it and, as the
// inverse, through an uncontrolled X, until a gate that acts otherwise on the
// bit needs them applied (pre) or the pass ends; in a round the phases that
// are due on the slots become one factor per register.
//
// complex64: a unitary one-target gate is g diag(1, p) R diag(1, q), R a real
// rotation: R alone is a sequence of shears (op_turn), and the phases join
// those that wait.  U3 layers with CZs between them so take, per four gates,
// four rotations and one set of factors: 32 multiply-adds per amplitude pair
// against the 64 (and 12 moves) of four dense gates, which round more: lists
// of 200 to 400 gates on 10 qubits end 0.35 to 0.93 times as far from their
// matrices in 80 bits as with one dense kernel per gate.
//
// complex128: a one-target gate is its matrix.  A rotation and phases are not:
// their own rounding, and what a matrix of rounded entries lacks of a unitary
// one, is as large as the arithmetic's (the same lists ended 1.25 to 2.9 times
// as far off).  With the matrices, phases in long double and runs multiplied
// in long double it is 0.85 to 1.01 times (20 layers of U3 + CZ: 0.99e-15 of
// the norm, gate by gate 1.01e-15).
bool unit(const cd& x) { return std::fabs(std::norm(x) - 1.0) < 4e-15; }
cd mulc(const cd& a, const cd& b) {
    return cd(a.real() * b.real() - a.imag() * b.imag(), a.real() * b.imag() + a.imag() * b.real());
}

// A complex number that is carried along, in long double: rounded at every
// gate, the factor of all amplitudes alone would be off by as much as the
// gates' own arithmetic.
struct Phase {
    long double re = 1.0L, im = 0.0L;
    Phase() = default;
    Phase(long double r, long double i) : re(r), im(i) {}
    explicit Phase(const cd& x) : re(x.real()), im(x.imag()) {}
    bool one() const { return re == 1.0L && im == 0.0L; }
    Phase inv() const {
        const long double q = re * re + im * im;
        return Phase(re / q, -im / q);
    }
    void by(const Phase& o) {
        const long double r = re * o.re - im * o.im;
        im = re * o.im + im * o.re;
        re = r;
    }
    cd value() const { return cd((double)re, (double)im); }
};

struct Euler { Phase g, p, q; double c, s; };

// u = g diag(1, p) [c -s; s c] diag(1, q), for a unitary u with no zero entry.
bool euler(const std::vector<cd>& u, Euler& e) {
    Phase w[4];
    long double r[4];
    for (int i = 0; i < 4; ++i) {
        const long double x = u[i].real(), y = u[i].imag();
        r[i] = sqrtl(x * x + y * y);
        if (!(r[i] > 0.0L) || !(r[i] < 2.0L)) return false;
        w[i] = Phase(x / r[i], y / r[i]);
    }
    // (the mean of both columns: what the entries' rounding leaves of the
    // matrix's norm stays in g)
    const long double c2 = r[0] * r[3], s2 = r[1] * r[2], h = sqrtl(c2 + s2), tol = 4e-15L;
    if (!(fabsl(h - 1.0L) < tol) || !(fabsl(r[0] - r[3]) < tol) || !(fabsl(r[1] - r[2]) < tol)) return false;
    e.c = (double)(sqrtl(c2) / h);
    e.s = (double)(sqrtl(s2) / h);
    e.g = w[0];
    e.p = w[2];
    e.p.by(w[0].inv());
    e.q = Phase(-w[1].re, -w[1].im);
    e.q.by(w[0].inv());
    Phase d = e.g;
    d.by(e.p);
    d.by(e.q);
    if (!(fabsl(d.re - w[3].re) * r[3] < tol) || !(fabsl(d.im - w[3].im) * r[3] < tol)) return false;
    e.g.re *= h;
    e.g.im *= h;
    return true;
}

// (own: ops that are not the list's)
// split: one-target gates as rotations and phases (complex64).
std::vector<PGate> pass_gates(const std::vector<GGate>& G, const std::vector<int>& ops, std::deque<LOp>& own, bool split) {
    const cd one(1.0, 0.0), zero(0.0, 0.0);
    std::vector<PGate> out;
    out.reserve(ops.size() + 2);
    Phase ph[QVM_MAX_QUBITS], all;               // of the amplitudes with the bit set; of every amplitude
    for (int i : ops) {
        const LOp& o = G[i].op;
        if (o.cls == OP_PHASE && pc(o.cond_mask) == 1 && unit(o.phase)) {
            Phase f(o.phase);
            if (!o.cond_val) {
                all.by(f);
                f = f.inv();
            }
            ph[__builtin_ctzll(o.cond_mask)].by(f);
            continue;
        }
        if (o.cls == OP_DIAG && o.k == 1 && o.cmask == 0 && unit(o.m[0]) && unit(o.m[1])) {
            Phase f(o.m[1]);
            f.by(Phase(o.m[0]).inv());
            ph[o.t[0]].by(f);
            all.by(Phase(o.m[0]));
            continue;
        }
        PGate g{&o, G[i].xq, G[i].zq, G[i].frac, false, 0, 0, 0, {}, {}};
        const bool lone = o.cls == OP_DENSE && o.k == 1 && o.cmask == 0;
        Phase after;                             // what it leaves on its bit
        Euler e;
        if (lone && o.m[0] == zero && o.m[3] == zero && unit(o.m[1]) && unit(o.m[2])) {
            // diag(m1, m2) X: all m1, then m2 / m1 on the bit
            after = Phase(o.m[2]);
            after.by(Phase(o.m[1]).inv());
            all.by(Phase(o.m[1]));
            own.push_back(classify(1, o.t, 0, {zero, one, one, zero}));
            g.op = &own.back();
        } else if (lone && !split) {
            g.lone = true;
        } else if (lone && euler(o.m, e)) {
            g.lone = true;
            g.a = -e.s / (1.0 + e.c);
            g.b = e.s;
            all.by(e.g);
            ph[o.t[0]].by(e.q);
            after = e.p;
        }
        for (uint64_t m = g.xq; m; m &= m - 1) {
            const int b = __builtin_ctzll(m);
            if (ph[b].one()) continue;
            if (g.op->cls == OP_SWAPPAIR && g.xq == 1ull << b && !g.zq) {
                all.by(ph[b]);
                ph[b] = ph[b].inv();
                continue;
            }
            g.bit[g.npre] = b;
            g.pre[g.npre++] = ph[b].value();
            ph[b] = Phase();
        }
        if (!after.one()) ph[__builtin_ctzll(g.xq)].by(after);
        out.push_back(std::move(g));
    }
    auto phase = [&](uint64_t bits, const Phase& f) {
        LOp o{};
        o.cls = OP_PHASE;
        o.cond_mask = o.cond_val = bits;
        o.phase = f.value();
        own.push_back(std::move(o));
        return PGate{&own.back(), 0, bits, std::ldexp(1.0, -pc(bits)), false, 0, 0, 0, {}, {}};
    };
    for (int b = 0; b < QVM_MAX_QUBITS; ++b)
        if (!ph[b].one()) out.push_back(phase(1ull << b, ph[b]));
    if (!all.one()) out.insert(out.begin(), phase(0, all));
    return out;
}

// The records of a round: gates `now` of P in order.  A diagonal gate waits
// until a gate acts otherwise on one of its bits, and then all that wait are
// applied: the ones on slots alone as factors, the signs together, others one
// by one.  A rotation takes with it the rotations of the other slots that can
// come as early.  Fewer records, because choosing an op takes a dozen
// branches (the head of this file has the times with a record per gate).
// Returns how many.
constexpr size_t kMaxSigns = 64;                 // conditions of a record

template <typename R>
uint32_t round_records(Emit<R>& E, const std::vector<PGate>& P, const std::vector<int>& now, double amps,
                       double& flops) {
    const cd one(1.0, 0.0), neg(-1.0, 0.0);
    const int NA = 1 << E.rs;
    uint32_t nops = 0;
    std::vector<char> used(now.size(), 0), pre_used(now.size(), 0);
    std::vector<size_t> wait;                    // diagonal gates not applied yet
    uint64_t wait_bits = 0;
    cd f[1 << kSlots], fs[1 << kSlots];          // factors to be applied next; fs: the signs among them
    std::vector<SignCond> signs;
    int items = 0;                               // in f
    const LOp* single = nullptr;
    std::deque<LOp> hold;                        // the phases in f that no gate of P is
    auto clear = [&]() {
        std::fill(f, f + NA, one);
        std::fill(fs, fs + NA, one);
        signs.clear();
        hold.clear();
        items = 0;
        single = nullptr;
    };
    clear();
    auto factor = [&](const LOp& o) {            // o on slots alone
        const bool sign = o.cls == OP_PHASE && o.phase == neg;
        E.slot_factors(o, sign ? fs : f);
        if (sign) return;
        ++items;
        single = &o;
    };
    auto pres = [&](size_t k) {
        const PGate& q = P[now[k]];
        if (pre_used[k]) return;
        pre_used[k] = 1;
        for (int b = 0; b < q.npre; ++b) {
            LOp o{};
            o.cls = OP_PHASE;
            o.cond_mask = o.cond_val = 1ull << q.bit[b];
            o.phase = q.pre[b];
            hold.push_back(o);
            factor(hold.back());
        }
    };
    auto release = [&]() {
        for (size_t k : wait) {
            const LOp& o = *P[now[k]].op;
            if (E.slot_factors(o, nullptr)) {
                factor(o);
            } else if (o.cls == OP_PHASE && o.phase == neg) {
                const OpHead h = E.head(GP_SIGNS, o.cond_mask, o.cond_val, 0);
                signs.push_back(SignCond{h.jbits, h.tm, h.tv, h.om, h.ov, {0, 0, 0}});
            } else {
                nops += (uint32_t)E.gate(o);
                flops += 6.0 * amps * P[now[k]].frac;
            }
        }
        wait.clear();
        wait_bits = 0;
    };
    // the factors and signs due, with the one-target gates at of the slots in mask
    auto apply = [&](uint32_t mask, const PGate* const* at) {
        const bool one = items == 1 && !mask;    // one gate's factors: on its own registers only
        const bool tab = items && !one;
        uint32_t nb = 0;
        for (int j = 0; j < NA; ++j) {
            if (tab) f[j] = mulc(f[j], fs[j]);
            else if (fs[j] == neg) nb |= 1u << j;
        }
        if (nb) signs.push_back(SignCond{nb, 0, 0, 0, 0, {0, 0, 0}});
        for (size_t k = 0; k < signs.size(); k += kMaxSigns) {
            E.signs(std::vector<SignCond>(signs.begin() + k, signs.begin() + std::min(signs.size(), k + kMaxSigns)));
            ++nops;
        }
        if (one) {
            nops += (uint32_t)E.gate(*single);
            flops += 3.0 * amps;
        }
        if (tab || mask) {
            E.layer(tab ? f : nullptr, mask, at);
            ++nops;
            flops += (tab ? 6.0 : 0.0) * amps + (sizeof(R) == 4 ? 6.0 : 16.0) * amps * __builtin_popcount(mask);
        }
        clear();
    };
    for (size_t i = 0; i < now.size(); ++i) {
        if (used[i]) continue;
        const PGate& g = P[now[i]];
        if (!g.xq) {
            wait.push_back(i);
            wait_bits |= g.zq;
            continue;
        }
        if (wait_bits & g.xq) release();
        pres(i);
        uint64_t bx = g.lone ? 0 : g.xq, bz = (g.lone ? 0 : g.zq) | wait_bits;   // bits of gates passed over
        uint32_t mask = 0;
        const PGate* at[kSlots] = {};
        uint64_t taken = 0;                      // slots in mask
        auto take = [&](const PGate& q) {
            const int k = __builtin_ctz(E.slot_bits(q.xq));
            mask |= 1u << k;
            at[k] = &q;
            taken |= q.xq;
        };
        if (g.lone) take(g);
        for (size_t k = i + 1; k < now.size(); ++k) {
            if (used[k]) continue;
            const PGate& q = P[now[k]];
            if (g.lone && q.lone && !(q.xq & (bx | bz | taken))) {
                pres(k);
                take(q);
                used[k] = 1;
                continue;
            }
            // (factors due later that can be applied already)
            if (items && q.npre && !(q.xq & (bx | taken))) pres(k);
            if (items && !q.xq && !(q.zq & (bx | taken)) && E.slot_factors(*q.op, nullptr)) {
                factor(*q.op);
                used[k] = 1;
                continue;
            }
            bx |= q.xq;
            bz |= q.zq;
        }
        apply(mask, at);
        if (!g.lone) {
            nops += (uint32_t)E.gate(*g.op);
            const double touched = g.frac * amps;
            flops += g.op->cls == OP_DENSE ? touched * 8.0 * (1 << g.op->k) : g.op->cls == OP_SWAPPAIR ? 0.0 : 6.0 * touched;
        }
    }
    release();
    apply(0, nullptr);
    return nops;
}

// Records of the passes of one call: in the workspace's plan area, in stream
// order (when it is full, the next pass's records go to its start: the passes
// before have run by then).
struct PassBuf {
    uint32_t* dev;
    size_t cap, used = 0;
    explicit PassBuf(qvm_sv* sv)
        : dev((uint32_t*)(sv->work + sv->lay.plan_off)), cap(sv->lay.plan_bytes / 4) {}
};

// One pass over tiles of the bits in qmask: the gates ops of G in order, then,
// if asked, the reduced density matrix of the bits in measure (to rho_part:
// its workgroups' partials; *blocks: how many).
template <typename R>
qvm_status launch_pass(qvm_sv* sv, PassBuf& buf, const std::vector<GGate>& G, const std::vector<int>& ops,
                       uint64_t qmask, int rs, uint64_t measure = 0, double* rho_part = nullptr,
                       uint32_t* blocks = nullptr) {
    using T = typename GT<R>::T;
    const int n = sv->n, L = pc(qmask);
    PassArgs A{};
    A.qmask = qmask;
    A.L = (uint32_t)L;
    {
        int k = kSlots;
        for (int b = n - 1; k > 0; --b)
            if ((qmask >> b) & 1) A.top[--k] = (uint32_t)b;
    }
    std::vector<uint32_t> tab;
    std::deque<LOp> own;
    const std::vector<PGate> P = pass_gates(G, ops, own, sizeof(R) == 4);
    if (P.empty() && !measure) return QVM_OK;                   // (the gates undo each other)
    std::vector<int> left(P.size()), next, now;
    for (size_t i = 0; i < P.size(); ++i) left[i] = (int)i;
    double flops = 0;
    std::vector<uint64_t> round_slots;
    while (!left.empty()) {
        Sched s;
        uint64_t sm = 0;
        next.clear();
        now.clear();
        for (size_t q = 0; q < left.size(); ++q) {
            const PGate& g = P[left[q]];
            if ((s.bx & qmask) != qmask && s.free(g) && pc(sm | g.xq) <= rs) {
                sm |= g.xq;
                now.push_back(left[q]);
            } else {
                s.hold(g);
                next.push_back(left[q]);
            }
        }
        for (int b = n - 1; b >= 0 && pc(sm) < rs; --b)         // free slots: the highest tile bits
            if ((qmask >> b) & 1) sm |= 1ull << b;
        const size_t at = tab.size();
        tab.resize(at + RND_WORDS);
        Emit<R> E{tab, qmask, sm, rs, {}};
        {
            int k = 0;
            for (uint64_t m = sm; m; m &= m - 1) E.slot_phys[k++] = m & (~m + 1);
        }
        const uint32_t nops = round_records(E, P, now, (double)(1ull << n), flops);
        RoundHead rh{};
        for (int k = 0; k < rs; ++k) {
            rh.bit[k] = local_bits(E.slot_phys[k], qmask);
            rh.lds[k] = tile_swizzle(rh.bit[k]) * (uint32_t)sizeof(T);
            rh.phys[k] = (uint32_t)__builtin_ctzll(E.slot_phys[k]);
        }
        rh.nops = nops;
        memcpy(&tab[at], &rh, sizeof(rh));
        round_slots.push_back(sm);
        ++A.nrounds;
        left.swap(next);
    }
    const uint64_t low = (1ull << std::min<int>(GT<R>::C, n)) - 1;
    if (A.nrounds) {
        if (!(round_slots.front() & low)) A.direct |= 1;
        if (!measure && !(round_slots.back() & low)) A.direct |= 2;
    }
    tab.resize((tab.size() + 31) & ~size_t(31));
    if (buf.used + tab.size() + 64 > buf.cap) buf.used = 0;
    if (tab.size() + 64 > buf.cap) return fail(QVM_ENOMEM, "gate pass records exceed the workspace plan area");
    A.words = (uint32_t)buf.used;
    qvm_status st = put_words(sv, buf.dev + buf.used, tab.data(), tab.size());
    if (st) return st;
    buf.used += tab.size();
    A.lines = (uint32_t)(tab.size() / 32);
    const unsigned threads = std::max(64u, 1u << (L - rs));
    size_t lds = A.direct == 3 && A.nrounds == 1 ? 0 : sizeof(T) << L;
    unsigned grid = 1u << (n - L);
    RdmArgs M{};
    if (measure) {
        M.ntiles = grid;
        M.store = A.nrounds ? 1 : 0;
        int ks = 0, kc = 0;
        for (int b = 0; b < L; ++b) {
            uint64_t m = qmask;                                 // the b-th lowest tile bit
            for (int i = 0; i < b; ++i) m &= m - 1;
            const uint32_t at = tile_swizzle(1u << b) * (uint32_t)sizeof(T);
            if (measure & m & (~m + 1)) M.slot[ks++] = at;
            else M.col[kc++] = at;
        }
        grid = std::min(grid, kRdmBlocks);
        *blocks = grid;
        lds = std::max(lds, (size_t)(threads / 64) * kRdmVals * sizeof(double));
    }
    const int tok = prof_begin(sv);
    T* amps = (T*)sv->amps;
    if (measure) {
        if (rs == 3)
            hipLaunchKernelGGL((k_gate_pass<R, 3, true>), dim3(grid), dim3(threads), lds, sv->stream, amps, A, buf.dev,
                               M, rho_part);
        else
            hipLaunchKernelGGL((k_gate_pass<R, 4, true>), dim3(grid), dim3(threads), lds, sv->stream, amps, A, buf.dev,
                               M, rho_part);
    } else {
        if (rs == 3)
            hipLaunchKernelGGL((k_gate_pass<R, 3, false>), dim3(grid), dim3(threads), lds, sv->stream, amps, A,
                               buf.dev, M, rho_part);
        else
            hipLaunchKernelGGL((k_gate_pass<R, 4, false>), dim3(grid), dim3(threads), lds, sv->stream, amps, A,
                               buf.dev, M, rho_part);
    }
    QVM_LAUNCH_CHECK(sv);
    const double S = (double)(1ull << n) * sizeof(T);
    prof_end(sv, tok, measure ? PK_RDM1 : PK_GATES, M.store || !measure ? 2.0 * S : S, flops);
    return QVM_OK;
}

// Amplitudes per thread (as a power of two) and widest tile of a pass.
//
// Below 21 qubits a pass has few tiles, and the time of one wave through its
// gates counts: 8 amplitudes a thread instead of 16; from 13 to 16 qubits
// also tiles of 2^11, for twice the workgroups, as far as the passes that
// smaller tiles need (each two launches) pay.  From 21 qubits on the chip is
// full and the fewest passes win.  Measured, microseconds a call (calls one
// after another), tiles of 2^10 / 2^11 / 2^12 with 8 amplitudes | the widest
// with 16:
//   12 qubits, 200 mixed gates, complex64        161 / 140 / 128 | 153
//   14 qubits, 200 mixed gates, complex64        186 / 163 / 170 | 199
//   14 qubits, 200 mixed gates, complex128       182 / 178 / 198 | 219
//   16 qubits, 188 gates in layers, complex128    88 /  86 / 100 |  95
//   17 qubits, 200 mixed gates, complex64        200 / 187 / 185 | 227
//   18 qubits, 212 gates in layers, complex64    107 / 100 /  92 | 106
//   20 qubits, 236 gates in layers, complex128   172 / 162 / 138 | 136
//   22 qubits, 352 rotations, CNOTs, complex64   390 / 355 / 340 | 298
//   28 qubits, 332 gates in layers, complex128             28.1 ms | 26.6 ms
int pass_slots(int n) { return n <= 20 ? 3 : 4; }
template <typename R> int pass_width(int n) {
    return std::min(n, n > 20 ? GT<R>::LMAX : n > 12 && n <= 16 ? 11 : 12);
}

// Passes over the gates of G in order until none is left, or, with bits to
// measure, until one pass whose tile holds those bits takes all that are
// left and measures.
template <typename R>
qvm_status run_segment(qvm_sv* sv, const std::vector<GGate>& G, uint64_t measure = 0, double* rho_part = nullptr,
                       uint32_t* blocks = nullptr) {
    using T = typename GT<R>::T;
    const int n = sv->n, c = GT<R>::C, rs = pass_slots(n);
    const double S = (double)(1ull << n) * sizeof(T);
    PassBuf buf(sv);
    std::vector<char> done(G.size(), 0);
    std::vector<int> ops;
    size_t remaining = G.size(), first = 0;
    while (remaining || measure) {
        while (first < G.size() && done[first]) ++first;
        if (measure) {
            // (the tile holds the low bits, the measured ones and four more)
            const int L = std::min(n, n <= 20 ? 12 : GT<R>::LMAX);
            const uint64_t qmask = take_pass(G, done, first, n, L, c, measure, ops);
            if (ops.size() == remaining) return launch_pass<R>(sv, buf, G, ops, qmask, rs, measure, rho_part, blocks);
        }
        const uint64_t qmask = take_pass(G, done, first, n, pass_width<R>(n), c, 0, ops);
        // one gate's kernel costs a launch (3 us) and its share of the
        // state's traffic (5.5 TB/s), a pass two launches and all of the
        // traffic (5 TB/s): a few phases or moves on large states, and one
        // or two gates on small ones, stay one kernel each
        double each = 0;
        for (int i : ops) each += 3e-6 + 2.0 * S * G[i].frac / 5.5e12;
        const bool pass = ops.size() > 1 && each > 8e-6 + 2.0 * S / 5.0e12;
        for (int i : ops) done[i] = 1;
        remaining -= ops.size();
        if (pass) {
            qvm_status st = launch_pass<R>(sv, buf, G, ops, qmask, rs);
            if (st) return st;
            continue;
        }
        for (int i : ops) {
            qvm_status st = launch_op(sv, G[i].op);
            if (st) return st;
        }
    }
    return QVM_OK;
}

// A gate list under construction: runs of uncontrolled one-target gates on a
// bit become one gate (their product in long double, rounded once).
class ListBuilder {
  public:
    ListBuilder() { std::fill(open_, open_ + QVM_MAX_QUBITS, -1); }
    void one(int bit, const cd* m) {
        Phase x[4];
        for (int e = 0; e < 4; ++e) x[e] = Phase(m[e]);
        if (open_[bit] < 0) {
            open_[bit] = (int)items_.size();
            Item it{};
            it.bit = bit;
            std::copy(x, x + 4, it.m);
            items_.push_back(std::move(it));
            return;
        }
        Phase* r = items_[open_[bit]].m;
        Phase p[4];
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) {
                Phase y = x[2 * a], z = x[2 * a + 1];
                y.by(r[b]);
                z.by(r[2 + b]);
                p[2 * a + b] = Phase(y.re + z.re, y.im + z.im);
            }
        std::copy(p, p + 4, r);
    }
    void any(LOp op, uint64_t bits) {
        for (uint64_t m = bits; m; m &= m - 1) open_[__builtin_ctzll(m)] = -1;
        Item it{};
        it.bit = -1;
        it.op = std::move(op);
        items_.push_back(std::move(it));
    }
    size_t size() const { return items_.size(); }
    std::vector<GGate> finish() {
        std::vector<GGate> G;
        G.reserve(items_.size());
        std::vector<cd> u;
        for (Item& it : items_) {
            if (it.bit >= 0) {
                u.resize(4);
                for (int e = 0; e < 4; ++e) u[e] = it.m[e].value();
                it.op = classify(1, &it.bit, 0, u);
            }
            if (it.op.cls == OP_PHASE && it.op.phase == cd(1.0, 0.0)) continue;      // identity
            G.push_back(placed(std::move(it.op)));
        }
        return G;
    }

  private:
    struct Item {
        int bit;                                 // >= 0: a run of one-target gates with product m
        Phase m[4];
        LOp op;
    };
    static GGate placed(LOp op) {
        GGate g{std::move(op), 0, 0, 0};
        const LOp& o = g.op;
        uint64_t tm = 0;
        for (int r = 0; r < o.k; ++r) tm |= 1ull << o.t[r];
        switch (o.cls) {
            case OP_PHASE:
                g.zq = o.cond_mask;
                g.frac = std::ldexp(1.0, -pc(o.cond_mask));
                break;
            case OP_DIAG:
                g.zq = o.cmask | tm;
                g.frac = std::ldexp(1.0, -pc(o.cmask));
                break;
            case OP_SWAPPAIR:
                g.xq = o.xmask;
                g.zq = o.cond_mask & ~o.xmask;
                g.frac = std::ldexp(2.0, -pc(o.cond_mask | o.hbit));
                break;
            default:
                g.xq = tm;
                g.zq = o.cmask;
                g.frac = std::ldexp(1.0, -pc(o.cmask));
        }
        return g;
    }
    std::vector<Item> items_;
    int open_[QVM_MAX_QUBITS];
};

// Lowers one validated gate into the list; returns the physical bits it touches.
qvm_status add_gate(qvm_sv* sv, ListBuilder& B, const qvm_gate& g, std::vector<cd>& u) {
    qvm_status st = gate_matrix(g, u);
    if (st) return st;
    if (g.k == 1 && g.ctrl_mask == 0) {
        B.one(sv->perm[g.targets[0]], u.data());
        return QVM_OK;
    }
    uint64_t bits = phys_mask(sv, g.ctrl_mask);
    for (int r = 0; r < g.k; ++r) bits |= 1ull << sv->perm[g.targets[r]];
    B.any(lower(sv, g, u), bits);
    return QVM_OK;
}

qvm_status run_list(qvm_sv* sv, const std::vector<GGate>& G) {
    if (sv->n < kSlots || G.size() < 2) {
        for (const GGate& g : G) {
            const qvm_status st = launch_op(sv, g.op);
            if (st) return st;
        }
        return QVM_OK;
    }
    return sv->dt == QVM_C64 ? run_segment<float>(sv, G) : run_segment<double>(sv, G);
}

}  // namespace

qvm_status put_words(qvm_sv* sv, uint32_t* dst, const uint32_t* src, size_t n) {
    PutArgs pa;
    pa.pad = 0;
    for (size_t o = 0; o < n; o += kPutWords) {
        pa.dst = dst + o;
        pa.n = (uint32_t)std::min<size_t>(kPutWords, n - o);
        memcpy(pa.w, src + o, pa.n * 4);
        hipLaunchKernelGGL(k_put, dim3(1), dim3(256), 0, sv->stream, pa);
        QVM_LAUNCH_CHECK(sv);
    }
    return QVM_OK;
}

// The gate list in segments (a noisy run's groups likewise): bounds the host's
// work lists, the scans of the scheduler and a pass's records.
constexpr size_t kSegment = 4096;

qvm_status run_gates(qvm_sv* sv, const qvm_gate* gates, size_t n_gates) {
    std::vector<cd> u;
    for (size_t s0 = 0; s0 < n_gates; s0 += kSegment) {
        ListBuilder B;
        for (size_t i = s0; i < std::min(n_gates, s0 + kSegment); ++i) {
            const qvm_status st = add_gate(sv, B, gates[i], u);
            if (st) return st;
        }
        const qvm_status st = run_list(sv, B.finish());
        if (st) return st;
    }
    return QVM_OK;
}

// ============================================================ trajectories
// A noisy run (qvm_run_trajectory).  Every branching needs its qubit's
// density matrix at that point of the program, so one pass per branching
// reads the whole state, a host round trip chooses, and one more pass
// applies the chosen operator (0.42 ms per branching at 26 qubits, complex64).  But
// the reduced density matrix of up to four qubits determines everything that
// happens on those four until another qubit joins in: gates and chosen
// operators act on it as on the state.  So the program is cut into groups of
// steps that stay within four qubits; a group costs one pass, which applies
// the previous group's gates and chosen operators and measures this group's
// 16 x 16 matrix, and the host plays the group's branchings on that.
//
// 26 qubits, complex64, 262 gates, 264 branchings: 110 -> 14.2 ms in 40
// groups, 355 us each: the pass 285 (its traffic alone 167), the partials'
// sum 15, the copy and the host's part 50.
//
// Branchings keep their program order (each one's weights depend on the
// choices before it).  Gates without a branching that share no qubit with
// the open group do not change its matrix when they are unitary (every named
// gate): they wait until the group ends.
namespace {

// rho <- op rho op^H for an op on the 16-dimensional register.
struct Rho {
    double re[16][16], im[16][16];
    // rows: v_i <- sum_j m_ij v_j over the register positions pos (with controls cm)
    void rows(const cd* m, int k, const int* pos, uint32_t cm) {
        uint32_t tm = 0;
        for (int r = 0; r < k; ++r) tm |= 1u << pos[r];
        const int D = 1 << k;
        for (uint32_t b = 0; b < 16; ++b) {
            if ((b & tm) || (b & cm) != cm) continue;
            uint32_t ix[8];
            for (int j = 0; j < D; ++j) {
                ix[j] = b;
                for (int r = 0; r < k; ++r)
                    if ((j >> r) & 1) ix[j] |= 1u << pos[r];
            }
            for (int c = 0; c < 16; ++c) {
                double xr[8], xi[8];
                for (int j = 0; j < D; ++j) {
                    xr[j] = re[ix[j]][c];
                    xi[j] = im[ix[j]][c];
                }
                for (int i = 0; i < D; ++i) {
                    double sr = 0, si = 0;
                    for (int j = 0; j < D; ++j) {
                        const double a = m[i * D + j].real(), d = m[i * D + j].imag();
                        sr += a * xr[j] - d * xi[j];
                        si += a * xi[j] + d * xr[j];
                    }
                    re[ix[i]][c] = sr;
                    im[ix[i]][c] = si;
                }
            }
        }
    }
    void adjoint() {
        for (int i = 0; i < 16; ++i) {
            im[i][i] = -im[i][i];
            for (int j = 0; j < i; ++j) {
                std::swap(re[i][j], re[j][i]);
                const double t = im[i][j];
                im[i][j] = -im[j][i];
                im[j][i] = -t;
            }
        }
    }
    void apply(const cd* m, int k, const int* pos, uint32_t cm) {
        rows(m, k, pos, cm);
        adjoint();
        rows(m, k, pos, cm);
        adjoint();
    }
    // one position's 2 x 2 matrix: {rho_00, rho_11, Re rho_01, Im rho_01}
    void one(int pos, double* r) const {
        r[0] = r[1] = r[2] = r[3] = 0;
        for (uint32_t b = 0; b < 16; ++b) {
            if ((b >> pos) & 1) {
                r[1] += re[b][b];
            } else {
                const uint32_t d = b | 1u << pos;
                r[0] += re[b][b];
                r[2] += re[b][d];
                r[3] += im[b][d];
            }
        }
    }
};

template <typename R>
qvm_status measure_t(qvm_sv* sv, const std::vector<GGate>& G, uint64_t bits, Rho& rho) {
    // (partials and the result: the staging area)
    double* part = (double*)(sv->work + sv->lay.io_off);
    double* res = part + (size_t)kRdmBlocks * kRdmVals;
    uint32_t blocks = 0;
    qvm_status st = run_segment<R>(sv, G, bits, part, &blocks);
    if (st) return st;
    hipLaunchKernelGGL(k_rdm_final, dim3(kRdmVals / 16), dim3(256), 0, sv->stream, part, blocks, res);
    QVM_LAUNCH_CHECK(sv);
    double v[kRdmVals];
    QVM_HIP(sv, hipMemcpyAsync(v, res, sizeof(v), hipMemcpyDeviceToHost, sv->stream));
    QVM_HIP(sv, hipStreamSynchronize(sv->stream));
    // register q of lane l: row l / 16 + 4 q, column l % 16
    for (int i = 0; i < 16; ++i)
        for (int j = 0; j < 16; ++j) {
            auto at = [&](int row, int col) { return 64 * (row >> 2) + 16 * (row & 3) + col; };
            rho.re[i][j] = v[at(i, j)];
            rho.im[i][j] = v[256 + at(i, j)] - v[256 + at(j, i)];
        }
    return QVM_OK;
}

}  // namespace

// One branching on its own, from the state as it is: its branch and the chosen
// operator k, not yet applied.
static qvm_status branch_alone(qvm_sv* sv, int bit, const Channel& ch, double uniform, int32_t* branch, cd* k) {
    double r[4];
    qvm_status st = rd_rdm1(sv, bit, r);
    if (st) return st;
    int j = 0;
    st = choose_branch(r, ch.n_ops, ch.ops, uniform, &j, k, nullptr);
    if (st) return st;
    *branch = j;
    return QVM_OK;
}

qvm_status run_trajectory(qvm_sv* sv, const qvm_gate* gates, size_t n_gates, const Branching* br,
                          const size_t* first, const std::vector<Channel>& chans, const double* uniforms,
                          int32_t* branches) {
    std::vector<cd> u;
    auto bits_of = [&](size_t i) {
        const qvm_gate& g = gates[i];
        uint64_t b = phys_mask(sv, g.ctrl_mask);
        for (int r = 0; r < g.k; ++r) b |= 1ull << sv->perm[g.targets[r]];
        for (size_t q = first[i]; q < first[i + 1]; ++q) b |= 1ull << sv->perm[br[q].qubit];
        return b;
    };
    std::vector<size_t> body, later;             // the group's gates, and those passed over
    ListBuilder B;                               // what the next pass applies
    size_t pos = 0;
    qvm_status st = QVM_OK;
    while (pos < n_gates) {
        // the next group: gates without noise up to the first branching, then
        // what stays within four qubits
        body.clear();
        later.clear();
        uint64_t grp = 0, held = 0;
        size_t i = pos, items = 0, nbr = 0;      // (a branching adds at most one item per qubit)
        for (; i < n_gates && items < kSegment; ++i) {
            const uint64_t b = bits_of(i);
            const bool noisy = first[i + 1] > first[i];
            if (!grp && !noisy) {
                if ((st = add_gate(sv, B, gates[i], u))) return st;
                if (B.size() >= kSegment) {
                    if ((st = run_list(sv, B.finish()))) return st;
                    B = ListBuilder();
                }
                continue;
            }
            if (!noisy && !(b & grp) && gates[i].kind != QVM_G_MATRIX) {
                later.push_back(i);
                held |= b;
                ++items;
                continue;
            }
            if ((b & held) || pc(grp | b) > kSlots || sv->n < kSlots) break;
            grp |= b;
            body.push_back(i);
            items += 1 + std::min<size_t>(kSlots, first[i + 1] - first[i]);
            nbr += first[i + 1] - first[i];
        }
        pos = i;
        if (body.empty()) {
            if (pos == n_gates) break;
            // a noisy gate on more than four qubits, or fewer than four in all
            if ((st = add_gate(sv, B, gates[pos], u)) || (st = run_list(sv, B.finish()))) return st;
            B = ListBuilder();
            for (size_t q = first[pos]; q < first[pos + 1]; ++q) {
                const int bit = sv->perm[br[q].qubit];
                std::vector<cd> k(4);
                if ((st = branch_alone(sv, bit, chans[br[q].channel], uniforms[q], branches + q, k.data()))) return st;
                if ((st = launch_op(sv, classify(1, &bit, 0, k)))) return st;
            }
            ++pos;
            continue;
        }
        // A branching that no other one shares a measurement with: its qubit's
        // 2 x 2 matrix takes a read of the state and is cheaper than a
        // measuring pass (one H and its branching, complex64, one call: 24
        // qubits 117 against 153 us, 26 qubits 378 against 459; five with a
        // layer of gates before each: even, -3 to +4%).
        if (nbr == 1) {
            for (size_t gi : body) {
                if ((st = add_gate(sv, B, gates[gi], u))) return st;
                if (first[gi] == first[gi + 1]) continue;
                if ((st = run_list(sv, B.finish()))) return st;
                B = ListBuilder();
                const size_t q = first[gi];
                const int bit = sv->perm[br[q].qubit];
                cd k[4];
                if ((st = branch_alone(sv, bit, chans[br[q].channel], uniforms[q], branches + q, k))) return st;
                B.one(bit, k);
            }
            for (size_t gi : later)
                if ((st = add_gate(sv, B, gates[gi], u))) return st;
            continue;
        }
        uint64_t m = grp;
        for (int q = sv->n - 1; q >= 0 && pc(m) < kSlots; --q) m |= 1ull << q;
        Rho rho;
        const std::vector<GGate> G = B.finish();
        st = sv->dt == QVM_C64 ? measure_t<float>(sv, G, m, rho) : measure_t<double>(sv, G, m, rho);
        if (st) return st;
        B = ListBuilder();
        auto reg = [&](int bit) { return pc(m & ((1ull << bit) - 1)); };
        for (size_t gi : body) {
            const qvm_gate& g = gates[gi];
            if ((st = gate_matrix(g, u))) return st;
            int p[3];
            uint32_t cm = 0;
            for (int r = 0; r < g.k; ++r) p[r] = reg(sv->perm[g.targets[r]]);
            for (uint64_t c = phys_mask(sv, g.ctrl_mask); c; c &= c - 1) cm |= 1u << reg(__builtin_ctzll(c));
            rho.apply(u.data(), g.k, p, cm);
            if ((st = add_gate(sv, B, g, u))) return st;
            for (size_t q = first[gi]; q < first[gi + 1]; ++q) {
                const int bit = sv->perm[br[q].qubit], rp = reg(bit);
                const Channel& ch = chans[br[q].channel];
                double r[4];
                rho.one(rp, r);
                int j = 0;
                cd k[4];
                if ((st = choose_branch(r, ch.n_ops, ch.ops, uniforms[q], &j, k, nullptr))) return st;
                branches[q] = j;
                rho.apply(k, 1, &rp, 0);
                B.one(bit, k);
            }
        }
        for (size_t gi : later)
            if ((st = add_gate(sv, B, gates[gi], u))) return st;
    }
    return run_list(sv, B.finish());
}

}  // namespace qvm
