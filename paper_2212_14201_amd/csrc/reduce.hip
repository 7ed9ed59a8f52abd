// Readout kernels: norm, probabilities and marginals, <Z_q> for every qubit,
// Pauli-string expectations, sampling, amplitude copies.
//
// All sums are accumulated in double precision (single-precision amplitudes
// are widened before squaring) over a fixed grid and reduced in a fixed
// order, so every readout is bitwise reproducible run to run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "internal.hpp"

namespace qvm {

template <typename R> struct C2r;
template <> struct C2r<float> { using T = float2; };
template <> struct C2r<double> { using T = double2; };

struct Perm {
    int n;
    int identity;
    int p[QVM_MAX_QUBITS];            // logical -> physical bit
};

static Perm make_perm(const qvm_sv* sv) {
    Perm P{};
    P.n = sv->n;
    P.identity = 1;
    for (int q = 0; q < sv->n; ++q) {
        P.p[q] = sv->perm[q];
        if (sv->perm[q] != q) P.identity = 0;
    }
    return P;
}

__device__ __forceinline__ uint64_t to_phys(uint64_t l, const Perm& P) {
    if (P.identity) return l;
    uint64_t r = 0;
    for (int q = 0; q < P.n; ++q) r |= ((l >> q) & 1ull) << P.p[q];
    return r;
}

template <typename T>
__device__ __forceinline__ double prob(const T& v) {
    double x = (double)v.x, y = (double)v.y;
    return x * x + y * y;
}

// Sum over a 256-thread block; the result is valid in thread 0.
__device__ double block_sum256(double v, double* sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Streaming shape of the readouts (measured on a 28-qubit complex64 state, 2
// GiB): a block takes consecutive 16-byte pieces, one per thread and
// iteration, several iterations' loads in flight.
typedef float rf4 __attribute__((ext_vector_type(4)));
typedef double rd2 __attribute__((ext_vector_type(2)));
typedef double rd4 __attribute__((ext_vector_type(4)));
template <typename R> struct Piece;
template <> struct Piece<float> {
    using V = rf4;
    static constexpr int EP = 2, LB = 9;         // amplitudes per piece, index bits of a block's row of pieces
};
template <> struct Piece<double> {
    using V = rd2;
    static constexpr int EP = 1, LB = 8;
};
template <typename V, typename T>
__device__ __forceinline__ V ld_piece(const T* p) { return __builtin_nontemporal_load((const V*)p); }
// amplitude e of a piece
__device__ __forceinline__ double2 amp(const rf4& v, int e) { return make_double2(v[2 * e], v[2 * e + 1]); }
__device__ __forceinline__ double2 amp(const rd2& v, int) { return make_double2(v[0], v[1]); }
__device__ __forceinline__ double sq(const double2& v) { return v.x * v.x + v.y * v.y; }

// ------------------------------------------------------------ norm / scale
template <typename R>
__global__ __launch_bounds__(256) void k_norm_partial(const typename C2r<R>::T* __restrict__ psi,
                                                      uint64_t N, double* __restrict__ part) {
    using V = typename Piece<R>::V;
    constexpr int EP = Piece<R>::EP;
    __shared__ double sh[4];
    const uint64_t np = N / EP, rows = (np + 255) / 256, per = (rows + gridDim.x - 1) / gridDim.x;
    const uint64_t r0 = min(blockIdx.x * per, rows), r1 = min(r0 + per, rows);
    double s = 0;
    // (a block's pieces one row after the other: 28 qubits, complex64, 330 us;
    // strided over the grid 390)
    for (uint64_t r = r0; r < r1; r += 8) {
        V v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint64_t i = (r + k) * 256 + threadIdx.x;
            v[k] = r + k < r1 && i < np ? ld_piece<V>(psi + EP * i) : V{};
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int e = 0; e < EP; ++e) s += sq(amp(v[k], e));
    }
    double r = block_sum256(s, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
}

// Column v of the partials (nb each, in order) into res[v]: one block per
// value.  (One block for all values, each a strided column: 50 us for the 29
// values of a 28-qubit <Z> readout, now 4.)
__global__ __launch_bounds__(256) void k_final(const double* __restrict__ part, uint32_t nb,
                                               double* __restrict__ res) {
    __shared__ double sh[4];
    const double* col = part + (size_t)blockIdx.x * nb;
    double s = 0;
    for (uint32_t b = threadIdx.x; b < nb; b += 256) s += col[b];
    const double r = block_sum256(s, sh);
    if (threadIdx.x == 0) res[blockIdx.x] = r;
}

// One 16-byte piece per thread, nontemporal both ways: the shape that
// streams fastest (2 GiB: 725 -> 660 us against 8-byte ordinary accesses).
template <typename R>
__global__ __launch_bounds__(256) void k_scale(typename C2r<R>::T* __restrict__ psi, uint64_t N,
                                               R f) {
    using V = typename Piece<R>::V;
    constexpr int EP = Piece<R>::EP;
    const uint64_t np = N / EP, stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < np; i += stride)
        __builtin_nontemporal_store(ld_piece<V>(psi + EP * i) * f, (V*)(psi + EP * i));
}

// ----------------------------------------------------- <Z_q> for every q
// Block b of 2^bb takes the indices whose top bb bits are b, thread t in
// iteration it the piece (it << 8) + t of them.  Bits below LB are the
// thread's, the ib bits above the iteration's: eight iterations at a time
// give the sums of their three low bits from one tree, the bits above add
// the tree's total, so an amplitude costs about three additions whatever n
// (one per bit from 19 up, and a load of 8 bytes at a time, took 758 us for
// 2 GiB; now 335, HBM's time).  Columns: 0 the total, 1 + q the sum over indices
// with bit q set, q < LB + ib; the block bits' sums follow from the totals.
constexpr int kZIter = QVM_MAX_QUBITS - 8 - 11;      // iteration bits, at most
template <typename R>
__global__ __launch_bounds__(256) void k_zall_partial(const typename C2r<R>::T* __restrict__ psi,
                                                      int n, int ib, double* __restrict__ part) {
    using V = typename Piece<R>::V;
    constexpr int EP = Piece<R>::EP, LB = Piece<R>::LB;
    __shared__ double sh[4][kZIter + 8];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const bool live = n >= LB || EP * t < (1u << n);
    const auto* P = psi + ((uint64_t)blockIdx.x << (LB + ib)) + (uint64_t)EP * t;
    double total = 0, odd = 0, mid[kZIter];
#pragma unroll
    for (int k = 0; k < kZIter; ++k) mid[k] = 0;
    if (live) {
        if (ib >= 3) {
            for (uint64_t it = 0; it < (1ull << ib); it += 8) {
                V v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = ld_piece<V>(P + ((it + k) << LB));
                double x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    x[k] = sq(amp(v[k], 0));
                    if constexpr (EP == 2) {
                        const double o = sq(amp(v[k], 1));
                        odd += o;
                        x[k] += o;
                    }
                }
                const double a = x[0] + x[1], b = x[2] + x[3], c = x[4] + x[5], d = x[6] + x[7];
                mid[0] += (x[1] + x[3]) + (x[5] + x[7]);
                mid[1] += b + d;
                mid[2] += c + d;
                const double s = (a + b) + (c + d);
                total += s;
#pragma unroll
                for (int k = 3; k < kZIter; ++k)
                    if (k < ib && ((it >> k) & 1)) mid[k] += s;
            }
        } else {
            for (uint32_t it = 0; it < (1u << ib); ++it) {
                const V v = ld_piece<V>(P + ((uint64_t)it << LB));
                double x = sq(amp(v, 0));
                if constexpr (EP == 2) {
                    const double o = sq(amp(v, 1));
                    odd += o;
                    x += o;
                }
                total += x;
                if (it & 1) mid[0] += x;
                if (it & 2) mid[1] += x;
            }
        }
    }
    auto wsum = [&](double v) {
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
        return v;
    };
    // per wave: [0] total, [1] odd amplitudes, [2..7] lane bits, [8 + k] iteration bits
    {
        const double v = wsum(total), o = EP == 2 ? wsum(odd) : 0.0;
        if (lane == 0) {
            sh[wave][0] = v;
            sh[wave][1] = o;
        }
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double v = wsum(((lane >> k) & 1) ? total : 0.0);
        if (lane == 0) sh[wave][2 + k] = v;
    }
#pragma unroll
    for (int k = 0; k < kZIter; ++k)
        if (k < ib) {
            const double v = wsum(mid[k]);
            if (lane == 0) sh[wave][8 + k] = v;
        }
    __syncthreads();
    const int nv = 1 + (n < LB ? n : LB) + ib;
    if ((int)t < nv) {
        double r;
        const int q = (int)t - 1, tb = q - (EP - 1);            // index bit, thread bit
        auto all = [&](int i) { return (sh[0][i] + sh[1][i]) + (sh[2][i] + sh[3][i]); };
        if (q < 0) r = all(0);
        else if (q >= LB) r = all(8 + q - LB);
        else if (tb < 0) r = all(1);
        else if (tb < 6) r = all(2 + tb);
        else r = tb == 6 ? sh[1][0] + sh[3][0] : sh[2][0] + sh[3][0];
        part[(size_t)t * gridDim.x + blockIdx.x] = r;
    }
}

// res[0] = total, res[1 + q] for every bit q: own columns below `cols`, the
// totals of the blocks with the bit set above.
__global__ __launch_bounds__(256) void k_zall_final(const double* __restrict__ part, uint32_t nb, int cols,
                                                    double* __restrict__ res) {
    __shared__ double sh[4];
    const int v = blockIdx.x;
    const double* col = part + (v < cols ? (size_t)v * nb : 0);
    const uint32_t need = v < cols ? 0u : 1u << (v - cols);
    double s = 0;
    for (uint32_t b = threadIdx.x; b < nb; b += 256)
        if ((b & need) == need) s += col[b];
    const double r = block_sum256(s, sh);
    if (threadIdx.x == 0) res[v] = r;
}

// ----------------------------------------------------- Pauli expectations
// For x = 0:   acc_t = sum_i p_i (-1)^{|z_t & i|}.
// For x != 0:  over pairs (i, i^x) with i's highest x bit 0, a =
//              conj(psi_{i^x}) psi_i, acc_t = sum (-1)^{|z_t & i|} * (Re a if
//              |x&z_t| even else Im a); the host applies the factor +-2 given
//              by |x & z_t| mod 4.
// A job is one x with two sets of up to 16 terms of one kind (Re or Im) each;
// one launch takes all jobs (grid y), so a sum of many strings costs one
// launch, one reduction and one copy to the host instead of three per x.
// The signs are a matrix: the 16 terms of a set times the wave's 64 values
// of one iteration are one FP64 MFMA per value of a piece, whose A operand
// (row = term, 4 columns = lane bits 4, 5) holds +-1 and whose 16 output
// columns are the lane's low bits, signed and summed once at the end.  A
// term then costs 4 matrix cycles per wave and piece value instead of a
// popcount, a select and an addition per amplitude.  27 Z-strings: 28 qubits
// complex64 2,171 -> 575 us (the matrix unit alone 220, the conversions and
// squares beside it), 27 qubits complex128 390 us (HBM 335); 40 random
// strings of 21 qubits 1,400 -> 85 us.
struct PauliJob {
    uint64_t x;
    uint32_t nt[2], im[2];           // terms and kind (1: Im) of the two sets
    uint32_t out, pad;               // first term's column of the partials
    uint64_t z[32];                  // set s at 16 s; unused entries 0
};
static_assert(sizeof(PauliJob) == 288 && sizeof(PauliJob) % 4 == 0, "records of whole words");

template <typename R>
__global__ __launch_bounds__(256) void k_pauli_partial(const typename C2r<R>::T* __restrict__ psi, int n,
                                                       const PauliJob* __restrict__ jobs,
                                                       double* __restrict__ part) {
    using V = typename Piece<R>::V;
    constexpr int EP = Piece<R>::EP, LB = Piece<R>::LB;
    __shared__ double sh[4][32];
    const PauliJob* __restrict__ J = jobs + blockIdx.y;
    const uint64_t x = J->x;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    // pairs: the highest bit of x is taken out of the enumeration where it
    // is above the block's row, else its upper half contributes nothing
    const int h = x ? 63 - __builtin_clzll(x) : -1;
    const bool cut = h >= LB;
    const int ebits = n - (cut ? 1 : 0);                         // enumeration bits
    const uint32_t low = EP * t;                                 // the thread's low index bits
    const bool live = ebits >= LB || low < (1u << ebits);
    const uint64_t rows = ebits > LB ? 1ull << (ebits - LB) : 1;
    const uint64_t per = (rows + gridDim.x - 1) / gridDim.x;
    const uint64_t r0 = min((uint64_t)blockIdx.x * per, rows), r1 = min(r0 + per, rows);
    // A operand of set s: lane's term l % 16, its sign over the lane bits 4,
    // 5 and the wave bits (index bits above EP's); the row part per iteration
    const uint64_t zt[2] = {J->z[lane & 15], J->z[16 + (lane & 15)]};
    const uint32_t lhi = low & ~(uint32_t)(16 * EP - 1);
    uint32_t sg[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) sg[s] = __popc((uint32_t)zt[s] & lhi);
    rd4 acc[2] = {rd4{0, 0, 0, 0}, rd4{0, 0, 0, 0}};
    const bool two = J->nt[1] != 0;
    const bool im0 = J->im[0] != 0, im1 = J->im[1] != 0;
    const uint64_t hm = cut ? (1ull << h) - 1 : ~0ull;
    auto row_index = [&](uint64_t r) {                           // r << LB with a zero at bit h
        const uint64_t i = r << LB;
        return cut ? ((i & ~hm) << 1) | (i & hm) : i;
    };
    constexpr int U = 2;                                         // iterations in flight
    for (uint64_t r = r0; r < r1; r += U) {
        V vi[U], vj[U];
        uint64_t ri[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            ri[k] = row_index(r + k < r1 ? r + k : r0);
            if (live && r + k < r1) {
                const uint64_t i = ri[k] | low;
                vi[k] = x ? *(const V*)(psi + i) : ld_piece<V>(psi + i);
                if (x) vj[k] = *(const V*)(psi + ((i ^ x) & ~(uint64_t)(EP - 1)));
            } else {
                vi[k] = V{};
                vj[k] = V{};
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (r + k >= r1) break;
            double sgn[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const uint32_t c = sg[s] + __popcll(zt[s] & ri[k]);
                sgn[s] = __hiloint2double(0x3ff00000 ^ (int)(c << 31), 0);
            }
#pragma unroll
            for (int e = 0; e < EP; ++e) {
                const double2 a = amp(vi[k], e);
                double re, im = 0;
                if (!x) {
                    re = sq(a);
                } else {
                    const double2 b = EP == 2 && (x & 1) ? amp(vj[k], EP - 1 - e) : amp(vj[k], e);
                    re = b.x * a.x + b.y * a.y;                  // Re conj(psi_j) psi_i
                    im = b.x * a.y - b.y * a.x;                  // Im conj(psi_j) psi_i
                    if (!cut && (((low | e) >> h) & 1)) re = im = 0;
                }
                if (e == 1) {
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        sgn[s] = __hiloint2double(__double2hiint(sgn[s]) ^ (int)((uint32_t)zt[s] << 31), 0);
                }
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(sgn[0], im0 ? im : re, acc[0], 0, 0, 0);
                if (two) acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(sgn[1], im1 ? im : re, acc[1], 0, 0, 0);
            }
        }
    }
    // register r of lane l: row l / 16 + 4 r, column l % 16 (the thread's low four bits)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t row = (lane >> 4) + 4 * r;
            const uint32_t c = __popc((uint32_t)J->z[16 * s + row] & (EP * (lane & 15)));
            double v = (c & 1) ? -acc[s][r] : acc[s][r];
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            if ((lane & 15) == 0) sh[wave][16 * s + row] = v;
        }
    __syncthreads();
    if (t < 32) {
        const uint32_t s = t >> 4, i = t & 15;
        if (i < J->nt[s])
            part[(size_t)(J->out + (s ? J->nt[0] : 0) + i) * gridDim.x + blockIdx.x] =
                (sh[0][t] + sh[1][t]) + (sh[2][t] + sh[3][t]);
    }
}

// --------------------------------------------------------- probabilities
template <typename R>
__global__ __launch_bounds__(256) void k_probs(const typename C2r<R>::T* __restrict__ psi,
                                               uint64_t first, uint64_t cnt, Perm P,
                                               double* __restrict__ out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < cnt; j += stride)
        out[j] = prob(psi[to_phys(first + j, P)]);
}

// Marginals.  A block takes whole rows of 2^LB consecutive amplitudes (one
// piece per thread) whose index bits above the row it fixes: every marginal
// qubit above the row, and as many others as give 2,048 blocks; it runs
// over the bits that are left, none of them a marginal qubit, so a thread
// adds into one register per amplitude of its piece, and only the row's own
// marginal qubits are sorted out, once, in LDS.  Reads are whole lines in
// any layout (one block per bucket read an amplitude at a time, its bits
// spread one by one: 670 us for 8 of 28 qubits, 3,970 for 16 of 30; now 335
// and 1,200, 6.4 and 7.1 TB/s).
struct MargArgs {
    uint64_t qhi, seg, iter;          // index bits above the row: marginal qubits, other block bits, the rest
    uint32_t qlo;                     // marginal qubits inside the row
    uint32_t mh, segs, niter;         // marginal qubits above the row; 2^(seg bits); 2^(iter bits)
    uint8_t lo_out[12], hi_out[24];   // output bit of the k-th lowest bit of qlo / qhi
    uint8_t hi_run;                   // hi_out ascends one by one
};

// x's bits on the set bits of mask, ascending, a run of them at a time.
__device__ __forceinline__ uint64_t place_bits(uint64_t x, uint64_t mask) {
    uint64_t r = 0;
    while (mask) {
        const uint64_t low = mask & (~mask + 1);
        const uint64_t run = ((mask + low) & ~mask) - low;
        r |= (x * low) & run;
        x >>= __builtin_popcountll(run);
        mask &= ~run;
    }
    return r;
}

template <typename R>
__global__ __launch_bounds__(256) void k_marg_partial(const typename C2r<R>::T* __restrict__ psi, int n,
                                                      MargArgs a, double* __restrict__ part) {
    using V = typename Piece<R>::V;
    constexpr int EP = Piece<R>::EP, LB = Piece<R>::LB;
    __shared__ double sum[1 << LB];
    const uint32_t t = threadIdx.x;
    const uint32_t qi = blockIdx.x & ((1u << a.mh) - 1), seg = blockIdx.x >> a.mh;
    const uint32_t len = n < LB ? 1u << n : 1u << LB;            // amplitudes of a row
    const uint64_t base = place_bits(qi, a.qhi) | place_bits(seg, a.seg);
    const bool live = EP * t < len;
    double acc[EP];
#pragma unroll
    for (int e = 0; e < EP; ++e) acc[e] = 0;
    if (live) {
        uint64_t ix = 0;                                         // the iteration's bits in place
        for (uint32_t it = 0; it < a.niter; it += 4) {
            V v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = it + k < a.niter ? ld_piece<V>(psi + (base | ix | EP * t)) : V{};
                ix = ((ix | ~a.iter) + 1) & a.iter;              // the next subset of the bits
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < EP; ++e) acc[e] += sq(amp(v[k], e));
        }
    }
    // fold the row's other bits: a piece's and a wave's in registers, the waves'
    // when the buckets are read.  (The 16 highest of 24 qubits, complex128,
    // 65,536 blocks of one row each: 260 us a level at a time in LDS, 220 so, 104
    // with the block's bits placed a run at a time instead of one by one.)
    if (EP == 2 && !(a.qlo & 1)) acc[0] += acc[EP - 1];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        if ((a.qlo >> (EP - 1 + k)) & 1) continue;
#pragma unroll
        for (int e = 0; e < EP; ++e) acc[e] += __shfl_xor(acc[e], 1 << k, 64);
    }
#pragma unroll
    for (int e = 0; e < EP; ++e) sum[EP * t + e] = acc[e];
    __syncthreads();
    constexpr uint32_t W0 = EP << 6, W1 = EP << 7;
    uint32_t jh = a.hi_run ? qi << a.hi_out[0] : 0;
    if (!a.hi_run)
        for (uint32_t k = 0; k < a.mh; ++k) jh |= ((qi >> k) & 1u) << a.hi_out[k];
    const uint32_t nlo = 1u << __popc(a.qlo);
    for (uint32_t i = t; i < nlo; i += 256) {
        uint32_t j = jh, e = 0, x = i, k = 0;
        for (uint32_t m = a.qlo; m; m &= m - 1, ++k, x >>= 1)
            if (x & 1) {
                e |= m & (~m + 1);
                j |= 1u << a.lo_out[k];
            }
        double v = sum[e];
        if (!(a.qlo & W0)) v += sum[e | W0];
        if (!(a.qlo & W1)) {
            double x = sum[e | W1];
            if (!(a.qlo & W0)) x += sum[e | W1 | W0];
            v += x;
        }
        part[(size_t)j * a.segs + seg] = v;
    }
}

__global__ __launch_bounds__(256) void k_marg_final(const double* __restrict__ part,
                                                    uint64_t nb, uint32_t segs,
                                                    double* __restrict__ out) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nb) return;
    double s = 0;
    for (uint32_t k = 0; k < segs; ++k) s += part[j * segs + k];
    out[j] = s;
}

// -------------------------------------------------------------- sampling
// The chunk sums (2^clog consecutive logical indices each) are the marginal
// over the logical qubits from clog up.

// Exclusive prefixes of the chunk sums inside groups of 1,024 chunks (infinity
// for a chunk of no probability: it is never drawn), and the groups' totals (at
// most 256).
constexpr uint32_t kGroup = 1024;
__global__ __launch_bounds__(256) void k_scan_chunks(const double* __restrict__ csum, uint64_t nchunks,
                                                     double* __restrict__ prefix, double* __restrict__ gtot) {
    __shared__ double sh[256];
    const uint64_t c0 = (uint64_t)blockIdx.x * kGroup + 4 * threadIdx.x;
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = c0 + k < nchunks ? csum[c0 + k] : 0.0;
    sh[threadIdx.x] = (v[0] + v[1]) + (v[2] + v[3]);
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const double u = threadIdx.x >= (unsigned)off ? sh[threadIdx.x - off] : 0.0;
        __syncthreads();
        sh[threadIdx.x] += u;
        __syncthreads();
    }
    double run = threadIdx.x ? sh[threadIdx.x - 1] : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (c0 + k < nchunks) prefix[c0 + k] = v[k] > 0.0 ? run : __builtin_inf();
        run += v[k];
    }
    if (threadIdx.x == 255) gtot[blockIdx.x] = sh[255];
}

// One block per sample: the last group and in it the last chunk whose offset is
// at most the target, then the chunk is scanned in order.  Offsets are sums
// associated in a tree and may decrease in the last place from one entry to
// the next, or grow by it over entries without probability, so the highest
// index that passes is taken (a bisection or a count would take them for
// sorted), and only groups, chunks and amplitudes of some probability are
// drawn: the first of them has offset 0 in its group, so one always passes.
// A state of one chunk needs no offsets (one sample of 12 qubits: 43 -> 35 us).  With E = 16 elements per thread
// (chunks of 4,096, up to 30 qubits) the probabilities stay in registers
// between the sum and the search.
template <typename R, int E16>
__global__ __launch_bounds__(256) void k_find(const typename C2r<R>::T* __restrict__ psi,
                                              int n, int clog, Perm P,
                                              const double* __restrict__ prefix, uint64_t nchunks,
                                              const double* __restrict__ gtot, uint32_t ngroups,
                                              const double* __restrict__ uni,
                                              uint64_t* __restrict__ out) {
    __shared__ double sh[5];
    __shared__ unsigned long long best, last;     // first amplitude past the target; last of the chunk with any probability
    __shared__ unsigned grp, chunk;               // 1 + the highest that passes
    const uint64_t N = 1ull << n;
    const uint64_t C = 1ull << clog;
    const uint32_t t = threadIdx.x;
    // the sums before each thread's value, and of all: within the waves, then
    // the waves' totals
    auto before = [&](double v, double& total) {
        const uint32_t lane = t & 63, wave = t >> 6;
        double x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double y = __shfl_up(x, o, 64);
            if (lane >= (uint32_t)o) x += y;
        }
        __syncthreads();
        if (lane == 63) sh[wave] = x;
        __syncthreads();
        double b = 0;
        for (uint32_t w = 0; w < wave; ++w) b += sh[w];
        total = (sh[0] + sh[1]) + (sh[2] + sh[3]);
        const double y = __shfl_up(x, 1, 64);
        return lane ? b + y : b;
    };
    if (t == 0) {
        best = ~0ull;
        last = 0;
        grp = chunk = 0;
    }
    const double u = uni[blockIdx.x];
    double total, target = 0, coff = 0;
    uint64_t c = 0;
    if (nchunks > 1) {
        const double mine = t < ngroups ? gtot[t] : 0.0;
        const double off = before(mine, total);
        target = u * total;
        if (mine > 0.0 && off <= target) atomicMax(&grp, t + 1);
        __syncthreads();
        if (grp == 0) {                                          // no probability at all, or not a number
            if (t == 0) out[blockIdx.x] = target == 0.0 ? N - 1 : C;
            return;
        }
        const uint32_t g = grp - 1;
        if (t == g) sh[4] = off;
        __syncthreads();
        const double goff = sh[4];
        unsigned top = 0;
        for (uint32_t k = t; k < kGroup; k += 256) {
            const uint64_t q = (uint64_t)g * kGroup + k;
            if (q < nchunks && goff + prefix[q] <= target) top = k + 1;
        }
        if (top) atomicMax(&chunk, top);
        __syncthreads();
        c = (uint64_t)g * kGroup + (chunk ? chunk - 1 : 0);
        coff = goff + prefix[c];
    }
    const uint64_t E = C >= 256 ? C / 256 : 1;
    const uint64_t e0 = min((uint64_t)t * E, C);
    const uint64_t e1 = min(e0 + E, C);
    const uint64_t base = c << clog;
    // e0 is a multiple of E, so phys(base + e0 + k) = phys(base + e0) | phys(k), k < E
    const uint64_t pb0 = to_phys(base + e0, P);
    double loc = 0, pr[E16 ? 16 : 1];
    if constexpr (E16) {
        typename C2r<R>::T v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = psi[pb0 | to_phys(k, P)];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            pr[k] = prob(v[k]);
            loc += pr[k];
        }
    } else {
        for (uint64_t e = e0; e < e1; ++e) loc += prob(psi[pb0 | to_phys(e - e0, P)]);
    }
    double run = coff + before(loc, total);
    if (nchunks == 1) target = u * total;
    uint64_t cand = ~0ull, nz = nchunks == 1 && !(total > 0.0) ? N - 1 : 0;
    if constexpr (E16) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            run += pr[k];
            if (cand == ~0ull && pr[k] > 0.0 && run > target) cand = base + e0 + k;
            if (pr[k] > 0.0) nz = base + e0 + k;
        }
    } else {
        for (uint64_t e = e0; e < e1; ++e) {
            const double x = prob(psi[pb0 | to_phys(e - e0, P)]);
            run += x;
            if (x > 0.0) nz = base + e;
            if (x > 0.0 && run > target) {
                cand = base + e;
                break;
            }
        }
    }
    if (cand != ~0ull) atomicMin(&best, (unsigned long long)cand);
    if (nz) atomicMax(&last, (unsigned long long)nz);
    __syncthreads();
    // (rounding may leave the target at or past the end of the chunk)
    if (t == 0) out[blockIdx.x] = best != ~0ull ? best : last;
}

// ------------------------------------------------------------ amplitudes
template <typename R>
__global__ __launch_bounds__(256) void k_copy(const typename C2r<R>::T* __restrict__ psi,
                                              uint64_t first, uint64_t cnt, Perm P,
                                              double2* __restrict__ out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < cnt; j += stride) {
        auto v = psi[to_phys(first + j, P)];
        out[j] = make_double2((double)v.x, (double)v.y);
    }
}

template <typename R>
__global__ __launch_bounds__(256) void k_gather(const typename C2r<R>::T* __restrict__ psi,
                                                const uint64_t* __restrict__ idx, uint64_t cnt,
                                                Perm P, double2* __restrict__ out) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= cnt) return;
    auto v = psi[to_phys(idx[j], P)];
    out[j] = make_double2((double)v.x, (double)v.y);
}

// ------------------------------------------ one qubit's reduced density matrix
// Over the pairs (i, j = i | 2^b) with physical bit b of i clear:
// part column [0] = sum |psi_i|^2, [1] = sum |psi_j|^2, [2] + i [3] = sum psi_i conj(psi_j).
template <typename R>
__global__ __launch_bounds__(256) void k_rdm1_partial(const typename C2r<R>::T* __restrict__ psi,
                                                      uint64_t half, int b, double* __restrict__ part) {
    __shared__ double sh[4];
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t low = (1ull << b) - 1;
    double r00 = 0, r11 = 0, re = 0, im = 0;
    for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < half; w += stride) {
        const uint64_t i = ((w & ~low) << 1) | (w & low);
        const auto x = psi[i], y = psi[i | (low + 1)];
        const double xr = x.x, xi = x.y, yr = y.x, yi = y.y;
        r00 += xr * xr + xi * xi;
        r11 += yr * yr + yi * yi;
        re += xr * yr + xi * yi;
        im += xi * yr - xr * yi;
    }
    const double v[4] = {r00, r11, re, im};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const double t = block_sum256(v[s], sh);
        if (threadIdx.x == 0) part[(size_t)s * gridDim.x + blockIdx.x] = t;
    }
}

// ============================================================ host side
static unsigned grid_of(uint64_t items) {
    uint64_t g = (items + 255) / 256;
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(g, 1u << 20));
}
// one item per thread up to 2^31 threads (the kernels loop over the rest)
static unsigned grid_one(uint64_t items) {
    uint64_t g = (items + 255) / 256;
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(g, 1u << 23));
}

static double* red_part(qvm_sv* sv) { return (double*)(sv->work + sv->lay.red_off); }
static double* red_res(qvm_sv* sv) { return red_part(sv) + (size_t)kRedBlocks * kRedSlots; }
static char* io(qvm_sv* sv) { return sv->work + sv->lay.io_off; }

constexpr size_t kPauliJobs = 512;                // jobs per launch (their records at the start of the staging area)

static qvm_status fetch(qvm_sv* sv, void* host, const void* dev, size_t bytes) {
    QVM_HIP(sv, hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, sv->stream));
    QVM_HIP(sv, hipStreamSynchronize(sv->stream));
    return QVM_OK;
}

template <typename R>
static qvm_status norm_t(qvm_sv* sv, double* out) {
    using T = typename C2r<R>::T;
    uint64_t N = 1ull << sv->n;
    hipLaunchKernelGGL((k_norm_partial<R>), dim3(kRedBlocks), dim3(256), 0, sv->stream,
                       (const T*)sv->amps, N, red_part(sv));
    QVM_LAUNCH_CHECK(sv);
    hipLaunchKernelGGL(k_final, dim3(1), dim3(256), 0, sv->stream, red_part(sv), (uint32_t)kRedBlocks, red_res(sv));
    QVM_LAUNCH_CHECK(sv);
    return fetch(sv, out, red_res(sv), sizeof(double));
}

qvm_status rd_norm(qvm_sv* sv, double* out) {
    return sv->dt == QVM_C64 ? norm_t<float>(sv, out) : norm_t<double>(sv, out);
}

qvm_status rd_scale(qvm_sv* sv, double f) {
    uint64_t N = 1ull << sv->n;
    if (sv->dt == QVM_C64)
        hipLaunchKernelGGL((k_scale<float>), dim3(grid_one(N / 2)), dim3(256), 0, sv->stream,
                           (float2*)sv->amps, N, (float)f);
    else
        hipLaunchKernelGGL((k_scale<double>), dim3(grid_one(N)), dim3(256), 0, sv->stream,
                           (double2*)sv->amps, N, f);
    QVM_LAUNCH_CHECK(sv);
    return QVM_OK;
}

template <typename R>
static qvm_status zall_t(qvm_sv* sv, double* total, double* bit) {
    using T = typename C2r<R>::T;
    constexpr int LB = Piece<R>::LB;
    const int above = std::max(0, sv->n - LB);                   // index bits above a row
    const int bb = std::min(above, 11), ib = above - bb;
    const uint32_t nb = 1u << bb;
    const int cols = 1 + std::min(sv->n, LB) + ib;
    static_assert((size_t)2048 * (1 + 9 + 15) <= (size_t)kRedBlocks * kRedSlots, "partials fit (34 qubits)");
    hipLaunchKernelGGL((k_zall_partial<R>), dim3(nb), dim3(256), 0, sv->stream,
                       (const T*)sv->amps, sv->n, ib, red_part(sv));
    QVM_LAUNCH_CHECK(sv);
    hipLaunchKernelGGL(k_zall_final, dim3(sv->n + 1), dim3(256), 0, sv->stream, red_part(sv), nb, cols,
                       red_res(sv));
    QVM_LAUNCH_CHECK(sv);
    double res[QVM_MAX_QUBITS + 1];
    qvm_status st = fetch(sv, res, red_res(sv), sizeof(double) * (sv->n + 1));
    if (st) return st;
    *total = res[0];
    for (int q = 0; q < sv->n; ++q) bit[q] = res[1 + q];
    return QVM_OK;
}

template <typename R>
static qvm_status rdm1_t(qvm_sv* sv, int pbit, double* out) {
    using T = typename C2r<R>::T;
    const int tok = prof_begin(sv);
    hipLaunchKernelGGL((k_rdm1_partial<R>), dim3(kRedBlocks), dim3(256), 0, sv->stream,
                       (const T*)sv->amps, 1ull << (sv->n - 1), pbit, red_part(sv));
    prof_end(sv, tok, PK_RDM1, (double)(1ull << sv->n) * sizeof(T), 8.0 * (double)(1ull << sv->n));
    QVM_LAUNCH_CHECK(sv);
    hipLaunchKernelGGL(k_final, dim3(4), dim3(256), 0, sv->stream, red_part(sv), (uint32_t)kRedBlocks, red_res(sv));
    QVM_LAUNCH_CHECK(sv);
    return fetch(sv, out, red_res(sv), 4 * sizeof(double));
}

qvm_status rd_rdm1(qvm_sv* sv, int pbit, double* out) {
    return sv->dt == QVM_C64 ? rdm1_t<float>(sv, pbit, out) : rdm1_t<double>(sv, pbit, out);
}

qvm_status rd_z_all(qvm_sv* sv, double* total, double* bit) {
    return sv->dt == QVM_C64 ? zall_t<float>(sv, total, bit) : zall_t<double>(sv, total, bit);
}

template <typename R>
static qvm_status pauli_t(qvm_sv* sv, const std::vector<PauliTerm>& terms, double* out) {
    using T = typename C2r<R>::T;
    constexpr int LB = Piece<R>::LB;
    std::vector<PauliJob> jobs;
    std::vector<size_t> order;                                   // term of each column
    auto flush = [&]() -> qvm_status {
        if (jobs.empty()) return QVM_OK;
        // blocks per job: about 4,096 in all, with eight rows or more each unless
        // that leaves fewer than 256 (one string, 22 qubits: complex64 49 us with
        // two rows, 41 with eight; complex128 52 and 46), within the partials
        const uint64_t rows = sv->n - 1 > LB ? 1ull << (sv->n - 1 - LB) : 1;
        uint64_t nb = 4096 / jobs.size();
        const uint64_t most = std::max<uint64_t>(rows / 8, std::min<uint64_t>(rows, 256));
        nb = std::min<uint64_t>({std::max<uint64_t>(nb, 1), most, (uint64_t)kRedBlocks * kRedSlots / order.size()});
        PauliJob* dj = (PauliJob*)io(sv);
        double* res = (double*)(io(sv) + kPauliJobs * sizeof(PauliJob));
        qvm_status st = put_words(sv, (uint32_t*)dj, (const uint32_t*)jobs.data(), jobs.size() * sizeof(PauliJob) / 4);
        if (st) return st;
        hipLaunchKernelGGL((k_pauli_partial<R>), dim3((unsigned)nb, (unsigned)jobs.size()), dim3(256), 0, sv->stream,
                           (const T*)sv->amps, sv->n, dj, red_part(sv));
        QVM_LAUNCH_CHECK(sv);
        hipLaunchKernelGGL(k_final, dim3((unsigned)order.size()), dim3(256), 0, sv->stream, red_part(sv),
                           (uint32_t)nb, res);
        QVM_LAUNCH_CHECK(sv);
        std::vector<double> r(order.size());
        st = fetch(sv, r.data(), res, sizeof(double) * r.size());
        if (st) return st;
        for (size_t i = 0; i < r.size(); ++i) {
            const PauliTerm& t = terms[order[i]];
            const int c = __builtin_popcountll(t.x & t.z) & 3;
            out[t.index] = t.x == 0 ? r[i] : (c == 0 || c == 3) ? 2.0 * r[i] : -2.0 * r[i];
        }
        jobs.clear();
        order.clear();
        return QVM_OK;
    };
    for (size_t i = 0; i < terms.size();) {
        // the terms of one x, Re kinds first (the caller sorts)
        size_t e = i, m = i;
        while (e < terms.size() && terms[e].x == terms[i].x) ++e;
        auto im = [&](size_t k) { return (uint32_t)(__builtin_popcountll(terms[k].x & terms[k].z) & 1); };
        while (m < e && !im(m)) ++m;
        struct Set { size_t a, b; };
        std::vector<Set> sets;
        for (size_t a = i; a < m; a += 16) sets.push_back({a, std::min(a + 16, m)});
        for (size_t a = m; a < e; a += 16) sets.push_back({a, std::min(a + 16, e)});
        for (size_t s = 0; s < sets.size(); s += 2) {
            if (jobs.size() == kPauliJobs) {
                const qvm_status st = flush();
                if (st) return st;
            }
            PauliJob j{};
            j.x = terms[i].x;
            j.out = (uint32_t)order.size();
            for (size_t k = s; k < std::min(s + 2, sets.size()); ++k) {
                j.nt[k - s] = (uint32_t)(sets[k].b - sets[k].a);
                j.im[k - s] = im(sets[k].a);
                for (size_t q = sets[k].a; q < sets[k].b; ++q) {
                    j.z[16 * (k - s) + (q - sets[k].a)] = terms[q].z;
                    order.push_back(q);
                }
            }
            jobs.push_back(j);
        }
        i = e;
    }
    return flush();
}

qvm_status rd_pauli(qvm_sv* sv, const std::vector<PauliTerm>& terms, double* out) {
    return sv->dt == QVM_C64 ? pauli_t<float>(sv, terms, out) : pauli_t<double>(sv, terms, out);
}

template <typename R>
static qvm_status probs_t(qvm_sv* sv, double* out) {
    using T = typename C2r<R>::T;
    const uint64_t N = 1ull << sv->n;
    const uint64_t cap = sv->lay.io_bytes / sizeof(double);
    Perm P = make_perm(sv);
    for (uint64_t f = 0; f < N; f += cap) {
        uint64_t cnt = std::min(cap, N - f);
        hipLaunchKernelGGL((k_probs<R>), dim3(grid_of(cnt)), dim3(256), 0, sv->stream,
                           (const T*)sv->amps, f, cnt, P, (double*)io(sv));
        QVM_LAUNCH_CHECK(sv);
        qvm_status st = fetch(sv, out + f, io(sv), cnt * sizeof(double));
        if (st) return st;
    }
    return QVM_OK;
}

qvm_status rd_probs_full(qvm_sv* sv, double* out) {
    return sv->dt == QVM_C64 ? probs_t<float>(sv, out) : probs_t<double>(sv, out);
}

// The marginal over physical bits pq (output bit r <-> pq[r]) into dst, with
// partials (if the blocks outnumber the buckets) in part.
template <typename R>
static qvm_status marginal_to(qvm_sv* sv, int m, const int* pq, double* dst, double* part, size_t part_doubles) {
    using T = typename C2r<R>::T;
    constexpr int LB = Piece<R>::LB;
    MargArgs a{};
    uint64_t q = 0;
    for (int r = 0; r < m; ++r) q |= 1ull << pq[r];
    const uint64_t rowm = (1ull << std::min(LB, sv->n)) - 1, above = ((1ull << sv->n) - 1) & ~rowm;
    a.qlo = (uint32_t)(q & rowm);
    a.qhi = q & above;
    a.mh = (uint32_t)__builtin_popcountll(a.qhi);
    for (int r = 0; r < m; ++r) {
        const uint64_t below = (1ull << pq[r]) - 1;
        if ((rowm >> pq[r]) & 1) a.lo_out[__builtin_popcountll(a.qlo & below)] = (uint8_t)r;
        else a.hi_out[__builtin_popcountll(a.qhi & below)] = (uint8_t)r;
    }
    a.hi_run = 1;
    for (uint32_t k = 1; k < a.mh; ++k) a.hi_run &= a.hi_out[k] == a.hi_out[0] + k;
    // the other bits above the row: the highest split the sum over blocks, as
    // long as a block keeps the four rows that it has in flight at once, and
    // from 256 blocks on (one a CU) sixteen: their sums take another launch
    uint64_t rest = above & ~q;
    uint32_t sb = 0;
    const size_t nb = (size_t)1 << m;
    while (__builtin_popcountll(rest) > (a.mh + sb < 8 ? 2 : 4) && a.mh + sb < 11 && (nb << (sb + 1)) <= part_doubles) {
        const uint64_t top = 1ull << (63 - __builtin_clzll(rest));
        a.seg |= top;
        rest ^= top;
        ++sb;
    }
    a.iter = rest;
    a.segs = 1u << sb;
    a.niter = 1u << __builtin_popcountll(rest);
    hipLaunchKernelGGL((k_marg_partial<R>), dim3(1u << (a.mh + sb)), dim3(256), 0, sv->stream,
                       (const T*)sv->amps, sv->n, a, sb ? part : dst);
    QVM_LAUNCH_CHECK(sv);
    if (sb) {
        // few buckets of many partials each: a block per bucket
        if (a.segs >= 64)
            hipLaunchKernelGGL(k_final, dim3((unsigned)nb), dim3(256), 0, sv->stream, part, a.segs, dst);
        else
            hipLaunchKernelGGL(k_marg_final, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, sv->stream,
                               part, (uint64_t)nb, a.segs, dst);
        QVM_LAUNCH_CHECK(sv);
    }
    return QVM_OK;
}

template <typename R>
static qvm_status marg_t(qvm_sv* sv, int m, const int* pq, double* out) {
    // one partial per bucket and 2^14 amplitudes must fit the staging area
    const int nO = sv->n - m;
    const uint64_t nb = 1ull << m, nblk = nb * (nO > 14 ? (1u << (nO - 14)) : 1u);
    if ((nblk + nb) * sizeof(double) > sv->lay.io_bytes)
        return fail(QVM_ENOMEM, "marginal partials exceed the staging area");
    double* res = (double*)io(sv);
    const qvm_status st = marginal_to<R>(sv, m, pq, res, res + nb, sv->lay.io_bytes / sizeof(double) - nb);
    if (st) return st;
    return fetch(sv, out, res, nb * sizeof(double));
}

qvm_status rd_marginal(qvm_sv* sv, int m, const int* pq, double* out) {
    return sv->dt == QVM_C64 ? marg_t<float>(sv, m, pq, out) : marg_t<double>(sv, m, pq, out);
}

template <typename R>
static qvm_status sample_t(qvm_sv* sv, size_t ns, const double* u, uint64_t* out) {
    using T = typename C2r<R>::T;
    const int clog = sv->lay.chunk_log;
    const uint64_t nchunks = 1ull << (sv->n - clog);
    double* csum = (double*)(sv->work + sv->lay.chunk_off);
    double* prefix = csum + nchunks;
    Perm P = make_perm(sv);
    const uint32_t ngroups = (uint32_t)((nchunks + kGroup - 1) / kGroup);
    double* gtot = red_part(sv);
    qvm_status st;
    if (nchunks > 1) {
        int pq[QVM_MAX_QUBITS];
        for (int q = clog; q < sv->n; ++q) pq[q - clog] = sv->perm[q];
        st = marginal_to<R>(sv, sv->n - clog, pq, csum, (double*)io(sv), sv->lay.io_bytes / sizeof(double));
        if (st) return st;
        hipLaunchKernelGGL(k_scan_chunks, dim3(ngroups), dim3(256), 0, sv->stream, csum, nchunks, prefix, gtot);
        QVM_LAUNCH_CHECK(sv);
    }
    const size_t cap = sv->lay.io_bytes / 16;
    double* du = (double*)io(sv);
    uint64_t* dout = (uint64_t*)(io(sv) + cap * sizeof(double));
    for (size_t s0 = 0; s0 < ns; s0 += cap) {
        size_t cnt = std::min(cap, ns - s0);
        QVM_HIP(sv, hipMemcpyAsync(du, u + s0, cnt * sizeof(double), hipMemcpyHostToDevice,
                                   sv->stream));
        if (clog == 12)
            hipLaunchKernelGGL((k_find<R, 1>), dim3((unsigned)cnt), dim3(256), 0, sv->stream, (const T*)sv->amps,
                               sv->n, clog, P, prefix, nchunks, gtot, ngroups, du, dout);
        else
            hipLaunchKernelGGL((k_find<R, 0>), dim3((unsigned)cnt), dim3(256), 0, sv->stream, (const T*)sv->amps,
                               sv->n, clog, P, prefix, nchunks, gtot, ngroups, du, dout);
        QVM_LAUNCH_CHECK(sv);
        st = fetch(sv, out + s0, dout, cnt * sizeof(uint64_t));
        if (st) return st;
    }
    return QVM_OK;
}

qvm_status rd_sample(qvm_sv* sv, size_t ns, const double* u, uint64_t* out) {
    if (ns == 0) return QVM_OK;
    return sv->dt == QVM_C64 ? sample_t<float>(sv, ns, u, out) : sample_t<double>(sv, ns, u, out);
}

template <typename R>
static qvm_status copy_t(qvm_sv* sv, uint64_t first, uint64_t count, double* out) {
    using T = typename C2r<R>::T;
    const uint64_t cap = sv->lay.io_bytes / 16;
    Perm P = make_perm(sv);
    for (uint64_t f = 0; f < count; f += cap) {
        uint64_t cnt = std::min(cap, count - f);
        hipLaunchKernelGGL((k_copy<R>), dim3(grid_of(cnt)), dim3(256), 0, sv->stream,
                           (const T*)sv->amps, first + f, cnt, P, (double2*)io(sv));
        QVM_LAUNCH_CHECK(sv);
        qvm_status st = fetch(sv, out + 2 * f, io(sv), cnt * 16);
        if (st) return st;
    }
    return QVM_OK;
}

qvm_status rd_copy(qvm_sv* sv, uint64_t first, uint64_t count, double* out) {
    if (!count) return QVM_OK;
    return sv->dt == QVM_C64 ? copy_t<float>(sv, first, count, out)
                             : copy_t<double>(sv, first, count, out);
}

template <typename R>
static qvm_status gather_t(qvm_sv* sv, size_t count, const uint64_t* idx, double* out) {
    using T = typename C2r<R>::T;
    const size_t cap = sv->lay.io_bytes / 24;
    Perm P = make_perm(sv);
    uint64_t* di = (uint64_t*)io(sv);
    double2* dv = (double2*)(io(sv) + ((cap * 8 + 255) & ~size_t(255)));
    for (size_t f = 0; f < count; f += cap) {
        size_t cnt = std::min(cap, count - f);
        QVM_HIP(sv, hipMemcpyAsync(di, idx + f, cnt * 8, hipMemcpyHostToDevice, sv->stream));
        hipLaunchKernelGGL((k_gather<R>), dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0,
                           sv->stream, (const T*)sv->amps, di, cnt, P, dv);
        QVM_LAUNCH_CHECK(sv);
        qvm_status st = fetch(sv, out + 2 * f, dv, cnt * 16);
        if (st) return st;
    }
    return QVM_OK;
}

qvm_status rd_gather(qvm_sv* sv, size_t count, const uint64_t* idx, double* out) {
    if (!count) return QVM_OK;
    return sv->dt == QVM_C64 ? gather_t<float>(sv, count, idx, out)
                             : gather_t<double>(sv, count, idx, out);
}

}  // namespace qvm
