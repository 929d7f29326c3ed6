// Row operations on operators whose blocks of 256 rows hold few distinct
// (offset, value) pairs: constant-coefficient stencils and the fine Galerkin and
// transfer operators made from them.  The entries are kept without loss as a
// table of the block's pairs (column minus the row's base column, value) and a
// code of one or two bytes per entry, its place in the table, so that a sweep
// moves 1 byte an entry where the SELL-64 copy moves 9 and is left with its
// vectors.
//
// Layout: a lane a row; the codes of a row packed into 32-bit words, the same
// number for every row of the operator, word k of a block's 256 rows
// contiguous; code 0 is the padding of shorter rows (never summed).  The base
// column is the row itself (square operators) or the row's first column.
// Codes, table and vectors have addresses known from the block alone, so they
// are requested together; the table goes to LDS, then every lane gathers its
// whole row and sums it in ascending column order.  The reciprocal diagonal of
// a sweep comes from the table too.  Every sum is formed with the operations of
// the form this one replaces, so results keep their bits.
//
// Bound by the vectors and by the two memory latencies of a block: 3D Poisson
// 128^3, us a launch, SELL-64 (P: LDS-staged) -> coded: A_0 residual 29.4 -> 16.1
// (67 MB, 4.2 TB/s), product 26.9 -> 16.0, last sweep 43.1 -> 20.2, A_1 residual
// 48.2 -> 17.7, sweep 44.7 -> 17.5, R_0 24.1 -> 14.9, R_1 16.2 -> 7.6, P_0 30 ->
// 21.7, P_1 13.9 -> 9.7.  No faster: two rows a lane, 2,048 or 4,096 workgroups
// looping; slower: a list of pairs per slice with a bit per pair and row
// (offsets and values in scalar registers, no LDS; A_1 residual 24.5 us).
#include "kernels.hpp"
#include "row_common.hpp"

#include <hip/hip_ext.h>

#include <algorithm>
#include <stdexcept>
#include <string>

namespace amg355 {
namespace {

constexpr int kGrid = 65536;    // workgroups; larger operators loop

template <int CB>
constexpr int kLimit = CB == 1 ? 256 : 1024;   // pairs of a block, the padding's included

template <class K, class... Args>
void launch(K kernel, dim3 grid, hipStream_t st, Args... args) {
    hipEvent_t a, b;
    if (take_launch_events(&a, &b)) hipExtLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, st, a, b, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, st, args...);
}

// acc + v g: one multiply-add (what the SELL-64 kernel's sum compiles to), or
// the product rounded, then added (the LDS-staged kernel's)
template <bool FUSED, class T>
__device__ __forceinline__ T add_term(T acc, T v, T g) {
    if constexpr (FUSED) {
        if constexpr (sizeof(T) == 8) return __builtin_fma(v, g, acc);
        else return __builtin_fmaf(v, g, acc);
    } else {
#pragma clang fp contract(off)
        const T p = v * g;
        return acc + p;
    }
}

template <int OP>
constexpr bool has_dot() {
    return OP == kResidNorm || OP == kJacobiDot || OP == kSpmvDot;
}

template <int CB>
__device__ __forceinline__ int code_of(const uint32_t* wd, int k) {
    if constexpr (CB == 1) return (int)((wd[k / 4] >> (8 * (k % 4))) & 255u);
    else return (int)((wd[k / 2] >> (16 * (k % 2))) & 65535u);
}

// NW: words of a row
template <class T, int NW, int OP, int CB, bool FUSED>
__global__ __launch_bounds__(kBlock) void coded_kernel(CsrT<T> a, const T* __restrict__ g, const T* u,
                                                       const T* __restrict__ dinv, T omega, T* y, T* y2,
                                                       DotTarget dot, int nblocks) {
    constexpr int U = NW * 4 / CB;
    constexpr bool kSweep = OP == kJacobi || OP == kJacobiDot;   // square: 1 / a_ii from the table
    __shared__ T tv[kLimit<CB>];
    __shared__ int to[kLimit<CB>];
    __shared__ T td[kSweep ? kLimit<CB> : 1];
    const int lb = xcd_logical_block();
    double contrib = 0.0;
    // with one block per workgroup a dot product's partial goes to the block's
    // own index, the same in both directions
    int pidx = lb;
    for (int lblk = lb; lblk < nblocks; lblk += gridDim.x) {
        const int blk = a.rev ? nblocks - 1 - lblk : lblk;
        if (nblocks <= (int)gridDim.x) pidx = blk;
        uint32_t wd[NW];
        const uint32_t* const word = a.pc_word + (size_t)blk * NW * kBlock + threadIdx.x;
#pragma unroll
        for (int k = 0; k < NW; ++k) wd[k] = word[k * kBlock];
        const int r = blk * kBlock + (int)threadIdx.x;
        const bool act = r < a.rows;
        const int base = !act ? 0 : a.pc_base ? a.pc_base[r] : r;
        T ui = T(0), gi = T(0), di = T(0);
        if (act) {
            if constexpr (OP != kSpmv && OP != kSpmvDot && OP != kSpmvScale) ui = u[r];
            if constexpr (OP == kJacobi || OP == kJacobiDot || OP == kSpmvDot) gi = g[r];
            if constexpr (OP == kZeroJacobiResid || OP == kSpmvScale) di = dinv[r];
        }
        if (lblk != lb) __syncthreads();   // the table of the block before is done with
        for (int t = threadIdx.x; t < a.pc_stride; t += kBlock) {
            to[t] = a.pc_tabo[(size_t)blk * a.pc_stride + t];
            tv[t] = (T)a.pc_tabv[(size_t)blk * a.pc_stride + t];
            if constexpr (kSweep) td[t] = (T)a.pc_tabr[(size_t)blk * a.pc_stride + t];
        }
        __syncthreads();
        T gg[U];
        int diag = 0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int c = code_of<CB>(wd, k);
            const int o = to[c];
            const int j = base + o;
            if constexpr (kSweep) diag = (c != 0 && o == 0) ? c : diag;
            if constexpr (OP == kZeroJacobiResid) gg[k] = omega * (dinv[j] * u[j]);
            else gg[k] = g[j];
        }
        T acc = T(0);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int c = code_of<CB>(wd, k);
            const T s = add_term<FUSED>(acc, tv[c], gg[k]);
            acc = c != 0 ? s : acc;
        }
        if constexpr (kSweep) di = td[diag];
        if (act) {
            if constexpr (OP == kSpmv) {
                y[r] = acc;
            } else if constexpr (OP == kSpmvAdd) {
                y[r] = ui + acc;
            } else if constexpr (OP == kResid || OP == kResidNorm) {
                const T rr = ui - acc;
                y[r] = rr;
                if constexpr (OP == kResidNorm) contrib += (double)rr * (double)rr;
            } else if constexpr (OP == kJacobi || OP == kJacobiDot) {
                const T xn = gi + omega * di * (ui - acc);
                y[r] = xn;
                if constexpr (OP == kJacobiDot) contrib += (double)ui * (double)xn;
            } else if constexpr (OP == kZeroJacobiResid) {
                y2[r] = omega * (di * ui);
                y[r] = ui - acc;
            } else if constexpr (OP == kSpmvDot) {
                y[r] = acc;
                contrib += (double)gi * (double)acc;
            } else if constexpr (OP == kSpmvScale) {
                y[r] = acc;
                y2[r] = omega * (di * acc);
            }
        }
    }
    if constexpr (has_dot<OP>()) store_block_partial(contrib, dot.partials, pidx);
}

// y = u - A g and y2 = u2 - A g2 with the block partials of ||y2||^2, every row
// summed as coded_kernel sums it
template <int NW>
__global__ __launch_bounds__(kBlock) void coded_dual_kernel(CsrView a, const double* __restrict__ g, const double* u,
                                                            double* y, const double* __restrict__ g2,
                                                            const double* u2, double* y2, DotTarget dot,
                                                            int nblocks) {
    constexpr int U = NW * 4;
    __shared__ double tv[kLimit<1>];
    __shared__ int to[kLimit<1>];
    const int lb = xcd_logical_block();
    double contrib = 0.0;
    int pidx = lb;
    for (int lblk = lb; lblk < nblocks; lblk += gridDim.x) {
        const int blk = a.rev ? nblocks - 1 - lblk : lblk;
        if (nblocks <= (int)gridDim.x) pidx = blk;
        uint32_t wd[NW];
        const uint32_t* const word = a.pc_word + (size_t)blk * NW * kBlock + threadIdx.x;
#pragma unroll
        for (int k = 0; k < NW; ++k) wd[k] = word[k * kBlock];
        const int r = blk * kBlock + (int)threadIdx.x;
        const bool act = r < a.rows;
        const int base = act ? r : 0;
        double ui = 0.0, u2i = 0.0;
        if (act) {
            ui = u[r];
            u2i = u2[r];
        }
        if (lblk != lb) __syncthreads();
        for (int t = threadIdx.x; t < a.pc_stride; t += kBlock) {
            to[t] = a.pc_tabo[(size_t)blk * a.pc_stride + t];
            tv[t] = a.pc_tabv[(size_t)blk * a.pc_stride + t];
        }
        __syncthreads();
        double gg[U], gg2[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int j = base + to[code_of<1>(wd, k)];
            gg[k] = g[j];
            gg2[k] = g2[j];
        }
        double acc = 0.0, acc2 = 0.0;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int c = code_of<1>(wd, k);
            const double v = tv[c];
            const double s = __builtin_fma(v, gg[k], acc), s2 = __builtin_fma(v, gg2[k], acc2);
            acc = c != 0 ? s : acc;
            acc2 = c != 0 ? s2 : acc2;
        }
        if (act) {
            y[r] = ui - acc;
            const double rr = u2i - acc2;
            y2[r] = rr;
            contrib += rr * rr;
        }
    }
    store_block_partial(contrib, dot.partials, pidx);
}

int coded_blocks(int rows) { return (rows + kBlock - 1) / kBlock; }

int coded_grid(int rows) { return round_up8(std::max(1, std::min(coded_blocks(rows), kGrid))); }

bool dot_op(RowOp op) { return op == kResidNorm || op == kJacobiDot || op == kSpmvDot; }

// a dot product's partials are independent of the direction only with one
// block per workgroup
template <class T>
CsrT<T> directed(const CsrT<T>& a, bool dot) {
    CsrT<T> d = a;
    if (dot && coded_blocks(a.rows) > coded_grid(a.rows)) d.rev = 0;
    return d;
}

// An operation or a row of words without an instance would leave its result
// unwritten.
[[noreturn]] void no_instance(int kind, int op, int words) {
    throw std::logic_error("pair-coded form " + std::to_string(kind) + " has no kernel for operation " +
                           std::to_string(op) + " on rows of " + std::to_string(words) + " words");
}

#define AMG_CODED_CASE(OPV)                                                                                  \
    case OPV:                                                                                                \
        launch(coded_kernel<T, NW, OPV, CB, FUSED>, dim3(grid), st, a, g, u, dinv, omega, y, y2, dot, nb);   \
        break;

// square operators: every operation but the interpolation's
template <class T, int NW>
void launch_square(RowOp op, const CsrT<T>& a, const T* g, const T* u, const T* dinv, T omega, T* y, T* y2,
                   DotTarget dot, hipStream_t st) {
    constexpr int CB = 1;
    constexpr bool FUSED = true;
    const int grid = coded_grid(a.rows), nb = coded_blocks(a.rows);
    switch (op) {
        AMG_CODED_CASE(kSpmv)
        AMG_CODED_CASE(kResid)
        AMG_CODED_CASE(kJacobi)
        AMG_CODED_CASE(kZeroJacobiResid)
        default:
            if constexpr (sizeof(T) == 8) {   // the FP32 cycle forms no dots
                switch (op) {
                    AMG_CODED_CASE(kResidNorm)
                    AMG_CODED_CASE(kJacobiDot)
                    AMG_CODED_CASE(kSpmvDot)
                    default: no_instance(a.pc_kind, op, NW);
                }
            } else {
                no_instance(a.pc_kind, op, NW);
            }
    }
}

// restriction operators
template <class T, int NW>
void launch_restrict(RowOp op, const CsrT<T>& a, const T* g, const T* u, const T* dinv, T omega, T* y, T* y2,
                     DotTarget dot, hipStream_t st) {
    constexpr int CB = 2;
    constexpr bool FUSED = true;
    const int grid = coded_grid(a.rows), nb = coded_blocks(a.rows);
    switch (op) {
        AMG_CODED_CASE(kSpmv)
        AMG_CODED_CASE(kSpmvScale)
        default: no_instance(a.pc_kind, op, NW);
    }
}

// interpolation operators
template <class T, int NW>
void launch_interp(RowOp op, const CsrT<T>& a, const T* g, const T* u, const T* dinv, T omega, T* y, T* y2,
                   DotTarget dot, hipStream_t st) {
    constexpr int CB = 1;
    constexpr bool FUSED = false;
    const int grid = coded_grid(a.rows), nb = coded_blocks(a.rows);
    switch (op) {
        AMG_CODED_CASE(kSpmvAdd)
        default: no_instance(a.pc_kind, op, NW);
    }
}
#undef AMG_CODED_CASE

template <class T>
int launch_op(RowOp op, const CsrT<T>& a_in, const T* g, const T* u, const T* dinv, T omega, T* y, T* y2,
              DotTarget dot, hipStream_t st) {
    const CsrT<T> a = directed(a_in, dot_op(op));
#define AMG_CODED_ARGS op, a, g, u, dinv, omega, y, y2, dot, st
    if (a.pc_kind == kCodedSquare || a.pc_kind == kCodedInterp) {
        const bool sq = a.pc_kind == kCodedSquare;
        switch (a.pc_words) {
#define AMG_CODED_WORDS(NW)                                             \
    case NW:                                                            \
        if (sq) launch_square<T, NW>(AMG_CODED_ARGS);                   \
        else launch_interp<T, NW>(AMG_CODED_ARGS);                      \
        break;
            AMG_CODED_WORDS(1)
            AMG_CODED_WORDS(2)
            AMG_CODED_WORDS(3)
            AMG_CODED_WORDS(4)
            AMG_CODED_WORDS(5)
            AMG_CODED_WORDS(6)
            AMG_CODED_WORDS(8)
#undef AMG_CODED_WORDS
            default: no_instance(a.pc_kind, op, a.pc_words);
        }
    } else {
        switch (a.pc_words) {
#define AMG_CODED_WORDS(NW) \
    case NW: launch_restrict<T, NW>(AMG_CODED_ARGS); break;
            AMG_CODED_WORDS(2)
            AMG_CODED_WORDS(3)
            AMG_CODED_WORDS(4)
            AMG_CODED_WORDS(5)
            AMG_CODED_WORDS(6)
            AMG_CODED_WORDS(8)
            AMG_CODED_WORDS(10)
            AMG_CODED_WORDS(12)
            AMG_CODED_WORDS(16)
#undef AMG_CODED_WORDS
            default: no_instance(a.pc_kind, op, a.pc_words);
        }
    }
#undef AMG_CODED_ARGS
    return dot_op(op) ? coded_grid(a.rows) : 0;
}

// ---- building ------------------------------------------------------------------

// The pairs of one block of 256 rows, collected by one wavefront in a hash
// table in LDS: 64 rows at a time, entry by entry, a lane a row; the lanes that
// miss a pair claim places together and look again.  Place 0 is the padding.
constexpr unsigned kEmpty = 0xffffffffu;
template <int CB>
struct PairTable {
    static constexpr int kSlots = 2 * kLimit<CB>;
    long long val[kSlots];
    int off[kSlots];
    unsigned pos[kSlots];
    __device__ __forceinline__ unsigned find(int o, long long v) const {
        unsigned long long h = (unsigned long long)v * 0x9E3779B97F4A7C15ull;
        h ^= (unsigned long long)(unsigned)o * 0xC2B2AE3D27D4EB4Full;
        h ^= h >> 29;
        h *= 0xBF58476D1CE4E5B9ull;
        unsigned s = (unsigned)(h >> 33) & (kSlots - 1);
        while (pos[s] != kEmpty && !(off[s] == o && val[s] == v)) s = (s + 1) & (kSlots - 1);
        return s;
    }
};

// Calls each(slice, k, place) for every entry slot k of the block's 64-row
// slices, padding included, and each(slice, -1, width) at a slice's end;
// returns the number of places, kLimit + 1 if they do not suffice.
template <int CB, class F>
__device__ __forceinline__ int collect_pairs(PairTable<CB>& t, int blk, int rows, bool square,
                                             const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                             const double* __restrict__ v, int32_t* tabo, double* tabv, double* tabr,
                                             F&& each) {
    const int lane = (int)threadIdx.x & 63;
    for (int i = lane; i < PairTable<CB>::kSlots; i += 64) t.pos[i] = kEmpty;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    int cnt = 1;
    for (int s = 0; s < kBlock / 64; ++s) {
        const int r = blk * kBlock + s * 64 + lane;
        const int beg = r < rows ? rp[r] : 0, len = r < rows ? rp[r + 1] - beg : 0;
        const int base = square ? r : len > 0 ? ci[beg] : 0;
        int w = len;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, 64));
        for (int k = 0; k < w; ++k) {
            const bool in = k < len;
            const int o = in ? ci[beg + k] - base : 0;
            const long long bits = in ? __double_as_longlong(v[beg + k]) : 0ll;
            int place = in ? -1 : 0;
            for (;;) {
                unsigned slot = 0;
                if (place < 0) {
                    slot = t.find(o, bits);
                    if (t.pos[slot] != kEmpty) place = (int)t.pos[slot];
                }
                const bool miss = place < 0;
                if (!__any(miss)) break;
                // of the lanes at one empty slot, the one whose claim comes
                // first takes it; the others look again
                const bool won = miss && atomicCAS(&t.pos[slot], kEmpty, 0u) == kEmpty;
                const unsigned long long winners = __ballot(won);
                const int n = __popcll(winners);
                if (cnt + n > kLimit<CB>) return kLimit<CB> + 1;
                if (won) {
                    place = cnt + __popcll(winners & ((1ull << lane) - 1ull));
                    t.off[slot] = o;
                    t.val[slot] = bits;
                    t.pos[slot] = (unsigned)place;
                    if (tabo) {
                        const double x = __longlong_as_double(bits);
                        tabo[place] = o;
                        tabv[place] = x;
                        if (tabr) tabr[place] = 1.0 / x;
                    }
                }
                cnt += n;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            each(s, k, place);
        }
        each(s, -1, w);
    }
    return cnt;
}

template <int CB>
__global__ __launch_bounds__(64) void coded_count_kernel(int rows, bool square, const int32_t* __restrict__ rp,
                                                         const int32_t* __restrict__ ci,
                                                         const double* __restrict__ v, int32_t* most) {
    __shared__ PairTable<CB> t;
    // an operator that is already out needs no more counting
    if (__hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > kLimit<CB>) return;
    int widest = 0;
    const int n = collect_pairs<CB>(t, blockIdx.x, rows, square, rp, ci, v, nullptr, nullptr, nullptr,
                                    [&](int, int k, int w) {
                                        if (k < 0) widest = max(widest, w);
                                    });
    // thousands of atomics on one word take longer than the counting: only the
    // blocks that raise it
    if (threadIdx.x == 0) {
        if (__hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n) atomicMax(most, n);
        if (__hip_atomic_load(most + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < widest)
            atomicMax(most + 1, widest);
    }
}

template <int CB>
__global__ __launch_bounds__(64) void coded_fill_kernel(int rows, bool square, const int32_t* __restrict__ rp,
                                                        const int32_t* __restrict__ ci,
                                                        const double* __restrict__ v, int words,
                                                        uint32_t* __restrict__ word, int32_t* __restrict__ base,
                                                        int stride, int32_t* __restrict__ tabo,
                                                        double* __restrict__ tabv, double* __restrict__ tabr) {
    __shared__ PairTable<CB> t;
    constexpr int PER = 4 / CB;
    const int blk = blockIdx.x, lane = threadIdx.x;
    const size_t tb = (size_t)blk * stride;
    uint32_t* const w0 = word + (size_t)blk * words * kBlock + lane;
    uint32_t acc = 0;
    const int n = collect_pairs<CB>(t, blk, rows, square, rp, ci, v, tabo + tb, tabv + tb, tabr ? tabr + tb : nullptr,
                                    [&](int s, int k, int place) {
                                        if (k >= 0) {
                                            acc |= (uint32_t)place << (8 * CB * (k % PER));
                                            if (k % PER == PER - 1) {
                                                w0[k / PER * kBlock + s * 64] = acc;
                                                acc = 0;
                                            }
                                            return;
                                        }
                                        // the slice's end (place: its width): the words after its entries
                                        for (int q = place / PER; q < words; ++q) {
                                            w0[q * kBlock + s * 64] = acc;
                                            acc = 0;
                                        }
                                    });
    // the padding, and the places past the block's pairs
    for (int i = lane; i < stride; i += 64)
        if (i == 0 || i >= n) {
            tabo[tb + i] = 0;
            tabv[tb + i] = 0.0;
            if (tabr) tabr[tb + i] = 0.0;
        }
    if (base)
        for (int s = 0; s < kBlock / 64; ++s) {
            const int r = blk * kBlock + s * 64 + lane;
            if (r < rows) base[r] = rp[r + 1] > rp[r] ? ci[rp[r]] : 0;
        }
}

}  // namespace

int coded_limit(CodedKind kind) { return kind == kCodedRestrict ? kLimit<2> : kLimit<1>; }

int coded_words(CodedKind kind, int longest) {
    static const int kOne[] = {1, 2, 3, 4, 5, 6, 8}, kTwo[] = {2, 3, 4, 5, 6, 8, 10, 12, 16};
    if (kind == kCodedRestrict) {
        for (int w : kTwo)
            if (2 * w >= longest) return w;
    } else {
        for (int w : kOne)
            if (4 * w >= longest) return w;
    }
    return 0;
}

int launch_coded_op(RowOp op, const CsrView& a, const double* g, const double* u, const double* dinv, double omega,
                    double* y, double* y2, DotTarget dot, hipStream_t st) {
    return launch_op<double>(op, a, g, u, dinv, omega, y, y2, dot, st);
}

int launch_coded_op(RowOp op, const CsrView32& a, const float* g, const float* u, const float* dinv, float omega,
                    float* y, float* y2, DotTarget dot, hipStream_t st) {
    return launch_op<float>(op, a, g, u, dinv, omega, y, y2, dot, st);
}

int launch_coded_dual_resid(const CsrView& a_in, const double* g, const double* u, double* y, const double* g2,
                            const double* u2, double* y2, DotTarget dot, hipStream_t st) {
    const CsrView a = directed(a_in, true);
    const int grid = coded_grid(a.rows), nb = coded_blocks(a.rows);
    switch (a.pc_words) {
#define AMG_CODED_DUAL(NW) \
    case NW: launch(coded_dual_kernel<NW>, dim3(grid), st, a, g, u, y, g2, u2, y2, dot, nb); break;
        AMG_CODED_DUAL(1)
        AMG_CODED_DUAL(2)
        AMG_CODED_DUAL(3)
        AMG_CODED_DUAL(4)
        AMG_CODED_DUAL(5)
        AMG_CODED_DUAL(6)
        AMG_CODED_DUAL(8)
#undef AMG_CODED_DUAL
        default: return 0;
    }
    return grid;
}

void launch_coded_count(int rows, CodedKind kind, const int32_t* rp, const int32_t* ci, const double* v,
                        int32_t* most, hipStream_t st) {
    const dim3 grid(coded_blocks(rows));
    if (kind == kCodedRestrict)
        hipLaunchKernelGGL(coded_count_kernel<2>, grid, dim3(64), 0, st, rows, false, rp, ci, v, most);
    else
        hipLaunchKernelGGL(coded_count_kernel<1>, grid, dim3(64), 0, st, rows, kind == kCodedSquare, rp, ci, v, most);
}

void launch_coded_fill(int rows, CodedKind kind, const int32_t* rp, const int32_t* ci, const double* v, int words,
                       uint32_t* word, int32_t* base, int stride, int32_t* tabo, double* tabv, double* tabr,
                       hipStream_t st) {
    const dim3 grid(coded_blocks(rows));
    if (kind == kCodedRestrict)
        hipLaunchKernelGGL(coded_fill_kernel<2>, grid, dim3(64), 0, st, rows, false, rp, ci, v, words, word, base,
                           stride, tabo, tabv, tabr);
    else
        hipLaunchKernelGGL(coded_fill_kernel<1>, grid, dim3(64), 0, st, rows, kind == kCodedSquare, rp, ci, v, words,
                           word, base, stride, tabo, tabv, tabr);
}

}  // namespace amg355
