// Device kernels of the hierarchy setup (Section 2, amg_setup).  Each kernel
// states the host-setup step it reproduces; the arithmetic of every value is
// the same sequence of IEEE operations in the same order, so the device
// hierarchy is bitwise the host one (for the same C/F split).
#include "setup_kernels.hpp"

#include "row_common.hpp"

#include <algorithm>
#include <climits>

// the order of every floating-point operation is the order written here
#pragma clang fp contract(off)

namespace amg355 {

namespace {

constexpr int kSB = 256;

int grid_of(int64_t n) {
    const int64_t b = (n + kSB - 1) / kSB;
    return round_up8((int)std::max<int64_t>(1, std::min<int64_t>(b, 16384)));
}

// neighbouring rows on one die: they gather from each other
#define GRID_STRIDE(i, n)                                                                       \
    for (int64_t i = (int64_t)xcd_logical_block() * blockDim.x + threadIdx.x; i < (int64_t)(n); \
         i += (int64_t)gridDim.x * blockDim.x)

__device__ inline int64_t find_col(const int32_t* ci, int64_t b, int64_t e, int col) {
    int64_t lo = b, hi = e;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ci[mid] < col) lo = mid + 1;
        else hi = mid;
    }
    return (lo < e && ci[lo] == col) ? lo : -1;
}

// ---------------------------------------------------------------------------
// input contract: 0-based non-decreasing row_ptr ending at nnz, in-range
// strictly ascending columns, finite values, positive stored diagonal,
// bitwise symmetry (a_ji stored with the same bits as a_ij)
// ---------------------------------------------------------------------------
// Eight lanes a row, so that neighbouring lanes read neighbouring entries
// (lognormal FV 120^3: 208 -> 145 us).
constexpr int kRowLanes = 8;

__global__ void validate_kernel(int n, int64_t nnz, const int32_t* __restrict__ rp,
                                const int32_t* __restrict__ ci, const double* __restrict__ v,
                                int* __restrict__ err) {
    const int lane = threadIdx.x % kRowLanes;
    GRID_STRIDE(t, (int64_t)n * kRowLanes) {
        const int i = (int)(t / kRowLanes);
        int bits = 0;
        const int64_t b = rp[i], e = rp[i + 1];
        if ((i == 0 && b != 0) || (i == n - 1 && e != nnz) || b < 0 || e < b || e > nnz) {
            bits = kErrRowPtr;
        } else {
            int diag = 0;
            for (int64_t p = b + lane; p < e; p += kRowLanes) {
                const int j = ci[p];
                if (j < 0 || j >= n) {
                    bits |= kErrColRange;
                    continue;
                }
                if (p > b && j <= ci[p - 1]) bits |= kErrColOrder;
                const double a = v[p];
                if (!isfinite(a)) bits |= kErrNonFinite;
                if (j == i) {
                    diag = 1;
                    if (!(a > 0.0)) bits |= kErrDiagSign;
                }
                const int64_t jb = rp[j], je = rp[j + 1];
                if (jb < 0 || je < jb || je > nnz) continue;   // row j reports its own pointers
                const int64_t q = find_col(ci, jb, je, i);
                if (q < 0 || __double_as_longlong(v[q]) != __double_as_longlong(a)) bits |= kErrAsymmetric;
            }
#pragma unroll
            for (int o = kRowLanes / 2; o > 0; o >>= 1) diag |= __shfl_xor(diag, o, kRowLanes);
            if (!diag) bits |= kErrNoDiag;
        }
        if (bits) {
            atomicOr(&err[0], bits);
            atomicMin(&err[1], i);
        }
    }
}

// ---------------------------------------------------------------------------
// A wave takes 64 rows, one a lane, whose entries it first brings into LDS with
// coalesced loads: a lane's walk through its row then costs LDS latency, not a
// cache line a step.  Rows that do not fit are walked in memory.  Lognormal FV
// 120^3, the second level (530,000 rows of 18), us: strength 465 + 507 in two
// walks with a scan and a readback between -> 104 in one, whose lists start where
// the rows of A do; interpolation 429 -> 111.
// ---------------------------------------------------------------------------
constexpr int kWaveRows = 64;

// rows a wave takes (fewer, if long, so that they fit) and the entries it has
// room for
struct Staging {
    int rows, cap;
};
Staging staging(int n, int64_t nnz) {
    const int64_t mean = n > 0 ? (nnz + n - 1) / n : 1;
    Staging s{kWaveRows, 0};
    while (s.rows > 4 && s.rows * (mean + mean / 4) > 2048) s.rows /= 2;
    s.cap = (int)std::min<int64_t>(4096, std::max<int64_t>(256, s.rows * (mean + mean / 4 + 1)));
    return s;
}

// ---------------------------------------------------------------------------
// strength: big = max(0, max_{k!=i} -a_ik); strong iff big > 0 and
// -a_ij >= fl(theta * big), j != i
// ---------------------------------------------------------------------------
__device__ inline bool strength_threshold(int i, int64_t b, int64_t e, const int32_t* ci, const double* v,
                                          double theta, double& thr) {
    double big = 0.0;
    for (int64_t p = b; p < e; ++p)
        if (ci[p] != i) {
            const double t = -v[p];
            big = (big < t) ? t : big;
        }
    thr = theta * big;
    return big > 0.0;
}

// the strong columns of row i, ascending, from sci[rp[i]] on (their number in
// cnt[i]), and lambda
__global__ __launch_bounds__(kWaveRows) void strength_kernel(int n, const int32_t* __restrict__ rp,
                                                             const int32_t* __restrict__ ci,
                                                             const double* __restrict__ v, double theta, Staging sg,
                                                             int32_t* __restrict__ cnt, int32_t* __restrict__ sci,
                                                             int32_t* __restrict__ lam) {
    extern __shared__ __align__(16) char lds[];
    double* lv = reinterpret_cast<double*>(lds);
    int32_t* lc = reinterpret_cast<int32_t*>(lv + sg.cap);
    const int r0 = xcd_logical_block() * sg.rows, r1 = min(n, r0 + sg.rows);
    if (r0 >= n) return;
    const int64_t base = rp[r0];
    const int total = (int)min<int64_t>(rp[r1] - base, INT_MAX);
    const int i = r0 + (int)threadIdx.x;
    const bool have = i < r1;
    const int64_t b = have ? rp[i] : 0, e = have ? rp[i + 1] : 0;
    // columns c and values w of the row, its list written to out
    auto row = [&](int64_t lo, int64_t hi, auto* c, auto* w, auto* out) {
        double thr;
        int k = 0;
        if (strength_threshold(i, lo, hi, c, w, theta, thr))
            for (int64_t p = lo; p < hi; ++p) {
                const int j = c[p];
                if (j != i && -w[p] >= thr) {
                    out[lo + k++] = j;
                    atomicAdd(&lam[j], 1);
                }
            }
        if (have) cnt[i] = k;
    };
    if (total > sg.cap) {
        row(b, e, ci, v, sci);
        return;
    }
#pragma unroll 4
    for (int q = threadIdx.x; q < total; q += kWaveRows) {
        lc[q] = ci[base + q];
        lv[q] = v[base + q];
    }
    __syncthreads();
    row(b - base, e - base, lc, lv, lc);   // in place: a list is no longer than its row
    __syncthreads();
    for (int q = threadIdx.x; q < total; q += kWaveRows) sci[base + q] = lc[q];
}

// ---------------------------------------------------------------------------
// PMIS
// ---------------------------------------------------------------------------
// SplitMix64 (Steele, Lea and Flood, OOPSLA 2014): output k >= 1 of the
// stream seeded with `seed` is the finaliser applied to seed + k * golden
__device__ inline uint64_t splitmix64_at(uint64_t seed, uint64_t k) {
    uint64_t z = seed + k * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void pmis_init_kernel(int n, const int32_t* __restrict__ lam, uint64_t seed, double* __restrict__ w,
                                 int32_t* __restrict__ state, int32_t* __restrict__ mark) {
    GRID_STRIDE(i, n) {
        const double u = (double)(splitmix64_at(seed, (uint64_t)i + 1) >> 11) * 0x1p-53;
        w[i] = (double)lam[i] + u;
        state[i] = lam[i] == 0 ? kPtF : kPtUndecided;
        mark[i] = 0;
    }
}

// i beats j: larger weight, equal weights: smaller index
__device__ inline bool beats(const double* w, int i, int j) { return w[i] > w[j] || (w[i] == w[j] && i < j); }

// every strong edge j -> k between undecided points marks its loser
__global__ void pmis_mark_kernel(int n, const int32_t* __restrict__ rp, const int32_t* __restrict__ cnt,
                                 const int32_t* __restrict__ sci, const double* __restrict__ w,
                                 const int32_t* __restrict__ state, int32_t* __restrict__ mark, int round,
                                 int32_t* __restrict__ undecided) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *undecided = 0;
    GRID_STRIDE(jj, n) {
        const int j = (int)jj;
        if (state[j] != kPtUndecided) continue;
        const int64_t b = rp[j], e = b + cnt[j];
        for (int64_t p = b; p < e; ++p) {
            const int k = sci[p];
            if (state[k] != kPtUndecided) continue;
            if (beats(w, j, k)) mark[k] = round;
            else mark[j] = round;
        }
    }
}

// undecided points without a mark of this round become C; those that depend
// strongly on a C point F; the rest are counted.  A point is C, whether its
// state says so yet or not, if it was undecided without a mark or C before, so
// what its neighbours find does not depend on the order of the threads.
__global__ __launch_bounds__(kSB) void pmis_decide_kernel(int n, const int32_t* __restrict__ rp,
                                                          const int32_t* __restrict__ cnt,
                                                          const int32_t* __restrict__ sci, int32_t* state,
                                                          const int32_t* __restrict__ mark, int round,
                                                          int32_t* __restrict__ undecided) {
    __shared__ int left[kSB / 64];
    int open = 0;
    GRID_STRIDE(jj, n) {
        const int j = (int)jj;
        if (state[j] != kPtUndecided) continue;
        if (mark[j] != round) {
            state[j] = kPtC;
            continue;
        }
        bool to_f = false;
        const int64_t b = rp[j], e = b + cnt[j];
        for (int64_t p = b; p < e && !to_f; ++p) {
            const int k = sci[p];
            const int sk = state[k];
            to_f = sk == kPtC || (sk == kPtUndecided && mark[k] != round);
        }
        if (to_f) state[j] = kPtF;
        else ++open;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) open += __shfl_xor(open, o, 64);
    if ((threadIdx.x & 63) == 0) left[threadIdx.x >> 6] = open;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kSB / 64; ++q) open += left[q];
        if (open) atomicAdd(undecided, open);
    }
}

// a C point's flag, and the entries of each row of P: a C point's one, an F
// point's strong C neighbours
__global__ void split_counts_kernel(int n, const int32_t* __restrict__ rp, const int32_t* __restrict__ cnt,
                                    const int32_t* __restrict__ sci, const int32_t* __restrict__ state,
                                    int32_t* __restrict__ flag, int32_t* __restrict__ pcnt) {
    GRID_STRIDE(ii, n) {
        const int i = (int)ii;
        const bool c = state[i] == kPtC;
        flag[i] = c;
        int k = 1;
        if (!c) {
            k = 0;
            const int64_t b = rp[i], e = b + cnt[i];
            for (int64_t p = b; p < e; ++p) k += state[sci[p]] == kPtC;
        }
        pcnt[i] = k;
    }
}

// the C points in order; code[i]: point i's coarse number, -1 for F points
__global__ void c_points_kernel(int n, const int32_t* __restrict__ state, const int32_t* __restrict__ cidx,
                                int32_t* __restrict__ c_points, int32_t* __restrict__ code) {
    GRID_STRIDE(i, n) {
        const bool c = state[i] == kPtC;
        code[i] = c ? cidx[i] : -1;
        if (c) c_points[cidx[i]] = (int32_t)i;
    }
}

// ---------------------------------------------------------------------------
// direct interpolation: C rows inject; an F row interpolates from its strong
// C neighbours with w_ij = -(alpha a_ij) / d, alpha = (sum of negative
// off-diagonals) / (sum of a_ij over strong C neighbours), d = a_ii + (sum
// of positive off-diagonals), every sum in ascending column order
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kWaveRows) void interp_fill_kernel(int n, const int32_t* __restrict__ rp,
                                                                const int32_t* __restrict__ ci,
                                                                const double* __restrict__ v, double theta, Staging sg,
                                                                const int32_t* __restrict__ code,
                                                                const int32_t* __restrict__ prp,
                                                                int32_t* __restrict__ pci, double* __restrict__ pv) {
    extern __shared__ __align__(16) char lds[];
    double* lv = reinterpret_cast<double*>(lds);
    int32_t* lc = reinterpret_cast<int32_t*>(lv + sg.cap);
    int32_t* lk = lc + sg.cap;
    const int r0 = xcd_logical_block() * sg.rows, r1 = min(n, r0 + sg.rows);
    if (r0 >= n) return;
    const int64_t base = rp[r0];
    const int total = (int)min<int64_t>(rp[r1] - base, INT_MAX);
    const int i = r0 + (int)threadIdx.x;
    const bool have = i < r1;
    const int64_t b = have ? rp[i] : 0, e = have ? rp[i + 1] : 0;
    int64_t w = have ? prp[i] : 0;
    const bool any = have && prp[i + 1] != w;
    const int mine = have ? code[i] : -1;
    // columns c, values x, and code_at(p) the code of entry p's column
    auto row = [&](int64_t lo, int64_t hi, auto* c, auto* x, auto code_at) {
        if (!any) return;
        if (mine >= 0) {
            pci[w] = mine;
            pv[w] = 1.0;
            return;
        }
        double thr;
        (void)strength_threshold(i, lo, hi, c, x, theta, thr);
        double dsum = 0.0;
        for (int64_t p = lo; p < hi; ++p)
            if (c[p] == i) dsum = x[p];
        double neg = 0.0, strong_c = 0.0;
        for (int64_t p = lo; p < hi; ++p) {
            if (c[p] == i) continue;
            const double t = x[p];
            if (t < 0.0) neg = neg + t;
            else if (t > 0.0) dsum = dsum + t;
            if (-t >= thr && code_at(p) >= 0) strong_c = strong_c + t;
        }
        const double alpha = neg / strong_c;
        for (int64_t p = lo; p < hi; ++p) {
            const double t = x[p];
            if (c[p] == i || !(-t >= thr)) continue;
            const int k = code_at(p);
            if (k < 0) continue;
            const double s = alpha * t;
            pci[w] = k;
            pv[w] = -s / dsum;
            ++w;
        }
    };
    if (total > sg.cap) {
        row(b, e, ci, v, [&](int64_t p) { return code[ci[p]]; });
        return;
    }
#pragma unroll 4
    for (int q = threadIdx.x; q < total; q += kWaveRows) {
        const int j = ci[base + q];
        lc[q] = j;
        lv[q] = v[base + q];
        lk[q] = code[j];
    }
    __syncthreads();
    row(b - base, e - base, lc, lv, [&](int64_t p) { return lk[p]; });
}

// ---------------------------------------------------------------------------
// transposes and products through sorted keys (row << col_bits | col): the
// general form, for products with rows and transposes with columns too long for
// the row kernels
// ---------------------------------------------------------------------------
__global__ void transpose_keys_kernel(int rows, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                      const double* __restrict__ v, int row_bits, uint64_t* __restrict__ keys,
                                      double* __restrict__ vals) {
    GRID_STRIDE(ii, rows) {
        const int i = (int)ii;
        for (int64_t p = rp[i]; p < rp[i + 1]; ++p) {
            keys[p] = ((uint64_t)(uint32_t)ci[p] << row_bits) | (uint64_t)(uint32_t)i;
            vals[p] = v[p];
        }
    }
}

// terms of each entry of X (nnz + 1 entries, the last 0)
template <bool LOOSE>
__global__ void entry_terms_kernel(ProductArgs a, int64_t nnz, int64_t* __restrict__ terms) {
    GRID_STRIDE(p, nnz + 1) {
        int64_t c = 0;
        if (p < nnz) {
            const int l = a.xci[p];
            c = LOOSE ? a.ylen[l] : a.yrp[l + 1] - a.yrp[l];
        }
        terms[p] = c;
    }
}

// The terms of X Y: row i lists, for each l of X's row in ascending order,
// x_il y_lJ over Y's row l.  G lanes an entry of X, which write next to each other;
// an entry finds its row in the row pointers.  Entries in parallel, not rows: the
// coarse rows of dense levels hold thousands of terms each (a thread a row, random
// graph of 20,000 vertices, all products: 17.9 ms; this 0.40).
template <int G, bool LOOSE>
__global__ __launch_bounds__(kSB) void expand_terms_kernel(ProductArgs a, int64_t nnz,
                                                           const int64_t* __restrict__ start, int col_bits,
                                                           uint64_t* __restrict__ keys, double* __restrict__ vals) {
    const int lane = threadIdx.x % G;
    GRID_STRIDE(t, nnz * G) {
        const int64_t p = t / G;
        int lo = 0, hi = a.rows;   // the last row that starts at or before p
        while (hi - lo > 1) {
            const int mid = lo + (hi - lo) / 2;
            if (a.xrp[mid] <= p) lo = mid;
            else hi = mid;
        }
        const uint64_t row = (uint64_t)(uint32_t)lo << col_bits;
        const int l = a.xci[p];
        const double x = a.xv[p];
        const int64_t o = start[p], len = start[p + 1] - o, b = LOOSE ? a.yoff[l] : a.yrp[l];
        for (int64_t q = lane; q < len; q += G) {
            keys[o + q] = row | (uint64_t)(uint32_t)a.yci[b + q];
            vals[o + q] = x * a.yv[b + q];
        }
    }
}

__global__ void loose_rows_kernel(int rows, const int32_t* __restrict__ rp, int64_t* __restrict__ off,
                                  int64_t* __restrict__ len) {
    GRID_STRIDE(i, (int64_t)rows + 1) {
        off[i] = rp[i];
        len[i] = i < rows ? rp[i + 1] - rp[i] : 0;
    }
}

// flags has m + 1 entries (the last 0)
__global__ void run_heads_kernel(int64_t m, const uint64_t* __restrict__ keys, int64_t* __restrict__ flags) {
    GRID_STRIDE(q, m + 1) flags[q] = q < m && (q == 0 || keys[q] != keys[q - 1]);
}

__global__ void run_sums_kernel(int64_t m, const uint64_t* __restrict__ keys, const double* __restrict__ vals,
                                const int64_t* __restrict__ head_index, int col_bits, int32_t* __restrict__ out_ci,
                                double* __restrict__ out_v, uint64_t* __restrict__ out_keys) {
    const uint64_t mask = (1ull << col_bits) - 1;
    GRID_STRIDE(q, m) {
        const uint64_t key = keys[q];
        if (q > 0 && keys[q - 1] == key) continue;
        double sum = vals[q];
        for (int64_t r = q + 1; r < m && keys[r] == key; ++r) sum = sum + vals[r];
        const int64_t s = head_index[q];
        out_ci[s] = (int32_t)(key & mask);
        out_v[s] = sum;
        out_keys[s] = key;
    }
}

__global__ void rowptr_from_keys_kernel(int64_t m, const uint64_t* __restrict__ keys, int col_bits, int rows,
                                        int32_t* __restrict__ rp) {
    if (m == 0) {
        GRID_STRIDE(c, (int64_t)rows + 1) rp[c] = 0;
        return;
    }
    GRID_STRIDE(q, m) {
        const int64_t r = (int64_t)(keys[q] >> col_bits);
        const int64_t prev = q == 0 ? -1 : (int64_t)(keys[q - 1] >> col_bits);
        for (int64_t c = prev + 1; c <= r; ++c) rp[c] = (int32_t)q;
        if (q == m - 1)
            for (int64_t c = r + 1; c <= rows; ++c) rp[c] = (int32_t)m;
    }
}

__global__ void unpack_keys_kernel(int64_t m, const uint64_t* __restrict__ keys, const double* __restrict__ vals,
                                   int col_bits, int32_t* __restrict__ ci, double* __restrict__ v) {
    const uint64_t mask = (1ull << col_bits) - 1;
    GRID_STRIDE(q, m) {
        ci[q] = (int32_t)(keys[q] & mask);
        v[q] = vals[q];
    }
}

__global__ void publish_words_kernel(PublishWords w, int64_t* host, uint32_t* flag, uint32_t seq) {
    const int t = threadIdx.x;
    if (t < w.count)
        host_store(host + t, w.bytes[t] == 8 ? *static_cast<const int64_t*>(w.src[t])
                                             : (int64_t) * static_cast<const int32_t*>(w.src[t]));
    host_flag(flag, seq);
}

}  // namespace

void launch_validate_csr(int n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v, int* err,
                         hipStream_t st) {
    hipLaunchKernelGGL(validate_kernel, dim3(grid_of((int64_t)n * kRowLanes)), dim3(kSB), 0, st, n, nnz, rp, ci, v, err);
}

void launch_strength(int n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v, double theta,
                     int32_t* cnt, int32_t* sci, int32_t* lam, hipStream_t st) {
    const Staging sg = staging(n, nnz);
    hipLaunchKernelGGL(strength_kernel, dim3(round_up8((n + sg.rows - 1) / sg.rows)), dim3(kWaveRows), (size_t)sg.cap * 12, st, n,
                       rp, ci, v, theta, sg, cnt, sci, lam);
}

void launch_pmis_init(int n, const int32_t* lam, uint64_t seed, double* w, int32_t* state, int32_t* mark,
                      hipStream_t st) {
    hipLaunchKernelGGL(pmis_init_kernel, dim3(grid_of(n)), dim3(kSB), 0, st, n, lam, seed, w, state, mark);
}

void launch_pmis_round(int n, const int32_t* rp, const int32_t* cnt, const int32_t* sci, const double* w,
                       int32_t* state, int32_t* mark, int round, int32_t* undecided, hipStream_t st) {
    hipLaunchKernelGGL(pmis_mark_kernel, dim3(grid_of(n)), dim3(kSB), 0, st, n, rp, cnt, sci, w, state, mark, round,
                       undecided);
    hipLaunchKernelGGL(pmis_decide_kernel, dim3(grid_of(n)), dim3(kSB), 0, st, n, rp, cnt, sci, state, mark, round,
                       undecided);
}

void launch_split_counts(int n, const int32_t* rp, const int32_t* cnt, const int32_t* sci, const int32_t* state,
                         int32_t* flag, int32_t* pcnt, hipStream_t st) {
    hipLaunchKernelGGL(split_counts_kernel, dim3(grid_of(n)), dim3(kSB), 0, st, n, rp, cnt, sci, state, flag, pcnt);
}

void launch_c_points(int n, const int32_t* state, const int32_t* cidx, int32_t* c_points, int32_t* code,
                     hipStream_t st) {
    hipLaunchKernelGGL(c_points_kernel, dim3(grid_of(n)), dim3(kSB), 0, st, n, state, cidx, c_points, code);
}

void launch_interp_fill(int n, int64_t nnz, const int32_t* rp, const int32_t* ci, const double* v, double theta,
                        const int32_t* code, const int32_t* prp, int32_t* pci, double* pv, hipStream_t st) {
    const Staging sg = staging(n, nnz);
    hipLaunchKernelGGL(interp_fill_kernel, dim3(round_up8((n + sg.rows - 1) / sg.rows)), dim3(kWaveRows), (size_t)sg.cap * 16, st,
                       n, rp, ci, v, theta, sg, code, prp, pci, pv);
}

void launch_transpose_keys(int rows, const int32_t* rp, const int32_t* ci, const double* v, int row_bits,
                           uint64_t* keys, double* vals, hipStream_t st) {
    hipLaunchKernelGGL(transpose_keys_kernel, dim3(grid_of(rows)), dim3(kSB), 0, st, rows, rp, ci, v, row_bits,
                       keys, vals);
}

void launch_entry_terms(const ProductArgs& a, int64_t nnz, int64_t* terms, hipStream_t st) {
    const dim3 grid(grid_of(nnz + 1));
    if (a.yrp) hipLaunchKernelGGL(entry_terms_kernel<false>, grid, dim3(kSB), 0, st, a, nnz, terms);
    else hipLaunchKernelGGL(entry_terms_kernel<true>, grid, dim3(kSB), 0, st, a, nnz, terms);
}

namespace {
template <int G>
void expand_terms(const ProductArgs& a, int64_t nnz, const int64_t* start, int col_bits, uint64_t* keys,
                  double* vals, hipStream_t st) {
    const dim3 grid(grid_of(nnz * G));
    if (a.yrp)
        hipLaunchKernelGGL((expand_terms_kernel<G, false>), grid, dim3(kSB), 0, st, a, nnz, start, col_bits, keys, vals);
    else
        hipLaunchKernelGGL((expand_terms_kernel<G, true>), grid, dim3(kSB), 0, st, a, nnz, start, col_bits, keys, vals);
}
}  // namespace

void launch_expand_terms(const ProductArgs& a, int64_t nnz, int64_t m, const int64_t* start, int col_bits,
                         uint64_t* keys, double* vals, hipStream_t st) {
    // lanes by the mean number of terms of an entry
    if (m <= 8 * nnz) expand_terms<4>(a, nnz, start, col_bits, keys, vals, st);
    else if (m <= 32 * nnz) expand_terms<16>(a, nnz, start, col_bits, keys, vals, st);
    else expand_terms<64>(a, nnz, start, col_bits, keys, vals, st);
}

void launch_loose_rows(int rows, const int32_t* rp, int64_t* off, int64_t* len, hipStream_t st) {
    hipLaunchKernelGGL(loose_rows_kernel, dim3(grid_of((int64_t)rows + 1)), dim3(kSB), 0, st, rows, rp, off, len);
}

void launch_run_heads(int64_t m, const uint64_t* keys, int64_t* flags, hipStream_t st) {
    hipLaunchKernelGGL(run_heads_kernel, dim3(grid_of(m + 1)), dim3(kSB), 0, st, m, keys, flags);
}

void launch_run_sums(int64_t m, const uint64_t* keys, const double* vals, const int64_t* head_index,
                     int col_bits, int32_t* out_ci, double* out_v, uint64_t* out_keys, hipStream_t st) {
    hipLaunchKernelGGL(run_sums_kernel, dim3(grid_of(m)), dim3(kSB), 0, st, m, keys, vals, head_index, col_bits,
                       out_ci, out_v, out_keys);
}

void launch_rowptr_from_keys(int64_t m, const uint64_t* keys, int col_bits, int rows, int32_t* rp,
                             hipStream_t st) {
    hipLaunchKernelGGL(rowptr_from_keys_kernel, dim3(grid_of(std::max<int64_t>(m, (int64_t)rows + 1))),
                       dim3(kSB), 0, st, m, keys, col_bits, rows, rp);
}

void launch_unpack_keys(int64_t m, const uint64_t* keys, const double* vals, int col_bits, int32_t* ci,
                        double* v, hipStream_t st) {
    hipLaunchKernelGGL(unpack_keys_kernel, dim3(grid_of(m)), dim3(kSB), 0, st, m, keys, vals, col_bits, ci, v);
}

void launch_publish_words(const PublishWords& w, int64_t* host, uint32_t* flag, uint32_t seq, hipStream_t st) {
    hipLaunchKernelGGL(publish_words_kernel, dim3(1), dim3(64), 0, st, w, host, flag, seq);
}

namespace {

// ---------------------------------------------------------------------------
// Exclusive scan of int64 counts and a stable LSD radix sort of (key, value)
// pairs: the sort that groups the Galerkin product's terms by (row, column)
// and the transpose's entries by (column, row).
// ---------------------------------------------------------------------------

// scan: 4,096 entries per block (256 threads, 16 consecutive entries each)
constexpr int kScanPer = 16;
constexpr int kScanTile64 = kSB * kScanPer;

// block-wide exclusive scan of one int64 per thread (wave shuffles, then the
// four wave totals through LDS); *total receives the block's sum
__device__ __forceinline__ int64_t block_exclusive_scan64(int64_t v, int64_t* wsum, int64_t* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < kSB / 64; ++k) {
        if (k < w) before += wsum[k];
        all += wsum[k];
    }
    *total = all;
    __syncthreads();
    return before + incl - v;
}

__global__ __launch_bounds__(kSB) void scan64_reduce_kernel(int64_t n, const int64_t* __restrict__ in,
                                                            int64_t* __restrict__ bsum) {
    __shared__ int64_t wsum[kSB / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile64;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const int64_t i = base + (int64_t)k * kSB + threadIdx.x;
        if (i < n) s += in[i];
    }
    int64_t tot;
    block_exclusive_scan64(s, wsum, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// the block sums, scanned in place by one workgroup of 1,024 threads, each
// owning a contiguous range
__global__ __launch_bounds__(1024) void scan64_blocks_kernel(int64_t nb, int64_t* bsum) {
    __shared__ int64_t part[1024];
    const int64_t per = (nb + 1023) / 1024;
    const int64_t lo = threadIdx.x * per, hi = std::min<int64_t>(nb, lo + per);
    int64_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += bsum[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int64_t t = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
        __syncthreads();
        part[threadIdx.x] += t;
        __syncthreads();
    }
    int64_t run = part[threadIdx.x] - s;
    for (int64_t i = lo; i < hi; ++i) {
        const int64_t v = bsum[i];
        bsum[i] = run;
        run += v;
    }
}

// each thread scans its 16 consecutive entries after the block-wide scan of
// the thread sums; entries staged through LDS so that both the loads and the
// stores are coalesced
__global__ __launch_bounds__(kSB) void scan64_apply_kernel(int64_t n, const int64_t* __restrict__ in,
                                                           const int64_t* __restrict__ boff,
                                                           int64_t* __restrict__ out) {
    __shared__ int64_t tile[kScanTile64 + kScanTile64 / 32];
    __shared__ int64_t wsum[kSB / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile64;
    // padded index: one spare slot every 32 entries keeps a thread's 16
    // consecutive entries off each other's LDS banks
    auto at = [](int i) { return i + (i >> 5); };
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const int i = k * kSB + threadIdx.x;
        tile[at(i)] = base + i < n ? in[base + i] : 0;
    }
    __syncthreads();
    int64_t v[kScanPer];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        v[k] = tile[at(threadIdx.x * kScanPer + k)];
        s += v[k];
    }
    int64_t tot;
    int64_t run = block_exclusive_scan64(s, wsum, &tot) + boff[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        tile[at(threadIdx.x * kScanPer + k)] = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const int i = k * kSB + threadIdx.x;
        if (base + i < n) out[base + i] = tile[at(i)];
    }
}

int64_t scan64_blocks(int64_t n) { return std::max<int64_t>(1, (n + kScanTile64 - 1) / kScanTile64); }

void launch_scan64(int64_t n, const int64_t* in, int64_t* out, int64_t* bsum, hipStream_t st) {
    const int64_t nb = scan64_blocks(n);
    hipLaunchKernelGGL(scan64_reduce_kernel, dim3((unsigned)nb), dim3(kSB), 0, st, n, in, bsum);
    hipLaunchKernelGGL(scan64_blocks_kernel, dim3(1), dim3(1024), 0, st, nb, bsum);
    hipLaunchKernelGGL(scan64_apply_kernel, dim3((unsigned)nb), dim3(kSB), 0, st, n, in, bsum, out);
}

// radix sort: 8-bit digits, 4,096 pairs per block (16 rounds of 256, pair
// r * 256 + t of the block held by thread t), so that a block's pairs in
// round order are its pairs in input order
constexpr int kRadixBits = 8;
constexpr int kRadixBins = 1 << kRadixBits;
constexpr int kRadixRounds = 16;
constexpr int kRadixTile = kSB * kRadixRounds;
static_assert(kRadixBins == kSB, "one digit per thread in the offset steps");

// lanes of this wave holding the same digit (lanes with valid = false take
// part in no group); eight ballots, one per digit bit
__device__ __forceinline__ uint64_t same_digit_lanes(int d, bool valid) {
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
        const uint64_t ones = __ballot((d >> b) & 1);
        peers &= ((d >> b) & 1) ? ones : ~ones;
    }
    return peers;
}

__device__ __forceinline__ uint64_t lanes_below() {
    return (1ull << (threadIdx.x & 63)) - 1ull;
}

// per-block digit counts, digit-major: cnt[d * nb + block]
__global__ __launch_bounds__(kSB) void radix_count_kernel(int64_t m, int shift, const uint64_t* __restrict__ keys,
                                                          int64_t* __restrict__ cnt, int64_t nb) {
    __shared__ int hist[kRadixBins];
    hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
    uint64_t k[kRadixRounds];
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r) {
        const int64_t e = base + (int64_t)r * kSB + threadIdx.x;
        k[r] = e < m ? keys[e] : 0;
    }
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r) {
        const bool valid = base + (int64_t)r * kSB + threadIdx.x < m;
        const int d = (int)((k[r] >> shift) & (kRadixBins - 1));
        const uint64_t peers = same_digit_lanes(d, valid);
        // the lowest lane of each group adds the group's size
        if (valid && (peers & lanes_below()) == 0) atomicAdd(&hist[d], __popcll(peers));
    }
    __syncthreads();
    cnt[(int64_t)threadIdx.x * nb + blockIdx.x] = hist[threadIdx.x];
}

// block-wide exclusive scan of one int per thread (kSB threads)
__device__ __forceinline__ int block_exclusive_scan_i32(int v, int* wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int k = 0; k < kSB / 64; ++k)
        if (k < w) before += wsum[k];
    __syncthreads();
    return before + incl - v;
}

// stable scatter.  Pair (r, t) of the block (held by thread t in round r)
// takes slot tstart[d] + (pairs of digit d in earlier rounds) + (in earlier
// waves of this round) + (in lower lanes of its wave) of the block's tile,
// tstart the block's exclusive scan of its digit counts, so that the slots
// hold the tile's pairs sorted stably by digit.  The pairs are staged in LDS
// in slot order, keys and then values, and written out slot by slot: slot q
// of digit d goes to first[d] + q - tstart[d], so consecutive threads write
// consecutive positions of one digit's run.
__global__ __launch_bounds__(kSB) void radix_scatter_kernel(int64_t m, int shift,
                                                            const uint64_t* __restrict__ kin,
                                                            const double* __restrict__ vin,
                                                            uint64_t* __restrict__ kout,
                                                            double* __restrict__ vout,
                                                            const int64_t* __restrict__ cnt,
                                                            const int64_t* __restrict__ first, int64_t nb) {
    constexpr int kWaves = kSB / 64;
    __shared__ int next[kRadixBins];              // next free slot per digit
    __shared__ int wcnt[kWaves][kRadixBins];      // this round's count per wave and digit
    __shared__ int wpos[kWaves][kRadixBins];      // this round's first slot per wave and digit
    __shared__ int64_t gbase[kRadixBins];         // output position of slot 0 of each digit
    __shared__ int wsum[kWaves];
    __shared__ uint64_t stage[kRadixTile];
    const int t = threadIdx.x, w = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
    uint64_t k[kRadixRounds];
    double v[kRadixRounds];
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r) {
        const int64_t e = base + (int64_t)r * kSB + t;
        k[r] = e < m ? kin[e] : 0;
        v[r] = e < m ? vin[e] : 0.0;
    }
    const int64_t ci = (int64_t)t * nb + blockIdx.x;
    const int tstart = block_exclusive_scan_i32((int)cnt[ci], wsum);
    next[t] = tstart;
    gbase[t] = first[ci] - tstart;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) wcnt[q][t] = 0;
    __syncthreads();
    int slot[kRadixRounds];
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r) {
        const bool valid = base + (int64_t)r * kSB + t < m;
        const int d = (int)((k[r] >> shift) & (kRadixBins - 1));
        const uint64_t peers = same_digit_lanes(d, valid);
        const int rank = __popcll(peers & lanes_below());
        if (valid && rank == 0) wcnt[w][d] = __popcll(peers);
        __syncthreads();
        {
            // thread t owns digit t: first slots of its waves, then clear
            int p = next[t];
#pragma unroll
            for (int q = 0; q < kWaves; ++q) {
                wpos[q][t] = p;
                p += wcnt[q][t];
                wcnt[q][t] = 0;
            }
            next[t] = p;
        }
        __syncthreads();
        slot[r] = valid ? wpos[w][d] + rank : -1;
    }
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r)
        if (slot[r] >= 0) stage[slot[r]] = k[r];
    __syncthreads();
    const int here = (int)min<int64_t>(kRadixTile, m - base);
    int dq[kRadixRounds];
#pragma unroll
    for (int q = 0; q < kRadixRounds; ++q) {
        const int idx = q * kSB + t;
        dq[q] = 0;
        if (idx < here) {
            const uint64_t key = stage[idx];
            dq[q] = (int)((key >> shift) & (kRadixBins - 1));
            kout[gbase[dq[q]] + idx] = key;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRadixRounds; ++r)
        if (slot[r] >= 0) stage[slot[r]] = __double_as_longlong(v[r]);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRadixRounds; ++q) {
        const int idx = q * kSB + t;
        if (idx < here) vout[gbase[dq[q]] + idx] = __longlong_as_double((long long)stage[idx]);
    }
}

size_t align_up(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

hipError_t sort_pairs(void* temp, size_t& temp_bytes, uint64_t* keys[2], double* vals[2], int64_t m, int bits,
                      int& result, hipStream_t st) {
    const int64_t nb = std::max<int64_t>(1, (m + kRadixTile - 1) / kRadixTile);
    const int64_t ncnt = nb * kRadixBins;
    const size_t cnt_bytes = align_up(sizeof(int64_t) * (size_t)ncnt);
    const size_t need = 2 * cnt_bytes + align_up(sizeof(int64_t) * (size_t)scan64_blocks(ncnt));
    const int passes = (std::max(bits, 0) + kRadixBits - 1) / kRadixBits;
    result = passes & 1;
    if (temp == nullptr) {
        temp_bytes = need;
        return hipSuccess;
    }
    if (temp_bytes < need) return hipErrorInvalidValue;
    if (m <= 0) return hipSuccess;
    if (nb > INT_MAX) return hipErrorInvalidValue;
    int64_t* cnt = static_cast<int64_t*>(temp);
    int64_t* first = reinterpret_cast<int64_t*>(static_cast<char*>(temp) + cnt_bytes);
    int64_t* bsum = reinterpret_cast<int64_t*>(static_cast<char*>(temp) + 2 * cnt_bytes);
    for (int p = 0; p < passes; ++p) {
        const int src = p & 1, dst = src ^ 1, shift = p * kRadixBits;
        hipLaunchKernelGGL(radix_count_kernel, dim3((unsigned)nb), dim3(kSB), 0, st, m, shift, keys[src], cnt, nb);
        launch_scan64(ncnt, cnt, first, bsum, st);
        hipLaunchKernelGGL(radix_scatter_kernel, dim3((unsigned)nb), dim3(kSB), 0, st, m, shift, keys[src],
                           vals[src], keys[dst], vals[dst], cnt, first, nb);
    }
    return hipGetLastError();
}

hipError_t scan_counts(void* temp, size_t& temp_bytes, const int64_t* in, int64_t* out, int64_t m,
                       hipStream_t st) {
    const int64_t n = m + 1;
    const size_t need = align_up(sizeof(int64_t) * (size_t)scan64_blocks(n));
    if (temp == nullptr) {
        temp_bytes = need;
        return hipSuccess;
    }
    if (temp_bytes < need || scan64_blocks(n) > INT_MAX) return hipErrorInvalidValue;
    launch_scan64(n, in, out, static_cast<int64_t*>(temp), st);
    return hipGetLastError();
}

}  // namespace amg355
