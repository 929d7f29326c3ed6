// Sparse products and transposes of the hierarchy setup, row by row: the rows
// of T = A P and C = P^T T are summed in tables in LDS, in the order in which
// the terms are listed, without the list ever reaching memory.
//
// A group of G lanes takes a row of the left factor and goes through its
// entries in order; the entries of the right factor's row, whose columns
// differ, go to the lanes.  Each finds its column in the group's hash table (or
// claims a slot) and adds its term there.  The steps of a group follow each
// other in one wave, so every sum takes its terms in list order, first term
// assigned: the bits of the listed, stably sorted and summed form, which moved
// 16 bytes of every term twelve times (sort passes of keys and values) where
// this reads the factors and writes the sums.  Bound by the latency of the
// gathers from the right factor (four rows are requested ahead) and of the LDS
// round trips of a step.  Lognormal FV 120^3 (PMIS), all levels: products and
// transposes 14 -> 4.5 ms, the setup 27.4 -> 9.5; the first A P (1.7 million rows,
// 39 million terms) takes 440 us, the first P^T (A P) (860,000 rows) 335.
//
// Rows are written where their number of terms lets them start (`off`), in
// ascending column order with their length beside: no pass that only counts.
// A row with more columns than its table holds is listed for a second kernel,
// whose table is larger; rows beyond that are counted, and the caller takes the
// sorted form for that product.
#include "setup_kernels.hpp"

#include "row_common.hpp"

#include <algorithm>
#include <climits>

// the order of every floating-point operation is the order written here
#pragma clang fp contract(off)

namespace amg355 {

namespace {

constexpr int kStepsAhead = 4;

// A table of H slots takes at most C columns, and holds few of them in most
// rows: every step waits for the longest search of the wave's lanes (with tables
// of half the slots coarse levels took 300 us a product, not 130).
struct Slot {
    int32_t key, pos;
};
constexpr size_t table_bytes(int H, int C) { return (size_t)H * sizeof(Slot) + (size_t)C * 16; }

// the wave's LDS writes before this point are seen by its lanes after it
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// ROWS: rows a group takes one after the other, its table cleared once
template <int G, int H, int C, int ROWS, bool LOOSE, bool LISTED>
__global__ __launch_bounds__(kBlock) void row_product_kernel(ProductArgs a, const int32_t* list,
                                                                            const int32_t* list_count,
                                                                            int32_t* over, int32_t* over_count) {
    extern __shared__ __align__(16) char lds[];
    static_assert(C % 4 == 0 && C < H);
    constexpr int kGroups = kBlock / G;
    constexpr int kShift = 32 - __builtin_ctz(H);
    const int group = threadIdx.x / G, lane = threadIdx.x % G;
    const int todo = LISTED ? *list_count : a.rows;
    const int chunk = LISTED ? 0 : (int)xcd_logical_block() * (kGroups * ROWS);
    if (LISTED ? (int)blockIdx.x * kGroups >= todo : chunk >= todo) return;
    // slots; then in the order the columns were claimed: sums, columns, slots
    Slot* tab = reinterpret_cast<Slot*>(lds + group * table_bytes(H, C));
    double* vals = reinterpret_cast<double*>(tab + H);
    int32_t* cols = reinterpret_cast<int32_t*>(vals + C);
    int32_t* slots = cols + C;
    for (int h = lane; h < H; h += G) tab[h].key = -1;
    wave_order();
    const int first_lane = (threadIdx.x & 63) - lane;
    const uint64_t group_mask = (G == 64 ? ~0ull : ((1ull << (G & 63)) - 1)) << first_lane;
    const uint64_t below = ((1ull << (threadIdx.x & 63)) - 1) & group_mask;
    const int begin = LISTED ? (int)blockIdx.x * kGroups + group : chunk + group;
    const int step = LISTED ? (int)gridDim.x * kGroups : kGroups;
    const int end = LISTED ? todo : min(todo, chunk + kGroups * ROWS);
    for (int at = begin; at < end; at += step) {
        const int row = LISTED ? list[at] : at;
        const int xb = a.xrp[row], xe = a.xrp[row + 1];
        int count = 0;
        bool fits = true;
        // one entry of the left factor: up to G columns
        auto add = [&](bool have, int J, double term) {
            bool claimed = false;
            int h = 0, pos = 0;
            if (have) {
                h = (int)(((uint32_t)J * 0x9E3779B1u) >> kShift);
                while (true) {
                    const Slot cur = tab[h];
                    pos = cur.pos;
                    if (cur.key == J) break;
                    if (cur.key == -1) {
                        claimed = atomicCAS(&tab[h].key, -1, J) == -1;
                        if (claimed) break;
                    }
                    h = (h + 1) & (H - 1);   // (a slot lost just now is another column's)
                }
            }
            const uint64_t news = __ballot(claimed) & group_mask;
            if (claimed) {
                pos = count + __popcll(news & below);
                tab[h].pos = pos;
                cols[pos] = J;
                slots[pos] = h;
            }
            if (have) vals[pos] = claimed ? term : vals[pos] + term;
            count += __popcll(news);
            wave_order();
        };
        for (int base = xb; base < xe && fits; base += G) {
            const bool have = base + lane < xe;
            int64_t start = 0;
            int len = 0;
            double x = 0.0;
            if (have) {
                const int l = a.xci[base + lane];
                x = a.xv[base + lane];
                if (LOOSE) {
                    start = a.yoff[l];
                    len = (int)a.ylen[l];
                } else {
                    start = a.yrp[l];
                    len = a.yrp[l + 1] - (int)start;
                }
            }
            const int here = min(G, xe - base);
            for (int e0 = 0; e0 < here && fits; e0 += kStepsAhead) {
                int64_t s[kStepsAhead];
                int n[kStepsAhead], J[kStepsAhead];
                double f[kStepsAhead], y[kStepsAhead];
#pragma unroll
                for (int u = 0; u < kStepsAhead; ++u) {
                    const int e = min(e0 + u, G - 1);
                    s[u] = __shfl(start, e, G);
                    n[u] = __shfl(len, e, G);
                    f[u] = __shfl(x, e, G);
                    if (e0 + u >= here) n[u] = 0;
                    J[u] = lane < n[u] ? a.yci[s[u] + lane] : 0;
                    y[u] = lane < n[u] ? a.yv[s[u] + lane] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < kStepsAhead; ++u) {
                    for (int c = 0; c < n[u]; c += G) {
                        fits = fits && count + G <= C;
                        if (!fits) break;
                        const bool in = c + lane < n[u];
                        if (c > 0 && in) {
                            J[u] = a.yci[s[u] + c + lane];
                            y[u] = a.yv[s[u] + c + lane];
                        }
                        add(in, J[u], f[u] * y[u]);
                    }
                }
            }
        }
        if (!fits && lane == 0) over[atomicAdd(over_count, 1)] = row;
        if (fits) {
            const int quads = (count + 3) / 4;
            if (lane < 4 * quads - count) cols[count + lane] = INT_MAX;
            wave_order();
            const int64_t o = a.off[row];
            for (int i = lane; i < count; i += G) {
                const int J = cols[i];
                int rank = 0;
                for (int q = 0; q < quads; ++q) {
                    const int4 c = reinterpret_cast<const int4*>(cols)[q];
                    rank += (c.x < J) + (c.y < J) + (c.z < J) + (c.w < J);
                }
                a.oci[o + rank] = J;
                a.ov[o + rank] = vals[i];
            }
        }
        for (int i = lane; i < count; i += G) tab[slots[i]].key = -1;
        if (lane == 0) a.olen[row] = fits ? count : 0;
        wave_order();
    }
}

// terms of each row (entry rows: 0), the most in most[0]
template <bool LOOSE>
__global__ __launch_bounds__(kBlock) void product_terms_kernel(int rows, const int32_t* __restrict__ xrp,
                                                               const int32_t* __restrict__ xci,
                                                               const int32_t* __restrict__ yrp,
                                                               const int64_t* __restrict__ ylen,
                                                               int64_t* __restrict__ terms, int32_t* most) {
    constexpr int G = 8;
    const int row = (int)(((int64_t)xcd_logical_block() * kBlock + threadIdx.x) / G), lane = threadIdx.x % G;
    int64_t c = 0;
    if (row < rows)
        for (int p = xrp[row] + lane; p < xrp[row + 1]; p += G) {
            const int l = xci[p];
            c += LOOSE ? ylen[l] : yrp[l + 1] - yrp[l];
        }
#pragma unroll
    for (int o = G / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, G);
    if (row <= rows && lane == 0) terms[row] = c;
    int top = (int)min<int64_t>(c, INT_MAX);
#pragma unroll
    for (int o = 32; o >= G; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
    if ((threadIdx.x & 63) == 0 && top > __hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(most, top);
}

// Entries of RB rows a workgroup, one a thread and turn: consecutive threads take
// consecutive entries and find their rows in the row pointers, kept in LDS.
// 256 rows, and 16 where that leaves fewer workgroups than the device holds.
constexpr int kFewRows = 65536;
template <int RB, class RP, class F>
__device__ __forceinline__ void for_entries(int rows, const RP* rp, F&& f) {
    __shared__ int64_t ptr[RB + 1];
    const int r0 = xcd_logical_block() * RB, here = min(RB, rows - r0);
    if (here <= 0) return;
    for (int t = threadIdx.x; t <= here; t += kBlock) ptr[t] = rp[r0 + t];
    __syncthreads();
    for (int64_t q = ptr[0] + threadIdx.x; q < ptr[here]; q += kBlock) {
        int lo = 0, hi = here;   // the last row that starts at or before q
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (ptr[mid] <= q) lo = mid;
            else hi = mid;
        }
        f(r0 + lo, q, ptr[lo], ptr[lo + 1]);
    }
}

// C in CSR from its loose rows, symmetrized: (c_ij + c_ji) / 2
template <int RB>
__global__ __launch_bounds__(kBlock) void pack_symmetrized_kernel(int n, const int64_t* __restrict__ off,
                                                                  const int64_t* __restrict__ len,
                                                                  const int32_t* __restrict__ lci,
                                                                  const double* __restrict__ lv,
                                                                  const int64_t* __restrict__ start,
                                                                  int32_t* __restrict__ rp, int32_t* __restrict__ ci,
                                                                  double* __restrict__ v, int* __restrict__ err) {
    const int r0 = xcd_logical_block() * RB;
    for (int t = threadIdx.x; t <= min(RB, n - r0); t += kBlock) rp[r0 + t] = (int32_t)start[r0 + t];
    for_entries<RB>(n, start, [&](int i, int64_t q, int64_t first, int64_t) {
        const int64_t p = off[i] + (q - first);
        const int j = lci[p];
        const int64_t b = off[j];
        int lo = 0, hi = (int)len[j];
        const int last = hi;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (lci[b + mid] < i) lo = mid + 1;
            else hi = mid;
        }
        ci[q] = j;
        if (lo < last && lci[b + lo] == i) {
            v[q] = 0.5 * (lv[p] + lv[b + lo]);
        } else {
            atomicOr(err, (int)kErrPattern);
            v[q] = lv[p];
        }
    });
}

// Transpose: every entry takes a place among those of its column, in any
// order; the rows of the transpose are then ordered by rank.
__global__ __launch_bounds__(kBlock) void column_places_kernel(int64_t nnz, const int32_t* __restrict__ ci,
                                                               int32_t* __restrict__ cnt,
                                                               int32_t* __restrict__ place, int32_t* most) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int top = 0;
    if (p < nnz) {
        const int k = atomicAdd(&cnt[ci[p]], 1);
        place[p] = k;
        top = k + 1;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
    if ((threadIdx.x & 63) == 0 && top > __hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(most, top);
}

template <int RB>
__global__ __launch_bounds__(kBlock) void column_fill_kernel(int rows, const int32_t* __restrict__ rp,
                                                             const int32_t* __restrict__ ci,
                                                             const double* __restrict__ v,
                                                             const int32_t* __restrict__ place,
                                                             const int32_t* __restrict__ trp,
                                                             int32_t* __restrict__ tci, double* __restrict__ tv) {
    for_entries<RB>(rows, rp, [&](int i, int64_t q, int64_t, int64_t) {
        const int64_t t = (int64_t)trp[ci[q]] + place[q];
        tci[t] = i;
        tv[t] = v[q];
    });
}

constexpr int kOrderStage = 4096;   // columns of a block kept in LDS

template <int RB>
__global__ __launch_bounds__(kBlock) void order_rows_kernel(int rows, const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ uci,
                                                            const double* __restrict__ uv,
                                                            int32_t* __restrict__ ci, double* __restrict__ v) {
    __shared__ int32_t col[kOrderStage];
    const int r0 = xcd_logical_block() * RB, r1 = min(rows, r0 + RB);
    if (r0 >= rows) return;
    const int64_t base = rp[r0];
    const bool staged = rp[r1] - base <= kOrderStage;
    if (staged)
        for (int64_t q = base + threadIdx.x; q < rp[r1]; q += kBlock) col[q - base] = uci[q];
    for_entries<RB>(rows, rp, [&](int, int64_t q, int64_t first, int64_t last) {
        const int me = uci[q];
        int rank = 0;
        if (staged)
            for (int64_t s = first; s < last; ++s) rank += col[s - base] < me;
        else
            for (int64_t s = first; s < last; ++s) rank += uci[s] < me;
        ci[first + rank] = me;
        v[first + rank] = uv[q];
    });
}

template <int G, int H, int C, bool LOOSE>
void launch_rows(const ProductArgs& a, int32_t* over, int32_t* over_count, hipStream_t st) {
    constexpr int groups = kBlock / G;
    constexpr size_t bytes = groups * table_bytes(H, C);
    static_assert(bytes <= 64 * 1024);
    // four rows a group once that leaves enough workgroups
    if (a.rows > kFewRows)
        hipLaunchKernelGGL((row_product_kernel<G, H, C, 4, LOOSE, false>),
                           dim3(round_up8((a.rows + 4 * groups - 1) / (4 * groups))), dim3(kBlock), bytes, st, a,
                           nullptr, nullptr, over, over_count);
    else
        hipLaunchKernelGGL((row_product_kernel<G, H, C, 1, LOOSE, false>),
                           dim3(round_up8((a.rows + groups - 1) / groups)), dim3(kBlock), bytes, st, a, nullptr,
                           nullptr, over, over_count);
}

// rows that the first kernel's tables do not hold
constexpr int kSecondTable = 1024, kSecondCap = 512;

template <bool LOOSE>
void launch_product(const ProductArgs& a, double mean_row, double mean_terms, int32_t* list, int32_t* counts,
                    hipStream_t st) {
    // lanes by the right factor's mean row, table by the mean number of terms: the
    // smallest that most rows fit, since the workgroups a CU holds hide the latency
    if (mean_row <= 4.0) {
        if (mean_terms <= 48.0) launch_rows<4, 32, 24, LOOSE>(a, list, counts, st);
        else launch_rows<8, 64, 48, LOOSE>(a, list, counts, st);
    } else if (mean_row <= 24.0) {
        if (mean_terms <= 160.0) launch_rows<16, 128, 64, LOOSE>(a, list, counts, st);
        else launch_rows<16, 256, 96, LOOSE>(a, list, counts, st);
    } else {
        launch_rows<64, 512, 256, LOOSE>(a, list, counts, st);
    }
    // their own list is not read any more when the next one's count is looked at:
    // it says only that there is one
    constexpr size_t bytes = kBlock / 64 * table_bytes(kSecondTable, kSecondCap);
    static_assert(bytes <= 64 * 1024);
    hipLaunchKernelGGL((row_product_kernel<64, kSecondTable, kSecondCap, 1, LOOSE, true>),
                       dim3(std::max(1, std::min(a.rows / (kBlock / 64), 512))), dim3(kBlock), bytes, st, a, list,
                       counts, list + a.rows, counts + 1);
}

}  // namespace

void launch_product_terms(const ProductArgs& a, int64_t* terms, int32_t* most, hipStream_t st) {
    const int blocks = round_up8((int)(((int64_t)(a.rows + 1) * 8 + kBlock - 1) / kBlock));
    if (a.yrp)
        hipLaunchKernelGGL(product_terms_kernel<false>, dim3(blocks), dim3(kBlock), 0, st, a.rows, a.xrp, a.xci, a.yrp,
                           a.ylen, terms, most);
    else
        hipLaunchKernelGGL(product_terms_kernel<true>, dim3(blocks), dim3(kBlock), 0, st, a.rows, a.xrp, a.xci, a.yrp,
                           a.ylen, terms, most);
}

void launch_row_product(const ProductArgs& a, double mean_row, double mean_terms, int32_t* list, int32_t* counts,
                        hipStream_t st) {
    if (a.yrp) launch_product<false>(a, mean_row, mean_terms, list, counts, st);
    else launch_product<true>(a, mean_row, mean_terms, list, counts, st);
}

void launch_pack_symmetrized(int n, const int64_t* off, const int64_t* len, const int32_t* lci, const double* lv,
                             const int64_t* start, int32_t* rp, int32_t* ci, double* v, int* err, hipStream_t st) {
    if (n > kFewRows) hipLaunchKernelGGL(pack_symmetrized_kernel<256>, dim3(round_up8((n + 255) / 256)), dim3(kBlock), 0, st, n, off, len, lci,
                       lv, start, rp, ci, v, err);
    else hipLaunchKernelGGL(pack_symmetrized_kernel<16>, dim3(round_up8((n + 15) / 16)), dim3(kBlock), 0, st, n, off, len, lci,
                       lv, start, rp, ci, v, err);
}

void launch_column_places(int64_t nnz, const int32_t* ci, int32_t* cnt, int32_t* place, int32_t* most,
                          hipStream_t st) {
    hipLaunchKernelGGL(column_places_kernel, dim3((unsigned)std::max<int64_t>(1, (nnz + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, st, nnz, ci, cnt, place, most);
}

void launch_column_fill(int rows, const int32_t* rp, const int32_t* ci, const double* v, const int32_t* place,
                        const int32_t* trp, int32_t* tci, double* tv, hipStream_t st) {
    if (rows > kFewRows) hipLaunchKernelGGL(column_fill_kernel<256>, dim3(round_up8((rows + 255) / 256)), dim3(kBlock), 0, st, rows, rp, ci, v,
                       place, trp, tci, tv);
    else hipLaunchKernelGGL(column_fill_kernel<16>, dim3(round_up8((rows + 15) / 16)), dim3(kBlock), 0, st, rows, rp, ci, v,
                       place, trp, tci, tv);
}

void launch_order_rows(int rows, const int32_t* rp, const int32_t* uci, const double* uv, int32_t* ci, double* v,
                       hipStream_t st) {
    if (rows > kFewRows) hipLaunchKernelGGL(order_rows_kernel<256>, dim3(round_up8((rows + 255) / 256)), dim3(kBlock), 0, st, rows, rp, uci, uv,
                       ci, v);
    else hipLaunchKernelGGL(order_rows_kernel<16>, dim3(round_up8((rows + 15) / 16)), dim3(kBlock), 0, st, rows, rp, uci, uv,
                       ci, v);
}

}  // namespace amg355
