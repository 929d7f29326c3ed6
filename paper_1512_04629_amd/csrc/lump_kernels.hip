// Strong-neighbour lumping kernels: every sum and share in the order the
// definition fixes (ascending columns; shares of a target in ascending order
// of their source entry), contraction off.  The threshold and the copy run
// one wave per row; the copy also lists every row's dropped entries, from
// rp[i] - new_rp[i] on.  The shares run a wave per row by those lists, rows of
// many dropped entries a workgroup with the row staged in LDS; the denominators
// the same or, on levels of short rows, a wave per row with its own stage (rows
// longer than the stage, and a launch forced to it, one wave per row without a
// stage or lists).
#include "lump_kernels.hpp"

#include "row_common.hpp"

#include <algorithm>
#include <cmath>
#include <cstdlib>

#pragma clang fp contract(off)

namespace amg355 {

namespace {

constexpr int kLB = 256;
constexpr int kWaves = kLB / 64;
constexpr int kWideCap = 256;   // row entries a workgroup stages in LDS (15 KB: eight workgroups a CU)
// below this mean row length, on levels with enough rows to fill the device
// with waves, the denominators run a wave per row with its own LDS stage
// (measured on 3D Poisson: faster at 174,772 and 27,542 rows of 34 and 57
// entries, slower at 129 rows of 65 and from 108 entries a row)
constexpr double kDenWaveMeanRow = 80.0;
constexpr int kDenWaveMinRows = 16384;

int wave_grid_of(int n) { return round_up8(std::max(1, std::min((n + kWaves - 1) / kWaves, 65536))); }

__device__ inline int find_in_row(const int32_t* ci, int b, int e, int col) {
    int lo = b, hi = e;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ci[mid] < col) lo = mid + 1;
        else hi = mid;
    }
    return (lo < e && ci[lo] == col) ? lo : -1;
}

__device__ inline bool strong_at(const int32_t* ci, const double* v, const double* thr, int j, int r) {
    return ci[r] != j && thr[j] > 0.0 && -v[r] >= thr[j];
}

// one wave per row i (kWaves per workgroup), lanes over the row's entries
// (neighbouring rows on one die: they read each other's rows)
#define WAVE_ROW_LOOP(i, n)                                                                               \
    for (int i = xcd_logical_block() * kWaves + (int)(threadIdx.x >> 6); i < (n); i += gridDim.x * kWaves)

// one wave per row: the kept entries of each 64-entry chunk go to the next
// free places in order (ballot, count of the lower lanes' kept entries)
__global__ void __launch_bounds__(kLB) compact_copy_kernel(int n, const int32_t* __restrict__ rp,
                                                           const int32_t* __restrict__ ci,
                                                           const double* __restrict__ v,
                                                           const uint8_t* __restrict__ keep,
                                                           const int32_t* __restrict__ new_rp,
                                                           int32_t* __restrict__ new_ci, double* __restrict__ new_v,
                                                           int32_t* __restrict__ dropped, int32_t* heavy_count) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) *heavy_count = 0;
    WAVE_ROW_LOOP(i, n) {
        const int ie = rp[i + 1];
        int w = new_rp[i];
        for (int p0 = rp[i]; p0 < ie; p0 += 64) {
            const int p = p0 + lane;
            const bool kp = p < ie && keep[p];
            const uint64_t mask = __ballot(kp);
            const int at = w + __popcll(mask & below);   // kept entries before p
            if (kp) {
                new_ci[at] = ci[p];
                new_v[at] = v[p];
            } else if (p < ie) {
                dropped[p - at] = p;
            }
            w += __popcll(mask);
        }
    }
}

// one wave per row: the largest -a_jm off the diagonal (a maximum, the same
// in any order)
__global__ void __launch_bounds__(kLB) lump_threshold_kernel(int n, const int32_t* __restrict__ rp,
                                                             const int32_t* __restrict__ ci,
                                                             const double* __restrict__ v, double theta,
                                                             double* __restrict__ thr) {
    const int lane = threadIdx.x & 63;
    WAVE_ROW_LOOP(j, n) {
        double big = 0.0;
        for (int p = rp[j] + lane; p < rp[j + 1]; p += 64)
            if (ci[p] != j && -v[p] > big) big = -v[p];
        for (int o = 32; o > 0; o >>= 1) {
            const double other = __shfl_xor(big, o);
            if (other > big) big = other;
        }
        if (lane == 0) thr[j] = big > 0.0 ? theta * big : -1.0;
    }
}

// den of every dropped entry of row i, one wave: a lane per dropped entry;
// the strong neighbours m of j in ascending order are matched against the
// ascending columns of row i by a merge walk
__device__ inline void lump_den_row(int i, int lane, const int32_t* rp, const int32_t* ci, const double* v,
                                    const uint8_t* keep, const double* thr, double* den) {
    const int ib = rp[i], ie = rp[i + 1];
    for (int p = ib + lane; p < ie; p += 64) {
        const int j = ci[p];
        if (j == i || keep[p]) continue;
        double d = 0.0;
        int w = ib;
        for (int r = rp[j]; r < rp[j + 1]; ++r) {
            if (!strong_at(ci, v, thr, j, r)) continue;
            const int m = ci[r];
            while (w < ie && ci[w] < m) ++w;
            if (w < ie && ci[w] == m && keep[w]) d = d + fabs(v[r]);
        }
        den[p] = d;
    }
}

__global__ void __launch_bounds__(kLB) lump_den_kernel(int n, const int32_t* __restrict__ rp,
                                                       const int32_t* __restrict__ ci,
                                                       const double* __restrict__ v,
                                                       const uint8_t* __restrict__ keep,
                                                       const double* __restrict__ thr, double* __restrict__ den) {
    const int lane = threadIdx.x & 63;
    WAVE_ROW_LOOP(i, n) { lump_den_row(i, lane, rp, ci, v, keep, thr, den); }
}

// First position w in the ascending a[0..len) with a[w] >= col.
__device__ inline int lower_bound_lds(const int32_t* a, int len, int col) {
    int lo = 0, hi = len;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < col) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ inline double lane_value(double x, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Ordered sum of the lanes' x where has is set, in lane order, onto acc
// (the same value in every lane).  The sum is a chain; a term read with
// readlane (the lane's number is uniform) joins it in tens of cycles where a
// shuffle through LDS took more than a hundred.
__device__ inline double ordered_add(double acc, bool has, double x) {
    for (uint64_t mask = __ballot(has); mask != 0; mask &= mask - 1)
        acc = acc + lane_value(x, __builtin_ctzll(mask));
    return acc;
}

// One workgroup per row i, its columns and keep flags staged in LDS; each
// wave takes a dropped entry (i,j) at a time, its lanes over the entries of
// row j (coalesced), and finds m among the staged columns by a binary search
// in LDS; the wave adds the terms in lane order, which is ascending m.  Rows
// longer than the stage take the one-wave path.
__global__ void __launch_bounds__(kLB) lump_den_wide_kernel(int n, const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ ci,
                                                            const double* __restrict__ v,
                                                            const uint8_t* __restrict__ keep,
                                                            const double* __restrict__ thr,
                                                            double* __restrict__ den) {
    __shared__ int32_t sc[kWideCap];
    __shared__ uint8_t sk[kWideCap];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int ib = rp[i], ie = rp[i + 1], len = ie - ib;
        if (len > kWideCap) {
            if (wave == 0) lump_den_row(i, lane, rp, ci, v, keep, thr, den);
            continue;
        }
        __syncthreads();   // the previous row's readers are done
        for (int t = threadIdx.x; t < len; t += kLB) {
            sc[t] = ci[ib + t];
            sk[t] = keep[ib + t];
        }
        __syncthreads();
        for (int u = wave; u < len; u += kWaves) {
            const int j = sc[u];
            if (j == i || sk[u]) continue;
            const int jb = rp[j], je = rp[j + 1];
            const double t = thr[j];
            double d = 0.0;
            for (int r0 = jb; r0 < je; r0 += 64) {
                const int r = r0 + lane;
                bool has = false;
                double a = 0.0;
                if (r < je && t > 0.0) {
                    const int m = ci[r];
                    a = v[r];
                    if (m != j && -a >= t) {
                        const int w = lower_bound_lds(sc, len, m);
                        has = w < len && sc[w] == m && sk[w];
                    }
                }
                d = ordered_add(d, has, fabs(a));
            }
            if (lane == 0) den[ib + u] = d;
        }
    }
}

// Short rows: the same per dropped entry, but one wave per row (each wave
// its own slice of LDS, so four rows of a workgroup are in flight at once);
// a row's stage is written and read by its own wave only, and its dropped
// entries come from their list.
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ void __launch_bounds__(kLB) lump_den_wave_kernel(int n, const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ ci,
                                                            const double* __restrict__ v,
                                                            const uint8_t* __restrict__ keep,
                                                            const int32_t* __restrict__ hrp,
                                                            const int32_t* __restrict__ hci,
                                                            const int32_t* __restrict__ dropped,
                                                            const double* __restrict__ thr,
                                                            double* __restrict__ den) {
    __shared__ int32_t scw[kWaves][kWideCap];
    const int lane = threadIdx.x & 63;
    int32_t* sc = scw[threadIdx.x >> 6];   // the row's kept columns
    WAVE_ROW_LOOP(i, n) {
        const int ib = rp[i], ie = rp[i + 1], hb = hrp[i], he = hrp[i + 1], nk = he - hb;
        if (ie - ib == nk) continue;
        if (nk > kWideCap) {
            lump_den_row(i, lane, rp, ci, v, keep, thr, den);
            continue;
        }
        wave_lds_sync();   // the previous row's reads are done
        for (int t = lane; t < nk; t += 64) sc[t] = hci[hb + t];
        wave_lds_sync();
        for (int o = ib - hb; o < ie - he; ++o) {
            const int p = dropped[o];
            const int j = ci[p];
            if (j == i) continue;
            const int jb = rp[j], je = rp[j + 1];
            const double t = thr[j];
            double d = 0.0;
            for (int r0 = jb; r0 < je; r0 += 64) {
                const int r = r0 + lane;
                bool has = false;
                double a = 0.0;
                if (r < je && t > 0.0) {
                    const int m = ci[r];
                    a = v[r];
                    if (m != j && -a >= t) {
                        const int w = lower_bound_lds(sc, nk, m);
                        has = w < nk && sc[w] == m;
                    }
                }
                d = ordered_add(d, has, fabs(a));
            }
            if (lane == 0) den[p] = d;
        }
    }
}

// Position of column col in the ascending columns ci[w..e), walking w
// forward (a merge against an ascending sequence of col); -1 if absent.
__device__ inline int walk_to(const int32_t* ci, int& w, int e, int col) {
    while (w < e && ci[w] < col) ++w;
    return (w < e && ci[w] == col) ? w : -1;
}

// acc plus the shares the dropped entries (s,j) of row s give to node x, in
// ascending j: (|a_jx| / den) a_sj where (j,x) is strong.  The operator is
// bitwise symmetric, so a_jx is read as a_xj from row x, found by a merge
// walk of row s against row x: no row j is touched.  (s,x) is kept, so x
// belongs to every such W and den > 0.
__device__ inline double pull_row(const int32_t* rp, const int32_t* ci, const double* v, const uint8_t* keep,
                                  const double* thr, const double* den, int s, int x, double acc) {
    int w = rp[x];
    const int we = rp[x + 1];
    for (int q = rp[s]; q < rp[s + 1]; ++q) {
        const int j = ci[q];
        if (j == s || keep[q]) continue;
        const int r = walk_to(ci, w, we, j);
        if (r < 0) continue;
        const double t = thr[j], ajx = v[r];
        if (t > 0.0 && -ajx >= t) acc = acc + (fabs(ajx) / den[q]) * v[q];
    }
    return acc;
}

// Row k of the lumped operator, one wave.  Kept sets are symmetric, so the
// shares an entry (k,m) receives come from exactly two rows: dropped (k,j)
// sharing with m, and dropped (m,j) sharing with k, added in ascending order
// of the source entry (the lower row first).  (m,k) receives the same shares
// in the same order from the same start value, so one lane per (k,m) with
// m > k adds them serially and writes both entries.  The diagonal receives
// shares from every row it keeps (itself included); the lanes form one chunk
// of 64 entries of a source row at a time and the wave adds the chunk's
// shares in lane order.  Requires a bitwise symmetric operator (every
// Galerkin and non-Galerkin coarse operator is).
__device__ inline void strong_lump_row(int k, int lane, const int32_t* rp, const int32_t* ci, const double* v,
                                       const uint8_t* keep, const double* thr, const double* den,
                                       const int32_t* hrp, const int32_t* hci, double* hv) {
    const int hb = hrp[k], he = hrp[k + 1];
    for (int t = hb + lane; t < he; t += 64) {
        const int m = hci[t];
        if (m <= k) continue;
        double acc = pull_row(rp, ci, v, keep, thr, den, k, m, hv[t]);
        acc = pull_row(rp, ci, v, keep, thr, den, m, k, acc);
        hv[t] = acc;
        const int tm = find_in_row(hci, hrp[m], hrp[m + 1], k);
        if (tm >= 0) hv[tm] = acc;   // always found: the kept pattern is symmetric
    }
    const int dk = find_in_row(hci, hb, he, k);
    if (dk < 0) return;   // every operator stores its diagonal; never taken (uniform over the wave)
    const int kb = rp[k], ke = rp[k + 1];
    double acc = hv[dk];
    for (int p = hb; p < he; ++p) {
        const int s = hci[p];
        const int sb = rp[s], se = rp[s + 1];
        for (int q0 = sb; q0 < se; q0 += 64) {
            const int q = q0 + lane;
            bool has = false;
            double c = 0.0;
            if (q < se && !keep[q]) {
                const int j = ci[q];
                const double d = den[q];
                if (j != s && s == k) {
                    if (d == 0.0) {
                        c = v[q];   // no strong neighbour kept: the whole entry
                        has = true;
                    } else {
                        // the share to k itself, with a_jk = a_kj
                        const double t = thr[j], a = v[q];
                        if (t > 0.0 && -a >= t) {
                            c = (fabs(a) / d) * a;
                            has = true;
                        }
                    }
                } else if (j != s && d != 0.0) {
                    // the share of (s,j) to k, with a_jk read as a_kj from row k
                    const int r = find_in_row(ci, kb, ke, j);
                    if (r >= 0) {
                        const double t = thr[j], a = v[r];
                        if (t > 0.0 && -a >= t) {
                            c = -((fabs(a) / d) * v[q]);   // a - c == a + (-c) exactly
                            has = true;
                        }
                    }
                }
            }
            acc = ordered_add(acc, has, c);
        }
    }
    if (lane == 0) hv[dk] = acc;
}

__global__ void __launch_bounds__(kLB) strong_lump_kernel(int n, const int32_t* __restrict__ rp,
                                                          const int32_t* __restrict__ ci,
                                                          const double* __restrict__ v,
                                                          const uint8_t* __restrict__ keep,
                                                          const double* __restrict__ thr,
                                                          const double* __restrict__ den,
                                                          const int32_t* __restrict__ hrp,
                                                          const int32_t* __restrict__ hci,
                                                          double* __restrict__ hv) {
    const int lane = threadIdx.x & 63;
    WAVE_ROW_LOOP(k, n) { strong_lump_row(k, lane, rp, ci, v, keep, thr, den, hrp, hci, hv); }
}

// Row k of the lumped operator by the lists of dropped entries, one wave.  Few
// entries are dropped (gamma 0.1: 4 % on the finest sparsified level, a quarter
// on the next), and only they give shares, so the work follows them and not the
// rows: with D_i row i's list,
// * (k,m), m > k, a lane each: the shares of D_k, one j after the other for all
//   lanes, row j staged in LDS and searched for m; then those of D_m, each lane
//   along its own list, j searched in the staged row k.  A lane adds its shares
//   one by one, so nothing has to be brought into order; pairs without shares
//   are left as copied;
// * the diagonal: the lists of the kept rows end to end, 64 at a time, a lane an
//   entry; the wave adds the chunk's shares in lane order.
// Rows longer than the stage (or next to one) and of more than kListDrops
// dropped entries go to the workgroup form below (`heavy`).  3D Poisson 90^3, us, workgroup form ->
// this: 60,749 rows of 33 entries (4 % dropped) 604 -> 234, 9,351 of 55 (28 %)
// 192 -> 153.
// Where more than a third of a level's entries are dropped all its rows go there:
// a wave's work grows with its row's drops, the workgroup's hardly.  A level's
// sparsification in us, workgroup form and lists, by the share dropped: 59,438
// rows of 27, 27 % 609 and 524, 37 % 604 and 601, 56 % 612 and 747; 27,542 of 57,
// 27 % 721 and 567, 39 % 724 and 705, 49 % 714 and 823; 174,772 of 34, 39 % 2324
// and 2187, 50 % 2385 and 2595; 9,318 of 40, 20 % 194 and 166, 43 % 196 and 253.
constexpr int kListCap = 128;
constexpr int kListDrops = 32;       // 16: 2.77 ms a step with its solve, 8: 2.87, this 2.65
constexpr int kListMinRows = 8192;   // fewer rows leave the device to one wave's latency

// (the same answer in every workgroup of both kernels, from counts on the device)
__device__ __forceinline__ bool mostly_dropped(int n, const int32_t* __restrict__ rp, const int32_t* __restrict__ hrp) {
    return 3 * (int64_t)(rp[n] - hrp[n]) > (int64_t)rp[n];
}

__global__ void __launch_bounds__(kLB) strong_lump_list_kernel(int n, const int32_t* __restrict__ rp,
                                                               const int32_t* __restrict__ ci,
                                                               const double* __restrict__ v,
                                                               const int32_t* __restrict__ dropped,
                                                               const double* __restrict__ thr,
                                                               const double* __restrict__ den,
                                                               const int32_t* __restrict__ hrp,
                                                               const int32_t* __restrict__ hci, double* hv,
                                                               int32_t* __restrict__ heavy, int32_t* heavy_count) {
    __shared__ double jvw[kWaves][kListCap];
    __shared__ double kvw[kWaves][kListCap];
    __shared__ int32_t kcw[kWaves][kListCap];        // row k's columns (and values)
    __shared__ int32_t jcw[kWaves][kListCap];        // row j's columns (and values)
    __shared__ int32_t ksw[kWaves][kListCap];        // the kept columns s of row k
    __shared__ int32_t dsw[kWaves][kListCap];        // where their lists start
    __shared__ int32_t offw[kWaves][kListCap + 1];   // the lists' offsets, end to end
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double *jv = jvw[wave], *kv = kvw[wave];
    int32_t *kc = kcw[wave], *jc = jcw[wave], *ks = ksw[wave], *ds = dsw[wave], *off = offw[wave];
    if (mostly_dropped(n, rp, hrp)) return;
    WAVE_ROW_LOOP(k, n) {
        const int kb = rp[k], ke = rp[k + 1], len = ke - kb;
        const int hb = hrp[k], he = hrp[k + 1], nk = he - hb, nd = len - nk;
        // the row's dropped entries (k,j), a lane each: row j's place and length (0
        // where it has no strong neighbour), j's threshold, den, a_kj
        bool fits = len <= kListCap && nd <= kListDrops;
        int jb_l = 0, lj_l = 0;
        double th_l = 0.0, d_l = 0.0, a_l = 0.0;
        if (fits && nd > 0) {
            if (lane < nd) {
                const int p = dropped[kb - hb + lane];
                const int j = ci[p];
                jb_l = rp[j];
                lj_l = rp[j + 1] - jb_l;
                th_l = thr[j];
                d_l = den[p];
                a_l = v[p];
                if (j == k || !(th_l > 0.0)) lj_l = 0;
            }
            fits = __ballot(lj_l > kListCap) == 0;
        }
        if (!fits) {
            if (lane == 0) heavy[atomicAdd(heavy_count, 1)] = k;
            continue;
        }
        wave_lds_sync();   // the previous row's reads are done
        int total = 0;
        for (int base = 0; base < nk; base += 64) {
            const int idx = base + lane;
            int x = 0;
            if (idx < nk) {
                const int s = hci[hb + idx];
                const int s0 = rp[s], h0 = hrp[s];
                x = (rp[s + 1] - s0) - (hrp[s + 1] - h0);
                ks[idx] = s;
                ds[idx] = s0 - h0;
            }
            int incl = x;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            if (idx < nk) off[idx] = total + incl - x;
            total += __shfl(incl, 63);
        }
        if (total == 0) continue;   // nothing dropped here or beside
        if (lane == 0) off[nk] = total;
        for (int t = lane; t < len; t += 64) {
            kc[t] = ci[kb + t];
            kv[t] = v[kb + t];
        }
        wave_lds_sync();
        const int dpos = lower_bound_lds(ks, nk, k);
        if (dpos >= nk || ks[dpos] != k) continue;   // every operator stores its diagonal; never taken
        for (int t0 = dpos + 1; t0 < nk; t0 += 64) {
            const int t = t0 + lane;
            const bool have = t < nk;
            const int m = have ? ks[t] : -1;
            double acc = have ? hv[hb + t] : 0.0;
            bool changed = false;
            // (k,j) dropped, (j,m) strong; the next row j is requested before this one is searched
            int c0 = -1, c1 = -1;
            double w0 = 0.0, w1 = 0.0;
            auto request = [&](int o) {
                const int jb = __builtin_amdgcn_readlane(jb_l, o), lj = __builtin_amdgcn_readlane(lj_l, o);
                if (lane < lj) {
                    c0 = ci[jb + lane];
                    w0 = v[jb + lane];
                }
                if (lane + 64 < lj) {
                    c1 = ci[jb + 64 + lane];
                    w1 = v[jb + 64 + lane];
                }
            };
            if (nd > 0) request(0);
            for (int o = 0; o < nd; ++o) {
                const int lj = __builtin_amdgcn_readlane(lj_l, o);
                wave_lds_sync();   // the last row j's reads are done
                if (lane < lj) {
                    jc[lane] = c0;
                    jv[lane] = w0;
                }
                if (lane + 64 < lj) {
                    jc[lane + 64] = c1;
                    jv[lane + 64] = w1;
                }
                wave_lds_sync();
                if (o + 1 < nd) request(o + 1);
                const double th = lane_value(th_l, o);
                const int w = lower_bound_lds(jc, lj, m);
                if (have && w < lj && jc[w] == m && th > 0.0 && -jv[w] >= th) {
                    acc = acc + (fabs(jv[w]) / lane_value(d_l, o)) * lane_value(a_l, o);
                    changed = true;
                }
            }
            // (m,j) dropped, (j,k) strong: a_jk read as a_kj
            const int ob = have ? ds[t] : 0, cnt = have ? off[t + 1] - off[t] : 0;
            for (int e0 = 0; e0 < cnt; e0 += 4) {
                // four entries' loads in flight (the list's last one stands for those past it)
                int j[4];
                double d[4], a[4], th[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int p = dropped[ob + min(e0 + u, cnt - 1)];
                    j[u] = ci[p];
                    d[u] = den[p];
                    a[u] = v[p];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) th[u] = thr[j[u]];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (e0 + u >= cnt || j[u] == m) continue;
                    const int w = lower_bound_lds(kc, len, j[u]);
                    if (w >= len || kc[w] != j[u]) continue;
                    const double akj = kv[w];
                    if (th[u] > 0.0 && -akj >= th[u]) {
                        acc = acc + (fabs(akj) / d[u]) * a[u];
                        changed = true;
                    }
                }
            }
            if (changed) {
                hv[hb + t] = acc;
                const int tm = find_in_row(hci, hrp[m], hrp[m + 1], k);
                if (tm >= 0) hv[tm] = acc;   // always found: the kept pattern is symmetric
            }
        }
        // the diagonal
        double acc = hv[hb + dpos];
        for (int f0 = 0; f0 < total; f0 += 64) {
            const int f = f0 + lane;
            bool has = false;
            double c = 0.0;
            if (f < total) {
                int lo = 0, hi = nk;   // off[lo] <= f < off[lo + 1]
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (off[mid] <= f) lo = mid;
                    else hi = mid;
                }
                const int s = ks[lo], p = dropped[ds[lo] + f - off[lo]];
                const int j = ci[p];
                const double d = den[p], a = v[p];
                if (j != s && s == k) {
                    const double th = thr[j];
                    if (d == 0.0) {
                        c = a;   // no strong neighbour kept: the whole entry
                        has = true;
                    } else if (th > 0.0 && -a >= th) {
                        c = (fabs(a) / d) * a;   // the share to k itself, a_jk = a_kj
                        has = true;
                    }
                } else if (j != s && d != 0.0) {
                    const int r = lower_bound_lds(kc, len, j);
                    if (r < len && kc[r] == j) {
                        const double th = thr[j], akj = kv[r];
                        if (th > 0.0 && -akj >= th) {
                            c = -((fabs(akj) / d) * a);   // a - c == a + (-c) exactly
                            has = true;
                        }
                    }
                }
            }
            acc = ordered_add(acc, has, c);
        }
        if (lane == 0) hv[hb + dpos] = acc;
    }
}

// One workgroup per row k (the listed ones, or all), row k of A (columns, values, keep flags,
// denominators, and the thresholds of its columns) staged in LDS.
// * (k,m), m > k, one wave each, its lanes over row m (coalesced): a lane
//   finds its column j in the staged row k by a binary search in LDS and
//   forms the share of dropped (k,j) (with a_jm read as a_mj); the wave adds
//   them in lane order, then, in a second pass, the shares of dropped (m,j)
//   (a_jk read as a_kj).  Every share needs j in row k, so its threshold is
//   a staged one.  Same terms, same order as the one-wave path.
// * the diagonal: the kept rows s of row k are laid end to end (offsets by a
//   scan), the workgroup computes kDiagPer x 256 consecutive entries' shares
//   at a time into LDS (a_kj by a binary search of the staged row k) and the
//   first wave adds them in order.
// Rows longer than the stage take the one-wave path.
constexpr int kDiagPer = 2;

// LB threads a workgroup: LB, or 1024 on levels too small to fill the
// device otherwise; eight waves a SIMD (at most 64 registers, no spills)
template <int LB>
__global__ void __launch_bounds__(LB) __attribute__((amdgpu_waves_per_eu(8, 8))) strong_lump_wide_kernel(int n, const int32_t* __restrict__ rp,
                                                               const int32_t* __restrict__ ci,
                                                               const double* __restrict__ v,
                                                               const uint8_t* __restrict__ keep,
                                                               const double* __restrict__ thr,
                                                               const double* __restrict__ den,
                                                               const int32_t* __restrict__ hrp,
                                                               const int32_t* __restrict__ hci,
                                                               double* __restrict__ hv,
                                                               const int32_t* heavy,
                                                               const int32_t* __restrict__ heavy_count) {
    __shared__ int32_t kc[kWideCap];
    __shared__ double kv[kWideCap];
    __shared__ double kd[kWideCap];
    __shared__ double kt[kWideCap];         // thr of the columns of row k
    __shared__ uint8_t kk[kWideCap];
    __shared__ int32_t ks[kWideCap];        // the kept columns s of row k
    __shared__ int32_t sb[kWideCap];        // rp[s]
    __shared__ int32_t off[kWideCap + 1];   // their rows' offsets, end to end
    __shared__ double slot_c[kDiagPer * LB];
    __shared__ uint8_t slot_h[kDiagPer * LB];
    __shared__ int wsum[(LB / 64)];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (heavy && mostly_dropped(n, rp, hrp)) heavy = nullptr;
    const int todo = heavy ? *heavy_count : n;   // listed rows, or all
    for (int it = blockIdx.x; it < todo; it += gridDim.x) {
        const int k = heavy ? heavy[it] : it;
        const int kb = rp[k], ke = rp[k + 1], len = ke - kb;
        if (len > kWideCap) {
            if (wave == 0) strong_lump_row(k, lane, rp, ci, v, keep, thr, den, hrp, hci, hv);
            continue;
        }
        const int hb = hrp[k], he = hrp[k + 1], nk = he - hb;   // nk <= len
        __syncthreads();   // the previous row's readers are done
        for (int t = threadIdx.x; t < len; t += LB) {
            const int p = kb + t;
            const int j = ci[p];
            kc[t] = j;
            kv[t] = v[p];
            kk[t] = keep[p];
            kd[t] = keep[p] ? 0.0 : den[p];   // den is written for dropped entries only
            kt[t] = thr[j];
        }
        // kept columns and their row lengths, scanned end to end
        int carry = 0;
        for (int base = 0; base < nk; base += LB) {
            const int idx = base + (int)threadIdx.x;
            int x = 0;
            if (idx < nk) {
                const int s = hci[hb + idx];
                const int s0 = rp[s];
                ks[idx] = s;
                sb[idx] = s0;
                x = rp[s + 1] - s0;
            }
            int incl = x;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            int before = 0, total = 0;
            for (int w = 0; w < (LB / 64); ++w) {
                before += w < wave ? wsum[w] : 0;
                total += wsum[w];
            }
            if (idx < nk) off[idx] = carry + before + incl - x;
            carry += total;
            __syncthreads();   // wsum is reused
        }
        if (threadIdx.x == 0) off[nk] = carry;
        __syncthreads();
        const int dpos = lower_bound_lds(ks, nk, k);
        if (dpos >= nk || ks[dpos] != k) continue;   // every operator stores its diagonal; never taken
        const int dk = hb + dpos;
        // off-diagonals (k,m), m > k: a wave per target, its lanes over row m;
        // the terms of dropped (k,j) first, then those of dropped (m,j), each
        // in ascending j (lane order)
        // a target's loads: its start value, the bounds of row m's kept
        // columns, and the first 64 entries of row m (a kept entry's den is
        // never written and is not used)
        struct Target {
            int m, mb, me, hm0, hm1, j0;
            double acc, a0, d0;
            uint8_t kp0;
        };
        auto fetch = [&](int tt) {
            Target g;
            g.m = ks[tt - hb];
            g.mb = sb[tt - hb];
            g.me = g.mb + off[tt - hb + 1] - off[tt - hb];
            g.hm0 = hrp[g.m];
            g.hm1 = hrp[g.m + 1];
            g.acc = hv[tt];
            const int r0 = min(g.mb + lane, g.me - 1);
            g.j0 = ci[r0];
            g.a0 = v[r0];
            g.d0 = den[r0];
            g.kp0 = keep[r0];
            return g;
        };
        Target nxt{};
        if (dk + 1 + wave < he) nxt = fetch(dk + 1 + wave);
        for (int t = dk + 1 + wave; t < he; t += (LB / 64)) {
            const Target cur = nxt;
            // the first chunk of the mirror row, then the next target's
            // loads: both in flight while this target's shares are formed
            const int hidx = cur.hm0 + lane;
            const int hc0 = hidx < cur.hm1 ? hci[hidx] : -1;
            if (t + (LB / 64) < he) nxt = fetch(t + (LB / 64));
            const int m = cur.m, mb = cur.mb, me = cur.me, hm0 = cur.hm0, hm1 = cur.hm1, j0 = cur.j0;
            const double a0 = cur.a0, d0 = cur.d0;
            const uint8_t kp0 = cur.kp0;
            double acc = cur.acc;
            const int w0 = lower_bound_lds(kc, len, j0);
            const bool at0 = w0 < len && kc[w0] == j0;   // j0 in row k
            for (int c0 = mb; c0 < me; c0 += 64) {   // (k,j) dropped, (j,m) strong: a_jm read as a_mj
                int j = j0, w = w0;
                double ajm = a0;
                bool at = at0;
                if (c0 != mb) {
                    const int r = min(c0 + lane, me - 1);
                    j = ci[r];
                    ajm = v[r];
                    w = lower_bound_lds(kc, len, j);
                    at = w < len && kc[w] == j;
                }
                bool has = false;
                double c = 0.0;
                if (c0 + lane < me && at && j != k && !kk[w]) {
                    const double th = kt[w];
                    if (th > 0.0 && -ajm >= th) {
                        c = (fabs(ajm) / kd[w]) * kv[w];
                        has = true;
                    }
                }
                acc = ordered_add(acc, has, c);
            }
            for (int c0 = mb; c0 < me; c0 += 64) {   // (m,j) dropped, (j,k) strong: a_jk read as a_kj
                int j = j0, w = w0;
                double a = a0, d = d0;
                bool at = at0, kp = kp0 != 0;
                if (c0 != mb) {
                    const int q = min(c0 + lane, me - 1);
                    j = ci[q];
                    a = v[q];
                    d = den[q];
                    kp = keep[q] != 0;
                    w = lower_bound_lds(kc, len, j);
                    at = w < len && kc[w] == j;
                }
                bool has = false;
                double c = 0.0;
                if (c0 + lane < me && j != m && !kp && at) {
                    const double th = kt[w], akj = kv[w];
                    if (th > 0.0 && -akj >= th) {
                        c = (fabs(akj) / d) * a;
                        has = true;
                    }
                }
                acc = ordered_add(acc, has, c);
            }
            // (m,k): the same value; its position by a coalesced search of row m
            int tm = -1;
            for (int c0 = hm0; c0 < hm1 && tm < 0; c0 += 64) {
                const int idx = c0 + lane;
                const int col = c0 == hm0 ? hc0 : (idx < hm1 ? hci[idx] : -1);
                const uint64_t hit = __ballot(idx < hm1 && col == k);
                if (hit) tm = c0 + __builtin_ctzll(hit);
            }
            if (lane == 0) {
                hv[t] = acc;
                if (tm >= 0) hv[tm] = acc;   // always found: the kept pattern is symmetric
            }
        }
        // the diagonal
        double acc = hv[dk];
        const int total = off[nk];
        for (int g = 0; g < total; g += kDiagPer * LB) {
            int qq[kDiagPer], ss[kDiagPer];
#pragma unroll
            for (int e = 0; e < kDiagPer; ++e) {
                const int f = g + e * LB + (int)threadIdx.x;
                qq[e] = -1;
                ss[e] = 0;
                if (f < total) {
                    int lo = 0, hi = nk;   // off[lo] <= f < off[lo + 1]
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (off[mid] <= f) lo = mid;
                        else hi = mid;
                    }
                    ss[e] = ks[lo];
                    qq[e] = sb[lo] + (f - off[lo]);
                }
            }
            int jj[kDiagPer];
            uint8_t kp[kDiagPer];
            double dd[kDiagPer], aa[kDiagPer];
#pragma unroll
            for (int e = 0; e < kDiagPer; ++e) {
                const int q = qq[e] < 0 ? kb : qq[e];   // a valid entry; unused when qq < 0
                jj[e] = ci[q];
                kp[e] = keep[q];
                dd[e] = den[q];
                aa[e] = v[q];
            }
#pragma unroll
            for (int e = 0; e < kDiagPer; ++e) {
                bool has = false;
                double c = 0.0;
                if (qq[e] >= 0 && !kp[e]) {
                    const int s = ss[e], j = jj[e];
                    const double d = dd[e];
                    if (j != s && s == k) {
                        if (d == 0.0) {
                            c = aa[e];   // no strong neighbour kept: the whole entry
                            has = true;
                        } else {
                            const double t = kt[qq[e] - kb], a = aa[e];   // the share to k itself, a_jk = a_kj
                            if (t > 0.0 && -a >= t) {
                                c = (fabs(a) / d) * a;
                                has = true;
                            }
                        }
                    } else if (j != s && d != 0.0) {
                        const int r = lower_bound_lds(kc, len, j);
                        if (r < len && kc[r] == j) {
                            const double t = kt[r], a = kv[r];
                            if (t > 0.0 && -a >= t) {
                                c = -((fabs(a) / d) * aa[e]);   // a - c == a + (-c) exactly
                                has = true;
                            }
                        }
                    }
                }
                slot_c[e * LB + threadIdx.x] = c;
                slot_h[e * LB + threadIdx.x] = has ? 1 : 0;
            }
            __syncthreads();
            if (wave == 0)
                for (int w = 0; w < kDiagPer * (LB / 64); ++w)
                    acc = ordered_add(acc, slot_h[w * 64 + lane] != 0, slot_c[w * 64 + lane]);
            __syncthreads();   // the slots are reused
        }
        if (threadIdx.x == 0) hv[dk] = acc;
    }
}

}  // namespace

void launch_compact_copy(int n, const int32_t* rp, const int32_t* ci, const double* v, const uint8_t* keep,
                         const int32_t* new_rp, int32_t* new_ci, double* new_v, const LumpLists& lists,
                         hipStream_t st) {
    hipLaunchKernelGGL(compact_copy_kernel, dim3(wave_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v, keep, new_rp,
                       new_ci, new_v, lists.dropped, lists.heavy + n);
}

void launch_lump_threshold(int n, const int32_t* rp, const int32_t* ci, const double* v, double theta,
                           double* thr, hipStream_t st) {
    hipLaunchKernelGGL(lump_threshold_kernel, dim3(wave_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v, theta, thr);
}

namespace {

bool use_wide(const LumpShapes& ls, double mean_row) { return mean_row >= ls.wide_mean_row; }

bool use_den_wave(const LumpShapes& ls, int n, double mean_row) {
    if (ls.den_wave_mean_row >= 0.0) return mean_row < ls.den_wave_mean_row;
    return n >= kDenWaveMinRows && mean_row < kDenWaveMeanRow;
}

int row_grid_of(int n) { return std::max(1, std::min(n, 65536)); }

}  // namespace

void launch_lump_den(int n, const int32_t* rp, const int32_t* ci, const double* v, const uint8_t* keep,
                     const int32_t* hrp, const int32_t* hci, const LumpLists& lists, const double* thr, double* den,
                     double mean_row, const LumpShapes& ls, hipStream_t st) {
    if (use_wide(ls, mean_row) && use_den_wave(ls, n, mean_row))
        hipLaunchKernelGGL(lump_den_wave_kernel, dim3(wave_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v, keep, hrp, hci,
                           lists.dropped, thr, den);
    else if (use_wide(ls, mean_row))
        hipLaunchKernelGGL(lump_den_wide_kernel, dim3(row_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v, keep, thr,
                           den);
    else
        hipLaunchKernelGGL(lump_den_kernel, dim3(wave_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v, keep, thr, den);
}

void launch_strong_lump(int n, const int32_t* rp, const int32_t* ci, const double* v, const uint8_t* keep,
                        const LumpLists& lists, const double* thr, const double* den, const int32_t* hrp,
                        const int32_t* hci, double* hv, double mean_row, const LumpShapes& ls, hipStream_t st) {
    if (!use_wide(ls, mean_row)) {
        hipLaunchKernelGGL(strong_lump_kernel, dim3(wave_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v, keep, thr, den,
                           hrp, hci, hv);
        return;
    }
    int32_t *heavy = nullptr, *count = nullptr;
    if (n >= kListMinRows) {
        heavy = lists.heavy;
        count = lists.heavy + n;
        hipLaunchKernelGGL(strong_lump_list_kernel, dim3(wave_grid_of(n)), dim3(kLB), 0, st, n, rp, ci, v,
                           lists.dropped, thr, den, hrp, hci, hv, heavy, count);
    }
    // a workgroup a row also where few rows may be listed: 4,096 looping took
    // 2569 instead of 2373 us where all rows come here (174,772), and save 10
    // where none does
    const dim3 grid(row_grid_of(n));
    if (n < ls.small_rows)
        hipLaunchKernelGGL(strong_lump_wide_kernel<1024>, grid, dim3(1024), 0, st, n, rp, ci, v, keep, thr, den, hrp,
                           hci, hv, heavy, count);
    else
        hipLaunchKernelGGL(strong_lump_wide_kernel<kLB>, grid, dim3(kLB), 0, st, n, rp, ci, v, keep, thr, den, hrp,
                           hci, hv, heavy, count);
}

}  // namespace amg355
