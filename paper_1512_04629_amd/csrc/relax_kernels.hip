// Hybrid Gauss-Seidel sweep: the rows of a block in order, each row's sum in
// ascending column order (the order and operations of the definition, so the
// result is the CPU's bit for bit).  Three forms: one thread per block, reading
// global memory (blocks of more than 1,024 rows); one lane per block on terms
// staged in LDS (small blocks on large levels); 16 or 64 lanes per chunk of
// blocks, the terms staged by other waves (everything else).
#include "relax_kernels.hpp"

#include <algorithm>

#pragma clang fp contract(off)

namespace amg355 {

namespace {

template <bool FORWARD>
__device__ inline void gs_block_rows(int r0, int r1, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                     const double* __restrict__ v, const double* __restrict__ b,
                                     const double* __restrict__ xold, double* xnew);

template <bool FORWARD>
__global__ __launch_bounds__(256) void hybrid_gs_kernel(int n, const int32_t* __restrict__ rp,
                                                        const int32_t* __restrict__ ci,
                                                        const double* __restrict__ v,
                                                        const double* __restrict__ b,
                                                        const double* __restrict__ xold, double* xnew,
                                                        int block) {
    const int64_t nblk = ((int64_t)n + block - 1) / block;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nblk;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int r0 = (int)(t * block);
        const int r1 = (int)std::min<int64_t>((int64_t)r0 + block, n);
        gs_block_rows<FORWARD>(r0, r1, rp, ci, v, b, xold, xnew);
    }
}

// Staged form, for blocks of fewer than kGsChainMin rows.  A workgroup owns a chunk
// of R consecutive rows (whole blocks).  First all its threads turn the
// chunk's entries into terms in LDS with coalesced loads: the product
// a_ij xold_j for a term with an old value (rounded exactly as the sweep
// rounds it), a_ij and the chunk-local row of j for a term with a new value,
// the diagonal marked.  Then one lane per block runs the block's rows in
// order from LDS, subtracting the terms in ascending column order: the same
// operations in the same order as hybrid_gs_kernel.  A chunk whose entries do
// not fit takes the per-block loop of hybrid_gs_kernel.
constexpr int kGsThreads = 256;
constexpr int kGsCap = 3072;      // staged terms per chunk
constexpr int kGsMaxRows = 256;   // rows per chunk
constexpr int16_t kGsDiag = -2, kGsOld = -1;

template <bool FORWARD>
__device__ inline void gs_block_rows(int r0, int r1, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                     const double* __restrict__ v, const double* __restrict__ b,
                                     const double* __restrict__ xold, double* xnew) {
    int last = -1;
    double last_x = 0.0;
    for (int k = 0; k < r1 - r0; ++k) {
        const int i = FORWARD ? r0 + k : r1 - 1 - k;
        double s = b[i], d = 0.0;
        for (int p = rp[i]; p < rp[i + 1]; ++p) {
            const int j = ci[p];
            if (j == i) {
                d = v[p];
                continue;
            }
            const bool visited = j >= r0 && j < r1 && (FORWARD ? j < i : j > i);
            const double y = visited ? (j == last ? last_x : xnew[j]) : xold[j];
            s = s - v[p] * y;
        }
        const double xi = s / d;
        xnew[i] = xi;
        last = i;
        last_x = xi;
    }
}

template <bool FORWARD>
__global__ __launch_bounds__(kGsThreads) void hybrid_gs_staged_kernel(int n, const int32_t* __restrict__ rp,
                                                                      const int32_t* __restrict__ ci,
                                                                      const double* __restrict__ v,
                                                                      const double* __restrict__ b,
                                                                      const double* __restrict__ xold,
                                                                      double* xnew, int block, int R) {
    __shared__ double term[kGsCap];
    __shared__ int16_t tag[kGsCap];
    __shared__ uint8_t rowid[kGsCap];   // chunk-local row of each staged entry
    __shared__ int32_t lrp[kGsMaxRows + 1];
    __shared__ double lb[kGsMaxRows], ly[kGsMaxRows];
    const int nchunk = (n + R - 1) / R;
    for (int c = blockIdx.x; c < nchunk; c += gridDim.x) {
        const int r0 = c * R, r1 = min(r0 + R, n), nr = r1 - r0;
        const int p0 = rp[r0], p1 = rp[r1];
        const int nb = (nr + block - 1) / block;
        if (p1 - p0 > kGsCap) {   // uniform over the workgroup
            for (int k = threadIdx.x; k < nb; k += blockDim.x)
                gs_block_rows<FORWARD>(r0 + k * block, min(r0 + (k + 1) * block, r1), rp, ci, v, b, xold, xnew);
            continue;
        }
        for (int t = threadIdx.x; t <= nr; t += blockDim.x) lrp[t] = rp[r0 + t] - p0;
        for (int t = threadIdx.x; t < nr; t += blockDim.x) lb[t] = b[r0 + t];
        __syncthreads();
        for (int t = threadIdx.x; t < nr; t += blockDim.x)
            for (int q = lrp[t]; q < lrp[t + 1]; ++q) rowid[q] = (uint8_t)t;
        __syncthreads();
        for (int q = threadIdx.x; q < p1 - p0; q += blockDim.x) {
            const int lo = rowid[q];
            const int i = r0 + lo;
            const int j = ci[p0 + q];
            const double a = v[p0 + q];
            if (j == i) {
                tag[q] = kGsDiag;
                term[q] = a;
                continue;
            }
            const int bs = r0 + (lo / block) * block;
            const int be = min(bs + block, r1);
            if (j >= bs && j < be && (FORWARD ? j < i : j > i)) {
                tag[q] = (int16_t)(j - r0);
                term[q] = a;
            } else {
                tag[q] = kGsOld;
                term[q] = a * xold[j];
            }
        }
        __syncthreads();
        // the chains are serial: let their wave issue ahead of the other
        // workgroups' staging waves on the same SIMD
        const bool chain_wave = (int)(threadIdx.x & ~63) < nb;
        if (chain_wave) __builtin_amdgcn_s_setprio(3);
        for (int k = threadIdx.x; k < nb; k += blockDim.x) {
            const int b0 = k * block, b1 = min(b0 + block, nr);
            int prev = -1;          // the row visited last: its value stays in a register
            double prev_x = 0.0;
            for (int s = 0; s < b1 - b0; ++s) {
                const int il = FORWARD ? b0 + s : b1 - 1 - s;
                double acc = lb[il], d = 0.0;
                for (int q0 = lrp[il], qe = lrp[il + 1]; q0 < qe; q0 += 8) {
                    // a group of up to 8 terms: the staged values first, then
                    // the new values they need, then the subtractions in order
                    double tv[8], yv[8];
                    int tg[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const bool ok = q0 + u < qe;
                        tg[u] = ok ? tag[q0 + u] : kGsOld;
                        tv[u] = ok ? term[q0 + u] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int f = tg[u];
                        yv[u] = f >= 0 ? (f == prev ? prev_x : ly[f]) : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (q0 + u >= qe) break;
                        const int f = tg[u];
                        if (f == kGsDiag) {
                            d = tv[u];
                            continue;
                        }
                        acc = acc - (f >= 0 ? tv[u] * yv[u] : tv[u]);
                    }
                }
                const double xi = acc / d;
                ly[il] = xi;
                xnew[r0 + il] = xi;
                prev = il;
                prev_x = xi;
            }
        }
        if (chain_wave) __builtin_amdgcn_s_setprio(0);
        __syncthreads();
    }
}

// Chain form, for blocks of up to kGsChainMaxRows rows.  The rows of a block
// are a serial chain, so what a sweep costs is the time of one row in its
// chain times the rows, and the instructions that time takes where the chains
// fill the machine.  A chunk of consecutive rows (whole blocks) belongs to W
// lanes of a workgroup's first wave: W = 64, one chunk to a workgroup (long
// rows, few chunks), or W = 16, four chunks side by side in the wave.  The
// other waves turn the next strip of every chunk (up to W rows and S entries)
// into terms in LDS, while the first runs the current one: the product
// a_ij xold_j where the old value is used, a_ij and the row's place in the
// chunk where the new one is, 0 for the diagonal, whose subtraction changes
// nothing; and subtract, lane by row, the terms that come before a row's first
// new value.  In the chain a row's other terms lie one to a lane, loaded two rows
// ahead, the new values they need one row ahead (the value of the row before
// from a register), and are subtracted in ascending column order by one
// multiply-add each, acc = (-1) t + acc, the term taken from its lane by the
// instruction's own row broadcast: exactly the subtraction, so the operations
// are those of the definition in its order and the bits those of the per-block
// kernel.  A row longer than a strip is summed from memory.
constexpr int kGsChainMaxRows = 1024;   // rows per chunk

// acc - t(lane 0) - t(lane 1) ... of each row of 16 lanes, 8 or 16 lanes in
// order (v_fmac_f64 with src1 = -1; a DPP source needs two wait states after
// the instruction that wrote it)
__device__ __forceinline__ double sub_row8(double acc, double t, double m1) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:7 row_mask:0xf bank_mask:0xf"
        : "+v"(acc) : "v"(t), "v"(m1));
    return acc;
}

__device__ __forceinline__ double sub_row8_high(double acc, double t, double m1) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:15 row_mask:0xf bank_mask:0xf"
        : "+v"(acc) : "v"(t), "v"(m1));
    return acc;
}

__device__ __forceinline__ double lane_read(double x, int lane) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// acc minus the first len (<= W) terms of the W lanes in order; lanes past len
// hold 0.  W = 64: acc is handed from each row of 16 lanes to the next and
// comes back in every lane.
template <int W>
__device__ __forceinline__ double sub_terms(double acc, double t, int len, double m1) {
    if constexpr (W == 16) {
        acc = sub_row8(acc, t, m1);
        if (__any(len > 8)) acc = sub_row8_high(acc, t, m1);
    } else {
        for (int r = 0; r < 4; ++r) {
            if (len <= 16 * r) break;
            acc = sub_row8(acc, t, m1);
            if (len > 16 * r + 8) acc = sub_row8_high(acc, t, m1);
            acc = lane_read(acc, 16 * r);
        }
    }
    return acc;
}

// a / d from the correctly rounded reciprocal y = 1 / d, correctly rounded
// (Markstein, IBM J. Res. Dev. 34, 1990: the correction of a quotient within
// one unit in the last place by an exact remainder is the rounded quotient;
// the first correction brings it there); far from the ends of the exponent
// range the remainders are exact, elsewhere (and for 0, infinities and NaN) the
// division itself.  y = 0 says that d is not in the range.
__device__ __forceinline__ bool mid_range(double a) {   // exponents -400 to 399, from the bits
    return (unsigned)((__double2hiint(a) & 0x7fffffff) - (623 << 20)) < (800u << 20);
}
__device__ __forceinline__ double quotient(double a, double d, double y) {
    if (mid_range(a) && __double2hiint(y) != 0) {
        double q = a * y;
        q = __builtin_fma(__builtin_fma(-d, q, a), y, q);
        return __builtin_fma(__builtin_fma(-d, q, a), y, q);
    }
    return a / d;
}

struct __align__(16) GsRow {      // a staged row
    double b, d, y;               // right-hand side, diagonal, its reciprocal (0: divide)
    int32_t off, len;             // its terms in the strip; len < 0: too long, not staged
};

template <bool FORWARD, int W, int NP, bool AHEAD>
__global__ __launch_bounds__(64 * (1 + NP)) void hybrid_gs_chain_kernel(
    int n, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, const double* __restrict__ v,
    const double* __restrict__ b, const double* __restrict__ xold, double* __restrict__ xnew, int block, int chunk) {
    constexpr int G = 64 / W;               // chunks of the workgroup
    constexpr int E = 8;                    // entries of a strip per staging lane
    constexpr int S = W * E * NP;           // entries per strip
    // one more of each: what a lane without an entry, or a step without a row, reads
    __shared__ double term[2][G][S + 1];
    __shared__ int16_t tag[2][G][S + 1];
    __shared__ GsRow rows[2][G][W + 1];
    __shared__ int32_t rows_in[2][G];
    __shared__ int32_t soff[NP][G][W];
    extern __shared__ double ly_all[];      // new values of the chunks' rows
    const int g = ((int)threadIdx.x & 63) / W, lane = (int)threadIdx.x & (W - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t start = ((int64_t)blockIdx.x * G + g) * chunk;
    const int r0 = (int)min(start, (int64_t)n), nr = (int)min((int64_t)chunk, (int64_t)n - r0);
    double* const ly = ly_all + (size_t)g * (chunk + 1);   // ly[chunk]: not a row
    if (threadIdx.x < 2 * G) {
        const int u = (int)threadIdx.x / G, w = (int)threadIdx.x % G;
        term[u][w][S] = 0.0;
        tag[u][w][S] = kGsOld;
        rows[u][w][W] = GsRow{0.0, 1.0, 1.0, 0, 0};
    }
    // strip entries of a staging wave: alternate rows of W, or its share end to end
    auto place = [&](int e, int part) { return lane + W * (AHEAD ? e + part * E : e * NP + part); };
    // row visited k-th of the chunk, relative to r0
    auto row_at = [&](int k) { return FORWARD ? k : nr - 1 - k; };
    // x of the group's lane l
    auto from = [&](int x, int l) {
        if constexpr (W == 64) return __builtin_amdgcn_readlane(x, l);
        else return __shfl(x, l, W);
    };
    int done = 0;                           // rows staged (or left to the long-row path) so far
    auto produce = [&](int buf) {
        const int part = wave - 1;
        const int left = nr - done;
        const bool have = lane < left;
        const int il = have ? row_at(done + lane) : 0;
        const int beg = have ? rp[r0 + il] : 0, end = have ? rp[r0 + il + 1] : 0;
        const double bi = have ? b[r0 + il] : 0.0;
        // entries of the strip up to and with this lane's row
        const int first = from(FORWARD ? beg : end, 0);
        const int upto = FORWARD ? end - first : first - beg;
        unsigned long long fit = __ballot(have && upto <= S);
        if constexpr (W < 64) fit = (fit >> (g * W)) & ((1ull << W) - 1ull);
        const int R = __popcll(fit);
        const bool lng = R == 0 && left > 0;
        const int lastl = max(R - 1, 0);
        const int p0 = FORWARD ? first : from(beg, lastl);
        const int total = R > 0 ? from(upto, lastl) : 0;
        const int ibs = il - il % block;     // the row's block in the chunk
        soff[part][g][lane] = lane < R ? beg - p0 : INT32_MAX;
        if (part == 0) {
            if (lane >= R) rows[buf][g][lane] = GsRow{0.0, 1.0, 1.0, 0, R == 0 && lane == 0 ? -1 : 0};
            if (lane == 0) rows_in[buf][g] = lng ? 1 : R;
            if (!AHEAD && lane < R) {
                GsRow& q = rows[buf][g][lane];
                q.b = bi;
                q.off = beg - p0;
                q.len = end - beg;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        int jj[E], kk[E];
        double aa[E], xx[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int q = place(e, part);
            jj[e] = q < total ? ci[p0 + q] : min(r0, n - 1);
            aa[e] = q < total ? v[p0 + q] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) xx[e] = xold[jj[e]];
        // the strip row (in memory order) holding each entry
#pragma unroll
        for (int e = 0; e < E; ++e) kk[e] = 0;
#pragma unroll
        for (int step = W / 2; step > 0; step >>= 1) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int m = kk[e] + step;
                const int st = m < R ? soff[part][g][FORWARD ? m : R - 1 - m] : INT32_MAX;
                if (st <= place(e, part)) kk[e] = m;
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = FORWARD ? kk[e] : max(R - 1 - kk[e], 0);
            const int bs = __shfl(ibs, k, W);
            const int q = place(e, part);
            if (q < total) {
                const int i = row_at(done + k), j = jj[e] - r0;
                if (j == i) {
                    rows[buf][g][k].d = aa[e];
                    // With many chunks of 64 lanes the registers bound the chains in
                    // flight: divided without a branch (82 registers, 104 with;
                    // 101 and 114 us on 2,731 chunks).  Elsewhere the branch, which
                    // shortens the staging (64^3, blocks of 64, a solve: 5.82 and
                    // 5.94 ms).
                    if constexpr (W == 64 && !AHEAD) {
                        const double y = 1.0 / aa[e];
                        rows[buf][g][k].y = mid_range(aa[e]) ? y : 0.0;
                    } else {
                        rows[buf][g][k].y = mid_range(aa[e]) ? 1.0 / aa[e] : 0.0;
                    }
                    tag[buf][g][q] = kGsDiag;
                    term[buf][g][q] = 0.0;
                } else {
                    const int be = min(bs + block, nr);
                    const bool fresh = j >= bs && j < be && (FORWARD ? j < i : j > i);
                    tag[buf][g][q] = fresh ? (int16_t)j : kGsOld;
                    term[buf][g][q] = fresh ? aa[e] : aa[e] * xx[e];
                }
            }
        }
        // AHEAD: a row's terms before the first that waits for a new value are
        // subtracted here (a lane a row, in order): the chain starts at that one.
        // A row whose entries two waves staged keeps them all.
        if (AHEAD && lane < R) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int off = beg - p0, len = end - beg;
            // (the wave that staged its first entry keeps the row)
            const bool mine = off + len <= (part + 1) * (W * E);
            if (part == min(off / (W * E), NP - 1)) {
                double acc = bi;
                int o = off;
                const int stop = off + len;
                bool open = mine;
                while (open && o < stop) {
                    double t[4];
                    int a[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int at = min(o + u, stop - 1);
                        t[u] = term[buf][g][at];
                        a[u] = o + u < stop ? (int)tag[buf][g][at] : 0;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        open = open && a[u] < 0;
                        if (open) {
                            acc = acc - t[u];
                            ++o;
                        }
                    }
                }
                GsRow& q = rows[buf][g][lane];
                q.b = acc;
                q.off = o;
                q.len = stop - o;
            }
        }
        done += lng ? 1 : R;
    };
    double m1 = -1.0;
    asm("" : "+v"(m1));
    int at = 0;                             // rows finished
    // a row too long for a strip: its terms from memory (all of a group's
    // lanes or none are here)
    auto long_row = [&]() {
        const int il = row_at(at), i = r0 + il;
        const int bs = il - il % block, be = min(bs + block, nr);
        const int beg = rp[i], end = rp[i + 1];
        double acc = b[i], d = 0.0;
        for (int p = beg; p < end; p += W) {
            const bool in = p + lane < end;
            const int j = in ? ci[p + lane] - r0 : il;
            const double a = in ? v[p + lane] : 0.0;
            const bool fresh = j >= bs && j < be && (FORWARD ? j < il : j > il);
            const double y = fresh ? ly[j] : xold[r0 + j];
            const double t = in && j != il ? a * y : 0.0;
            if (in && j == il) d = a;
            acc = sub_terms<W>(acc, t, end - p, m1);
        }
        // exactly one lane holds the diagonal
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) d += __shfl_xor(d, o, W);
        const double xi = acc / d;
        if (lane == 0) {
            ly[il] = xi;
            xnew[i] = xi;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    auto consume = [&](int buf, int Rmax) {
        const int R = rows_in[buf][g];
        const GsRow* const row = rows[buf][g];
        const double* const tm = term[buf][g];
        const int16_t* const tg = tag[buf][g];
        const bool lng = R == 1 && row[0].len < 0;
        if (__any(lng)) {
            if (lng) long_row();
        }
        const int Rs = lng ? 0 : R;         // staged rows of this group
        // headers three rows ahead, terms two, new values one: nothing a row asks
        // for is waited for in the same step.  No branches either: lanes and steps
        // without an entry read and write spare places, so that the compiler
        // counts what is in flight.
        auto head = [&](int k) { return row[min(k, W)]; };
        auto load = [&](const GsRow& h, double& t, int& q) {
            const int p = lane < h.len ? h.off + lane : S;
            t = tm[p];
            q = (int)tg[p];
        };
        double t0, t1, y0;
        int q0, q1;
        GsRow h0 = head(0), h1 = head(1), h2 = head(2);
        load(h0, t0, q0);
        load(h1, t1, q1);
        y0 = ly[max(q0, 0)];
        int prev = -1;
        double prev_x = 0.0;
        for (int k = 0; k < Rmax; ++k) {
            const double y1 = ly[max(q1, 0)];
            double t2;
            int q2;
            load(h2, t2, q2);
            const GsRow h3 = head(k + 3);
            const double t = q0 >= 0 ? t0 * (q0 == prev ? prev_x : y0) : t0;
            double acc = sub_terms<W>(h0.b, t, h0.len, m1);
            for (int o = W; __any(o < h0.len); o += W) {
                const bool in = o + lane < h0.len;
                double tq = in ? tm[h0.off + o + lane] : 0.0;
                const int qq = in ? (int)tg[h0.off + o + lane] : (int)kGsOld;
                const double yq = ly[max(qq, 0)];
                tq = qq >= 0 ? tq * (qq == prev ? prev_x : yq) : tq;
                acc = sub_terms<W>(acc, tq, h0.len - o, m1);
            }
            const double xi = quotient(acc, h0.d, h0.y);
            const int il = row_at(at + k);
            ly[k < Rs ? il : chunk] = xi;      // every lane the same
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the store before later rows' loads
            prev = il;
            prev_x = xi;
            t0 = t1;
            q0 = q1;
            h0 = h1;
            y0 = y1;
            t1 = t2;
            q1 = q2;
            h1 = h2;
            h2 = h3;
        }
        if (lane < Rs) {
            const int il = row_at(at + lane);
            xnew[r0 + il] = ly[il];
        }
        at += R;
    };
    if (wave > 0) produce(0);
    else __builtin_amdgcn_s_setprio(2);   // the chain ahead of the staging waves of its SIMD
    __syncthreads();
    for (int buf = 0;; buf ^= 1) {
        int Rmax = 0;
#pragma unroll
        for (int c = 0; c < G; ++c) Rmax = max(Rmax, rows_in[buf][c]);
        Rmax = __builtin_amdgcn_readfirstlane(Rmax);
        if (Rmax == 0) break;               // every chunk is done, in every wave
        if (wave > 0) produce(buf ^ 1);
        else consume(buf, Rmax);
        __syncthreads();
    }
}

}  // namespace

// The chain form takes blocks of at least kGsChainMin rows, and blocks of two
// rows or more on levels of up to kGsChainRowsFew rows; below that the staged
// form's one lane per block has chains enough and is faster where rows are
// short.  A chunk is the whole blocks that fit kGsChainRows rows, fewer where
// the level has too few rows for kGsChainChunks chunks.  16 lanes to a chunk
// where rows are short and there are chunks to fill the machine four to a
// workgroup, else 64.
// A forward sweep in us, one lane per block (staged form) -> chain form, 3D
// Poisson hierarchies, levels 0, 1, 2, ...:
//   64^3, blocks of 64:   102 236 279 779 1298 675 -> 28 35 38 40 56 42
//   128^3, blocks of 64:  623 1493 942 879 1782 1760 902 -> 146 152 101 43 74 74 46
//   128^3, blocks of 16:  190 418 254 160 240 222 136 -> 149 152 101 31 26 25 19
//   128^3, blocks of 8:   126 230 130 76 295 290 80 -> 154 153 102 33 19 17 12
//   128^3, blocks of 2:   82 124 54 23 91 95 27 -> 153 153 102 30 20 9 9
//   64^3, blocks of 1024 (per-block form): 4000 11372 15617 13706 9643 996 ->
//                         336 348 405 500 412 59
// 64 lanes to a chunk on the two finest levels, blocks of 64: 99 and 77 us at
// 64^3, 658 and 409 at 128^3; 16 lanes on the third (rows of 32 entries, 342
// chunks at 64^3): 74 us.
constexpr int kGsChainMin = 16;
constexpr int kGsChainRowsFew = 16384;
constexpr int kGsChainRows = 64;
constexpr int64_t kGsChainChunks = 2048;
constexpr int64_t kGsShortRowChunks = 1024;
constexpr double kGsShortRow = 24.0;
// More staging waves where a chunk takes several strips and the chunks do not
// fill the machine (then they only share its instructions): 16 lanes, one wave or
// two (rows of 8: sixteen rows, a strip, fit one wave's); 64 lanes, two or four.
// Terms are subtracted ahead there and on rows of up to 8, not where the chunk is
// one strip, which the chain would only wait for.  us, one wave (16 lanes) or two
// and nothing ahead -> this rule: 64^3, blocks of 64, levels 0 to 4: 31 53 42 44 62
// -> 28 35 38 40 56.  Where the rule says no: four waves on 2,731 chunks of 64 rows
// 103 -> 233; terms ahead on 16,384 chunks of rows above 8 155 -> 173, on short
// chunks (blocks of 2, 128^3, level 4) 20 -> 46.
constexpr double kGsOneWaveRow = 8.0;
constexpr int kGsLongChunk = 32;
constexpr double kGsStage16 = 256.0, kGsStage64 = 1024.0;   // entries of two waves' strip
constexpr int64_t kGsFewChunks16 = 4096, kGsFewChunks64 = 512;

template <int W, int NP, bool AHEAD>
static void launch_chain(bool forward, int n, const int32_t* rp, const int32_t* ci, const double* v, const double* b,
                         const double* xold, double* xnew, int block, int chunk, hipStream_t st) {
    constexpr int G = 64 / W;
    const int64_t per = (int64_t)chunk * G;
    const dim3 grid((unsigned)((n + per - 1) / per)), threads(64 * (1 + NP));
    const size_t lds = sizeof(double) * (size_t)(G * (chunk + 1));
    if (forward)
        hipLaunchKernelGGL((hybrid_gs_chain_kernel<true, W, NP, AHEAD>), grid, threads, lds, st, n, rp, ci, v, b, xold, xnew,
                           block, chunk);
    else
        hipLaunchKernelGGL((hybrid_gs_chain_kernel<false, W, NP, AHEAD>), grid, threads, lds, st, n, rp, ci, v, b, xold, xnew,
                           block, chunk);
}

void launch_hybrid_gs(bool forward, int n, const int32_t* rp, const int32_t* ci, const double* v,
                      const double* b, const double* xold, double* xnew, int block, double mean_row,
                      hipStream_t st) {
    if (n <= 0) return;
    if (block <= kGsChainMaxRows && (block >= kGsChainMin || (block >= 2 && n <= kGsChainRowsFew))) {
        const int64_t most = std::max<int64_t>(1, kGsChainRows / block);
        const int64_t per = std::max<int64_t>(1, std::min<int64_t>(most, n / (kGsChainChunks * block)));
        const int chunk = (int)(per * block);
        const int64_t chunks = ((int64_t)n + chunk - 1) / chunk;
        // (blocks of a few rows: the chain is short, whatever the staging)
        const double entries = chunk >= kGsLongChunk ? mean_row * chunk : 0.0;
        if (mean_row <= kGsShortRow && chunks >= kGsShortRowChunks) {
            if (mean_row > kGsOneWaveRow && entries > kGsStage16 && chunks <= kGsFewChunks16)
                launch_chain<16, 2, true>(forward, n, rp, ci, v, b, xold, xnew, block, chunk, st);
            else if (mean_row <= kGsOneWaveRow && entries > kGsStage16)
                launch_chain<16, 1, true>(forward, n, rp, ci, v, b, xold, xnew, block, chunk, st);
            else launch_chain<16, 1, false>(forward, n, rp, ci, v, b, xold, xnew, block, chunk, st);
        } else if (entries > kGsStage64 && chunks <= kGsFewChunks64) {
            launch_chain<64, 4, true>(forward, n, rp, ci, v, b, xold, xnew, block, chunk, st);
        } else {
            launch_chain<64, 2, false>(forward, n, rp, ci, v, b, xold, xnew, block, chunk, st);
        }
        return;
    }
    if (block <= kGsMaxRows) {
        // chunks of whole blocks whose entries usually fit the staging buffer
        const int per = std::max(1, std::min(kGsMaxRows / block,
                                             (int)(kGsCap / (1.15 * std::max(mean_row, 1.0) * block))));
        const int R = per * block;
        const int nchunk = (n + R - 1) / R;
        const int grid = std::max(1, std::min(nchunk, 65535));
        if (forward)
            hipLaunchKernelGGL(hybrid_gs_staged_kernel<true>, dim3(grid), dim3(kGsThreads), 0, st, n, rp, ci, v, b,
                               xold, xnew, block, R);
        else
            hipLaunchKernelGGL(hybrid_gs_staged_kernel<false>, dim3(grid), dim3(kGsThreads), 0, st, n, rp, ci, v, b,
                               xold, xnew, block, R);
        return;
    }
    const int64_t nblk = ((int64_t)n + block - 1) / block;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((nblk + 255) / 256, 65535));
    if (forward)
        hipLaunchKernelGGL(hybrid_gs_kernel<true>, dim3(grid), dim3(256), 0, st, n, rp, ci, v, b, xold, xnew, block);
    else
        hipLaunchKernelGGL(hybrid_gs_kernel<false>, dim3(grid), dim3(256), 0, st, n, rp, ci, v, b, xold, xnew,
                           block);
}

}  // namespace amg355
