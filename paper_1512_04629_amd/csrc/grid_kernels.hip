// The V-cycle on the small levels (a few thousand rows, down to the coarsest)
// in one launch, and whole PCG solves of systems that small.  Launched step by
// step a level costs four launches of 3 to 5 us whatever its work (2.4 us from
// one dependent launch to the next, and a chain of cold loads), a CG iteration
// nine more and a round trip to the host.  Here kGridWgs workgroups share the
// rows of every level and meet at a barrier where one's rows need another's; a
// last workgroup holds the coarsest levels in its LDS and runs them when the
// others have restricted to them.
//
// Barriers: the workgroups wait for each other, so all of them must be on the
// device at once, which nothing promises: other streams and other processes may
// hold the compute units.  The first barrier of a launch settles it in one word,
// the gate: the last workgroup, which has the least to do before, opens it when it
// has seen all of them, one whose time runs out before that closes it, both with a
// compare-and-swap, so that all workgroups, the late ones too, find one and the
// same verdict.  Where it was closed nobody meets: the one that closed it does the
// cycle alone, far slower and with the same result to rounding (a solve tells the
// host, which launches it step by step), the others leave.  Past the gate all are
// running, and every later wait ends.  The first residual is formed before the gate
// has to be passed: a cycle takes no longer with it (501^2: 112 us), a 64^2 solve
// 366 us instead of 363.
//
// Those later barriers: every workgroup stores the number of its barrier in a
// word of its own, and one wave of each polls all words (two cache lines) until
// none is behind.  The vectors that cross workgroups are stored and loaded with
// agent-scope atomics (relaxed: they go past the L2s, which are not coherent
// with each other), and every wave waits for its stores before the workgroup's
// word is written, so no cache is written back or invalidated.  A barrier with
// the exchange around it is four trips to memory, about 3 us; with release and
// acquire fences the barrier alone took 5 at 64 workgroups.  The words go on
// counting from launch to launch: a launch reads the number to start from in
// its own word, so a captured launch can be replayed.  The polls of a wait are
// counted all the same: should one run out (a device that takes some of a
// running launch's workgroups off for seconds), the result is not a number, the
// words are unequal from then on, and `failed` keeps later launches from using
// them until the host has reported it and set them back.
//
// Two barriers a level and cycle: a workgroup forms the residual in all rows its
// share of the next level restricts from (b and dinv give the first sweep
// there), and interpolates to all columns its share of the rows needs, in LDS,
// again where its neighbours do so too: a few rows of a small level more, where
// each would be a barrier more.  Where that would repeat too much of A (dense
// small levels) the residual is exchanged instead.  Operator entries of a
// lane's first row are requested before the barrier.
#include "grid_kernels.hpp"

#include "per_device.hpp"

#include <algorithm>
#include <climits>

namespace amg355 {
namespace {

constexpr int kThreads = 1024;
constexpr int kAhead = 4;                             // entries a lane requests before a barrier
// Dynamic LDS of a launch: half a compute unit's, so that a workgroup of another
// kernel finds room beside (of these kernels the registers let one on a unit).
constexpr size_t kLdsShare = 80 * 1024;

template <class U>
using Global = __attribute__((address_space(1))) U*;
template <class U>
using Lds = __attribute__((address_space(3))) U*;
template <class U>
__device__ __forceinline__ Global<U> gp(U* p) {
    return (Global<U>)p;
}

// values that cross workgroups: past the L2s
template <class U>
__device__ __forceinline__ U xld(const U* p, int i) {
    return __hip_atomic_load(gp(p) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class U>
__device__ __forceinline__ void xst(U* p, int i, U v) {
    __hip_atomic_store(gp(p) + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct Barrier {
    unsigned* words;
    unsigned at;         // number of the last barrier announced
    bool ok;             // past every barrier so far
};

template <class U>
__device__ __forceinline__ void to_host(U* p, U v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ uint32_t* told(const Barrier& b) {
    return (uint32_t*)((uint64_t)xld(b.words, kWordTold) | (uint64_t)xld(b.words, kWordTold + 1) << 32);
}

// all stores of this wave are at their place
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ void announce(Barrier& b) {
    stores_done();
    __syncthreads();
    b.at += 1;
    if (threadIdx.x == 0) xst(b.words, blockIdx.x, b.at);
}

// every workgroup has announced this barrier or a later one (differences, so
// that the count may wrap); false if the wait ran out
__device__ __forceinline__ bool await_all(Barrier& b) {
    __shared__ int reached;
    static_assert(kGridWgs < 64);
    if (threadIdx.x < 64) {
        bool all = false;
        for (unsigned poll = 0;; ++poll) {
            all = __all((int)threadIdx.x > kGridWgs || (int)(xld(b.words, threadIdx.x) - b.at) >= 0);
            if (all || ((poll & 255) == 255 && poll >= xld(b.words, kWordPolls))) break;
        }
        if (threadIdx.x == 0) {
            reached = all ? 1 : 0;
            if (!all) {
                xst(b.words, kWordFailed, 1u);
                to_host(told(b) + kToldLost, 1u);
            }
        }
    }
    __syncthreads();
    b.ok = b.ok && reached != 0;
    return b.ok;
}

// The gate: whether the workgroups of this launch met at its first barrier.  The
// word's values are the barrier's own, so nothing has to be cleared.
enum Verdict : int {
    kOpen,      // all are here
    kClosed,    // leave
    kAlone      // this workgroup closed it
};

// the first wave: the gate, seen as g, says v from now on, unless it has said
// otherwise
__device__ __forceinline__ bool decide(const Barrier& b, unsigned g, unsigned v) {
    int won = 0;
    if (threadIdx.x == 0)
        while (!won && g != 2u * b.at && g != 2u * b.at + 1u)
            won = __hip_atomic_compare_exchange_strong(gp(b.words) + kWordGate, &g, v, __ATOMIC_RELAXED,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_amdgcn_readfirstlane(won) != 0;
}

// the first barrier's wait (announced)
__device__ __forceinline__ Verdict pass_gate(const Barrier& b) {
    __shared__ int found;
    if (threadIdx.x < 64) {
        const unsigned go = 2u * b.at, shut = go + 1u;
        const unsigned long long start = __builtin_amdgcn_s_memrealtime();
        const unsigned ticks = xld(b.words, kWordTicks), absent = xld(b.words, kWordAbsent);
        int verdict = -1;
        do {
            unsigned g = 0;
            for (int poll = 0; poll < 32 && verdict < 0; ++poll) {
                g = __builtin_amdgcn_readfirstlane(xld(b.words, kWordGate));
                if (g == go) verdict = kOpen;
                else if (g == shut) verdict = kClosed;
                else if (blockIdx.x == kGridWgs && absent != kAbsentAtGate &&
                         __all((int)threadIdx.x > kGridWgs || (int)(xld(b.words, threadIdx.x) - b.at) >= 0))
                    verdict = decide(b, g, go) ? kOpen : kClosed;
            }
            if (verdict < 0 && __builtin_amdgcn_s_memrealtime() - start >= ticks && decide(b, g, shut))
                verdict = kAlone;   // (else it was decided meanwhile: the next look says how)
        } while (verdict < 0);
        if (threadIdx.x == 0) {
            found = verdict;
            if (verdict == kAlone) to_host(told(b) + kToldClosed, 1u);
        }
    }
    __syncthreads();
    return (Verdict)found;
}

// rows [lo, hi) and the lanes each is given
struct Rows {
    int lo, hi, lanes;
};
__device__ __forceinline__ Rows rows_of(int lo, int hi, int most) {
    int w = 1;
    while (w < most && 2 * w * (hi - lo) <= kThreads) w *= 2;
    return Rows{lo, hi, w};
}
template <class T>
__device__ __forceinline__ Rows share_of(const GridOp<T>& op) {
    const int per = (op.rows + kGridWgs - 1) / kGridWgs;
    const int lo = min(op.rows, (int)blockIdx.x * per);
    return rows_of(lo, min(op.rows, lo + per), op.lanes);
}
template <class T>
__device__ __forceinline__ int window(const GridLevel<T>& L, int k) {
    return gp(L.win)[kWinInts * blockIdx.x + k];
}

// entries of the first row this lane's group takes (column -1: none)
template <class T>
struct Ahead {
    int beg, end;
    int c[kAhead];
    T v[kAhead];
};
template <class T>
__device__ __forceinline__ Ahead<T> request(const GridOp<T>& op, const Rows& s) {
    Ahead<T> h;
    const int row = s.lo + (int)threadIdx.x / s.lanes, lane = (int)threadIdx.x & (s.lanes - 1);
    const bool have = row < s.hi;
    h.beg = have ? gp(op.rp)[row] : 0;
    h.end = have ? gp(op.rp)[row + 1] : 0;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
        const int p = h.beg + lane + k * s.lanes;
        const bool in = p < h.end;
        h.c[k] = in ? gp(op.ci)[p] : -1;
        h.v[k] = in ? gp(op.v)[p] : T(0);
    }
    return h;
}

// put(row, sum over the row of v g) for every row, in the first lane of its
// group; g in LDS, its first entry standing for column c0
template <class T, class F>
__device__ __forceinline__ void row_sums(const GridOp<T>& op, const Rows& s, const Ahead<T>& h, Lds<T> g, int c0,
                                         F&& put) {
    const int W = s.lanes, lane = (int)threadIdx.x & (W - 1);
    const int first = s.lo + (int)threadIdx.x / W, stride = kThreads / W;
    for (int row = first; row < s.hi; row += stride) {
        T sum = T(0);
        int p, end;
        if (row == first) {
#pragma unroll
            for (int k = 0; k < kAhead; ++k)
                if (h.c[k] >= 0) sum += h.v[k] * g[h.c[k] - c0];
            p = h.beg + lane + kAhead * W;
            end = h.end;
        } else {
            p = gp(op.rp)[row] + lane;
            end = gp(op.rp)[row + 1];
        }
        for (; p + 3 * W < end; p += 4 * W) {
            int c[4];
            T v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = gp(op.ci)[p + q * W];
                v[q] = gp(op.v)[p + q * W];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) sum += v[q] * g[c[q] - c0];
        }
        for (; p < end; p += W) sum += gp(op.v)[p] * g[gp(op.ci)[p] - c0];
        for (int o = W / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) put(row, sum);
    }
}

// to(i, from[i]) for i in [lo, hi), four loads in flight
template <class T, class F>
__device__ __forceinline__ void fetch(const T* from, int lo, int hi, F&& to) {
    for (int i = lo + (int)threadIdx.x; i < hi; i += 4 * kThreads) {
        T t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k * kThreads < hi) t[k] = xld(from, i + k * kThreads);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k * kThreads < hi) to(i + k * kThreads, t[k]);
    }
}

// ---- the coarsest levels in the last workgroup's LDS -------------------------------

constexpr int kTailLanes = 8;

template <class U>
__device__ __forceinline__ Lds<U> at(Lds<unsigned char> m, uint32_t off) {
    return (Lds<U>)(m + off);
}

template <int STEP, class T>
__device__ __forceinline__ void tail_step(Lds<unsigned char> m, const GridTailMat& a, uint32_t g, uint32_t u,
                                          uint32_t dinv, T omega, uint32_t y, uint32_t y2) {
    const Lds<int32_t> rp = at<int32_t>(m, a.rp), ci = at<int32_t>(m, a.ci);
    const Lds<T> v = at<T>(m, a.v), gv = at<T>(m, g), yv = at<T>(m, y);
    const int lane = threadIdx.x & (kTailLanes - 1);
    for (int row = threadIdx.x / kTailLanes; row < a.rows; row += kThreads / kTailLanes) {
        const int end = rp[row + 1];
        int p = rp[row] + lane;
        T s = T(0);
        for (; p + 3 * kTailLanes < end; p += 4 * kTailLanes) {
            int c[4];
            T w[4], x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = ci[p + q * kTailLanes];
                w[q] = v[p + q * kTailLanes];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) x[q] = gv[c[q]];
#pragma unroll
            for (int q = 0; q < 4; ++q) s += w[q] * x[q];
        }
        for (; p < end; p += kTailLanes) s += v[p] * gv[ci[p]];
#pragma unroll
        for (int o = kTailLanes / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kTailLanes);
        if (lane == 0) {
            if constexpr (STEP == 0) yv[row] = at<T>(m, u)[row] - s;
            else if constexpr (STEP == 1) {
                yv[row] = s;
                at<T>(m, y2)[row] = omega * (at<T>(m, dinv)[row] * s);
            } else if constexpr (STEP == 2) yv[row] = s;
            else if constexpr (STEP == 3) yv[row] = at<T>(m, u)[row] + s;
            else yv[row] = gv[row] + omega * at<T>(m, dinv)[row] * (at<T>(m, u)[row] - s);
        }
    }
    __syncthreads();
}

// copies the arrays a wave-wide load (64 words) at a time straight into LDS;
// waited for at the next barrier
template <class T>
__device__ __forceinline__ void tail_stage(const GridArgs<T>& a, Lds<unsigned char> m) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    for (int q = 0; q < a.runs; ++q) {
        const GridRun r = a.run[q];
        for (uint32_t w = 64 * wave; w < r.words; w += kThreads) {
            const uint32_t dst = __builtin_amdgcn_readfirstlane(r.dst + 4 * w);
            if (w + lane < r.words)
                __builtin_amdgcn_global_load_lds((Global<const void>)(r.src + w + lane), (Lds<void>)(m + dst), 4, 0, 0);
        }
    }
}

template <class T>
__device__ __forceinline__ void tail_cycle(const GridArgs<T>& a, Lds<unsigned char> m) {
    const int last = a.tail_count - 1;
    const GridTailLevel& F = a.tl[0];
    for (int i = threadIdx.x; i < F.n; i += kThreads) {
        const T bi = xld(a.tail_b, i);
        at<T>(m, F.b)[i] = bi;
        if (last > 0) at<T>(m, F.x)[i] = a.omega * (at<T>(m, F.dinv)[i] * bi);
    }
    __syncthreads();
    for (int k = 0; k < last; ++k) {
        const GridTailLevel &L = a.tl[k], &N = a.tl[k + 1];
        tail_step<0, T>(m, L.A, L.x, L.b, 0, a.omega, L.r, 0);
        if (k + 1 < last) tail_step<1, T>(m, L.R, L.r, 0, N.dinv, a.omega, N.b, N.x);
        else tail_step<2, T>(m, L.R, L.r, 0, 0, a.omega, N.b, 0);
    }
    {
        // x = inverse b: 16 lanes a row
        const GridTailLevel& C = a.tl[last];
        const Lds<double> inv = at<double>(m, a.inv);
        const int lane = threadIdx.x & 15;
        for (int i = threadIdx.x / 16; i < C.n; i += kThreads / 16) {
            double s = 0.0;
            for (int j = lane; j < C.n; j += 16) s += inv[i * C.n + j] * (double)at<T>(m, C.b)[j];
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 16);
            if (lane == 0) at<T>(m, C.x)[i] = (T)s;
        }
        __syncthreads();
    }
    for (int k = last - 1; k >= 0; --k) {
        const GridTailLevel &L = a.tl[k], &N = a.tl[k + 1];
        tail_step<3, T>(m, L.P, k + 1 == last ? N.x : N.xt, L.x, 0, a.omega, L.x, 0);
        tail_step<4, T>(m, L.A, L.x, L.b, L.dinv, a.omega, L.xt, 0);
    }
    for (int i = threadIdx.x; i < F.n; i += kThreads) xst(a.tail_out, i, at<T>(m, last > 0 ? F.xt : F.x)[i]);
}

// ---- the cycle -----------------------------------------------------------------

// One cycle from zero: on entry the barrier after lv[0].b's last store is
// announced, not awaited, or (GATED) lv[0].b is there and first() is the launch's
// gate, passed before anything is stored; on exit lv[0].xt is stored, its
// barrier not announced.  ready() runs after the first barrier and returns
// whether to go on; done(row, value) sees the share's rows of the result.  False:
// the workgroups do not meet (any more), or ready() said so.
template <bool GATED, class T, class First, class Ready, class Done>
__device__ __forceinline__ bool cycle(const GridArgs<T>& a, Barrier& b, Lds<unsigned char> m, First&& first,
                                      Ready&& ready, Done&& done) {
    const T omega = a.omega;
    auto meet = [&] { return await_all(b); };
    if (blockIdx.x == kGridWgs) {
        const unsigned absent = xld(b.words, kWordAbsent);
        for (int k = 0; k < a.count; ++k) {
            if (!(GATED && k == 0 ? first() : meet())) return false;
            if (k == 0 && !ready()) return false;
            if (!a.lv[k].fused) {
                announce(b);
                if (!meet()) return false;
            }
            announce(b);
        }
        if (!meet()) return false;
        if (absent == kAbsentLater) {
            b.ok = false;
            return false;
        }
        tail_cycle(a, m);
        announce(b);
        for (int k = a.count - 1; k > 0; --k) {
            if (!meet()) return false;
            announce(b);
        }
        return meet();
    }
    for (int k = 0; k < a.count; ++k) {
        const GridLevel<T>& L = a.lv[k];
        const Rows coarse = share_of(L.R);
        const int f0 = window(L, kWinF0), f1 = window(L, kWinF1);
        T* const nb = k + 1 < a.count ? a.lv[k + 1].b : a.tail_b;
        // the residual: in every row the share of the next level restricts from,
        // or in the level's own share, to be exchanged
        const Rows fine = L.fused ? rows_of(f0, f1, L.A.lanes) : share_of(L.A);
        const int x0 = window(L, L.fused ? kWinX0 : kWinY0), x1 = window(L, L.fused ? kWinX1 : kWinY1);
        const Lds<T> x = (Lds<T>)m;
        Lds<T> r = x + (x1 - x0);
        const Ahead<T> ha = request(L.A, fine);
        const bool gate = GATED && k == 0;
        if (!gate && !meet()) return false;
        fetch(L.b, x0, x1, [&](int i, T bi) {
            x[i - x0] = omega * (gp(L.dinv)[i] * bi);
            if (i >= fine.lo && i < fine.hi) r[i - fine.lo] = bi;
        });
        if (k == 0 && !ready()) return false;
        const Ahead<T> hr = request(L.R, coarse);
        __syncthreads();
        if (gate && !L.fused && !first()) return false;
        row_sums(L.A, fine, ha, x, x0, [&](int i, T t) {
            const T ri = r[i - fine.lo] - t;
            if (L.fused) r[i - fine.lo] = ri;
            else xst(L.r, i, ri);
        });
        if (L.fused) {
            __syncthreads();
            if (gate && !first()) return false;
        } else {
            announce(b);
            if (!meet()) return false;
            r = x;
            fetch(L.r, f0, f1, [&](int i, T ri) { r[i - f0] = ri; });
            __syncthreads();
        }
        row_sums(L.R, coarse, hr, r, f0, [&](int i, T t) { xst(nb, i, t); });
        announce(b);
    }
    if (!meet()) return false;   // the tail's right-hand side
    announce(b);
    for (int k = a.count - 1; k >= 0; --k) {
        const GridLevel<T>& L = a.lv[k];
        const Rows own = share_of(L.A);
        const int y0 = window(L, kWinY0), y1 = window(L, kWinY1), c0 = window(L, kWinC0), c1 = window(L, kWinC1);
        const Rows reach = rows_of(y0, y1, L.P.lanes);
        const Lds<T> x = (Lds<T>)m, bo = x + (y1 - y0), xc = bo + (own.hi - own.lo);
        // what does not depend on the coarse result: the first sweep, entries
        fetch(L.b, y0, y1, [&](int i, T bi) {
            x[i - y0] = omega * (gp(L.dinv)[i] * bi);
            if (i >= own.lo && i < own.hi) bo[i - own.lo] = bi;
        });
        const Ahead<T> hp = request(L.P, reach);
        if (!meet()) return false;
        fetch(k + 1 < a.count ? a.lv[k + 1].xt : a.tail_out, c0, c1, [&](int i, T v) { xc[i - c0] = v; });
        const Ahead<T> ha = request(L.A, own);
        __syncthreads();
        row_sums(L.P, reach, hp, xc, c0, [&](int i, T s) { x[i - y0] = x[i - y0] + s; });
        __syncthreads();
        row_sums(L.A, own, ha, x, y0, [&](int i, T s) {
            const T xn = x[i - y0] + omega * gp(L.dinv)[i] * (bo[i - own.lo] - s);
            xst(L.xt, i, xn);
            if (k == 0) done(i, xn);
        });
        if (k > 0) announce(b);
    }
    return true;
}

// The same cycle by one workgroup, the vectors in memory.
template <class T, class Get, class Put>
__device__ __forceinline__ void rows_alone(const GridOp<T>& op, Get&& get, Put&& put) {
    const int W = op.lanes, lane = (int)threadIdx.x & (W - 1);
    for (int row = (int)threadIdx.x / W; row < op.rows; row += kThreads / W) {
        T sum = T(0);
        for (int p = gp(op.rp)[row] + lane; p < gp(op.rp)[row + 1]; p += W) sum += gp(op.v)[p] * get(gp(op.ci)[p]);
        for (int o = W / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) put(row, sum);
    }
    stores_done();
    __syncthreads();
}

template <class T>
__device__ __forceinline__ void cycle_alone(const GridArgs<T>& a, Lds<unsigned char> m) {
    for (int k = 0; k < a.count; ++k) {
        const GridLevel<T>& L = a.lv[k];
        T* const nb = k + 1 < a.count ? a.lv[k + 1].b : a.tail_b;
        rows_alone(L.A, [&](int j) { return a.omega * (gp(L.dinv)[j] * xld(L.b, j)); },
                   [&](int i, T t) { xst(L.r, i, xld(L.b, i) - t); });
        rows_alone(L.R, [&](int j) { return xld(L.r, j); }, [&](int i, T t) { xst(nb, i, t); });
    }
    tail_stage(a, m);
    stores_done();     // (the loads to LDS count with them)
    __syncthreads();
    tail_cycle(a, m);
    stores_done();
    __syncthreads();
    for (int k = a.count - 1; k >= 0; --k) {
        const GridLevel<T>& L = a.lv[k];
        const T* const xc = k + 1 < a.count ? a.lv[k + 1].xt : a.tail_out;
        rows_alone(L.P, [&](int j) { return xld(xc, j); },
                   [&](int i, T t) { xst(L.r, i, a.omega * (gp(L.dinv)[i] * xld(L.b, i)) + t); });
        rows_alone(L.A, [&](int j) { return xld(L.r, j); }, [&](int i, T t) {
            xst(L.xt, i, xld(L.r, i) + a.omega * gp(L.dinv)[i] * (xld(L.b, i) - t));
        });
    }
}

// number of the last barrier of the launches before this one, which are done:
// every workgroup's word holds it, unless one of them was lost
template <class T>
__device__ __forceinline__ Barrier first_barrier(const GridArgs<T>& a) {
    const unsigned at = xld(a.words, blockIdx.x), failed = xld(a.words, kWordFailed);
    return Barrier{a.words, (unsigned)__builtin_amdgcn_readfirstlane(at), __builtin_amdgcn_readfirstlane(failed) == 0};
}

template <class T>
__global__ __launch_bounds__(kThreads) void grid_cycle_kernel(GridArgs<T> a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds<unsigned char> m = (Lds<unsigned char>)smem;
    Barrier b = first_barrier(a);
    Verdict gate = kOpen;
    if (b.ok) {
        announce(b);     // nothing to wait for: the launch before stored lv[0].b
        if (blockIdx.x == kGridWgs) tail_stage(a, m);
        (void)cycle<true>(a, b, m, [&] { return (gate = pass_gate(b)) == kOpen; }, [] { return true; }, [](int, T) {});
    }
    if (gate == kAlone) cycle_alone(a, m);
    if (!b.ok && blockIdx.x < kGridWgs) {
        // lost: the result is not a number
        const Rows s = share_of(a.lv[0].A);
        for (int i = s.lo + (int)threadIdx.x; i < s.hi; i += kThreads) xst(a.lv[0].xt, i, (T)__builtin_nanf(""));
    }
}

// ---- PCG ------------------------------------------------------------------------

// sum of the workgroups' partials of a slot, the same in every wave
__device__ __forceinline__ double total(const double* part, int slot) {
    const int lane = (int)threadIdx.x & 63;
    double v = lane < kGridWgs ? xld(part, slot * kGridWgs + lane) : 0.0;
#pragma unroll
    for (int o = kGridWgs / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return __shfl(v, 0, 64);
}

// this workgroup's partial of a slot: v summed over its threads
__device__ __forceinline__ void put_partial(double* part, int slot, double v) {
    __shared__ double wsum[kThreads / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x / 64] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = wsum[0];
        for (int w = 1; w < kThreads / 64; ++w) t += wsum[w];
        xst(part, slot * kGridWgs + (int)blockIdx.x, t);
    }
}

enum { kPartNorm = 0, kPartPq = 1, kPartRz = 2, kPartTrue = 3 };

// The iteration of `solve` (amg_lib.hip): the same tests in the same order, all
// workgroups taking them on the same numbers.
template <class T>
__global__ __launch_bounds__(kThreads) void grid_solve_kernel(GridArgs<T> a, GridSolve s) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds<unsigned char> m = (Lds<unsigned char>)smem;
    const Lds<double> win = (Lds<double>)smem;
    const GridLevel<T>& F = a.lv[0];
    // the end of the launch for the host (one thread)
    auto tell = [&](double status, int iters) {
        to_host(s.out + kGridOutStatus, status);
        to_host(s.out + kGridOutIters, (double)iters);
        stores_done();
        to_host(s.done, s.seq);
    };
    const bool worker = blockIdx.x < kGridWgs, teller = blockIdx.x == 0 && threadIdx.x == 0;
    const Rows own = worker ? share_of(s.A) : Rows{0, 0, 1};
    const int y0 = worker ? window(F, kWinY0) : 0, y1 = worker ? window(F, kWinY1) : 0;
    Barrier b = first_barrier(a);
    if (!b.ok) {                      // (the host sets the words back before it launches)
        if (teller) tell(-1.0, s.iters);
        return;
    }
    announce(b);                      // the gate's barrier: workers store what follows before the next one
    if (!worker) tail_stage(a, m);
    // y = b - A x in the share's rows and its squared norm in a slot
    auto residual = [&](double* y, int slot) {
        double n2 = 0.0;
        if (worker) {
            const Ahead<double> h = request(s.A, own);
            fetch(s.x, y0, y1, [&](int i, double v) { win[i - y0] = v; });
            __syncthreads();
            row_sums(s.A, own, h, win, y0, [&](int i, double t) {
                const double ri = gp(s.b)[i] - t;
                xst(y, i, ri);
                n2 += ri * ri;
            });
            put_partial(s.part, slot, n2);
        }
    };
    // the cycle's right-hand side in the share's rows
    auto precision = [&](int i, double ri) { xst(F.b, i, (T)ri); };
    double nr0 = s.nr0, nws = s.nws, rz = 0.0, nrt = -1.0;
    int iters = s.iters, inwin = 0, status = kGridMaxit;
    bool live = true;                 // the solve goes on; b.ok: so does the launch
    if (s.start == 0) {
        residual(s.r, kPartNorm);
        if (worker) {
            __syncthreads();
            for (int i = own.lo + (int)threadIdx.x; i < own.hi; i += kThreads) precision(i, xld(s.r, i));
        }
    } else if (worker) {
        double n2 = 0.0;
        for (int i = own.lo + (int)threadIdx.x; i < own.hi; i += kThreads) {
            if (s.start == 1) {
                const double bi = gp(s.b)[i];
                xst(s.x, i, 0.0);
                xst(s.r, i, bi);
                precision(i, bi);
                n2 += bi * bi;
            } else {
                precision(i, xld(s.r, i));
            }
        }
        put_partial(s.part, kPartNorm, n2);
    }
    if (worker)
        for (int i = own.lo + (int)threadIdx.x; i < own.hi; i += kThreads) xst(s.xw, i, s.start == 1 ? 0.0 : xld(s.x, i));
    if (const Verdict gate = pass_gate(b); gate != kOpen) {
        // x, and for a resumed solve r, are as they were (x = 0 for a zero guess)
        if (gate == kAlone && threadIdx.x == 0) tell(kGridClosed, iters);
        return;
    }
    announce(b);
    auto meet = [&] { return await_all(b); };
    double *p = s.p, *p2 = s.p2;
    bool fresh = true;                // p = z
    for (;;) {
        // the residual is stored and its barrier announced; its norm decides
        double rzp = 0.0;
        auto ready = [&] {
            if (fresh && s.start != 2) {
                nr0 = sqrt(total(s.part, kPartNorm));
                nws = nr0;
                if (teller) to_host(s.hist, nr0);
                if (s.singular && *s.singular != 0) {
                    live = false;                // the host reports it; x stays as it is
                } else if (!isfinite(nr0)) {
                    status = kGridBreakdown;
                    live = false;
                } else if (nr0 == 0.0) {
                    status = kGridConverged;
                    live = false;
                }
            } else if (!fresh) {
                const double nr = sqrt(total(s.part, kPartNorm));
                iters += 1;
                inwin += 1;
                if (teller) to_host(s.hist + iters, nr);
                const bool window_end = s.adaptive && inwin == s.k;
                if (window_end) nrt = sqrt(total(s.part, kPartTrue));
                if (!isfinite(nr)) {
                    status = kGridBreakdown;
                    live = false;
                } else if (nr <= s.rtol * nr0) {
                    status = kGridConverged;
                    live = false;
                } else if (window_end) {
                    if (nrt / nws > s.window_limit && s.any_gamma) {
                        status = kGridReintroduce;
                        live = false;
                    } else {
                        if (worker)
                            for (int i = own.lo + (int)threadIdx.x; i < own.hi; i += kThreads)
                                xst(s.xw, i, xld(s.x, i));
                        nws = nrt;
                        nrt = -1.0;
                        inwin = 0;
                    }
                }
            }
            if (live && iters >= s.maxit) live = false;
            return live;
        };
        const bool cycled = cycle<false>(a, b, m, meet, ready, [&](int i, T z) { rzp += xld(s.r, i) * (double)z; });
        if (!cycled) break;
        if (worker) put_partial(s.part, kPartRz, rzp);
        announce(b);
        // p = z + beta p in the columns the share's rows have, q = A p
        const Ahead<double> h = request(s.A, own);
        if (!meet()) break;
        const double rz_new = total(s.part, kPartRz);
        const double beta = fresh ? 0.0 : rz_new / rz;
        rz = rz_new;
        double pq = 0.0;
        if (worker) {
            for (int i = y0 + (int)threadIdx.x; i < y1; i += 2 * kThreads) {
                double z[2], po[2];
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (i + k * kThreads < y1) {
                        z[k] = (double)xld(F.xt, i + k * kThreads);
                        po[k] = fresh ? 0.0 : xld(p, i + k * kThreads);
                    }
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (i + k * kThreads < y1) {
                        const int j = i + k * kThreads;
                        const double pj = fresh ? z[k] : z[k] + beta * po[k];
                        win[j - y0] = pj;
                        if (j >= own.lo && j < own.hi) xst(p2, j, pj);
                    }
            }
            __syncthreads();
            row_sums(s.A, own, h, win, y0, [&](int i, double t) {
                xst(s.q, i, t);
                pq += win[i - y0] * t;
            });
            put_partial(s.part, kPartPq, pq);
        }
        double* const was = p;
        p = p2;
        p2 = was;
        fresh = false;
        announce(b);
        if (!meet()) break;
        // x += alpha p, r -= alpha q
        const double den = total(s.part, kPartPq);
        if (!(den > 0.0 && isfinite(den))) {
            status = kGridBreakdown;
            live = false;
            break;
        }
        const double alpha = rz / den;
        double n2 = 0.0;
        if (worker) {
            for (int i = own.lo + (int)threadIdx.x; i < own.hi; i += kThreads) {
                xst(s.x, i, xld(s.x, i) + alpha * xld(p, i));
                const double ri = xld(s.r, i) - alpha * xld(s.q, i);
                xst(s.r, i, ri);
                precision(i, ri);
                n2 += ri * ri;
            }
            put_partial(s.part, kPartNorm, n2);
        }
        announce(b);
        if (s.adaptive && inwin + 1 == s.k) {
            // a window ends with this iteration: the true residual
            if (!meet()) break;
            residual(s.rt, kPartTrue);
            announce(b);
        }
    }
    // the true residual of the result; a finished window has it
    if (b.ok && nrt < 0.0) {
        announce(b);
        if (meet()) {
            residual(s.rt, kPartTrue);
            announce(b);
            if (meet()) nrt = sqrt(total(s.part, kPartTrue));
        }
    }
    if (teller) {
        to_host(s.out + kGridOutNorm0, nr0);
        to_host(s.out + kGridOutTrue, nrt);
        to_host(s.out + kGridOutWindow, nws);
        to_host(s.out + kGridOutSingular, s.singular ? (double)*s.singular : 0.0);
        tell(b.ok ? (double)status : -1.0, iters);
    }
}

// ---- setup ----------------------------------------------------------------------

// smallest first and largest last column of rows [lo, hi) (columns ascend)
__device__ __forceinline__ int2 span_of(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, int lo, int hi) {
    __shared__ int lo_s[4], hi_s[4];
    int a = INT_MAX, z = 0;
    for (int r = lo + (int)threadIdx.x; r < hi; r += 256) {
        const int b = rp[r], e = rp[r + 1];
        if (e > b) {
            a = min(a, ci[b]);
            z = max(z, ci[e - 1] + 1);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a = min(a, __shfl_xor(a, o, 64));
        z = max(z, __shfl_xor(z, o, 64));
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        lo_s[threadIdx.x / 64] = a;
        hi_s[threadIdx.x / 64] = z;
    }
    __syncthreads();
    a = min(min(lo_s[0], lo_s[1]), min(lo_s[2], lo_s[3]));
    z = max(max(hi_s[0], hi_s[1]), max(hi_s[2], hi_s[3]));
    return a < z ? make_int2(a, z) : make_int2(0, 0);
}

__global__ __launch_bounds__(256) void grid_windows_kernel(int rows, int coarse, const int32_t* __restrict__ a_rp,
                                                           const int32_t* __restrict__ a_ci,
                                                           const int32_t* __restrict__ r_rp,
                                                           const int32_t* __restrict__ r_ci,
                                                           const int32_t* __restrict__ p_rp,
                                                           const int32_t* __restrict__ p_ci, int32_t* __restrict__ win,
                                                           int32_t* most) {
    const int w = blockIdx.x;
    const int cper = (coarse + kGridWgs - 1) / kGridWgs, per = (rows + kGridWgs - 1) / kGridWgs;
    const int2 f = span_of(r_rp, r_ci, min(coarse, w * cper), min(coarse, w * cper + cper));
    const int2 x = span_of(a_rp, a_ci, f.x, f.y);
    const int lo = min(rows, w * per), hi = min(rows, lo + per);
    const int2 y = span_of(a_rp, a_ci, lo, hi);
    const int2 c = span_of(p_rp, p_ci, y.x, y.y);
    if (threadIdx.x == 0) {
        int32_t* q = win + kWinInts * w;
        q[kWinF0] = f.x;
        q[kWinF1] = f.y;
        q[kWinX0] = x.x;
        q[kWinX1] = x.y;
        q[kWinY0] = y.x;
        q[kWinY1] = y.y;
        q[kWinC0] = c.x;
        q[kWinC1] = c.y;
        atomicMax(most, max((x.y - x.x) + (f.y - f.x), (y.y - y.x) + (hi - lo) + (c.y - c.x)));
        atomicMax(most + 1, a_rp[f.y] - a_rp[f.x]);
        atomicMax(most + 2, a_rp[hi] - a_rp[lo]);
    }
}

}  // namespace

void launch_grid_windows(int rows, int coarse, const int32_t* a_rp, const int32_t* a_ci, const int32_t* r_rp,
                         const int32_t* r_ci, const int32_t* p_rp, const int32_t* p_ci, int32_t* win, int32_t* most,
                         hipStream_t st) {
    hipLaunchKernelGGL(grid_windows_kernel, dim3(kGridWgs), dim3(256), 0, st, rows, coarse, a_rp, a_ci, r_rp, r_ci,
                       p_rp, p_ci, win, most);
}

GridLimits grid_limits() {
    return per_device([](int dev) {
        int per_block = 0, cus = 0;
        if (hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return GridLimits{};
        const void* const kernels[] = {
            reinterpret_cast<const void*>(grid_cycle_kernel<double>), reinterpret_cast<const void*>(grid_cycle_kernel<float>),
            reinterpret_cast<const void*>(grid_solve_kernel<double>), reinterpret_cast<const void*>(grid_solve_kernel<float>)};
        size_t lds = (size_t)per_block;
        for (const void* k : kernels) {
            hipFuncAttributes fa{};
            if (hipFuncGetAttributes(&fa, k) != hipSuccess || (size_t)per_block <= fa.sharedSizeBytes) return GridLimits{};
            const size_t dyn = (size_t)per_block - fa.sharedSizeBytes;
            if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn) != hipSuccess)
                return GridLimits{};
            lds = std::min(lds, std::min(dyn, kLdsShare - fa.sharedSizeBytes));
        }
        int per_cu = INT_MAX;
        for (const void* k : kernels) {
            int here = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&here, k, kThreads, lds) != hipSuccess) return GridLimits{};
            per_cu = std::min(per_cu, here);
        }
        return GridLimits{lds, grid_launches(cus, per_cu)};
    });
}

void launch_grid_cycle(const GridArgs<double>& a, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL(grid_cycle_kernel<double>, dim3(kGridWgs + 1), dim3(kThreads), lds, st, a);
}
void launch_grid_cycle(const GridArgs<float>& a, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL(grid_cycle_kernel<float>, dim3(kGridWgs + 1), dim3(kThreads), lds, st, a);
}
void launch_grid_solve(const GridArgs<double>& a, const GridSolve& s, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL(grid_solve_kernel<double>, dim3(kGridWgs + 1), dim3(kThreads), lds, st, a, s);
}
void launch_grid_solve(const GridArgs<float>& a, const GridSolve& s, size_t lds, hipStream_t st) {
    hipLaunchKernelGGL(grid_solve_kernel<float>, dim3(kGridWgs + 1), dim3(kThreads), lds, st, a, s);
}

}  // namespace amg355
