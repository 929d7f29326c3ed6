// Small levels and small systems in one launch: the V(1,1) Jacobi cycle from a
// level of a few thousand rows down, and whole PCG solves where the finest
// level is that small.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace amg355 {

// Workgroups that share the levels' rows (one more keeps the coarsest levels
// in its LDS), and the most levels of either kind a launch takes.
constexpr int kGridWgs = 32;
constexpr int kGridLevels = 6;
constexpr int kGridTailLevels = 4;

// A handle's barrier words, kept from launch to launch: one a workgroup and, in a
// cache line of their own, the gate of a launch and whether a launch was lost
// (grid_kernels.hip); then how long workgroups wait, at the gate in ticks of the
// 100 MHz clock and at later barriers in polls (0.7 us), what a test takes away,
// and the address of the words the host reads (two words).
enum {
    kWordGate = 64, kWordFailed, kWordTicks = 96, kWordPolls, kWordAbsent, kWordTold, kGridWords = kWordTold + 2
};
enum { kToldClosed = 0, kToldLost, kToldWords };
constexpr unsigned kGateTicks = 10000000;   // 0.1 s: the device is shared
constexpr unsigned kLatePolls = 1u << 23;   // 6 s
// For tests: the gate does not open, in any launch or in those that resume a
// solve, or the coarsest levels' workgroup leaves instead of running them.
enum { kAbsentAtGate = 1, kAbsentLater = 2, kAbsentResumed = 3 };

template <class T>
struct GridOp {
    const int32_t* rp;
    const int32_t* ci;
    const T* v;
    int rows;
    int lanes;           // most lanes a row is given (a power of two)
};
// Index ranges of a level, per workgroup (win[8 w + ...]): the level's rows that
// its share of the next level's rows restricts from, the columns A has in
// them; the columns A has in its share of the level's own rows, and the next
// level's points that P reaches from those.
enum { kWinF0 = 0, kWinF1, kWinX0, kWinX1, kWinY0, kWinY1, kWinC0, kWinC1, kWinInts };
template <class T>
struct GridLevel {
    GridOp<T> A, R, P;   // R to the next level, P from it
    const T* dinv;
    const int32_t* win;
    T *b, *xt, *r;       // right-hand side, result, residual
    int fused;           // the residual is formed again by every workgroup that restricts from it
};
// An array the last workgroup copies into its LDS at the start.
struct GridRun {
    const uint32_t* src;
    uint32_t words, dst;     // 4-byte words; byte offset in LDS
};
struct GridTailMat {
    uint32_t rp, ci, v;      // byte offsets in LDS
    int32_t rows;
};
struct GridTailLevel {
    GridTailMat A, R, P;
    uint32_t dinv, b, x, xt, r;
    int32_t n;
};
template <class T>
struct GridArgs {
    GridLevel<T> lv[kGridLevels];
    int count;                               // shared levels
    GridTailLevel tl[kGridTailLevels];
    int tail_count;                          // levels of the last workgroup, the coarsest one last
    GridRun run[10 * kGridTailLevels];
    int runs;
    uint32_t inv;                            // LDS offset of the coarsest inverse (FP64)
    T *tail_b, *tail_out;                    // in memory: the first tail level's right-hand side and result
    T omega;
    unsigned* words;                         // kGridWords
};

// What a solve adds; the cycle's lv[0] is the finest level.  Numbers the host
// reads are written to host-coherent memory, `done` last.
// (closed: the workgroups were not there together, nothing was done)
enum { kGridConverged = 0, kGridMaxit = 1, kGridBreakdown = 2, kGridReintroduce = 3, kGridClosed = 4 };
enum { kGridOutStatus = 0, kGridOutIters, kGridOutNorm0, kGridOutTrue, kGridOutWindow, kGridOutSingular, kGridOutInts };
struct GridSolve {
    GridOp<double> A;                        // the finest operator, FP64
    const double* b;
    double *x, *r, *p, *p2, *q, *xw, *rt;
    double* part;                            // 4 kGridWgs partial sums
    double* out;                             // kGridOut* values (host-coherent)
    double* hist;                            // residual norms by iteration (host-coherent)
    const int* singular;
    uint32_t* done;
    uint32_t seq;
    double rtol;
    double window_limit;                     // of the residuals' quotient over a window
    double nr0, nws;                         // resumed solves: the first residual norm, the window's
    int maxit, adaptive, k, any_gamma;
    int start;                               // 0: from x, 1: from zero, 2: resumed from r
    int iters;                               // resumed solves: iterations so far
};

// The index ranges of a level (A, R, P with `rows`, `coarse`, `rows` rows; win
// as above); most[0..2]: the largest of the LDS entries a workgroup needs, of
// the entries of A it reads to form the residual again, of its share's.
void launch_grid_windows(int rows, int coarse, const int32_t* a_rp, const int32_t* a_ci, const int32_t* r_rp,
                         const int32_t* r_ci, const int32_t* p_rp, const int32_t* p_ci, int32_t* win, int32_t* most,
                         hipStream_t st);

// Launches whose workgroups are on the device together whatever the others do: the
// workgroups go round the dies of 32 compute units, so the fullest die counts.  At
// 128 registers and 1,024 threads a unit takes one: six launches on 256 units, one
// on a partition of 64, none on one of 32.
constexpr int grid_launches(int cus, int per_cu) {
    constexpr int kDieCus = 32;
    const int dies = cus > kDieCus ? cus / kDieCus : 1;
    const int share = (kGridWgs + 1 + dies - 1) / dies;
    return cus / dies * per_cu / share;
}
static_assert(grid_launches(256, 1) == 6 && grid_launches(256, 2) == 12 && grid_launches(128, 1) == 3 &&
              grid_launches(64, 1) == 1 && grid_launches(32, 1) == 0 && grid_launches(256, 0) == 0);

// What the current device gives the kernels: dynamic LDS of a launch (bytes) and
// launches at the same time; 0 if it cannot be found out.
struct GridLimits {
    size_t lds = 0;
    int launches = 0;
};
GridLimits grid_limits();

// Levels lv[0..count) and the tail below them: on entry lv[0].b holds the
// right-hand side, on exit lv[0].xt the result of the cycle from zero.  lds: the
// larger of the widest windows and the tail's arrays.
void launch_grid_cycle(const GridArgs<double>& a, size_t lds, hipStream_t st);
void launch_grid_cycle(const GridArgs<float>& a, size_t lds, hipStream_t st);
// PCG with that cycle (FP64, or FP32 values and vectors in the cycle)
void launch_grid_solve(const GridArgs<double>& a, const GridSolve& s, size_t lds, hipStream_t st);
void launch_grid_solve(const GridArgs<float>& a, const GridSolve& s, size_t lds, hipStream_t st);

}  // namespace amg355
