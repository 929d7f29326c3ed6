// What the row kernels of several files share (gfx950, wave64): the block
// order over the dies and the reduction of a workgroup's dot product.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace amg355 {
namespace {

constexpr int kBlock = 256;
constexpr int kXcds = 8;            // MI355X: 8 accelerator complex dies, each with its own L2

// Workgroups are handed to the XCDs round-robin.  Remap so that XCD x works on
// a contiguous range of logical blocks: neighbouring rows gather neighbouring
// entries of x, which then stay in one L2.  The grid is a multiple of 8.
__device__ __forceinline__ int xcd_logical_block() {
    const int per = gridDim.x / kXcds;
    return (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
}

inline int round_up8(int b) { return (b + kXcds - 1) / kXcds * kXcds; }

// Block-wide sum of v; the total is valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double* lds) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int wid = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) lds[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) {
        t = lds[0];
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) t += lds[w];
    }
    __syncthreads();
    return t;
}

// Deterministic grid reduction, first pass: every block stores its partial
// sum; dot_finish_kernel adds the partials in a fixed order.  (A single-pass
// last-block scheme would need an agent-scope release fence per block, which
// on gfx950 writes back the XCD's L2 and stalls the block.)
__device__ __forceinline__ void store_block_partial(double v, double* partials, int lb) {
    __shared__ double lds[kBlock / 64];
    const double t = block_sum(v, lds);
    if (threadIdx.x == 0) partials[lb] = t;
}

// Values for the host, then the flag it polls: stores of system scope go to
// memory themselves, so the flag waits for them alone and no cache is written
// back (a release fence here cost 3 us).  Every thread calls host_flag.
template <class T>
__device__ __forceinline__ void host_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void host_flag(uint32_t* flag, uint32_t seq) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) host_store(flag, seq);
}

}  // namespace
}  // namespace amg355
