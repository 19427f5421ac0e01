// bmg_check.h -- the convergence test of a cycle, as a device function: it runs
// as a launch of its own (k_finalize_check) or as an extra workgroup of the
// next cycle's first coarse kernel.
#pragma once
#include "bmg_internal.h"

namespace hbmg {

// Sum of the first 256 threads' values (every thread of the workgroup calls):
// a butterfly within each wave, then the four wave sums in turn.  The result is
// thread 0's.
__device__ __forceinline__ double sum256(double acc, double *sh)
{
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0 && threadIdx.x < 256) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    return ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// values to a host-mapped slot, then the tag the host polls for: the fence
// orders the two
__device__ __forceinline__ void slot_write(double *slot, double v0, double v1, double v2, double tag)
{
    volatile double *v = slot;
    v[0] = v0;
    v[1] = v1;
    v[2] = v2;
    __threadfence_system();
    v[3] = tag;
}

// test k's flag; a large streaming leg's tiles may read it on the way
__device__ __forceinline__ void set_flag(const CheckArgs &c, int run)
{
    __hip_atomic_store(c.flags + (c.k & 1), run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// thread 0, with the partials' sum: the test and its outcome
__device__ __forceinline__ void check_sum(const CheckArgs &c, double sum)
{
    const double rel = sqrt(sum) / c.denom[0];
    int run = 1;
    if (!isfinite(rel) || rel <= c.tol) run = 0;
    set_flag(c, run);
    slot_write(c.slot, rel, (double)run, (double)(run ? 0 : c.k), c.tag);
}

// whether an earlier cycle met the test: then so does this one (no slot is written)
__device__ __forceinline__ bool check_over(const CheckArgs &c)
{
    if (c.flags[(c.k - 1) & 1]) return false;
    if (threadIdx.x == 0) set_flag(c, 0);
    return true;
}

// the whole workgroup (at least 256 threads) calls
__device__ __forceinline__ void cycle_check(const CheckArgs &c)
{
    __shared__ double sh[4];
    if (check_over(c)) return;
    double acc = 0.0;
    if (threadIdx.x < 256)
        for (int m = threadIdx.x; m < c.n; m += 256) acc += c.partials[m];
    const double sum = sum256(acc, sh);
    if (threadIdx.x == 0) check_sum(c, sum);
}

// the same bits from one wave: each lane stands for four of the 256 threads
__device__ __forceinline__ void cycle_check_wave(const CheckArgs &c)
{
    if (check_over(c)) return;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int m = threadIdx.x; m < c.n; m += 256)
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[w] += m + 64 * w < c.n ? c.partials[m + 64 * w] : 0.0;
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[w] += __shfl_xor(acc[w], off, 64);
    if (threadIdx.x == 0) check_sum(c, ((acc[0] + acc[1]) + acc[2]) + acc[3]);
}

}  // namespace hbmg
