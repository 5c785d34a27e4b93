// Exact sums of products on the device: every inner product of the library is the
// double nearest the exact sum (exact products through fma, compensated
// accumulation, one rounding), so any summation order gives the same double.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace ftk {

// Sums of exact products as an unevaluated pair: hi the running double sum, lo the
// sum of every rounding error (TwoProd and TwoSum), together as accurate as twice
// the working precision.  hi depends on one addition per term, the errors are
// added off that chain, which is what a step's latency is made of.
__device__ __forceinline__ void pair_add(double &hi, double &lo, double bh, double bl)
{
    const double t = hi + bh;
    const double z = t - hi;
    const double e = (hi - (t - z)) + (bh - z);
    hi = t;
    lo = (lo + bl) + e;
}

__device__ __forceinline__ void pair_prod(double &hi, double &lo, double a, double b)
{
    const double p = a * b;
    pair_add(hi, lo, p, fma(a, b, -p));
}

template <int CTRL>
__device__ __forceinline__ double dpp(double x)
{
    union {
        double d;
        int i[2];
    } u;
    u.d = x;
    u.i[0] = __builtin_amdgcn_update_dpp(0, u.i[0], CTRL, 0xf, 0xf, true);
    u.i[1] = __builtin_amdgcn_update_dpp(0, u.i[1], CTRL, 0xf, 0xf, true);
    return u.d;
}

// Pair sum over groups of 2^LEVELS consecutive lanes, the same value in each of
// them: lane ^ 1, lane ^ 2, then mirrors within 8 and 16 lanes (their groups of 4
// and 8 already agree), then the rows of 16 and the halves exchanged.
template <int LEVELS>
__device__ __forceinline__ void lane_sum(double &hi, double &lo)
{
    if (LEVELS > 0) pair_add(hi, lo, dpp<0xB1>(hi), dpp<0xB1>(lo));
    if (LEVELS > 1) pair_add(hi, lo, dpp<0x4E>(hi), dpp<0x4E>(lo));
    if (LEVELS > 2) pair_add(hi, lo, dpp<0x141>(hi), dpp<0x141>(lo));
    if (LEVELS > 3) pair_add(hi, lo, dpp<0x140>(hi), dpp<0x140>(lo));
#pragma unroll
    for (int level = 4; level < LEVELS; ++level) {
        union U {
            double d;
            unsigned i[2];
        } h, l, h2, l2;
        h.d = hi;
        l.d = lo;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // first: rows (halves) 0 0 2 2, second: 1 1 3 3
            const auto a = level == 4 ? __builtin_amdgcn_permlane16_swap(h.i[j], h.i[j], false, false)
                                      : __builtin_amdgcn_permlane32_swap(h.i[j], h.i[j], false, false);
            const auto b = level == 4 ? __builtin_amdgcn_permlane16_swap(l.i[j], l.i[j], false, false)
                                      : __builtin_amdgcn_permlane32_swap(l.i[j], l.i[j], false, false);
            h.i[j] = a[0];
            h2.i[j] = a[1];
            l.i[j] = b[0];
            l2.i[j] = b[1];
        }
        hi = h.d;
        lo = l.d;
        pair_add(hi, lo, h2.d, l2.d);
    }
}

// The launch-invariant data behind p, read through the scalar cache.
template <class T>
__device__ __forceinline__ const T *constant(const T *p)
{
    return (const T *)(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// Barrier over LDS only: global stores (the recorded coefficients) stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int log2c(int x) { return x <= 1 ? 0 : 1 + log2c(x / 2); }

// a value that every lane holds, in scalar registers
__device__ __forceinline__ double uniform(double x)
{
    union {
        double d;
        int i[2];
    } u;
    u.d = x;
    u.i[0] = __builtin_amdgcn_readfirstlane(u.i[0]);
    u.i[1] = __builtin_amdgcn_readfirstlane(u.i[1]);
    return u.d;
}

// Sum over the workgroup, rounded, in every thread; sh holds one pair per wave.
// One barrier, which also ends the phase before it.
template <int T>
__device__ __forceinline__ double block_sum(double hi, double lo, double2 *sh)
{
    lane_sum<6>(hi, lo);
    if (T > 64) {
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_double2(hi, lo);
        lds_barrier();
        const double2 p = sh[threadIdx.x & (T / 64 - 1)];
        hi = p.x;
        lo = p.y;
        lane_sum<log2c(T / 64)>(hi, lo);
    } else {
        lds_barrier();
    }
    return uniform(hi + lo);
}

// Sum over the workgroup of pairs; the same pair in every thread.  One barrier, between
// the waves' writes and the reads: a wave may be past it while another still reads, so two
// sums with no barrier between them need different memory.  A kernel's leading sums (the
// partials of the launch before) and the one that ends it each have their own; a second of
// the same kind needs a barrier before it.
enum SumSlot { kLead, kEnd };
template <int BLOCK, SumSlot SLOT>
__device__ __forceinline__ void block_pair(double &hi, double &lo)
{
    __shared__ double2 sh[BLOCK / 64];
    lane_sum<6>(hi, lo);
    if (BLOCK > 64) {
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_double2(hi, lo);
        __syncthreads();
        const double2 p = sh[threadIdx.x & (BLOCK / 64 - 1)];
        hi = p.x;
        lo = p.y;
        lane_sum<log2c(BLOCK / 64)>(hi, lo);
    }
}

// Sum of nparts (hi, lo) partials, rounded, in every thread of a block.
template <int BLOCK = kBlock>
__device__ __forceinline__ double reduce_partials(const double *partials, int nparts)
{
    double hi = 0.0, lo = 0.0;
    for (int i = threadIdx.x; i < nparts; i += BLOCK) pair_add(hi, lo, partials[2 * i], partials[2 * i + 1]);
    block_pair<BLOCK, kLead>(hi, lo);
    return hi + lo;
}

template <int BLOCK>
__device__ __forceinline__ void write_partial(double *partials, double hi, double lo)
{
    block_pair<BLOCK, kEnd>(hi, lo);
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = hi;
        partials[2 * blockIdx.x + 1] = lo;
    }
}

}  // namespace ftk
