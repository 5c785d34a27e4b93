// Exact sums of products on the device: every inner product of the library is the
// double nearest the exact sum (exact products through fma, compensated
// accumulation, one rounding), so any summation order gives the same double.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace ftk {

// A sum of exact products: hi the running double sum, lo the sum of what its additions
// rounded off (Knuth's TwoSum), er the sum of what the products did (TwoProd through fma).
// hi depends on one addition per term, the rest is added off that chain, which is what a
// step's latency is made of.  What additions round off are multiples of the terms' last
// places, so lo is exact over terms of like size; the products' errors, which have bits
// far below, would round it at every term and so have a sum of their own.  Error (rms) of
// the whole sum against double-double with a normalisation per term and as its tree's additions,
// on host models of the kernels' shapes over random vectors: 0.4 to 1.0 times (with both errors
// in one sum, never normalised: 1.2 to 1.5 times at 6 to 20 sites, 5 at 24, 50 at 30; that
// is faster by 1 to 2 % at 8 and 12 sites and by 3 % for COCG's five sums).
struct Sum {
    double hi = 0.0, lo = 0.0, er = 0.0;

    __device__ __forceinline__ double two_sum(double b)
    {
        const double t = hi + b;
        const double z = t - hi;
        const double e = (hi - (t - z)) + (b - z);
        hi = t;
        return e;
    }
    // + a b
    __device__ __forceinline__ void product(double a, double b)
    {
        const double p = a * b;
        er = er + fma(a, b, -p);
        lo = lo + two_sum(p);
    }
    // + a pair that was read back (its lo has bits as far below as a product's error)
    __device__ __forceinline__ void pair(double h, double l)
    {
        er = er + l;
        lo = lo + two_sum(h);
    }
    __device__ __forceinline__ void add(double h, double l, double r)
    {
        er = er + r;
        lo = (lo + l) + two_sum(h);
    }
    // lo within half a unit of hi's last place (Dekker's FastTwoSum); a long sum does this
    // every few terms, so that lo's own additions stay exact
    __device__ __forceinline__ void normalise()
    {
        const double t = hi + lo;
        lo = lo - (t - hi);
        hi = t;
    }
    // the sum as a pair: hi and this
    __device__ __forceinline__ double low()
    {
        normalise();
        return lo + er;
    }
    __device__ __forceinline__ double rounded()
    {
        const double l = low();
        return hi + l;
    }
};

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

// A thread that takes an element a turn normalises its sums after every eighth: turn counts
// them from 0.
__device__ __forceinline__ bool settles(int turn) { return (turn & 7) == 7; }

// Sum over groups of 2^LEVELS consecutive lanes, the same value in each of
// them: lane ^ 1, lane ^ 2, then mirrors within 8 and 16 lanes (their groups of 4
// and 8 already agree), then the rows of 16 and the halves exchanged.
template <int CTRL>
__device__ __forceinline__ void lane_add(Sum &s)
{
    s.add(dpp<CTRL>(s.hi), dpp<CTRL>(s.lo), dpp<CTRL>(s.er));
}
// rows (LEVEL 4) or halves (5) of x exchanged: first 0 0 2 2, second 1 1 3 3
template <int LEVEL>
__device__ __forceinline__ double swap_rows(double &x)
{
    union U {
        double d;
        unsigned i[2];
    } a, b;
    a.d = x;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const auto r = LEVEL == 4 ? __builtin_amdgcn_permlane16_swap(a.i[j], a.i[j], false, false)
                                  : __builtin_amdgcn_permlane32_swap(a.i[j], a.i[j], false, false);
        a.i[j] = r[0];
        b.i[j] = r[1];
    }
    x = a.d;
    return b.d;
}
template <int LEVEL>
__device__ __forceinline__ void row_add(Sum &s)
{
    const double h = swap_rows<LEVEL>(s.hi), l = swap_rows<LEVEL>(s.lo), r = swap_rows<LEVEL>(s.er);
    s.add(h, l, r);
}
template <int LEVELS>
__device__ __forceinline__ void lane_sum(Sum &s)
{
    if (LEVELS > 0) lane_add<0xB1>(s);
    if (LEVELS > 1) lane_add<0x4E>(s);
    if (LEVELS > 2) lane_add<0x141>(s);
    if (LEVELS > 3) lane_add<0x140>(s);
    if (LEVELS > 4) row_add<4>(s);
    if (LEVELS > 5) row_add<5>(s);
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

// The workgroup's sum in every thread, by way of sh (a pair per wave; three numbers are no
// faster) and a barrier.
template <int T, class Barrier>
__device__ __forceinline__ void wave_sums(Sum &s, double2 *sh, Barrier &&barrier)
{
    s.normalise();
    lane_sum<6>(s);
    if (T > 64) {
        const double l = s.low();
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_double2(s.hi, l);
        barrier();
        const double2 p = sh[threadIdx.x & (T / 64 - 1)];
        s = Sum{p.x, 0.0, p.y};
        lane_sum<log2c(T / 64)>(s);
    }
}

// Sum over the workgroup, rounded, in every thread; sh holds one pair per wave.
// One barrier, which also ends the phase before it.
template <int T>
__device__ __forceinline__ double block_sum(Sum s, double2 *sh)
{
    wave_sums<T>(s, sh, lds_barrier);
    if (T == 64) lds_barrier();
    return uniform(s.rounded());
}

// Sum over the workgroup; the same in every thread.  One barrier, between
// the waves' writes and the reads: a wave may be past it while another still reads, so two
// sums with no barrier between them need different memory.  A kernel's leading sums (the
// partials of the launch before) and the one that ends it each have their own; a second of
// the same kind needs a barrier before it.
enum SumSlot { kLead, kEnd };
template <int BLOCK, SumSlot SLOT>
__device__ __forceinline__ void block_total(Sum &s)
{
    __shared__ double2 sh[BLOCK / 64];
    wave_sums<BLOCK>(s, sh, [] { __syncthreads(); });
}

// Sum of nparts (hi, lo) partials, rounded, in every thread of a block.
template <int BLOCK = kBlock>
__device__ __forceinline__ double reduce_partials(const double *partials, int nparts)
{
    Sum s;
    for (int i = threadIdx.x; i < nparts; i += BLOCK) s.pair(partials[2 * i], partials[2 * i + 1]);
    block_total<BLOCK, kLead>(s);
    return s.rounded();
}

template <int BLOCK>
__device__ __forceinline__ void write_partial(double *partials, Sum s)
{
    block_total<BLOCK, kEnd>(s);
    const double l = s.low();
    if (threadIdx.x == 0) {
        partials[2 * blockIdx.x] = s.hi;
        partials[2 * blockIdx.x + 1] = l;
    }
}

}  // namespace ftk
