// The per-shift recurrence of a Green's-function sequence, shared by the kernels that run it.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace ftk {

// One step of the forward LDL^T recurrence of (z - T)^{-1}_{00} for the shift z = zr + i zi
// (App. A.3): d_k, the running product p_k and the accumulated G; alpha = alpha_k,
// bk = beta_k.
__device__ __forceinline__ void shift_update(ShiftState &q, double zr, double zi, double alpha, double bk, int k)
{
    if (k == 0) {
        q.dr = zr - alpha;
        q.di = zi;
        q.pr = 1.0;
        q.pi = 0.0;
        const double den = q.dr * q.dr + q.di * q.di;
        q.gr = q.dr / den;
        q.gi = -q.di / den;
    } else {
        const double den = q.dr * q.dr + q.di * q.di;
        const double rr = q.dr / den, ri = -q.di / den;  // 1/d_{k-1}
        const double fr = bk * rr, fi = bk * ri;         // beta_k / d_{k-1}
        const double pr = q.pr * fr - q.pi * fi;
        const double pi = q.pr * fi + q.pi * fr;
        const double b2 = bk * bk;
        q.dr = (zr - alpha) - b2 * rr;
        q.di = zi - b2 * ri;
        q.pr = pr;
        q.pi = pi;
        const double p2r = pr * pr - pi * pi, p2i = 2.0 * pr * pi;
        const double dn = q.dr * q.dr + q.di * q.di;
        q.gr = q.gr + (p2r * q.dr + p2i * q.di) / dn;
        q.gi = q.gi + (p2i * q.dr - p2r * q.di) / dn;
    }
}

// Galerkin residual of a shift after a step, per unit right-hand side: |p_k| beta_{k+1} / |d_k|
__device__ __forceinline__ double shift_residual(const ShiftState &q, double bn)
{
    return sqrt((q.pr * q.pr + q.pi * q.pi) / (q.dr * q.dr + q.di * q.di)) * bn;
}

// maximum over a block of BLOCK threads; valid in thread 0
template <int BLOCK>
__device__ __forceinline__ double block_max(double v)
{
    __shared__ double sh[BLOCK / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double m = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < BLOCK / 64; ++i) m = sh[i] > m ? sh[i] : m;
    return m;
}

}  // namespace ftk
