// Shifted COCG with seed switching: per-sequence state and launchers (cocg.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "exact_sum.h"
#include "kernels.h"

namespace ftk {

// Shifted COCG with seed switching (complex-symmetric Lanczos basis + per-shift
// scalar recurrences; cocg.hip), per sequence.
struct CocgState {
    double invr, invi;  // inv_k = 1/b_k (1/delta_0 at k = 0)
    double ipr, ipi;    // inv_{k-1}
    double bkr, bki;    // b_k (0 at k = 0)
    double akr, aki;    // a_k
    double c2r, c2i;    // -(a_k inv_k)
    double ckr, cki;    // c_k = <chi|q_k>
    double hn, hn0;     // ||q_k||^2, ||q_0||^2
    double d0r, d0i;    // delta_0 = csqrt(chi^T chi)
    double alr, ali;    // seed alpha_{k-1}
    double ber, bei;    // seed beta_{k-1}
    double dr, di;      // seed residual scale delta_k
    double norm2;       // ||chi||^2
    double shift_re;    // real offset of every shift (E_m)
    double max_resid;   // largest residual 2-norm over the shifts after the last step
    int seed;           // index of the seed shift
    int done, steps, numeric_error;
};
struct CocgShift {
    double pr, pi;    // pi_k
    double por, poi;  // pi_{k-1}
    double Pr, Pi;    // <chi|p_{k-1}> of the shift
    double gr, gi;    // <chi|x_k> of the shift
    double res;       // residual 2-norm after the shift's last update (+inf before the first)
};
// A batch of B sequences run in lockstep: sequence r's vectors lie 2 * 2^N doubles after
// sequence r - 1's, its state, shifts and recorded scalars one row further.
struct CocgBatch {
    int B, n;                 // sequences; steps (rows of a and b: n entries, of c: n + 1)
    const double *lam;        // the projection vectors (chi for a spectrum)
    double *Hw;               // work vectors, needed by cocg_work_vectors(op)
    double *pa, *pb;          // partial sums, B * 10 * vec_grid doubles each
    CocgState *st;
    CocgShift *sh;
    const double *omega;
    int n_omega;
    double eta, tol, rtol, seed_tol;
    double *a, *b, *c;        // a_k, b_{k+1}, c_{k+1} (c_0 at the start), complex
};
// H v one element per thread takes the first half step as its epilogue; the other forms
// leave H w in work vectors.
bool cocg_work_vectors(const HvOp &op);
// the first half step in that epilogue (kernels.hip): u over U, partial sums to pa
void launch_hv_cocg(const HvOp &op, const double *Wcur, const double *Wprev, double *U, const CocgState *st,
                    double *pa, int first, int B, hipStream_t s);
// states from the right-hand sides chi and E_m
void launch_cocg_start(uint32_t dim, const double *chi, const CocgBatch &q, const BatchShifts &shift_re, hipStream_t s);
// step k: Wcur = w_{k-1} (chi at k = 0), Wprev = w_{k-2} (chi at k = 1, unused at
// k = 0); U (may be Wprev) receives w_k
void launch_cocg_step(const HvOp &op, const CocgBatch &q, const double *Wcur, const double *Wprev, double *U, int k,
                      hipStream_t s);
// g [B][n_omega]
void launch_cocg_finish(const CocgBatch &q, double *g, hipStream_t s);

#if defined(__HIPCC__)
// complex products of the vector updates: (fma(ar, br, -(ai bi)), fma(ar, bi, ai br))
__device__ __forceinline__ void cmul_v(double ar, double ai, double br, double bi, double &r, double &i)
{
    r = fma(ar, br, -(ai * bi));
    i = fma(ar, bi, ai * br);
}

// up to 5 exact sums per block, (hi, lo) pairs in partials[(block * 5 + j) * 2]
template <int NS>
__device__ __forceinline__ void write_partials5(double *partials, Sum (&sum)[NS])
{
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        block_total<kBlock, kEnd>(sum[j]);
        const double l = sum[j].low();
        if (threadIdx.x == 0) {
            partials[(blockIdx.x * 5 + j) * 2] = sum[j].hi;
            partials[(blockIdx.x * 5 + j) * 2 + 1] = l;
        }
        __syncthreads();
    }
}

template <int NS>
__device__ __forceinline__ void normalise(Sum (&sum)[NS])
{
#pragma unroll
    for (int j = 0; j < NS; ++j) sum[j].normalise();
}

// u = (H w_{k-1}) inv_k + c1 w_{k-2}, one element; its part of the sums of w_{k-1}^T u
struct CocgA {
    double ir, ii, c1r, c1i;
    Sum sum[2];
    __device__ __forceinline__ void init(const CocgState *st)
    {
        ir = st->invr, ii = st->invi;
        cmul_v(st->bkr, st->bki, st->ipr, st->ipi, c1r, c1i);
        c1r = -c1r;
        c1i = -c1i;
    }
    __device__ __forceinline__ double2 operator()(double hr, double him, const double2 &wc, const double2 &wp, int first)
    {
        double tr, ti;
        cmul_v(hr, him, ir, ii, tr, ti);
        double ur = tr, ui = ti;
        if (!first) {
            ur = fma(c1r, wp.x, fma(-c1i, wp.y, tr));
            ui = fma(c1r, wp.y, fma(c1i, wp.x, ti));
        }
        sum[0].product(wc.x, ur);
        sum[0].product(-wc.y, ui);
        sum[1].product(wc.x, ui);
        sum[1].product(wc.y, ur);
        return make_double2(ur, ui);
    }
};
#endif

}  // namespace ftk
