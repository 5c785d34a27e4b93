// Krylov sequences of small clusters (2^6 .. 2^12 states): one workgroup runs one
// sequence from its start vector to its last step.  Compiled with
// -ffp-contract=off; the operations per element are those of the per-step kernels
// (kernels.hip), and every inner product is the double nearest the exact sum, so
// the coefficients are theirs bit for bit.
//
// Why: a step of such a vector is a few microseconds of work, less than the four
// launches it took, and the per-step kernels of 16 sequences filled 16 to 128 of
// the 1024 SIMDs.  Here the step's two reductions are two workgroup barriers,
// nothing but the coefficients leaves the compute unit, and all sequences of a
// call run side by side.
#include <hip/hip_runtime.h>

#include "resident.h"
#include "shift_update.h"
#include "spin_ops.h"

namespace ftk {

// ---------------------------------------------------------------------------
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

// Barrier over LDS only: global stores (the recorded coefficients) stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

constexpr int log2c(int x) { return x <= 1 ? 0 : 1 + log2c(x / 2); }

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
    return hi + lo;
}

// the start vectors of the sequences, 2^N entries each
__global__ void __launch_bounds__(kBlock) k_start_vectors(int n_sites, int load, ResidentRun R, double2 *__restrict__ chi)
{
    const uint32_t x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= 1u << n_sites) return;
    const ResidentSeq q = R.seq[blockIdx.y];
    double2 *out = chi + ((size_t)blockIdx.y << n_sites);
    if (load == kLoadSpin) {
        const SqParams &P = R.sq[q.op];
        out[x] = sq_part(n_sites, P.alpha, P.h, q.phi, x);
    } else {
        const SpinOpParams &A = R.a[q.op >> 2], &B = R.b[q.op >> 2];
        out[x] = polarize_part(q.op & 3, spin_op_part(n_sites, A.h, q.phi, x), spin_op_part(n_sites, B.h, q.phi, x));
    }
}

// A bond for one thread: its amplitudes for the elements whose register bits it
// flips with even and odd parity, and the register bits it flips.
struct BondAt {
    double even, odd;
    uint32_t mr;
};

// One fma per element; a bond that flips no register bit takes one amplitude for all.
template <int E>
__device__ __forceinline__ void accumulate(double (&re)[E], double (&im)[E], const double2 (&v)[E], BondAt at)
{
    const double even = at.even, odd = at.odd;
    if (at.mr == 0) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            re[e] = fma(even, v[e].x, re[e]);
            im[e] = fma(even, v[e].y, im[e]);
        }
    } else {
        uint32_t sel = 0;  // bit e: element e takes the odd amplitude
        if (at.mr & 1u) sel ^= 0xAAu;
        if (at.mr & 2u) sel ^= 0xCCu;
        if (at.mr & 4u) sel ^= 0xF0u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double a = ((sel >> e) & 1u) ? odd : even;
            re[e] = fma(a, v[e].x, re[e]);
            im[e] = fma(a, v[e].y, im[e]);
        }
    }
}

// Element e of a thread is state tid + e T: the register bits are the highest
// sites.  The current vector w_{k-1} is in LDS (partners) and in registers (own
// elements) with w_{k-2}; bond constants sit one bond per lane and are read into
// scalar registers, so the bond loop waits for LDS data only.  Its LDS reads
// (16 B per element and bond at 128 B per clock) bound the larger sizes, the two
// reductions' latency the smaller ones.
template <int LOGT, int E>
__global__ void __launch_bounds__(1 << LOGT) k_resident(HvParams P, ResidentRun R)
{
    constexpr int T = 1 << LOGT;
    constexpr uint32_t dim = T * E;
    __shared__ double2 tile[dim];
    __shared__ double2 sh_a[T / 64], sh_b[T / 64];
    const ResidentSeq q = R.seq[blockIdx.x];
    const uint32_t tid = threadIdx.x;
    SeqState *st = R.st + q.out;
    double *alpha = R.alpha + (size_t)q.out * R.stride, *beta = R.beta + (size_t)q.out * R.stride;
    const int nb = P.n_bonds;
    const int bl = (int)(tid & 63) < nb ? (int)(tid & 63) : 0;
    const int c_code = (int)P.code[bl];
    const double ap0 = P.ap3[0], ap1 = P.ap3[1], ap2 = P.ap3[2];
    const double aa0 = P.aa3[0], aa1 = P.aa3[1], aa2 = P.aa3[2];

    // bond parities of the thread's element 0 and the diagonal of its elements
    uint64_t par64 = 0;
#pragma unroll
    for (int l = 0; l < LOGT; ++l)
        if ((tid >> l) & 1u) par64 ^= P.smask[l];
    const uint32_t par_lo = (uint32_t)par64, par_hi = (uint32_t)(par64 >> 32);
    const int nz = __popcll(P.zmask);
    double D[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        uint64_t pe = par64;
        if (e & 1) pe ^= P.smask[LOGT];
        if (e & 2) pe ^= P.smask[LOGT + 1];
        if (e & 4) pe ^= P.smask[LOGT + 2];
        const int s_all = nb - 2 * __popcll(pe);
        const int s_z = nz - 2 * __popcll(pe & P.zmask);
        D[e] = fma(P.kq, (double)s_z, P.jq * (double)s_all);
    }

    double2 wc[E], wp[E];
    double inv, inv_prev, bcur;
    double *carry = R.carry ? R.carry + (size_t)blockIdx.x * 4 * dim : nullptr;
    int bad;  // 1 + the first step after which a scalar was not finite (1: the start), 0 none
    if (R.k0 == 0) {
        const double2 *start = R.chi ? (const double2 *)R.chi + (size_t)blockIdx.x * dim : q.phi;
        double hi = 0.0, lo = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t x = tid + e * T;
            wc[e] = start[x];
            wp[e] = make_double2(0.0, 0.0);
            tile[x] = wc[e];
            pair_prod(hi, lo, wc[e].x, wc[e].x);
            pair_prod(hi, lo, wc[e].y, wc[e].y);
        }
        const double s = block_sum<T>(hi, lo, sh_b);
        const double nrm = sqrt(s);
        inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
        inv_prev = 0.0;
        bcur = 0.0;
        bad = isfinite(s) ? 0 : 1;
        if (tid == 0) {
            st->norm2 = s;
            st->norm = nrm;
            st->inv_cur = inv;
            st->inv_prev = 0.0;
            st->beta_cur = 0.0;
            st->alpha_cur = 0.0;
            st->shift_re = q.shift_re;
            st->max_resid = 0.0;
            st->done = nrm > 0.0 ? 0 : 1;
            st->steps = 0;
            st->numeric_error = bad;
            st->pad = bad;
        }
        if (!(nrm > 0.0)) return;
    } else {
        if (st->done) return;
        inv = st->inv_cur;
        inv_prev = st->inv_prev;
        bcur = st->beta_cur;
        bad = st->pad;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t x = tid + e * T;
            wc[e] = ((const double2 *)carry)[x];
            wp[e] = ((const double2 *)carry)[dim + x];
            tile[x] = wc[e];
        }
        lds_barrier();
    }

    // bond b and its partners of the thread's elements
    auto bond = [&](int b, double2 (&v)[E]) {
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane(c_code, b);
        const uint32_t m = c & 0x3fffffffu, type = c >> 30;
        const double p0 = ap0, p1 = ap1, p2 = ap2, q0 = aa0, q1 = aa1, q2 = aa2;
        const double ap = type == 0 ? p0 : type == 1 ? p1 : p2;
        const double aa = type == 0 ? q0 : type == 1 ? q1 : q2;
        const bool anti = ((b < 32 ? par_lo : par_hi) & (1u << (b & 31))) != 0;
        const BondAt at{anti ? aa : ap, anti ? ap : aa, m >> LOGT};
        const double2 *src = tile + (tid ^ (m & (T - 1)));
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = src[((uint32_t)e ^ at.mr) << LOGT];
        return at;
    };

    double2 *vout = R.vout ? (double2 *)(R.vout + (size_t)blockIdx.x * R.vstride) : nullptr;
    int k = R.k0, done = 0;
    double a = 0.0;
    for (; k < R.k1 && !done; ++k) {
        double re[E], im[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            re[e] = D[e] * wc[e].x;
            im[e] = D[e] * wc[e].y;
        }
        int b = 0;
        for (; b + 1 < nb; b += 2) {  // two bonds' reads in flight, their fmas in list order
            double2 v0[E], v1[E];
            const BondAt b0 = bond(b, v0), b1 = bond(b + 1, v1);
            accumulate<E>(re, im, v0, b0);
            accumulate<E>(re, im, v1, b1);
        }
        if (b < nb) {
            double2 v0[E];
            const BondAt b0 = bond(b, v0);
            accumulate<E>(re, im, v0, b0);
        }
        // u = (H w_{k-1}) inv + c1 w_{k-2}; alpha_k
        const double c1 = (-bcur) * inv_prev;
        double hi = 0.0, lo = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            double ur = re[e] * inv, ui = im[e] * inv;
            if (k > 0) {
                ur = fma(c1, wp[e].x, ur);
                ui = fma(c1, wp[e].y, ui);
            }
            re[e] = ur;
            im[e] = ui;
            pair_prod(hi, lo, wc[e].x, ur);
            pair_prod(hi, lo, wc[e].y, ui);
        }
        if (vout) {
#pragma unroll
            for (int e = 0; e < E; ++e) vout[(size_t)(k - R.k0) * dim + tid + e * T] = wc[e];
        }
        a = inv * block_sum<T>(hi, lo, sh_a);  // the barrier ends the reads of the tile
        // w_k = u + c2 w_{k-1}; beta_{k+1}
        const double c2 = -(a * inv);
        hi = lo = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double wr = fma(c2, wc[e].x, re[e]);
            const double wi = fma(c2, wc[e].y, im[e]);
            tile[tid + e * T] = make_double2(wr, wi);
            pair_prod(hi, lo, wr, wr);
            pair_prod(hi, lo, wi, wi);
            wp[e] = wc[e];
            wc[e] = make_double2(wr, wi);
        }
        const double bn = sqrt(block_sum<T>(hi, lo, sh_b));
        if (tid == 0) {
            alpha[k] = a;
            beta[k] = bn;
        }
        if (bad == 0 && !(isfinite(a) && isfinite(bn))) bad = k + 2;
        if (!(bn > R.tol)) {
            done = 1;  // invariant subspace
        } else {
            inv_prev = inv;
            inv = 1.0 / bn;
            bcur = bn;
        }
    }
    if (tid == 0) {
        st->inv_cur = inv;
        st->inv_prev = inv_prev;
        st->beta_cur = bcur;
        st->alpha_cur = a;
        st->done = done;
        st->steps = k;
        st->numeric_error = bad != 0;
        st->pad = bad;
    }
    if (carry && !done) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t x = tid + e * T;
            ((double2 *)carry)[x] = wc[e];
            ((double2 *)carry)[dim + x] = wp[e];
        }
    }
}

template <int LOGT, int E>
static void launch_resident_t(const HvParams &P, const ResidentRun &run, int n_seq, hipStream_t s)
{
    hipLaunchKernelGGL((k_resident<LOGT, E>), dim3(n_seq), dim3(1 << LOGT), 0, s, P, run);
}

void launch_start_vectors(int n_sites, ResidentLoad load, const ResidentRun &run, int n_seq, hipStream_t s)
{
    if (n_seq <= 0) return;
    hipLaunchKernelGGL(k_start_vectors, dim3(((1u << n_sites) + kBlock - 1) / kBlock, n_seq), dim3(kBlock), 0, s, n_sites,
                       (int)load, run, (double2 *)run.chi);
}

bool resident(const HvOp &op)
{
    return forced_hv_mode() < 0 && op.P.n_sites >= kResidentMinSites && op.P.n_sites <= kResidentMaxSites;
}

void launch_resident(const HvOp &op, const ResidentRun &run, int n_seq, hipStream_t s)
{
    if (n_seq <= 0) return;
    switch (op.P.n_sites) {
    // 256 threads with one element each hide more latency than 64 with four (8 sites,
    // 192 sequences of 64 steps: 0.35 against 0.40 ms a call); at 12 sites 512 threads
    // with eight elements share the bonds' scalar work and the reductions among fewer
    // waves than 1024 with four (48 sequences of 300 steps: 3.00 against 3.24 ms)
    case 6: launch_resident_t<6, 1>(op.P, run, n_seq, s); break;
    case 7: launch_resident_t<7, 1>(op.P, run, n_seq, s); break;
    case 8: launch_resident_t<8, 1>(op.P, run, n_seq, s); break;
    case 9: launch_resident_t<8, 2>(op.P, run, n_seq, s); break;
    case 10: launch_resident_t<8, 4>(op.P, run, n_seq, s); break;
    case 11: launch_resident_t<9, 4>(op.P, run, n_seq, s); break;
    case 12: launch_resident_t<9, 8>(op.P, run, n_seq, s); break;
    default: break;
    }
}

// ---------------------------------------------------------------------------
// The multi-shift update needs nothing but a sequence's coefficients, so it runs
// once per sequence with a thread per shift (state in registers, coefficients
// staged in LDS) instead of once per step.
constexpr int kShiftThreads = 128;
constexpr int kShiftStage = 256;  // coefficients staged at a time

__global__ void __launch_bounds__(kShiftThreads) k_shifts(ShiftRun R)
{
    __shared__ double2 ab[kShiftStage];
    const size_t r = blockIdx.y;
    SeqState *st = R.st + r;
    const double *al = R.alpha + r * R.stride, *be = R.beta + r * R.stride;
    const int n = st->steps;
    const int j = blockIdx.x * kShiftThreads + threadIdx.x;
    const bool live = j < R.n_omega;
    const double zr = (live ? R.omega[j] : 0.0) + st->shift_re, zi = R.eta;
    ShiftState q = {};
    for (int k0 = 0; k0 < n; k0 += kShiftStage) {
        const int cnt = n - k0 < kShiftStage ? n - k0 : kShiftStage;
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += kShiftThreads)
            ab[i] = make_double2(al[k0 + i], k0 + i > 0 ? be[k0 + i - 1] : 0.0);
        __syncthreads();
        for (int i = 0; i < cnt; ++i) shift_update(q, zr, zi, ab[i].x, ab[i].y, k0 + i);
    }
    double rs = 0.0;
    if (n > 0 && live) {
        const double v = shift_residual(q, be[n - 1]);
        rs = v > 0.0 ? v : 0.0;
    }
    if (live) {
        const double n2 = st->norm2;
        double2 *g = (double2 *)R.g + r * R.n_omega;
        g[j] = n > 0 ? make_double2(n2 * q.gr, n2 * q.gi) : make_double2(0.0, 0.0);
    }
    const double m = block_max<kShiftThreads>(rs);
    // residuals are not negative, so their bit patterns order as they do
    if (threadIdx.x == 0 && n > 0)
        atomicMax((unsigned long long *)&st->max_resid, (unsigned long long)__double_as_longlong(m * st->norm));
}

void launch_shifts(const ShiftRun &run, int n_seq, hipStream_t s)
{
    if (n_seq <= 0) return;
    hipLaunchKernelGGL(k_shifts, dim3((run.n_omega + kShiftThreads - 1) / kShiftThreads, n_seq), dim3(kShiftThreads), 0,
                       s, run);
}

// With a residual test per step the sequence's shifts share one workgroup.
constexpr int kUntilThreads = 512;
__global__ void __launch_bounds__(kUntilThreads) k_shifts_until(ShiftRun R, int k0, int k1, double rtol, ShiftState *sh)
{
    __shared__ double s_max;
    const size_t r = blockIdx.x;
    SeqState *st = R.st + r;
    const double *al = R.alpha + r * R.stride, *be = R.beta + r * R.stride;
    double2 *g = (double2 *)R.g + r * R.n_omega;
    sh += r * R.n_omega;
    const int n = st->steps;
    const double n2 = st->norm2, off = st->shift_re;
    if (k0 == 0 && n == 0)  // an empty start vector
        for (int j = threadIdx.x; j < R.n_omega; j += kUntilThreads) g[j] = make_double2(0.0, 0.0);
    int k = k0;
    double m = 0.0;
    bool stop = false;
    for (; k < k1 && k < n && !stop; ++k) {
        const double a = al[k], b = k > 0 ? be[k - 1] : 0.0, bn = be[k];
        double rmax = 0.0;
        for (int j = threadIdx.x; j < R.n_omega; j += kUntilThreads) {
            ShiftState q = k > 0 ? sh[j] : ShiftState{};
            shift_update(q, R.omega[j] + off, R.eta, a, b, k);
            sh[j] = q;
            g[j] = make_double2(n2 * q.gr, n2 * q.gi);
            const double rs = shift_residual(q, bn);
            rmax = rs > rmax ? rs : rmax;
        }
        m = block_max<kUntilThreads>(rmax);
        if (threadIdx.x == 0) s_max = m;
        __syncthreads();
        m = s_max;
        stop = m <= rtol;
    }
    if (threadIdx.x == 0 && k > k0) {
        st->max_resid = m * st->norm;
        if (stop) {
            st->done = 1;
            st->steps = k;
            st->numeric_error = st->pad != 0 && st->pad <= k + 1;  // none after the last step
        }
    }
}

void launch_shifts_until(const ShiftRun &run, int k0, int k1, double rtol, ShiftState *sh, int n_seq, hipStream_t s)
{
    if (n_seq <= 0) return;
    hipLaunchKernelGGL(k_shifts_until, dim3(n_seq), dim3(kUntilThreads), 0, s, run, k0, k1, rtol, sh);
}

}  // namespace ftk
