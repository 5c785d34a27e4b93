// Krylov sequences of small clusters (2^6 .. 2^14 states): one workgroup runs one
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

#include "bond_ops.h"
#include "device_checks.h"
#include "exact_sum.h"
#include "resident.h"
#include "shift_update.h"
#include "spin_ops.h"

namespace ftk {

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

// The sequence's state after its start vector and after the steps of a launch; pad
// keeps 1 + the first step after which a scalar was not finite (1: the start).
__device__ __forceinline__ void start_state(SeqState *st, double norm2, double norm, double inv, double shift_re, int bad)
{
    st->norm2 = norm2;
    st->norm = norm;
    st->inv_cur = inv;
    st->inv_prev = 0.0;
    st->beta_cur = 0.0;
    st->alpha_cur = 0.0;
    st->shift_re = shift_re;
    st->max_resid = 0.0;
    st->done = norm > 0.0 ? 0 : 1;
    st->steps = 0;
    st->numeric_error = bad;
    st->pad = bad;
}
__device__ __forceinline__ void end_state(SeqState *st, double inv, double inv_prev, double bcur, double a, int done,
                                          int steps, int bad)
{
    st->inv_cur = inv;
    st->inv_prev = inv_prev;
    st->beta_cur = bcur;
    st->alpha_cur = a;
    st->done = done;
    st->steps = steps;
    st->numeric_error = bad != 0;
    st->pad = bad;
}

// Bit e: element e of a thread takes a bond's odd amplitude.  One code path for every
// bond: a branch on the register bits costs more in copies of the sums, which the two
// sides keep in different registers, than the selects it saves.
__device__ __forceinline__ uint32_t odd_elements(uint32_t mr)
{
    uint32_t sel = 0;
    if (mr & 1u) sel ^= 0xAAAAu;
    if (mr & 2u) sel ^= 0xCCCCu;
    if (mr & 4u) sel ^= 0xF0F0u;
    if (mr & 8u) sel ^= 0xFF00u;
    return sel;
}

// Element e of a thread is state tid + e T: the register bits are the highest
// sites.  The current vector w_{k-1} is in LDS (partners) and in registers (own
// elements) with w_{k-2}; bond constants sit one bond per lane and are read into
// scalar registers, so the bond loop waits for LDS data only.  fp64 issue bounds the
// larger sizes, the latency of the two reductions the smaller ones: a step of 48
// sequences takes 2.7 us at 8 sites, 4.0 at 10 and 8.4 at 12 (before: 17.5 ms for 192
// sequences of 64 steps at 8 sites, now 0.34; 28.0 ms for 48 of 300 at 12, now 2.82).
template <int LOGT, int E>
__global__ void __launch_bounds__(1 << LOGT) k_resident(HvParams P, ResidentRun R)
{
    constexpr int T = 1 << LOGT;
    constexpr uint32_t dim = T * E;
    __shared__ double2 tile[dim];
    __shared__ double2 sh_a[T / 64], sh_b[T / 64];
    // eight elements: the real and the imaginary parts apart, as bond16 reads them
    constexpr bool kPlanar = E == 8;
    auto put = [&](uint32_t x, double2 w) {
        if constexpr (kPlanar) {
            ((double *)tile)[x] = w.x;
            ((double *)tile)[dim + x] = w.y;
        } else {
            tile[x] = w;
        }
    };
    const uint32_t tile_at = lds_address(tile);
    const ResidentSeq q = R.seq[blockIdx.x];
    const uint32_t tid = FTK_IDX(threadIdx.x, (E - 1) * T, dim, 14);
    SeqState *st = R.st + q.out;
    double *alpha = R.alpha + (size_t)q.out * R.stride, *beta = R.beta + (size_t)q.out * R.stride;
    const int nb = P.n_bonds;
    // bond parities of the thread's element 0 and the diagonal of its elements
    uint64_t par64 = 0;
#pragma unroll
    for (int l = 0; l < LOGT; ++l)
        if ((tid >> l) & 1u) par64 ^= P.smask[l];
    const Bonds bonds(P, P.code, nb, par64);
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
        Sum sum;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t x = tid + e * T;
            wc[e] = start[x];
            wp[e] = make_double2(0.0, 0.0);
            put(x, wc[e]);
            sum.product(wc[e].x, wc[e].x);
            sum.product(wc[e].y, wc[e].y);
        }
        const double s = block_sum<T>(sum, sh_b);
        const double nrm = sqrt(s);
        inv = uniform(nrm > 0.0 ? 1.0 / nrm : 0.0);
        inv_prev = 0.0;
        bcur = 0.0;
        bad = isfinite(s) ? 0 : 1;
        if (tid == 0) start_state(st, s, nrm, inv, q.shift_re, bad);
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
            put(x, wc[e]);
        }
        lds_barrier();
    }

    double2 *vout = R.vout ? (double2 *)(R.vout + (size_t)blockIdx.x * R.vstride) : nullptr;
    int k = R.k0, done = 0;
    double a = 0.0;
    for (; k < R.k1 && !done; ++k) {
        double acc[2 * E];  // the real parts, then the imaginary ones
#pragma unroll
        for (int e = 0; e < E; ++e) {
            acc[e] = D[e] * wc[e].x;
            acc[E + e] = D[e] * wc[e].y;
        }
        if constexpr (kPlanar) {
            for (int b = 0; b < nb; ++b) {
                const BondAt c = bonds.at(b);
                const uint32_t t0 = tile_at + FTK_IDX(tid ^ (c.m & (T - 1)), (E - 1) * T, dim, 15) * 8;
                bond16<T * 8>(acc, t0, t0 + 8 * dim, c.m >> LOGT, c.even, c.odd);
            }
        } else {
            auto partners = [&](uint32_t m, double2 (&v)[E]) {
#pragma unroll
                for (int e = 0; e < E; ++e) v[e] = tile[FTK_IDX((tid ^ m) ^ (uint32_t)(e * T), 0, dim, 15)];
            };
            auto add = [&](const BondAt &c, const double2 (&v)[E]) {
                const double even = c.even, odd = c.odd;
                const uint32_t sel = odd_elements(c.m >> LOGT);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const double amp = ((sel >> e) & 1u) ? odd : even;
                    acc[e] = fma(amp, v[e].x, acc[e]);
                    acc[E + e] = fma(amp, v[e].y, acc[E + e]);
                }
            };
            int b = 0;
            for (; b + 1 < nb; b += 2) {  // two bonds' reads in flight, their fmas in list order
                const BondAt c0 = bonds.at(b), c1 = bonds.at(b + 1);
                double2 v0[E], v1[E];
                partners(c0.m, v0);
                partners(c1.m, v1);
                add(c0, v0);
                add(c1, v1);
            }
            if (b < nb) {
                const BondAt c0 = bonds.at(b);
                double2 v0[E];
                partners(c0.m, v0);
                add(c0, v0);
            }
        }
        // u = (H w_{k-1}) inv + c1 w_{k-2}; alpha_k
        const double c1 = uniform((-bcur) * inv_prev);
        Sum sum;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            double ur = acc[e] * inv, ui = acc[E + e] * inv;
            if (k > 0) {
                ur = fma(c1, wp[e].x, ur);
                ui = fma(c1, wp[e].y, ui);
            }
            acc[e] = ur;
            acc[E + e] = ui;
            sum.product(wc[e].x, ur);
            sum.product(wc[e].y, ui);
        }
        if (vout) {
#pragma unroll
            for (int e = 0; e < E; ++e) vout[(size_t)(k - R.k0) * dim + tid + e * T] = wc[e];
        }
        a = uniform(inv * block_sum<T>(sum, sh_a));  // the barrier ends the reads of the tile
        // w_k = u + c2 w_{k-1}; beta_{k+1}
        const double c2 = uniform(-(a * inv));
        sum = Sum();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double wr = fma(c2, wc[e].x, acc[e]);
            const double wi = fma(c2, wc[e].y, acc[E + e]);
            put(tid + e * T, make_double2(wr, wi));
            sum.product(wr, wr);
            sum.product(wi, wi);
            wp[e] = wc[e];
            wc[e] = make_double2(wr, wi);
        }
        const double bn = uniform(sqrt(block_sum<T>(sum, sh_b)));
        if (tid == 0) {
            alpha[k] = a;
            beta[k] = bn;
        }
        if (bad == 0 && !(isfinite(a) && isfinite(bn))) bad = k + 2;
        if (!(bn > R.tol)) {
            done = 1;  // invariant subspace
        } else {
            inv_prev = inv;
            inv = uniform(1.0 / bn);
            bcur = bn;
        }
    }
    if (tid == 0) end_state(st, inv, inv_prev, bcur, a, done, k, bad);
    if (carry && !done) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t x = tid + e * T;
            ((double2 *)carry)[x] = wc[e];
            ((double2 *)carry)[dim + x] = wp[e];
        }
    }
}

// A sequence's carried vectors through a buffer descriptor: entry tid + i with i
// uniform is one register of lane offset and one scalar (a flat address takes two
// registers for each of a thread's 16 entries), and is bounds-checked by the hardware.
struct Carried {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t lane;  // byte offset of entry tid
    uint32_t entries;
    __device__ Carried(double *p, uint32_t n)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)(n * sizeof(double)), 0x00027000)),
          lane(threadIdx.x * (uint32_t)sizeof(double)), entries(n)
    {
    }
    __device__ __forceinline__ double get(uint32_t i) const
    {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, lane, FTK_IDX(i, blockDim.x - 1, entries, 16) * 8, 0));
    }
    __device__ __forceinline__ void set(uint32_t i, double x) const
    {
        typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, x), rsrc, lane, FTK_IDX(i, blockDim.x - 1, entries, 16) * 8, 0);
    }
};

// The same for vectors of two planes (real, imaginary) too large to keep complex in
// LDS: H is real, so a step multiplies one plane after the other, each staged in LDS
// (128 KiB at 14 sites) with its sums in registers.  w_{k-1} and w_{k-2} live in the
// sequence's carry buffer (planar, re-read from L2): w_k overwrites w_{k-2}.  LDS
// reads bound a step (8 B per element, plane and bond).
template <int LOGT, int E>
__global__ void __launch_bounds__(1 << LOGT) k_resident_planes(HvParams P, ResidentRun R)
{
    constexpr int T = 1 << LOGT;
    constexpr uint32_t dim = T * E;
    __shared__ double plane[dim];
    __shared__ double2 sh_a[T / 64], sh_b[T / 64];
    const ResidentSeq q = R.seq[blockIdx.x];
    const uint32_t tid = FTK_IDX(threadIdx.x, (E - 1) * T, dim, 14);
    SeqState *st = R.st + q.out;
    double *alpha = R.alpha + (size_t)q.out * R.stride, *beta = R.beta + (size_t)q.out * R.stride;
    const int nb = P.n_bonds;
    uint64_t par = 0;
#pragma unroll
    for (int l = 0; l < LOGT; ++l)
        if ((tid >> l) & 1u) par ^= P.smask[l];
    const Bonds bonds(P, P.code, nb, par);
    const int nz = __popcll(P.zmask);
    // the diagonal as its two bond sums, 8 bits each, two elements a word
    uint32_t dsum[E / 2];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        uint64_t pe = par;
        if (e & 1) pe ^= P.smask[LOGT];
        if (e & 2) pe ^= P.smask[LOGT + 1];
        if (e & 4) pe ^= P.smask[LOGT + 2];
        if (e & 8) pe ^= P.smask[LOGT + 3];
        const uint32_t c = (uint32_t)__popcll(pe) | (uint32_t)__popcll(pe & P.zmask) << 8;
        if (e & 1) dsum[e >> 1] |= c << 16;
        else dsum[e >> 1] = c;
    }
    auto diagonal = [&](int e) {
        const uint32_t c = dsum[e >> 1] >> (16 * (e & 1));
        const int s_all = nb - 2 * (int)(c & 0xffu);
        const int s_z = nz - 2 * (int)(c >> 8 & 0xffu);
        return fma(P.kq, (double)s_z, P.jq * (double)s_all);
    };

    // a thread's own entries: two bases, so that every offset fits the instruction
    uint32_t upper = tid + 8 * T;
    asm volatile("" : "+v"(upper));
    auto own = [&](int e) -> double & { return plane[(e < 8 ? tid : upper) + (e & 7) * T]; };

    const uint32_t plane_at = lds_address(plane);
    const Carried buf(R.carry + (size_t)blockIdx.x * 4 * dim, 4 * dim);  // w_k at entry (k & 1) 2 dim
    double inv, inv_prev, bcur;
    int bad;  // 1 + the first step after which a scalar was not finite (1: the start), 0 none
    if (R.k0 == 0) {
        const double2 *start = R.chi ? (const double2 *)R.chi + (size_t)blockIdx.x * dim : q.phi;
        Sum sum;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t x = tid + e * T;
            const double2 c = start[x];
            own(e) = c.x;
            buf.set(2 * dim + e * T, c.x);
            buf.set(3 * dim + e * T, c.y);
            sum.product(c.x, c.x);
            sum.product(c.y, c.y);
            if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
        const double s = block_sum<T>(sum, sh_b);
        const double nrm = sqrt(s);
        inv = uniform(nrm > 0.0 ? 1.0 / nrm : 0.0);
        inv_prev = 0.0;
        bcur = 0.0;
        bad = isfinite(s) ? 0 : 1;
        if (tid == 0) start_state(st, s, nrm, inv, q.shift_re, bad);
        if (!(nrm > 0.0)) return;
    } else {
        if (st->done) return;
        inv = st->inv_cur;
        inv_prev = st->inv_prev;
        bcur = st->beta_cur;
        bad = st->pad;
        const uint32_t w = ((R.k0 - 1) & 1) * 2 * dim;
#pragma unroll
        for (int e = 0; e < E; ++e) own(e) = buf.get(w + e * T);
        lds_barrier();
    }

    double2 *vout = R.vout ? (double2 *)(R.vout + (size_t)blockIdx.x * R.vstride) : nullptr;
    int k = R.k0, done = 0;
    double a = 0.0;
    for (; k < R.k1 && !done; ++k) {
        const bool first = k == 0;
        const uint32_t wnew = (k & 1) * 2 * dim;       // w_{k-2}, then w_k
        const uint32_t wcur = ((k + 1) & 1) * 2 * dim;  // w_{k-1}
        const double c1 = uniform((-bcur) * inv_prev);
        double acc[E];
        Sum sum;
        // u = (H w_{k-1}) inv + c1 w_{k-2} of the plane in LDS, into acc; its share of alpha_k
        auto half = [&](uint32_t wp) {
            double prev[E];  // read while the bonds run (step 0 has none and drops what it reads)
#pragma unroll
            for (int e = 0; e < E; ++e) prev[e] = buf.get(wp + e * T);
#pragma unroll
            for (int i = 0; i < E / 2; ++i) asm volatile("" : "+v"(dsum[i]));  // decoded here, not kept for all steps
#pragma unroll
            for (int e = 0; e < E; ++e) {
                acc[e] = diagonal(e) * own(e);
                if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            for (int b = 0; b < nb; ++b) {
                const BondAt c = bonds.at(b);
                if constexpr (E == 16) {
                    const uint32_t t0 = plane_at + FTK_IDX(tid ^ (c.m & (T - 1)), (E - 1) * T, dim, 15) * 8;
                    bond16<T * 8>(acc, t0, t0 + 64 * T, c.m >> LOGT, c.even, c.odd);
                    continue;
                }
                const double even = c.even, odd = c.odd;
                const uint32_t sel = odd_elements(c.m >> LOGT);
                const char *src = (const char *)plane;
                const uint32_t base = FTK_IDX(tid ^ c.m, 0, dim, 15) * (uint32_t)sizeof(double);
                double v[E];
#pragma unroll
                for (int e = 0; e < E; ++e)
                    v[e] = *(const double *)(src + (base ^ (uint32_t)(e * T * sizeof(double))));
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = fma(((sel >> e) & 1u) ? odd : even, v[e], acc[e]);
            }
            asm volatile("" ::: "memory");  // own entries are read again below, not kept over the bonds
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const double t = acc[e] * inv, u = fma(c1, prev[e], t);
                acc[e] = first ? t : u;
            }
            Sum part;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                part.product(own(e), acc[e]);
                if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            // added up here, to two registers: not their 32 factors kept to the end
            const double low = part.low();
            sum.pair(part.hi, low);
            sum.er = sum.low();
            sum.lo = 0.0;
            asm volatile("" : "+v"(sum.hi), "+v"(sum.er));
        };
        double own_re[E], own_im[E];
        half(wnew);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            own_im[e] = buf.get(wcur + dim + e * T);
            buf.set(wnew + e * T, acc[e]);  // u's real part, in the place of w_{k-2}'s
        }
        lds_barrier();  // the real plane is no longer read
#pragma unroll
        for (int e = 0; e < E; ++e) own(e) = own_im[e];
        lds_barrier();
        half(wnew + dim);
        double u_re[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            own_re[e] = buf.get(wcur + e * T);
            u_re[e] = buf.get(wnew + e * T);
        }
        a = uniform(inv * block_sum<T>(sum, sh_a));  // nor the imaginary one
        if (vout) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                (vout + (size_t)(k - R.k0) * dim + e * T)[tid] = make_double2(own_re[e], own(e));
                if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            asm volatile("" ::: "memory");
        }
        const double c2 = uniform(-(a * inv));
        sum = Sum();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const double ci = own(e);
            const double wr = fma(c2, own_re[e], u_re[e]);
            const double wi = fma(c2, ci, acc[e]);
            own(e) = wr;
            buf.set(wnew + e * T, wr);
            buf.set(wnew + dim + e * T, wi);
            sum.product(wr, wr);
            sum.product(wi, wi);
            if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
        }
        const double bn = uniform(sqrt(block_sum<T>(sum, sh_b)));
        if (tid == 0) {
            alpha[k] = a;
            beta[k] = bn;
        }
        if (bad == 0 && !(isfinite(a) && isfinite(bn))) bad = k + 2;
        if (!(bn > R.tol)) {
            done = 1;  // invariant subspace
        } else {
            inv_prev = inv;
            inv = uniform(1.0 / bn);
            bcur = bn;
        }
    }
    if (tid == 0) end_state(st, inv, inv_prev, bcur, a, done, k, bad);
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
    // 192 sequences of 64 steps: 0.35 against 0.40 ms a call), as do 256 with four
    // against 128 with eight (10 sites, 48 sequences of 200 steps: 0.87 against 1.12 ms);
    // at 12 sites 512 threads with eight elements share the bonds' scalar work and the
    // reductions among fewer waves than 1024 with four (48 sequences of 300 steps: 3.00
    // against 3.24 ms, both with selects in place of bond16)
    case 6: launch_resident_t<6, 1>(op.P, run, n_seq, s); break;
    case 7: launch_resident_t<7, 1>(op.P, run, n_seq, s); break;
    case 8: launch_resident_t<8, 1>(op.P, run, n_seq, s); break;
    case 9: launch_resident_t<8, 2>(op.P, run, n_seq, s); break;
    case 10: launch_resident_t<8, 4>(op.P, run, n_seq, s); break;
    case 11: launch_resident_t<9, 4>(op.P, run, n_seq, s); break;
    case 12: launch_resident_t<9, 8>(op.P, run, n_seq, s); break;
    case 13: hipLaunchKernelGGL((k_resident_planes<10, 8>), dim3(n_seq), dim3(1024), 0, s, op.P, run); break;
    case 14: hipLaunchKernelGGL((k_resident_planes<10, 16>), dim3(n_seq), dim3(1024), 0, s, op.P, run); break;
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

#ifdef FTK_DEVICE_CHECKS
bool resident_checks_read(unsigned int out[3], bool clear) { return dchk_read(out, clear); }
#endif

}  // namespace ftk
