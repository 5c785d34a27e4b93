// Linear spin operators on a state vector, shared by the kernels that apply them.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_checks.h"

namespace ftk {

// chi = S^alpha_{+Q} phi (Sec. V): x and y flip one spin, z is diagonal.
// <down|S^y|up> = +i/2 and <up|S^y|down> = -i/2 (bit 1 = spin down).  h holds
// the per-site factors (interleaved), the 1/2 of S = sigma/2 included.
template <class Coef>
__device__ __forceinline__ double2 sq_part(int n_sites, int alpha, const Coef &h, const double2 *__restrict__ phi,
                                           uint32_t x)
{
    double re = 0.0, im = 0.0;
    if (alpha == 2) {
        double cr = 0.0, ci = 0.0;
        for (int l = 0; l < n_sites; ++l) {
            if ((x >> l) & 1u) {
                cr = cr - h[2 * l];
                ci = ci - h[2 * l + 1];
            } else {
                cr = cr + h[2 * l];
                ci = ci + h[2 * l + 1];
            }
        }
        const double2 p = phi[x];
        re = cr * p.x - ci * p.y;
        im = cr * p.y + ci * p.x;
    } else {
        for (int l = 0; l < n_sites; ++l) {
            double cr = h[2 * l], ci = h[2 * l + 1];
            if (alpha == 1) {
                if ((x >> l) & 1u) {
                    const double t = cr;
                    cr = -ci;
                    ci = t;
                } else {
                    const double t = cr;
                    cr = ci;
                    ci = -t;
                }
            }
            const double2 p = phi[FTK_IDX(x ^ (1u << l), 0, 1u << n_sites, 12)];
            const double tr = cr * p.x - ci * p.y;
            const double ti = cr * p.y + ci * p.x;
            re = re + tr;
            im = im + ti;
        }
    }
    return make_double2(re, im);
}

// (A phi)[x] for a linear spin operator (operators A, B of Sec. III.B): the three
// components formed as above, added in the order (x + y) + z.
template <class Coef>
__device__ __forceinline__ double2 spin_op_part(int n_sites, const Coef &h, const double2 *__restrict__ phi, uint32_t x)
{
    const double2 a = sq_part(n_sites, 0, h[0], phi, x);
    const double2 b = sq_part(n_sites, 1, h[1], phi, x);
    const double2 c = sq_part(n_sites, 2, h[2], phi, x);
    return make_double2((a.x + b.x) + c.x, (a.y + b.y) + c.y);
}

// entry of the start vector k of the polarization identity: lam + rho, lam - rho,
// lam + i rho, lam - i rho for k = 0..3
__device__ __forceinline__ double2 polarize_part(int k, double2 a, double2 b)
{
    if (k == 0) return make_double2(a.x + b.x, a.y + b.y);
    if (k == 1) return make_double2(a.x - b.x, a.y - b.y);
    if (k == 2) return make_double2(a.x - b.y, a.y + b.x);
    return make_double2(a.x + b.y, a.y - b.x);
}

}  // namespace ftk
