// The bond loop of the kernels that hold a tile of a vector in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace ftk {

// The bond constants of a thread: one bond's code per lane, the amplitudes by bond
// type (scalar), the bond parities of the thread's element 0.
struct BondAt {
    double even, odd;  // amplitudes of elements whose register bits the bond flips with even, odd parity
    uint32_t m;        // flip mask
};
struct Bonds {
    int code;
    double ap0, ap1, ap2, aa0, aa1, aa2;
    uint32_t par_lo, par_hi;
    // n bonds' codes (flip mask of a thread's tile | bond type << 30), bit b of par the
    // parity of bond b at the thread's element 0
    __device__ Bonds(const HvParams &P, const uint32_t *codes, int n, uint64_t par)
        : ap0(P.ap3[0]), ap1(P.ap3[1]), ap2(P.ap3[2]), aa0(P.aa3[0]), aa1(P.aa3[1]), aa2(P.aa3[2]),
          par_lo((uint32_t)par), par_hi((uint32_t)(par >> 32))
    {
        const int l = (int)(threadIdx.x & 63);
        code = (int)codes[l < n ? l : 0];
    }
    __device__ __forceinline__ BondAt at(int b) const
    {
        const uint32_t c = (uint32_t)__builtin_amdgcn_readlane(code, b);
        const uint32_t type = c >> 30;
        const double p0 = ap0, p1 = ap1, p2 = ap2, q0 = aa0, q1 = aa1, q2 = aa2;
        const double ap = type == 0 ? p0 : type == 1 ? p1 : p2;
        const double aa = type == 0 ? q0 : type == 1 ? q1 : q2;
        const bool anti = ((b < 32 ? par_lo : par_hi) & (1u << (b & 31))) != 0;
        return BondAt{anti ? aa : ap, anti ? ap : aa, c & 0x3fffffffu};
    }
};

// One bond on 16 sums of a thread.  Sum e takes entry e ^ mr of the 16 entries STRIDE
// bytes apart at LDS address t0 (entries 8..15 at t8 = t0 + 8 STRIDE, so that every
// offset fits the instruction) with the amplitude of the parity of e & mr; mr, the
// register bits the bond flips, has at most two bits set.  Each value of mr has its
// own offsets and amplitude registers, so a sum costs one fma; written as one asm
// block because the compiler keeps the sums of different cases in different
// registers and copies all of them for every bond, and without the cases each sum
// takes two selects and an address (14 sites, 200 steps of 64 sequences: 12.2 ms
// with selects).  Eight reads are in flight; they return in order, and every one is
// waited for in the block.
#define FTK_RD(r, base, k) "ds_read_b64 %[v" #r "], %[" #base "] offset:" #k "*%[st]\n\t"
#define FTK_RD_0(r) FTK_RD(r, t0, 0)
#define FTK_RD_1(r) FTK_RD(r, t0, 1)
#define FTK_RD_2(r) FTK_RD(r, t0, 2)
#define FTK_RD_3(r) FTK_RD(r, t0, 3)
#define FTK_RD_4(r) FTK_RD(r, t0, 4)
#define FTK_RD_5(r) FTK_RD(r, t0, 5)
#define FTK_RD_6(r) FTK_RD(r, t0, 6)
#define FTK_RD_7(r) FTK_RD(r, t0, 7)
#define FTK_RD_8(r) FTK_RD(r, t8, 0)
#define FTK_RD_9(r) FTK_RD(r, t8, 1)
#define FTK_RD_10(r) FTK_RD(r, t8, 2)
#define FTK_RD_11(r) FTK_RD(r, t8, 3)
#define FTK_RD_12(r) FTK_RD(r, t8, 4)
#define FTK_RD_13(r) FTK_RD(r, t8, 5)
#define FTK_RD_14(r) FTK_RD(r, t8, 6)
#define FTK_RD_15(r) FTK_RD(r, t8, 7)
#define FTK_WAIT(n) "s_waitcnt lgkmcnt(" #n ")\n\t"
#define FTK_FMA(e, r, c) "v_fmac_f64_e32 %[a" #e "], %[" #c "], %[v" #r "]\n\t"
#define FTK_CASE(mr, p0, p1, p2, p3, p4, p5, p6, p7, p8, p9, p10, p11, p12, p13, p14, p15, c0, c1, c2, c3, c4, c5, c6, \
                 c7, c8, c9, c10, c11, c12, c13, c14, c15)                                                              \
    ".Lftk_case" #mr "_%=:\n\t" FTK_RD_##p0(0) FTK_RD_##p1(1) FTK_RD_##p2(2) FTK_RD_##p3(3) FTK_RD_##p4(4)             \
        FTK_RD_##p5(5) FTK_RD_##p6(6) FTK_RD_##p7(7) FTK_WAIT(7) FTK_FMA(0, 0, c0) FTK_RD_##p8(0) FTK_WAIT(7)            \
            FTK_FMA(1, 1, c1) FTK_RD_##p9(1) FTK_WAIT(7) FTK_FMA(2, 2, c2) FTK_RD_##p10(2) FTK_WAIT(7) FTK_FMA(3, 3, c3)  \
                FTK_RD_##p11(3) FTK_WAIT(7) FTK_FMA(4, 4, c4) FTK_RD_##p12(4) FTK_WAIT(7) FTK_FMA(5, 5, c5)               \
                    FTK_RD_##p13(5) FTK_WAIT(7) FTK_FMA(6, 6, c6) FTK_RD_##p14(6) FTK_WAIT(7) FTK_FMA(7, 7, c7)           \
                        FTK_RD_##p15(7) FTK_WAIT(7) FTK_FMA(8, 0, c8) FTK_WAIT(6) FTK_FMA(9, 1, c9) FTK_WAIT(5)           \
                            FTK_FMA(10, 2, c10) FTK_WAIT(4) FTK_FMA(11, 3, c11) FTK_WAIT(3) FTK_FMA(12, 4, c12)           \
                                FTK_WAIT(2) FTK_FMA(13, 5, c13) FTK_WAIT(1) FTK_FMA(14, 6, c14) FTK_WAIT(0)               \
                                    FTK_FMA(15, 7, c15) "s_branch .Lftk_done_%=\n"
#define FTK_GOTO(mr) "s_cmp_eq_u32 %[mr], " #mr "\n\ts_cbranch_scc1 .Lftk_case" #mr "_%=\n\t"
#define FTK_CASES \
    FTK_CASE(0, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev, ev) \
    FTK_CASE(1, 1, 0, 3, 2, 5, 4, 7, 6, 9, 8, 11, 10, 13, 12, 15, 14, ev, od, ev, od, ev, od, ev, od, ev, od, ev, od, ev, od, ev, od) \
    FTK_CASE(2, 2, 3, 0, 1, 6, 7, 4, 5, 10, 11, 8, 9, 14, 15, 12, 13, ev, ev, od, od, ev, ev, od, od, ev, ev, od, od, ev, ev, od, od) \
    FTK_CASE(3, 3, 2, 1, 0, 7, 6, 5, 4, 11, 10, 9, 8, 15, 14, 13, 12, ev, od, od, ev, ev, od, od, ev, ev, od, od, ev, ev, od, od, ev) \
    FTK_CASE(4, 4, 5, 6, 7, 0, 1, 2, 3, 12, 13, 14, 15, 8, 9, 10, 11, ev, ev, ev, ev, od, od, od, od, ev, ev, ev, ev, od, od, od, od) \
    FTK_CASE(5, 5, 4, 7, 6, 1, 0, 3, 2, 13, 12, 15, 14, 9, 8, 11, 10, ev, od, ev, od, od, ev, od, ev, ev, od, ev, od, od, ev, od, ev) \
    FTK_CASE(6, 6, 7, 4, 5, 2, 3, 0, 1, 14, 15, 12, 13, 10, 11, 8, 9, ev, ev, od, od, od, od, ev, ev, ev, ev, od, od, od, od, ev, ev) \
    FTK_CASE(8, 8, 9, 10, 11, 12, 13, 14, 15, 0, 1, 2, 3, 4, 5, 6, 7, ev, ev, ev, ev, ev, ev, ev, ev, od, od, od, od, od, od, od, od) \
    FTK_CASE(9, 9, 8, 11, 10, 13, 12, 15, 14, 1, 0, 3, 2, 5, 4, 7, 6, ev, od, ev, od, ev, od, ev, od, od, ev, od, ev, od, ev, od, ev) \
    FTK_CASE(10, 10, 11, 8, 9, 14, 15, 12, 13, 2, 3, 0, 1, 6, 7, 4, 5, ev, ev, od, od, ev, ev, od, od, od, od, ev, ev, od, od, ev, ev) \
    FTK_CASE(12, 12, 13, 14, 15, 8, 9, 10, 11, 4, 5, 6, 7, 0, 1, 2, 3, ev, ev, ev, ev, od, od, od, od, od, od, od, od, ev, ev, ev, ev)

template <int STRIDE>
__device__ __forceinline__ void bond16(double (&acc)[16], uint32_t t0, uint32_t t8, uint32_t mr, double even, double odd)
{
    double v0, v1, v2, v3, v4, v5, v6, v7;
    asm volatile(
        "s_waitcnt lgkmcnt(0)\n\t"  // only the block's own reads are counted below
        FTK_GOTO(0) FTK_GOTO(1) FTK_GOTO(2) FTK_GOTO(4) FTK_GOTO(8) FTK_GOTO(3) FTK_GOTO(5) FTK_GOTO(6) FTK_GOTO(9)
            FTK_GOTO(10) FTK_GOTO(12) "s_branch .Lftk_done_%=\n" FTK_CASES ".Lftk_done_%=:\n"
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]), [a4] "+v"(acc[4]), [a5] "+v"(acc[5]),
          [a6] "+v"(acc[6]), [a7] "+v"(acc[7]), [a8] "+v"(acc[8]), [a9] "+v"(acc[9]), [a10] "+v"(acc[10]),
          [a11] "+v"(acc[11]), [a12] "+v"(acc[12]), [a13] "+v"(acc[13]), [a14] "+v"(acc[14]), [a15] "+v"(acc[15]),
          [v0] "=&v"(v0), [v1] "=&v"(v1), [v2] "=&v"(v2), [v3] "=&v"(v3), [v4] "=&v"(v4), [v5] "=&v"(v5), [v6] "=&v"(v6),
          [v7] "=&v"(v7)
        : [t0] "v"(t0), [t8] "v"(t8), [mr] "s"(mr), [ev] "v"(even), [od] "v"(odd), [st] "n"(STRIDE)
        : "scc", "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

}  // namespace ftk
