// Device bounds checks of the debug build (-DFTK_DEVICE_CHECKS, libftkw_check.so):
// FTK_IDX(i, top, lim, site) states that indices i .. i + top of a buffer with lim
// entries are read or written.  In the debug build a violation is counted in the
// translation unit's g_dcheck (count, site of the first, its index) and index 0 is used instead, so
// the kernel finishes and the host reports it; the release build compiles the
// check away.  Sites: 1 single-element H v gather, 2/3 blocked and tiled gathers
// (global, LDS), 4 own elements of the blocked/tiled forms, 5 own LDS entries of
// the tiled form, 6/7 multi-pass global element and LDS tile entries, 8 multi-pass
// LDS partners, 10/11 batch-layout own elements
// and partners, 12 S^alpha_Q gathers, 13 filter accumulation, 14 resident sequences' own
// entries (LDS and global), 15 their LDS partners, 16 their carried vectors.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#ifdef FTK_DEVICE_CHECKS
namespace ftk {

static __device__ unsigned int g_dcheck[3];
__device__ __forceinline__ uint32_t dchk(uint32_t i, uint32_t top, uint32_t lim, uint32_t site)
{
    if (i < lim && top < lim - i) return i;
    if (atomicAdd(&g_dcheck[0], 1u) == 0u) {
        g_dcheck[1] = site;
        g_dcheck[2] = i;
    }
    return 0u;
}
// this unit's counters added to out (count, first site, its index)
static inline bool dchk_read(unsigned int out[3], bool clear)
{
    unsigned int r[3] = {0u, 0u, 0u};
    hipError_t e = hipMemcpyFromSymbol(r, HIP_SYMBOL(g_dcheck), sizeof r);
    if (e == hipSuccess && clear) {
        const unsigned int z[3] = {0u, 0u, 0u};
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_dcheck), z, sizeof z);
    }
    if (out[0] == 0u) out[1] = r[1], out[2] = r[2];
    out[0] += r[0];
    return e == hipSuccess;
}

}  // namespace ftk
#define FTK_IDX(i, top, lim, site) ftk::dchk((uint32_t)(i), (uint32_t)(top), (uint32_t)(lim), (site))
#else
#define FTK_IDX(i, top, lim, site) (i)
#endif
