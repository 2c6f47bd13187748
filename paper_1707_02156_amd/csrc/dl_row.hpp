// Product of one stored double-layer row with a density (gfx950, FP64): the
// body of k_dl_apply_multi and of the row blocks of k_synth_rows.
#pragma once
#include "internal.hpp"

#include <hip/hip_runtime.h>

namespace bim {

// One target row: (o0, o1, o2) = M_t (u0, u1, u2) over the six symmetric pair
// rows of length nc2 (even; rows and densities 16-byte aligned), read as
// double2 by one wavefront, two iterations of loads in flight per lane.
__device__ inline void dl_row(const double *__restrict__ Mt, const double *__restrict__ u, long ustride, int nc2,
                              int lane, double &o0, double &o1, double &o2)
{
    const int h = nc2 >> 1;
    const double2 *M0 = reinterpret_cast<const double2 *>(Mt), *M1 = M0 + h, *M2 = M1 + h, *M3 = M2 + h,
                  *M4 = M3 + h, *M5 = M4 + h;
    const double2 *U0 = reinterpret_cast<const double2 *>(u), *U1 = reinterpret_cast<const double2 *>(u + ustride),
                  *U2 = reinterpret_cast<const double2 *>(u + 2 * ustride);
    o0 = o1 = o2 = 0.0;
#pragma unroll 2
    for (int e = lane; e < h; e += 64) {
        const double2 a = U0[e], b = U1[e], c = U2[e];
        const double2 m00 = M0[e], m01 = M1[e], m02 = M2[e], m11 = M3[e], m12 = M4[e], m22 = M5[e];
        o0 = fma(m00.x, a.x, fma(m01.x, b.x, fma(m02.x, c.x, o0)));
        o1 = fma(m01.x, a.x, fma(m11.x, b.x, fma(m12.x, c.x, o1)));
        o2 = fma(m02.x, a.x, fma(m12.x, b.x, fma(m22.x, c.x, o2)));
        o0 = fma(m00.y, a.y, fma(m01.y, b.y, fma(m02.y, c.y, o0)));
        o1 = fma(m01.y, a.y, fma(m11.y, b.y, fma(m12.y, c.y, o1)));
        o2 = fma(m02.y, a.y, fma(m12.y, b.y, fma(m22.y, c.y, o2)));
    }
    for (int o = 32; o > 0; o >>= 1) {
        o0 += __shfl_down(o0, o, 64);
        o1 += __shfl_down(o1, o, 64);
        o2 += __shfl_down(o2, o, 64);
    }
}

}  // namespace bim
