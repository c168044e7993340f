// canonical.h -- reading and writing canonical complex128 [site][12] buffers.
#pragma once
#include "views.h"

namespace tmq {

__device__ __forceinline__ void load_canonical(const double2 *in, long site, spinor<double> &s)
{
    const double2 *q = in + site * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        double2 v = q[k];
        s.c[k / 3][k % 3] = cx<double>{v.x, v.y};
    }
}

__device__ __forceinline__ void store_canonical(double2 *out, long site, const spinor<double> &s)
{
    double2 *q = out + site * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) q[k] = make_double2(s.c[k / 3][k % 3].re, s.c[k / 3][k % 3].im);
}

// parity of canonical site s
__device__ __forceinline__ int site_parity(const Geom &g, long s)
{
    const unsigned su = (unsigned)s;
    const unsigned x = su % (unsigned)g.LX;
    unsigned r = su / (unsigned)g.LX;
    const unsigned y = r % (unsigned)g.LY;
    r /= (unsigned)g.LY;
    const unsigned z = r % (unsigned)g.LZ;
    const unsigned t = r / (unsigned)g.LZ;
    return (int)((t + z + y + x) & 1u);
}

}  // namespace tmq
