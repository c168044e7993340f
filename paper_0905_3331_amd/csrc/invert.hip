// invert.hip -- the vector passes of M psi = phi (see invert.h).
//
// Streams of whole FP64 fields, bound by memory: what counts is how often a
// field is passed over.  A source was converted, copied times g5, normed and
// multiplied by (M_ee)^-1 in passes of its own, a solution added to zeros, the
// residual formed against the g5 copy, multiplied by g5 and normed, and each
// right-hand side converted in launches of its own.  Here a source is read
// once on entry and once more for the residual, where g5 is a sign.
// Twelve sources at 16^3x32 (302 MB a field), us: entry 430 -> 130, odd source
// to the solver 150 -> 65, residual 340 -> 184 (4.9 TB/s), exit 190 -> 133, and
// the solution's zeros and addition, 165, are gone: the inversion 11960 -> 11200.
// Lanes take canonical sites in order, so that a buffer is read in order and
// the two parities of a field in two.
#include "invert.h"
#include "canonical.h"
#include "devutil.h"

namespace tmq {

#define BLOCK_RHS(rl) const int rhs = (rl).idx[blockIdx.y]

__device__ __forceinline__ void norm_partial(const spinor<double> &s, bool on, double *partial)
{
    double n = 0.0;
    if (on)
#pragma unroll
        for (int k = 0; k < 12; k++) n += norm2(s.c[k / 3][k % 3]);
    n = wave_sum(n);
    if ((threadIdx.x & 63) == 0) partial[(long)PARTS * blockIdx.x + (threadIdx.x >> 6)] = n;
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_m_enter(Geom g, CanList phi, BatchView<SpF64> r, BatchView<SpF64> te,
                                                        double2 cu, double2 cd, RhsList rl, double *partial,
                                                        long pstride)
{
    BLOCK_RHS(rl);
    const long s = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    const bool on = s < 2 * g.vh;
    spinor<double> v;
    if (on) {
        load_canonical(phi.p[rhs], s, v);
        const int par = site_parity(g, s);
        r.at(rhs).store(par * g.vh + (s >> 1), v);
        if (par == 0) {
            const cx<double> u = {cu.x, cu.y}, d = {cd.x, cd.y};
            spinor<double> w;
#pragma unroll
            for (int k = 0; k < 12; k++) w.c[k / 3][k % 3] = (k < 6 ? u : d) * v.c[k / 3][k % 3];
            te.at(rhs).store(s >> 1, w);
        }
    }
    norm_partial(v, on, partial + rhs * pstride);
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_m_residual(Geom g, CanList phi, BatchView<SpF64> q, BatchView<SpF64> r,
                                                           RhsList rl, double *partial, long pstride)
{
    BLOCK_RHS(rl);
    const long s = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    const bool on = s < 2 * g.vh;
    spinor<double> v;
    if (on) {
        const long h = site_parity(g, s) * g.vh + (s >> 1);
        spinor<double> a;
        load_canonical(phi.p[rhs], s, v);
        q.at(rhs).load(h, a);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            cx<double> &c = v.c[k / 3][k % 3];
            c = k < 6 ? c - a.c[k / 3][k % 3] : c + a.c[k / 3][k % 3];
        }
        r.at(rhs).store(h, v);
    }
    norm_partial(v, on, partial + rhs * pstride);
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_m_to_canonical(BatchView<SpF64> in, BatchView<SpF64> can, double down,
                                                               long n, RhsList rl)
{
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<double> v;
        in.at(rhs).load(h, v);
#pragma unroll
        for (int k = 6; k < 12; k++) {
            cx<double> &c = v.c[k / 3][k % 3];
            c = cx<double>{down * c.re, down * c.im};
        }
        store_canonical(can.at(rhs).p, h, v);
    }
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_m_from_canonical(BatchView<SpF64> can, BatchView<SpF64> out, long n,
                                                                 RhsList rl)
{
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<double> v;
        load_canonical(can.at(rhs).p, h, v);
        out.at(rhs).store(h, v);
    }
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_m_leave(Geom g, BatchView<SpF64> x, CanList psi, RhsList rl)
{
    BLOCK_RHS(rl);
    const long s = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (s < 2 * g.vh) {
        spinor<double> v;
        x.at(rhs).load(site_parity(g, s) * g.vh + (s >> 1), v);
        store_canonical(psi.p[rhs], s, v);
    }
}

#define LAUNCH_M(K, sites, ...)                                                                              \
    if (rl.n <= 0) return hipSuccess;                                                                      \
    hipLaunchKernelGGL(K, dim3(blas_grid(sites), rl.n), dim3(BLAS_BLOCK), 0, st, __VA_ARGS__);             \
    return hipGetLastError()

hipError_t launch_m_enter(const Geom &g, const CanList &phi, const FieldDesc &r, const FieldDesc &te, double2 cu,
                          double2 cd, const RhsList &rl, double *partial, long pstride, hipStream_t st)
{
    if (r.prec != P64 || te.prec != P64 || r.n != 2 * g.vh || te.n != g.vh) return hipErrorInvalidValue;
    LAUNCH_M(k_m_enter, r.n, g, phi, make_bv<SpF64>(r), make_bv<SpF64>(te), cu, cd, rl, partial, pstride);
}

hipError_t launch_m_residual(const Geom &g, const CanList &phi, const FieldDesc &q, const FieldDesc &r,
                             const RhsList &rl, double *partial, long pstride, hipStream_t st)
{
    if (q.prec != P64 || r.prec != P64 || q.n != 2 * g.vh || r.n != 2 * g.vh) return hipErrorInvalidValue;
    LAUNCH_M(k_m_residual, r.n, g, phi, make_bv<SpF64>(q), make_bv<SpF64>(r), rl, partial, pstride);
}

hipError_t launch_m_to_canonical(const FieldDesc &in, const FieldDesc &can, double down, const RhsList &rl,
                                 hipStream_t st)
{
    if (in.prec != P64 || can.prec != P64 || in.n != can.n) return hipErrorInvalidValue;
    LAUNCH_M(k_m_to_canonical, in.n, make_bv<SpF64>(in), make_bv<SpF64>(can), down, in.n, rl);
}

hipError_t launch_m_from_canonical(const FieldDesc &can, const FieldDesc &out, const RhsList &rl, hipStream_t st)
{
    if (out.prec != P64 || can.prec != P64 || out.n != can.n) return hipErrorInvalidValue;
    LAUNCH_M(k_m_from_canonical, out.n, make_bv<SpF64>(can), make_bv<SpF64>(out), out.n, rl);
}

hipError_t launch_m_leave(const Geom &g, const FieldDesc &x, const CanList &psi, const RhsList &rl, hipStream_t st)
{
    if (x.prec != P64 || x.n != 2 * g.vh) return hipErrorInvalidValue;
    LAUNCH_M(k_m_leave, x.n, g, make_bv<SpF64>(x), psi, rl);
}

}  // namespace tmq
