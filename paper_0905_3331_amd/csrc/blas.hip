// blas.hip -- site-parallel vector kernels of the CG solvers and their scalars.
//
// One lane per lattice site (all 12 spin-colour components), so that the
// per-site scaled 16-bit formats can be decoded and re-encoded in registers.
// Grid: x over the sites, y over the RHS of the launch.  Every reduction
// writes one FP64 partial per wavefront; a single-block-per-RHS scalar kernel
// sums the partials in a fixed order, which makes norms, inner products and
// therefore iteration counts bit-reproducible from run to run and
// independent of the batch an RHS is solved in.
#include "devutil.h"
#include "views.h"

namespace tmq {

RhsList rhs_all(int n)
{
    RhsList l;
    l.n = n < 0 ? 0 : (n > MAX_RHS ? MAX_RHS : n);
    for (int i = 0; i < l.n; i++) l.idx[i] = (unsigned char)i;
    return l;
}

template <typename R>
__device__ __forceinline__ R site_norm2(const spinor<R> &s)
{
    R n = R(0);
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) n += norm2(s.c[i][j]);
    return n;
}

// RHS of this block (grid y)
#define BLOCK_RHS(rl) const int rhs = (rl).idx[blockIdx.y]

#define WRITE_PARTIAL(ptr, pstride, part)                                                             \
    {                                                                                                 \
        const double s_ = wave_sum(part);                                                             \
        if ((threadIdx.x & 63) == 0)                                                                  \
            (ptr)[rhs * (pstride) + (long)PARTS * blockIdx.x + (threadIdx.x >> 6)] = s_;              \
    }

template <class F>
__global__ __launch_bounds__(BLAS_BLOCK) void k_norm2(BatchView<F> v, long n, RhsList rl, double *partial,
                                                      long pstride)
{
    using R = typename F::real;
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double part = 0.0;
    if (h < n) {
        spinor<R> s;
        v.at(rhs).load(h, s);
        part = (double)site_norm2(s);
    }
    WRITE_PARTIAL(partial, pstride, part)
}

template <class FI, class FO>
__global__ __launch_bounds__(BLAS_BLOCK) void k_convert(BatchView<FI> in, BatchView<FO> out, long n, RhsList rl)
{
    using R = typename FI::real;
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<R> s;
        in.at(rhs).load(h, s);
        out.at(rhs).store(h, s);
    }
}

template <class F>
__global__ __launch_bounds__(BLAS_BLOCK) void k_zero(BatchView<F> v, long n, RhsList rl)
{
    using R = typename F::real;
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<R> s;
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) s.c[i][j] = cx<R>{R(0), R(0)};
        v.at(rhs).store(h, s);
    }
}

// x += alpha p ; r -= alpha ap ; partial |r|^2
template <class FX, class F>
__global__ __launch_bounds__(BLAS_BLOCK) void k_axpy_norm(BatchView<FX> x, BatchView<F> p, BatchView<F> r,
                                                           BatchView<F> ap, long n, RhsList rl,
                                                           const CgScalars *sc, double *partial, long pstride,
                                                           int skip_done)
{
    using R = typename F::real;
    using RX = typename FX::real;
    BLOCK_RHS(rl);
    if (skip_done && sc[rhs].done) return;
    const double alpha = sc[rhs].alpha;
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double part = 0.0;
    if (h < n) {
        spinor<R> ps, rs, as;
        spinor<RX> xs;
        p.at(rhs).load(h, ps);
        r.at(rhs).load(h, rs);
        ap.at(rhs).load(h, as);
        x.at(rhs).load(h, xs);
        const R a = (R)alpha;
        const RX ax = (RX)alpha;
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                xs.c[i][j].re = fmad(ax, (RX)ps.c[i][j].re, xs.c[i][j].re);
                xs.c[i][j].im = fmad(ax, (RX)ps.c[i][j].im, xs.c[i][j].im);
                rs.c[i][j].re = fmad(-a, as.c[i][j].re, rs.c[i][j].re);
                rs.c[i][j].im = fmad(-a, as.c[i][j].im, rs.c[i][j].im);
            }
        x.at(rhs).store(h, xs);
        r.at(rhs).store(h, rs);
        part = (double)site_norm2(rs);
    }
    WRITE_PARTIAL(partial, pstride, part)
}

// out = cu * in on spins 0, 1 and cd * in on spins 2, 3 (a site-local
// a + i b gamma_5, FP64)
__global__ __launch_bounds__(BLAS_BLOCK) void k_twist(BatchView<SpF64> in, BatchView<SpF64> out, long n, RhsList rl,
                                                      double2 cu, double2 cd)
{
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<double> s;
        in.at(rhs).load(h, s);
        const cx<double> u = {cu.x, cu.y}, d = {cd.x, cd.y};
#pragma unroll
        for (int c = 0; c < 3; c++) {
            s.c[0][c] = u * s.c[0][c];
            s.c[1][c] = u * s.c[1][c];
            s.c[2][c] = d * s.c[2][c];
            s.c[3][c] = d * s.c[3][c];
        }
        out.at(rhs).store(h, s);
    }
}

// x += alpha p where pending, then p = r + beta p.  The update of x was in
// the half-sweep that forms r, which read p for it a second time; here p is at
// hand (a CG iteration moves one field less: FP16 52, FP64 192 bytes per site).
template <class FX, class F>
__global__ __launch_bounds__(BLAS_BLOCK) void k_xpay(BatchView<F> r, BatchView<F> p, BatchView<FX> x, long n,
                                                     RhsList rl, const CgScalars *sc, int skip_done, int has_x,
                                                     int only_x)
{
    using R = typename F::real;
    using RX = typename FX::real;
    BLOCK_RHS(rl);
    const bool up_x = has_x && sc[rhs].xpend, up_p = !only_x && !(skip_done && sc[rhs].done);
    if (!up_x && !up_p) return;
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<R> rs, ps;
        p.at(rhs).load(h, ps);
        if (up_p) r.at(rhs).load(h, rs);
        if (up_x) {
            const RX a = (RX)sc[rhs].alpha;
            spinor<RX> xs;
            if (sc[rhs].fresh) {
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int j = 0; j < 3; j++) xs.c[i][j] = cx<RX>{RX(0), RX(0)};
            } else {
                x.at(rhs).load(h, xs);
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    xs.c[i][j].re = fmad(a, (RX)ps.c[i][j].re, xs.c[i][j].re);
                    xs.c[i][j].im = fmad(a, (RX)ps.c[i][j].im, xs.c[i][j].im);
                }
            x.at(rhs).store(h, xs);
        }
        if (up_p) {
            const R b = (R)sc[rhs].beta;
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    ps.c[i][j].re = fmad(b, ps.c[i][j].re, rs.c[i][j].re);
                    ps.c[i][j].im = fmad(b, ps.c[i][j].im, rs.c[i][j].im);
                }
            p.at(rhs).store(h, ps);
        }
    }
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_residual(BatchView<SpF64> b, BatchView<SpF64> ax,
                                                         BatchView<SpF64> r, long n, RhsList rl, double *partial,
                                                         long pstride)
{
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double part = 0.0;
    if (h < n) {
        spinor<double> bs, as;
        b.at(rhs).load(h, bs);
        ax.at(rhs).load(h, as);
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) bs.c[i][j] = bs.c[i][j] - as.c[i][j];
        r.at(rhs).store(h, bs);
        part = site_norm2(bs);
    }
    WRITE_PARTIAL(partial, pstride, part)
}

// x += xs, xs completed by its pending alpha p on the way (not stored: it is
// fresh after this).  What counts as zero is not read.
template <class F>
__global__ __launch_bounds__(BLAS_BLOCK) void k_accumulate(BatchView<SpF64> x, BatchView<SpF32> xs, BatchView<F> p,
                                                           long n, RhsList rl, const CgScalars *sc)
{
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<double> a;
        spinor<float> d, ps;
        if (sc[rhs].reliable) {
            x.at(rhs).load(h, a);
        } else {
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) a.c[i][j] = cx<double>{0.0, 0.0};
        }
        if (sc[rhs].fresh) {
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) d.c[i][j] = cx<float>{0.f, 0.f};
        } else {
            xs.at(rhs).load(h, d);
        }
        if (sc[rhs].xpend) {
            const float al = (float)sc[rhs].alpha;
            p.at(rhs).load(h, ps);
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    d.c[i][j].re = fmad(al, ps.c[i][j].re, d.c[i][j].re);
                    d.c[i][j].im = fmad(al, ps.c[i][j].im, d.c[i][j].im);
                }
        }
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                a.c[i][j].re += (double)d.c[i][j].re;
                a.c[i][j].im += (double)d.c[i][j].im;
            }
        x.at(rhs).store(h, a);
    }
}

__global__ __launch_bounds__(BLAS_BLOCK) void k_add(BatchView<SpF64> x, BatchView<SpF64> d, long n, RhsList rl)
{
    BLOCK_RHS(rl);
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    if (h < n) {
        spinor<double> a, b;
        x.at(rhs).load(h, a);
        d.at(rhs).load(h, b);
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) a.c[i][j] = a.c[i][j] + b.c[i][j];
        x.at(rhs).store(h, a);
    }
}

// b, r and p of a new right-hand side from its canonical source, with |b|^2:
// one pass instead of a conversion, three copies and a norm of their own
template <class F>
__global__ __launch_bounds__(BLAS_BLOCK) void k_join(const double2 *src, SpF64 b, F r, F p, long n, double *partial)
{
    constexpr int rhs = 0;
    const long h = (long)blockIdx.x * BLAS_BLOCK + threadIdx.x;
    double part = 0.0;
    if (h < n) {
        spinor<double> s;
        const double2 *q = src + h * 12;
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const double2 v = q[k];
            s.c[k / 3][k % 3] = cx<double>{v.x, v.y};
        }
        b.store(h, s);
        r.store(h, s);
        if constexpr (F::coded) {  // p is a copy of the stored r
            spinor<float> t;
            r.load(h, t);
            p.store(h, t);
        } else {
            p.store(h, s);
        }
        part = site_norm2(s);
    }
    WRITE_PARTIAL(partial, 0, part)
}

// ------------------------------------------------------------- scalars

constexpr int SC_THREADS = 1024;

// the wavefronts' sums of n blocks: a block's in the order of its wavefronts
// (as block_sum), the blocks in a fixed order
__device__ __forceinline__ double det_sum(const double *partial, int n, double *sh)
{
    static_assert(PARTS == 4, "a block's partial sums are two 16-byte words");
    double v = 0.0;
    constexpr int U = 4;  // loads asked for together
    for (int i = threadIdx.x; i < n; i += U * SC_THREADS) {
        double2 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int k = min(i + u * SC_THREADS, n - 1);
            a[u] = ((const double2 *)partial)[2 * k];
            b[u] = ((const double2 *)partial)[2 * k + 1];
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (i + u * SC_THREADS < n) v += (((0.0 + a[u].x) + a[u].y) + b[u].x) + b[u].y;
    }
    return block_sum_n<SC_THREADS / 64>(v, sh);  // valid in thread 0
}

// two such sums over n <= SC_THREADS blocks, their loads together (sh: twice the room)
__device__ __forceinline__ double2 det_sum2(const double *pa, const double *pb, int n, double *sh)
{
    double a = 0.0, b = 0.0;
    if ((int)threadIdx.x < n) {
        const double2 *qa = (const double2 *)pa + 2 * threadIdx.x, *qb = (const double2 *)pb + 2 * threadIdx.x;
        const double2 a0 = qa[0], a1 = qa[1], b0 = qb[0], b1 = qb[1];
        a += (((0.0 + a0.x) + a0.y) + a1.x) + a1.y;
        b += (((0.0 + b0.x) + b0.y) + b1.x) + b1.y;
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if ((threadIdx.x & 63) == 0) {
        sh[2 * (threadIdx.x >> 6)] = a;
        sh[2 * (threadIdx.x >> 6) + 1] = b;
    }
    __syncthreads();
    double2 s = make_double2(0.0, 0.0);
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < SC_THREADS / 64; i++) {
            s.x += sh[2 * i];
            s.y += sh[2 * i + 1];
        }
    return s;  // valid in thread 0
}

__device__ __forceinline__ int finite(double v) { return isfinite(v) ? 1 : 0; }

// one block per RHS of rl (grid x); PAP: SC_ALPHA_BETA
template <bool PAP>
__global__ __launch_bounds__(SC_THREADS) void k_scalar(int op, RhsList rl, const double *partial, long pstride,
                                                       int nparts, CgScalars *sc, double tol2, int relative,
                                                       int skip_done, int defer, CgScalars *publish,
                                                       const double *pap)
{
    const int rhs = rl.idx[blockIdx.x];
    // (the scalars are read ahead of the sum and written back whole)
    CgScalars c = sc[rhs], *s = &c;
    if ((PAP || op == SC_BETA) && s->xpend) {
        s->fresh = 0;
        s->xpend = 0;
    }
    if (skip_done && s->done) {
        if (threadIdx.x == 0) {
            sc[rhs] = c;
            if (publish) publish[rhs] = c;
        }
        return;
    }
    __shared__ double sh[(PAP ? 2 : 1) * SC_THREADS / 64];
    double sum;
    if constexpr (PAP) {
        const double2 w = det_sum2(pap + rhs * pstride, partial + rhs * pstride, nparts, sh);
        s->pAp = w.x;
        s->alpha = s->rr / w.x;
        if (!finite(s->alpha)) {  // (the half-sweep did nothing)
            s->nan = 1, s->done = 1;
            op = -1;
        } else {
            op = SC_BETA;
        }
        sum = w.y;
    } else {
        sum = det_sum(partial + rhs * pstride, nparts, sh);
    }
    if (threadIdx.x != 0) return;
    switch (op) {
    case SC_INIT:  // sum = ||b||^2 = ||r_0||^2 (x_0 = 0)
        s->bb = sum;
        s->rr = s->rr_prev = sum;
        s->target = tol2 * (relative ? sum : 1.0);
        s->alpha = s->beta = s->pAp = 0.0;
        s->iter = 0;
        s->reliable = 0;
        s->xpend = 0;
        s->fresh = defer;
        s->last_true = 1;
        s->nan = !finite(sum);
        s->done = (sum < s->target || sum == 0.0 || s->nan) ? 1 : 0;
        break;
    case SC_ALPHA:  // sum = <p, A p>
        s->pAp = sum;
        s->alpha = s->rr / sum;
        if (!finite(s->alpha)) s->nan = 1, s->done = 1;
        break;
    case SC_BETA:  // sum = ||r||^2 of the updated iterated residual
        s->rr_prev = s->rr;
        s->rr = sum;
        s->beta = sum / s->rr_prev;
        s->iter += 1;
        s->last_true = 0;
        s->xpend = defer;
        if (!finite(sum) || !finite(s->beta)) s->nan = 1;
        s->done = (sum < s->target || s->nan) ? 1 : 0;
        break;
    case SC_RELIABLE:  // sum = ||b - A x||^2 recomputed in FP64; replaces the iterated residual
        s->rr = sum;
        s->beta = s->rr_prev > 0.0 ? sum / s->rr_prev : 0.0;
        s->reliable += 1;
        s->last_true = 1;
        s->xpend = 0;
        s->fresh = defer;
        if (!finite(sum)) s->nan = 1;
        s->done = (sum < s->target || sum == 0.0 || s->nan) ? 1 : 0;
        break;
    }
    sc[rhs] = c;
    if (publish) publish[rhs] = c;
}

// the pending update of x has been applied: x holds it (one lane per RHS)
__global__ __launch_bounds__(MAX_RHS) void k_x_applied(RhsList rl, CgScalars *sc)
{
    if ((int)threadIdx.x >= rl.n) return;
    CgScalars &s = sc[rl.idx[threadIdx.x]];
    if (s.xpend) {
        s.xpend = 0;
        s.fresh = 0;
    }
}

// out[i] = the sum of RHS rl.idx[i]
__global__ __launch_bounds__(SC_THREADS) void k_sums(RhsList rl, const double *partial, long pstride, int nparts,
                                                     double *out)
{
    __shared__ double sh[SC_THREADS / 64];
    const double sum = det_sum(partial + rl.idx[blockIdx.x] * pstride, nparts, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = sum;
}

constexpr int SUM_THREADS = 1024;

__global__ __launch_bounds__(SUM_THREADS) void k_max(const double *partial, int n, double *out)
{
    __shared__ double sh[SUM_THREADS / 64];
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += SUM_THREADS) v = fmax(v, partial[i]);
    const double m = block_max(v, sh);
    if (threadIdx.x == 0) *out = m;
}

// plain streaming copy, 16 bytes per lane, for bandwidth calibration
__global__ __launch_bounds__(256) void k_stream_copy(const float4 *__restrict__ a, float4 *__restrict__ b, long n)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) b[i] = a[i];
}

// ------------------------------------------------------------- dispatch

#define DISPATCH_SP TMQ_DISPATCH_SP

static dim3 grid2(long n, const RhsList &rl) { return dim3((unsigned)blas_grid(n), (unsigned)rl.n); }

#define LAUNCH(KERNEL, NSITES, RL, STREAM, ...)                                                          \
    do {                                                                                                  \
        if ((RL).n > 0 && (NSITES) > 0)                                                                   \
            hipLaunchKernelGGL(KERNEL, grid2(NSITES, RL), dim3(BLAS_BLOCK), 0, STREAM, __VA_ARGS__);      \
    } while (0)

hipError_t launch_norm2(const FieldDesc &v, const RhsList &rl, double *partial, long pstride, hipStream_t st)
{
    DISPATCH_SP(v.prec, F, LAUNCH(k_norm2<F>, v.n, rl, st, make_bv<F>(v), v.n, rl, partial, pstride));
    return hipGetLastError();
}

hipError_t launch_zero(const FieldDesc &v, const RhsList &rl, hipStream_t st)
{
    DISPATCH_SP(v.prec, F, LAUNCH(k_zero<F>, v.n, rl, st, make_bv<F>(v), v.n, rl));
    return hipGetLastError();
}

hipError_t launch_twist(const FieldDesc &in, const FieldDesc &out, const RhsList &rl, double2 cu, double2 cd,
                        hipStream_t st)
{
    if (in.prec != P64 || out.prec != P64 || in.n != out.n) return hipErrorInvalidValue;
    LAUNCH(k_twist, in.n, rl, st, make_bv<SpF64>(in), make_bv<SpF64>(out), in.n, rl, cu, cd);
    return hipGetLastError();
}

hipError_t launch_convert(const FieldDesc &in, const FieldDesc &out, const RhsList &rl, hipStream_t st)
{
    if (in.n != out.n) return hipErrorInvalidValue;
    DISPATCH_SP(in.prec, FI,
                DISPATCH_SP(out.prec, FO,
                            LAUNCH((k_convert<FI, FO>), in.n, rl, st, make_bv<FI>(in), make_bv<FO>(out), in.n, rl)));
    return hipGetLastError();
}

hipError_t launch_axpy_norm(const FieldDesc &x, const FieldDesc &p, const FieldDesc &r, const FieldDesc &ap,
                            const RhsList &rl, const CgScalars *s, double *partial, long pstride, bool skip_done,
                            hipStream_t st)
{
    if (p.prec != r.prec || p.prec != ap.prec) return hipErrorInvalidValue;
    const long n = p.n;
    const int sk = skip_done ? 1 : 0;
    if (x.prec == P64 && p.prec == P64)
        LAUNCH((k_axpy_norm<SpF64, SpF64>), n, rl, st, make_bv<SpF64>(x), make_bv<SpF64>(p), make_bv<SpF64>(r),
               make_bv<SpF64>(ap), n, rl, s, partial, pstride, sk);
    else if (x.prec == P32) {
        DISPATCH_SP(p.prec, F,
                    LAUNCH((k_axpy_norm<SpF32, F>), n, rl, st, make_bv<SpF32>(x), make_bv<F>(p), make_bv<F>(r),
                           make_bv<F>(ap), n, rl, s, partial, pstride, sk));
    } else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_xpay(const FieldDesc &r, const FieldDesc &p, const FieldDesc &x, const RhsList &rl,
                       const CgScalars *s, bool skip_done, bool only_x, hipStream_t st)
{
    const int hx = x.data ? 1 : 0, sk = skip_done ? 1 : 0, ox = only_x ? 1 : 0;
    if (r.prec != p.prec || (hx && x.prec != (p.prec == P64 ? P64 : P32))) return hipErrorInvalidValue;
    if (p.prec == P64) {
        LAUNCH((k_xpay<SpF64, SpF64>), p.n, rl, st, make_bv<SpF64>(r), make_bv<SpF64>(p), make_bv<SpF64>(x), p.n, rl,
               s, sk, hx, ox);
        return hipGetLastError();
    }
    DISPATCH_SP(p.prec, F,
                LAUNCH((k_xpay<SpF32, F>), p.n, rl, st, make_bv<F>(r), make_bv<F>(p), make_bv<SpF32>(x), p.n, rl, s, sk,
                       hx, ox));
    return hipGetLastError();
}

hipError_t launch_residual(const FieldDesc &b, const FieldDesc &ax, const FieldDesc &r, const RhsList &rl,
                           double *partial, long pstride, hipStream_t st)
{
    if (b.prec != P64 || ax.prec != P64 || r.prec != P64) return hipErrorInvalidValue;
    LAUNCH(k_residual, b.n, rl, st, make_bv<SpF64>(b), make_bv<SpF64>(ax), make_bv<SpF64>(r), b.n, rl, partial,
           pstride);
    return hipGetLastError();
}

hipError_t launch_accumulate(const FieldDesc &x64, const FieldDesc &xs, const FieldDesc &p, const RhsList &rl,
                             const CgScalars *s, hipStream_t st)
{
    if (x64.prec != P64 || xs.prec != P32 || p.prec == P64) return hipErrorInvalidValue;
    DISPATCH_SP(p.prec, F,
                LAUNCH(k_accumulate<F>, x64.n, rl, st, make_bv<SpF64>(x64), make_bv<SpF32>(xs), make_bv<F>(p), x64.n,
                       rl, s));
    return hipGetLastError();
}

hipError_t launch_add(const FieldDesc &x, const FieldDesc &d, const RhsList &rl, hipStream_t st)
{
    if (x.prec != P64 || d.prec != P64 || x.n != d.n) return hipErrorInvalidValue;
    LAUNCH(k_add, x.n, rl, st, make_bv<SpF64>(x), make_bv<SpF64>(d), x.n, rl);
    return hipGetLastError();
}

hipError_t launch_join(const double2 *src, const FieldDesc &b, const FieldDesc &r, const FieldDesc &p, double *partial,
                       hipStream_t st)
{
    if (b.prec != P64 || r.prec != p.prec || r.n != b.n || p.n != b.n) return hipErrorInvalidValue;
    DISPATCH_SP(r.prec, F,
                hipLaunchKernelGGL(k_join<F>, dim3(blas_grid(b.n)), dim3(BLAS_BLOCK), 0, st, src, make_sp<SpF64>(b),
                                   make_sp<F>(r), make_sp<F>(p), b.n, partial));
    return hipGetLastError();
}

hipError_t launch_scalar(int op, const RhsList &rl, const double *partial, long pstride, int nparts,
                         CgScalars *s, double tol2, int relative, bool skip_done, bool defer,
                         CgScalars *publish, hipStream_t st, const double *pap)
{
    if (rl.n <= 0) return hipSuccess;
    if (op == SC_ALPHA_BETA && (!pap || nparts > SC_THREADS)) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(rl.n), dim3(SC_THREADS), 0, st, op, rl, partial, pstride, nparts, s, tol2,
                           relative, skip_done ? 1 : 0, defer ? 1 : 0, publish, pap);
    };
    if (op == SC_ALPHA_BETA)
        go(k_scalar<true>);
    else
        go(k_scalar<false>);
    return hipGetLastError();
}

hipError_t launch_x_applied(const RhsList &rl, CgScalars *s, hipStream_t st)
{
    if (rl.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_x_applied, dim3(1), dim3(MAX_RHS), 0, st, rl, s);
    return hipGetLastError();
}

hipError_t launch_sums(const RhsList &rl, const double *partial, long pstride, int nparts, double *out, hipStream_t st)
{
    if (rl.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sums, dim3(rl.n), dim3(SC_THREADS), 0, st, rl, partial, pstride, nparts, out);
    return hipGetLastError();
}

hipError_t launch_max(const double *partial, int n, double *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_max, dim3(1), dim3(SUM_THREADS), 0, st, partial, n, out);
    return hipGetLastError();
}

hipError_t launch_stream_copy(const void *src, void *dst, size_t bytes, hipStream_t st)
{
    const long n = (long)(bytes / 16);
    hipLaunchKernelGGL(k_stream_copy, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const float4 *)src,
                       (float4 *)dst, n);
    return hipGetLastError();
}

FieldDesc field_sub(const FieldDesc &f, long off, long n)
{
    FieldDesc o = f;
    o.data = (char *)f.data + off * (long)field_blocks(f.prec) * (long)field_elem_bytes(f.prec);
    o.scale = f.scale ? f.scale + off : nullptr;
    o.n = n;
    return o;
}

FieldDesc field_rhs(const FieldDesc &f, int r)
{
    FieldDesc o = f;
    o.data = (char *)f.data + (long)r * f.rhs_elems * (long)field_elem_bytes(f.prec);
    o.scale = f.scale ? f.scale + (long)r * f.rhs_sites : nullptr;
    o.nrhs = 1;
    return o;
}

size_t field_elem_bytes(int) { return 16; }  // double2, float4, uint4
int field_blocks(int prec) { return prec == P64 ? 12 : prec == P32 ? 6 : 3; }

}  // namespace tmq
