// small_cg.hip -- the whole full-lattice CG of a tiny lattice in one launch.
//
// On a lattice of a few hundred sites every kernel of a CG iteration is a
// handful of wavefronts, and the iteration costs what the GPU needs to start
// its nine dependent kernels (about 5 us each).  Here one launch runs textbook
// CG on Q^+ Q^- (Sec. 4.4, eq. (eo1) on both parities) from start to finish.
//
// A block of eight wavefronts owns 64 sites of the stacked lattice, as in the
// split half-sweep (hop_split.h): wavefront W forms hop W of its sites, whose
// link it keeps in registers for the whole solve, and wavefronts 0 .. 5 each
// sum, and own in registers, two complex components of x, r and p.  The
// neighbours' r, p and t pass through global memory, and an iteration has two
// grid barriers, which carry the inner products: t = Q^- p with |t|^2, then
// A p = Q^+ t with the update and |r|^2.  The new search direction p = r +
// beta p is formed by whoever reads it, from the r and the previous p of the
// site.  Sums run in a fixed order, the same in every block, so that all take
// the same decisions and results are reproducible.
//
// What bounds it: the latency of the chain neighbour load -> hop -> LDS -> sum
// -> store -> barrier, twice per iteration.  One workgroup of 256 lanes with
// all eight hops of a site in a lane, which this replaces, took 16 us per
// iteration at 4^4 (1.73 ms for 107, here 0.87) and four times that at 1024
// sites (here 10).  Passing the vectors as device-scope atomics (8 bytes at a
// time, past the L2), without the fences of the exchange, took 11.6 us.
//
// After the iterated residual meets the target the kernel recomputes the
// true residual b - A x and leaves the decision to the host, which calls it
// again (CG restarted from the true residual) if the true residual has not
// met the target.
#include <type_traits>

#include "devutil.h"
#include "views.h"

namespace tmq {

constexpr int SMALL_SITES = 64, SMALL_THREADS = 512;
constexpr int SMALL_BLOCKS = (int)(SMALL_CG_MAX_SITES / SMALL_SITES);
constexpr int SMALL_UNITS = 6;  // wavefronts that own components, two each
static_assert(SMALL_BLOCKS < 64, "a wavefront polls the slots of every block and the abort word");
static_assert(3 * SMALL_BLOCKS + 1 <= SMALL_SYNC_WORDS, "slots of three exchanges and the abort word");

template <class LK>
struct SmallCgArgs {
    Geom g;
    SpF64 b, x, r, t, p[2];  // stacked (even, odd) full-lattice fields
    LK lk;
    double ph[4][2];
    int phase_mask;
    double kappa, mut, tol2;
    int relative, max_iter;
    CgScalars *sc;             // in/out: counters and residuals across calls
    unsigned long long *sync;  // SMALL_SYNC_WORDS words, all ones at the start
    long long spin;            // clock ticks a block waits for the others
};

namespace {

constexpr unsigned long long SMALL_EMPTY = ~0ull;

struct SmallShared {
    double2 sh[8][6][SMALL_SITES];  // half spinors of the hops
    double red[SMALL_UNITS];
    double sum[2];
    int fail;
};

// Every block passes its v on and waits for those of all blocks: a grid
// barrier that returns their sum (in the order of the blocks).  Exchange k
// uses the slots k % 3; a block empties its slot of exchange k + 1 before it
// fills that of k (a block that has filled k - 1 has read all of k - 2, which
// used the same slot).  What the block stored before is visible to every block
// after it.  Waits are bounded: a block that has waited `spin` ticks, or sees
// that another has, gives up, and so do all others; returns false then.
template <class LK>
__device__ __forceinline__ bool small_exchange(const SmallCgArgs<LK> &a, SmallShared &S, int W, int lane, int k,
                                               double v, double *sum)
{
    // this wavefront's stores are in the L2
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    v = wave_sum(v);
    if (W < SMALL_UNITS && lane == 0) S.red[W] = v;
    __syncthreads();
    if (W == 0) {
        const int nb = gridDim.x, b = blockIdx.x;
        unsigned long long *slot = a.sync + (k % 3) * SMALL_BLOCKS, *abort = a.sync + 3 * SMALL_BLOCKS;
        if (lane == 0) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < SMALL_UNITS; q++) s += S.red[q];
            unsigned long long bits = (unsigned long long)__double_as_longlong(s);
            if (bits == SMALL_EMPTY) bits ^= 1;  // another NaN
            __hip_atomic_store(a.sync + ((k + 1) % 3) * SMALL_BLOCKS + b, SMALL_EMPTY, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(slot + b, bits, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        }
        // lane i < nb waits for block i, the last lane looks at the abort word
        unsigned long long got;
        bool fail = false;
        const long long t0 = wall_clock64();
        while (true) {
            got = lane < nb || lane == 63 ? __hip_atomic_load(lane == 63 ? abort : slot + lane, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT)
                                          : 0ull;
            if (__ballot(lane < nb && got == SMALL_EMPTY) == 0) break;
            fail = __ballot(lane == 63 && got != SMALL_EMPTY) != 0 || wall_clock64() - t0 > a.spin;
            if (fail) {
                if (lane == 0) __hip_atomic_store(abort, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        double s = 0.0;
        const double d = __longlong_as_double((long long)got);
        for (int i = 0; i < nb; i++) s += __shfl(d, i, 64);
        if (lane == 0) {
            S.sum[k & 1] = s;
            S.fail = fail;
        }
    }
    __syncthreads();
    *sum = S.sum[k & 1];
    return !S.fail;
}

// spin I of hop (MU, S) rebuilt from the half spinors of the hop and added
// (reconstruct_add of spin.h, one component)
template <int K, int J>
__device__ __forceinline__ void small_add(const SmallShared &S, int lane, cx<double> &acc)
{
    constexpr int I = K / 3, A = K % 3, MU = J >> 1, SG = (J & 1) == 0 ? +1 : -1;
    constexpr int row = I < 2 ? I : (MU == 0 || MU == 3) ? I - 2 : 3 - I;
    const double2 v = S.sh[J][row * 3 + A][lane];
    const cx<double> h = {v.x, v.y};
    if (I < 2)
        acc = acc + h;
    else if (MU == 0)
        acc = SG > 0 ? acc - h : acc + h;
    else if (MU == 1)
        acc = acc + (SG > 0 ? ipl(h) : imi(h));
    else if (MU == 2)
        acc = (SG > 0) == (I == 2) ? acc + h : acc - h;
    else
        acc = acc + ((SG > 0) == (I == 2) ? ipl(h) : imi(h));
}

// what wavefront W's lane knows of its site: stacked index s, neighbour sn, the link of its hop
template <class LK>
struct SmallSite {
    bool active;
    long s, sn;
    typename LK::Loaded u;
};

// the two components of out = g5 [(1 + sign i mut g5) v - kappa H in] that
// wavefront W owns, v its own components of in; `in` gives the neighbour's
// spinor.  Ends with the block's reads of LDS done by its own wavefront only:
// an exchange has to follow.
template <int W, class LK, class IN>
__device__ __forceinline__ void small_q(const SmallCgArgs<LK> &a, SmallShared &S, const SmallSite<LK> &p, int lane,
                                        int sign, const cx<double> (&v)[2], cx<double> (&o)[2], IN in)
{
    constexpr int MU = W >> 1;
    constexpr bool BACK = W & 1;
    if (p.active) {
        spinor<double> nb;
        in(p.sn, nb);
        half<double> h, w;
        project<MU, BACK ? -1 : +1>(nb, h);
        a.lk.template apply<BACK>(p.u, h, w);
        if ((a.phase_mask >> MU) & 1) {
            const cx<double> ph = {a.ph[MU][0], a.ph[MU][1]};
            half_scale(w, BACK ? conj(ph) : ph);
        }
#pragma unroll
        for (int c = 0; c < 6; c++) S.sh[W][c][lane] = make_double2(w.c[c / 3][c % 3].re, w.c[c / 3][c % 3].im);
    }
    __syncthreads();
    if constexpr (W < SMALL_UNITS) {
        const double m = sign * a.mut;
        auto comp = [&](auto nc) {
            constexpr int N = decltype(nc)::value, K = 2 * W + N;
            cx<double> acc = {0.0, 0.0};
            small_add<K, 0>(S, lane, acc);
            small_add<K, 1>(S, lane, acc);
            small_add<K, 2>(S, lane, acc);
            small_add<K, 3>(S, lane, acc);
            small_add<K, 4>(S, lane, acc);
            small_add<K, 5>(S, lane, acc);
            small_add<K, 6>(S, lane, acc);
            small_add<K, 7>(S, lane, acc);
            const cx<double> A = {K < 6 ? 1.0 : -1.0, m}, B = {K < 6 ? -a.kappa : a.kappa, 0.0};
            o[N] = fma(A, v[N], B * acc);
        };
        if (p.active) {
            comp(std::integral_constant<int, 0>{});
            comp(std::integral_constant<int, 1>{});
        }
    }
}

__device__ __forceinline__ double norm2_of(const cx<double> (&v)[2])
{
    return fmad(v[0].re, v[0].re, fmad(v[0].im, v[0].im, fmad(v[1].re, v[1].re, v[1].im * v[1].im)));
}
__device__ __forceinline__ void load2(const SpF64 &f, long s, int W, cx<double> (&v)[2])
{
    const double2 *q = f.p + aidx(s, 2 * W, 12);
    const double2 a = q[0], b = q[8];
    v[0] = {a.x, a.y}, v[1] = {b.x, b.y};
}
__device__ __forceinline__ void store2(const SpF64 &f, long s, int W, const cx<double> (&v)[2])
{
    double2 *q = f.p + aidx(s, 2 * W, 12);
    q[0] = make_double2(v[0].re, v[0].im);
    q[8] = make_double2(v[1].re, v[1].im);
}

template <int W, class LK>
__device__ __forceinline__ void small_cg_role(const SmallCgArgs<LK> &a, SmallShared &S, int lane)
{
    constexpr int MU = W >> 1;
    constexpr bool BACK = W & 1, UNIT = W < SMALL_UNITS;
    const Geom &g = a.g;
    SmallSite<LK> p;
    p.s = (long)blockIdx.x * SMALL_SITES + lane;
    p.active = p.s < 2 * g.vh;
    p.sn = 0;
    const bool own = UNIT && p.active;
    if (p.active) {
        const int par = p.s >= g.vh ? 1 : 0;
        const long h = p.s - par * g.vh;
        const unsigned hu = (unsigned)h;
        const unsigned xh = hu % (unsigned)g.XH;
        unsigned rr = hu / (unsigned)g.XH;
        const int y = (int)(rr % (unsigned)g.LY);
        rr /= (unsigned)g.LY;
        const int z = (int)(rr % (unsigned)g.LZ);
        const int t = (int)(rr / (unsigned)g.LZ);
        const int x = 2 * (int)xh + ((par + t + z + y) & 1);
        const long row = h - xh, sy = g.XH, sz = (long)g.LY * g.XH, stt = (long)g.LZ * sz;
        long hn;
        if (MU == 0)
            hn = BACK ? (t == 0 ? h + (g.T - 1) * stt : h - stt) : (t + 1 == g.T ? h - (g.T - 1) * stt : h + stt);
        else if (MU == 1)
            hn = row + ((BACK ? (x == 0 ? g.LX - 1 : x - 1) : (x + 1 == g.LX ? 0 : x + 1)) >> 1);
        else if (MU == 2)
            hn = BACK ? (y == 0 ? h + (g.LY - 1) * sy : h - sy) : (y + 1 == g.LY ? h - (g.LY - 1) * sy : h + sy);
        else
            hn = BACK ? (z == 0 ? h + (g.LZ - 1) * sz : h - sz) : (z + 1 == g.LZ ? h - (g.LZ - 1) * sz : h + sz);
        a.lk.template load_link<false>(BACK ? par ^ 1 : par, MU, BACK ? hn : h, p.u);
        p.sn = (1 - par) * g.vh + hn;
    }
    CgScalars C = *a.sc;
    int k = 0;
    double rr = 0.0, sum = 0.0;
    bool ok = true;
    cx<double> b[2], x[2], r[2], pp[2], v[2], o[2];
    if (own) {
        load2(a.b, p.s, W, b);
        load2(a.x, p.s, W, x);
    }
    auto from = [&](const SpF64 &f) { return [&f](long s, spinor<double> &q) { f.load(s, q); }; };
    // v = Q^- (field f, own components fv), exchanged through t with the sum of |v|^2, then o = Q^+ v
    auto apply_a = [&](auto in, const cx<double>(&fv)[2]) {
        small_q<W>(a, S, p, lane, -1, fv, v, in);
        if (own) store2(a.t, p.s, W, v);
        ok = small_exchange(a, S, W, lane, k++, own ? norm2_of(v) : 0.0, &sum);
    };
    // r = b - A x (x as left by the previous call, zero at the start), p = r
    const bool first = C.iter == 0 && C.reliable == 0;
    if (first) {
#pragma unroll
        for (int n = 0; n < 2; n++) r[n] = b[n];
    } else {
        apply_a(from(a.x), x);
        if (ok) small_q<W>(a, S, p, lane, +1, v, o, from(a.t));
#pragma unroll
        for (int n = 0; n < 2; n++) r[n] = b[n] - o[n];
    }
    const cx<double> zero[2] = {{0.0, 0.0}, {0.0, 0.0}};
    pp[0] = pp[1] = {0.0, 0.0};
    if (own) {
        store2(a.r, p.s, W, r);
        store2(a.p[0], p.s, W, zero);
    }
    if (ok) ok = small_exchange(a, S, W, lane, k++, own ? norm2_of(r) : 0.0, &rr);
    if (first) {
        C.bb = rr;
        C.target = a.tol2 * (a.relative ? rr : 1.0);
    }
    bool nan = !isfinite(rr);
    double beta = 0.0;
    int cur = 0;  // p[cur]: the previous search direction
    // CG from r (Sec. 4.4): alpha = rr / |Q^- p|^2, x += alpha p, r -= alpha A p, beta = rr' / rr
    while (ok && !nan && rr >= C.target && rr > 0.0 && C.iter < a.max_iter) {
        const SpF64 &pold = a.p[cur], &pnew = a.p[cur ^ 1];
        if (own) {
#pragma unroll
            for (int n = 0; n < 2; n++) {
                pp[n].re = fmad(beta, pp[n].re, r[n].re);
                pp[n].im = fmad(beta, pp[n].im, r[n].im);
            }
            store2(pnew, p.s, W, pp);
        }
        apply_a(
            [&](long s, spinor<double> &q) {
                spinor<double> w;
                a.r.load(s, q);
                pold.load(s, w);
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int c = 0; c < 3; c++) {
                        q.c[i][c].re = fmad(beta, w.c[i][c].re, q.c[i][c].re);
                        q.c[i][c].im = fmad(beta, w.c[i][c].im, q.c[i][c].im);
                    }
            },
            pp);
        if (!ok) break;
        const double alpha = rr / sum;
        small_q<W>(a, S, p, lane, +1, v, o, from(a.t));
        if (own) {
#pragma unroll
            for (int n = 0; n < 2; n++) {
                x[n].re = fmad(alpha, pp[n].re, x[n].re);
                x[n].im = fmad(alpha, pp[n].im, x[n].im);
                r[n].re = fmad(-alpha, o[n].re, r[n].re);
                r[n].im = fmad(-alpha, o[n].im, r[n].im);
            }
            store2(a.r, p.s, W, r);
        }
        double rr_new;
        ok = small_exchange(a, S, W, lane, k++, own ? norm2_of(r) : 0.0, &rr_new);
        if (!ok) break;
        beta = rr_new / rr;
        rr = rr_new;
        C.iter += 1;
        nan = !isfinite(rr) || !isfinite(alpha) || !isfinite(beta);
        cur ^= 1;
    }
    // the true residual b - A x
    if (own) store2(a.x, p.s, W, x);
    if (ok) ok = small_exchange(a, S, W, lane, k++, 0.0, &sum);
    if (ok) apply_a(from(a.x), x);
    double rt = 0.0;
    if (ok) {
        small_q<W>(a, S, p, lane, +1, v, o, from(a.t));
#pragma unroll
        for (int n = 0; n < 2; n++) r[n] = b[n] - o[n];
        ok = small_exchange(a, S, W, lane, k++, own ? norm2_of(r) : 0.0, &rt);
    }
    if (W == 0 && lane == 0 && (blockIdx.x == 0 || !ok)) {
        if (!ok) {
            a.sc->pad = 1;  // (any block that gave up; nothing else of the scalars is written then)
        } else {
            C.rr = rt;
            C.reliable += 1;
            C.last_true = 1;
            C.nan = (nan || !isfinite(rt)) ? 1 : 0;
            C.done = (C.nan || rt < C.target || rt == 0.0) ? 1 : 0;
            C.pad = 0;
            *a.sc = C;
        }
    }
}

}  // namespace

template <class LK>
__global__ __launch_bounds__(SMALL_THREADS) void k_small_cg(SmallCgArgs<LK> a)
{
    __shared__ SmallShared S;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // (the eight roles run through the same barriers)
    switch (w) {
    case 0: small_cg_role<0>(a, S, lane); break;
    case 1: small_cg_role<1>(a, S, lane); break;
    case 2: small_cg_role<2>(a, S, lane); break;
    case 3: small_cg_role<3>(a, S, lane); break;
    case 4: small_cg_role<4>(a, S, lane); break;
    case 5: small_cg_role<5>(a, S, lane); break;
    case 6: small_cg_role<6>(a, S, lane); break;
    default: small_cg_role<7>(a, S, lane); break;
    }
}

template <class LK>
static hipError_t go_small(const Geom &g, const FieldDesc *f, const LinkDesc &lk, const OpParams &op, double tol2,
                           int relative, int max_iter, CgScalars *sc, unsigned long long *sync, long long spin,
                           hipStream_t st)
{
    SmallCgArgs<LK> a;
    a.g = g;
    a.b = make_sp<SpF64>(f[0]);
    a.x = make_sp<SpF64>(f[1]);
    a.r = make_sp<SpF64>(f[2]);
    a.p[0] = make_sp<SpF64>(f[3]);
    a.p[1] = make_sp<SpF64>(f[5]);
    a.t = make_sp<SpF64>(f[4]);
    a.lk = make_lk<LK>(lk);
    for (int mu = 0; mu < 4; mu++) a.ph[mu][0] = op.ph[mu][0], a.ph[mu][1] = op.ph[mu][1];
    a.phase_mask = hop_phase_mask(op);
    a.kappa = op.kappa[0];
    a.mut = op.mut[0];
    a.tol2 = tol2;
    a.relative = relative;
    a.max_iter = max_iter;
    a.sc = sc;
    a.sync = sync;
    a.spin = spin;
    const int blocks = (int)((2 * g.vh + SMALL_SITES - 1) / SMALL_SITES);
    const hipError_t e = hipMemsetAsync(sync, 0xFF, sizeof(unsigned long long) * SMALL_SYNC_WORDS, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_small_cg<LK>, dim3(blocks), dim3(SMALL_THREADS), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_small_cg(const Geom &g, const FieldDesc *f, const LinkDesc &lk, const OpParams &op, double tol2,
                           int relative, int max_iter, CgScalars *sc, unsigned long long *sync, long long spin,
                           hipStream_t st)
{
    if (2 * g.vh > SMALL_CG_MAX_SITES) return hipErrorInvalidValue;
    for (int i = 0; i < 6; i++)
        if (f[i].prec != P64 || f[i].n != 2 * g.vh) return hipErrorInvalidValue;
    if (lk.fmt == LK64R) return go_small<L64R>(g, f, lk, op, tol2, relative, max_iter, sc, sync, spin, st);
    if (lk.fmt == LK64F) return go_small<L64F>(g, f, lk, op, tol2, relative, max_iter, sc, sync, spin, st);
    return hipErrorInvalidValue;
}

}  // namespace tmq
