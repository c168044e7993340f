// hop_split_nd.h -- the split half-sweep of one flavour doublet (FP64 and FP32).
//
// As hop_split_kernel, with both flavours of a site in the same block: a
// wavefront loads the link of its hop once and forms the hop of the upper
// flavour, then of the lower one, through the same LDS; the units hold the two
// hop sums of their components, mix them by the doublet's site terms (nd_mix
// in hop_impl.h, operation by operation) and store both.  The sums of |out|^2
// are those of hop_kernel's lane pairs: 32 sites of two flavours each.
#pragma once
#include "hop_split.h"

namespace tmq {

template <class SP, class LK>
struct SplitNdArgs {
    using R = typename LK::real;
    Geom g;
    int out_par, epi, ord;
    int phase_mask;
    int tiles;    // 64-site tiles per XCD
    int doublet;  // batch index of the doublet: its scalars
    SP in[2], self[2], out[2];
    LK lk;
    double ph[4][2];
    double *partial;  // of this doublet
    const CgScalars *scal;
    float one;
    SP cg_r[2];      // r (CG update) or b (true residual)
    AnyView res[2];  // the true residual, in its format
    SiteDiv dv;
    // site terms rounded from FP64: K1 {c, c m, c e}, K2 {m, e}
    R co[3];
};

// wavefront W's work
template <int W, class SP, class LK, bool SELF, bool NORM, int EP>
__device__ __forceinline__ void split_nd_role(const SplitNdArgs<SP, LK> &a, SplitShared<SP> &S, const SplitSite &p)
{
    using IO = SplitIo<SP>;
    using R = typename IO::R;
    using R2 = typename IO::R2;
    constexpr int UC = IO::UC, NU = IO::NU;
    constexpr bool XY1 = __is_same(SP, SpF64) && !SELF;
    constexpr int MU = k1_order<XY1>(W >> 1);
    constexpr bool BACK = W & 1;
    constexpr bool UNIT = W < NU;
    const Geom &g = a.g;
    const int lane = p.lane;
    const uint32_t h = p.h;
    cx<R> sf[2][UC], rr[2][UC], acc[2][UC];
    typename LK::Loaded u;
    typename IO::Raw raw;
    uint32_t hn = 0;
    if (p.active) {
        const uint32_t XH = (uint32_t)g.XH, plane = (uint32_t)g.LY * XH;
        if constexpr (MU == 1) {
            const uint32_t LX = (uint32_t)g.LX;
            hn = h - p.xh + ((BACK ? (p.x == 0 ? LX - 1 : p.x - 1) : (p.x + 1 == LX ? 0u : p.x + 1)) >> 1);
        } else {
            const uint32_t c = MU == 0 ? p.t : MU == 2 ? p.y : p.z;
            const uint32_t E = (uint32_t)(MU == 0 ? g.T : MU == 2 ? g.LY : g.LZ);
            const uint32_t s = MU == 0 ? (uint32_t)g.LZ * plane : MU == 2 ? XH : plane;
            hn = BACK ? h - s + (c == 0 ? E * s : 0u) : h + s - (c + 1 == E ? E * s : 0u);
        }
        a.lk.template load_link<true>(BACK ? a.out_par ^ 1 : a.out_par, MU, BACK ? hn : h, u);
        IO::load(a.in[0], hn, raw);
    }
#pragma unroll
    for (int f = 0; f < 2; f++) {
        if (p.active) {
            half<R> hv;
            float sc = 0.f;
            split_hop<MU, BACK ? 1 : 0>(a, u, raw, hv, sc);
            // (the lower flavour's neighbour, and what the unit needs of its own
            // site, arrive while the upper one's sum is formed)
            if (f == 0) IO::load(a.in[1], hn, raw);
            if constexpr (UNIT) {
                if (SELF) IO::load_unit(a.self[f], h, W, sf[f]);
            }
#pragma unroll
            for (int c = 0; c < 6; c++) {
                R2 v;
                v.x = hv.c[c / 3][c % 3].re, v.y = hv.c[c / 3][c % 3].im;
                S.sh[W][c][lane] = v;
            }
        }
        __syncthreads();
        if constexpr (UNIT) {
            auto comp = [&](auto kc) {
                constexpr int N = decltype(kc)::value;
                acc[f][N] = cx<R>{R(0), R(0)};
                split_sum<W * UC + N, XY1, false>(S.sh, S.shs, lane, acc[f][N]);
            };
            if (p.active) {
                comp(std::integral_constant<int, 0>{});
                comp(std::integral_constant<int, 1>{});
            }
        }
        if constexpr (UNIT && (EP == EP_CG || EP == EP_RES)) {
            // (late: with the lower flavour's neighbour they would not fit 128 registers)
            if (f == 1 && p.active) {
                IO::load_unit(a.cg_r[0], h, W, rr[0]);
                IO::load_unit(a.cg_r[1], h, W, rr[1]);
            }
        }
        __syncthreads();  // the sums are read
    }
    R n2[2][UC];
    cx<R> o[2][UC];
    if constexpr (UNIT) {
        auto comp = [&](auto kc) {
            constexpr int N = decltype(kc)::value, K = W * UC + N;
            constexpr bool UP = K < 6;  // gamma_5 = +1 on the upper spins
            if constexpr (!SELF) {
                // c (1 -+ i m g5) own - c e other (upper / lower flavour)
                const cx<R> pm = {a.co[0], -a.co[1]}, pp = {a.co[0], a.co[1]};
                o[0][N] = fma(UP ? pm : pp, acc[0][N], (-a.co[2]) * acc[1][N]);
                o[1][N] = fma(UP ? pp : pm, acc[1][N], (-a.co[2]) * acc[0][N]);
            } else {
                // A self = (1 +- i m g5) own + e other
                const cx<R> pm = {R(1), a.co[0]}, mm = {R(1), -a.co[0]};
                const cx<R> a0 = fma(UP ? pm : mm, sf[0][N], a.co[1] * sf[1][N]);
                const cx<R> a1 = fma(UP ? mm : pm, sf[1][N], a.co[1] * sf[0][N]);
                const cx<R> o0 = a0 - acc[0][N], o1 = a1 - acc[1][N];
                o[0][N] = UP ? o0 : -o0;
                o[1][N] = UP ? o1 : -o1;
            }
#pragma unroll
            for (int f = 0; f < 2; f++) {
                if constexpr (EP == EP_CG) {
                    const R ar = (R)a.scal[a.doublet].alpha;
                    o[f][N].re = fmad(-ar, o[f][N].re, rr[f][N].re);
                    o[f][N].im = fmad(-ar, o[f][N].im, rr[f][N].im);
                }
                if constexpr (EP == EP_RES) o[f][N] = rr[f][N] - o[f][N];
                if constexpr (NORM) n2[f][N] = norm2(o[f][N]);
            }
        };
        if (p.active) {
            comp(std::integral_constant<int, 0>{});
            comp(std::integral_constant<int, 1>{});
#pragma unroll
            for (int f = 0; f < 2; f++) {
                if constexpr (EP == EP_RES) {
                    if (a.res[f].prec == P64)
                        SplitIo<SpF64>::store_unit(SpF64{(double2 *)a.res[f].data}, h, W, o[f]);
                    else if (a.res[f].prec == P32)
                        st<false>((float4 *)a.res[f].data + aidx(h, W, 6),
                                  make_float4((float)o[f][0].re, (float)o[f][0].im, (float)o[f][1].re, (float)o[f][1].im));
                } else {
                    IO::store_unit(EP == EP_STORE ? a.out[f] : a.cg_r[f], h, W, o[f]);
                }
            }
        }
    }
    if constexpr (NORM) {
        // |out|^2 per component and flavour, and a 16-bit residual's values
        R *shn = (R *)S.sh;                                   // [flavour][component][site]
        float2 *shr = (float2 *)(shn + 24 * SPLIT_SITES);     // the same
        const bool res16 = EP == EP_RES && a.res[0].prec != P64 && a.res[0].prec != P32;
        if constexpr (UNIT) {
#pragma unroll
            for (int f = 0; f < 2; f++)
#pragma unroll
                for (int n = 0; n < UC; n++) {
                    shn[(f * 12 + W * UC + n) * SPLIT_SITES + lane] = p.active ? n2[f][n] : R(0);
                    if (res16)
                        shr[(f * 12 + W * UC + n) * SPLIT_SITES + lane] =
                            make_float2((float)o[f][n].re, (float)o[f][n].im);
                }
        }
        __syncthreads();
        if constexpr (EP == EP_RES && (W == 2 || W == 3)) {
            if (res16 && p.active) {
                spinor<float> v;
#pragma unroll
                for (int c = 0; c < 12; c++) {
                    const float2 q = shr[((W - 2) * 12 + c) * SPLIT_SITES + lane];
                    v.c[c / 3][c % 3] = {q.x, q.y};
                }
                store_any(a.res[W - 2], 0, h, v);
            }
        }
        if constexpr (W < 2) {
            // sites 32 W .. 32 W + 31, the two flavours of one in neighbouring lanes
            R n = R(0);
#pragma unroll
            for (int c = 0; c < 12; c++) n += shn[((lane & 1) * 12 + c) * SPLIT_SITES + 32 * W + (lane >> 1)];
            const double s = wave_sum((double)n);
            if (lane == 0) a.partial[p.pidx + W] = s;
        }
    }
}

template <class SP, class LK, bool SELF, bool NORM, int EP>
__global__ __launch_bounds__(SPLIT_THREADS, 4) void hop_split_nd_kernel(SplitNdArgs<SP, LK> a)
{
    if (a.scal && a.scal[a.doublet].done) return;
    __shared__ SplitShared<SP> S;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    SplitSite p;
    split_site<2>(a, p);
    switch (w) {
    case 0: split_nd_role<0, SP, LK, SELF, NORM, EP>(a, S, p); break;
    case 1: split_nd_role<1, SP, LK, SELF, NORM, EP>(a, S, p); break;
    case 2: split_nd_role<2, SP, LK, SELF, NORM, EP>(a, S, p); break;
    case 3: split_nd_role<3, SP, LK, SELF, NORM, EP>(a, S, p); break;
    case 4: split_nd_role<4, SP, LK, SELF, NORM, EP>(a, S, p); break;
    case 5: split_nd_role<5, SP, LK, SELF, NORM, EP>(a, S, p); break;
    case 6: split_nd_role<6, SP, LK, SELF, NORM, EP>(a, S, p); break;
    default: split_nd_role<7, SP, LK, SELF, NORM, EP>(a, S, p); break;
    }
}

// a half-sweep of the one doublet of rl (RHS 2d, 2d + 1; arguments as
// launch_hop, checked by go(); nblk for two lanes per site)
template <class SP, class LK>
hipError_t launch_split_nd(const Geom &g, int out_par, const FieldDesc &in, const FieldDesc &self,
                           const FieldDesc &out, const LinkDesc &lk, const OpParams &op, int epi, int sign,
                           const RhsList &rl, double *partial, long pstride, const CgScalars *scal, int ord, int nblk,
                           hipStream_t st, const CgFields *cg)
{
    using R = typename LK::real;
    const int ep = epi == EPI_K2_CG ? EP_CG : epi == EPI_K2_RES ? EP_RES : EP_STORE;
    const int d = rl.idx[0] >> 1;
    SplitNdArgs<SP, LK> a;
    a.g = g;
    a.out_par = out_par;
    a.epi = ep == EP_STORE ? epi : EPI_K2;
    a.ord = ord;
    a.phase_mask = hop_phase_mask(op);
    a.tiles = nblk * PARTS / 8 / 2;
    a.doublet = d;
    for (int f = 0; f < 2; f++) {
        auto field = [&](const FieldDesc &v) { return make_sp<SP>(v.data ? field_rhs(v, 2 * d + f) : v); };
        a.in[f] = field(in);
        a.self[f] = field(self);
        a.out[f] = field(out);
        if (ep != EP_STORE) a.cg_r[f] = field(ep == EP_CG ? cg->r : cg->b);
        if (ep == EP_RES) a.res[f] = make_any(field_rhs(cg->r, 2 * d + f));
    }
    a.lk = make_lk<LK>(lk);
    for (int mu = 0; mu < 4; mu++) a.ph[mu][0] = op.ph[mu][0], a.ph[mu][1] = op.ph[mu][1];
    a.partial = partial ? partial + d * pstride : nullptr;
    a.scal = scal;
    a.one = 1.0f;
    a.dv = make_site_div(g, ord, nblk, 1, 1);
    const double kap = op.kappa[d], m = sign * op.mut[d], e = op.eps[d];
    if (a.epi == EPI_K1) {
        const double c = kap * kap / (1.0 + m * m - e * e);
        a.co[0] = (R)c, a.co[1] = (R)(c * m), a.co[2] = (R)(c * e);
    } else {
        a.co[0] = (R)m, a.co[1] = (R)e, a.co[2] = R(0);
    }
    const dim3 grid(8 * a.tiles), block(SPLIT_THREADS);
    const bool s = a.epi != EPI_K1, n = partial != nullptr;
    if (ep == EP_CG)
        hipLaunchKernelGGL((hop_split_nd_kernel<SP, LK, true, true, EP_CG>), grid, block, 0, st, a);
    else if (ep == EP_RES) {
        if constexpr (__is_same(SP, SpF64))
            hipLaunchKernelGGL((hop_split_nd_kernel<SP, LK, true, true, EP_RES>), grid, block, 0, st, a);
    } else if (s && n)
        hipLaunchKernelGGL((hop_split_nd_kernel<SP, LK, true, true, EP_STORE>), grid, block, 0, st, a);
    else if (s)
        hipLaunchKernelGGL((hop_split_nd_kernel<SP, LK, true, false, EP_STORE>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((hop_split_nd_kernel<SP, LK, false, false, EP_STORE>), grid, block, 0, st, a);
    return hipGetLastError();
}

}  // namespace tmq
