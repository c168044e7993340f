// hop_split.h -- the hopping half-sweep of one field with the eight hops of a
// site in eight wavefronts.
//
// The arithmetic of hop_kernel (hop_impl.h), operation by operation, so that
// the two give the same numbers; what differs is who does it.  A block of
// eight wavefronts owns 64 consecutive output sites of the block order:
//   hops    wavefront W forms hop W of the sum (direction k1_order(W / 2),
//           forward for even W) for the 64 sites: it loads the link and the
//           neighbour, projects, multiplies, applies the phase, and leaves the
//           half spinor in LDS;
//   units   wavefronts 0 .. NU-1 each own one piece of the output spinor (UC
//           complex components, 16 or 32 bytes): they sum the eight half
//           spinors in the order of the sum, apply the site terms and store.
//
// What bounds it.  A lane of hop_kernel walks through eight dependent loads
// and about 1500 vector instructions, so a launch of few blocks takes the time
// of one lane, and a full one needs 164-180 registers in FP64 (two or three
// wavefronts per SIMD).  Here a lane has one hop: every load of a site is in
// flight at once, 56 registers in FP32 and 108 in FP64 leave 8 and 4
// wavefronts per SIMD, and for the same bytes in flight a third as many sites,
// so more of a site's neighbours are still in the XCD's L2 when they are used
// again (FP64 K1 at 32^3x64 reads 1.07-1.11 GB instead of 1.36, 1.01 without
// any re-read).  K1 in us, hop_kernel -> here on one box: FP64 8^3x16 9.8 ->
// 4.9, 24^3x48 83.4 -> 71.5, 32^3x64 223 -> 213 (5.7 TB/s of operands,
// HBM-bound; 203-212 on others); FP32
// 7.9 -> 4.0, 42.8 -> 37.6, 109 -> 104; FP16 8^3x16 6.0 -> 4.0.
// The exchange costs vector instructions and LDS traffic, which the 16-bit
// half-sweep, bound by its vector instructions once the chip is full, cannot
// afford: hop_takes_split draws the line.
#pragma once
#include "hop_impl.h"

namespace tmq {

constexpr int SPLIT_SITES = 64;    // sites per block
constexpr int SPLIT_THREADS = 512;  // eight wavefronts

// EP_CG with alpha formed from the partials of <p, A p> (SplitArgs::pap; an
// instantiation of its own: the registers it takes cost the others 0.7 % of an
// FP64 solve at 24^3x48)
constexpr int EP_CG_OWN = 4;

// which operands are canonical complex128 buffers: the input, the own-site
// field, the output; and whether these hold the whole lattice
enum SplitCan { CAN_IN = 1, CAN_SELF = 2, CAN_OUT = 4, CAN_FULL = 8 };

template <class SP, class LK>
struct SplitArgs {
    using R = typename LK::real;
    Geom g;
    int out_par, epi, ord;
    int phase_mask;
    int tiles;  // 64-site tiles per XCD
    int rhs;    // batch index of the field: its scalars and partial sums
    SP in, self, out;
    LK lk;
    double ph[4][2];
    double *partial;  // of this right-hand side
    const CgScalars *scal;
    float one;  // 1.0, opaque to the compiler (see code_lo in fields.h)
    SP cg_r;      // fused epilogues: r (CG update) or b (true residual)
    const double *pap;  // EP_CG_OWN: the partials of <p, A p> of npap blocks
    int npap;
    AnyView res;  // the true residual, in its format
    const double2 *cin, *cself;  // canonical operands (SplitCan)
    double2 *cout;
    SiteDiv dv;
    // site-term coefficients, formed on the host in FP64 by the operations of
    // hop_epilogue and rounded once: K1 {c, c m}, K2 {m}, FULL {m, kappa}, SRC
    // {kappa}, REC {c, c m, kappa c, kappa c m}
    R co[4];
};

// which of T = identity, negation, i, -i rebuilds spin I of hop (MU, S) from
// row split_row(MU, I) of its half spinor (the table of spin.h)
constexpr int split_sel(int MU, int S, int I)
{
    return I < 2     ? 0
           : MU == 0 ? (S > 0 ? 1 : 0)
           : MU == 1 ? (S > 0 ? 2 : 3)
           : MU == 2 ? ((S > 0) == (I == 2) ? 0 : 1)
                     : ((S > 0) == (I == 2) ? 2 : 3);
}
constexpr int split_row(int MU, int I)
{
    return I < 2 ? I : (MU == 0 || MU == 3) ? I - 2 : 3 - I;
}

// a neighbour spinor as loaded, and the pieces of fields that the units own
template <class SP>
struct SplitIo;

template <>
struct SplitIo<SpF64> {
    using R = double;
    using R2 = double2;
    static constexpr int UC = 2, NU = 6;
    using Raw = spinor<double>;
    static __device__ __forceinline__ void load(const SpF64 &f, long h, Raw &r) { f.load(h, r); }
    static __device__ __forceinline__ void to_canonical(double2 *q, const cx<R> (&v)[UC], float)
    {
        q[0] = make_double2(v[0].re, v[0].im);
        q[1] = make_double2(v[1].re, v[1].im);
    }
    static __device__ __forceinline__ void load_unit(const SpF64 &f, long h, int u, cx<R> (&v)[UC])
    {
        const double2 *q = f.p + aidx(h, 2 * u, 12);
        const double2 a = q[0], b = q[8];
        v[0] = {a.x, a.y}, v[1] = {b.x, b.y};
    }
    static __device__ __forceinline__ void store_unit(const SpF64 &f, long h, int u, const cx<R> (&v)[UC])
    {
        double2 *q = f.p + aidx(h, 2 * u, 12);
        st<true>(q, make_double2(v[0].re, v[0].im));
        st<true>(q + 8, make_double2(v[1].re, v[1].im));
    }
};

template <>
struct SplitIo<SpF32> {
    using R = float;
    using R2 = float2;
    static constexpr int UC = 2, NU = 6;
    using Raw = spinor<float>;
    static __device__ __forceinline__ void load(const SpF32 &f, long h, Raw &r) { f.load(h, r); }
    static __device__ __forceinline__ void to_canonical(double2 *q, const cx<R> (&v)[UC], float)
    {
        q[0] = make_double2((double)v[0].re, (double)v[0].im);
        q[1] = make_double2((double)v[1].re, (double)v[1].im);
    }
    static __device__ __forceinline__ void load_unit(const SpF32 &f, long h, int u, cx<R> (&v)[UC])
    {
        const float4 a = f.p[aidx(h, u, 6)];
        v[0] = {a.x, a.y}, v[1] = {a.z, a.w};
    }
    static __device__ __forceinline__ void store_unit(const SpF32 &f, long h, int u, const cx<R> (&v)[UC])
    {
        st<true>(f.p + aidx(h, u, 6), make_float4(v[0].re, v[0].im, v[1].re, v[1].im));
    }
};

template <bool BF>
struct SplitIo<Sp16<BF>> {
    using R = float;
    using R2 = float2;
    static constexpr int UC = 4, NU = 3;
    struct Raw {
        uint32_t c[12];
        float sc;
    };
    static __device__ __forceinline__ void load(const Sp16<BF> &f, long h, Raw &r) { f.load_codes(h, r.c, r.sc); }
    static __device__ __forceinline__ void load_unit(const Sp16<BF> &f, long h, int u, cx<R> (&v)[UC])
    {
        const float sc = f.scale[h];
        const uint4 q = f.p[aidx(h, u, 3)];
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int k = 0; k < 4; k++)
            v[k] = {code_to_f32<BF>(lo16(w[k])) * sc, code_to_f32<BF>(hi16(w[k])) * sc};
    }
    // the unit's part of Sp16::store, given the site's largest magnitude
    static __device__ __forceinline__ void store_unit(const Sp16<BF> &f, long h, int u, const cx<R> (&v)[UC], float m)
    {
        const bool bad = !(m <= 3.0e38f), tiny = m < 1.17549435e-38f;
        const float inv = tiny ? 0.f : 1.0f / m;
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; k++) w[k] = pack16(f32_to_code<BF>(v[k].re * inv), f32_to_code<BF>(v[k].im * inv));
        f.p[aidx(h, u, 3)] = make_uint4(w[0], w[1], w[2], w[3]);
        if (u == 0) f.scale[h] = bad ? __int_as_float(0x7fc00000) : (tiny ? 0.f : m);
    }
    // the same piece as it would be read back, to a canonical buffer
    static __device__ __forceinline__ void to_canonical(double2 *q, const cx<R> (&v)[UC], float m)
    {
        const bool bad = !(m <= 3.0e38f), tiny = m < 1.17549435e-38f;
        const float inv = tiny ? 0.f : 1.0f / m, sc = bad ? __int_as_float(0x7fc00000) : (tiny ? 0.f : m);
#pragma unroll
        for (int k = 0; k < 4; k++)
            q[k] = make_double2((double)(code_to_f32<BF>(f32_to_code<BF>(v[k].re * inv)) * sc),
                                (double)(code_to_f32<BF>(f32_to_code<BF>(v[k].im * inv)) * sc));
    }
};

// hop (MU, DIR) of the sum from the loaded neighbour: the half spinor w, and
// for 16-bit spinors the factor sc it is accumulated with
template <int MU, int DIR, template <class, class> class A, class SP, class LK, typename R>
__device__ __forceinline__ void split_hop(const A<SP, LK> &a, const typename LK::Loaded &u,
                                          const typename SplitIo<SP>::Raw &r, half<R> &w, float &sc)
{
    const bool phase = (a.phase_mask >> MU) & 1;  // uniform over the launch
    half<R> p;
    if constexpr (SP::coded) {
        project_codes<MU, DIR == 0 ? +1 : -1, SP::bf>(r.c, a.one, p);
        a.lk.template apply<DIR == 1>(u, p, w);
        sc = r.sc;
        if (phase) {
            const cx<R> ph = {(R)a.ph[MU][0], (R)a.ph[MU][1]};
            const cx<R> phd = DIR == 0 ? ph : conj(ph);
            half_scale(w, cx<R>{sc * phd.re, sc * phd.im});
            sc = 1.0f;
        }
    } else {
        project<MU, DIR == 0 ? +1 : -1>(r, p);
        a.lk.template apply<DIR == 1>(u, p, w);
        if (phase) {
            const cx<R> ph = {(R)a.ph[MU][0], (R)a.ph[MU][1]};
            half_scale(w, DIR == 0 ? ph : conj(ph));
        }
    }
}

// component K = 3 spin + colour of the hop sum added to acc (XY1: the order of
// the sum, as k1_order); sh: the half spinors, shs: the 16-bit factors
template <int K, bool XY1, bool CODED, typename R, typename R2>
__device__ __forceinline__ void split_sum(const R2 (*sh)[6][SPLIT_SITES], const float (*shs)[SPLIT_SITES], int lane,
                                          cx<R> &acc)
{
    constexpr int I = K / 3, A = K % 3;
    auto one = [&](auto jc) {
        constexpr int J = decltype(jc)::value;
        constexpr int MU = k1_order<XY1>(J >> 1), S = (J & 1) == 0 ? +1 : -1;
        constexpr int T = split_sel(MU, S, I);
        const R2 v = sh[J][split_row(MU, I) * 3 + A][lane];
        const cx<R> h = {v.x, v.y};
        if constexpr (CODED) {
            acc_fma<T>(acc, h, shs[J][lane]);
        } else {
            if (T == 0) acc = acc + h;
            if (T == 1) acc = acc - h;
            if (T == 2) acc = acc + ipl(h);
            if (T == 3) acc = acc + imi(h);
        }
    };
    one(std::integral_constant<int, 0>{});
    one(std::integral_constant<int, 1>{});
    one(std::integral_constant<int, 2>{});
    one(std::integral_constant<int, 3>{});
    one(std::integral_constant<int, 4>{});
    one(std::integral_constant<int, 5>{});
    one(std::integral_constant<int, 6>{});
    one(std::integral_constant<int, 7>{});
}

// the block's place on the lattice, the same for its eight wavefronts
struct SplitSite {
    uint32_t t, z, y, xh, x, h, pidx;
    bool active;  // the lane has a site
    int lane;
    // index in a canonical buffer of one parity, or (FULL) of the whole lattice
    template <bool FULL>
    __device__ __forceinline__ uint32_t site() const
    {
        return FULL ? 2 * (h - xh) + x : h;
    }
};

// LDS of a block
template <class SP>
struct SplitShared {
    using R2 = typename SplitIo<SP>::R2;
    R2 sh[8][6][SPLIT_SITES];                                // the half spinors of the hops
    float shs[SP::coded ? 8 : 1][SPLIT_SITES];               // their factors (16-bit spinors)
    float shm[SP::coded ? SplitIo<SP>::NU : 1][SPLIT_SITES];  // largest magnitude of each unit's components
    double pap[SPLIT_THREADS / 64];                          // <p, A p>, the sums of the wavefronts
};

// wavefront W's work
template <int W, class SP, class LK, bool SELF, bool NORM, int EP, int CAN>
__device__ __forceinline__ void split_role(const SplitArgs<SP, LK> &a, SplitShared<SP> &S, const SplitSite &p)
{
    using IO = SplitIo<SP>;
    using R = typename IO::R;
    using R2 = typename IO::R2;
    constexpr int UC = IO::UC, NU = IO::NU;
    constexpr bool XY1 = (SP::coded || __is_same(SP, SpF64)) && !SELF;
    constexpr int MU = k1_order<XY1>(W >> 1);
    constexpr bool BACK = W & 1;
    constexpr bool UNIT = W < NU;
    constexpr bool CG = EP == EP_CG || EP == EP_CG_OWN;
    const Geom &g = a.g;
    const int lane = p.lane;
    const uint32_t h = p.h;
    // the partial sums of <p, A p> of block 64 W + lane, summed as the scalar kernels do
    double2 pa = make_double2(0.0, 0.0), pb = pa;
    if constexpr (EP == EP_CG_OWN) {
        const int k = W * 64 + lane;
        if (k < a.npap) {
            pa = ((const double2 *)a.pap)[2 * k];
            pb = ((const double2 *)a.pap)[2 * k + 1];
        }
    }
    // what the unit needs of its own site, asked for with the hop's operands
    cx<R> sf[UC], rr[UC];
    if (p.active) {
        // the wavefront's neighbour (eo index hn; x coordinate xn) and link
        uint32_t hn, xn = p.x;
        const uint32_t XH = (uint32_t)g.XH, plane = (uint32_t)g.LY * XH;
        if constexpr (MU == 1) {
            const uint32_t LX = (uint32_t)g.LX;
            xn = BACK ? (p.x == 0 ? LX - 1 : p.x - 1) : (p.x + 1 == LX ? 0u : p.x + 1);
            hn = h - p.xh + (xn >> 1);
        } else {
            const uint32_t c = MU == 0 ? p.t : MU == 2 ? p.y : p.z;
            const uint32_t E = (uint32_t)(MU == 0 ? g.T : MU == 2 ? g.LY : g.LZ);
            const uint32_t s = MU == 0 ? (uint32_t)g.LZ * plane : MU == 2 ? XH : plane;
            hn = BACK ? h - s + (c == 0 ? E * s : 0u) : h + s - (c + 1 == E ? E * s : 0u);
        }
        typename LK::Loaded u;
        typename IO::Raw raw;
        a.lk.template load_link<true>(BACK ? a.out_par ^ 1 : a.out_par, MU, BACK ? hn : h, u);
        if constexpr (CAN & CAN_IN) {
            // the conversion to the device format is this rounding
            const double2 *q = a.cin + 12L * ((CAN & CAN_FULL) ? 2 * (hn - (xn >> 1)) + xn : hn);
#pragma unroll
            for (int c = 0; c < 12; c++) {
                const double2 v = q[c];
                raw.c[c / 3][c % 3] = cx<R>{(R)v.x, (R)v.y};
            }
        } else {
            IO::load(a.in, hn, raw);
        }
        if constexpr (UNIT) {
            if constexpr ((CAN & CAN_SELF) && SELF) {
                const double2 *q = a.cself + 12L * p.site<(CAN & CAN_FULL) != 0>() + W * UC;
#pragma unroll
                for (int n = 0; n < UC; n++) {
                    const double2 v = q[n];
                    sf[n] = cx<R>{(R)v.x, (R)v.y};
                }
            } else if (SELF) {
                IO::load_unit(a.self, h, W, sf);
            }
            if (CG || EP == EP_RES) IO::load_unit(a.cg_r, h, W, rr);
        }
        half<R> hv;
        float sc = 0.f;
        split_hop<MU, BACK ? 1 : 0>(a, u, raw, hv, sc);
#pragma unroll
        for (int c = 0; c < 6; c++) {
            R2 v;
            v.x = hv.c[c / 3][c % 3].re, v.y = hv.c[c / 3][c % 3].im;
            S.sh[W][c][lane] = v;
        }
        if constexpr (SP::coded) S.shs[W][lane] = sc;
    }
    if constexpr (EP == EP_CG_OWN) {
        const double s = wave_sum((((0.0 + pa.x) + pa.y) + pb.x) + pb.y);
        if (lane == 0) S.pap[W] = s;
    }
    __syncthreads();
    R ar = R(0);  // alpha
    if constexpr (EP == EP_CG_OWN) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < SPLIT_THREADS / 64; i++) s += S.pap[i];
        const double al = a.scal[a.rhs].rr / s;
        if (!isfinite(al)) return;  // (all wavefronts: the scalar kernel ends the solve)
        ar = (R)al;
    }

    // the units: sum, site terms, update
    cx<R> o[UC];
    float m = 0.f;
    R n2[UC];
    if constexpr (UNIT) {
        const bool pre = SELF && EP == EP_STORE && a.epi == EPI_K2;
        auto comp = [&](auto kc) {
            constexpr int N = decltype(kc)::value, K = W * UC + N;
            constexpr bool UP = K < 6;  // gamma_5 = +1 on the upper spins
            cx<R> acc = {R(0), R(0)};
            if (pre) {  // k2_self_first
                const cx<R> A = cx<R>{UP ? R(1) : R(-1), a.co[0]};
                acc = UP ? -(A * sf[N]) : A * sf[N];
            }
            split_sum<K, XY1, SP::coded>(S.sh, S.shs, lane, acc);
            if (pre) {
                o[N] = UP ? -acc : acc;
            } else if (!SELF) {
                o[N] = cx<R>{a.co[0], UP ? -a.co[1] : a.co[1]} * acc;
            } else {
                cx<R> A, B;
                if (EP == EP_STORE && a.epi == EPI_SRC) {
                    A = cx<R>{R(1), R(0)};
                    B = cx<R>{a.co[0], R(0)};
                } else if (EP == EP_STORE && a.epi == EPI_REC) {
                    A = cx<R>{a.co[0], UP ? -a.co[1] : a.co[1]};
                    B = cx<R>{a.co[2], UP ? -a.co[3] : a.co[3]};
                } else {
                    const R b = EP == EP_STORE ? a.co[1] : R(1);  // FULL: kappa
                    A = cx<R>{UP ? R(1) : R(-1), a.co[0]};
                    B = cx<R>{UP ? -b : b, R(0)};
                }
                o[N] = fma(A, sf[N], B * acc);
            }
            if constexpr (CG) {
                // r -= alpha (A p)
                if constexpr (EP == EP_CG) ar = (R)a.scal[a.rhs].alpha;
                o[N].re = fmad(-ar, o[N].re, rr[N].re);
                o[N].im = fmad(-ar, o[N].im, rr[N].im);
            }
            if constexpr (EP == EP_RES) o[N] = rr[N] - o[N];
            if constexpr (NORM) n2[N] = norm2(o[N]);
            if constexpr (SP::coded) {
                const float f0 = fabsf(o[N].re), f1 = fabsf(o[N].im);
                if (!(f0 <= 3.0e38f) || !(f1 <= 3.0e38f)) m = __builtin_inff();  // (non-finite: Sp16::store)
                m = fmaxf(m, fmaxf(f0, f1));
            }
        };
        if (p.active) {
            comp(std::integral_constant<int, 0>{});
            comp(std::integral_constant<int, 1>{});
            if constexpr (UC == 4) {
                comp(std::integral_constant<int, 2>{});
                comp(std::integral_constant<int, 3>{});
            }
            if constexpr (EP == EP_RES) {
                // (FP64 and FP32 residuals from here, 16-bit ones below: they need the whole site)
                if (a.res.prec == P64)
                    SplitIo<SpF64>::store_unit(SpF64{(double2 *)a.res.data}, h, W, o);
                else if (a.res.prec == P32)
                    st<false>((float4 *)a.res.data + aidx(h, W, 6),
                              make_float4((float)o[0].re, (float)o[0].im, (float)o[1].re, (float)o[1].im));
            } else if constexpr (SP::coded)
                S.shm[W][lane] = m;
            else if constexpr (CAN & CAN_OUT)
                IO::to_canonical(a.cout + 12L * p.site<(CAN & CAN_FULL) != 0>() + W * UC, o, 0.f);
            else
                IO::store_unit(EP == EP_STORE ? a.out : a.cg_r, h, W, o);
        }
    }
    if constexpr (SP::coded || NORM) {
        __syncthreads();  // the sums are read, the largest magnitudes written
        // |out|^2 per component, for the sum over a site in the order of its components
        R *shn = (R *)S.sh;
        // a 16-bit residual: the site's values (rounded to FP32 first, as Sp16::store does)
        float2 *shr = (float2 *)(shn + 12 * SPLIT_SITES);
        const bool res16 = EP == EP_RES && a.res.prec != P64 && a.res.prec != P32;
        if constexpr (UNIT) {
            if (p.active) {
                if constexpr (NORM)
#pragma unroll
                    for (int n = 0; n < UC; n++) shn[(W * UC + n) * SPLIT_SITES + lane] = n2[n];
                if constexpr (EP == EP_RES)
                    if (res16)
#pragma unroll
                        for (int n = 0; n < UC; n++)
                            shr[(W * UC + n) * SPLIT_SITES + lane] = make_float2((float)o[n].re, (float)o[n].im);
                if constexpr (SP::coded) {
                    const float mx = fmaxf(S.shm[0][lane], fmaxf(S.shm[1][lane], S.shm[2][lane]));
                    if constexpr (CAN & CAN_OUT)
                        IO::to_canonical(a.cout + 12L * h + W * UC, o, mx);
                    else
                        IO::store_unit(EP == EP_STORE ? a.out : a.cg_r, h, W, o, mx);
                }
            }
        }
        if constexpr (NORM) {
            __syncthreads();
            if constexpr (EP == EP_RES && W == 1) {
                // (wavefront 0 sums the norm meanwhile)
                if (res16 && p.active) {
                    spinor<float> v;
#pragma unroll
                    for (int c = 0; c < 12; c++) {
                        const float2 q = shr[c * SPLIT_SITES + lane];
                        v.c[c / 3][c % 3] = {q.x, q.y};
                    }
                    store_any(a.res, 0, h, v);
                }
            }
            if constexpr (W == 0) {
                double s = 0.0;
                if (p.active) {
                    R n = R(0);
#pragma unroll
                    for (int c = 0; c < 12; c++) n += shn[c * SPLIT_SITES + lane];
                    s = (double)n;
                }
                s = wave_sum(s);
                if (lane == 0) a.partial[p.pidx] = s;
            }
        }
    }
}

// the site of a lane, and the index of its block's (first) partial sum: a
// 64-site tile is a quarter of a block of hop_kernel, or half of one with two
// lanes per site (LPS), whose wavefronts leave their sums at PARTS * block +
// wavefront
template <int LPS, class A>
__device__ __forceinline__ void split_site(const A &a, SplitSite &p)
{
    const Geom &g = a.g;
    const uint32_t j = blockIdx.x & 7, sb = blockIdx.x >> 3;
    constexpr uint32_t TPB = PARTS / LPS;  // tiles of such a block
    p.lane = threadIdx.x & 63;
    const uint32_t XH = (uint32_t)g.XH, LY = (uint32_t)g.LY, LZ = (uint32_t)g.LZ, T = (uint32_t)g.T;
    const uint32_t plane = LY * XH;
    if (a.ord == ORD_PLAIN) {
        const uint32_t lb = j * (uint32_t)a.tiles + sb, l = lb * SPLIT_SITES + p.lane;
        p.active = l < (uint32_t)g.vh;
        const uint32_t hu = p.active ? l : 0u;
        const uint32_t r = fdiv(hu, a.dv.xh), r1 = fdiv(r, a.dv.ly);
        p.xh = hu - r * XH;
        p.y = r - r1 * LY;
        p.t = fdiv(r1, a.dv.lz);
        p.z = r1 - p.t * LZ;
        p.pidx = LPS * lb;
    } else {
        // slabs of z (t outermost) or of t (z outermost), an extent in 8 parts
        const bool zs = a.ord == ORD_ZSLAB;
        const uint32_t E = zs ? LZ : T, O = zs ? T : LZ;
        const uint32_t eb = E >> 3, er = E & 7;
        const uint32_t ec = eb + (j < er ? 1 : 0), e0 = j * eb + (j < er ? j : er);
        const uint32_t S1 = ec * plane, l = sb * SPLIT_SITES + p.lane;
        p.active = l < O * S1;
        const uint32_t lu = p.active ? l : 0u;
        const uint32_t o = fdiv(lu, a.dv.slab[j < er ? 1 : 0]), rem = lu - o * S1;
        const uint32_t e = fdiv(rem, a.dv.plane), r2 = rem - e * plane;
        p.y = fdiv(r2, a.dv.xh);
        p.xh = r2 - p.y * XH;
        p.t = zs ? o : e0 + e;
        p.z = zs ? e0 + e : o;
        p.pidx = PARTS * (8 * (sb / TPB) + j) + LPS * (sb % TPB);
    }
    p.h = ((p.t * LZ + p.z) * LY + p.y) * XH + p.xh;
    p.x = 2 * p.xh + ((a.out_par + p.t + p.z + p.y) & 1);  // (t + z + y + x) = out_par mod 2
}

template <class SP, class LK, bool SELF, bool NORM, int EP, int CAN = 0>
__global__ __launch_bounds__(SPLIT_THREADS) void hop_split_kernel(SplitArgs<SP, LK> a)
{
    if (a.scal && a.scal[a.rhs].done) return;
    __shared__ SplitShared<SP> S;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    SplitSite p;
    split_site<1>(a, p);
    // (the eight roles run through the same barriers)
    switch (w) {
    case 0: split_role<0, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    case 1: split_role<1, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    case 2: split_role<2, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    case 3: split_role<3, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    case 4: split_role<4, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    case 5: split_role<5, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    case 6: split_role<6, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    default: split_role<7, SP, LK, SELF, NORM, EP, CAN>(a, S, p); break;
    }
}

// a half-sweep of the one field of rl through the split kernel (arguments as
// launch_hop, checked by go(); instantiated in hop_split_*.hip)
template <class SP, class LK>
hipError_t launch_split(const Geom &g, int out_par, const FieldDesc &in, const FieldDesc &self, const FieldDesc &out,
                        const LinkDesc &lk, const OpParams &op, int epi, int sign, const RhsList &rl, double *partial,
                        long pstride, const CgScalars *scal, int ord, int nblk, hipStream_t st, const CgFields *cg)
{
    using R = typename LK::real;
    static_assert(SPLIT_SITES * PARTS == HOP_BLOCK, "a tile is the sites of one partial sum");
    const int ep = epi == EPI_K2_CG ? EP_CG : epi == EPI_K2_RES ? EP_RES : EP_STORE;
    const int r = rl.idx[0];
    auto field = [&](const FieldDesc &f) { return make_sp<SP>(f.data && !f.layout ? field_rhs(f, r) : f); };
    SplitArgs<SP, LK> a;
    a.g = g;
    a.out_par = out_par;
    a.epi = ep == EP_STORE ? epi : EPI_K2;
    a.ord = ord;
    a.phase_mask = hop_phase_mask(op);
    a.tiles = nblk * PARTS / 8;
    a.rhs = r;
    a.in = field(in);
    a.self = field(self);
    a.out = field(out);
    a.lk = make_lk<LK>(lk);
    for (int mu = 0; mu < 4; mu++) a.ph[mu][0] = op.ph[mu][0], a.ph[mu][1] = op.ph[mu][1];
    a.partial = partial ? partial + r * pstride : nullptr;
    a.scal = scal;
    a.one = 1.0f;
    if (ep != EP_STORE) {
        a.cg_r = field(ep == EP_CG ? cg->r : cg->b);
        if (ep == EP_RES) a.res = make_any(field_rhs(cg->r, r));
    }
    a.pap = ep == EP_CG && cg->pap ? cg->pap + r * pstride : nullptr;
    a.npap = a.pap ? cg->npap : 0;
    if (a.npap > SPLIT_THREADS) return hipErrorInvalidValue;
    // canonical operands: the input with the own-site field (if any), the output
    const bool fused = ep != EP_STORE, sl = self.data != nullptr;
    const int full = in.layout == LAY_CANONICAL_FULL || out.layout == LAY_CANONICAL_FULL ? CAN_FULL : 0;
    const int can = (in.layout ? CAN_IN : 0) | (sl && self.layout ? CAN_SELF : 0) |
                    (!fused && out.layout ? CAN_OUT : 0) | full;
    if (can && (fused || partial || r != 0)) return hipErrorInvalidValue;
    a.cin = (const double2 *)in.data;
    a.cself = (const double2 *)self.data;
    a.cout = (double2 *)out.data;
    a.dv = make_site_div(g, ord, nblk, 1, 1);
    const double kap = op.kappa[r], m = sign * op.mut[r];
    double e[4] = {m, kap, 0.0, 0.0};
    if (a.epi == EPI_K1) {
        e[0] = kap * kap / (1.0 + m * m);
        e[1] = e[0] * m;
    } else if (a.epi == EPI_SRC) {
        e[0] = kap;
    } else if (a.epi == EPI_REC) {
        const double c = 1.0 / (1.0 + m * m);
        e[0] = c, e[1] = c * m, e[2] = kap * c, e[3] = kap * c * m;
    }
    for (int q = 0; q < 4; q++) a.co[q] = (R)e[q];
    const dim3 grid(nblk * PARTS), block(SPLIT_THREADS);
    const bool s = a.epi != EPI_K1, n = partial != nullptr;
    if (can) {
#define SPLIT_CAN(SELF, CAN)                                                                              \
    if (s == SELF && can == (CAN)) {                                                                      \
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, SELF, false, EP_STORE, CAN>), grid, block, 0, st, a); \
        return hipGetLastError();                                                                         \
    }
        SPLIT_CAN(true, CAN_OUT)
        if constexpr (!SP::coded) {
            SPLIT_CAN(false, CAN_IN)
            SPLIT_CAN(true, CAN_SELF | CAN_OUT)
        }
        if constexpr (__is_same(SP, SpF64)) {
            SPLIT_CAN(true, CAN_SELF)
            SPLIT_CAN(true, CAN_OUT | CAN_FULL)
            SPLIT_CAN(true, CAN_IN | CAN_SELF | CAN_OUT | CAN_FULL)
        }
#undef SPLIT_CAN
        return hipErrorInvalidValue;
    }
    if (a.pap)
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, true, true, EP_CG_OWN>), grid, block, 0, st, a);
    else if (ep == EP_CG)
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, true, true, EP_CG>), grid, block, 0, st, a);
    else if (ep == EP_RES) {
        if constexpr (__is_same(SP, SpF64))
            hipLaunchKernelGGL((hop_split_kernel<SP, LK, true, true, EP_RES>), grid, block, 0, st, a);
    } else if (s && n)
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, true, true, EP_STORE>), grid, block, 0, st, a);
    else if (s)
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, true, false, EP_STORE>), grid, block, 0, st, a);
    else if (n)
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, false, true, EP_STORE>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((hop_split_kernel<SP, LK, false, false, EP_STORE>), grid, block, 0, st, a);
    return hipGetLastError();
}

}  // namespace tmq
