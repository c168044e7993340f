// kernels.h -- host-side declarations of the device kernels' launch wrappers.
//
// Host code (the lattice object, the solvers, the C ABI) is format-agnostic:
// it passes FieldDesc / LinkDesc descriptors and the wrappers dispatch to the
// template instantiations in hop.hip, blas.hip and codec.hip.
//
// Every vector kernel works on a batch of right-hand sides (RHS): a field
// holds nrhs fields of n sites each, and a launch covers the RHS named in an
// RhsList.  One block handles one RHS, so per-RHS scalars, "done" flags and
// partial sums stay separate, and each RHS is computed exactly as if it were
// alone (a single solve is the batch of one).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fastdiv.h"
#include "hop_grid.h"

namespace tmq {

enum Prec { P64 = 0, P32 = 1, P16 = 2, PB16 = 3 };  // same values as tmq_prec
// LK32F: FP32 full 3x3 links, the reduced-precision copy of a gauge field
// that is not SU(3) (two-row storage rebuilds row 2 assuming SU(3))
enum LinkFmt { LK64F = 0, LK64R = 1, LK32R = 2, LK16R = 3, LK32F = 4 };
constexpr int N_LINK_FMT = 8;  // stride of the (spinor precision, link format) tuning keys

constexpr int MAX_RHS = 64;

// How a field is laid out: the device layout of its precision, or a caller's
// canonical complex128 buffer that a half-sweep reads or writes itself
// (rounded to the precision on the way: the numbers are those of a conversion
// pass), [V/2][12] of one parity or [V][12] of the whole lattice.
enum Layout { LAY_DEVICE = 0, LAY_CANONICAL = 1, LAY_CANONICAL_FULL = 2 };

// A batch of spinor fields, each of n sites (one parity, or both parities
// stacked: even sites 0..V/2-1, odd sites V/2..V-1) in the 8-site chunked
// layout of fields.h; RHS r starts rhs_elems elements (and rhs_sites scales)
// after RHS 0.
struct FieldDesc {
    int prec = P64;
    int layout = LAY_DEVICE;
    void *data = nullptr;   // element type by prec: double2, float4, uint4
    float *scale = nullptr; // FP32 per-site scale of 16-bit formats
    long n = 0;             // sites per RHS (a multiple of 8)
    int nrhs = 1;
    long rhs_elems = 0;
    long rhs_sites = 0;
};

// a canonical buffer as the input or output of a half-sweep in precision prec
inline FieldDesc canonical_desc(int prec, const void *buf, long n, int layout)
{
    FieldDesc d;
    d.prec = prec;
    d.layout = layout;
    d.data = (void *)buf;
    d.n = n;
    return d;
}
// sub-view starting at site `off` (a multiple of 8), n sites, every RHS
FieldDesc field_sub(const FieldDesc &f, long off, long n);
// the single field of RHS r
FieldDesc field_rhs(const FieldDesc &f, int r);
size_t field_elem_bytes(int prec);
int field_blocks(int prec);  // component blocks per site: 12, 6, 3, 3

// The RHS a launch covers (indices into the batch).
struct RhsList {
    int n = 0;
    unsigned char idx[MAX_RHS];
};
RhsList rhs_all(int n);

struct LinkDesc {
    int fmt = LK64F;
    const void *a = nullptr;  // main array
    const void *b = nullptr;  // second array (LK16R)
    long vh = 0;              // sites per parity
};

// Operator parameters of a launch: boundary phases common to the batch,
// kappa and mut = 2 kappa mu per RHS (indexed by the batch index).
//
// nd = 1: the flavour doublet of eq. (Dh) (mut is 2 kappa mubar, eps is
// 2 kappa epsbar).  A doublet field is one field of twice the sites, the
// upper flavour's sites first; doublet d of a batch has its parameters at
// index d.  Host wrappers present the launch to the kernel as a batch of
// single-flavour fields in which doublet d is the pair 2d, 2d + 1.
struct OpParams {
    double ph[4][2];  // e^{i theta_mu pi / L_mu} (re, im), mu = t, x, y, z
    double kappa[MAX_RHS];
    double mut[MAX_RHS];
    double eps[MAX_RHS];
    int nd = 0;
};

// Epilogue of a hop half-sweep at output site h (spin s; upper = spins 0,1
// where gamma_5 = +1, lower = spins 2,3), with sigma = sign of Qhat^{+-}:
//   EPI_K1   out = kappa^2/(1+mut^2) (1 - sigma i mut g5) acc              (eq. (eo3))
//   EPI_K2   out = g5 [(1 + sigma i mut g5) self - acc]                    (eq. (eo4))
//   EPI_FULL out = g5 [(1 + sigma i mut g5) self - kappa acc]              (eq. (eo1))
//   EPI_SRC  out = self + kappa acc                                       (even/odd source, App. B)
//   EPI_REC  out = (1 - sigma i mut g5)/(1+mut^2) (self + kappa acc)      (even-site solution, App. B)
//   EPI_K2_CG  as EPI_K2, then the CG update of the residual with the RHS's
//              alpha (device scalars): r -= alpha out ; norm of the new r; out
//              is not stored (x += alpha p goes with the update of p)
//   EPI_K2_RES as EPI_K2, then r = b - out (the true residual) with its norm;
//              out is not stored, r is stored in any spinor format
// For a doublet (OpParams::nd) a lane pair holds the two flavours (f, f') of
// a site and, with A = 1 + sigma i mubar g5 tau^3 + epsbar tau^1 the site term
// and d = 1 + mubar^2 - epsbar^2,
//   EPI_K1   out = kappa^2 / d (1 - sigma i mubar g5 tau^3 - epsbar tau^1) acc
//   EPI_K2   out = g5 [A self - acc]
// and the fused epilogues as above, per flavour, with the doublet's scalars;
// the norm is over both flavours.  Other epilogues are refused.
enum HopEpi { EPI_K1 = 0, EPI_K2 = 1, EPI_FULL = 2, EPI_K2_CG = 3, EPI_K2_RES = 4, EPI_SRC = 5, EPI_REC = 6 };

// Vectors of the fused epilogues: r (in the hop's spinor format for
// EPI_K2_CG), and for EPI_K2_RES b in the hop's format.
struct CgFields {
    FieldDesc r, b;
    // EPI_K2_CG of a launch of hop_sums_alpha: partial sums of <p, A p> of npap
    // blocks, from which the half-sweep forms alpha itself (else scal's)
    const double *pap = nullptr;
    int npap = 0;
};

// Device scalars of a CG solve (one struct per right-hand side).
struct CgScalars {
    double rr;       // current ||r||^2 (iterated, or true after a reliable update)
    double rr_prev;  // ||r||^2 at the start of the last iteration
    double pAp;      // <p, A p> = ||Qhat^- p||^2
    double alpha, beta;
    double bb;       // ||b||^2
    double target;   // stop when rr < target
    int iter;        // iterations done
    int done;        // 1 once rr < target or nan (kernels told to skip done RHS then do nothing)
    int nan;         // 1 once a non-finite scalar appeared
    int reliable;    // number of true-residual recomputations
    int last_true;   // 1 if rr is a recomputed true residual
    int pad;
    int xpend;       // 1: x += alpha p of the last iteration is still to be done
    int fresh;       // 1: the solution (correction) holds nothing yet and counts as zero
};

// whether the (spinor precision, link format) pairing has every variant; the
// others always run variant 0 whatever HopTune asks for
bool hop_all_variants(int prec, int link_fmt);

// bit mu set when the boundary phase of direction mu is not 1
inline int hop_phase_mask(const OpParams &op)
{
    int m = 0;
    for (int mu = 0; mu < 4; mu++)
        if (op.ph[mu][0] != 1.0 || op.ph[mu][1] != 0.0) m |= 1 << mu;
    return m;
}
// whether a single-field launch (not a doublet's) runs in the split kernel
// (hop_split.h), in the block order of its variant (2 as 1, 4 as 3), without a
// cap.  FP64 and FP32: always; it is the faster one from 4^4 (FP64 K1 4.3
// against 7.1 us) to 32^3x64 (213 against 223 us).  16-bit: up to three
// quarters of a 256-lane block per CU.  Below, the lanes of the 16-bit kernel
// leave CUs idle (K1 6.0 us at 8^3x16 and 7.0 us at 20x10x14x18, split 4.0 and
// 5.1 us); from one block per CU on its vector instructions bound it and the
// split kernel executes more of them (6.7 against 7.1 us at 16^3x32, 57 against
// 78 us at 32^3x64).
inline bool hop_takes_split(const Geom &g, int prec, int link_fmt)
{
    if (prec == P64) return true;
    if (prec == P32) return link_fmt == LK32R;
    return link_fmt == LK16R && g.vh <= 49152;
}
// whether the CG half-sweep of a single field sums the nparts blocks' partials
// of <p, A p> itself (SC_ALPHA_BETA follows it): a launch and the wait between
// two kernels less per iteration, for as many reads of the partials as there are
// blocks.  A wavefront takes 64 of them, so a block's eight take 512.  Solves
// repeated on the same inputs, a launch of its own -> here, us: FP32 8^3x16 (16
// blocks) 1138 -> 1069, 16^3x32 (256) 2207 -> 2154; FP64 1197 -> 1145, 3240 ->
// 3170; with 512 blocks (16^3x64) FP32 3489 -> 3460, FP64 5660 -> 5630, half a
// per cent, so the line is drawn there.
inline bool hop_sums_alpha(const Geom &g, int prec, int link_fmt, int nparts)
{
    return hop_takes_split(g, prec, link_fmt) && nparts <= 512;
}
// whether a launch of 16-bit spinors on FP16 two-row links runs in the 16-bit
// kernel (hop16_kernel): 32-bit offsets (V/2 < 2^26) and a boundary phase in
// time only, or none
inline bool hop16_ok(const Geom &g, int phase_mask) { return g.vh < (1L << 26) && (phase_mask == 0 || phase_mask == 1); }
// lanes per site of a doublet launch: 1 in the 16-bit kernel (both flavours
// in a lane), 2 in the general kernel (a lane pair)
inline int hop_nd_lanes(const Geom &g, int prec, int link_fmt, const OpParams &op)
{
    return (prec == P16 || prec == PB16) && link_fmt == LK16R && hop16_ok(g, hop_phase_mask(op)) ? 1 : 2;
}

// Which single-field half-sweeps take canonical buffers (Layout).  Output (no
// norm, no fused update): the split kernel and the 16-bit kernel, at any size:
// it saves the conversion pass (Qhat at 32^3x64: FP64 614 -> 560 us, FP32 352
// -> 325, FP16 250 -> 236; at 8^3x16 19.2 -> 16.1).  Input: the split kernel in
// FP64 and FP32 (a 16-bit site would be encoded eight times), of buffers of at
// most 32 K sites (6 MB): a launch less (Qhat FP64 8^3x16 16.1 -> 13.2 us,
// 20x10x14x18 25.1 -> 22.1); above, its 192-byte strides, read eight times
// over, cost more than the pass (16^3x32 41.5 -> 42.0, FP32 at 32^3x64 325 ->
// 410, the full operator 768 -> 944).
inline bool hop_reads_canonical(const Geom &g, int prec, int link_fmt, long sites)
{
    return (prec == P64 || prec == P32) && hop_takes_split(g, prec, link_fmt) && sites <= 32768;
}
inline bool hop_writes_canonical(const Geom &g, int prec, int link_fmt, const OpParams &op)
{
    return hop_takes_split(g, prec, link_fmt) ||
           ((prec == P16 || prec == PB16) && link_fmt == LK16R && hop16_ok(g, hop_phase_mask(op)));
}

// Hop half-sweep: out(h) over the V/2 sites of parity out_par for every RHS
// of rl; `in` holds parity 1 - out_par; `self` (data may be nullptr unless
// the epilogue needs it) holds parity out_par.  partial != nullptr: sums of
// |out|^2 per wavefront at partial[r * pstride + PARTS * block + wavefront].  scal != nullptr: blocks of
// RHS r with scal[r].done set do nothing.
// Launch shape of a hop half-sweep, chosen by the autotuner.
struct HopTune {
    int variant = 0;   // block order (see above)
    int group = 0;     // RHS per L2 group of a batched launch (0: sized from the L2 capacity)
    int rpl = 1;       // RHS per lane in a batched launch: 1 or 2 (FP32-arithmetic formats)
    unsigned lds = 0;  // LDS bytes reserved per block (unused by the kernel; a value above
                       // the CU's LDS / (c + 1) caps the blocks resident per CU at c)
};
hipError_t launch_hop(const Geom &g, int out_par, const FieldDesc &in, const FieldDesc &self,
                      const FieldDesc &out, const LinkDesc &lk, const OpParams &op, int epi, int sign,
                      const RhsList &rl, double *partial, long pstride, const CgScalars *scal, const HopTune &tu,
                      hipStream_t st, const CgFields *cg = nullptr);

// Vector kernels over the n sites of each RHS of rl.  Reductions write the
// wavefronts' sums of blas_grid(n) blocks at partial[r * pstride + PARTS * block + wavefront]; scalars come
// from scal[r]; skip_done: blocks of RHS with scal[r].done do nothing.
hipError_t launch_norm2(const FieldDesc &v, const RhsList &rl, double *partial, long pstride, hipStream_t st);
hipError_t launch_convert(const FieldDesc &in, const FieldDesc &out, const RhsList &rl, hipStream_t st);
hipError_t launch_zero(const FieldDesc &v, const RhsList &rl, hipStream_t st);
// x += alpha p ; r -= alpha ap ; partial |r|^2
hipError_t launch_axpy_norm(const FieldDesc &x, const FieldDesc &p, const FieldDesc &r, const FieldDesc &ap,
                            const RhsList &rl, const CgScalars *scal, double *partial, long pstride,
                            bool skip_done, hipStream_t st);
// x += alpha p where that is pending (xpend; x may have no data: nothing), then
// p = r + beta p (not for done RHS if skip_done, not at all if only_x)
hipError_t launch_xpay(const FieldDesc &r, const FieldDesc &p, const FieldDesc &x, const RhsList &rl,
                       const CgScalars *scal, bool skip_done, bool only_x, hipStream_t st);
// r = b - ax (FP64), partial |r|^2
hipError_t launch_residual(const FieldDesc &b, const FieldDesc &ax, const FieldDesc &r, const RhsList &rl,
                           double *partial, long pstride, hipStream_t st);
// out = cu in (spins 0, 1), cd in (spins 2, 3); FP64 fields
hipError_t launch_twist(const FieldDesc &in, const FieldDesc &out, const RhsList &rl, double2 cu, double2 cd,
                        hipStream_t st);
// x64 += xs, with the pending xs += alpha p; x64 counts as zero before the first
// true residual, xs while it is fresh
hipError_t launch_accumulate(const FieldDesc &x64, const FieldDesc &xs, const FieldDesc &p, const RhsList &rl,
                             const CgScalars *scal, hipStream_t st);
// x += d (FP64)
hipError_t launch_add(const FieldDesc &x, const FieldDesc &d, const RhsList &rl, hipStream_t st);
// a right-hand side enters a solve: b (FP64), r and p (one format) of RHS 0 of
// each field from the canonical source, and the partials of |b|^2
hipError_t launch_join(const double2 *src, const FieldDesc &b, const FieldDesc &r, const FieldDesc &p, double *partial,
                       hipStream_t st);

// Scalar kernels (one block per RHS): deterministic sums of the partials of nparts blocks.
enum ScalarOp {
    SC_INIT = 0,     // bb = rr = sum ; target = tol2 * (relative ? bb : 1) ; counters cleared
    SC_ALPHA = 1,    // pAp = sum ; alpha = rr / pAp
    SC_BETA = 2,     // rr_prev = rr ; rr = sum ; beta = rr / rr_prev ; iter++ ; done = rr < target
    SC_RELIABLE = 3,  // rr = sum (true residual) ; beta = rr / rr_prev ; done = rr < target
    SC_ALPHA_BETA = 4  // SC_ALPHA of the partials at pap, then SC_BETA (nparts at most 1024)
};
// defer: the solve leaves x += alpha p to launch_xpay: SC_INIT and SC_RELIABLE
// set fresh to it (and xpend to 0), SC_BETA xpend (0 for a skipped RHS; an
// update pending before was done by then, so x is not fresh any more).
// publish != nullptr: the scalars of RHS r are finally copied to publish[r]
// (host-mapped memory), also when the block is skipped.
hipError_t launch_scalar(int op, const RhsList &rl, const double *partial, long pstride, int nparts,
                         CgScalars *scal, double tol2, int relative, bool skip_done, bool defer,
                         CgScalars *publish, hipStream_t st, const double *pap = nullptr);
// xpend = 0 after launch_xpay has applied the update, and x not fresh: for RHS
// that go on without the iteration whose SC_BETA would do this
hipError_t launch_x_applied(const RhsList &rl, CgScalars *scal, hipStream_t st);
// out[i] = sum of the partials of nparts blocks of RHS rl.idx[i], in the order of the scalar kernels
hipError_t launch_sums(const RhsList &rl, const double *partial, long pstride, int nparts, double *out, hipStream_t st);
// out[0] = deterministic maximum of partial[0..n)
hipError_t launch_max(const double *partial, int n, double *out, hipStream_t st);
// b = a, bytes / 16 lanes of 16 bytes (bandwidth calibration)
hipError_t launch_stream_copy(const void *src, void *dst, size_t bytes, hipStream_t st);

// BiCGstab on one odd-site system (FP64, RHS 0 of each field), scalars on
// the device; every kernel does nothing once `done` is set (see bicgstab.hip)
struct BicgScalars {
    double rho[2], alpha[2], omega[2], beta[2];  // complex (re, im)
    double rr, bb, target;
    int iter, restarts, done, nan, breakdown;
    int max_iter;  // done once iter reaches it (set by the host before the start)
};
enum BicgOp {
    BI_START = 0,  // r = rhat: sums <rhat, r>, |r|^2 ; alpha = omega = 1, beta = 0
    BI_ALPHA = 1,  // sum <rhat, v> ; alpha = rho / <rhat, v>
    BI_OMEGA = 2,  // sums <t, s>, |t|^2 ; omega = <t, s> / |t|^2
    BI_UPDATE = 3  // sums <rhat, r>, |r|^2 of the new r ; beta = (rho' / rho)(alpha / omega) ; done
};
// <a, b> -> p0 (re), p1 (im); |a|^2 -> p2, one partial per block (blas_grid(n))
hipError_t launch_bi_dot(const FieldDesc &a, const FieldDesc &b, const BicgScalars *sc, double *p0, double *p1,
                         double *p2, hipStream_t st);
// p = r + beta (p - omega v)
hipError_t launch_bi_p(const FieldDesc &r, const FieldDesc &p, const FieldDesc &v, const BicgScalars *sc,
                       hipStream_t st);
// s = r - alpha v
hipError_t launch_bi_s(const FieldDesc &r, const FieldDesc &v, const FieldDesc &s, const BicgScalars *sc,
                       hipStream_t st);
// x += alpha p + omega s ; r = s - omega t ; <rhat, r> -> p0, p1 ; |r|^2 -> p2
hipError_t launch_bi_xr(const FieldDesc &x, const FieldDesc &p, const FieldDesc &s, const FieldDesc &t,
                        const FieldDesc &r, const FieldDesc &rhat, const BicgScalars *sc, double *p0, double *p1,
                        double *p2, hipStream_t st);
// one scalar step (BicgOp) from nparts partials of p0, p1, p2; publish: copy of the scalars
hipError_t launch_bi_scalar(int op, const double *p0, const double *p1, const double *p2, int nparts,
                            BicgScalars *s, double tol2, int relative, BicgScalars *publish, hipStream_t st);

// the whole full-lattice FP64 CG on Q^+ Q^- of a tiny lattice in one launch
// (small_cg.hip): f = {b, x, r, p, t, p'}, stacked full fields; continues from
// x and the counters in *sc (zeroed before the first call), ends with the true
// residual in sc->rr and sc->done set if it met the target.  sync: device
// memory of SMALL_SYNC_WORDS words for the blocks' exchanges; a block waits at
// most `spin` wall-clock ticks for the others (they wait for a place on the
// device while other launches fill it), then all give up: sc->pad is 1 and the
// solve has to be done another way.
constexpr long SMALL_CG_MAX_SITES = 1024;
constexpr int SMALL_SYNC_WORDS = 64;
hipError_t launch_small_cg(const Geom &g, const FieldDesc *f, const LinkDesc &lk, const OpParams &op, double tol2,
                           int relative, int max_iter, CgScalars *sc, unsigned long long *sync, long long spin,
                           hipStream_t st);

// a 4x4 complex spin matrix (row-major)
struct SpinMat {
    double2 m[4][4];
};
// per time slice t and block b of it: partial sums of psi^+ Gamma psi over the
// slice's sites (psi canonical full-lattice complex128 [V][12]) at
// pre / pim[t * ts_bilinear_blocks(g) + b]
int ts_bilinear_blocks(const Geom &g);
hipError_t launch_ts_bilinear(const Geom &g, const double2 *psi, const SpinMat &m, double *pre, double *pim,
                              hipStream_t st);

// codec: canonical complex128 [site][12] <-> one device field (RHS 0 of the view)
hipError_t launch_from_canonical(const double2 *in, const FieldDesc &out, hipStream_t st);
hipError_t launch_to_canonical(const FieldDesc &in, double2 *out, hipStream_t st);
// full-lattice fields: canonical site s of parity p -> stacked view site p * V/2 + (s >> 1)
hipError_t launch_full_from_canonical(const Geom &g, const double2 *in, const FieldDesc &out, hipStream_t st);
hipError_t launch_full_to_canonical(const Geom &g, const FieldDesc &in, double2 *out, hipStream_t st);
// canonical full field (complex128 [V][12], lexicographic sites) <-> canonical
// even and odd fields ([V/2][12], eo index = site >> 1); split skips a null
// parity, merge writes zeros for one
hipError_t launch_split_eo(const Geom &g, const double2 *full, double2 *even, double2 *odd, hipStream_t st);
hipError_t launch_merge_eo(const Geom &g, const double2 *even, const double2 *odd, double2 *full, hipStream_t st);
// export 16-bit codes of a field in canonical [site][24] order plus scales
hipError_t launch_export_codes(const FieldDesc &in, uint16_t *codes, float *scale, hipStream_t st);

// gauge ingest from canonical complex128 [site][mu][3][3]: writes the enabled
// formats (null pointers skip) and per-block maxima of |U U^+ - 1| and |det U - 1|
struct GaugeOut {
    double2 *full64;  // LK64F
    double2 *row64;   // LK64R
    float4 *row32;    // LK32R
    uint4 *row16a;    // LK16R
    uint2 *row16b;
    float2 *full32;   // LK32F
};
hipError_t launch_gauge_ingest(const Geom &g, const double2 *U, const GaugeOut &o, double *partial_max,
                               hipStream_t st);

}  // namespace tmq
