// hop.hip -- dispatch of the hopping half-sweep to the per-format translation
// units.
#include "devutil.h"
#include "views.h"

namespace tmq {

bool hop_all_variants(int prec, int link_fmt)
{
    // the pairings of a solve's inner iteration and of FP64; the others
    // (FP32 spinors on FP16 links, 16-bit spinors on FP32 links) are
    // instantiated with the plain order only
    if (prec == P64) return true;
    if (prec == P32) return link_fmt == LK32R;
    return link_fmt == LK16R;
}

// per-format entry points (hop_f64.hip, hop_f32.hip, hop_f16.hip)
#define TMQ_HOP_ARGS                                                                                       \
    const Geom &g, int out_par, const FieldDesc &in, const FieldDesc &self, const FieldDesc &out,           \
        const LinkDesc &lk, const OpParams &op, int epi, int sign, const RhsList &rl, double *partial,      \
        long pstride, const CgScalars *scal, const HopTune &tu, hipStream_t st, const CgFields *cg
hipError_t launch_hop_f64(TMQ_HOP_ARGS);
hipError_t launch_hop_f32(TMQ_HOP_ARGS);
hipError_t launch_hop_f16(TMQ_HOP_ARGS);
hipError_t launch_hop_b16(TMQ_HOP_ARGS);

hipError_t launch_hop(TMQ_HOP_ARGS)
{
    const bool fused = epi == EPI_K2_CG || epi == EPI_K2_RES;  // no output field
    if ((!fused && in.prec != out.prec) || (self.data && self.prec != in.prec)) return hipErrorInvalidValue;
    switch (in.prec) {
    case P64: return launch_hop_f64(g, out_par, in, self, out, lk, op, epi, sign, rl, partial, pstride, scal, tu, st, cg);
    case P32: return launch_hop_f32(g, out_par, in, self, out, lk, op, epi, sign, rl, partial, pstride, scal, tu, st, cg);
    case P16: return launch_hop_f16(g, out_par, in, self, out, lk, op, epi, sign, rl, partial, pstride, scal, tu, st, cg);
    case PB16: return launch_hop_b16(g, out_par, in, self, out, lk, op, epi, sign, rl, partial, pstride, scal, tu, st, cg);
    }
    return hipErrorInvalidValue;
}

}  // namespace tmq
