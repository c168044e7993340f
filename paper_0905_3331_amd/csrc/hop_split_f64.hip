// hop_split_f64.hip -- instantiations of the split half-sweep for one spinor format.
#include "hop_split_nd.h"

namespace tmq {

template hipError_t launch_split<SpF64, L64F>(const Geom &, int, const FieldDesc &, const FieldDesc &,
                                                const FieldDesc &, const LinkDesc &, const OpParams &, int, int,
                                                const RhsList &, double *, long, const CgScalars *, int, int,
                                                hipStream_t, const CgFields *);
template hipError_t launch_split<SpF64, L64R>(const Geom &, int, const FieldDesc &, const FieldDesc &,
                                                const FieldDesc &, const LinkDesc &, const OpParams &, int, int,
                                                const RhsList &, double *, long, const CgScalars *, int, int,
                                                hipStream_t, const CgFields *);
template hipError_t launch_split_nd<SpF64, L64F>(const Geom &, int, const FieldDesc &, const FieldDesc &,
                                                   const FieldDesc &, const LinkDesc &, const OpParams &, int, int,
                                                   const RhsList &, double *, long, const CgScalars *, int, int,
                                                   hipStream_t, const CgFields *);
template hipError_t launch_split_nd<SpF64, L64R>(const Geom &, int, const FieldDesc &, const FieldDesc &,
                                                   const FieldDesc &, const LinkDesc &, const OpParams &, int, int,
                                                   const RhsList &, double *, long, const CgScalars *, int, int,
                                                   hipStream_t, const CgFields *);

}  // namespace tmq
