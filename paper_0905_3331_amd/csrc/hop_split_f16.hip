// hop_split_f16.hip -- instantiations of the split half-sweep for one spinor format.
#include "hop_split.h"

namespace tmq {

template hipError_t launch_split<SpH16, L16R>(const Geom &, int, const FieldDesc &, const FieldDesc &,
                                                const FieldDesc &, const LinkDesc &, const OpParams &, int, int,
                                                const RhsList &, double *, long, const CgScalars *, int, int,
                                                hipStream_t, const CgFields *);

}  // namespace tmq
