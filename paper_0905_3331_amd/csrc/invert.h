// invert.h -- the vector passes of M psi = phi through the even/odd system
// (solve_M_batch), each one launch for all right-hand sides.  Fields are FP64;
// partial sums are left as launch_norm2 leaves them, for blas_grid(2 vh) blocks.
#pragma once
#include "kernels.h"

namespace tmq {

// a canonical buffer per right-hand side
struct CanList {
    double2 *p[MAX_RHS];
};

// r = phi (full lattice), te = diag(cu, cd) phi on the even sites, partial |phi|^2
hipError_t launch_m_enter(const Geom &g, const CanList &phi, const FieldDesc &r, const FieldDesc &te, double2 cu,
                          double2 cd, const RhsList &rl, double *partial, long pstride, hipStream_t st);
// r = phi - g5 q (full lattice), partial |r|^2
hipError_t launch_m_residual(const Geom &g, const CanList &phi, const FieldDesc &q, const FieldDesc &r,
                             const RhsList &rl, double *partial, long pstride, hipStream_t st);
// a batched field to the canonical buffers of a like batch (lower spins times down = 1 or -1), and back
hipError_t launch_m_to_canonical(const FieldDesc &in, const FieldDesc &can, double down, const RhsList &rl,
                                 hipStream_t st);
hipError_t launch_m_from_canonical(const FieldDesc &can, const FieldDesc &out, const RhsList &rl, hipStream_t st);
// psi = x (full lattice)
hipError_t launch_m_leave(const Geom &g, const FieldDesc &x, const CanList &psi, const RhsList &rl, hipStream_t st);

}  // namespace tmq
