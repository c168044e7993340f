// Host build of the half-sweeps' launch grids (hop_grid.h), so that the room
// for their partial sums can be checked on the CPU.
#include "../../paper_0905_3331_amd/csrc/hop_grid.h"

using namespace tmq;

static Geom geom(const int *d) { return Geom{d[0], d[1], d[2], d[3], d[3] / 2, (long)d[0] * d[1] * d[2] * d[3] / 2}; }

extern "C" long grid_partials(const int *d) { return hop_partials(geom(d)); }
extern "C" int grid_variant(const int *d, int v, int lanes) { return hop_grid_variant(geom(d), v, lanes); }
extern "C" int grid_vector(long n) { return blas_grid(n); }
