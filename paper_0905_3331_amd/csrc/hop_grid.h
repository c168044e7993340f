// hop_grid.h -- lattice geometry and the launch grids of the half-sweeps, plain
// C++ (host code, and the bound of the partial sums' array checked on the CPU).
#pragma once

namespace tmq {

// Lattice geometry.  Extents (T, LZ, LY, LX) all even; V/2 sites per parity,
// eo index h = site >> 1 with site = ((t*LZ + z)*LY + y)*LX + x.
struct Geom {
    int T, LZ, LY, LX;
    int XH;   // LX / 2
    long vh;  // V / 2
};

constexpr int HOP_BLOCK = 256;
constexpr int BLAS_BLOCK = 256;
// partial sums that a block of 256 lanes leaves, one per wavefront (the split
// half-sweep's blocks hold a wavefront's sites, so a sum does not depend on the kernel)
constexpr int PARTS = 4;

inline int blas_grid(long n) { return (int)((n + BLAS_BLOCK - 1) / BLAS_BLOCK); }
inline int hop_grid(long n)
{
    long g = (n + HOP_BLOCK - 1) / HOP_BLOCK;
    g = (g + 7) / 8 * 8;  // a multiple of the XCD count for the remap
    return (int)g;
}

// hop kernel variants (see hop_impl.h): 0 plain order, 1 z-slabs per XCD, 2
// z-slabs + scheduling barriers, 3 t-slabs per XCD, 4 t-slabs + barriers.
// z-slabs need LZ >= 8, t-slabs T >= 8.  Links are loaded non-temporally in
// single-RHS launches and cached in batched ones.
enum HopOrder { ORD_PLAIN = 0, ORD_ZSLAB = 1, ORD_TSLAB = 2 };
constexpr int HOP_VARIANTS = 5;
inline int hop_order(int v) { return v == 0 ? ORD_PLAIN : v <= 2 ? ORD_ZSLAB : ORD_TSLAB; }
inline bool hop_variant_valid(const Geom &g, int v)
{
    if (v < 0 || v >= HOP_VARIANTS) return false;
    if (hop_order(v) == ORD_ZSLAB) return g.LZ >= 8;
    if (hop_order(v) == ORD_TSLAB) return g.T >= 8;
    return true;
}
// blocks of HOP_BLOCK lanes per RHS of variant v (PARTS partial sums each with a
// norm): every XCD has as many as the largest slab needs.  lanes_per_site = 2
// for doublets in the general kernel (a lane pair per site) and in the split one.
inline int hop_grid_variant(const Geom &g, int v, int lanes_per_site = 1)
{
    const long L = lanes_per_site;
    if (!hop_variant_valid(g, v) || hop_order(v) == ORD_PLAIN) return hop_grid(L * g.vh);
    const bool zs = hop_order(v) == ORD_ZSLAB;
    const long extent = zs ? g.LZ : g.T, other = zs ? g.T : g.LZ;
    const long sites = other * ((extent + 7) / 8) * g.LY * g.XH;
    return (int)(8 * ((L * sites + HOP_BLOCK - 1) / HOP_BLOCK));
}

// room for the partial sums of one RHS (or doublet): those of any half-sweep,
// and of any vector pass over 2 V/2 sites.  With an extent that eight does not
// divide, a slab order has more blocks than the plain one (1.6 times for 10).
inline long hop_partials(const Geom &g)
{
    long n = blas_grid(2 * g.vh);
    for (int v = 0; v < HOP_VARIANTS; v++)
        for (int lanes = 1; lanes <= 2; lanes++) {
            const long k = hop_grid_variant(g, v, lanes);
            if (k > n) n = k;
        }
    return PARTS * n;
}

}  // namespace tmq
