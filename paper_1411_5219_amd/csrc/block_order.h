// Where a block and a work-item of a stencil launch work: the output site of
// the work-item in the launch's block order and the neighbours of that site.
// Shared by the Wilson and the staggered hop kernels, which walk the lattice
// the same way.
#pragma once

#include "lqcd_device.h"
#include "lqcd_kernels.h"

namespace lqcd {

// Neighbour of an output site for hop K = 2 mu + (0 forward, 1 backward):
// the neighbour's parity-local index, the link block (mu, parity) and the
// parity-local site the link is stored at, and whether the hop crosses the
// lattice boundary (and so takes the boundary phase).
// Parity-local indices fit 32 bits (the library limits V/2 to 21 * 2^20),
// which keeps them in one register each.
struct Nbr {
    int nb, lsite;
    int lblk;
    bool cross;
};

struct SiteGeo {
    int x, y, z, t, p, Lx, Ly, Lz, Lt;
    int h, base, hy, hz, ht;

    template <int K>
    __device__ __forceinline__ Nbr get() const
    {
        constexpr int MU = K >> 1;
        constexpr bool FWD = (K & 1) == 0;
        Nbr n;
        if constexpr (MU == 0) {
            if constexpr (FWD) {
                n.cross = x == Lx - 1;
                n.nb = base + ((n.cross ? 0 : x + 1) >> 1);
            } else {
                n.cross = x == 0;
                n.nb = base + ((n.cross ? Lx - 1 : x - 1) >> 1);
            }
        } else {
            const int c = MU == 1 ? y : MU == 2 ? z : t;
            const int Lc = MU == 1 ? Ly : MU == 2 ? Lz : Lt;
            const int hc = MU == 1 ? hy : MU == 2 ? hz : ht;
            if constexpr (FWD) {
                n.cross = c == Lc - 1;
                n.nb = n.cross ? h - (Lc - 1) * hc : h + hc;
            } else {
                n.cross = c == 0;
                n.nb = n.cross ? h + (Lc - 1) * hc : h - hc;
            }
        }
        // U_mu(x) for forward hops, U_mu(x - mu) (stored at the neighbour) for backward ones
        n.lblk = 2 * MU + (FWD ? p : 1 - p);
        n.lsite = FWD ? h : n.nb;
        return n;
    }
};

__device__ __forceinline__ SiteGeo site_geo(const Geom& g, const SitePos& s, int p)
{
    const int Lxh = g.Lxh, Ly = g.L[1], Lz = g.L[2];
    return SiteGeo{s.x, s.y, s.z, s.t, p, g.L[0], Ly, Lz, g.L[3], s.h, s.h - s.xh, Lxh, Lxh * Ly, Lxh * Ly * Lz};
}

}  // namespace lqcd
