// Host build of the choice of a hop launch's kernel (csrc/hop_form.h) for tests/test_hop_form.py.
#include "hop_form.h"

using namespace lqcd;

static ChunkGrid grid(const int* L) { return {{L[0], L[1], L[2], L[3]}, L[0] / 2, L[0] / 2 * L[1] * L[2] * L[3]}; }

extern "C" {

// The form for n lattices (L: 4 extents each) together, and the shape of a
// launch of it: out = split, halves, tile, lnt, next, built.
int form_of(int prec, int recon, int full, const int* L, int n, int nrhs, int rare, int* out)
{
    ChunkGrid g[16];
    for (int i = 0; i < n; ++i) g[i] = grid(L + 4 * i);
    const int form = hop_form(prec, recon, full != 0, g, n, nrhs, rare != 0);
    const HopShape h = hop_shape(prec, recon, full != 0, g[0], nrhs, form);
    out[0] = h.split;
    out[1] = h.halves;
    out[2] = h.tile;
    out[3] = h.lnt;
    out[4] = h.next;
    out[5] = hop_built(prec, recon, h.split, h.lnt, h.next);
    return form;
}

// Every hardware block of a launch of `slots` blocks per tile: counts[tile *
// slots + block] is raised for each that runs; returns the first inconsistency (0: none).
int block_cover(int slots, int tile, int adjacent, int nrhs, int swizzle, int* counts)
{
    ChunkArgs c = {};
    const int grid = (int)plan_tiles(&c, slots, tile, adjacent != 0, nrhs);
    const int ntiles = (nrhs + tile - 1) / tile;
    for (int bx = 0; bx < grid; ++bx) {
        uint32_t t, b;
        if (adjacent) tile_by_tile(c, swizzle, bx, &t, &b);
        else if (!tile_after_tile(c, swizzle, bx, &t, &b)) continue;
        if ((int)t >= ntiles) return 1;
        if ((int)b >= slots) return 2;
        ++counts[(int)t * slots + (int)b];
    }
    return 0;
}

// rhs_per_launch, and the work-items along x of a launch of that many.
int parts_of(int slots, int tile, int threads, int nrhs, long long* items)
{
    ChunkArgs c = {};
    const int n = rhs_per_launch(slots, tile, threads, nrhs);
    long long worst = 0;
    for (int adjacent = 0; adjacent < 2; ++adjacent) {
        const long long v = (long long)plan_tiles(&c, slots, tile, adjacent != 0, n) * threads;
        worst = v > worst ? v : worst;
    }
    *items = worst;
    return n;
}
}
