// Host build of the choice of a hop launch's kernel (csrc/hop_form.h) for tests/test_hop_form.py.
#include "hop_form.h"

using namespace lqcd;

static ChunkGrid grid(const int* L) { return {{L[0], L[1], L[2], L[3]}, L[0] / 2, L[0] / 2 * L[1] * L[2] * L[3]}; }

extern "C" {

// The form for n lattices (L: 4 extents each) together, and the shape of a
// launch of it: out = split, halves, tile, lnt, built.
int form_of(int prec, int recon, int full, const int* L, int n, int nrhs, int* out)
{
    ChunkGrid g[16];
    for (int i = 0; i < n; ++i) g[i] = grid(L + 4 * i);
    const int form = hop_form(prec, recon, full != 0, g, n, nrhs);
    const HopShape h = hop_shape(form, full != 0, nrhs);
    out[0] = h.split;
    out[1] = h.halves;
    out[2] = h.tile;
    out[3] = h.lnt;
    out[4] = hop_built(prec, h.split, h.lnt);
    return form;
}
}
