// Which waves serve the sites and the right-hand sides of a Wilson hop launch
// (plain C++: compiled into the library by hipcc and by a host compiler for
// its test).
#pragma once

#include <stdint.h>

#include "chunks.h"

namespace lqcd {

constexpr int kSimds = 1024;  // 256 compute units of 4 SIMDs

// Right-hand sides of a block (the kernel's bound).  Their spinors share the
// XCD's L2: 32^3x8 FP32/12 Schur on 12 right-hand sides 207 us with 4 per
// block, 218 with 3, 245 with 2; 8 per block read more from beyond L2 (296).
constexpr int kMaxTile = 4;

// How the waves of a Wilson hop share sites and right-hand sides: one wave or
// a pair of waves per chunk of 64 sites and right-hand side, or a tile of
// right-hand sides per chunk with its links in LDS, and in this one wave per
// right-hand side, or (FORM_TILE only, by size) two.
enum HopForm { FORM_BY_SIZE = 0, FORM_WAVE = 1, FORM_PAIR = 2, FORM_TILE = 3, FORM_TILE_WAVE = 4 };

// Which waves serve a launch's sites and right-hand sides, for the n systems
// of a batch together.
// One right-hand side: a pair of waves per chunk (see dslash_block) except
// where one wave per chunk fills every wave slot of the chip, two per SIMD at
// its register count, planes split evenly into blocks of such waves, and each
// link is read once and whole: there FP64/18, which streams at the memory's
// rate either way, loses by the second wave's indices and the exchange
// (48^3x12 186 us with one wave, 193 with two; 32^3x8, exactly full, 36.5 and
// 38.2; 24^3x8, half full, 20.2 and 18.5; 40^3x6, uneven, 66 and 59; FP64/12
// 48^3x8 103 and 99).
// Several: a tile of them per block (hop_rhs.h) once the pairs of all of them
// would no longer run at once, two waves per SIMD in FP64 and three below;
// before that the pairs are faster, each on its own right-hand side (Schur
// complement, FP32/12: 8^3x4 with four 9.8 us against 13.3, 16^3x8 with four
// 15.0 against 16.8, with twelve 33.1 against 29.7; FP64/18 20^3x8 with two
// 35.6 against 45.5, 20^3x6 with four 47 against 41).  FP64/12 stays with pairs
// up to five waves per SIMD: tiles hold all 18 reals in LDS (20^3x8 with four
// 53 against 61, 24^3x8 with three 71 against 68); so does FP16 storage with
// two or three, whose tiles wait for LDS (48^3x12 with two 135 against 147,
// 28^3x8 with three 34.0 against 36.4, with four 41.0 against 40.6).
inline int hop_form(int prec, int recon, bool full, const ChunkGrid* g, int n, int nrhs)
{
    int64_t chunks = 0;
    bool even = true;
    for (int i = 0; i < n; ++i) {
        const ChunkArgs c = plan_chunk_order(g[i], 1, 256, 1, 4);
        chunks += (g[i].Vh + kChunk - 1) / kChunk;
        even = even && c.planes == 1 && c.nsub > 1 && c.chunks % c.nsub == 0;
    }
    if (nrhs > 1) {
        const int64_t waves = 2 * chunks * nrhs;
        const bool pair = prec == 64 ? waves <= (recon == 12 ? 5 : 2) * kSimds
                                     : waves <= 3 * kSimds || (prec == 16 && nrhs <= 3);
        return pair ? FORM_PAIR : FORM_TILE;
    }
    return prec == 64 && recon == 18 && !full && even && chunks >= 2 * kSimds ? FORM_WAVE : FORM_PAIR;
}

// What a launch of a form runs: the kernel (split, halves, lnt) and its blocks.
struct HopShape {
    int split;   // waves per chunk of sites, 0: several right-hand sides per block
    int halves;  // split = 0: waves per right-hand side
    int tile;    // right-hand sides per block
    bool lnt;    // streaming link loads (no other block of the launch reads the links)
};
inline HopShape hop_shape(int form, bool full, int nrhs)
{
    if (form == FORM_TILE || form == FORM_TILE_WAVE) {
        // several right-hand sides share a block and the links in its LDS: as
        // few tiles of at most kMaxTile as there can be, of even sizes
        const int ntiles = (nrhs + kMaxTile - 1) / kMaxTile, tile = (nrhs + ntiles - 1) / ntiles;
        return {0, form == FORM_TILE && tile <= 2 ? 2 : 1, tile, false};
    }
    return {form == FORM_WAVE ? 1 : 2, 1, 1, nrhs == 1 && !full};
}

// Whether the launch's kernel is built.  One wave per chunk is built only
// where it can be the faster split: FP64 on one parity and right-hand side.
constexpr bool hop_built(int prec, int split, bool lnt) { return split != 1 || (prec == 64 && lnt); }

}  // namespace lqcd
