// Which waves serve the sites and the right-hand sides of a Wilson hop launch
// (plain C++: compiled into the library by hipcc and by a host compiler for
// its test).
#pragma once

#include <stdint.h>

#include "chunks.h"

namespace lqcd {

constexpr int kSimds = 1024;  // 256 compute units of 4 SIMDs

// Right-hand sides of a block (the kernel's bound).  Their spinors share the
// XCD's L2: 32^3x8 FP32/12 Schur on 12 right-hand sides 206 us with 4 per
// block, 218 with 3, 245 with 2; 8 per block read more from beyond L2 (296).
constexpr int kMaxTile = 4;

// How the waves of a Wilson hop share sites and right-hand sides: one wave or
// a pair of waves per chunk of 64 sites and right-hand side, the right-hand
// sides one after the other or (FORM_NEXT, pairs) next to each other in the
// block order, or a tile of right-hand sides per chunk with its links in LDS,
// and in this one wave per right-hand side, or (tiles of two) two.  FORM_WAVE on
// several right-hand sides, next to each other, is the persistent kernel's.
enum HopForm { FORM_BY_SIZE = 0, FORM_WAVE = 1, FORM_PAIR = 2, FORM_TILE = 3, FORM_NEXT = 5 };

// What hop_form and hop_shape know of a lattice: whether its planes leave
// lanes of their last chunk idle, so that chunks run over several of them, and
// whether with that its time extent is long.  The blocks of such a layer lie
// t, then the layer's sites, apart from their z neighbours, which leave the L2
// meanwhile; in memory order the sites between a block and its t neighbours are
// one spatial volume.  Four right-hand sides, layers against memory order,
// FP64/18: tiles 24^3x48 306 us against 244; pairs 18^3x12 27.5 against 25.5,
// 20^3x10 32.6 against 29.0, 24^3x8 38.8 against 38.0; where planes split evenly
// memory order loses (32^3x8 tiles 81.0 against 97.2).
inline bool layered(const ChunkGrid& g) { return layer_planes(g, 20) > 1; }
inline bool long_layers(const ChunkGrid& g) { return layered(g) && g.L[3] >= 10; }

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
// Several: pairs, or tiles of up to four per block with the links in LDS
// (hop_rhs.h).  Pairs while all of them run at once (two waves per SIMD in FP64,
// three below: FP32/12 Schur complement 8^3x4 with four 9.8 us against 13.3,
// 16^3x8 with four 15.0 against 16.8), one right-hand side after the other, which
// is 0.1 to 0.2 us shorter; the full matrix of FP64/12 on
// small lattices up to five waves (12^3x8 n16 33.0 us, next to each other 36.4;
// 16^3x8 n8 37.8 and 39.9; but 18^3x8 n6 47.5 and 46.7).  Beyond that pairs with the right-hand sides of a
// chunk next to each other, so that all but one find its links in L2 (FP64/18
// 24^3x8 n8 104 -> 66.4 us); us of one hop as such pairs and as tiles, n
// right-hand sides:
//   FP64: tiles where they all run at once, two blocks per compute unit (18:
//     16^3x8 n6 17.6 and 15.3, 20^3x8 n3 20.4 and 18.5; 12: 10x14x18x22 n4 20.5
//     and 18.9), not for both parities (16^3x8 n6 32.8 and 32.9, 20^3x6 n8 64.0
//     and 76.9).  Then pairs while links and spinors take up to twice the
//     Infinity Cache (18: 24^3x8 n8 66.4 and 81.0, n16 125 and 156, 26^3x8 n12
//     128 and 159, 28^3x8 n12 178 and 197, n16 275 and 261), or with whole planes
//     while the lattice gives a SIMD less than two chunks (18: 22^3x8 n16 104
//     and 125, 16^3x32 n12 112 and 155; 32^3x8 n4 82.4 and 80.7, n12 280 and 246).
//   rare: the FP64 hops of a mixed solve's reliable updates, which hardly any
//     launch finds pending: tiles, whose launch then costs less (k_hop_rhs_update).
//   FP32: tiles with 18-real links (36^3x8 n2 37.1 and 36.0) and for both parities
//     (24^3x8 n8, 12 reals 59.3 and 55.5; 32^3x8 n12 268 and 193).  One parity,
//     12 reals: pairs up to three right-hand sides (32^3x8 n3 26.5 and 30.0, n2
//     20.2 and 21.8; 48^3x8 n3, 425 MB, 116 and 101) and on large lattices in
//     layers (36^3x8 n4 49.9 and 56.7, n8 91.4 and 108.6), both up to 400 MB, and on
//     long ones in layers (24^3x16 n8 58.0 and 65.5); else tiles (32^3x8 n4 33.0
//     and 33.0, n12 99 and 84; 24^3x8 n8 30.5 and 30.1; 26^3x8 n16 75 and 70).
//   FP16 with two or three, whose tiles wait for LDS: pairs (48^3x12 Schur n2
//     135 and 147, 28^3x8 n3 34.0 and 36.4, n4 41.0 and 40.6) up to 512 MB
//     (48^3x24 n2 147 and 137, n3 209 and 197).
inline int hop_form(int prec, int recon, bool full, const ChunkGrid* g, int n, int nrhs, bool rare = false)
{
    int64_t chunks = 0, sites = 0, in_layers = 0, in_long = 0;
    for (int i = 0; i < n; ++i) {
        chunks += (g[i].Vh + kChunk - 1) / kChunk;
        sites += g[i].Vh;
    }
    if (nrhs == 1) {
        bool wave = prec == 64 && recon == 18 && !full && chunks >= 2 * kSimds;
        for (int i = 0; wave && i < n; ++i) {
            const ChunkArgs c = plan_chunk_order(g[i], 1, 256, 1, 4);
            wave = c.planes == 1 && c.nsub > 1 && c.chunks % c.nsub == 0;
        }
        return wave ? FORM_WAVE : FORM_PAIR;
    }
    const int waves = prec != 64 ? 3 : recon == 12 && full && 4 * chunks <= kSimds ? 5 : 2;  // per SIMD
    if (2 * chunks * nrhs <= waves * kSimds) return FORM_PAIR;
    for (int i = 0; i < n; ++i) {
        const int64_t own = (g[i].Vh + kChunk - 1) / kChunk;
        in_layers += layered(g[i]) ? own : 0;
        in_long += long_layers(g[i]) ? own : 0;
    }
    // links once, each spinor of the hop's parity or parities read and written once
    const int spinor = 3 * prec + (prec == 16 ? 4 : 0);  // bytes (FP16: with the site's scale)
    const int64_t mb = sites * (recon * prec + (full ? 4 : 2) * nrhs * spinor) / 1000000;
    const bool layers = 2 * in_layers > chunks;
    bool pair;
    if (prec == 16) pair = nrhs <= 3 && mb <= 512;
    else if (prec == 64)
        pair = !rare && (full || chunks * ((nrhs + kMaxTile - 1) / kMaxTile) > kSimds / 2) && mb <= 512 &&
               (layers || chunks < 2 * kSimds);
    else if (full || recon == 18) pair = false;
    else if (2 * in_long > chunks && nrhs >= 4) pair = mb <= 512;
    else pair = mb <= 400 && (nrhs <= 3 || (layers && chunks > 2 * kSimds));
    return pair ? FORM_NEXT : FORM_TILE;
}

// What a launch of a form runs: the kernel (split, halves, lnt), its blocks and
// their order.
struct HopShape {
    int split;   // waves per chunk of sites, 0: several right-hand sides per block
    int halves;  // split = 0: waves per right-hand side
    int tile;    // right-hand sides per block
    bool lnt;    // streaming link loads (no other block of the launch reads the links)
    bool next;   // right-hand sides next to each other in the block order
    int idle;    // idle lanes of a layer: at most one of these (plan_chunk_order)
    bool memory; // memory order where the order asked for is 1
};
// idle, for several right-hand sides: a plane of which an eighth is idle runs by
// itself where the L2 is crowded and more than a few rounds of blocks follow:
// FP64 tiles (18 reals, 30^3x8 n16 343 -> 309 us against a sixteenth, 36^3x8 n8
// 299 -> 283; in few rounds they take the layers with the fewest idle lanes,
// 20^3x8 n3 makes 512 blocks of five planes, 520 of four: 52 -> 41), and both
// parities of FP32/12 (26^3x8 n8 82.2 -> 70.9, 30^3x8 n8 128 -> 104; not with two
// or three on small lattices, 24^3x8 n3 24.2 against 26.6, nor on long ones,
// 24^3x48 n3 170 against 183); else FP32 tiles a sixteenth (44^3x6 n4 175 -> 145;
// an eighth 28^3x8 n8 45.3 against 49.7) and FP32 pairs next to each other a
// twelfth (36^3x8 n4 53.0 -> 49.9, 44^3x6 n3 56.2 -> 48.9; an eighth 28^3x8 n2
// 15.0 against 16.6).
inline HopShape hop_shape(int prec, int recon, bool full, const ChunkGrid& g, int nrhs, int form)
{
    HopShape s = {};
    const int64_t chunks = (g.Vh + kChunk - 1) / kChunk;
    if (form == FORM_TILE) {
        // several right-hand sides share a block and the links in its LDS: as
        // few tiles of at most kMaxTile as there can be, of even sizes
        const int ntiles = (nrhs + kMaxTile - 1) / kMaxTile;
        s.tile = (nrhs + ntiles - 1) / ntiles;
        s.halves = s.tile <= 2 ? 2 : 1;
        const bool crowded = full && recon == 12 && g.L[3] < 10 && (nrhs >= 4 || chunks > kSimds);
        s.idle = prec == 16 ? 20 : prec == 64 ? (chunks * ntiles <= 2 * kSimds ? 40 : 8) : crowded ? 8 : 16;
        s.memory = prec == 64 && nrhs > 1 && long_layers(g);
        return s;
    }
    s.split = form == FORM_WAVE ? 1 : 2;
    s.halves = 1;
    s.tile = 1;
    s.lnt = nrhs == 1 && !full;
    s.next = form == FORM_NEXT || (form == FORM_WAVE && nrhs > 1);
    s.idle = s.next && prec == 32 ? 12 : 20;
    s.memory = nrhs > 1 && long_layers(g) && (prec == 64 || (s.next && prec == 32 && recon == 12 && !full && nrhs >= 4));
    // the persistent kernel's blocks have four waves: all of them busy
    if (form == FORM_WAVE && nrhs > 1) s.memory = plan_chunk_order(g, 1, 256, 1, 4, s.idle).nsub < 4;
    return s;
}

// Whether the launch's kernel is built: what hop_form chooses.  One wave per
// chunk can be the faster split with FP64/18 on one parity and right-hand side,
// pairs next to each other with every storage but FP32/18.
constexpr bool hop_built(int prec, int recon, int split, bool lnt, bool next)
{
    return split == 1   ? prec == 64 && recon == 18 && lnt && !next
           : split == 2 ? !next || (!lnt && !(prec == 32 && recon == 18))
                        : !lnt && !next;
}

}  // namespace lqcd
