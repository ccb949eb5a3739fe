// The order in which the blocks of a hop launch walk the lattice (plain C++:
// compiled into the library by hipcc and by a host compiler for its test).
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define LQCD_CHUNK_FN __host__ __device__ __forceinline__
#else
#define LQCD_CHUNK_FN inline
#endif

namespace lqcd {

constexpr int kChunk = 64;  // sites of a chunk, one per lane of a wave

// Division of 31-bit numbers by a launch constant: n / d = mulhi(n, m) >> s
// with m = ceil(2^(31 + l) / d), l = ceil(log2 d), s = l - 1, exact for
// n < 2^31 (m d - 2^(31 + l) < d <= 2^l); m = 0 stands for d = 1.
struct FastDiv {
    uint32_t d, m, s;
};
inline FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f{d, 0, 0};
    if (d <= 1) return f;
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    f.m = (uint32_t)(((1ull << (31 + l)) + d - 1) / d);
    f.s = l - 1;
    return f;
}
LQCD_CHUNK_FN uint32_t fdiv(const FastDiv& f, uint32_t n)
{
    return f.m ? (uint32_t)(((uint64_t)n * f.m) >> 32) >> f.s : n;
}

// Block order of a hop launch.  The sites of one parity are cut into layers of
// `planes` consecutive xy planes and these into chunks of 64 consecutive sites
// (the last chunk of a layer may be ragged); a block covers nsub consecutive
// chunks, and the spatial blocks run z within a slab of ztile layers fastest,
// then t, then `group` neighbouring blocks of the layer, then the slab, then
// the next group: the t and z neighbours a block reads were loaded by blocks
// that ran just before it on the same XCD, and with a group the rows just
// outside its chunks too.  chunks = 0: chunks of the whole parity in memory
// order.  Full-lattice launches alternate the parities of each spatial block.
struct ChunkArgs {
    int chunks;      // chunks per layer (0: memory order)
    int planes;      // xy planes of a layer
    int nsub;        // chunks per block
    int nsp;         // spatial blocks per parity
    int tile;        // right-hand sides per block
    int nblk;        // blocks of one right-hand-side tile
    // Tiles run one after the other, or (hops by pairs of waves) next to each
    // other on each spatial block.
    FastDiv stride;  // one after the other: hardware blocks of a tile, nblk, with several rounded up to a multiple of 8
    FastDiv tiles;   // next to each other: how many
    FastDiv Lxh, Ly, Lz, Lt, plane, group, slabs, ztile;
};

// Extents (x, y, z, t), sites per parity and sites per half x-row.
struct ChunkGrid {
    int L[4];
    int Lxh, Vh;
};

// xy planes of a layer: one where its last chunk leaves at most one of idle_max
// of the lanes idle, else the fewest planes (a divisor of Lz up to 8) that do,
// or that leave the fewest idle: 20^3x8 has 200 sites per plane, 78% of four
// chunks, but 800 in four planes, 96% of 13 (FP64 Schur complement on four
// right-hand sides 66.7 us with one plane, 59.9 with four).
inline int layer_planes(const ChunkGrid& g, int idle_max)
{
    const int plane = g.Lxh * g.L[1];
    auto lanes_of = [&](int n) { return (int64_t)((plane * n + kChunk - 1) / kChunk) * kChunk; };
    int planes = 1;
    for (int n = 1; n <= 8 && n <= g.L[2]; ++n) {
        if (g.L[2] % n) continue;
        const int64_t idle = lanes_of(n) - (int64_t)plane * n, best = lanes_of(planes) - (int64_t)plane * planes;
        if (idle_max * best <= lanes_of(planes)) break;
        if (idle * lanes_of(planes) < best * lanes_of(n)) planes = n;
    }
    return planes;
}

// Plan for blocks of at most maxsub chunks of 64 sites.  order 0: memory
// order; k >= 1: layers, in z-slabs of the largest divisor of the layers with at most
// k planes; block and ygroup: the sites of a layer that are neighbours in the order
// (block requests of work-items, one per site, times ygroup).
inline ChunkArgs plan_chunk_order(const ChunkGrid& g, int order, int block, int ygroup, int maxsub, int idle_max = 20)
{
    ChunkArgs c = {};
    const int plane = g.Lxh * g.L[1];
    const int64_t flat = (g.Vh + kChunk - 1) / kChunk;
    auto chunks_of = [&](int n) { return (plane * n + kChunk - 1) / kChunk; };
    c.planes = layer_planes(g, idle_max);
    const int per = chunks_of(c.planes), layers = g.L[2] / c.planes;
    // chunks of layers unless memory order is asked for; a lattice so wide and
    // flat that its ragged layers would take more slots than the caller's
    // partials hold (one per x-row or per 64 sites) runs in memory order too
    const int64_t rows = (int64_t)g.L[1] * g.L[2] * g.L[3];
    c.chunks = order == 0 || (int64_t)per * layers * g.L[3] > (rows > flat ? rows : flat) ? 0 : per;
    c.nsub = 1;
    int group = 1, ztile = 1;
    if (c.chunks) {
        // most chunks per block that fill every wave, or else waste at most a fifth of a layer's
        for (int n = 2; n <= maxsub; ++n)
            if (c.chunks % n == 0) c.nsub = n;
        for (int n = 2; n <= maxsub && c.nsub == 1; ++n)
            if (5 * c.chunks >= 4 * ((c.chunks + n - 1) / n) * n) c.nsub = n;
        const int blocks = (c.chunks + c.nsub - 1) / c.nsub;
        const int want = (block / kChunk + c.nsub - 1) / c.nsub * (ygroup > 1 ? ygroup : 1);
        // a layer of several planes is one group: its z neighbours are its own
        // chunks; a plane a little larger than the request is too
        if (c.planes > 1 || 2 * blocks <= 3 * want) group = blocks;
        else
            for (int d = 1; d <= want; ++d)
                if (blocks % d == 0) group = d;
        for (int d = 1; d <= layers && d * c.planes <= order; ++d)
            if (layers % d == 0) ztile = d;
        c.nsp = blocks * layers * g.L[3];
    } else {
        c.nsub = maxsub;
        c.nsp = (int)((flat + maxsub - 1) / maxsub);
    }
    c.Lxh = make_fastdiv((uint32_t)g.Lxh);
    c.Ly = make_fastdiv((uint32_t)g.L[1]);
    c.Lz = make_fastdiv((uint32_t)g.L[2]);
    c.Lt = make_fastdiv((uint32_t)g.L[3]);
    c.plane = make_fastdiv((uint32_t)plane);
    c.group = make_fastdiv((uint32_t)group);
    c.slabs = make_fastdiv((uint32_t)(layers / ztile));
    c.ztile = make_fastdiv((uint32_t)ztile);
    return c;
}

// Lays out a launch of `slots` blocks per tile (all parities); returns its
// hardware blocks.
inline unsigned plan_tiles(ChunkArgs* c, int slots, int tile, bool adjacent, int nrhs)
{
    const unsigned ntiles = (unsigned)((nrhs + tile - 1) / tile), n = (unsigned)slots;
    const unsigned stride = ntiles > 1 && !adjacent ? (n + 7) / 8 * 8 : n;
    c->tile = tile;
    c->nblk = slots;
    c->tiles = make_fastdiv(ntiles);
    c->stride = make_fastdiv(stride);
    return stride * ntiles;
}

// Right-hand sides of one launch whose blocks, `slots` to a tile of them, have
// `threads` work-items: as even parts as keep the work-items along x below 2^32,
// HIP's limit (plan_tiles adds at most 7 blocks to a tile).
inline int rhs_per_launch(int slots, int tile, int threads, int nrhs)
{
    const int64_t most = (int64_t)0xffffffff / threads / ((int64_t)slots + 7) * tile;
    const int64_t parts = (nrhs + most - 1) / most;
    return (int)((nrhs + parts - 1) / parts);
}

// Block index remap that hands each XCD a contiguous range of logical
// blocks.  Workgroups are dispatched round-robin over the 8 XCDs, so
// hardware block b runs on XCD b % 8; giving that XCD logical blocks
// [start(b%8), start(b%8) + count) keeps neighbouring sites in one L2.
LQCD_CHUNK_FN int xcd_swizzle(int b, int nb)
{
    const int q = nb >> 3, rem = nb & 7;
    const int xcd = b & 7, k = b >> 3;
    const int start = xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q;
    return start + k;
}

// Right-hand-side tile and logical block of hardware block bx, tiles one after
// the other.  Every tile takes a multiple of 8 hardware blocks, so that with
// the XCD remap a spatial block runs on the same XCD for every tile and a later
// tile can find the links in that XCD's L2; false for the padding.
LQCD_CHUNK_FN bool tile_after_tile(const ChunkArgs& c, int swizzle, int bx, uint32_t* tile, uint32_t* b)
{
    *tile = fdiv(c.stride, (uint32_t)bx);
    const int x = bx - (int)(*tile * c.stride.d);
    if (x >= c.nblk) return false;
    *b = (uint32_t)(swizzle ? xcd_swizzle(x, c.nblk) : x);
    return true;
}

// The same with the tiles next to each other: with the XCD remap they run one
// after the other on one XCD, and all but the first find the links in its L2.
// No hardware block is padding: a second test at the top of the kernel, or the
// two orders as one function, lengthened the smallest hops by 0.1 to 0.8 us.
LQCD_CHUNK_FN void tile_by_tile(const ChunkArgs& c, int swizzle, int bx, uint32_t* tile, uint32_t* b)
{
    const uint32_t y = (uint32_t)(swizzle ? xcd_swizzle(bx, c.nblk * (int)c.tiles.d) : bx);
    *b = fdiv(c.tiles, y);
    *tile = y - *b * c.tiles.d;
}

struct SitePos {
    int h;            // parity-local index of the output site
    int xh, x, y, z, t;
    bool valid;       // false for lanes past the end, which repeat the last site
    bool some;        // some lane of the wave is valid (uniform)
};

// Site of lane `lane` of parity p in chunk `sub` of spatial block b.
// Divisions are by launch constants (FastDiv), and t is uniform over the
// wave unless the chunks run in memory order, and so is z with one plane per
// layer.
LQCD_CHUNK_FN SitePos chunk_site(const ChunkArgs& c, int Lxh, int Ly, int Lz, int Vh, uint32_t b, int sub, int p,
                                 int lane)
{
    SitePos s;
    if (c.chunks == 0) {
        const int first = ((int)b * c.nsub + sub) * kChunk;
        s.some = first < Vh;
        s.valid = first + lane < Vh;
        s.h = first + lane < Vh ? first + lane : Vh - 1;
        const uint32_t r = fdiv(c.Lxh, (uint32_t)s.h);
        s.xh = s.h - (int)r * Lxh;
        const uint32_t q = fdiv(c.Ly, r);
        s.y = (int)r - (int)q * Ly;
        s.t = (int)fdiv(c.Lz, q);
        s.z = (int)q - s.t * Lz;
    } else {
        uint32_t q = fdiv(c.ztile, b);
        const int zl = (int)(b - q * c.ztile.d);
        b = fdiv(c.Lt, q);
        s.t = (int)(q - b * c.Lt.d);
        q = fdiv(c.group, b);
        const int gi = (int)(b - q * c.group.d);
        b = fdiv(c.slabs, q);
        s.z = ((int)((q - b * c.slabs.d) * c.ztile.d) + zl) * c.planes;
        const int plane = Lxh * Ly, sites = plane * c.planes;
        const int first = (((int)(b * c.group.d) + gi) * c.nsub + sub) * kChunk;
        s.some = first < sites;
        s.valid = first + lane < sites;
        int i = first + lane < sites ? first + lane : sites - 1;
        s.h = i + plane * (s.z + Lz * s.t);
        if (c.planes > 1) {
            const int dz = (int)fdiv(c.plane, (uint32_t)i);
            s.z += dz;
            i -= dz * plane;
        }
        s.y = (int)fdiv(c.Lxh, (uint32_t)i);
        s.xh = i - s.y * Lxh;
    }
    s.x = 2 * s.xh + ((s.y + s.z + s.t + p) & 1);
    return s;
}

}  // namespace lqcd
