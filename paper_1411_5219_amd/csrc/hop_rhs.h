// Even-odd Wilson / twisted-mass Dslash on several right-hand sides (kernel
// templates; each storage precision is instantiated in its own translation
// unit).
//
// A block serves 64 output sites for up to four right-hand sides, one per
// wave (two of them: two waves each).  The waves first share the loading of
// the eight links of the sites and leave them in LDS with their third row
// rebuilt; after one barrier each wave runs the hops of its right-hand side
// with the spinors from memory and the links from LDS.
//
// Bounds: reads from beyond L2 (each XCD works on an eighth of the lattice and
// re-reads its surface), and VALU issue in FP16 storage.  Against one
// right-hand side per work-item with the links re-read through the caches
// (and for FP16 two of them in registers): a link's third row is rebuilt once
// for four right-hand sides and the link loads of a hop are one LDS read.
// 32^3x8 Schur, 12 right-hand sides, calls back to back: FP32/12 241 -> 206 us
// (a call by itself 260 -> 217), FP16/12 188 -> 139, FP64/18 683 -> 565.  Links
// are loaded with the normal policy: the next tile finds them in the Infinity
// Cache (streamed: FP32/12 219 us instead of 206, both parities of FP32/18 on
// four 81 instead of 61; FP64/18 gains, 533 instead of 565).
#pragma once

#include "dslash_impl.h"

namespace lqcd {

// The links of a block's sites, [hop][words of the link][site]: nine entries,
// or for FP16 storage the halves of rows 0 and 1 and the third row in FP32.
template <int PREC, int RECON>
struct RhsLinks {
    using R = typename SpinorIO<PREC>::R;
    struct alignas(4 * sizeof(R)) Two {
        cplx<R> a, b;
    };
    Two w[8][4][kChunk];
    cplx<R> last[8][kChunk];
    __device__ __forceinline__ void put(int k, int lane, const Lnk<PREC, RECON>& L)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[k][i][lane] = {L.u.u[2 * i / 3][2 * i % 3], L.u.u[(2 * i + 1) / 3][(2 * i + 1) % 3]};
        last[k][lane] = L.u.u[2][2];
    }
    template <bool ADJ>
    __device__ __forceinline__ void mul(int k, int lane, const cplx<R> (&h)[2][3], cplx<R> (&o)[2][3]) const
    {
        Link<R> L;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Two t = w[k][i][lane];
            L.u[2 * i / 3][2 * i % 3] = t.a;
            L.u[(2 * i + 1) / 3][(2 * i + 1) % 3] = t.b;
        }
        L.u[2][2] = last[k][lane];
        link_mul<R, ADJ>(L, h, o);
    }
};

template <>
struct RhsLinks<16, 12> {
    uint4 w[8][3][kChunk];
    __device__ __forceinline__ void put(int k, int lane, const Lnk<16, 12>& L)
    {
        cplx<float> t[3];
        L.third(t);
        w[k][0][lane] = make_uint4(L.w[0], L.w[1], L.w[2], L.w[3]);
        w[k][1][lane] = make_uint4(L.w[4], L.w[5], __float_as_uint(t[0].x), __float_as_uint(t[0].y));
        w[k][2][lane] = make_uint4(__float_as_uint(t[1].x), __float_as_uint(t[1].y), __float_as_uint(t[2].x),
                                   __float_as_uint(t[2].y));
    }
    template <bool ADJ>
    __device__ __forceinline__ void mul(int k, int lane, const cplx<float> (&h)[2][3], cplx<float> (&o)[2][3]) const
    {
        const uint4 a = w[k][0][lane], b = w[k][1][lane], c = w[k][2][lane];
        const Lnk<16, 12> L = {{a.x, a.y, a.z, a.w, b.x, b.y}};
        const cplx<float> t[3] = {{__uint_as_float(b.z), __uint_as_float(b.w)},
                                  {__uint_as_float(c.x), __uint_as_float(c.y)},
                                  {__uint_as_float(c.z), __uint_as_float(c.w)}};
        L.mul<ADJ>(t, h, o);
    }
};

// Neighbour spinors in flight per wave and waves per SIMD.  FP64 issues the
// next hop's loads after a hop's registers are free again (242 registers at
// two waves, no spills; ahead of the link product it spills 32).
template <int PREC>
struct RhsTune {
    static constexpr int depth = PREC == 64 ? 1 : 2;
    static constexpr int waves = PREC == 64 ? 2 : PREC == 32 ? 3 : 4;
};

// Hops K0 .. K1 - 1 of one right-hand side.
template <int PREC, int RECON, bool DAG, int K0, int K1>
struct RhsPipe {
    using R = typename SpinorIO<PREC>::R;
    static constexpr int D = RhsTune<PREC>::depth;
    static_assert(D == 1 || D == 2, "loads of first()");
    const RhsLinks<PREC, RECON>& lds;
    const DslashArgs& a;
    const SiteGeo& g;
    const char* in;
    int lane;
    Nbs<PREC> nb[D];
    Spinor<R> acc;

    template <int K>
    __device__ __forceinline__ void load()
    {
        if constexpr (K < K1) nb[K % D].load(in, a.g.S, g.template get<K>().nb);
    }
    template <int K>
    __device__ __forceinline__ void step()
    {
        constexpr int MU = K >> 1;
        constexpr bool FWD = (K & 1) == 0;
        constexpr int SIG = FWD != DAG ? 1 : -1;
        cplx<R> h[2][3], w[2][3];
        nb[K % D].template half<MU, SIG>(h);
        if constexpr (PREC == 32) load<K + D>();
        lds.template mul<!FWD>(K, lane, h, w);
        if (g.template get<K>().cross) {
            const cplx<R> ph = uniform<R>(a.g.ph[MU]);
            phase_mul(w, FWD ? ph : conj(ph));
        }
        nb[K % D].template add<MU, SIG>(acc, w);
        if constexpr (PREC != 32) load<K + D>();
        __builtin_amdgcn_sched_barrier(0);  // or the scheduler reads the next hops' links early and spills
    }
    __device__ __forceinline__ void first()
    {
        load<K0>();
        if constexpr (D > 1) load<K0 + 1>();
    }
    __device__ __forceinline__ void run()
    {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc.s[s][c] = {R(0), R(0)};
        step<K0>();
        step<K0 + 1>();
        step<K0 + 2>();
        step<K0 + 3>();
        if constexpr (K1 - K0 == 8) {
            step<4>();
            step<5>();
            step<6>();
            step<7>();
        }
    }
};

// Block bx of the launch.  HALVES = 2: two waves per right-hand side, wave 0 of
// them runs the x and y hops, wave 1 the z and t hops, whose sum it leaves in
// LDS.  For tiles of two: their links take the LDS of a tile of four, which
// lets two blocks of two waves run on a compute unit in FP64 and four in FP32,
// half the waves its registers allow (two right-hand sides: FP32/12 Schur
// complement 48^3x6 117 -> 101 us, 26^3x8 35 -> 32; FP64/18 32^3x8 118 -> 110;
// FP64/12 full matrix 24^3x8 48 -> 41).
template <int PREC, int RECON, bool DAG, int RED, int HALVES>
__device__ __forceinline__ void rhs_block(const DslashArgs& a, int bx, RhsLinks<PREC, RECON>& lds)
{
    using R = typename SpinorIO<PREC>::R;
    constexpr int N = RedN<RED>::N;
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    uint32_t tile, b;
    if (!tile_after_tile(a.ch, a.swizzle, bx, &tile, &b)) return;
    const int rhs0 = (int)tile * a.ch.tile, nr = min(a.ch.tile, a.nrhs - rhs0);
    // right-hand sides of the tile that run
    const bool on = lane < nr && !pred_skip(a.pred, a.ctl ? a.ctl + rhs0 + min(lane, nr - 1) : nullptr);
    const uint32_t mask = (uint32_t)__ballot(on);
    if (!mask) return;  // uniform over the block
    int p = a.parity;
    if (a.full) {
        p = (int)(b & 1u);
        b >>= 1;
    }
    const SitePos s = chunk_site(a.ch, a.g.Lxh, a.g.L[1], a.g.L[2], a.g.Vh, b, 0, p, lane);
    const SiteGeo geo = site_geo(a.g, s, p);
    const int64_t S = a.g.S;
    const int64_t poff = a.full ? p * a.par_bytes : 0, ioff = a.full ? (1 - p) * a.par_bytes : 0;
    const int mine = HALVES == 2 ? wave >> 1 : wave;
    const bool run = (mask >> mine) & 1u;
    const int64_t rr = rhs0 + mine;
    const char* in = static_cast<const char*>(a.in) + rr * a.st_in + ioff;
    auto links = [&]() {
        for (int k = wave; k < 8; k += nw) {
            // link of hop k: of this site (forward) or of the neighbour (backward)
            int l = s.h;
            if (k == 1) l = geo.get<1>().nb;
            else if (k == 3) l = geo.get<3>().nb;
            else if (k == 5) l = geo.get<5>().nb;
            else if (k == 7) l = geo.get<7>().nb;
            Lnk<PREC, RECON> L;
            L.template load<false>(a.U, S, (k & ~1) + ((k & 1) ? 1 - p : p), l);
            lds.put(k, lane, L);
        }
    };
    Spinor<R> acc;
    if constexpr (HALVES == 1) {
        RhsPipe<PREC, RECON, DAG, 0, 8> pipe{lds, a, geo, in, lane, {}, {}};
        if (run) pipe.first();
        links();
        __syncthreads();
        if (!run) return;
        pipe.run();
        acc = pipe.acc;
    } else {
        links();
        __syncthreads();
        if (run) {
            if ((wave & 1) == 0) {
                RhsPipe<PREC, RECON, DAG, 0, 4> pipe{lds, a, geo, in, lane, {}, {}};
                pipe.first();
                pipe.run();
                acc = pipe.acc;
            } else {
                RhsPipe<PREC, RECON, DAG, 4, 8> pipe{lds, a, geo, in, lane, {}, {}};
                pipe.first();
                pipe.run();
                acc = pipe.acc;
            }
        }
        __syncthreads();  // the links have been read
        cplx<R>* sum = reinterpret_cast<cplx<R>*>(&lds) + (mine * 12) * kChunk + lane;
        static_assert(sizeof(lds) >= 2 * 12 * kChunk * sizeof(cplx<R>), "the sums of a tile of two fit");
        if (run && (wave & 1)) {
#pragma unroll
            for (int k = 0; k < 12; ++k) sum[k * kChunk] = acc.s[k / 3][k % 3];
        }
        __syncthreads();
        if (!run || (wave & 1)) return;
#pragma unroll
        for (int k = 0; k < 12; ++k) acc.s[k / 3][k % 3] = acc.s[k / 3][k % 3] + sum[k * kChunk];
    }
    double tot[N];
#pragma unroll
    for (int j = 0; j < N; ++j) tot[j] = 0.0;
    hop_store<PREC, RED>(a, rr, poff, s.h, s.valid, acc, tot);
    if constexpr (RED != RED_NONE) {
        wave_reduce<N>(tot);
        const int64_t nsl = a.ch.nsp * (a.full ? 2 : 1), slot = (int)b + p * (a.full ? a.ch.nsp : 0);
        if (lane == 0)
#pragma unroll
            for (int j = 0; j < N; ++j) a.r.partials[(rr * nsl + slot) * N + j] = tot[j];
    }
}

template <int PREC, int RECON, bool DAG, int RED, int HALVES>
__global__ void __launch_bounds__(64 * kMaxTile) __attribute__((amdgpu_waves_per_eu(RhsTune<PREC>::waves)))
k_hop_rhs(const DslashArgs a)
{
    __shared__ RhsLinks<PREC, RECON> lds;
    rhs_block<PREC, RECON, DAG, RED, HALVES>(a, blockIdx.x, lds);
}

// The hops of a reliable update, which hardly any launch finds pending: as many
// blocks as run at once stride over the launch's blocks, so that one that finds
// nothing to do ends with its first blocks: 12.4 us of a launch of 8192 blocks
// whose LDS lets two run per compute unit (32^3x8, FP32 inner, sixteen right-hand
// sides 54.4 -> 53.9 ms; FP16 inner, twelve 38.5 -> 38.0).  Below four rounds the
// launch costs no more (24^3x6, FP16 inner, four: 6.32 ms against 6.45 strided).
constexpr int kLoopBlocks = 512;  // two per compute unit (a multiple of the XCDs)
template <int RECON, int RED>
__global__ void __launch_bounds__(64 * kMaxTile) __attribute__((amdgpu_waves_per_eu(RhsTune<64>::waves)))
k_hop_rhs_update(const DslashArgs a)
{
    __shared__ RhsLinks<64, RECON> lds;
    const int lane = (int)threadIdx.x & 63;
    const bool on = lane < a.nrhs && !pred_skip(a.pred, a.ctl ? a.ctl + lane : nullptr);
    if (!__ballot(on)) return;  // uniform over the grid
    for (int bx = blockIdx.x; bx < a.gx; bx += gridDim.x) {
        rhs_block<64, RECON, false, RED, 1>(a, bx, lds);
        __syncthreads();  // every wave is done with the links
    }
}

template <int PREC, int RECON, bool DAG, int RED, int HALVES>
__global__ void __launch_bounds__(64 * kMaxTile) __attribute__((amdgpu_waves_per_eu(RhsTune<PREC>::waves)))
k_hop_rhs_batch(const DslashArgs* __restrict__ tab, const int* __restrict__ offs, int nsys)
{
    __shared__ RhsLinks<PREC, RECON> lds;
    int bx;
    const int s = batch_system(offs, nsys, &bx);
    if (bx >= tab[s].gx) return;  // padding of the system's range
    rhs_block<PREC, RECON, DAG, RED, HALVES>(tab[s], bx, lds);
}

template <int PREC, int RECON, bool DAG, int RED, int HALVES>
static hipError_t rhs_one(const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if constexpr (PREC == 64 && !DAG && HALVES == 1 && (RED == RED_NONE || RED == RED_NORM_LOW))
        if (!L.tab && L.a->pred == PRED_UPDATE && grid.x > 4u * kLoopBlocks) {
            hipLaunchKernelGGL((k_hop_rhs_update<RECON, RED>), dim3(kLoopBlocks), block, 0, s, *L.a);
            return hipGetLastError();
        }
    if (L.tab) hipLaunchKernelGGL((k_hop_rhs_batch<PREC, RECON, DAG, RED, HALVES>), grid, block, 0, s, L.tab, L.offs, L.nsys);
    else hipLaunchKernelGGL((k_hop_rhs<PREC, RECON, DAG, RED, HALVES>), grid, block, 0, s, *L.a);
    return hipGetLastError();
}

template <int PREC, int RECON, bool DAG, int HALVES>
static hipError_t rhs_red(int red, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    switch (red) {
    case RED_NONE: return rhs_one<PREC, RECON, DAG, RED_NONE, HALVES>(L, grid, block, s);
    case RED_NORM: return rhs_one<PREC, RECON, DAG, RED_NORM, HALVES>(L, grid, block, s);
    case RED_NORM_DS: return rhs_one<PREC, RECON, DAG, RED_NORM_DS, HALVES>(L, grid, block, s);
    case RED_DOT_AUX: return rhs_one<PREC, RECON, DAG, RED_DOT_AUX, HALVES>(L, grid, block, s);
    default: break;
    }
    if constexpr (PREC == 64 && !DAG)
        if (red == RED_NORM_LOW) return rhs_one<PREC, RECON, DAG, RED_NORM_LOW, HALVES>(L, grid, block, s);
    return hipErrorInvalidValue;
}

template <int PREC, int RECON>
inline hipError_t launch_rhs(int halves, bool dag, int red, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if (halves == 2)
        return dag ? rhs_red<PREC, RECON, true, 2>(red, L, grid, block, s)
                   : rhs_red<PREC, RECON, false, 2>(red, L, grid, block, s);
    return dag ? rhs_red<PREC, RECON, true, 1>(red, L, grid, block, s)
               : rhs_red<PREC, RECON, false, 1>(red, L, grid, block, s);
}

}  // namespace lqcd
