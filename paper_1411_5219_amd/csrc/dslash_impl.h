// Even-odd Wilson / twisted-mass Dslash for gfx950 (kernel templates; each
// storage precision is instantiated in its own translation unit).
//
// For each of the 8 hops of an output site of parity p the neighbour spinor
// of parity 1-p is loaded, projected to a 2x3 half spinor with (1 -+ gamma_mu),
// multiplied by the link (or its adjoint) and by the boundary phase on hops
// that cross the boundary, and the lower spin components are rebuilt from the
// upper ones.  A wave holds 64 sites, one per lane; one or two waves share the
// hops of its sites.  The site-diagonal twisted-mass terms are fused into the
// store (out = add + a*site + c*hop) together with FP64 reductions, so a
// Schur-complement application or a residual never needs a separate vector
// pass.
//
// Bounds: FP64 and FP32 on large lattices by memory (48^3x12 FP64/18 186 us,
// FP32/12 75.5 us), FP16 storage by memory and VALU issue together (33.9 us;
// 39.7 with operands converted before use), small lattices by launch and
// latency.  Both parities in one launch are bound by memory too, with each
// link read once: 48^3x12 FP64/18 386 -> 320 us against two parities one after
// the other.
//
// In the chiral basis gamma_mu = [[0, B_mu], [B_mu^+, 0]] with
//   B_x = -i sigma_1, B_y = -i sigma_2, B_z = -i sigma_3, B_t = 1,
// so (1 - s gamma_mu) psi = (h ; -s B_mu^+ h) with h = psi_up - s B_mu psi_lo;
// only h is multiplied by the link.
#pragma once

#include "block_order.h"
#include "lqcd.h"
#include "lqcd_device.h"
#include "lqcd_fin.h"
#include "lqcd_kernels.h"

#include <type_traits>

namespace lqcd {

// h = u - SIG * B_MU l   (u = spins 0,1; l = spins 2,3)
template <class R, int MU, int SIG>
__device__ __forceinline__ void project(const Spinor<R>& p, cplx<R> (&h)[2][3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cplx<R> u0 = p.s[0][c], u1 = p.s[1][c], l0 = p.s[2][c], l1 = p.s[3][c];
        cplx<R> b0, b1;
        if (MU == 0) { b0 = mti(l1); b1 = mti(l0); }        // -i sigma_1
        else if (MU == 1) { b0 = -l1; b1 = l0; }            // -i sigma_2
        else if (MU == 2) { b0 = mti(l0); b1 = ti(l1); }    // -i sigma_3
        else { b0 = l0; b1 = l1; }                          // 1
        if (SIG > 0) { h[0][c] = u0 - b0; h[1][c] = u1 - b1; }
        else { h[0][c] = u0 + b0; h[1][c] = u1 + b1; }
    }
}

// acc += (w ; -SIG * B_MU^+ w)
template <class R, int MU, int SIG>
__device__ __forceinline__ void accumulate(Spinor<R>& acc, const cplx<R> (&w)[2][3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const cplx<R> w0 = w[0][c], w1 = w[1][c];
        acc.s[0][c] = acc.s[0][c] + w0;
        acc.s[1][c] = acc.s[1][c] + w1;
        cplx<R> d0, d1;  // B^+ w
        if (MU == 0) { d0 = ti(w1); d1 = ti(w0); }          // i sigma_1
        else if (MU == 1) { d0 = w1; d1 = -w0; }            // i sigma_2
        else if (MU == 2) { d0 = ti(w0); d1 = mti(w1); }    // i sigma_3
        else { d0 = w0; d1 = w1; }
        if (SIG > 0) { acc.s[2][c] = acc.s[2][c] - d0; acc.s[3][c] = acc.s[3][c] - d1; }
        else { acc.s[2][c] = acc.s[2][c] + d0; acc.s[3][c] = acc.s[3][c] + d1; }
    }
}

// w = U h (ADJ = false) or U^+ h (ADJ = true), on both spin components.
template <class R, bool ADJ>
__device__ __forceinline__ void link_mul(const Link<R>& U, const cplx<R> (&h)[2][3], cplx<R> (&w)[2][3])
{
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) w[s][a] = su3_row<R, ADJ>(U.u, a, h[s]);
}

template <class R>
__device__ __forceinline__ void phase_mul(cplx<R> (&w)[2][3], cplx<R> ph)
{
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int a = 0; a < 3; ++a) w[s][a] = ph * w[s][a];
}

// A launch constant in scalar registers at precision R (converted in vector
// registers it would stay there across the whole kernel).
template <class R>
__device__ __forceinline__ cplx<R> uniform(const double (&v)[2])
{
    if constexpr (sizeof(R) == 8) return {v[0], v[1]};
    else
        return {__builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, (float)v[0]))),
                __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, (float)v[1])))};
}

// ---------------------------------------------------------------------------
// Operands of one hop as they are loaded.
//
// FP64 and FP32 storage: the neighbour spinor and the link as numbers.
// FP16 storage: the words themselves, 19 registers instead of 42 for the
// loads in flight, and used as half operands of mixed-precision fused
// multiply-adds: the projection of the unscaled halves u -+ B l is one
// instruction per real (it is exact up to one FP32 rounding), the link
// product takes its matrix elements as halves, and the site's scale is the
// factor of the accumulation's fused multiply-adds.  The kernel is bound by
// its VALU issue (a wave instruction takes four cycles of a SIMD): converting
// and scaling each operand first takes 24 + 12 instructions more per hop.

template <int PREC>
struct Nbs {
    using R = typename SpinorIO<PREC>::R;
    Spinor<R> v;
    __device__ __forceinline__ void load(const void* in, int64_t S, int site) { SpinorIO<PREC>::load(in, S, site, v); }
    template <int MU, int SIG>
    __device__ __forceinline__ void half(cplx<R> (&h)[2][3]) const
    {
        project<R, MU, SIG>(v, h);
    }
    template <int MU, int SIG>
    __device__ __forceinline__ void add(Spinor<R>& acc, const cplx<R> (&w)[2][3]) const
    {
        accumulate<R, MU, SIG>(acc, w);
    }
};

__device__ __forceinline__ float half_lo(uint32_t w) { return (float)__builtin_bit_cast(_Float16, (unsigned short)w); }
__device__ __forceinline__ float half_hi(uint32_t w)
{
    return (float)__builtin_bit_cast(_Float16, (unsigned short)(w >> 16));
}

template <>
struct Nbs<16> {
    uint32_t w[12];  // complex component k: real in the low half, imaginary in the high half
    float scale;
    __device__ __forceinline__ void load(const void* in, int64_t S, int site)
    {
        const rsrc_t r = make_rsrc(in, 52 * S);
        scale = bload<float>(r, static_cast<uint32_t>(site) * 4u, (uint32_t)(3 * S * 16));
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint4 d = bload<uint4>(r, static_cast<uint32_t>(site) * 16u, (uint32_t)(k * S * 16));
            w[4 * k] = d.x;
            w[4 * k + 1] = d.y;
            w[4 * k + 2] = d.z;
            w[4 * k + 3] = d.w;
        }
    }
    // (u - SIG * B_MU l) / scale
    template <int MU, int SIG>
    __device__ __forceinline__ void half(cplx<float> (&h)[2][3]) const
    {
        // one: 1 in a scalar register that the compiler does not know, so that u + l stays a fused multiply-add
        // of halves instead of two conversions and an addition
        float one = 1.0f;
        asm("" : "+s"(one));
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint32_t u0 = w[c], u1 = w[3 + c], l0 = w[6 + c], l1 = w[9 + c];
            const uint32_t b0 = MU < 2 ? l1 : l0, b1 = MU < 2 ? l0 : l1;
            // sign of b in h, and B's factor: -i, (-1 | +1), (-i | +i), 1
            constexpr float g = SIG > 0 ? -1.f : 1.f;
            if (MU == 0 || MU == 2) {
                constexpr float g1 = MU == 0 ? g : -g;
                h[0][c] = {fmar(half_lo(u0), one, g * half_hi(b0)), fmar(half_hi(u0), one, -g * half_lo(b0))};
                h[1][c] = {fmar(half_lo(u1), one, g1 * half_hi(b1)), fmar(half_hi(u1), one, -g1 * half_lo(b1))};
            } else {
                constexpr float g0 = MU == 1 ? -g : g;
                h[0][c] = {fmar(half_lo(u0), one, g0 * half_lo(b0)), fmar(half_hi(u0), one, g0 * half_hi(b0))};
                h[1][c] = {fmar(half_lo(u1), one, g * half_lo(b1)), fmar(half_hi(u1), one, g * half_hi(b1))};
            }
        }
    }
    // acc += scale * (w ; -SIG * B_MU^+ w)
    template <int MU, int SIG>
    __device__ __forceinline__ void add(Spinor<float>& acc, const cplx<float> (&v)[2][3]) const
    {
        auto fma2 = [&](cplx<float>& a, cplx<float> b) { a = {fmar(scale, b.x, a.x), fmar(scale, b.y, a.y)}; };
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const cplx<float> w0 = v[0][c], w1 = v[1][c];
            cplx<float> d0, d1;  // B^+ w
            if (MU == 0) { d0 = ti(w1); d1 = ti(w0); }
            else if (MU == 1) { d0 = w1; d1 = -w0; }
            else if (MU == 2) { d0 = ti(w0); d1 = mti(w1); }
            else { d0 = w0; d1 = w1; }
            fma2(acc.s[0][c], w0);
            fma2(acc.s[1][c], w1);
            fma2(acc.s[2][c], SIG > 0 ? -d0 : d0);
            fma2(acc.s[3][c], SIG > 0 ? -d1 : d1);
        }
    }
};

template <int PREC, int RECON>
struct Lnk {
    using R = typename SpinorIO<PREC>::R;
    Link<R> u;
    template <bool LNT>
    __device__ __forceinline__ void load(const void* U, int64_t S, int blk, int site)
    {
        if constexpr (LNT) LinkIO<PREC, RECON>::template load<>(U, S, blk, site, u);
        else LinkIO<PREC, RECON>::template load<0>(U, S, blk, site, u);
    }
    template <bool ADJ>
    __device__ __forceinline__ void mul(const cplx<R> (&h)[2][3], cplx<R> (&w)[2][3]) const
    {
        link_mul<R, ADJ>(u, h, w);
    }
};

template <>
struct Lnk<16, 12> {
    uint32_t w[6];  // rows 0 and 1
    template <bool LNT>
    __device__ __forceinline__ void load(const void* U, int64_t S, int blk, int site)
    {
        const rsrc_t r = make_rsrc(static_cast<const char*>(U) + blk * 24 * S, 24 * S);
        const uint4 d = bload<uint4, LQCD_LINK16_AUX>(r, static_cast<uint32_t>(site) * 16u, 0u);
        const uint2 e = bload<uint2, LQCD_LINK16_AUX>(r, static_cast<uint32_t>(site) * 8u, (uint32_t)(16 * S));
        w[0] = d.x;
        w[1] = d.y;
        w[2] = d.z;
        w[3] = d.w;
        w[4] = e.x;
        w[5] = e.y;
    }
    __device__ __forceinline__ float lo(int k) const { return half_lo(w[k]); }
    __device__ __forceinline__ float hi(int k) const { return half_hi(w[k]); }
    // third row: conj(a b - c d) of row-0 and row-1 entries
    __device__ __forceinline__ void third(cplx<float> (&t)[3]) const
    {
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int a = (j + 1) % 3, b = 3 + (j + 2) % 3, c = (j + 2) % 3, d = 3 + (j + 1) % 3;
            float re = fmar(lo(a), lo(b), 0.f), im = fmar(-lo(a), hi(b), 0.f);
            re = fmar(-hi(a), hi(b), re);
            im = fmar(-hi(a), lo(b), im);
            re = fmar(-lo(c), lo(d), re);
            im = fmar(lo(c), hi(d), im);
            re = fmar(hi(c), hi(d), re);
            im = fmar(hi(c), lo(d), im);
            t[j] = {re, im};
        }
    }
    template <bool ADJ>
    __device__ __forceinline__ void mul(const cplx<float> (&t)[3], const cplx<float> (&h)[2][3],
                                        cplx<float> (&o)[2][3]) const
    {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                float re = 0.f, im = 0.f;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const int row = ADJ ? k : a, col = ADJ ? a : k;
                    const float ux = row < 2 ? lo(3 * row + col) : t[col].x;
                    const float uy = row < 2 ? hi(3 * row + col) : t[col].y;
                    re = fmar(ux, h[s][k].x, re);
                    im = fmar(ux, h[s][k].y, im);
                    re = fmar(ADJ ? uy : -uy, h[s][k].y, re);
                    im = fmar(ADJ ? -uy : uy, h[s][k].x, im);
                }
                o[s][a] = {re, im};
            }
    }
    template <bool ADJ>
    __device__ __forceinline__ void mul(const cplx<float> (&h)[2][3], cplx<float> (&o)[2][3]) const
    {
        cplx<float> t[3];
        third(t);
        mul<ADJ>(t, h, o);
    }
};

// Per storage precision: waves per SIMD the register allocation must allow
// and the depth of the software pipeline over the hops (the loads of hop
// K + depth are issued right after hop K has been applied).  FP64 holds 84
// registers of operands per hop: two waves per SIMD either way, with one hop
// in flight where a wave runs all eight (242 registers), with two where it
// runs four (8^3x4 to 12^3x8: 5.6-7.0 us a hop against 6.8-8.2 with one).
// FP32 and FP16 keep three waves or more with two hops in flight (three: no
// faster).
template <int PREC, int SPLIT>
struct HopTune {
    static constexpr int waves = hop_waves(PREC);
    static constexpr int depth = PREC == 64 && SPLIT == 1 ? 1 : 2;
};

// Hops K0 .. K1 - 1 of one site added into acc.  At depth 1 the neighbour
// spinor is loaded and projected before the link is loaded, so the full
// spinor and the link are not live together.
template <int PREC, int RECON, bool DAG, bool LNT, int D, int K0, int K1>
struct HopPipe {
    using R = typename SpinorIO<PREC>::R;
    static_assert(D == 1 || D == 2, "loads of run()");
    const char* in;
    const DslashArgs& a;
    const SiteGeo& g;
    Spinor<R>& acc;
    Nbs<PREC> nb[D];
    Lnk<PREC, RECON> lk[D];

    template <int K>
    __device__ __forceinline__ void load()
    {
        if constexpr (K < K1) {
            const Nbr n = g.template get<K>();
            lk[K % D].template load<LNT>(a.U, a.g.S, n.lblk, n.lsite);
            nb[K % D].load(in, a.g.S, n.nb);
        }
    }
    template <int K>
    __device__ __forceinline__ void step()
    {
        if constexpr (K < K1) {
            constexpr int MU = K >> 1;
            constexpr bool FWD = (K & 1) == 0;
            constexpr int SIG = FWD != DAG ? 1 : -1;  // projector (1 - SIG gamma)
            const Nbr n = g.template get<K>();
            cplx<R> h[2][3], w[2][3];
            if constexpr (D == 1) nb[0].load(in, a.g.S, n.nb);
            nb[K % D].template half<MU, SIG>(h);
            if constexpr (D == 1) lk[0].template load<LNT>(a.U, a.g.S, n.lblk, n.lsite);
            lk[K % D].template mul<!FWD>(h, w);
            if (n.cross) {
                const cplx<R> ph = uniform<R>(a.g.ph[MU]);
                phase_mul(w, FWD ? ph : conj(ph));
            }
            nb[K % D].template add<MU, SIG>(acc, w);
            if constexpr (D > 1) load<K + D>();
        }
    }
    __device__ __forceinline__ void run()
    {
        if constexpr (D > 1) {
            load<K0>();
            load<K0 + 1>();
        }
        step<K0>();
        step<K0 + 1>();
        step<K0 + 2>();
        step<K0 + 3>();
        step<K0 + 4>();
        step<K0 + 5>();
        step<K0 + 6>();
        step<K0 + 7>();
    }
};

template <int RED>
struct RedN {
    static constexpr int N = RED == RED_NONE ? 1 : RED == RED_NORM || RED == RED_NORM_LOW ? 1 : RED == RED_DOT_AUX ? 2 : 3;
};

// out = add + a * site + c * acc of one right-hand side, with the sums of the reduction.
template <int PREC, int RED>
__device__ __forceinline__ void hop_store(const DslashArgs& a, int64_t rr, int64_t poff, int h, bool valid,
                                          const Spinor<typename SpinorIO<PREC>::R>& acc, double (&tot)[RedN<RED>::N])
{
    using R = typename SpinorIO<PREC>::R;
    constexpr int N = RedN<RED>::N;
    const int64_t S = a.g.S;
    const cplx<R> cu = uniform<R>(a.c.up), cl = uniform<R>(a.c.lo);
    Spinor<R> o, st;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) o.s[s][c] = (s < 2 ? cu : cl) * acc.s[s][c];
    if (a.site) {
        const cplx<R> au = uniform<R>(a.a.up), al = uniform<R>(a.a.lo);
        SpinorIO<PREC>::load(static_cast<const char*>(a.site) + rr * a.st_site + poff, S, h, st);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) o.s[s][c] = o.s[s][c] + (s < 2 ? au : al) * st.s[s][c];
    }
    if (a.add) {
        Spinor<R> ad;
        SpinorIO<PREC>::load(static_cast<const char*>(a.add) + rr * a.st_add + poff, S, h, ad);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) o.s[s][c] = o.s[s][c] + ad.s[s][c];
    }
    if (!valid) return;
    if (a.out) SpinorIO<PREC>::template store<LQCD_OUT_AUX>(static_cast<char*>(a.out) + rr * a.st_out + poff, S, h, o);
    if constexpr (RED == RED_NORM_LOW) {
        // the residual of a reliable update, in the storage of the inner solve
        // (as a branch of RED_NORM it slowed every FP64 hop by 2%)
        Spinor<float> f;
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) f.s[s][c] = {(float)o.s[s][c].x, (float)o.s[s][c].y};
        char* low = static_cast<char*>(a.low) + rr * a.st_low;
        if (a.low_prec == 32) SpinorIO<32>::store(low, S, h, f);
        else SpinorIO<16>::store(low, S, h, f);
    }
    if (RED == RED_NORM || RED == RED_NORM_DS || RED == RED_NORM_LOW) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) tot[0] += (double)norm2(o.s[s][c]);
    }
    if (RED == RED_NORM_DS) {  // <out, site>
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const cplx<R> v = cmulc(o.s[s][c], st.s[s][c]);
                tot[N - 2] += (double)v.x;
                tot[N - 1] += (double)v.y;
            }
    }
    if (RED == RED_DOT_AUX) {  // <aux, out>
        Spinor<R> ax;
        SpinorIO<PREC>::load(static_cast<const char*>(a.aux) + rr * a.st_aux + poff, S, h, ax);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const cplx<R> v = cmulc(ax.s[s][c], o.s[s][c]);
                tot[N - 2] += (double)v.x;
                tot[N - 1] += (double)v.y;
            }
    }
}

// The sum wave 1 of a two-wave block leaves for wave 0.
template <class R, int SPLIT>
struct SplitLds {
    cplx<R> v[12][kChunk];
};
template <class R>
struct SplitLds<R, 1> {};

// One right-hand side per block, block bx of the launch.  SPLIT = 1: every wave of the block
// serves its own chunk of 64 sites.  SPLIT = 2: a block is two waves that
// share one chunk, wave 0 runs the x and y hops and wave 1 the z and t hops,
// and wave 0 adds the two sums through LDS and stores.  What the split buys:
// half the chain of dependent loads per wave and twice the waves, where a
// lattice does not fill the chip (FP64/18 hop 16^3x8 9.3 -> 6.3 us, 12^3x8
// 13.9 -> 7.0, 24^3x8 20.2 -> 18.5; FP32/12 20^3x6 8.1 -> 6.3), and a shorter
// drain at the end of a large launch (48^3x12 FP32/12 77.0 -> 75.5).  The
// plan chooses (see plan_dslash).
template <int PREC, int RECON, bool DAG, int RED, bool LNT, int SPLIT, bool NEXT>
__device__ __forceinline__ void dslash_block(const DslashArgs& a, int bx)
{
    using R = typename SpinorIO<PREC>::R;
    constexpr int N = RedN<RED>::N;
    constexpr int D = HopTune<PREC, SPLIT>::depth;
    __shared__ SplitLds<R, SPLIT> lds;
    uint32_t rhs, b;
    if constexpr (NEXT) tile_by_tile(a.ch, a.swizzle, bx, &rhs, &b);
    else if (!tile_after_tile(a.ch, a.swizzle, bx, &rhs, &b)) return;
    if (pred_skip(a.pred, a.ctl ? a.ctl + rhs : nullptr)) return;
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int p = a.parity;
    if (a.full) {  // both parities in one launch, adjacent in the block order: the second finds the links in L2
        p = (int)(b & 1u);
        b >>= 1;
    }
    const int64_t poff = a.full ? p * a.par_bytes : 0, ioff = a.full ? (1 - p) * a.par_bytes : 0;
    const SitePos s = chunk_site(a.ch, a.g.Lxh, a.g.L[1], a.g.L[2], a.g.Vh, b, SPLIT > 1 ? 0 : wave, p, lane);
    double tot[N];
#pragma unroll
    for (int j = 0; j < N; ++j) tot[j] = 0.0;
    if (SPLIT > 1 || (s.some && wave < a.ch.nsub)) {  // (a batched launch may have more waves than this system's blocks)
        const SiteGeo geo = site_geo(a.g, s, p);
        const char* in = static_cast<const char*>(a.in) + (int64_t)rhs * a.st_in + ioff;
        Spinor<R> acc;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc.s[i][c] = {R(0), R(0)};
        auto hops = [&](auto part) {
            constexpr int Q = decltype(part)::value;
            HopPipe<PREC, RECON, DAG, LNT, D, Q * (8 / SPLIT), (Q + 1) * (8 / SPLIT)> pipe{in, a, geo, acc, {}, {}};
            pipe.run();
        };
        if constexpr (SPLIT == 1) hops(std::integral_constant<int, 0>{});
        else {
            if (wave == 0) hops(std::integral_constant<int, 0>{});
            else {
                hops(std::integral_constant<int, 1>{});
#pragma unroll
                for (int k = 0; k < 12; ++k) lds.v[k][lane] = acc.s[k / 3][k % 3];
            }
            __syncthreads();
            if (wave == 0)
#pragma unroll
                for (int k = 0; k < 12; ++k) acc.s[k / 3][k % 3] = acc.s[k / 3][k % 3] + lds.v[k][lane];
        }
        if (SPLIT == 1 || wave == 0) hop_store<PREC, RED>(a, rhs, poff, s.h, s.valid, acc, tot);
    }
    if constexpr (RED != RED_NONE) {
        const int slot = (int)(rhs * a.ch.nblk) + (int)b + p * (a.full ? a.ch.nsp : 0);
        if constexpr (SPLIT == 1) block_reduce_store<N>(tot, a.r.partials, slot);
        else if (wave == 0) {
            wave_reduce<N>(tot);
            if (lane == 0)
#pragma unroll
                for (int j = 0; j < N; ++j) a.r.partials[(int64_t)slot * N + j] = tot[j];
        }
    }
}

template <int PREC, int RECON, bool DAG, int RED, bool LNT, int SPLIT, bool NEXT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HopTune<PREC, SPLIT>::waves)))
k_dslash_eo(const DslashArgs a)
{
    dslash_block<PREC, RECON, DAG, RED, LNT, SPLIT, NEXT>(a, blockIdx.x);
}

// Several systems (lattices of different sizes) in one launch: block x of the
// flattened grid belongs to system s with offs[s] <= x < offs[s + 1]; each
// system's arguments come from the device table tab.
template <int PREC, int RECON, bool DAG, int RED, bool LNT, int SPLIT, bool NEXT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HopTune<PREC, SPLIT>::waves)))
k_dslash_eo_batch(const DslashArgs* __restrict__ tab, const int* __restrict__ offs, int nsys)
{
    int bx;
    const int s = batch_system(offs, nsys, &bx);
    // blocks past the system's own grid are padding
    if (bx >= tab[s].gx) return;
    dslash_block<PREC, RECON, DAG, RED, LNT, SPLIT, NEXT>(tab[s], bx);
}

template <int PREC, int RECON, bool DAG, int RED, bool LNT, int SPLIT, bool NEXT>
static hipError_t launch_one(const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if (L.tab)
        hipLaunchKernelGGL((k_dslash_eo_batch<PREC, RECON, DAG, RED, LNT, SPLIT, NEXT>), grid, block, 0, s, L.tab, L.offs,
                           L.nsys);
    else hipLaunchKernelGGL((k_dslash_eo<PREC, RECON, DAG, RED, LNT, SPLIT, NEXT>), grid, block, 0, s, *L.a);
    return hipGetLastError();
}

template <int PREC, int RECON, bool DAG, bool LNT, int SPLIT, bool NEXT>
static hipError_t launch_red(int red, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    switch (red) {
    case RED_NONE: return launch_one<PREC, RECON, DAG, RED_NONE, LNT, SPLIT, NEXT>(L, grid, block, s);
    case RED_NORM: return launch_one<PREC, RECON, DAG, RED_NORM, LNT, SPLIT, NEXT>(L, grid, block, s);
    case RED_NORM_DS: return launch_one<PREC, RECON, DAG, RED_NORM_DS, LNT, SPLIT, NEXT>(L, grid, block, s);
    case RED_DOT_AUX: return launch_one<PREC, RECON, DAG, RED_DOT_AUX, LNT, SPLIT, NEXT>(L, grid, block, s);
    default: break;
    }
    if constexpr (PREC == 64 && !DAG)
        if (red == RED_NORM_LOW) return launch_one<PREC, RECON, DAG, RED_NORM_LOW, LNT, SPLIT, NEXT>(L, grid, block, s);
    return hipErrorInvalidValue;
}

template <int PREC, int RECON, bool LNT, int SPLIT, bool NEXT>
static hipError_t launch_dag(bool dag, int red, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    return dag ? launch_red<PREC, RECON, true, LNT, SPLIT, NEXT>(red, L, grid, block, s)
               : launch_red<PREC, RECON, false, LNT, SPLIT, NEXT>(red, L, grid, block, s);
}

// Streaming link loads for one parity (each link has one reader), cached ones
// for both parities in one launch (each link has two).
template <int PREC, int RECON>
inline hipError_t launch_hop(int split, bool lnt, bool next, bool dag, int red, const DslashLaunch& L, dim3 grid,
                             dim3 block, hipStream_t s)
{
    if constexpr (hop_built(PREC, RECON, 2, false, true))
        if (split == 2 && next && !lnt) return launch_dag<PREC, RECON, false, 2, true>(dag, red, L, grid, block, s);
    if (split == 2 && !next)
        return lnt ? launch_dag<PREC, RECON, true, 2, false>(dag, red, L, grid, block, s)
                   : launch_dag<PREC, RECON, false, 2, false>(dag, red, L, grid, block, s);
    if constexpr (hop_built(PREC, RECON, 1, true, false))
        if (split == 1 && lnt && !next) return launch_dag<PREC, RECON, true, 1, false>(dag, red, L, grid, block, s);
    return hipErrorInvalidValue;
}

}  // namespace lqcd
