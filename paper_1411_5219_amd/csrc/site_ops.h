// Site-local block routines shared by the standalone kernels (blas.hip) and
// the persistent batched solver (persist.hip): the fused BLAS-1 steps of the
// solvers with their FP64 block reductions, precision conversion, and the
// block-order sum of reduction partials.
#pragma once

#include "lqcd.h"
#include "lqcd_device.h"
#include "lqcd_fin.h"
#include "lqcd_kernels.h"

namespace lqcd {

template <int OP>
struct BlasRed {
    static constexpr int N = (OP == BLAS_NORM || OP == BLAS_AXMY_NORM) ? 1
                             : (OP == BLAS_BI_XR || OP == BLAS_NORM_DOT || OP == BLAS_BL_ORTH ||
                                OP == BLAS_BL_MR)                                          ? 3
                             : OP == BLAS_BL_GRAM                                          ? 5
                                                                                          : 0;
};

// Scalar steps a BLAS step takes over from its producers (CtlFold): the values
// of the last step's partials and its Fin (FIN_NONE: none).
template <int KIND, int OP>
struct BlasFold {
    static constexpr int FIN = OP == BLAS_AXMY_NORM ? (KIND == KIND_COLOUR ? FIN_MS_ALPHA : FIN_CG_ALPHA)
                               : OP == BLAS_CG_XP   ? FIN_CG_BETA
                               : OP == BLAS_MS_XP   ? FIN_MS_BETA
                                                    : FIN_NONE;
    static constexpr int N = FIN == FIN_MS_ALPHA ? 3 : 1;
    static constexpr bool MS = FIN == FIN_MS_ALPHA || FIN == FIN_MS_BETA;
};

// Sum of one right-hand side's partials by one block: each thread adds its
// strided share four blocks' partials at a time (the four loads issued
// together: the partials were just written on other XCDs and each round trip
// is long).
template <int N>
__device__ __forceinline__ void sum_partials(const double* p, int nblocks, double (&v)[N])
{
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = 0.0;
    const int T = blockDim.x;
    for (int b0 = threadIdx.x; b0 < nblocks; b0 += 4 * T) {
        double t[4][N];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + u * T;
#pragma unroll
            for (int j = 0; j < N; ++j) t[u][j] = b < nblocks ? p[(int64_t)b * N + j] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] += t[u][j];
    }
}

// The folded scalar steps of a block.  A launch of its own for each step costs
// 4.7 to 6 us and the gap before it on an otherwise idle chip; here every block
// repeats the sum and the step, which lengthens a short kernel by 3.5 us (the
// update of r at 24^3x8 in FP64 5.6 -> 9.5 us) and is hidden under the blocks
// before it in a long one.  Loading the fields before the step gains 0.4 us of
// this and costs occupancy where nothing is folded (48^3x12 FP16 20.2 -> 22.1).
// ctl: the nctl control blocks (cur the one that steps) as the last launch
// left them; returns their new state, in LDS.
constexpr int kFoldWaves = 16;  // of a block, at most
template <int N, int NCTL>
struct FoldLds {
    double part[N + 1][kFoldWaves];
    uint32_t ctl[NCTL * sizeof(Ctl) / 4];
};
// The block's totals, in every lane of wave 0, from its waves' sums.
template <int N, int NCTL>
__device__ __forceinline__ void fold_totals(const FoldLds<N, NCTL>& lds, bool pre, double (&t)[6], double (&pt)[6])
{
    const int nw = (int)blockDim.x >> 6, lane = (int)threadIdx.x;
    double v[N + 1];
#pragma unroll
    for (int j = 0; j <= N; ++j) v[j] = lane < nw && (j < N || pre) ? lds.part[j][lane] : 0.0;
#pragma unroll
    for (int off = kFoldWaves / 2; off > 0; off >>= 1)
#pragma unroll
        for (int j = 0; j <= N; ++j) v[j] += __shfl_xor(v[j], off, 64);
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        t[j] = j < N ? __shfl(v[j], 0, 64) : 0.0;
        pt[j] = j == 0 ? __shfl(v[N], 0, 64) : 0.0;
    }
}
template <int N, int FIN, int NCTL>
__device__ __forceinline__ const Ctl* fold_ctl(const CtlFold& f, const Ctl* ctl, Ctl* out, int nctl, int cur,
                                               int64_t rhs, bool write, FoldLds<N, NCTL>& lds)
{
    static_assert(sizeof(Ctl) % 8 == 0, "copied by words");
    const int wave = (int)threadIdx.x >> 6;
    const int words = nctl * (int)(sizeof(Ctl) / 4);
    const uint32_t* src = reinterpret_cast<const uint32_t*>(ctl);
    for (int i = threadIdx.x; i < words; i += blockDim.x) lds.ctl[i] = src[i];
    double v[N], u[1] = {0.0};
    sum_partials<N>(f.partials + rhs * f.slots * N, f.slots, v);
    wave_reduce<N>(v);
    const bool pre = f.pre_partials != nullptr;
    if (pre) {
        sum_partials<1>(f.pre_partials + rhs * f.pre_slots, f.pre_slots, u);
        wave_reduce<1>(u);
    }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) lds.part[j][wave] = v[j];
        lds.part[N][wave] = u[0];
    }
    __syncthreads();
    Ctl* c = reinterpret_cast<Ctl*>(lds.ctl);
    if (wave == 0) {
        double t[6], pt[6];
        fold_totals(lds, pre, t, pt);
        // the first step is one of two: the kernel holds only their code
        const int pf = !pre ? FIN_NONE : f.pre_fin == FIN_RU_RR ? FIN_RU_RR : FIN_CG_RR;
        ctl_step_wave(c + cur, pf, pt, FIN, t);
    }
    __syncthreads();
    if (write) {
        uint32_t* dst = reinterpret_cast<uint32_t*>(out);
        for (int i = threadIdx.x; i < words; i += blockDim.x) dst[i] = lds.ctl[i];
    }
    return c;
}

template <class R>
__device__ __forceinline__ cplx<R> cval(const double* d) { return {R(d[0]), R(d[1])}; }

// The work of block bx of nbx (x) and by (right-hand side) of a launch, on
// fields of kind KIND (spinors or colour vectors) stored at precision PREC.
template <int PREC, int KIND, int OP>
__device__ __forceinline__ void blas_block(const BlasArgs& a, int bx, int nbx, int by)
{
    using F = FieldIO<PREC, KIND>;
    using R = typename F::R;
    using Vec = typename F::Vec;
    constexpr int NC = F::NC;
    constexpr int N = BlasRed<OP>::N;
    constexpr int NN = N > 0 ? N : 1;
    // BLAS_MS_XP (one right-hand side): by is a share of the shifts
    const int rhs = OP == BLAS_MS_XP ? 0 : by;
    // each sub-field covers nbs whole blocks, so the sub-field is uniform per block
    const int nbs = nbx / a.nsub;
    const int sub = bx / nbs;
    const int64_t h = (int64_t)(bx - sub * nbs) * blockDim.x + threadIdx.x;
    const int64_t soff = (int64_t)sub * a.sub_stride;
    const int64_t r64 = rhs;
    const int64_t S = a.S;
    auto P = [&](void* base, int64_t st) { return static_cast<char*>(base) + r64 * st + soff; };

    const Ctl* ctl = a.ctl ? a.ctl + rhs : nullptr;
    constexpr int FIN = BlasFold<KIND, OP>::FIN;
    if constexpr (FIN != FIN_NONE) {
        constexpr bool MS = BlasFold<KIND, OP>::MS;
        if (a.fold.out) {
            __shared__ FoldLds<BlasFold<KIND, OP>::N, MS ? kMaxShifts : 1> lds;
            // multi-shift: the whole family steps with its base system
            const int n = MS ? a.fam_n : 1, cur = MS ? a.fam_base : 0;
            const Ctl* c0 = OP == BLAS_AXMY_NORM ? ctl - cur : ctl;
            c0 = fold_ctl<BlasFold<KIND, OP>::N, FIN>(a.fold, c0, a.fold.out + rhs, n, cur, rhs,
                                                       bx == 0 && (OP != BLAS_MS_XP || by == 0), lds);
            ctl = OP == BLAS_AXMY_NORM ? c0 + cur : c0;
            if (OP == BLAS_AXMY_NORM && ctl->done) return;
        } else if (OP == BLAS_AXMY_NORM && pred_skip(a.pred, ctl)) {
            return;
        }
        if (OP == BLAS_CG_XP && !ctl->xdo && ctl->done) return;
    } else if (pred_skip(a.pred, ctl)) {
        return;
    }

    double red[NN];
#pragma unroll
    for (int j = 0; j < NN; ++j) red[j] = 0.0;

    if (h < a.Vh) {
        if (OP == BLAS_CG_XP) {
            // one pass over p for both updates: five fields in and out of
            // memory here and three in BLAS_AXMY_NORM, against six and three
            // with x updated beside r
            const R al = R(ctl->alpha), be = R(ctl->beta);
            const bool dox = ctl->xdo != 0, dop = ctl->done == 0;
            Vec x, p, z;
            F::load(P(a.y, a.st_y), S, h, p);
            if (dox) F::load(P(a.x, a.st_x), S, h, x);
            if (dop) F::load(P(a.z, a.st_z), S, h, z);
            if (dox) {
#pragma unroll
                for (int k = 0; k < NC; ++k) F::at(x, k) = F::at(x, k) + al * F::at(p, k);
                F::store(P(a.x, a.st_x), S, h, x);
            }
            if (dop) {
#pragma unroll
                for (int k = 0; k < NC; ++k) F::at(p, k) = F::at(z, k) + be * F::at(p, k);
                F::store(P(a.y, a.st_y), S, h, p);
            }
        } else if (OP == BLAS_COPY) {
            Vec x;
            F::load(P(a.x, a.st_x), S, h, x);
            F::store(P(a.y, a.st_y), S, h, x);
        } else if (OP == BLAS_ZERO) {
            Vec x;
#pragma unroll
            for (int k = 0; k < NC; ++k) F::at(x, k) = {R(0), R(0)};
            F::store(P(a.y, a.st_y), S, h, x);
        } else if (OP == BLAS_SPIN_SCALE) {
            // spinors: coef.up on spins 0, 1 and coef.lo on spins 2, 3; colour vectors: coef.up
            const cplx<R> cu = cval<R>(a.coef.up), cl = cval<R>(a.coef.lo);
            Vec x;
            F::load(P(a.x, a.st_x), S, h, x);
#pragma unroll
            for (int k = 0; k < NC; ++k) F::at(x, k) = (KIND == KIND_COLOUR || k < 6 ? cu : cl) * F::at(x, k);
            F::store(P(a.y, a.st_y), S, h, x);
        } else if (OP == BLAS_NORM) {
            Vec x;
            F::load(P(a.x, a.st_x), S, h, x);
#pragma unroll
            for (int k = 0; k < NC; ++k) red[0] += (double)norm2(F::at(x, k));
        } else if (OP == BLAS_NORM_DOT) {
            Vec x, r0;
            F::load(P(a.x, a.st_x), S, h, x);
            F::load(static_cast<const char*>(a.r0) + r64 * a.st_r0 + soff, S, h, r0);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                red[0] += (double)norm2(F::at(x, k));
                const cplx<R> d = cmulc(F::at(r0, k), F::at(x, k));
                red[1] += (double)d.x;
                red[2] += (double)d.y;
            }
        } else if (OP == BLAS_XPY) {
            Vec x, y;
            F::load(P(a.x, a.st_x), S, h, x);
            F::load(P(a.y, a.st_y), S, h, y);
#pragma unroll
            for (int k = 0; k < NC; ++k) F::at(y, k) = F::at(y, k) + F::at(x, k);
            F::store(P(a.y, a.st_y), S, h, y);
        } else if (OP == BLAS_BI_P) {
            // beta = (rho / rho_old) (alpha / omega), computed in FP64
            double t1[2], t2[2], be[2];
            cdiv(ctl->rho, ctl->rho_old, t1);
            cdiv(ctl->balpha, ctl->omega, t2);
            be[0] = t1[0] * t2[0] - t1[1] * t2[1];
            be[1] = t1[0] * t2[1] + t1[1] * t2[0];
            const cplx<R> b = cval<R>(be), om = cval<R>(ctl->omega);
            Vec p, r, v;
            F::load(P(a.y, a.st_y), S, h, p);
            F::load(P(a.z, a.st_z), S, h, r);
            F::load(P(a.v, a.st_v), S, h, v);
#pragma unroll
            for (int k = 0; k < NC; ++k) F::at(p, k) = F::at(r, k) + b * (F::at(p, k) - om * F::at(v, k));
            F::store(P(a.y, a.st_y), S, h, p);
        } else if (OP == BLAS_BI_S) {
            const cplx<R> al = cval<R>(ctl->balpha);
            Vec r, v;
            F::load(P(a.z, a.st_z), S, h, r);
            F::load(P(a.v, a.st_v), S, h, v);
#pragma unroll
            for (int k = 0; k < NC; ++k) F::at(r, k) = F::at(r, k) - al * F::at(v, k);
            F::store(P(a.w, a.st_w), S, h, r);
        } else if (OP == BLAS_BI_XR) {
            // omega of this step (0 when ||t|| = 0: x += alpha p, r = s)
            const cplx<R> al = cval<R>(ctl->balpha), om = cval<R>(ctl->omega_step);
            Vec x, p, sv, t, r0, r;
            F::load(P(a.x, a.st_x), S, h, x);
            F::load(P(a.y, a.st_y), S, h, p);
            F::load(P(a.w, a.st_w), S, h, sv);
            F::load(P(a.v, a.st_v), S, h, t);
            F::load(static_cast<const char*>(a.r0) + r64 * a.st_r0 + soff, S, h, r0);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(x, k) = F::at(x, k) + al * F::at(p, k) + om * F::at(sv, k);
                F::at(r, k) = F::at(sv, k) - om * F::at(t, k);
                red[0] += (double)norm2(F::at(r, k));
                const cplx<R> d = cmulc(F::at(r0, k), F::at(r, k));
                red[1] += (double)d.x;
                red[2] += (double)d.y;
            }
            F::store(P(a.x, a.st_x), S, h, x);
            F::store(P(a.z, a.st_z), S, h, r);
        } else if (OP == BLAS_MS_XP) {
            // every shift's x_i += alpha_i p_i ; p_i = zeta_i z + beta_i p_i,
            // z and each p_i read once for both; shifts by, by + fam_gy, ...
            Vec z;
            F::load(P(a.z, a.st_z), S, h, z);
            char *xi = static_cast<char*>(a.x) + soff + by * a.st_x, *pi = static_cast<char*>(a.y) + soff + by * a.st_y;
            for (int i = by; i < a.fam_n; i += a.fam_gy, xi += a.fam_gy * a.st_x, pi += a.fam_gy * a.st_y) {
                const Ctl& c = ctl[i];
                const bool dox = c.xdo != 0, dop = c.done == 0;
                if (!dox && !dop) continue;
                const R al = R(c.alpha), ze = R(c.zeta), be = R(c.beta);
                Vec x, p;
                F::load(pi, S, h, p);
                if (dox) {
                    F::load(xi, S, h, x);
#pragma unroll
                    for (int k = 0; k < NC; ++k) F::at(x, k) = F::at(x, k) + al * F::at(p, k);
                    F::store(xi, S, h, x);
                }
                if (dop) {
#pragma unroll
                    for (int k = 0; k < NC; ++k) F::at(p, k) = ze * F::at(z, k) + be * F::at(p, k);
                    F::store(pi, S, h, p);
                }
            }
        } else if (OP == BLAS_BL_U0) {
            const cplx<R> be = cval<R>(ctl->bl_beta), g1 = cval<R>(ctl->bl_g1), g2 = cval<R>(ctl->bl_g2);
            Vec u0, r0v, u1, u2;
            F::load(P(a.y, a.st_y), S, h, u0);
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, u1);
            F::load(P(a.v, a.st_v), S, h, u2);
#pragma unroll
            for (int k = 0; k < NC; ++k)
                F::at(u0, k) = F::at(r0v, k) - be * (F::at(u0, k) - g1 * F::at(u1, k) - g2 * F::at(u2, k));
            F::store(P(a.y, a.st_y), S, h, u0);
        } else if (OP == BLAS_BL_XR0) {
            const cplx<R> al = cval<R>(ctl->balpha);
            Vec x, u0, r0v, u1;
            F::load(P(a.x, a.st_x), S, h, x);
            F::load(P(a.y, a.st_y), S, h, u0);
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, u1);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(x, k) = F::at(x, k) + al * F::at(u0, k);
                F::at(r0v, k) = F::at(r0v, k) - al * F::at(u1, k);
            }
            F::store(P(a.x, a.st_x), S, h, x);
            F::store(P(a.z, a.st_z), S, h, r0v);
        } else if (OP == BLAS_BL_U01) {
            const cplx<R> be = cval<R>(ctl->bl_beta);
            Vec u0, r0v, u1, r1;
            F::load(P(a.y, a.st_y), S, h, u0);
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, u1);
            F::load(P(a.v, a.st_v), S, h, r1);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(u0, k) = F::at(r0v, k) - be * F::at(u0, k);
                F::at(u1, k) = F::at(r1, k) - be * F::at(u1, k);
            }
            F::store(P(a.y, a.st_y), S, h, u0);
            F::store(P(a.w, a.st_w), S, h, u1);
        } else if (OP == BLAS_BL_XR01) {
            const cplx<R> al = cval<R>(ctl->balpha);
            Vec x, u0, r0v, u1, r1, u2;
            F::load(P(a.x, a.st_x), S, h, x);
            F::load(P(a.y, a.st_y), S, h, u0);
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, u1);
            F::load(P(a.v, a.st_v), S, h, r1);
            F::load(static_cast<const char*>(a.r0) + r64 * a.st_r0 + soff, S, h, u2);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(x, k) = F::at(x, k) + al * F::at(u0, k);
                F::at(r0v, k) = F::at(r0v, k) - al * F::at(u1, k);
                F::at(r1, k) = F::at(r1, k) - al * F::at(u2, k);
            }
            F::store(P(a.x, a.st_x), S, h, x);
            F::store(P(a.z, a.st_z), S, h, r0v);
            F::store(P(a.v, a.st_v), S, h, r1);
        } else if (OP == BLAS_BL_GRAM) {
            Vec r0v, r1, r2;
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, r1);
            F::load(P(a.v, a.st_v), S, h, r2);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                red[0] += (double)norm2(F::at(r1, k));
                const cplx<R> d12 = cmulc(F::at(r1, k), F::at(r2, k));
                const cplx<R> d10 = cmulc(F::at(r1, k), F::at(r0v, k));
                red[1] += (double)d12.x;
                red[2] += (double)d12.y;
                red[3] += (double)d10.x;
                red[4] += (double)d10.y;
            }
        } else if (OP == BLAS_BL_ORTH) {
            const cplx<R> ta = cval<R>(ctl->bl_tau);
            Vec r0v, r1, r2;
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, r1);
            F::load(P(a.v, a.st_v), S, h, r2);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(r2, k) = F::at(r2, k) - ta * F::at(r1, k);
                red[0] += (double)norm2(F::at(r2, k));
                const cplx<R> d = cmulc(F::at(r2, k), F::at(r0v, k));
                red[1] += (double)d.x;
                red[2] += (double)d.y;
            }
            F::store(P(a.v, a.st_v), S, h, r2);
        } else if (OP == BLAS_BL_MR) {
            const cplx<R> g1 = cval<R>(ctl->bl_g1), g2 = cval<R>(ctl->bl_g2);
            const cplx<R> gp1 = cval<R>(ctl->bl_gp1), gp2 = cval<R>(ctl->bl_gp2);
            Vec x, r0v, r1, r2, rt;
            F::load(P(a.x, a.st_x), S, h, x);
            F::load(P(a.z, a.st_z), S, h, r0v);
            F::load(P(a.w, a.st_w), S, h, r1);
            F::load(P(a.v, a.st_v), S, h, r2);
            F::load(static_cast<const char*>(a.r0) + r64 * a.st_r0 + soff, S, h, rt);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(x, k) = F::at(x, k) + g1 * F::at(r0v, k) + g2 * F::at(r1, k);
                F::at(r0v, k) = F::at(r0v, k) - gp1 * F::at(r1, k) - gp2 * F::at(r2, k);
                red[0] += (double)norm2(F::at(r0v, k));
                const cplx<R> d = cmulc(F::at(rt, k), F::at(r0v, k));
                red[1] += (double)d.x;
                red[2] += (double)d.y;
            }
            F::store(P(a.x, a.st_x), S, h, x);
            F::store(P(a.z, a.st_z), S, h, r0v);
        } else if (OP == BLAS_AXMY_NORM) {
            // z -= alpha w ; red ||z||^2
            const R al = R(ctl->alpha);
            Vec z, w;
            F::load(P(a.z, a.st_z), S, h, z);
            F::load(P(a.w, a.st_w), S, h, w);
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                F::at(z, k) = F::at(z, k) - al * F::at(w, k);
                red[0] += (double)norm2(F::at(z, k));
            }
            F::store(P(a.z, a.st_z), S, h, z);
        }
    }

    if (N > 0) block_reduce_store<NN>(red, a.r.partials + (int64_t)rhs * nbx * NN, bx);
}

// dst = src (ACC = 0), dst += src (1) or dst += src + alpha p (2, the grid
// strides over the sites: hardly any launch finds an update pending, and 512
// blocks that leave cost less than one per 256 sites).
template <int PD, int PS, int ACC>
__device__ __forceinline__ void convert_block(const ConvertArgs& a, int bx, int nbx, int by)
{
    const int rhs = by;
    const Ctl* ctl = a.ctl ? a.ctl + rhs : nullptr;
    using RD = typename SpinorIO<PD>::R;
    using RS = typename SpinorIO<PS>::R;
    RS al = RS(0);
    int sub = 0;
    int64_t h = (int64_t)bx * blockDim.x + threadIdx.x, step = (int64_t)nbx * blockDim.x;
    if constexpr (ACC == 2) {
        if (a.fold.out) {
            __shared__ FoldLds<1, 1> lds;
            ctl = fold_ctl<1, FIN_CG_RR>(a.fold, ctl, a.fold.out + rhs, 1, 0, rhs, bx == 0, lds);
            if (ctl->done || !ctl->update) return;
        } else if (pred_skip(a.pred, ctl)) {
            return;
        }
        al = RS(ctl->alpha);
    } else {
        if (pred_skip(a.pred, ctl)) return;
        const int nbs = nbx / a.nsub;
        sub = bx / nbs;
        h -= (int64_t)sub * nbs * blockDim.x;
        step = a.Vh;
    }
    char* dst = static_cast<char*>(a.dst) + rhs * a.rhs_stride_dst + sub * a.sub_stride_dst;
    char* src = static_cast<char*>(a.src) + rhs * a.rhs_stride_src + sub * a.sub_stride_src;
    for (; h < a.Vh; h += step) {
        Spinor<RS> v;
        SpinorIO<PS>::load(src, a.S, h, v);
        if constexpr (ACC == 2) {
            Spinor<RS> p;
            SpinorIO<PS>::load(static_cast<const char*>(a.p) + rhs * a.rhs_stride_p, a.S, h, p);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < 3; ++c) v.s[s][c] = v.s[s][c] + al * p.s[s][c];
        }
        Spinor<RD> d;
        if (ACC) SpinorIO<PD>::load(dst, a.S, h, d);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const cplx<RD> cv = {RD(v.s[s][c].x), RD(v.s[s][c].y)};
                d.s[s][c] = ACC ? d.s[s][c] + cv : cv;
            }
        SpinorIO<PD>::store(dst, a.S, h, d);
        if (a.zero_src) {
            Spinor<RS> z;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int c = 0; c < 3; ++c) z.s[s][c] = {RS(0), RS(0)};
            SpinorIO<PS>::store(src, a.S, h, z);
        }
    }
}

constexpr int kFinThreads = 1024;

// One right-hand side's finalize by a block: its steps' totals, then the steps,
// on a copy of the control block in LDS (the step reads a dozen scalars one
// after the other; from memory that took 3 us longer).
template <int N>
__device__ __forceinline__ void finalize_block(const FinArgs& f, int rhs, int count)
{
    constexpr int kWords = (int)(sizeof(Ctl) / 4);
    __shared__ FoldLds<N, 1> lds;
    Ctl* ctl = f.ctl + rhs;
    uint32_t* mem = reinterpret_cast<uint32_t*>(ctl);
    const bool ms = f.fin == FIN_MS_ALPHA || f.fin == FIN_MS_BETA || f.fin == FIN_MS_INIT || f.fin == FIN_MS_INIT_KEEP;
    for (int i = threadIdx.x; i < kWords; i += blockDim.x) lds.ctl[i] = mem[i];
    double v[N], u[1] = {0.0};
    sum_partials<N>(f.partials + (int64_t)rhs * f.nblocks * N, count, v);
    wave_reduce<N>(v);
    const bool pre = f.pre_partials != nullptr;
    if (pre) {
        sum_partials<1>(f.pre_partials + (int64_t)rhs * f.pre_slots, f.pre_slots, u);
        wave_reduce<1>(u);
    }
    const int wave = (int)threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) lds.part[j][wave] = v[j];
        lds.part[N][wave] = u[0];
    }
    __syncthreads();
    if (wave != 0) return;
    Ctl* c = reinterpret_cast<Ctl*>(lds.ctl);
    const bool skip = f.pred != PRED_ALWAYS && (c->done || (f.pred == PRED_UPDATE && !c->update) ||
                                                (f.pred == PRED_NO_UPDATE && c->update));
    if (skip && !closes_iteration(f.fin)) return;
    double t[6], pt[6];
    fold_totals(lds, pre, t, pt);
    if (ms) {  // the family is stepped in memory
        ctl_step_wave(ctl, FIN_NONE, pt, f.fin, t, f.pred == PRED_ALWAYS);
        return;
    }
    ctl_step_wave(c, pre ? f.pre_fin : FIN_NONE, pt, f.fin, t, f.pred == PRED_ALWAYS);
    __builtin_amdgcn_wave_barrier();
    for (int i = threadIdx.x; i < kWords; i += 64) mem[i] = lds.ctl[i];
}

}  // namespace lqcd
