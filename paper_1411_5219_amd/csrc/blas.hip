// Site-local kernels: the fused BLAS-1 steps of CGNR and BiCGStab with
// FP64 reductions, precision conversion, canonical <-> internal packing,
// and small utilities (zero fill, control-block set-up).
//
// Every kernel maps one work-item to one site of a parity field and walks
// that site's planes, so loads of one plane are coalesced across the
// wavefront and padding sites are never touched.
#include "lqcd.h"
#include "lqcd_device.h"
#include "lqcd_fin.h"
#include "lqcd_kernels.h"
#include "site_ops.h"

namespace lqcd {

template <int PREC, int KIND, int OP>
__global__ void __launch_bounds__(256) k_blas(const BlasArgs a)
{
    blas_block<PREC, KIND, OP>(a, blockIdx.x, gridDim.x, blockIdx.y);
}

template <int PREC, int KIND, int OP>
__global__ void __launch_bounds__(256) k_blas_batch(const BlasArgs* __restrict__ tab, const int* __restrict__ offs,
                                                   int nsys)
{
    int bx;
    const int s = batch_system(offs, nsys, &bx);
    if (bx >= tab[s].gx) return;  // padding of the system's range
    blas_block<PREC, KIND, OP>(tab[s], bx, tab[s].gx, blockIdx.y);
}

struct BlasLaunch {
    const BlasArgs* a;
    const BlasArgs* tab;
    const int* offs;
    int nsys;
};

template <int PREC, int KIND, int OP>
static hipError_t blas_one(const BlasLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if (L.tab) hipLaunchKernelGGL((k_blas_batch<PREC, KIND, OP>), grid, block, 0, s, L.tab, L.offs, L.nsys);
    else hipLaunchKernelGGL((k_blas<PREC, KIND, OP>), grid, block, 0, s, *L.a);
    return hipGetLastError();
}

#define LQCD_BLAS_CASE(OP) \
    case OP: return blas_one<PREC, KIND, OP>(L, grid, block, s);

// Spinor fields: every operation.
template <int PREC, int KIND>
static hipError_t blas_op(int op, const BlasLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if constexpr (KIND == KIND_SPINOR) {
        switch (op) {
            LQCD_BLAS_CASE(BLAS_CG_XP)
            LQCD_BLAS_CASE(BLAS_AXMY_NORM)
            LQCD_BLAS_CASE(BLAS_COPY)
            LQCD_BLAS_CASE(BLAS_ZERO)
            LQCD_BLAS_CASE(BLAS_SPIN_SCALE)
            LQCD_BLAS_CASE(BLAS_NORM)
            LQCD_BLAS_CASE(BLAS_BI_P)
            LQCD_BLAS_CASE(BLAS_BI_S)
            LQCD_BLAS_CASE(BLAS_BI_XR)
            LQCD_BLAS_CASE(BLAS_XPY)
            LQCD_BLAS_CASE(BLAS_NORM_DOT)
            LQCD_BLAS_CASE(BLAS_BL_U0)
            LQCD_BLAS_CASE(BLAS_BL_XR0)
            LQCD_BLAS_CASE(BLAS_BL_U01)
            LQCD_BLAS_CASE(BLAS_BL_XR01)
            LQCD_BLAS_CASE(BLAS_BL_GRAM)
            LQCD_BLAS_CASE(BLAS_BL_ORTH)
            LQCD_BLAS_CASE(BLAS_BL_MR)
        default: return hipErrorInvalidValue;
        }
    } else {
        // colour vectors: what the staggered CG and multi-shift CG use
        switch (op) {
            LQCD_BLAS_CASE(BLAS_COPY)
            LQCD_BLAS_CASE(BLAS_ZERO)
            LQCD_BLAS_CASE(BLAS_SPIN_SCALE)
            LQCD_BLAS_CASE(BLAS_NORM)
            LQCD_BLAS_CASE(BLAS_XPY)
            LQCD_BLAS_CASE(BLAS_MS_XP)
            LQCD_BLAS_CASE(BLAS_AXMY_NORM)
        default: return hipErrorInvalidValue;
        }
    }
}
#undef LQCD_BLAS_CASE

static hipError_t blas_prec(int prec, int kind, int op, const BlasLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if (kind == KIND_SPINOR) {
        if (prec == 64) return blas_op<64, KIND_SPINOR>(op, L, grid, block, s);
        if (prec == 32) return blas_op<32, KIND_SPINOR>(op, L, grid, block, s);
        if (prec == 16) return blas_op<16, KIND_SPINOR>(op, L, grid, block, s);
    } else if (kind == KIND_COLOUR) {
        if (prec == 64) return blas_op<64, KIND_COLOUR>(op, L, grid, block, s);
        if (prec == 32) return blas_op<32, KIND_COLOUR>(op, L, grid, block, s);
    }
    return hipErrorInvalidValue;
}

// Shares of the shifts of a multi-shift update: a thread passes over the shifts
// one after the other, each a load and a store later, and few blocks do not hide
// this; so as many shares as give the card's SIMDs a wave each (a solve with 32
// shifts: 8^3x4 5.13 -> 3.16 ms, 12^3x8 8.09 -> 6.06, 16^3x8 8.21 -> 6.83;
// one share from 24^3x8 on).
static int shift_shares(int64_t blocks, int blk, int nshift)
{
    const int64_t waves = blocks * (blk / 64);
    return (int)std::max<int64_t>(1, std::min<int64_t>(nshift, kSimds / waves));
}

hipError_t plan_blas(int prec, int op, const BlasArgs& a, int nrhs, const Launch& cfg, BlasPlan* out)
{
    if (prec != 64 && prec != 32 && prec != 16) return hipErrorInvalidValue;
    BlasPlan& p = *out;
    p.a = a;
    p.prec = prec;
    p.op = op;
    p.nrhs = nrhs;
    const int blk = cfg.block;
    const unsigned nbs = (unsigned)((a.Vh + blk - 1) / blk);
    p.a.fam_gy = op == BLAS_MS_XP ? shift_shares(nbs * a.nsub, blk, a.fam_n) : 1;
    p.grid = dim3(nbs * a.nsub, op == BLAS_MS_XP ? p.a.fam_gy : nrhs);
    p.a.gx = (int)p.grid.x;
    p.block = dim3(blk);
    p.nfin = (op == BLAS_NORM || op == BLAS_AXMY_NORM)                                           ? 1
             : (op == BLAS_BI_XR || op == BLAS_NORM_DOT || op == BLAS_BL_ORTH || op == BLAS_BL_MR) ? 3
             : op == BLAS_BL_GRAM                                                                 ? 5
                                                                                                  : 0;
    p.slots = (int)p.grid.x;
    if (p.nfin && p.slots > a.r.capacity) return hipErrorInvalidValue;  // partials too small
    if (a.r.fin == FIN_NONE) p.nfin = 0;
    return hipSuccess;
}

hipError_t exec_blas(const BlasPlan& p, hipStream_t s)
{
    BlasLaunch L{&p.a, nullptr, nullptr, 1};
    const hipError_t e = blas_prec(p.prec, p.a.kind, p.op, L, p.grid, p.block, s);
    if (e != hipSuccess || p.nfin == 0) return e;
    return launch_finalize(p.nfin, fin_args(p.a.r, p.slots, p.a.ctl, p.a.pred), p.nrhs, s);
}

hipError_t exec_blas_batch(const BlasPlan* plans, int n, const BlasArgs* tab, const int* offs, int total_blocks,
                           const FinArgs* fin_tab, hipStream_t s)
{
    if (n < 1) return hipErrorInvalidValue;
    const BlasPlan& p0 = plans[0];
    unsigned gx = 0;
    for (int i = 0; i < n; ++i) gx = plans[i].grid.x > gx ? plans[i].grid.x : gx;
    const BatchGrid bg = batch_grid(n, gx, p0.grid.y, (unsigned)total_blocks, offs);
    BlasLaunch L{nullptr, tab, bg.offs, n};
    const hipError_t e = blas_prec(p0.prec, p0.a.kind, p0.op, L, bg.grid, p0.block, s);
    if (e != hipSuccess || p0.nfin == 0) return e;
    return launch_finalize_batch(p0.nfin, fin_tab, n, p0.nrhs, s);
}

hipError_t launch_blas(int prec, int op, const BlasArgs& a, int nrhs, const Launch& cfg, hipStream_t s)
{
    BlasPlan p;
    hipError_t e = plan_blas(prec, op, a, nrhs, cfg, &p);
    if (e != hipSuccess) return e;
    if (Recorder* r = active_recorder()) {
        r->steps.push_back(Step{});
        r->steps.back().kind = STEP_BLAS;
        r->steps.back().b = p;
        return hipSuccess;
    }
    return exec_blas(p, s);
}

thread_local Recorder* g_recorder = nullptr;
Recorder* active_recorder() { return g_recorder; }
void set_recorder(Recorder* r) { g_recorder = r; }

template <int N>
__global__ void __launch_bounds__(kFinThreads) k_finalize(const FinArgs f, int count)
{
    finalize_block<N>(f, blockIdx.x, count);
}

// One block per (system, right-hand side): the finalize of every system of a batched launch.
template <int N>
__global__ void __launch_bounds__(kFinThreads) k_finalize_batch(const FinArgs* __restrict__ tab, int nrhs)
{
    const FinArgs& f = tab[blockIdx.x / nrhs];
    finalize_block<N>(f, blockIdx.x % nrhs, f.nblocks);
}

hipError_t launch_finalize_batch(int N, const FinArgs* tab, int nsys, int nrhs, hipStream_t s)
{
    dim3 g((unsigned)(nsys * nrhs)), b(kFinThreads);
    if (N == 1) hipLaunchKernelGGL(k_finalize_batch<1>, g, b, 0, s, tab, nrhs);
    else if (N == 2) hipLaunchKernelGGL(k_finalize_batch<2>, g, b, 0, s, tab, nrhs);
    else if (N == 3) hipLaunchKernelGGL(k_finalize_batch<3>, g, b, 0, s, tab, nrhs);
    else if (N == 5) hipLaunchKernelGGL(k_finalize_batch<5>, g, b, 0, s, tab, nrhs);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_finalize(int N, const FinArgs& f, int nrhs, hipStream_t s, int count)
{
    if (!f.ctl) return hipErrorInvalidValue;
    if (count < 0 || count > f.nblocks) count = f.nblocks;
    dim3 g(nrhs), b(kFinThreads);
    if (N == 1) hipLaunchKernelGGL(k_finalize<1>, g, b, 0, s, f, count);
    else if (N == 2) hipLaunchKernelGGL(k_finalize<2>, g, b, 0, s, f, count);
    else if (N == 3) hipLaunchKernelGGL(k_finalize<3>, g, b, 0, s, f, count);
    else if (N == 5) hipLaunchKernelGGL(k_finalize<5>, g, b, 0, s, f, count);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Precision conversion

template <int PD, int PS, int ACC>
__global__ void __launch_bounds__(256) k_convert(const ConvertArgs a)
{
    convert_block<PD, PS, ACC>(a, blockIdx.x, gridDim.x, blockIdx.y);
}

template <int PD, int PS, int ACC>
__global__ void __launch_bounds__(256) k_convert_batch(const ConvertArgs* __restrict__ tab,
                                                      const int* __restrict__ offs, int nsys)
{
    int bx;
    const int s = batch_system(offs, nsys, &bx);
    if (bx >= tab[s].gx) return;  // padding of the system's range
    convert_block<PD, PS, ACC>(tab[s], bx, tab[s].gx, blockIdx.y);
}

struct ConvertLaunch {
    const ConvertArgs* a;
    const ConvertArgs* tab;
    const int* offs;
    int nsys;
};

template <int PD, int PS, int ACC>
static hipError_t convert_one(const ConvertLaunch& L, dim3 g, dim3 b, hipStream_t s)
{
    if (L.tab) hipLaunchKernelGGL((k_convert_batch<PD, PS, ACC>), g, b, 0, s, L.tab, L.offs, L.nsys);
    else hipLaunchKernelGGL((k_convert<PD, PS, ACC>), g, b, 0, s, *L.a);
    return hipGetLastError();
}

static hipError_t convert_any(int pd, int ps, int acc, const ConvertLaunch& L, dim3 g, dim3 b, hipStream_t s)
{
#define LQCD_CONV(D, S_, A) \
    if (pd == D && ps == S_ && acc == A) return convert_one<D, S_, A>(L, g, b, s);
    LQCD_CONV(64, 64, 0)
    LQCD_CONV(64, 32, 0)
    LQCD_CONV(64, 16, 0)
    LQCD_CONV(32, 64, 0)
    LQCD_CONV(32, 32, 0)
    LQCD_CONV(32, 16, 0)
    LQCD_CONV(16, 64, 0)
    LQCD_CONV(16, 32, 0)
    LQCD_CONV(16, 16, 0)
    LQCD_CONV(64, 64, 1)
    LQCD_CONV(64, 32, 1)
    LQCD_CONV(64, 16, 1)
    LQCD_CONV(64, 32, 2)
    LQCD_CONV(64, 16, 2)
#undef LQCD_CONV
    return hipErrorInvalidValue;
}

hipError_t plan_convert(int pd, int ps, const ConvertArgs& a, int nrhs, ConvertPlan* out)
{
    const int blk = 256;
    unsigned nbs = (unsigned)((a.Vh + blk - 1) / blk);
    if (a.accumulate == 2) {
        if (a.nsub != 1) return hipErrorInvalidValue;
        const unsigned most = (unsigned)(512 / nrhs > 0 ? 512 / nrhs : 1);
        if (nbs > most) nbs = most;
    }
    out->a = a;
    out->pd = pd;
    out->ps = ps;
    out->grid = dim3(nbs * a.nsub, nrhs);
    out->a.gx = (int)out->grid.x;
    out->block = dim3(blk);
    return hipSuccess;
}

hipError_t exec_convert(const ConvertPlan& p, hipStream_t s)
{
    ConvertLaunch L{&p.a, nullptr, nullptr, 1};
    return convert_any(p.pd, p.ps, p.a.accumulate, L, p.grid, p.block, s);
}

hipError_t exec_convert_batch(const ConvertPlan* plans, int n, const ConvertArgs* tab, const int* offs,
                              int total_blocks, hipStream_t s)
{
    if (n < 1) return hipErrorInvalidValue;
    const ConvertPlan& p0 = plans[0];
    unsigned gx = 0;
    for (int i = 0; i < n; ++i) gx = plans[i].grid.x > gx ? plans[i].grid.x : gx;
    const BatchGrid bg = batch_grid(n, gx, p0.grid.y, (unsigned)total_blocks, offs);
    ConvertLaunch L{nullptr, tab, bg.offs, n};
    return convert_any(p0.pd, p0.ps, p0.a.accumulate, L, bg.grid, p0.block, s);
}

hipError_t launch_convert(int pd, int ps, const ConvertArgs& a, int nrhs, hipStream_t s)
{
    ConvertPlan p;
    hipError_t e = plan_convert(pd, ps, a, nrhs, &p);
    if (e != hipSuccess) return e;
    if (Recorder* r = active_recorder()) {
        r->steps.push_back(Step{});
        r->steps.back().kind = STEP_CONVERT;
        r->steps.back().c = p;
        return hipSuccess;
    }
    return exec_convert(p, s);
}

// ---------------------------------------------------------------------------
// Canonical complex128 <-> internal layouts

// A canonical array holds one record of NC complex128 per site, x fastest; site
// 2h and 2h + 1 of it are the two sites h of the parity fields, so a block's 64
// sites of both parities are 128 records in a row.  Records are moved between
// memory and LDS 16 bytes per lane in address order and between LDS and the
// planes one site per lane; reading them from memory one per lane, as pieces
// 16 bytes wide and 192 apart, bounded the conversions by L1 requests (32^3x8,
// four FP64 spinors: in 91 -> 83 us, out 105 -> 73, links 74 -> 64, which is
// 4.7 to 5.5 TB/s; 32 or 128 sites, or streaming accesses, within 2%).
constexpr int kPackSites = 64;  // per parity and block
template <int NC>
struct PackLds {
    // an odd record length in units of 16 bytes: a wave reading one record per
    // lane then meets every bank equally often
    static constexpr int LD = NC | 1;
    double2 v[2 * kPackSites * LD];

    __device__ __forceinline__ void fill(const double2* canon, int n)
    {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int e = (int)threadIdx.x + 2 * kPackSites * k;
            if (e < n * NC) v[e + (LD - NC) * (e / NC)] = canon[e];
        }
    }
    __device__ __forceinline__ void drain(double2* canon, int n) const
    {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int e = (int)threadIdx.x + 2 * kPackSites * k;
            if (e < n * NC) canon[e] = v[e + (LD - NC) * (e / NC)];
        }
    }
};
// Which of the records 2h, 2h + 1 is the site of parity p.
__device__ __forceinline__ int pack_odd(const Geom& g, int p, int h)
{
    const int row = h / g.Lxh, q = row / g.L[1], t = q / g.L[2];
    return (row - q * g.L[1] + q - t * g.L[2] + t + p) & 1;
}

// Canonical (V, NC) complex128 per right-hand side <-> internal parity
// fields of kind KIND (NC = 12 for spinors, 3 for colour vectors).
template <int PREC, int KIND, bool PACK>
__global__ void __launch_bounds__(2 * kPackSites) k_pack_field(const Geom g, const double2* canon_c, double2* canon_m,
                                                              const char* in, char* out)
{
    using F = FieldIO<PREC, KIND>;
    using R = typename F::R;
    constexpr int NC = F::NC;
    __shared__ PackLds<NC> lds;
    const int rhs = blockIdx.y, h0 = (int)blockIdx.x * kPackSites, n = min(kPackSites, g.Vh - h0);
    const int64_t first = ((int64_t)rhs * 2 * g.Vh + 2 * h0) * NC;
    const int p = (int)threadIdx.x / kPackSites, l = (int)threadIdx.x % kPackSites, h = h0 + l;
    const int64_t par_bytes = field_parity_bytes(KIND, PREC, g.S);
    const int64_t foff = (int64_t)rhs * 2 * par_bytes + p * par_bytes;
    double2* c = lds.v + (2 * l + (l < n ? pack_odd(g, p, h) : 0)) * PackLds<NC>::LD;
    typename F::Vec v;
    if (PACK) {
        lds.fill(canon_c + first, 2 * n);
        __syncthreads();
        if (l >= n) return;
#pragma unroll
        for (int k = 0; k < NC; ++k) F::at(v, k) = {R(c[k].x), R(c[k].y)};
        F::store(out + foff, g.S, h, v);
    } else {
        if (l < n) {
            F::load(in + foff, g.S, h, v);
#pragma unroll
            for (int k = 0; k < NC; ++k) c[k] = make_double2((double)F::at(v, k).x, (double)F::at(v, k).y);
        }
        __syncthreads();
        lds.drain(canon_m + first, 2 * n);
    }
}

template <int KIND>
static hipError_t pack_kind(int prec, bool pack, const Geom& g, const void* canon, const void* in, void* out, int nrhs,
                            hipStream_t s)
{
    dim3 b(2 * kPackSites), gr((unsigned)((g.Vh + kPackSites - 1) / kPackSites), nrhs);
    const double2* cc = static_cast<const double2*>(canon);
    double2* cm = static_cast<double2*>(const_cast<void*>(canon));
    const char* i = static_cast<const char*>(in);
    char* o = static_cast<char*>(out);
#define LQCD_PACK(P)                                                                                         \
    if (prec == P) {                                                                                         \
        if (pack) hipLaunchKernelGGL((k_pack_field<P, KIND, true>), gr, b, 0, s, g, cc, nullptr, nullptr, o); \
        else hipLaunchKernelGGL((k_pack_field<P, KIND, false>), gr, b, 0, s, g, nullptr, cm, i, nullptr);    \
        return hipGetLastError();                                                                            \
    }
    LQCD_PACK(64)
    LQCD_PACK(32)
    LQCD_PACK(16)
#undef LQCD_PACK
    return hipErrorInvalidValue;
}

hipError_t launch_pack_spinor(int prec, const Geom& g, const void* canon, void* out, int nrhs, hipStream_t s)
{
    return pack_kind<KIND_SPINOR>(prec, true, g, canon, nullptr, out, nrhs, s);
}

hipError_t launch_unpack_spinor(int prec, const Geom& g, const void* in, void* canon, int nrhs, hipStream_t s)
{
    return pack_kind<KIND_SPINOR>(prec, false, g, canon, in, nullptr, nrhs, s);
}

hipError_t launch_pack_colour(int prec, const Geom& g, const void* canon, void* out, int nrhs, hipStream_t s)
{
    return pack_kind<KIND_COLOUR>(prec, true, g, canon, nullptr, out, nrhs, s);
}

hipError_t launch_unpack_colour(int prec, const Geom& g, const void* in, void* canon, int nrhs, hipStream_t s)
{
    return pack_kind<KIND_COLOUR>(prec, false, g, canon, in, nullptr, nrhs, s);
}

// Canonical (4, V, 9) complex128 links into storage (PREC, RECON).
template <int PREC, int RECON>
__global__ void __launch_bounds__(2 * kPackSites) k_pack_gauge(const Geom g, const double2* canon, void* out)
{
    __shared__ PackLds<9> lds;
    const int mu = blockIdx.y, h0 = (int)blockIdx.x * kPackSites, n = min(kPackSites, g.Vh - h0);
    const int p = (int)threadIdx.x / kPackSites, l = (int)threadIdx.x % kPackSites, h = h0 + l;
    lds.fill(canon + ((int64_t)mu * 2 * g.Vh + 2 * h0) * 9, 2 * n);
    __syncthreads();
    if (l >= n) return;
    const double2* c = lds.v + (2 * l + pack_odd(g, p, h)) * PackLds<9>::LD;
    Link<double> U;
#pragma unroll
    for (int k = 0; k < 9; ++k) U.u[k / 3][k % 3] = {c[k].x, c[k].y};
    LinkIO<PREC, RECON>::store(out, g.S, mu * 2 + p, h, U);
}

// Links of the internal FP64 field with SRC_RECON reals per link into storage
// (PREC, RECON) (a 12-real source has its third row rebuilt in FP64 first).
template <int PREC, int RECON, int SRC_RECON>
__global__ void __launch_bounds__(256) k_convert_gauge(const Geom g, const void* U64, void* out)
{
    const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int blk = blockIdx.y;  // mu * 2 + parity
    if (h >= g.Vh) return;
    Link<double> U;
    LinkIO<64, SRC_RECON>::load(U64, g.S, blk, h, U);
    LinkIO<PREC, RECON>::store(out, g.S, blk, h, U);
}

template <int PREC, int RECON>
static hipError_t gauge_one(const Geom& g, const void* canon, const void* U64, int src_recon, void* out, hipStream_t s)
{
    if (canon) {
        const dim3 gr((unsigned)((g.Vh + kPackSites - 1) / kPackSites), 4);
        hipLaunchKernelGGL((k_pack_gauge<PREC, RECON>), gr, dim3(2 * kPackSites), 0, s, g,
                           static_cast<const double2*>(canon), out);
    } else {
        const dim3 b(256), gr((unsigned)((g.Vh + 255) / 256), 8);
        if (src_recon == 12) hipLaunchKernelGGL((k_convert_gauge<PREC, RECON, 12>), gr, b, 0, s, g, U64, out);
        else if (src_recon == 18) hipLaunchKernelGGL((k_convert_gauge<PREC, RECON, 18>), gr, b, 0, s, g, U64, out);
        else return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

static hipError_t gauge_any(int prec, int recon, const Geom& g, const void* canon, const void* U64, int src_recon,
                            void* out, hipStream_t s)
{
    if (prec == 64 && recon == 18) return gauge_one<64, 18>(g, canon, U64, src_recon, out, s);
    if (prec == 64 && recon == 12) return gauge_one<64, 12>(g, canon, U64, src_recon, out, s);
    if (prec == 32 && recon == 18) return gauge_one<32, 18>(g, canon, U64, src_recon, out, s);
    if (prec == 32 && recon == 12) return gauge_one<32, 12>(g, canon, U64, src_recon, out, s);
    if (prec == 16 && recon == 12) return gauge_one<16, 12>(g, canon, U64, src_recon, out, s);
    return hipErrorInvalidValue;
}

hipError_t launch_pack_gauge(int prec, int recon, const Geom& g, const void* canon, void* out, hipStream_t s)
{
    if (!canon) return hipErrorInvalidValue;
    return gauge_any(prec, recon, g, canon, nullptr, 0, out, s);
}

hipError_t launch_convert_gauge(int prec, int recon, const Geom& g, const void* U64, int src_recon, void* out,
                                hipStream_t s)
{
    return gauge_any(prec, recon, g, nullptr, U64, src_recon, out, s);
}

// ---------------------------------------------------------------------------

__global__ void k_fill_zero(uint4* p, int64_t n16, unsigned char* tail, int ntail)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n16) p[i] = make_uint4(0u, 0u, 0u, 0u);
    if (i < ntail) tail[i] = 0;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return hipSuccess;
    const int64_t n16 = (int64_t)(bytes / 16);
    const int ntail = (int)(bytes - 16 * n16);
    const int64_t n = n16 > ntail ? n16 : ntail;
    dim3 b(256), g((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL(k_fill_zero, g, b, 0, s, static_cast<uint4*>(p), n16,
                       static_cast<unsigned char*>(p) + 16 * n16, ntail);
    return hipGetLastError();
}

__global__ void k_ctl_init(Ctl* ctl, int nrhs, CtlInit in)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrhs) return;
    ctl[i] = ctl_make(in);
}

hipError_t launch_ctl_init(Ctl* ctl, int nrhs, const CtlInit& in, hipStream_t s)
{
    hipLaunchKernelGGL(k_ctl_init, dim3((nrhs + 63) / 64), dim3(64), 0, s, ctl, nrhs, in);
    return hipGetLastError();
}

hipError_t launch_ctl_init(Ctl* ctl, int nrhs, double tol, double delta, int iter_limit, hipStream_t s)
{
    CtlInit in{};
    in.tol = tol;
    in.delta = delta;
    in.iter_limit = iter_limit;
    return launch_ctl_init(ctl, nrhs, in, s);
}

__global__ void k_ctl_init_shifts(Ctl* ctl, int n, int base, ShiftList shifts)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    ctl[i].sigma = shifts.s[i] - shifts.s[base];
    ctl[i].ms_index = i;
    ctl[i].ms_n = n;
    ctl[i].ms_base = base;
}

hipError_t launch_ctl_init_shifts(Ctl* ctl, int n, int base, const ShiftList& shifts, hipStream_t s)
{
    if (n < 1 || n > kMaxShifts || base < 0 || base >= n) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ctl_init_shifts, dim3(1), dim3(64), 0, s, ctl, n, base, shifts);
    return hipGetLastError();
}

__global__ void k_ctl_reopen(Ctl* ctl, int nrhs, unsigned mask, int no_fallback)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nrhs || !((mask >> i) & 1u)) return;
    ctl[i].done = 0;
    ctl[i].status = 0;
    ctl[i].update = 0;
    ctl[i].reset_p = 0;
    ctl[i].outer_req = 0;
    if (no_fallback) ctl[i].fallback_ok = 0;
}

hipError_t launch_ctl_reopen(Ctl* ctl, int nrhs, unsigned mask, hipStream_t s, bool no_fallback)
{
    hipLaunchKernelGGL(k_ctl_reopen, dim3((nrhs + 63) / 64), dim3(64), 0, s, ctl, nrhs, mask, no_fallback ? 1 : 0);
    return hipGetLastError();
}

}  // namespace lqcd
