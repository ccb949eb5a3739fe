// Kernel argument blocks and the host-side launchers of every kernel in the
// library (the solvers' control block is in solver_ctl.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "chunks.h"
#include "hop_form.h"
#include "solver_ctl.h"

namespace lqcd {

// Lattice geometry as the kernels see it.
struct Geom {
    int L[4];        // extents x, y, z, t (all even)
    int Lxh;         // L[0] / 2
    int Vh;          // sites per parity
    int64_t S;       // plane stride in sites (Vh rounded up to an odd multiple of 16)
    double ph[4][2]; // exp(i theta_mu): applied on hops that cross the boundary
};

// Spin-block coefficients (upper spins 0,1 / lower spins 2,3), complex.
struct SpinCoef {
    double up[2];
    double lo[2];
};

// Which scalars a reduction produces (totals per right-hand side):
//   RED_NONE
//   RED_NORM    : ||out||^2
//   RED_NORM_DS : ||out||^2, <out, site>          (re, im)
//   RED_DOT_AUX : <aux, out>                      (re, im)
//   RED_NORM_LOW: ||out||^2, and out is also stored at low_prec (FP64 Wilson hops)
enum Red { RED_NONE = 0, RED_NORM = 1, RED_NORM_DS = 2, RED_DOT_AUX = 3, RED_NORM_LOW = 4 };

// Predicates on the control block evaluated at the top of a kernel.
enum Pred {
    PRED_ALWAYS = 0,      // ignore the control block
    PRED_ACTIVE = 1,      // skip when done
    PRED_UPDATE = 2,      // run only while a reliable update is pending (and not done)
    PRED_NO_UPDATE = 3,   // run only while no update is pending (and not done)
};

// Most values one reduction produces per block (BiCGStab(2)'s Gram step).
constexpr int kMaxFin = 5;

struct RedArgs {
    double* partials;       // [nrhs][nblocks][N]
    int capacity;           // blocks the partials hold per right-hand side (N <= kMaxFin)
    int fin;                // Fin
    int fin_even;           // full-lattice launches: a second Fin on the even-parity blocks' partials (0: none)
    // a scalar step of an earlier launch run before fin (null: none): its partials, slots and Fin
    const double* pre_partials;
    int pre_slots, pre_fin;
};

// Scalar steps that the blocks of a consuming kernel run themselves instead of
// a launch of their own: every block sums the partials in the same order, runs
// the steps on its copy of the control block and goes on with the result;
// block 0 writes it to out, a copy no block of the launch reads.
struct CtlFold {
    Ctl* out;               // per right-hand side; null: nothing folded, a.ctl is up to date
    const double* partials; // [nrhs][slots][N]
    int slots;
    const double* pre_partials;  // [nrhs][pre_slots] (null: no first step)
    int pre_slots, pre_fin;
};

// Dslash_eo with a fused epilogue:
//   out = add + a * site + c * (sum of the 8 hops of `in` onto parity `parity`)
// with a, c spin-block coefficients; `add`, `site`, `out` may be null.
struct DslashArgs {
    Geom g;
    int parity;
    int pred;
    const void* in;
    void* out;
    const void* site;
    const void* add;
    const void* aux;
    const void* U;
    void* low;              // RED_NORM_LOW
    int low_prec;
    SpinCoef a, c;
    // bytes between right-hand sides of each field
    int64_t st_in, st_out, st_site, st_add, st_aux, st_low;
    int full;               // 1: both parities in one launch (fields are full-lattice)
    int64_t par_bytes;      // bytes of one parity field (full = 1)
    RedArgs r;
    Ctl* ctl;               // per right-hand side, or null
    int swizzle;
    int nrhs;               // right-hand sides (set by the launcher)
    int gx;                 // planned grid.x (batched launches pad each system's range)
    ChunkArgs ch;
};

// Waves per SIMD the one-right-hand-side hop kernels are compiled for (their
// register budget): FP64 holds about 250 registers at two waves, FP32 and FP16
// keep three.
__host__ __device__ constexpr int hop_waves(int prec) { return prec == 64 ? 2 : 3; }

// Launch configuration picked per kernel (autotuned).
struct Launch {
    int block = 128;
    int swizzle = 1;
    int order = 0;     // 0: memory order, 1: t-fastest chunks of xy planes, k > 1: z-slabs of k planes (hops)
    int rhs_tile = 4;  // rhs_tile, rhs_group, rhs_lanes: part of the C ABI's struct, without effect
    int rhs_group = 4; // (hop_form chooses how right-hand sides share links)
    int ygroup = 1;    // blocks of a plane interleaved after t, in units of the block request (1: none)
    int rhs_lanes = 1;
    int form = FORM_BY_SIZE;  // HopForm of Wilson hops (given where several launches must run the same kernel)
};

// hop_form of the n lattices g.
int hop_form(int prec, int recon, bool full, const Geom* g, int n, int nrhs, bool rare = false);

// Finalize of one reduction of one system.
struct FinArgs {
    const double* partials;
    int nblocks;
    int fin;
    Ctl* ctl;
    int pred;
    const double* pre_partials;  // as in RedArgs
    int pre_slots, pre_fin;
};
inline FinArgs fin_args(const RedArgs& r, int slots, Ctl* ctl, int pred)
{
    return FinArgs{r.partials, slots, r.fin, ctl, pred, r.pre_partials, r.pre_slots, r.pre_fin};
}
// Sum N block partials per right-hand side in block order and run the
// solver's scalar steps on the totals; one block per right-hand side.
// count < nblocks sums only the first count partials of each right-hand
// side (nblocks stays the stride between right-hand sides).
hipError_t launch_finalize(int N, const FinArgs& f, int nrhs, hipStream_t s, int count = -1);

// ---- launchers (return hipError_t) ----
hipError_t launch_dslash(int prec, int recon, bool dagger, int red, const DslashArgs& a, int nrhs,
                         const Launch& cfg, hipStream_t s);
// The staggered even-odd hop with the same arguments: out = add + a * site +
// c * sum_mu eta_mu [U chi(x + mu) - U^+ chi(x - mu)] (a, c: the up entries of
// the coefficients), one right-hand side per work-item, reductions NONE, NORM
// or NORM_DS.
hipError_t launch_stag(int prec, int recon, int red, const DslashArgs& args, int nrhs, const Launch& cfg,
                       hipStream_t s);

// Grid of a batched launch.  Systems of about one size lie along z, each padded
// to the widest, so that a block knows its system at once; offs is null then.
// Others lie one after the other along x and a block searches offs, a trip to
// memory before the one for its arguments (mixed solves of four lattices of 1728
// to 4096 sites, four right-hand sides each: 5.85 ms searched, 5.55 along z).
struct BatchGrid {
    dim3 grid;
    const int* offs;
};
inline BatchGrid batch_grid(int nsys, unsigned widest, unsigned gy, unsigned total, const int* offs)
{
    const unsigned gx = (widest + 7) / 8 * 8;  // whole rounds over the XCDs
    if ((uint64_t)gx * nsys <= 2 * (uint64_t)total) return {dim3(gx, gy, (unsigned)nsys), nullptr};
    return {dim3(total, gy), offs};
}
#if defined(__HIPCC__)
__device__ __forceinline__ int batch_system(const int* offs, int nsys, int* bx)
{
    const int x = blockIdx.x;
    if (!offs) {
        *bx = x;
        return blockIdx.z;
    }
    int s = 0;
    while (s + 1 < nsys && x >= offs[s + 1]) ++s;
    *bx = x - offs[s];
    return s;
}
#endif

// One Dslash launch, or a batch of nsys argument sets in device memory.
struct DslashLaunch {
    const DslashArgs* a;
    const DslashArgs* tab;
    const int* offs;
    int nsys;
};

// A planned Dslash launch (final arguments, grid, kernel selectors).
// Stencil of a planned hop launch.
enum PlanKind { PLAN_WILSON = 0, PLAN_STAG = 1 };

struct DslashPlan {
    DslashArgs a;
    dim3 grid, block;
    int kind;   // PlanKind
    int prec, recon, red;
    int split;  // waves per chunk of sites, 0: several right-hand sides per block
    int halves; // split = 0: waves per right-hand side
    bool dag;
    bool lnt;   // streaming link loads (no other block of the launch reads the links)
    bool next;  // right-hand sides next to each other in the block order
    int nfin;   // values per finalize (0: no reduction)
    int slots;  // partial slots per right-hand side
};
hipError_t plan_dslash(int prec, int recon, bool dagger, int red, const DslashArgs& args, int nrhs, const Launch& cfg,
                       DslashPlan* out);
hipError_t plan_stag_hop(int prec, int recon, int red, const DslashArgs& args, int nrhs, const Launch& cfg,
                         DslashPlan* out);
hipError_t exec_dslash(const DslashPlan& p, hipStream_t s);
// plans[0..n) share kernel selectors; tab / offs / fin_tab are their device
// tables (arguments, block offsets with offs[n] = total_blocks, finalizes).
hipError_t exec_dslash_batch(const DslashPlan* plans, int n, const DslashArgs* tab, const int* offs, int total_blocks,
                             const FinArgs* fin_tab, hipStream_t s);
hipError_t launch_finalize_batch(int N, const FinArgs* tab, int nsys, int nrhs, hipStream_t s);

// Site-local BLAS-1 on parity fields of precision prec (all operands the same).
enum Blas {
    BLAS_CG_XP = 1,       // x += alpha p (while xdo); p = z + beta p (while not done)
    BLAS_COPY = 2,        // y = x
    BLAS_ZERO = 3,        // y = 0
    BLAS_SPIN_SCALE = 4,  // y = coef * x                          (spin-block coefficient)
    BLAS_NORM = 5,        // red ||x||^2
    BLAS_BI_P = 6,        // p = r + beta (p - omega v), beta = (rho/rho_old)(alpha/omega)
    BLAS_BI_S = 7,        // s = r - alpha v
    BLAS_BI_XR = 8,       // x += alpha p + omega s; r = s - omega t; red ||r||^2, <r0, r>
    BLAS_XPY = 9,         // y += x
    BLAS_NORM_DOT = 10,   // red ||x||^2, <r0, x>
    BLAS_MS_XP = 11,      // x_i += alpha_i p_i (while xdo); p_i = zeta_i z + beta_i p_i (while not done), every shift
    BLAS_AXMY_NORM = 13,  // z -= alpha w;                         red ||z||^2
    // BiCGStab(2) (coefficients from each right-hand side's Ctl): y = u_0,
    // z = r_0, w = u_1 or r_1, v = u_2, r_1 or r_2, r0 = u_2 or rt
    BLAS_BL_U0 = 14,      // u_0 = r_0 - beta (u_0 - g1 u_1 - g2 u_2)         (y, z, w = u_1, v = u_2)
    BLAS_BL_XR0 = 15,     // x += alpha u_0; r_0 -= alpha u_1                 (x, y, z, w = u_1)
    BLAS_BL_U01 = 16,     // u_0 = r_0 - beta u_0; u_1 = r_1 - beta u_1       (y, z, w = u_1, v = r_1)
    BLAS_BL_XR01 = 17,    // x += alpha u_0; r_0 -= alpha u_1; r_1 -= alpha u_2 (x, y, z, w = u_1, v = r_1, r0 = u_2)
    BLAS_BL_GRAM = 18,    // red ||r_1||^2, <r_1, r_2>, <r_1, r_0>            (z, w = r_1, v = r_2)
    BLAS_BL_ORTH = 19,    // r_2 -= tau r_1; red ||r_2||^2, <r_2, r_0>         (z, w = r_1, v = r_2)
    BLAS_BL_MR = 20,      // x += g1 r_0 + g2 r_1; r_0 -= gp1 r_1 + gp2 r_2; red ||r_0||^2, <rt, r_0>
                          //                                                  (x, z, w = r_1, v = r_2, r0 = rt)
};

struct BlasArgs {
    int kind;               // FieldKind of every operand (0: spinor, 1: colour vector)
    int Vh;
    int64_t S;
    int nsub;               // sub-fields of Vh sites each (1: parity field, 2: full lattice)
    int64_t sub_stride;     // bytes between sub-fields
    int pred;
    void* x;
    void* y;
    void* z;
    void* w;
    void* v;
    const void* r0;
    SpinCoef coef;
    // bytes between right-hand sides of each operand
    int64_t st_x, st_y, st_z, st_w, st_v, st_r0;
    RedArgs r;
    Ctl* ctl;
    int fam_n, fam_base;    // multi-shift: systems and index of the base system
    int fam_gy;             // BLAS_MS_XP: shares of the shifts, one along grid.y each (plan_blas)
    CtlFold fold;           // BLAS_AXMY_NORM, BLAS_CG_XP, BLAS_MS_XP
    int gx;                 // planned grid.x (batched launches)
};

hipError_t launch_blas(int prec, int op, const BlasArgs& a, int nrhs, const Launch& cfg, hipStream_t s);

struct BlasPlan {
    BlasArgs a;
    dim3 grid, block;
    int prec, op, nrhs;
    int nfin, slots;
};
hipError_t plan_blas(int prec, int op, const BlasArgs& a, int nrhs, const Launch& cfg, BlasPlan* out);
hipError_t exec_blas(const BlasPlan& p, hipStream_t s);
hipError_t exec_blas_batch(const BlasPlan* plans, int n, const BlasArgs* tab, const int* offs, int total_blocks,
                           const FinArgs* fin_tab, hipStream_t s);

// Precision conversion of a parity field: dst(prec_dst) = src(prec_src);
// accumulate = 1: dst += src (dst FP64); 2: dst += src + alpha p, p at src's
// precision, the reliable update of a CG iteration whose x still lacks alpha p.
struct ConvertArgs {
    int Vh;
    int64_t S;
    int nsub;
    int64_t sub_stride_dst, sub_stride_src;
    int64_t rhs_stride_dst, rhs_stride_src;
    void* dst;
    void* src;
    int accumulate;
    const void* p;          // accumulate = 2
    int64_t rhs_stride_p;
    CtlFold fold;           // accumulate = 2
    int zero_src;           // src = 0 afterwards
    int pred;
    Ctl* ctl;
    int gx;                 // planned grid.x (batched launches)
};
hipError_t launch_convert(int prec_dst, int prec_src, const ConvertArgs& a, int nrhs, hipStream_t s);

struct ConvertPlan {
    ConvertArgs a;
    dim3 grid, block;
    int pd, ps;
};
hipError_t plan_convert(int prec_dst, int prec_src, const ConvertArgs& a, int nrhs, ConvertPlan* out);
hipError_t exec_convert(const ConvertPlan& p, hipStream_t s);
hipError_t exec_convert_batch(const ConvertPlan* plans, int n, const ConvertArgs* tab, const int* offs, int total_blocks,
                              hipStream_t s);

// Recording: while a recorder is active on the calling thread, launch_dslash,
// launch_blas and launch_convert append their plans instead of launching.
// The solver uses it to record one iteration per system and replay the
// recorded steps of all systems as batched launches.
enum StepKind { STEP_DSLASH = 0, STEP_BLAS = 1, STEP_CONVERT = 2 };
struct Step {
    int kind;
    DslashPlan d;
    BlasPlan b;
    ConvertPlan c;
};
struct Recorder {
    std::vector<Step> steps;
};
Recorder* active_recorder();
void set_recorder(Recorder* r);

// Canonical complex128 <-> internal layouts.
hipError_t launch_pack_spinor(int prec, const Geom& g, const void* canon, void* out, int nrhs, hipStream_t s);
hipError_t launch_unpack_spinor(int prec, const Geom& g, const void* in, void* canon, int nrhs, hipStream_t s);
// The twisted-mass pseudo-fermion force of full-lattice FP64 fields X and Wf
// (Z = gamma_5 Wf) into canonical F[mu][site][3][3]: F = scale * force
// (accumulate = 0) or F += scale * force.
hipError_t launch_tm_force(int recon, const Geom& g, const void* U, const void* X, const void* Wf, void* F,
                           double kappa, double scale, int accumulate, hipStream_t s);
hipError_t launch_pack_colour(int prec, const Geom& g, const void* canon, void* out, int nrhs, hipStream_t s);
hipError_t launch_unpack_colour(int prec, const Geom& g, const void* in, void* canon, int nrhs, hipStream_t s);
hipError_t launch_pack_gauge(int prec, int recon, const Geom& g, const void* canon, void* out, hipStream_t s);
// Re-encode an internal FP64/18 gauge field at another precision / recon.
hipError_t launch_convert_gauge(int prec, int recon, const Geom& g, const void* U64, int src_recon, void* out,
                                hipStream_t s);

// Fill memory with zero bytes through a kernel (graph-capture safe).
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);

// ---- persistent batched solver (persist.hip)
// Block routines a phase of the persistent kernel runs: the steps of the
// mixed-precision CGNR iteration with FP32/12 inner and FP64/18 outer hops on
// several right-hand sides (one wave per chunk of sites and right-hand side).
enum PRoutine {
    PR_HOP32_12_D0_NONE = 0,
    PR_HOP32_12_D0_NORM,
    PR_HOP32_12_D1_NONE,
    PR_HOP32_12_D1_NORM,
    PR_HOP64_18_D0_NONE,
    PR_HOP64_18_D0_NORM_LOW,
    PR_BLAS32_AXMY,
    PR_BLAS32_CG_XP,
    PR_CONV64_32_ACC,
    PR_NONE = -1,
};
constexpr int kPersistThreads = 256;   // block size of the persistent kernel
constexpr int kMaxPersistSteps = 32;

// One step of the batched iteration as a phase: its routine, the blocks of
// all systems (total along x, each system's range starting at offs[s]; gy
// along y), the per-system argument table, and the finalize of its
// reduction (nfin values, per-system FinArgs; 0: none).
struct PStep {
    int routine;
    int total;
    int gy;
    int nfin;
    int pred;  // the step's predicate (the same for every system)
    const void* tab;
    const int* offs;
    const FinArgs* fin;
};

struct PProgram {
    PStep step[kMaxPersistSteps];
    int nsteps;
    int nsys, nrhs;
    int ctl_stride;        // control block of system s, right-hand side r: ctl[s * ctl_stride + r]
    Ctl* ctl;
    int max_iter;          // iterations this launch may run
    int spin_limit;        // polls of a barrier word before the kernel gives up
    unsigned* bar;         // arrival slots [kMaxPersistBlocks], then release slots (zero before the launch)
    int* flag;             // [0] give-up request from the host, [1] a barrier gave up (zero before the launch)
};

// Largest grid of the persistent kernel (one arrival and one release slot each).
constexpr int kMaxPersistBlocks = 2048;

// Blocks the device keeps resident at once for the persistent kernel
// (hipErrorNotSupported without cooperative launch).
hipError_t persistent_grid(int* blocks);
// Cooperative launch of the persistent kernel on prog_dev (device memory).
hipError_t launch_batch_persistent(const PProgram* prog_dev, int blocks, hipStream_t s);
// Zero the nslots barrier slots at words and set the two flags after them to
// (give_up, 0), with a kernel (capturable without a memset node).
hipError_t launch_persist_reset(unsigned* words, int nslots, int give_up, hipStream_t s);

// Initialise control blocks on the device (every right-hand side from in;
// the short form: a plain or reliable-update solve without stagnation
// handling or outer steps).
hipError_t launch_ctl_init(Ctl* ctl, int nrhs, const CtlInit& in, hipStream_t s);
hipError_t launch_ctl_init(Ctl* ctl, int nrhs, double tol, double delta, int iter_limit, hipStream_t s);
// Multi-shift control blocks: ctl[i].sigma = shifts[i] - shifts[base],
// ms_index = i, ms_n = n, ms_base = base (after launch_ctl_init).
constexpr int kMaxShifts = 32;
struct ShiftList {
    double s[kMaxShifts];
};
hipError_t launch_ctl_init_shifts(Ctl* ctl, int n, int base, const ShiftList& shifts, hipStream_t s);
// Re-open the solves whose bit is set in mask (done = 0, status = 0) after a
// failed true-residual check or a fall back to FP32 storage (no_fallback:
// the reopened solves may not fall back again).
hipError_t launch_ctl_reopen(Ctl* ctl, int nrhs, unsigned mask, hipStream_t s, bool no_fallback = false);

}  // namespace lqcd
