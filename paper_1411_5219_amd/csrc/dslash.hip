// Host side of the Dslash launches: block order and shape, how right-hand sides
// share them, grid, and the finalize step of fused reductions.  The kernels are
// instantiated per storage precision in dslash64/32/16.hip.
#include "lqcd.h"
#include "lqcd_kernels.h"

namespace lqcd {

hipError_t launch_dslash_64(int recon, int split, bool lnt, bool next, bool dag, int red, const DslashLaunch& L,
                            dim3 grid, dim3 block, hipStream_t s);
hipError_t launch_dslash_32(int recon, int split, bool lnt, bool next, bool dag, int red, const DslashLaunch& L,
                            dim3 grid, dim3 block, hipStream_t s);
hipError_t launch_dslash_16(int recon, int split, bool lnt, bool next, bool dag, int red, const DslashLaunch& L,
                            dim3 grid, dim3 block, hipStream_t s);

hipError_t launch_stag_64(int recon, int red, bool lnt, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s);
hipError_t launch_stag_32(int recon, int red, bool lnt, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s);
hipError_t launch_stag_16(int recon, int red, bool lnt, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s);

hipError_t launch_rhs_64(int recon, int halves, bool dag, int red, const DslashLaunch& L, dim3 grid, dim3 block,
                         hipStream_t s);
hipError_t launch_rhs_32(int recon, int halves, bool dag, int red, const DslashLaunch& L, dim3 grid, dim3 block,
                         hipStream_t s);
hipError_t launch_rhs_16(int recon, int halves, bool dag, int red, const DslashLaunch& L, dim3 grid, dim3 block,
                         hipStream_t s);

static hipError_t launch_dslash_prec(const DslashPlan& p, const DslashLaunch& L, dim3 grid, hipStream_t s)
{
    if (p.kind == PLAN_STAG) {
        if (p.prec == 64) return launch_stag_64(p.recon, p.red, p.lnt, L, grid, p.block, s);
        if (p.prec == 32) return launch_stag_32(p.recon, p.red, p.lnt, L, grid, p.block, s);
        if (p.prec == 16) return launch_stag_16(p.recon, p.red, p.lnt, L, grid, p.block, s);
        return hipErrorInvalidValue;
    }
    if (p.split == 0) {
        if (p.prec == 64) return launch_rhs_64(p.recon, p.halves, p.dag, p.red, L, grid, p.block, s);
        if (p.prec == 32) return launch_rhs_32(p.recon, p.halves, p.dag, p.red, L, grid, p.block, s);
        if (p.prec == 16) return launch_rhs_16(p.recon, p.halves, p.dag, p.red, L, grid, p.block, s);
        return hipErrorInvalidValue;
    }
    if (p.prec == 64) return launch_dslash_64(p.recon, p.split, p.lnt, p.next, p.dag, p.red, L, grid, p.block, s);
    if (p.prec == 32) return launch_dslash_32(p.recon, p.split, p.lnt, p.next, p.dag, p.red, L, grid, p.block, s);
    if (p.prec == 16) return launch_dslash_16(p.recon, p.split, p.lnt, p.next, p.dag, p.red, L, grid, p.block, s);
    return hipErrorInvalidValue;
}

static ChunkGrid chunk_grid(const Geom& g) { return ChunkGrid{{g.L[0], g.L[1], g.L[2], g.L[3]}, g.Lxh, g.Vh}; }

// Block order and grid of a launch whose blocks cover at most maxsub chunks
// of 64 sites each, for `tile` right-hand sides per block.
static void plan_chunks(const Launch& cfg, int maxsub, int tile, bool adjacent, int nrhs, DslashPlan* p, int idle_max = 20)
{
    DslashArgs& a = p->a;
    a.swizzle = cfg.swizzle;
    a.nrhs = nrhs;
    a.ch = plan_chunk_order(chunk_grid(a.g), cfg.order, cfg.block, cfg.ygroup, maxsub, idle_max);
    p->slots = a.ch.nsp * (a.full ? 2 : 1);
    p->grid = dim3(plan_tiles(&a.ch, p->slots, tile, adjacent, nrhs));
    a.gx = (int)p->grid.x;
}

static hipError_t finish_plan(int red, DslashPlan* p)
{
    if (red != RED_NONE && p->slots > p->a.r.capacity) return hipErrorInvalidValue;  // partials too small
    p->nfin = red == RED_NONE || p->a.r.fin == FIN_NONE ? 0 : red == RED_NORM || red == RED_NORM_LOW ? 1 : red == RED_DOT_AUX ? 2 : 3;
    return hipSuccess;
}

static bool storage_built(int prec, int recon)
{
    return (prec == 64 && (recon == 18 || recon == 12)) || (prec == 32 && (recon == 18 || recon == 12)) ||
           (prec == 16 && recon == 12);
}

int hop_form(int prec, int recon, bool full, const Geom* g, int n, int nrhs, bool rare)
{
    std::vector<ChunkGrid> c;
    for (int i = 0; i < n; ++i) c.push_back(chunk_grid(g[i]));
    return hop_form(prec, recon, full, c.data(), n, nrhs, rare);
}

hipError_t plan_dslash(int prec, int recon, bool dagger, int red, const DslashArgs& args, int nrhs, const Launch& cfg,
                       DslashPlan* out)
{
    if (!storage_built(prec, recon)) return hipErrorInvalidValue;
    DslashPlan& p = *out;
    p.kind = PLAN_WILSON;
    p.prec = prec;
    p.recon = recon;
    p.dag = dagger;
    p.red = red;
    p.a = args;
    const ChunkGrid grid = chunk_grid(args.g);
    const int form = cfg.form != FORM_BY_SIZE ? cfg.form : hop_form(prec, recon, args.full != 0, &grid, 1, nrhs);
    const HopShape h = hop_shape(prec, recon, args.full != 0, grid, nrhs, form);
    p.split = h.split;
    p.halves = h.halves;
    p.lnt = h.lnt;
    p.next = h.next;
    Launch c = cfg;
    // half the group of blocks where a tile's spinors are twice as large or
    // both parities share the L2 (32^3x8, 4 right-hand sides: FP64 Schur 198 us
    // against 204, FP64 full 173 against 203, FP32/18 full 61 against 75; FP32
    // Schur, 12 right-hand sides, is faster in groups of 4: 206 us against 211;
    // one right-hand side, FP64/18 full 32^3x8 54.8 -> 50.4, 48^3x12 326 -> 319,
    // but FP32/12 48^3x12 136 us with whole groups, 138 with halves)
    if (h.split == 0 ? prec == 64 || args.full : prec == 64 && args.full) c.block = cfg.block / 2;
    if (h.memory && cfg.order == 1) c.order = 0;
    plan_chunks(c, h.split == 1 ? cfg.block / kChunk : 1, h.tile, h.next, nrhs, &p, h.idle);
    const int waves = h.split == 0 ? h.tile * h.halves : h.split == 2 ? 2 : p.a.ch.nsub;
    p.block = dim3((unsigned)(kChunk * waves));
    return finish_plan(red, &p);
}

hipError_t exec_dslash(const DslashPlan& p, hipStream_t s)
{
    DslashLaunch L{&p.a, nullptr, nullptr, 1};
    const hipError_t e = launch_dslash_prec(p, L, p.grid, s);
    if (e != hipSuccess || p.nfin == 0) return e;
    FinArgs fa = fin_args(p.a.r, p.slots, p.a.ctl, p.a.pred);
    const hipError_t f = launch_finalize(p.nfin, fa, p.a.nrhs, s);
    // both parities in one launch: the even-parity blocks hold the first half of the partials
    if (f != hipSuccess || !p.a.full || !p.a.r.fin_even) return f;
    fa.fin = p.a.r.fin_even;
    fa.pre_partials = nullptr;
    return launch_finalize(p.nfin, fa, p.a.nrhs, s, p.slots / 2);
}

hipError_t exec_dslash_batch(const DslashPlan* plans, int n, const DslashArgs* tab, const int* offs, int total_blocks,
                             const FinArgs* fin_tab, hipStream_t s)
{
    if (n < 1) return hipErrorInvalidValue;
    const DslashPlan& p0 = plans[0];
    unsigned bx = p0.block.x, gx = p0.grid.x;
    for (int i = 1; i < n; ++i) {
        gx = plans[i].grid.x > gx ? plans[i].grid.x : gx;
        bx = plans[i].block.x > bx ? plans[i].block.x : bx;
    }
    DslashPlan q = p0;
    q.block = dim3(bx);
    const BatchGrid bg = batch_grid(n, gx, 1, (unsigned)total_blocks, offs);
    DslashLaunch L{nullptr, tab, bg.offs, n};
    const hipError_t e = launch_dslash_prec(q, L, bg.grid, s);
    if (e != hipSuccess || p0.nfin == 0) return e;
    return launch_finalize_batch(p0.nfin, fin_tab, n, p0.a.nrhs, s);
}

// Very many right-hand sides (an application of the matrix, no reduction and no
// control blocks): several launches, each on at most n of them.
template <class F>
static hipError_t launch_parts(int red, DslashArgs a, int nrhs, int n, F launch)
{
    if (red != RED_NONE || a.ctl) return hipErrorInvalidValue;
    for (int k = 0; k < nrhs; k += n) {
        const hipError_t e = launch(a, nrhs - k < n ? nrhs - k : n);
        if (e != hipSuccess) return e;
        a.in = static_cast<const char*>(a.in) + n * a.st_in;
        a.out = static_cast<char*>(a.out) + n * a.st_out;
        if (a.site) a.site = static_cast<const char*>(a.site) + n * a.st_site;
        if (a.add) a.add = static_cast<const char*>(a.add) + n * a.st_add;
    }
    return hipSuccess;
}

hipError_t launch_dslash(int prec, int recon, bool dagger, int red, const DslashArgs& args, int nrhs,
                         const Launch& cfg, hipStream_t s)
{
    DslashPlan p;
    hipError_t e = plan_dslash(prec, recon, dagger, red, args, nrhs, cfg, &p);
    if (e != hipSuccess) return e;
    const int n = rhs_per_launch(p.slots, p.a.ch.tile, (int)p.block.x, nrhs);
    if (n < nrhs)
        return launch_parts(red, args, nrhs, n, [&](const DslashArgs& a, int m) {
            return launch_dslash(prec, recon, dagger, red, a, m, cfg, s);
        });
    if (Recorder* r = active_recorder()) {
        r->steps.push_back(Step{});
        r->steps.back().kind = STEP_DSLASH;
        r->steps.back().d = p;
        return hipSuccess;
    }
    return exec_dslash(p, s);
}

hipError_t plan_stag_hop(int prec, int recon, int red, const DslashArgs& args, int nrhs, const Launch& cfg,
                         DslashPlan* out)
{
    if (red != RED_NONE && red != RED_NORM && red != RED_NORM_DS) return hipErrorInvalidValue;
    if (!storage_built(prec, recon)) return hipErrorInvalidValue;
    DslashPlan& p = *out;
    p.kind = PLAN_STAG;
    p.prec = prec;
    p.recon = recon;
    p.dag = false;
    p.red = red;
    p.a = args;
    p.split = 1;
    p.halves = 1;
    p.next = false;
    p.lnt = nrhs == 1 && !args.full;
    plan_chunks(cfg, cfg.block / kChunk, 1, false, nrhs, &p);
    p.block = dim3((unsigned)(kChunk * p.a.ch.nsub));
    return finish_plan(red, &p);
}

hipError_t launch_stag(int prec, int recon, int red, const DslashArgs& args, int nrhs, const Launch& cfg,
                       hipStream_t s)
{
    DslashPlan p;
    hipError_t e = plan_stag_hop(prec, recon, red, args, nrhs, cfg, &p);
    if (e != hipSuccess) return e;
    const int n = rhs_per_launch(p.slots, 1, (int)p.block.x, nrhs);
    if (n < nrhs)
        return launch_parts(red, args, nrhs, n, [&](const DslashArgs& a, int m) {
            return launch_stag(prec, recon, red, a, m, cfg, s);
        });
    if (Recorder* r = active_recorder()) {
        r->steps.push_back(Step{});
        r->steps.back().kind = STEP_DSLASH;
        r->steps.back().d = p;
        return hipSuccess;
    }
    return exec_dslash(p, s);
}

}  // namespace lqcd
