// Host build of a CG iteration's scalar steps: one by one, each as a launch
// that a finished solve skips, and by ctl_step, which runs a step late together
// with the next one.  Compiled by the tests; not part of the library.
#include <cstring>

#include "solver_ctl.h"

using namespace lqcd;

namespace {

// Totals of iteration k.
struct It {
    double ww, rr, ru, zz;
};

void start(Ctl* c, double delta, double tol_inner, int limit, int stag_window, int max_stag)
{
    CtlInit in{};
    in.tol = 1e-3;
    in.delta = delta;
    in.tol_inner = tol_inner;
    in.iter_limit = limit;
    in.stag_window = stag_window;
    in.max_stag = max_stag;
    in.fallback_ok = max_stag > 0;
    *c = ctl_make(in);
    c->bb = 1.0;
    c->thresh = c->tol2;
    c->zz = 1.0;
    double rr0[6] = {1.0};
    if (delta > 0.0) finalize_totals(FIN_RR_INIT, c, rr0);
}

void one(Ctl* c, int fin, double v)
{
    if (c->done || (fin == FIN_RU_RR && !c->update)) return;
    const double t[6] = {v};
    finalize_totals(fin, c, t);
}

void step(Ctl* c, int pre, double pv, int fin, double v)
{
    const double p[6] = {pv}, t[6] = {v};
    ctl_step(c, pre, p, fin, t);
}

}  // namespace

extern "C" {

// n iterations either way; returns 0 when the control blocks agree after each
// and log[k] = xdo + 2 * done + 4 * updates so far, or k + 1 where they differ.
int compare(const double* tot, int n, double delta, double tol_inner, int limit, int stag_window, int max_stag, int* log)
{
    Ctl a, b;
    start(&a, delta, tol_inner, limit, stag_window, max_stag);
    start(&b, delta, tol_inner, limit, stag_window, max_stag);
    const bool mixed = delta > 0.0;
    for (int k = 0; k < n; ++k) {
        const It& t = reinterpret_cast<const It*>(tot)[k];
        one(&a, FIN_CG_ALPHA, t.ww);
        one(&a, FIN_CG_RR, t.rr);
        if (mixed) one(&a, FIN_RU_RR, t.ru);
        one(&a, FIN_CG_BETA, t.zz);
        step(&b, FIN_NONE, 0.0, FIN_CG_ALPHA, t.ww);
        if (mixed) {
            step(&b, FIN_NONE, 0.0, FIN_CG_RR, t.rr);
            step(&b, FIN_RU_RR, t.ru, FIN_CG_BETA, t.zz);
        } else {
            step(&b, FIN_CG_RR, t.rr, FIN_CG_BETA, t.zz);
        }
        log[k] = b.xdo + 2 * b.done + 4 * b.nupdates;
        if (b.xpend) return k + 1;
        Ctl x = a, y = b;
        x.xpend = y.xpend = x.xdo = y.xdo = 0;
        if (std::memcmp(&x, &y, sizeof x)) return k + 1;
    }
    return 0;
}

// The multi-shift steps of a family of n: every system's x takes alpha p in
// the iteration that ends it and in none after.  log[k * n + i] as above.
void family(const double* tot, int n, int base, int iters, const double* sigma, int* log)
{
    Ctl c[32];
    CtlInit in{};
    in.tol = 1e-3;
    in.iter_limit = 1000;
    for (int i = 0; i < n; ++i) {
        c[i] = ctl_make(in);
        c[i].sigma = sigma[i];
        c[i].ms_index = i;
        c[i].ms_n = n;
        c[i].ms_base = base;
    }
    const double one_[6] = {1.0};
    finalize_totals(FIN_MS_INIT, c + base, one_);
    for (int k = 0; k < iters; ++k) {
        const double w[6] = {0.0, tot[2 * k]}, r[6] = {tot[2 * k + 1]};
        ctl_step(c + base, FIN_NONE, w, FIN_MS_ALPHA, w);
        ctl_step(c + base, FIN_NONE, r, FIN_MS_BETA, r);
        for (int i = 0; i < n; ++i) log[k * n + i] = c[i].xdo + 2 * c[i].done;
    }
}
}
