// HMC entry points and the leapfrog trajectory driver (hybrid Monte Carlo, the gauge-field
// generation algorithm in the paper's list, after Duane et al.).  The driver sequences
// the library's own kernels: the gauge kick with the link update, the fermion solve and kick
// (the CG on M^H M, Y = M X, the link-wise force kernel), and the reductions that give H.
#include <chrono>
#include <cmath>
#include <string>

#include "cola.h"
#include "handle.h"
#include "hmc_stages.h"
#include "launch.h"

using namespace cola;

namespace {

hipStream_t hstream(void *s) { return (hipStream_t)s; }

size_t nlinks(const cola_handle_t *h) { return (size_t)8 * h->g.Vh; }

// device scalars of the trajectory: the parts of H at its start and end (the plaquette sum
// four times over)
enum Scalar { KIN0, RETR0, SF0, RETR1, SF1, KIN1, NSCALAR };

// device scratch of the trajectory: packed links (the step reads one and writes the other)
// and momenta, fermion vectors
struct HmcWork {
    void *U[2] = {nullptr, nullptr}, *P = nullptr;
    void *X = nullptr;                 // canonical spinor: the CG's solution and next guess
    void *Xp = nullptr, *Yp = nullptr; // packed FP64 full-lattice spinors
    double *sc = nullptr;              // NSCALAR device scalars
};

int scalars(cola_handle_t *h, double **sc) {
    void *p;
    COLA_TRY(get_vec(h, "hmc_sc", NSCALAR * sizeof(double), &p));
    *sc = (double *)p;
    return COLA_OK;
}

int work(cola_handle_t *h, bool fermions, HmcWork *w) {
    const size_t gb = (size_t)8 * 9 * 16 * h->g.S;
    COLA_TRY(get_vec(h, "links_w0", gb, &w->U[0]));
    COLA_TRY(get_vec(h, "links_w1", gb, &w->U[1]));
    COLA_TRY(get_vec(h, "hmc_P", gb, &w->P));
    COLA_TRY(scalars(h, &w->sc));
    if (!fermions) return COLA_OK;
    const size_t sb = (size_t)2 * h->g.Vh * 12 * 16;
    const size_t pb = cola_field_bytes(h, COLA_FP64, 1, -1);
    COLA_TRY(get_vec(h, "hmc_X", sb, &w->X));
    COLA_TRY(get_vec(h, "hmc_Xp", pb, &w->Xp));
    COLA_TRY(get_vec(h, "hmc_Yp", pb, &w->Yp));
    return COLA_OK;
}

double read_scalar(cola_handle_t *h, const double *d, hipStream_t st, int *rc) {
    double v = 0.0;
    hipError_t e = hipMemcpyAsync(&v, d, sizeof(double), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) *rc = hip_error(h, e, "hmc scalar read-back");
    return v;
}

// The fermion force at the links U (packed) kicks the momenta: P -= eps F_f; sf (device, may
// be null) receives S_f = Re <phi, X>.  X of the previous call is the CG's starting guess.
//
// Full lattice: X = (M^H M)^{-1} phi, Y = M X.  Even-odd pseudofermion
// S_f = phi_e^H (S^H S)^{-1} phi_e (plain Wilson): with X_e = (S^H S)^{-1} phi_e and
// Y_e = S X_e,
//   dS_f = 2 kappa^2 Re[Y_e^H dD_eo X_o + Y_o^H dD_oe X_e],  X_o = D_oe X_e, Y_o = D_eo^H Y_e,
// which is the full-lattice fermion force of (X_e, X_o) and (Y_e, Y_o) with kappa^2 in
// place of kappa.
int fermion_kick(cola_handle_t *h, const void *U, const void *phi, const cola_hmc_params_t *p,
                 HmcWork &w, bool first, double eps, double *sf, int *iters, int *status,
                 hipStream_t st) {
    COLA_TRY(set_links(h, U, true, st));
    cola_cg_params_t cp{};
    cp.system = p->eo ? COLA_SYS_SCHUR : COLA_SYS_MDAGM;
    cp.scheme = p->cg_scheme;
    cp.tol = p->cg_tol;
    cp.max_iter = p->cg_max_iter;
    cp.reliable_interval = 50;
    cp.use_x0 = first ? 0 : 1;
    double res = 0.0;
    cola_cg_result_t cr{};
    cr.true_rel_residual = &res;
    COLA_TRY(cola_cg_solve(h, w.X, phi, 1, &cp, &cr, st));  // even-odd: odd sites of X set to 0
    *iters += cr.iterations;
    if (cr.status != COLA_OK) *status = COLA_NOT_CONVERGED;
    COLA_TRY(cola_pack_spinor(h, w.Xp, w.X, COLA_FP64, 1, -1, st));
    if (p->eo) {
        const size_t blk = cola_field_bytes(h, COLA_FP64, 1, 0);
        char *xe = (char *)w.Xp, *xo = xe + blk, *ye = (char *)w.Yp, *yo = ye + blk;
        COLA_TRY(cola_dslash_apply(h, xo, xe, COLA_OP_HOP, 1, COLA_FP64, 1, st));
        COLA_TRY(cola_dslash_apply(h, ye, xe, COLA_OP_SCHUR, 0, COLA_FP64, 1, st));
        COLA_TRY(cola_dslash_apply(h, yo, ye, COLA_OP_HOP_DAG, 1, COLA_FP64, 1, st));
    } else {
        COLA_TRY(cola_dslash_apply(h, w.Yp, w.Xp, COLA_OP_M, -1, COLA_FP64, 1, st));
    }
    if (sf)
        COLA_HIP(h, launch_redot(phi, w.X, (size_t)2 * h->g.Vh * 12, h->partial, sf, st));
    COLA_HIP(h, launch_fermion_kick(h->g, U, w.Xp, w.Yp, w.P,
                                    p->eo ? h->kappa * h->kappa : h->kappa, h->phase, eps, st));
    return COLA_OK;
}

}  // namespace

int cola_gauge_force(cola_handle_t *h, void *F, const void *U, double beta, void *stream) {
    if (!h) return COLA_EINVAL;
    if (!F || !U) return set_error(h, COLA_EINVAL, "null pointer");
    COLA_HIP(h, launch_gauge_force(h->g, U, F, beta, hstream(stream)));
    return COLA_OK;
}

int cola_fermion_action(cola_handle_t *h, const void *phi, void *X, void *Y, double tol,
                        double *S, int *iterations, void *stream) {
    if (!h) return COLA_EINVAL;
    if (!phi || !X || !Y || !S) return set_error(h, COLA_EINVAL, "null pointer");
    if (!(tol > 0.0) || !std::isfinite(tol)) return set_error(h, COLA_EINVAL, "need tol > 0");
    if (h->csw != 0.0)
        return set_error(h, COLA_EINVAL, "the action's force exists for plain Wilson only");
    if (!h->gauge_set) return set_error(h, COLA_ESTATE, "no gauge field set");
    hipStream_t st = hstream(stream);
    void *Xp, *Yp;
    double *sc;
    const size_t pb = cola_field_bytes(h, COLA_FP64, 1, -1);
    COLA_TRY(get_vec(h, "fa_Xp", pb, &Xp));
    COLA_TRY(get_vec(h, "fa_Yp", pb, &Yp));
    COLA_TRY(scalars(h, &sc));
    // X = (M^H M)^{-1} phi from x = 0
    cola_cg_params_t cp{};
    cp.system = COLA_SYS_MDAGM;
    cp.scheme = COLA_CG_FP64;
    cp.tol = tol;
    cp.max_iter = 100000;
    cp.reliable_interval = 50;
    double res = 0.0;
    cola_cg_result_t cr{};
    cr.true_rel_residual = &res;
    COLA_TRY(cola_cg_solve(h, X, phi, 1, &cp, &cr, st));
    if (iterations) *iterations = cr.iterations;
    // Y = M X through the packed FP64 field; S = Re <phi, X>
    COLA_TRY(cola_pack_spinor(h, Xp, X, COLA_FP64, 1, -1, st));
    COLA_TRY(cola_dslash_apply(h, Yp, Xp, COLA_OP_M, -1, COLA_FP64, 1, st));
    COLA_TRY(cola_unpack_spinor(h, Y, Yp, COLA_FP64, 1, -1, st));
    COLA_HIP(h, launch_redot(phi, X, (size_t)2 * h->g.Vh * 12, h->partial, sc + 3, st));
    int rc = COLA_OK;
    *S = read_scalar(h, sc + 3, st, &rc);
    COLA_TRY(rc);
    return cr.status == COLA_OK ? COLA_OK : cr.status;
}

int cola_gauge_action(cola_handle_t *h, const void *U, double beta, double *S, void *stream) {
    if (!h) return COLA_EINVAL;
    if (!U || !S) return set_error(h, COLA_EINVAL, "null pointer");
    double *sc;
    COLA_TRY(scalars(h, &sc));
    hipStream_t st = hstream(stream);
    COLA_HIP(h, launch_plaquette_sum(h->g, U, h->partial, sc, st));
    int rc = COLA_OK;
    const double plaq = read_scalar(h, sc, st, &rc);
    COLA_TRY(rc);
    *S = beta * (6.0 * 2.0 * h->g.Vh - plaq / 3.0);
    return COLA_OK;
}

int cola_link_update(cola_handle_t *h, void *U, const void *P, double eps, void *stream) {
    if (!h) return COLA_EINVAL;
    if (!U || !P) return set_error(h, COLA_EINVAL, "null pointer");
    if (!std::isfinite(eps)) return set_error(h, COLA_EINVAL, "non-finite step");
    COLA_HIP(h, launch_link_update(U, P, eps, nlinks(h), hstream(stream)));
    return COLA_OK;
}

int cola_momentum_update(cola_handle_t *h, void *P, const void *F1, const void *F2, double eps,
                         void *stream) {
    if (!h) return COLA_EINVAL;
    if (!P || !F1) return set_error(h, COLA_EINVAL, "null pointer");
    COLA_HIP(h, launch_momentum_update(P, F1, F2, eps, nlinks(h), hstream(stream)));
    return COLA_OK;
}

int cola_hmc_trajectory(cola_handle_t *h, void *U, void *P, const void *phi,
                        const cola_hmc_params_t *p, cola_hmc_result_t *r, void *stream) {
    if (!h) return COLA_EINVAL;
    if (!U || !P || !p || !r) return set_error(h, COLA_EINVAL, "null pointer");
    if (p->nsteps < 1 || !(p->eps > 0.0) || !std::isfinite(p->eps) || !std::isfinite(p->beta))
        return set_error(h, COLA_EINVAL, "need nsteps >= 1, finite eps > 0 and finite beta");
    if (phi && h->csw != 0.0)
        return set_error(h, COLA_EINVAL, "fermion force of the clover term not available");
    if (h->flic)
        return set_error(h, COLA_EINVAL,
                         "the trajectory driver runs the Wilson operator (the FLIC force, "
                         "through the smearing, is not built)");
    if (phi && (!(p->cg_tol > 0.0) || p->cg_max_iter < 1))
        return set_error(h, COLA_EINVAL, "need cg_tol > 0 and cg_max_iter >= 1");
    if (phi && (p->cg_scheme < COLA_CG_FP64 || p->cg_scheme > COLA_CG_FP32_DEFECT))
        return set_error(h, COLA_EINVAL, "unknown cg_scheme");
    if (p->integrator < 0 || p->integrator > 2)
        return set_error(h, COLA_EINVAL,
                         "integrator must be 0 (leapfrog), 1 (Omelyan) or 2 (two time scales)");
    if (p->integrator == 2 && p->n_gauge < 1)
        return set_error(h, COLA_EINVAL, "n_gauge must be >= 1");
    hipStream_t st = hstream(stream);
    const auto t0 = std::chrono::steady_clock::now();
    HmcWork w;
    COLA_TRY(work(h, phi != nullptr, &w));
    *r = cola_hmc_result_t{};
    r->status = COLA_OK;
    int status = COLA_OK, iters = 0;

    // The trajectory runs on packed copies; the caller's fields receive its end.  The parts of
    // H are left on the device and read once, after the last launch.
    const size_t n = nlinks(h) * 9;
    COLA_HIP(h, launch_sqnorm(P, n, h->partial, w.sc + KIN0, st));
    COLA_HIP(h, launch_md_pack(h->g, U, P, w.U[0], w.P, st));
    const long long count = stage_count(*p);
    int cur = 0;
    for (long long k = 0; k < count; ++k) {
        const Stage s = stage_at(*p, k);
        const bool first = k == 0, last = k + 1 == count;
        if (phi && s.fermions)
            COLA_TRY(fermion_kick(h, w.U[cur], phi, p, w, first, s.eps_f,
                                  first  ? w.sc + SF0
                                  : last ? w.sc + SF1
                                         : nullptr,
                                  &iters, &status, st));
        COLA_HIP(h, launch_md_step(h->g, w.U[cur], last ? nullptr : w.U[1 - cur], w.P, p->beta,
                                   s.eps_g, s.eps_u, h->partial,
                                   first  ? w.sc + RETR0
                                   : last ? w.sc + RETR1
                                          : nullptr,
                                   st));
        if (!last) cur = 1 - cur;
    }
    COLA_HIP(h, launch_md_unpack(h->g, U, P, w.U[cur], w.P, st));
    COLA_HIP(h, launch_sqnorm(P, n, h->partial, w.sc + KIN1, st));
    double sc[NSCALAR];
    COLA_HIP(h, hipMemcpyAsync(sc, w.sc, sizeof sc, hipMemcpyDeviceToHost, st));
    COLA_HIP(h, hipStreamSynchronize(st));
    const auto gauge = [&](double retr) {
        return p->beta * (6.0 * 2.0 * h->g.Vh - 0.25 * retr / 3.0);
    };
    r->kinetic0 = 0.5 * sc[KIN0];
    r->kinetic1 = 0.5 * sc[KIN1];
    r->gauge0 = gauge(sc[RETR0]);
    r->gauge1 = gauge(sc[RETR1]);
    r->fermion0 = phi ? sc[SF0] : 0.0;
    r->fermion1 = phi ? sc[SF1] : 0.0;
    r->H0 = r->kinetic0 + r->gauge0 + r->fermion0;
    r->H1 = r->kinetic1 + r->gauge1 + r->fermion1;
    r->dH = r->H1 - r->H0;
    r->cg_iterations = iters;
    r->status = status;
    r->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return COLA_OK;
}
