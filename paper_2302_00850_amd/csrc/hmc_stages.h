// The stages of a trajectory's integrator, each computed from its place: no list is kept, so a
// trajectory of any length takes no host memory for it.
#pragma once

#include "../../include/cola.h"

namespace cola {

// One stage at the current links: the fermion kick (if any), then the gauge kick and, unless
// it is the last stage, the link update.
struct Stage {
    bool fermions;
    double eps_f, eps_g, eps_u;
};

inline long long stage_count(const cola_hmc_params_t &p) {
    const long long n = p.nsteps;
    return p.integrator == 0 ? n + 1 : p.integrator == 1 ? 2 * n + 1 : n * p.n_gauge + 1;
}

inline Stage stage_at(const cola_hmc_params_t &p, long long k) {
    const double eps = p.eps;
    const bool end = k == 0 || k == stage_count(p) - 1;
    if (p.integrator == 0) {
        // leapfrog: P eps/2, then per step U eps and P eps (eps/2 after the last)
        const double e = end ? 0.5 * eps : eps;
        return {true, e, e, eps};
    }
    if (p.integrator == 1) {
        // Omelyan: P lambda eps, then per step U eps/2, P (1 - 2 lambda) eps, U eps/2 and
        // P 2 lambda eps (the next step's first momentum step merged; lambda eps after the
        // last)
        const double lam = 0.1931833275037836;
        const double e = (k % 2 ? 1.0 - 2.0 * lam : end ? lam : 2.0 * lam) * eps;
        return {true, e, e, 0.5 * eps};
    }
    // two time scales: fermion kicks of eps around n_gauge gauge leapfrog sub-steps of
    // eps / n_gauge; the half gauge kicks that end one step and start the next are one
    const double hs = eps / p.n_gauge;
    if (k % p.n_gauge) return {false, 0.0, hs, hs};
    return {true, end ? 0.5 * eps : eps, end ? 0.5 * hs : hs, hs};
}

}  // namespace cola
