// Conjugate-gradient solvers on the normal operator (M^H M on the full lattice
// or S^H S on even sites), built from the hop and site kernels.
//
// All right-hand sides advance in lockstep (one batched hop per operator
// factor).  Per-rhs scalars (rho, pi, alpha, beta) live on the device; the
// host reads the residual norms back every `check_interval` iterations only.
//
// Schemes (the paper's benchmark is a mixed-precision solver with 32-bit
// inner iterations and a 64-bit outer solver):
//   FP64          plain CG; when the iterated residual meets tol the true
//                 residual b - A x is recomputed and CG continues from it if
//                 needed.
//   FP32_RELIABLE FP32 CG (FP32 vectors, 12-real FP32 links) with an FP64
//                 solution accumulator: every reliable_interval iterations
//                 (and when the iterated residual meets tol) x64 += x32,
//                 r = b - A64 x64 in FP64, and the FP32 residual is replaced;
//                 the search direction is kept.
//   FP16/FP32_DEFECT  FP64 defect correction: R = B - A64 X, inner CG on
//                 A E = R/|R| in FP16 storage (FP32 arithmetic) or FP32 down
//                 to inner_tol, X += |R| E.  Three cycles that contract the
//                 residual by less than 2x switch an FP16 inner solve to FP32.
#include <algorithm>
#include <chrono>
#include <cstddef>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "handle.h"

namespace cola {

namespace {

enum Slot {
    RHO = 0,
    RHO_NEW = 1,
    PI = 2,
    BNORM = 3,
    SCALE = 4,
    TRUE_RES = 5,
    TMP = 6
};

struct Ctx {
    cola_handle_t *h;
    hipStream_t st;
    int R;
    int full;  // 1: M^H M on the full lattice (2 blocks), 0: S^H S on even sites
    int nblk() const { return full ? 2 : 1; }
    size_t bytes(SpinorFmt f) const { return spinor_block_bytes(h->g, f, R) * nblk(); }
    BlasShape shape() const { return blas_shape(h->g, R, nblk()); }
    // RHO and RHO_NEW trade places each iteration (rotate_rho)
    mutable int flip = 0;
    // x += alpha p of the last step is still to be done (with the update of p, or finish_x)
    mutable bool x_due = false;
    int place(int s) const { return s <= RHO_NEW ? s ^ flip : s; }
    double *slot(int s) const { return scal_slot(h, place(s)); }
    // RHO_NEW and PI of one rhs may still be partial sums (count > 0), which the kernels that
    // follow add; keep: steps may leave them so.  slot() and reduce() are for whole
    // scalars: after settle(), or to write one (fresh()).
    mutable int parts[3] = {0, 0, 0};
    mutable double *part_buf = nullptr;  // 3 x kSumMax
    mutable bool keep = false;
    Sum sum(int s) const {
        const int n = parts[place(s)];
        return n > 0 ? Sum{part_buf + place(s) * kSumMax, n} : Sum{slot(s), 0};
    }
    NormTo norm_to(int s) const {
        return {slot(s), keep ? part_buf + place(s) * kSumMax : nullptr, &parts[place(s)]};
    }
    double *fresh(int s) const {
        if (s <= PI) parts[place(s)] = 0;
        return slot(s);
    }
    Reduce reduce(int s) const {
        fresh(s);
        return reduce_into(h, place(s));
    }
};

// Iterations between host convergence checks when the caller leaves it to the library.
// A check reads the residual norms back and waits for them (some 10-20 us during which
// the device idles), and the solve stops only at a check, overshooting by up to
// check - 1 iterations.  Where an iteration moves at least 2^20 site-rhs through the
// operator (a millisecond or more) the wait costs under 2% and every iteration is
// checked; smaller solves check every `small` iterations.
int default_check(const Ctx &c, int small) {
    const double work = (double)c.h->g.Vh * c.R * c.nblk();
    return work >= 1048576.0 ? 1 : small;
}

int vec(const Ctx &c, const char *tag, SpinorFmt f, void **out) {
    std::string t = std::string("cg_") + tag + "_" + std::to_string((int)f) + "_" +
                    std::to_string(c.R) + "_" + std::to_string(c.full);
    return get_vec(c.h, t, c.bytes(f), out);
}

// add the partial sums that RHO, RHO_NEW or PI still is
int settle(const Ctx &c, int s) {
    const Sum v = c.sum(s);
    if (v.n > 0) COLA_HIP(c.h, launch_reduce_partials(v.v, v.n, 1, c.fresh(s), c.st));
    return COLA_OK;
}

// steps of this solve may leave partial sums (one rhs)
int keep_sums(const Ctx &c, bool on) {
    c.keep = on && c.R == 1;
    if (!c.keep) return COLA_OK;
    void *v;
    COLA_TRY(get_vec(c.h, "cg_parts", 3 * kSumMax * sizeof(double), &v));
    c.part_buf = (double *)v;
    return COLA_OK;
}

// out = A in, |first factor output|^2 -> PI
int normal(const Ctx &c, int prec, void *out, const void *in) {
    if (!c.full)
        return apply_op(c.h, out, in, COLA_OP_SCHUR_DAGSCHUR, 0, prec, c.R, c.st, c.fresh(PI));
    cola_handle_t *h = c.h;
    const SpinorFmt sf = spinor_fmt(prec);
    void *t;
    COLA_TRY(get_vec(h, "cg_full_t_" + std::to_string((int)sf) + "_" + std::to_string(c.R),
                     c.bytes(sf), &t));
    COLA_TRY(apply_op(h, t, in, COLA_OP_M, -1, prec, c.R, c.st, c.fresh(PI)));
    return apply_op(h, out, t, COLA_OP_MDAG, -1, prec, c.R, c.st);
}

// One CG step: Ap = A p, pi = <p, Ap>, then r -= alpha Ap and rho_new = |r|^2, and
// x += alpha p.  With x, r and p in the operator's storage r is updated inside the last hop
// (Ap is never stored; the last hop of S^dag S on the even-odd system, the hop of M^dag on
// the full lattice) and x together with p, which is then read once for both;
// COLA_CG_FUSE=0 selects a separate update kernel of x and r.
int full_normal_cg_step(const Ctx &c, int prec, void *r, void *pv, const double *rho,
                        const NormTo &rho_new) {
    cola_handle_t *h = c.h;
    const SpinorFmt sf = spinor_fmt(prec);
    void *t;
    COLA_TRY(get_vec(h, "cg_full_t_" + std::to_string((int)sf) + "_" + std::to_string(c.R),
                     c.bytes(sf), &t));
    const bool clover = h->csw != 0.0;
    const NormTo pi = c.norm_to(PI);
    COLA_TRY(apply_op(h, t, pv, COLA_OP_M, -1, prec, c.R, c.st, nullptr, nullptr, &pi));
    // M^dag t with the update of r, both parities in one launch
    HopCall hc{r, t, 0, 1};
    hc.both = true;
    hc.epi = clover ? EPI_CLOV_XPAY_CG : EPI_XPAY_CG;
    hc.x = t;
    hc.a = -h->kappa;
    hc.clov = sf == SpinorFmt::F64 ? h->clov64 : h->clov32;
    hc.norm_result = rho_new.result;
    hc.norm_partial = rho_new.partial;
    hc.norm_n = rho_new.n;
    hc.cg_r = r;
    hc.cg_rho = rho;
    const Sum ps = c.sum(PI);
    hc.cg_pi = ps.v;
    hc.cg_pi_n = ps.n;
    hc.cg_active = h->active;
    return hop(h, hc, prec, c.R, c.st);
}

int cg_step(const Ctx &c, int prec, SpinorFmt fx, void *x, void *r, void *pv, void *ap) {
    cola_handle_t *h = c.h;
    const SpinorFmt fp = spinor_fmt(prec);
    const char *env = getenv("COLA_CG_FUSE");
    const bool fuse = fx == fp && !(env && env[0] == '0');
    c.x_due = fuse;
    if (fuse && c.full)
        return full_normal_cg_step(c, prec, r, pv, c.slot(RHO), c.norm_to(RHO_NEW));
    if (fuse)
        return schur_normal_cg_step(h, prec, c.R, c.st, r, pv, c.slot(RHO), c.norm_to(PI),
                                    h->active, c.norm_to(RHO_NEW));
    COLA_TRY(normal(c, prec, ap, pv));
    COLA_HIP(h, launch_cg_xr(c.shape(), fx, fp, fx, fp, x, pv, r, ap, c.slot(RHO), c.slot(PI),
                             h->active, c.reduce(RHO_NEW), c.st));
    return COLA_OK;
}

// r = b - A x in FP64 (x may be all zero); |r|^2 -> slot
int true_residual(const Ctx &c, void *r, const void *b, const void *x, int slot) {
    void *ax;
    COLA_TRY(vec(c, "ax64", SpinorFmt::F64, &ax));
    COLA_TRY(normal(c, COLA_FP64, ax, x));
    const Reduce red = reduce_into(c.h, slot);
    COLA_HIP(c.h, launch_residual(c.shape(), r, b, ax, red, c.st));
    return COLA_OK;
}

// The starting residual: b - A x, or b itself (and |b|^2, already in BNORM) when the
// solve starts from x = 0, which saves the four FP64 hops of the normal operator.
int initial_residual(const Ctx &c, void *r, const void *b, const void *x, bool x_zero) {
    if (!x_zero) return true_residual(c, r, b, x, TRUE_RES);
    COLA_HIP(c.h, hipMemcpyAsync(r, b, c.bytes(SpinorFmt::F64), hipMemcpyDeviceToDevice, c.st));
    COLA_HIP(c.h, hipMemcpyAsync(c.slot(TRUE_RES), c.slot(BNORM), sizeof(double) * c.R,
                                 hipMemcpyDeviceToDevice, c.st));
    return COLA_OK;
}

int read_slot(const Ctx &c, int slot, double *out) {
    if (slot <= PI) COLA_TRY(settle(c, slot));
    COLA_HIP(c.h, hipMemcpyAsync(out, c.slot(slot), sizeof(double) * c.R, hipMemcpyDeviceToHost,
                                 c.st));
    COLA_HIP(c.h, hipStreamSynchronize(c.st));
    return COLA_OK;
}

int write_active(const Ctx &c, const std::vector<int> &act) {
    memcpy(c.h->host_active, act.data(), sizeof(int) * c.R);
    COLA_HIP(c.h, hipMemcpyAsync(c.h->active, c.h->host_active, sizeof(int) * c.R,
                                 hipMemcpyHostToDevice, c.st));
    COLA_HIP(c.h, hipStreamSynchronize(c.st));  // the pinned staging area is reused
    return COLA_OK;
}

int write_slot(const Ctx &c, int slot, const std::vector<double> &v) {
    std::vector<double> tmp(v);
    COLA_HIP(c.h, hipMemcpyAsync(c.slot(slot), tmp.data(), sizeof(double) * c.R,
                                 hipMemcpyHostToDevice, c.st));
    COLA_HIP(c.h, hipStreamSynchronize(c.st));
    return COLA_OK;
}

bool finite_all(const double *v, int n) {
    for (int i = 0; i < n; ++i)
        if (!std::isfinite(v[i])) return false;
    return true;
}

// the new |r|^2 becomes the old one: the slots trade places (a copy in a launch of its own
// took 4.5 us of a 16^3 x 32 iteration's 90)
void rotate_rho(const Ctx &c) { c.flip ^= 1; }

// p = r + beta p, with the x update that is due; the new |r|^2 becomes the old one
int update_p(const Ctx &c, SpinorFmt f, void *x, const void *r, void *p) {
    COLA_HIP(c.h, launch_cg_xp(c.shape(), f, c.x_due ? x : nullptr, r, p, c.sum(RHO_NEW),
                               c.slot(RHO), c.x_due ? c.sum(PI) : Sum{c.slot(PI), 0},
                               c.h->active, c.slot(RHO_NEW), c.st));
    c.fresh(RHO_NEW);  // whole now
    c.x_due = false;
    rotate_rho(c);
    return COLA_OK;
}

// The x update that is due, without p: before x is read and before the active columns change.
int finish_x(const Ctx &c, SpinorFmt f, void *x, void *p) {
    if (c.x_due)
        COLA_HIP(c.h, launch_cg_xp(c.shape(), f, x, nullptr, p, Sum{c.slot(RHO_NEW), 0},
                                   c.slot(RHO), c.sum(PI), c.h->active, nullptr, c.st));
    c.x_due = false;
    return COLA_OK;
}

// x64 += x (the sloppy solution, with the x update that is due), x = 0
int fold_x(const Ctx &c, SpinorFmt f, void *x64, void *x, const void *p) {
    if (c.x_due) COLA_TRY(settle(c, PI));
    COLA_HIP(c.h, launch_accum(c.shape(), f, x64, x, nullptr, 1, c.st, c.x_due ? p : nullptr,
                               c.slot(RHO), c.slot(PI), c.h->active));
    c.x_due = false;
    return COLA_OK;
}

struct Outcome {
    int status = COLA_OK;
    int iterations = 0;
    int outer = 0;
    int reliable = 0;
    std::vector<double> final_tr;  // true |r|^2 of the returned x, when the solver has it
};

// ---------------------------------------------------------------- iteration blocks

// Small solves are bound by launch latency (an FP32 iteration at 16^3 x 32 is six dependent
// launches of 9 to 12 us), so with COLA_GRAPHS=1 the n iterations between two convergence
// checks -- (step, p update) x (n - 1), step -- are captured once as a HIP
// graph and replayed (large solves check every iteration and launch directly).  Capture
// needs every launch shape settled (the first block of a solve runs directly, which
// tunes) and no per-launch timing.  Off by default: solves at 16^3 x 32 took 9 to 14% longer
// with replays (FP32 with reliable updates 6.02 and 6.88 ms) and at 8^3 x 16 8 to 26%; replays
// add their partial sums in launches of their own.
bool graphs_wanted(const Ctx &c) {
    const char *env = getenv("COLA_GRAPHS");
    if (!env || env[0] != '1') return false;
    if ((c.h->flags & COLA_FLAG_TIMING) || c.h->tune_mode == 2) return false;
    return (double)c.h->g.Vh * c.R * c.nblk() < 1048576.0;
}

int cg_block(const Ctx &c, int prec, SpinorFmt fx, void *x, void *r, void *pv, void *ap, int n,
             bool graph) {
    cola_handle_t *h = c.h;
    auto body = [&](const Ctx &cc) -> int {
        for (int k = 0; k < n; ++k) {
            COLA_TRY(cg_step(cc, prec, fx, x, r, pv, ap));
            if (k + 1 < n) COLA_TRY(update_p(cc, fx, x, r, pv));
        }
        return COLA_OK;
    };
    if (!graph || n < 2) return body(c);
    if (!h->gstream) {
        COLA_HIP(h, hipStreamCreateWithFlags(&h->gstream, hipStreamNonBlocking));
        COLA_HIP(h, hipEventCreateWithFlags(&h->gevent, hipEventDisableTiming));
    }
    // everything the captured launches hold: vectors, fields, operator, shape
    char key[512];
    const char *fuse = getenv("COLA_CG_FUSE");
    snprintf(key, sizeof key, "%d %d %d %d %d %d %p %p %p %p %p %p %p %p %p %p %p %p %p %p %p %p %d %c",
             prec, (int)fx, c.R, c.full, n, c.flip, x, r, pv, ap, h->gauge[0], h->gauge[1], h->gauge[2],
             h->gauge[3], h->fat[0], h->fat[1], h->fat[2], h->fat[3], h->clov32, h->clov64,
             h->clovinv32, h->clovinv64, h->flic ? 1 : 0, fuse ? fuse[0] : '-');
    hipGraphExec_t exec;
    auto it = h->graphs.find(key);
    if (it != h->graphs.end()) {
        exec = it->second;
    } else {
        Ctx cg = c;
        cg.st = h->gstream;
        COLA_HIP(h, hipStreamBeginCapture(h->gstream, hipStreamCaptureModeRelaxed));
        const int rc = body(cg);
        hipGraph_t graph = nullptr;
        const hipError_t ec = hipStreamEndCapture(h->gstream, &graph);
        if (rc != COLA_OK) {
            if (graph) hipGraphDestroy(graph);
            return rc;
        }
        COLA_HIP(h, ec);
        const hipError_t ei = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        hipGraphDestroy(graph);
        COLA_HIP(h, ei);
        h->graphs[key] = exec;
    }
    // ordered after the caller's stream, and the caller's stream after it
    COLA_HIP(h, hipEventRecord(h->gevent, c.st));
    COLA_HIP(h, hipStreamWaitEvent(h->gstream, h->gevent, 0));
    COLA_HIP(h, hipGraphLaunch(exec, h->gstream));
    COLA_HIP(h, hipEventRecord(h->gevent, h->gstream));
    COLA_HIP(h, hipStreamWaitEvent(c.st, h->gevent, 0));
    c.flip ^= (n - 1) & 1;
    c.x_due = !(fuse && fuse[0] == '0');
    return COLA_OK;
}

}  // namespace

void graphs_clear(cola_handle_t *h) {
    for (auto &kv : h->graphs) hipGraphExecDestroy(kv.second);
    h->graphs.clear();
}

namespace {

// ---------------------------------------------------------------- FP64 / FP32 reliable

int solve_reliable(const Ctx &c, int sloppy_prec, const cola_cg_params_t &p, void *x64,
                   const void *b64, const std::vector<double> &thr, Outcome *o) {
    const bool x_zero = !p.use_x0;
    cola_handle_t *h = c.h;
    const BlasShape sh = c.shape();
    const SpinorFmt fs = spinor_fmt(sloppy_prec);
    const bool same = fs == SpinorFmt::F64;
    const int check = p.check_interval > 0 ? p.check_interval : default_check(c, same ? 8 : 5);
    const int interval = same ? (1 << 30) : std::max(1, p.reliable_interval);
    // also update once the iterated residual has fallen by delta since the last
    // update (Clark et al.): a sloppy residual far below the true one would make
    // beta = rho_true / rho_iter huge and leave p pointing the stale way
    const double delta2 = 1e-2;
    void *r64, *xs, *rs, *ps, *aps;
    COLA_TRY(vec(c, "r64", SpinorFmt::F64, &r64));
    COLA_TRY(vec(c, "ps", fs, &ps));
    COLA_TRY(vec(c, "aps", fs, &aps));
    if (same) {
        xs = x64;
        rs = r64;
    } else {
        COLA_TRY(vec(c, "xs", fs, &xs));
        COLA_TRY(vec(c, "rs", fs, &rs));
        COLA_HIP(h, hipMemsetAsync(xs, 0, c.bytes(fs), c.st));
    }
    // r = b - A x0, rho = |r|^2
    COLA_TRY(initial_residual(c, r64, b64, x64, x_zero));
    std::vector<double> rho(c.R), tr(c.R);
    COLA_TRY(read_slot(c, TRUE_RES, tr.data()));
    if (!finite_all(tr.data(), c.R)) {
        o->status = COLA_BREAKDOWN;
        return COLA_OK;
    }
    std::vector<int> act(c.R);
    std::vector<double> ref(tr);  // true |r|^2 at the last reliable update
    bool all_done = true;
    for (int q = 0; q < c.R; ++q) {
        act[q] = tr[q] > thr[q];
        all_done &= !act[q];
    }
    if (all_done) {
        o->final_tr = tr;
        return COLA_OK;
    }
    COLA_TRY(write_active(c, act));
    const Reduce red_rho = c.reduce(RHO);
    if (!same) COLA_HIP(h, launch_convert(sh, fs, SpinorFmt::F64, rs, r64, nullptr, 0, &red_rho, c.st));
    else COLA_HIP(h, hipMemcpyAsync(c.fresh(RHO), c.slot(TRUE_RES), sizeof(double) * c.R, hipMemcpyDeviceToDevice, c.st));
    COLA_HIP(h, launch_convert(sh, fs, fs, ps, rs, nullptr, 0, nullptr, c.st));
    int last_rel = 0;
    int it = 0;
    const bool graphs = graphs_wanted(c);
    COLA_TRY(keep_sums(c, !graphs));  // replays would need the counts
    while (it < p.max_iter) {
        // the iterations up to the next check (it % check == 0 or the cap)
        const int n = std::min(check - it % check, p.max_iter - it);
        COLA_TRY(cg_block(c, sloppy_prec, fs, xs, rs, ps, aps, n, graphs && it > 0));
        it += n;
        bool stop = false;
        {
            COLA_TRY(read_slot(c, RHO_NEW, rho.data()));
            if (!finite_all(rho.data(), c.R)) {
                o->status = COLA_BREAKDOWN;
                break;
            }
            bool iter_conv = true, dropped = false;
            for (int q = 0; q < c.R; ++q) {
                iter_conv &= !act[q] || rho[q] <= thr[q];
                dropped |= act[q] && rho[q] < delta2 * ref[q];
            }
            if (iter_conv || dropped || it - last_rel >= interval || it == p.max_iter) {
                if (same)
                    COLA_TRY(finish_x(c, fs, xs, ps));
                else
                    COLA_TRY(fold_x(c, fs, x64, xs, ps));
                COLA_TRY(true_residual(c, r64, b64, x64, TRUE_RES));
                COLA_TRY(read_slot(c, TRUE_RES, tr.data()));
                ++o->reliable;
                last_rel = it;
                bool done = true, restart = false;
                std::vector<int> keep(c.R);
                for (int q = 0; q < c.R; ++q) {
                    act[q] = tr[q] > thr[q];
                    done &= !act[q];
                    ref[q] = tr[q];
                    // true residual far above the iterated one: restart p = r
                    keep[q] = act[q] && !(tr[q] > 1e4 * rho[q]);
                    restart |= act[q] && !keep[q];
                }
                if (done) {
                    stop = true;
                    o->final_tr = tr;  // x64 holds the whole solution (xs was folded in)
                } else {
                    const Reduce red_new = c.reduce(RHO_NEW);
                    if (!same)
                        COLA_HIP(h, launch_convert(sh, fs, SpinorFmt::F64, rs, r64, nullptr, 0,
                                                   &red_new, c.st));
                    else
                        COLA_HIP(h, hipMemcpyAsync(c.fresh(RHO_NEW), c.slot(TRUE_RES),
                                                   sizeof(double) * c.R, hipMemcpyDeviceToDevice,
                                                   c.st));
                    if (restart) {
                        // beta = 0 for the restarted columns: p = r
                        COLA_TRY(write_active(c, keep));
                        COLA_TRY(update_p(c, fs, xs, rs, ps));
                        COLA_TRY(write_active(c, act));
                        continue;
                    }
                    COLA_TRY(write_active(c, act));
                }
            }
        }
        if (stop) break;
        COLA_TRY(update_p(c, fs, xs, rs, ps));
    }
    if (same) {
        COLA_TRY(finish_x(c, fs, xs, ps));
    } else if (o->status == COLA_OK) {
        // fold any remaining sloppy solution in (no-op after a final reliable update)
        COLA_TRY(fold_x(c, fs, x64, xs, ps));
    }
    c.x_due = false;
    o->iterations += it;
    if (o->status == COLA_OK && it >= p.max_iter) {
        COLA_TRY(true_residual(c, r64, b64, x64, TRUE_RES));
        COLA_TRY(read_slot(c, TRUE_RES, tr.data()));
        for (int q = 0; q < c.R; ++q)
            if (tr[q] > thr[q]) o->status = COLA_NOT_CONVERGED;
        o->final_tr = tr;
    }
    return COLA_OK;
}

// ---------------------------------------------------------------- defect correction

// CG iterations on the normal system in precision prec (all vectors in that storage, FP32
// arithmetic throughout).
int inner_cg(const Ctx &c, int prec, void *x, void *r, void *pv, void *ap,
             const std::vector<double> &inner_tol2, int max_it, std::vector<int> act, int check,
             int *iters, int *status) {
    const SpinorFmt f = spinor_fmt(prec);
    COLA_TRY(write_active(c, act));
    std::vector<double> rho(c.R);
    int it = 0;
    const bool graphs = graphs_wanted(c);
    COLA_TRY(keep_sums(c, !graphs));  // replays would need the counts
    while (it < max_it) {
        // the iterations up to the next check
        const int n = std::min(check - it % check, max_it - it);
        COLA_TRY(cg_block(c, prec, f, x, r, pv, ap, n, graphs && it > 0));
        it += n;
        if (it % check == 0) {
            COLA_TRY(read_slot(c, RHO_NEW, rho.data()));
            if (!finite_all(rho.data(), c.R)) {
                *status = COLA_BREAKDOWN;
                break;
            }
            bool any = false, change = false;
            for (int q = 0; q < c.R; ++q) {
                if (act[q] && rho[q] <= inner_tol2[q]) {
                    act[q] = 0;
                    change = true;
                }
                any |= act[q] != 0;
            }
            if (!any) break;
            if (change) {
                COLA_TRY(finish_x(c, f, x, pv));
                COLA_TRY(write_active(c, act));
            }
        }
        COLA_TRY(update_p(c, f, x, r, pv));
    }
    COLA_TRY(finish_x(c, f, x, pv));
    *iters = it;
    return COLA_OK;
}

// ---------------------------------------------------------------- block CG

// O'Leary block CG on A E = R (R given in r32, E accumulated in x32), all active
// columns sharing one Krylov space, A = S^H S on the even sites:
//   T = S P, Q = S^H T; alpha = (T^H T)^-1 (R^H R); E += P alpha; R -= Q alpha;
//   beta = (R^H R)_old^-1 (R^H R)_new; P = R + P beta.
// P^H Q is taken as T^H T (the same matrix, Hermitian positive semi-definite by
// construction, and one field read instead of two).  The Gram matrices and the two small
// Hermitian solves (Cholesky with deflation of dependent directions, block_solve_kernel)
// stay on the device; R^H R comes out of the update kernel itself.  The host reads the
// diagonal of R^H R every `check` iterations to stop once every active column's
// |R_q|^2 <= inner_tol2 (the columns start at 1).
int inner_block_cg(const Ctx &c, int prec, void *x32, void *r32,
                   const std::vector<double> &inner_tol2, int max_it, std::vector<int> act,
                   int check, int *iters, int *status) {
    cola_handle_t *h = c.h;
    const int n = c.R;
    const SpinorFmt fp = spinor_fmt(prec);
    const SpinorFmt fx = SpinorFmt::F32;
    const int S = h->g.S;
    void *P, *Pn, *Q, *T, *mats;
    COLA_TRY(vec(c, "bP", fp, &P));
    COLA_TRY(vec(c, "bPn", fp, &Pn));
    COLA_TRY(vec(c, "bQ", fp, &Q));
    COLA_TRY(vec(c, "bT", fp, &T));
    // five n x n complex matrices: T^H T, R^H R (two, alternating), alpha, beta
    const size_t mat = (size_t)2 * kMaxRhs * kMaxRhs;
    COLA_TRY(get_vec(h, "block_mats", sizeof(double) * 5 * mat, &mats));
    double *Gpi = (double *)mats, *Grho[2] = {Gpi + mat, Gpi + 2 * mat}, *alpha = Gpi + 3 * mat,
           *beta = Gpi + 4 * mat;
    std::vector<double> host(2 * (size_t)n * n);
    unsigned mask_bits = 0;
    // inactive columns take no part: zero their residual so they stay at E = 0
    std::vector<double> mask(n);
    for (int q = 0; q < n; ++q) {
        mask[q] = act[q] ? 1.0 : 0.0;
        if (act[q]) mask_bits |= 1u << q;
    }
    COLA_TRY(write_slot(c, TMP, mask));
    const BlasShape sh = c.shape();
    COLA_HIP(h, launch_convert(sh, fx, fx, r32, r32, c.slot(TMP), 0, nullptr, c.st));
    COLA_HIP(h, launch_convert(sh, fp, fx, P, r32, nullptr, 0, nullptr, c.st));
    auto red = [&](double *out) { return Reduce{h->partial, h->counter, out}; };
    int cur = 0;
    COLA_HIP(h, launch_gram(S, n, h->num_cu, fx, fx, r32, r32, red(Grho[cur]), c.st));
    int it = 0;
    while (it < max_it) {
        COLA_TRY(apply_op(h, T, P, COLA_OP_SCHUR, 0, prec, n, c.st));
        COLA_HIP(h, launch_gram(S, n, h->num_cu, fp, fp, T, T, red(Gpi), c.st));
        COLA_TRY(apply_op(h, Q, T, COLA_OP_SCHUR_DAG, 0, prec, n, c.st));
        COLA_HIP(h, launch_block_solve(Gpi, Grho[cur], mask_bits, n, alpha, c.st));
        const Reduce rr = red(Grho[1 - cur]);
        COLA_HIP(h, launch_block_axpy(S, n, h->num_cu, fx, fp, x32, P, r32, Q, alpha, &rr,
                                      c.st));
        ++it;
        if (it % check == 0 || it == max_it) {
            COLA_HIP(h, hipMemcpyAsync(host.data(), Grho[1 - cur], sizeof(double) * host.size(),
                                       hipMemcpyDeviceToHost, c.st));
            COLA_HIP(h, hipStreamSynchronize(c.st));
            bool any = false, bad = false;
            for (int q = 0; q < n; ++q) {
                const double d = host[2 * (q * n + q)];  // (R^H R)_qq
                bad |= !std::isfinite(d);
                any |= act[q] && d > inner_tol2[q];
            }
            if (bad) {
                *status = COLA_BREAKDOWN;
                break;
            }
            if (!any) break;
        }
        COLA_HIP(h, launch_block_solve(Grho[cur], Grho[1 - cur], mask_bits, n, beta, c.st));
        COLA_HIP(h, launch_block_xpay(S, n, h->num_cu, fx, fp, Pn, r32, P, beta, c.st));
        std::swap(P, Pn);
        cur = 1 - cur;
    }
    *iters = it;
    return COLA_OK;
}

int solve_defect(const Ctx &c, int inner_prec, const cola_cg_params_t &p, void *x64,
                 const void *b64, const std::vector<double> &thr, Outcome *o) {
    cola_handle_t *h = c.h;
    const BlasShape sh = c.shape();
    const int check = p.check_interval > 0 ? p.check_interval : default_check(c, 8);
    // default inner reductions: about as deep as the inner storage keeps the iterated
    // residual honest (FP16 ~5e-4 per rounding, FP32 ~6e-8), so that few restarts throw
    // away Krylov spaces: FP16 1e-2, FP32 1e-5 (two cycles for a 1e-10 solve)
    const double itol = p.inner_tol > 0 ? p.inner_tol : (inner_prec == COLA_FP16 ? 1e-2 : 1e-5);
    void *r64, *x32, *r32;
    COLA_TRY(vec(c, "r64", SpinorFmt::F64, &r64));
    COLA_TRY(vec(c, "x32", SpinorFmt::F32, &x32));
    COLA_TRY(vec(c, "r32", SpinorFmt::F32, &r32));
    std::vector<double> tr(c.R), prev(c.R, -1.0), s(c.R);
    int slow = 0;
    int prec = inner_prec;
    while (true) {
        COLA_TRY(initial_residual(c, r64, b64, x64, !p.use_x0 && o->outer == 0));
        COLA_TRY(read_slot(c, TRUE_RES, tr.data()));
        if (!finite_all(tr.data(), c.R)) {
            o->status = COLA_BREAKDOWN;
            return COLA_OK;
        }
        std::vector<int> act(c.R);
        bool done = true;
        double worst = 0;
        for (int q = 0; q < c.R; ++q) {
            act[q] = tr[q] > thr[q];
            done &= !act[q];
            s[q] = std::sqrt(tr[q]);
            if (act[q] && prev[q] > 0) worst = std::max(worst, std::sqrt(tr[q] / prev[q]));
        }
        if (done) {
            o->final_tr = tr;
            return COLA_OK;
        }
        if (o->iterations >= p.max_iter) {
            o->status = COLA_NOT_CONVERGED;
            return COLA_OK;
        }
        // Inner target per column (relative to |R|): the scheme's reduction, relaxed to
        // ten times below what the column still needs so the last cycle does not solve
        // far past the tolerance.
        std::vector<double> itol2(c.R, itol * itol);
        for (int q = 0; q < c.R; ++q)
            if (act[q] && tr[q] > 0) itol2[q] = std::max(itol * itol, 1e-2 * thr[q] / tr[q]);
        if (o->outer > 0 && worst > 0.5) {
            if (++slow >= 3 && prec == COLA_FP16) {
                prec = COLA_FP32;
                slow = 0;
            }
        } else {
            slow = 0;
        }
        prev = tr;
        COLA_TRY(write_slot(c, SCALE, s));
        const SpinorFmt fp = spinor_fmt(prec);
        void *pv, *ap;
        COLA_TRY(vec(c, "dp", fp, &pv));
        COLA_TRY(vec(c, "dap", fp, &ap));
        const Reduce red_rho = c.reduce(RHO);
        // Inner vectors: r = R / |R| (rho = |r|^2), p = r, x = 0.  Block CG keeps x and r in
        // FP32; the lockstep solver stores them like p, in the inner precision (FP16 rounds
        // them to about 5e-4 per update, far below the inner solve's 1e-2 reduction, and
        // saves a third of the bytes of the update kernels).
        const SpinorFmt fxr = p.block ? SpinorFmt::F32 : fp;
        void *xs = x32, *rs = r32;
        if (fxr != SpinorFmt::F32) {
            COLA_TRY(vec(c, "dx", fxr, &xs));
            COLA_TRY(vec(c, "dr", fxr, &rs));
        }
        COLA_HIP(h, launch_convert(sh, fxr, SpinorFmt::F64, rs, r64, c.slot(SCALE), 1, &red_rho,
                                   c.st));
        COLA_HIP(h, launch_convert(sh, fp, fxr, pv, rs, nullptr, 0, nullptr, c.st));
        COLA_HIP(h, hipMemsetAsync(xs, 0, c.bytes(fxr), c.st));
        int its = 0, st = COLA_OK;
        if (p.block)
            COLA_TRY(inner_block_cg(c, prec, x32, r32, itol2, p.max_iter - o->iterations, act,
                                    check, &its, &st));
        else
            COLA_TRY(inner_cg(c, prec, xs, rs, pv, ap, itol2, p.max_iter - o->iterations, act,
                              check, &its, &st));
        o->iterations += its;
        ++o->outer;
        if (st != COLA_OK) {
            o->status = st;
            return COLA_OK;
        }
        // X += |R| E
        COLA_HIP(h, launch_accum(sh, fxr, x64, xs, c.slot(SCALE), 0, c.st));
    }
}

}  // namespace

int cg_solve_impl(cola_handle_t *h, void *x, const void *b, int nrhs, const cola_cg_params_t *p,
                  cola_cg_result_t *r, hipStream_t st) {
    const auto t0 = std::chrono::steady_clock::now();
    Ctx c{h, st, nrhs, p->system == COLA_SYS_MDAGM ? 1 : 0};
    const BlasShape sh = c.shape();
    const size_t bb64 = spinor_block_bytes(h->g, SpinorFmt::F64, nrhs);
    void *b64, *x64, *bfull = nullptr;
    COLA_TRY(vec(c, "b64", SpinorFmt::F64, &b64));
    COLA_TRY(vec(c, "x64", SpinorFmt::F64, &x64));
    const bool clover = h->csw != 0.0;

    if (p->system == COLA_SYS_MDAGM) {
        COLA_HIP(h, launch_pack_spinor(h->g, SpinorFmt::F64, b64, b, nrhs, -1, st));
    } else if (p->system == COLA_SYS_SCHUR) {
        COLA_HIP(h, launch_pack_spinor(h->g, SpinorFmt::F64, b64, b, nrhs, 0, st));
    } else {
        // b_hat_e = b_e + kappa D_eo A_oo^-1 b_o ; rhs = S^H b_hat_e
        COLA_TRY(get_vec(h, "prop_b_full_" + std::to_string(nrhs), 2 * bb64, &bfull));
        COLA_HIP(h, launch_pack_spinor(h->g, SpinorFmt::F64, bfull, b, nrhs, -1, st));
        void *to, *bhat;
        COLA_TRY(get_vec(h, "prop_to_" + std::to_string(nrhs), bb64, &to));
        COLA_TRY(get_vec(h, "prop_bhat_" + std::to_string(nrhs), bb64, &bhat));
        const void *bo = (const char *)bfull + bb64;
        if (clover) {
            COLA_HIP(h, launch_clover_site(blas_shape(h->g, nrhs, 1), SpinorFmt::F64, 1, to, bo,
                                           h->clovinv64, 1, st));
        } else {
            COLA_HIP(h, hipMemcpyAsync(to, bo, bb64, hipMemcpyDeviceToDevice, st));
        }
        HopCall hc{bhat, to, 0, 0};
        hc.epi = EPI_XPAY;
        hc.x = bfull;
        hc.a = h->kappa;
        COLA_TRY(hop(h, hc, COLA_FP64, nrhs, st));
        COLA_TRY(apply_op(h, b64, bhat, COLA_OP_SCHUR_DAG, 0, COLA_FP64, nrhs, st));
    }
    if (p->use_x0) {
        COLA_HIP(h, hipMemsetAsync(x64, 0, c.bytes(SpinorFmt::F64), st));
        COLA_HIP(h, launch_pack_spinor(h->g, SpinorFmt::F64, x64, x, nrhs, c.full ? -1 : 0, st));
    } else {
        COLA_HIP(h, hipMemsetAsync(x64, 0, c.bytes(SpinorFmt::F64), st));
    }
    // thresholds tol^2 |b_q|^2
    std::vector<double> bn(nrhs), thr(nrhs);
    const Reduce red_b = reduce_into(h, BNORM);
    COLA_HIP(h, launch_norm2(sh, SpinorFmt::F64, b64, red_b, st));
    COLA_TRY(read_slot(c, BNORM, bn.data()));
    for (int q = 0; q < nrhs; ++q) thr[q] = p->tol * p->tol * bn[q];

    Outcome o;
    cola_cg_params_t pp = *p;
    auto run = [&]() -> int {
        o.final_tr.clear();
        switch (pp.scheme) {
            case COLA_CG_FP64: return solve_reliable(c, COLA_FP64, pp, x64, b64, thr, &o);
            case COLA_CG_FP32_RELIABLE: return solve_reliable(c, COLA_FP32, pp, x64, b64, thr, &o);
            case COLA_CG_FP16_DEFECT: return solve_defect(c, COLA_FP16, pp, x64, b64, thr, &o);
            case COLA_CG_FP32_DEFECT: return solve_defect(c, COLA_FP32, pp, x64, b64, thr, &o);
            default: return set_error(h, COLA_EINVAL, "unknown solver scheme");
        }
    };
    // final FP64 true residual of the solved system (the solver's last one when it
    // computed it for the returned x)
    std::vector<double> tr(nrhs);
    auto system_residual = [&]() -> int {
        if ((int)o.final_tr.size() == nrhs) {
            tr = o.final_tr;
        } else {
            void *r64;
            COLA_TRY(vec(c, "r64", SpinorFmt::F64, &r64));
            COLA_TRY(true_residual(c, r64, b64, x64, TRUE_RES));
            COLA_TRY(read_slot(c, TRUE_RES, tr.data()));
        }
        for (int q = 0; q < nrhs; ++q)
            if (!(tr[q] <= thr[q]) && o.status == COLA_OK) o.status = COLA_NOT_CONVERGED;
        return COLA_OK;
    };
    COLA_TRY(run());
    COLA_TRY(system_residual());

    if (p->system == COLA_SYS_PROPAGATOR) {
        // x_o = A_oo^-1 (b_o + kappa D_oe x_e) and the residual of M x = b on the full
        // lattice, one parity block at a time in the solver's FP64 residual block:
        // t = A_pp x_p - kappa D x_{1-p}, then t = b_p - t.  With x_o reconstructed
        // exactly, b - M x is (b_hat - S x_e) on the even sites and zero on the odd ones,
        // which the normal equations bound only up to the condition of S: a column whose
        // full residual misses tol has its normal-system threshold cut by
        // (tol / residual / 2)^2 and the solve continues from x (at most three times).
        void *xfull, *t;
        COLA_TRY(get_vec(h, "prop_x_full_" + std::to_string(nrhs), 2 * bb64, &xfull));
        COLA_TRY(vec(c, "r64", SpinorFmt::F64, &t));
        std::vector<double> bf(nrhs);
        const BlasShape sh1 = blas_shape(h->g, nrhs, 1);
        const BlasShape shf = blas_shape(h->g, nrhs, 2);
        const Reduce red_bf = reduce_into(h, BNORM);
        COLA_HIP(h, launch_norm2(shf, SpinorFmt::F64, bfull, red_bf, st));
        COLA_TRY(read_slot(c, BNORM, bf.data()));
        auto full_residual = [&]() -> int {
            COLA_HIP(h, hipMemcpyAsync(xfull, x64, bb64, hipMemcpyDeviceToDevice, st));
            HopCall hc{(char *)xfull + bb64, x64, 1, 0};
            hc.epi = clover ? EPI_XPAY_CLOV : EPI_XPAY;
            hc.x = (const char *)bfull + bb64;
            hc.a = h->kappa;
            hc.clov = h->clovinv64;
            COLA_TRY(hop(h, hc, COLA_FP64, nrhs, st));
            for (int q = 0; q < 2; ++q) {
                HopCall hm{t, (const char *)xfull + (1 - q) * bb64, q, 0};
                hm.epi = clover ? EPI_CLOV_XPAY : EPI_XPAY;
                hm.x = (const char *)xfull + q * bb64;
                hm.a = -h->kappa;
                hm.clov = h->clov64;
                COLA_TRY(hop(h, hm, COLA_FP64, nrhs, st));
                COLA_HIP(h, launch_residual(sh1, t, (const char *)bfull + q * bb64, t,
                                            reduce_into(h, q == 0 ? TRUE_RES : TMP), st));
            }
            COLA_HIP(h, launch_scalar_add(c.slot(TRUE_RES), c.slot(TMP), nrhs, st));
            return read_slot(c, TRUE_RES, tr.data());
        };
        COLA_TRY(full_residual());
        for (int round = 0; round < 3 && o.status == COLA_OK; ++round) {
            bool again = false;
            for (int q = 0; q < nrhs; ++q) {
                const double lim = p->tol * p->tol * bf[q];
                if (tr[q] > lim) {
                    thr[q] *= 0.25 * lim / tr[q];
                    again = true;
                }
            }
            if (!again) break;
            pp.use_x0 = 1;
            COLA_TRY(run());
            COLA_TRY(system_residual());
            COLA_TRY(full_residual());
        }
        for (int q = 0; q < nrhs; ++q)
            if (!(tr[q] <= p->tol * p->tol * bf[q]) && o.status == COLA_OK)
                o.status = COLA_NOT_CONVERGED;
        bn = bf;
        COLA_HIP(h, launch_unpack_spinor(h->g, SpinorFmt::F64, x, xfull, nrhs, -1, st));
    } else if (p->system == COLA_SYS_SCHUR) {
        COLA_HIP(h, hipMemsetAsync(x, 0, (size_t)h->g.Vh * 2 * 12 * 16 * nrhs, st));
        COLA_HIP(h, launch_unpack_spinor(h->g, SpinorFmt::F64, x, x64, nrhs, 0, st));
    } else {
        COLA_HIP(h, launch_unpack_spinor(h->g, SpinorFmt::F64, x, x64, nrhs, -1, st));
    }
    COLA_HIP(h, hipStreamSynchronize(st));
    if (r) {
        r->status = o.status;
        r->iterations = o.iterations;
        r->outer_cycles = o.outer;
        r->reliable_updates = o.reliable;
        if (r->true_rel_residual)
            for (int q = 0; q < nrhs; ++q)
                r->true_rel_residual[q] = bn[q] > 0 ? std::sqrt(tr[q] / bn[q]) : 0.0;
        r->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    return o.status;
}

// ---------------------------------------------------------------- multi-shift CG

// (A + sigma_q) x_q = b for nshift shifts sigma_q >= 0 from the Krylov space of the
// unshifted CG on A (M^H M or S^H S, FP64, one rhs).  The shifted residuals stay
// collinear with the base residual, r_q = zeta_q r, and with the base CG's alpha, beta
//   zeta_q' = zeta_q zeta_q^old alpha^old /
//             (alpha beta^old (zeta_q^old - zeta_q) + zeta_q^old alpha^old (1 + sigma_q alpha))
//   x_q += alpha zeta_q'/zeta_q p_q ;  p_q = zeta_q' r' + beta (zeta_q'/zeta_q)^2 p_q
// (zeta = zeta^old = 1, alpha^old = 1, beta^old = 0, p_q = b at the start).  Each shift's x
// and p are one-rhs fields; the scalar recursion runs on the device.  The base CG's own x is
// not needed and not formed.  A shift stops once zeta_q^2 |r|^2 <= tol^2
// |b|^2; its true residual is then checked against twice that.
int cg_multishift_impl(cola_handle_t *h, void *x, const void *b, int nshift, const double *sigma,
                       const cola_cg_params_t *p, cola_cg_result_t *res, hipStream_t st) {
    const auto t0 = std::chrono::steady_clock::now();
    const int full = p->system == COLA_SYS_MDAGM ? 1 : 0;
    Ctx c{h, st, 1, full};
    Ctx cn{h, st, nshift, full};
    const BlasShape sh1 = c.shape(), shn = cn.shape();
    void *b64, *r64, *p64, *xs, *ps, *axs;
    COLA_TRY(vec(c, "b64", SpinorFmt::F64, &b64));
    COLA_TRY(vec(c, "r64", SpinorFmt::F64, &r64));
    COLA_TRY(vec(c, "ms_p", SpinorFmt::F64, &p64));
    COLA_TRY(vec(cn, "ms_xs", SpinorFmt::F64, &xs));
    COLA_TRY(vec(cn, "ms_ps", SpinorFmt::F64, &ps));
    COLA_TRY(vec(cn, "ms_axs", SpinorFmt::F64, &axs));
    COLA_HIP(h, launch_pack_spinor(h->g, SpinorFmt::F64, b64, b, 1, full ? -1 : 0, st));
    const size_t b1 = c.bytes(SpinorFmt::F64), bn_ = cn.bytes(SpinorFmt::F64);
    COLA_HIP(h, hipMemcpyAsync(r64, b64, b1, hipMemcpyDeviceToDevice, st));
    COLA_HIP(h, hipMemcpyAsync(p64, b64, b1, hipMemcpyDeviceToDevice, st));
    COLA_HIP(h, hipMemsetAsync(xs, 0, bn_, st));
    COLA_HIP(h, hipMemsetAsync(ps, 0, bn_, st));
    // the shift recursion lives on the device (MsState): init writes the first update's
    // coefficients (p_q = b); each iteration's advance kernel reads the base CG's rho'
    // and pi where the reductions left them.  The host only reads the state's flags at
    // the convergence checks.
    void *state_v;
    COLA_TRY(get_vec(h, "ms_state", sizeof(MsState), &state_v));
    MsState *state = (MsState *)state_v;
    COLA_HIP(h, launch_norm2(sh1, SpinorFmt::F64, b64, reduce_into(h, BNORM), st));
    COLA_HIP(h, launch_ms_init(state, sigma, nshift, p->tol * p->tol, c.slot(BNORM), st));
    const size_t n = b1 / sizeof(Cplx64);
    double *rho = c.slot(RHO), *rho_new = c.slot(RHO_NEW);
    COLA_HIP(h, launch_ms_update(xs, ps, r64, nullptr, &state->coef, nshift, rho_new, rho, n, st));
    double bnorm = 0.0;
    COLA_TRY(read_slot(c, BNORM, &bnorm));
    COLA_HIP(h, hipMemcpyAsync(c.slot(RHO), c.slot(BNORM), sizeof(double),
                               hipMemcpyDeviceToDevice, st));
    COLA_TRY(write_active(c, std::vector<int>{1}));
    const double thr = p->tol * p->tol * bnorm;
    const int check = p->check_interval > 0 ? p->check_interval : default_check(c, 8);
    int status = COLA_OK, it = 0, iters = 0;
    // flags read back from the state: finished, status, iterations (consecutive ints)
    static_assert(offsetof(MsState, status) + sizeof(int) == offsetof(MsState, finished) &&
                      offsetof(MsState, finished) + sizeof(int) == offsetof(MsState, iterations),
                  "state flag order");
    bool finished = bnorm == 0.0;
    int flags[3] = {COLA_OK, finished ? 1 : 0, 0};
    while (!finished) {
        if (it >= p->max_iter) {
            status = COLA_NOT_CONVERGED;
            break;
        }
        if (full)
            COLA_TRY(full_normal_cg_step(c, COLA_FP64, r64, p64, rho,
                                         NormTo{rho_new, nullptr, nullptr}));
        else
            COLA_TRY(schur_normal_cg_step(h, COLA_FP64, 1, st, r64, p64, rho,
                                          NormTo{c.slot(PI), nullptr, nullptr}, h->active,
                                          NormTo{rho_new, nullptr, nullptr}));
        COLA_HIP(h, launch_ms_advance(state, rho_new, c.slot(PI), st));
        COLA_HIP(h, launch_ms_update(xs, ps, r64, p64, &state->coef, nshift, rho_new, rho, n, st));
        std::swap(rho, rho_new);
        ++it;
        if (it % check == 0 || it >= p->max_iter) {
            COLA_HIP(h, hipMemcpyAsync(flags, &state->status, sizeof flags,
                                       hipMemcpyDeviceToHost, st));
            COLA_HIP(h, hipStreamSynchronize(st));
            // flags: status, finished, iterations
            if (flags[0] != COLA_OK) {
                status = flags[0];
                break;
            }
            finished = flags[1] != 0;
        }
    }
    iters = finished ? flags[2] : it;
    // true residuals |b - (A + sigma_q) x_q| / |b|, all shifts in one multi-rhs pass
    std::vector<double> tr(nshift, 0.0);
    void *xr = ps;  // the directions are done with
    COLA_HIP(h, launch_ms_gather(xr, xs, nshift, n, st));
    COLA_TRY(normal(cn, COLA_FP64, axs, xr));
    COLA_HIP(h, launch_ms_residual(shn, b64, axs, xr, sigma, reduce_into(h, TRUE_RES), st));
    COLA_TRY(read_slot(cn, TRUE_RES, tr.data()));
    // the recursive residuals drift from the true ones by rounding: a shift counts as
    // converged within twice the tolerance
    for (int q = 0; q < nshift; ++q)
        if (!(tr[q] <= 4.0 * thr) && status == COLA_OK) status = COLA_NOT_CONVERGED;
    if (!full) COLA_HIP(h, hipMemsetAsync(x, 0, (size_t)h->g.Vh * 2 * 12 * 16 * nshift, st));
    COLA_HIP(h, launch_unpack_spinor(h->g, SpinorFmt::F64, x, xr, nshift, full ? -1 : 0, st));
    COLA_HIP(h, hipStreamSynchronize(st));
    if (res) {
        res->status = status;
        res->iterations = iters;
        res->outer_cycles = 0;
        res->reliable_updates = 0;
        if (res->true_rel_residual)
            for (int q = 0; q < nshift; ++q)
                res->true_rel_residual[q] = bnorm > 0 ? std::sqrt(tr[q] / bnorm) : 0.0;
        res->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    return status;
}

}  // namespace cola
