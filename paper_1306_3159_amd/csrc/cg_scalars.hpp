// The scalars of a CG solve and the formulas that advance them: plain functions of the scalars,
// compiled for the device by the kernels and for the host by the tests.
#pragma once

#include <math.h>

#include <cstdint>

#ifdef __HIPCC__
#define BRD_HD __host__ __device__ __forceinline__
#else
#define BRD_HD inline
#endif

namespace brd {

// Device-resident scalars of one CG solve. Every kernel of an iteration reads
// `done` first and returns if it is set, so the host can enqueue iterations
// without waiting for convergence. `done` is set by the finalize kernel only, whose one
// work-group nobody else's entry test can race with.
struct Scalars {
    double pq;        // p . B p
    double alpha;     // CG step
    double beta;      // CG direction update (Polak-Ribiere form)
    double rr;        // r . r
    double rsum;      // sum r
    double qsum;      // sum q
    double tol2;      // stop when rr <= tol2
    double shift;     // constant added to the V-cycle output z (null-space handling)
    double mean_r;    // mean removed from r before the V-cycle (projected problems)
    double mean_next; // mean of the next r predicted from sum r and sum q (fused update + V-cycle entry)
    double inv_ncell; // 1 / (nx ny nz)
    double eBe_inv;   // 1 / (e^T B e) for the reactive alpha = 0 constant mode (0 otherwise)
    double rr0;       // r . r of the initial residual
    double gg;        // right-hand side g . g
    int32_t done;     // 1: converged (or failed); kernels become no-ops
    int32_t iters;    // completed CG iterations
    int32_t project;  // 1: alpha = 0 problem, work on mean-zero vectors
    int32_t status;   // 0 ok, 1 breakdown/non-finite
    int32_t xzero;    // 1: x starts at zero and its first step writes it (no prior fill)
    int32_t xsteps;   // iterations whose steps x holds
    int32_t halt[2];  // breakdown found by the direction's (0), the update's (1) launch in the sums it
                      // finished itself; the next finalize launch turns it into status and done
    double rz[2];     // z . r (with the constant shift) of the last two iterates (iteration k: rz[k & 1])
    double step[2];   // CG steps of the last two iterations (iteration k: step[k & 1])
};

BRD_HD bool is_finite_d(double v) { return v == v && v - v == 0.0; }

// Entry tests of the direction's and of the update's launch. Where such a launch finishes a
// reduction itself, its first block stores the results while other blocks (and other waves of a
// block) are still to come: neither these tests nor the sums' formulas read a field which that
// launch stores, so all of a launch's waves decide alike.
BRD_HD bool cg_dir_runs(const Scalars* sc) { return !sc->done; }
BRD_HD bool cg_update_runs(const Scalars* sc) { return !sc->done && !sc->halt[0]; }

// The CG step from p.q and sum q, with its roundings fixed (formed by the finalize kernel or by
// every block of the update). sum(r - alpha q) = sum r - alpha sum q: the mean the fused update
// removes.
struct CgAlpha {
    double alpha, mean;
    bool bad;
};
BRD_HD CgAlpha cg_alpha(double pq, double qs, const Scalars* sc) {
#pragma clang fp contract(off)
    const double rz = sc->rz[sc->iters & 1];
    CgAlpha c{0.0, 0.0, !(pq > 0.0) || !is_finite_d(pq) || !is_finite_d(rz)};
    if (!c.bad) {
        c.alpha = rz / pq;
        if (sc->project) c.mean = fma(-c.alpha, qs, sc->rsum) * sc->inv_ncell;
    }
    return c;
}
BRD_HD void cg_stop(Scalars* sc) {
    sc->status = 1;
    sc->done = 1;
}
// folded: stored by the update's own launch
BRD_HD void cg_alpha_store(const CgAlpha& c, double pq, double qs, Scalars* sc, bool folded) {
    sc->pq = pq;
    sc->qsum = qs;
    sc->mean_next = c.mean;
    sc->alpha = c.alpha;
    sc->xsteps = sc->iters & ~1;  // the direction's launch has applied these
    if (!c.bad) sc->step[sc->iters & 1] = c.alpha;
    else if (folded) sc->halt[1] = 1;
    else cg_stop(sc);
}

// The direction's scalars from sum z, z.r and z.q, likewise (Polak-Ribiere form).
struct CgBeta {
    double shift, rz, beta;
    bool bad;
};
BRD_HD CgBeta cg_beta(double zs, double zr, double zq, const Scalars* sc) {
#pragma clang fp contract(off)
    CgBeta c;
    c.shift = sc->project ? fma(sc->rsum, sc->eBe_inv, -(zs * sc->inv_ncell)) : 0.0;
    c.rz = fma(c.shift, sc->rsum, zr);
    const double zq_full = fma(c.shift, sc->qsum, zq);
    c.beta = sc->iters == 0 ? 0.0 : -sc->alpha * zq_full / sc->rz[(sc->iters & 1) ^ 1];
    c.bad = !is_finite_d(c.rz) || !is_finite_d(c.beta);
    return c;
}
// folded: stored by the direction's own launch
BRD_HD void cg_beta_store(const CgBeta& c, Scalars* sc, bool folded) {
    sc->shift = c.shift;
    sc->beta = c.beta;
    sc->rz[sc->iters & 1] = c.rz;
    if (!c.bad) return;
    if (folded) sc->halt[0] = 1;
    else cg_stop(sc);
}

// Whether a launch of this iteration has found a breakdown that is still to be raised.
BRD_HD bool cg_halted(const Scalars* sc) { return sc->halt[0] || sc->halt[1]; }

}  // namespace brd
