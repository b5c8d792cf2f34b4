// Host-side pieces shared by the solver and batch runtimes.
#pragma once

#include <stdint.h>

#include "ace_internal.h"

namespace ace {

// Validated problem of one handle or batch instance (Sec. 2 notation).
struct Problem {
    int d, bc;
    int64_t N[3], M[3], total;
    double L[3], R[3];
    double dx, dt, eps, kappa, h;
    int nit;
    int start2;  // second-order start of the root iteration
    int rv;      // root variant of the implicit scheme (ROOT_*), and its polynomial
    double q[ROOT_MAX_DEG + 1];
    int cond_ok;
    int scheme;  // ACE_SCHEME_*
};

// True if the environment variable ACE_LOG is set: the library then reports
// HIP errors, handle parameters, graph captures and autotuner choices on
// stderr, one "[ace]" line each.
bool log_enabled();
int hip_status(hipError_t e);
int64_t nodes_per_axis(int64_t N, int bc);
// Fills p.nit, p.start2, p.rv and p.q from p.h.
void choose_root(Problem &p);
// ACE_OK, ACE_W_CONDITIONS or a negative error.
int derive(int d, const int64_t *N, const double *L, const double *R, double eps, double dt,
           int bc, Problem &p);
Shape shape_of(const Problem &p);
StepCoef coef_of(const Problem &p);
// E = dxd (bulk + cg grad) with dxd = dx^d and cg = kappa / (2 dt).
void energy_coefs(const Problem &p, double *dxd, double *cg);
double energy_from(const Problem &p, const double *trip);
// Waits for a handle's old stream before its work moves to `next`.  Not where
// either is under capture: a wait would break the old stream's, and a new
// stream's cannot wait for another (the caller has ordered them).
void leave_stream(hipStream_t old, hipStream_t next);
// (Re)allocates *ptr to hold at least need doubles of device memory.
int grow(double **ptr, int64_t *cap, int64_t need);

}  // namespace ace
