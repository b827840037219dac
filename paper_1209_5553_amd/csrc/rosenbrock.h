// Shifted linear solves (sigma I - J) x = b for the Rosenbrock-type and
// theta-Euler steps (Sec. 3.2.1-3.2.3): BiCGSTAB with Jacobi (diagonal)
// right preconditioning on the stencil of J, scalars resident on the device.
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace erem {

// Most workgroups, and partials per inner product, that the next kernel's
// wavefronts add up (ROS2(1) on 512 x 512, two coupled steps: 4.91 / 4.65 / 4.89 ms
// with 256 / 512 / 1024).
constexpr int kBicgBlocks = 512;
int bicg_blocks(const Dims& d);

// Scalars of the BiCGSTAB iteration.  Its inner products are kept as
// partial sums, one per workgroup, in a ring of four iterations; every consumer
// adds a product's partials in order (wave_part_sum), so results do not depend
// on the order in which workgroups ran.  The arrays live in one allocation of
// bicg_parts_words(nb) doubles.
struct BicgState {
  int done;         // 1 once converged (or broken down)
  int it_done;      // iteration at which the test passed
  int breakdown;    // rho = 0, omega = 0 or a non-finite scalar
  int bad;          // the last K1 found no usable beta
  int nb;           // partial slots per inner product
  double tol2;      // rtol^2
  double rho_v[4];  // (rhat, r_it)
  double alpha[4];
  double* bb_sl;    // [nb] ||b||^2
  double* rr;       // [4][nb] (r_it, r_it)
  double* rv;       // [4][nb] (rhat, v_it)
  double* ts;       // [4][nb] (t_it, s_it)
  double* tt;       // [4][nb] (t_it, t_it)
  double* hs;       // [4][nb] (rhat, s_it)
  double* ht;       // [4][nb] (rhat, t_it)
};
inline size_t bicg_parts_words(int nb) { return static_cast<size_t>(25) * nb; }
inline void bicg_bind_parts(BicgState* st, double* parts, int nb) {
  st->nb = nb;
  double** p[] = {&st->rr, &st->rv, &st->ts, &st->tt, &st->hs, &st->ht};
  st->bb_sl = parts;
  parts += nb;
  for (double** q : p) {
    *q = parts;
    parts += 4 * static_cast<size_t>(nb);
  }
}

// Vectors of one solve (N values each, device).
struct BicgBufs {
  double *r, *rhat, *p[2], *v[2], *s, *t, *dinv;
};

hipError_t launch_bicg_reset(BicgState* st, double tol2, hipStream_t s);
// r = rhat = b, x = 0, 1 / (sigma - J_ii), ||b||^2
hipError_t launch_bicg_start(const Dims& d, double sigma, const double* coef, const double* b, double* x,
                             const BicgBufs& B, BicgState* st, hipStream_t s);
// One iteration `it` (two kernels); with events, kernel-level timing of each
// (e[0..3]).
hipError_t launch_bicg_iteration(const Dims& d, const double* coef, double* x, const BicgBufs& B, BicgState* st,
                                 int it, hipStream_t s, const hipEvent_t* e = nullptr);
// out = sum_{m < n} w[m] in[m] (elementwise; out may alias in[0])
struct LinComb {
  const double* in[4];
  double w[4];
  int n;
};
hipError_t launch_lincomb(const Dims& d, double* out, const LinComb& lc, hipStream_t s);

}  // namespace erem
