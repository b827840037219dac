// Shifted solves (sigma I - J) x = b for the Rosenbrock-type steps (Eq. ROS,
// Eq. ROSMh) and the Newton iterations of theta-Euler (Eq. temscheme): the
// paper solves these systems with BiCGSTAB; here BiCGSTAB runs with Jacobi
// right preconditioning, M = diag(sigma - J_ii), two kernels per iteration,
// every inner product reduced into a ring of partial sums that the next kernel
// adds up, a wavefront per sum (no host round trip per iteration).
//
// With y = M^{-1} p and z = M^{-1} s, iteration `it` is
//   K1: (it > 0) omega = (t, s) / (t, t),  x += alpha y + omega z,
//       r = s - omega t of the iteration before,  (r, r);
//       p = r + beta (p_old - omega v_old),  v = A y,  (rhat, v)
//   K2: stop test on (r, r);  alpha = (rhat, r) / (rhat, v),  s = r - alpha v,
//       t = A z,  (t, s), (t, t), (rhat, s), (rhat, t)
// where A = sigma I - J.  beta needs (rhat, r) of the new r before K1 has formed
// it: it is (rhat, s) - omega (rhat, t), which takes the place of a third kernel
// and its pass.  The difference cancels where an iteration shortens r much (by a
// factor f it loses log10 f digits of beta, which r and x do not inherit): over
// four operators, sigma from 1e-3 to 1e-9 and rtol from 1e-6 to 1e-15 the
// iterations were 0.88 .. 1.08 times those with (rhat, r) summed, the same up to
// 40, and the residuals alike.  (r, r), which the stop test compares over many orders, is summed
// from r itself.  A kernel that needs a neighbour's p (or s) forms it from the
// neighbour's operands, so p and v alternate between two buffers.
//
// On 512 x 512 the kernels are chains of latencies (launch, loads, sums,
// shuffles), 10 and 8 us; with three kernels per iteration, up to seven sums on
// one wavefront and a division per neighbour an iteration took 27.6 us.
#include <hip/hip_runtime.h>

#include "rosenbrock.h"

#include <algorithm>

namespace erem {

namespace {

// Sum of NV values over the 256-thread block; valid in thread 0.
template <int NV>
__device__ inline void rb_block_sum(double (&v)[NV]) {
  __shared__ double sh[kThreads / 64][NV];
#pragma unroll
  for (int n = 0; n < NV; ++n) v[n] = wave_sum(v[n]);
  const int t = threadIdx.x;
  if ((t & 63) == 0) {
#pragma unroll
    for (int n = 0; n < NV; ++n) sh[t >> 6][n] = v[n];
  }
  __syncthreads();
  if (t == 0) {
#pragma unroll
    for (int n = 0; n < NV; ++n) v[n] = sh[0][n] + sh[1][n] + sh[2][n] + sh[3][n];
  }
}

// First slot of iteration it's partials in a ring of four.
__device__ inline int slot_of(const BicgState* st, int it) { return (it & 3) * st->nb; }

// Neighbour k of cell (x, y, z) in the stencil's order (-x, +x, -y, +y, -z,
// +z); a missing neighbour maps to the cell itself (its coefficient is 0).
template <int NB>
struct Nbrs {
  int idx[NB];
  __device__ Nbrs(const Dims& d, int x, int y, int z, int i) {
    const int pl = d.nx * d.ny;
    idx[0] = x > 0 ? i - 1 : i;
    idx[1] = x + 1 < d.nx ? i + 1 : i;
    idx[2] = y > 0 ? i - d.nx : i;
    idx[3] = y + 1 < d.ny ? i + d.nx : i;
    if (NB == 6) {
      idx[NB == 6 ? 4 : 0] = z > 0 ? i - pl : i;
      idx[NB == 6 ? 5 : 0] = z + 1 < d.nz ? i + pl : i;
    }
  }
};

// Scalars of a new solve (every producer overwrites all partial slots, so they
// need no clearing).
__global__ void k_bicg_reset(BicgState* st, double tol2) {
  if (threadIdx.x == 0) {
    st->done = 0;
    st->it_done = 0;
    st->breakdown = 0;
    st->bad = 0;
    st->tol2 = tol2;
  }
}

// The cell bands (64 x 4 cells) of the grid, dealt to the workgroups in turn.
struct Bands {
  int gx, gy, n;
  __device__ explicit Bands(const Dims& d) : gx((d.nx + kBX - 1) / kBX), gy((d.ny + kBY - 1) / kBY), n(gx * gy * d.nz) {}
  __device__ void cell(int b, int& x, int& y, int& z) const {
    x = (b % gx) * kBX + (threadIdx.x & 63);
    y = ((b / gx) % gy) * kBY + (threadIdx.x >> 6);
    z = b / (gx * gy);
  }
};

__global__ __launch_bounds__(kThreads) void k_bicg_start(Dims d, double sigma, const double* __restrict__ coef,
                                               const double* __restrict__ b, double* __restrict__ xv,
                                               double* __restrict__ r, double* __restrict__ rhat,
                                               double* __restrict__ dinv, BicgState* st) {
  double s[1] = {0.0};
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < d.N; i += gridDim.x * kThreads) {
    const double bi = b[i];
    r[i] = bi;
    rhat[i] = bi;
    xv[i] = 0.0;
    dinv[i] = 1.0 / (sigma - coef[i]);
    s[0] += bi * bi;
  }
  rb_block_sum<1>(s);
  if (threadIdx.x == 0) st->bb_sl[blockIdx.x] = s[0];  // also (rhat, r_0) and (r_0, r_0)
}

// Operands of one cell in K1 (the neighbours' loads go out with the cell's own).
template <int NB>
struct PvCell {
  bool in;
  int i;
  double r, s, t, p, v, rh, dv, x;
  double ns[NB], nt[NB], np[NB], nv[NB], nd[NB], ck[NB];
};

// K1 of iteration `it` (see above).
template <int NB>
__global__ __launch_bounds__(kThreads) void k_bicg_pv(Dims d, const double* __restrict__ coef,
                                            double* __restrict__ r, const double* __restrict__ sv,
                                            const double* __restrict__ tv, const double* __restrict__ pold,
                                            const double* __restrict__ vold, double* __restrict__ pnew,
                                            double* __restrict__ vnew, const double* __restrict__ rhat,
                                            const double* __restrict__ dinv, double* __restrict__ xv,
                                            BicgState* st, int it) {
  __shared__ double sums[4];
  const Bands B(d);
  const int N = d.N, t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int stopped = *(volatile const int*)&st->done;  // only K2 writes it
  auto load = [&](int b) {
    PvCell<NB> c;
    int x, y, z;
    B.cell(b, x, y, z);
    c.in = x < d.nx && y < d.ny;
    c.i = c.in ? x + d.nx * (y + d.ny * z) : 0;
    if (!c.in) x = y = z = 0;
    const Nbrs<NB> nb(d, x, y, z, c.i);
    c.rh = rhat[c.i];
    c.dv = dinv[c.i];
    if (it == 0) {
      c.r = r[c.i];
    } else {
      c.s = sv[c.i];
      c.t = tv[c.i];
      c.p = pold[c.i];
      c.v = vold[c.i];
      c.x = xv[c.i];
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int j = nb.idx[k];
      c.nd[k] = dinv[j];
      c.ck[k] = coef[static_cast<size_t>(k + 1) * N + c.i];
      if (it == 0) {
        c.ns[k] = r[j];
      } else {
        c.ns[k] = sv[j];
        c.nt[k] = tv[j];
        c.np[k] = pold[j];
        c.nv[k] = vold[j];
      }
    }
    return c;
  };
  int band = blockIdx.x;
  PvCell<NB> c = load(band);  // in flight while the sums are added up
  double om = 0.0, beta = 0.0, alpha = 0.0;
  if (it > 0) {
    const double* src[4] = {st->hs, st->ht, st->ts, st->tt};
    const double v = wave_part_sum(src[wave] + slot_of(st, it - 1), st->nb);
    if (lane == 0) sums[wave] = v;
    const double rho_p = st->rho_v[(it - 1) & 3];
    alpha = st->alpha[(it - 1) & 3];
    __syncthreads();
    om = sums[3] > 0.0 ? sums[2] / sums[3] : 0.0;
    const double rho = sums[0] - om * sums[1];
    beta = (rho / rho_p) * (alpha / om);
    const bool bad = rho == 0.0 || !isfinite(beta);
    if (bad) beta = 0.0;  // K2 decides: converged, or broken down
    if (blockIdx.x == 0 && t == 0 && !stopped) {
      st->rho_v[it & 3] = rho;
      st->bad = bad ? 1 : 0;
    }
  }
  if (stopped) return;
  double s[2] = {0.0, 0.0};
  for (;;) {
    if (c.in) {
      double rc, p;
      if (it == 0) {
        rc = c.r;
        p = rc;
      } else {
        rc = c.s - om * c.t;
        p = rc + beta * (c.p - om * c.v);
        xv[c.i] = c.x + (alpha * c.p + om * c.s) * c.dv;
        r[c.i] = rc;
      }
      double v = p;  // the preconditioned operator's own-cell term
#pragma unroll
      for (int k = 0; k < NB; ++k) {
        const double pk = it == 0 ? c.ns[k] : (c.ns[k] - om * c.nt[k]) + beta * (c.np[k] - om * c.nv[k]);
        v -= c.ck[k] * (pk * c.nd[k]);
      }
      pnew[c.i] = p;
      vnew[c.i] = v;
      s[0] += c.rh * v;
      s[1] += rc * rc;
    }
    band += gridDim.x;
    if (band >= B.n) break;
    c = load(band);
  }
  rb_block_sum<2>(s);
  if (t == 0) {
    st->rv[slot_of(st, it) + blockIdx.x] = s[0];
    st->rr[slot_of(st, it) + blockIdx.x] = s[1];
  }
}

template <int NB>
struct StCell {
  bool in;
  int i;
  double r, v, rh;
  double nr[NB], nv[NB], nd[NB], ck[NB];
};

// K2 of iteration `it` (see above).
template <int NB>
__global__ __launch_bounds__(kThreads) void k_bicg_st(Dims d, const double* __restrict__ coef,
                                            const double* __restrict__ r, const double* __restrict__ v,
                                            const double* __restrict__ rhat, const double* __restrict__ dinv,
                                            double* __restrict__ sv, double* __restrict__ tv, BicgState* st,
                                            int it) {
  __shared__ double sums[3];
  __shared__ int stop_sh;
  const Bands B(d);
  const int N = d.N, t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  auto load = [&](int b) {
    StCell<NB> c;
    int x, y, z;
    B.cell(b, x, y, z);
    c.in = x < d.nx && y < d.ny;
    c.i = c.in ? x + d.nx * (y + d.ny * z) : 0;
    if (!c.in) x = y = z = 0;
    const Nbrs<NB> nb(d, x, y, z, c.i);
    c.r = r[c.i];
    c.v = v[c.i];
    c.rh = rhat[c.i];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int j = nb.idx[k];
      c.nr[k] = r[j];
      c.nv[k] = v[j];
      c.nd[k] = dinv[j];
      c.ck[k] = coef[static_cast<size_t>(k + 1) * N + c.i];
    }
    return c;
  };
  int band = blockIdx.x;
  StCell<NB> c = load(band);
  if (wave < 3) {
    const double* src[3] = {st->rr + slot_of(st, it), st->rv + slot_of(st, it), st->bb_sl};
    const double w = wave_part_sum(src[wave], st->nb);
    if (lane == 0) sums[wave] = w;
  }
  // one reading of the flag for the whole workgroup: workgroup 0 may set it
  if (t == 0) stop_sh = *(volatile const int*)&st->done;
  const double rho_v = it > 0 ? st->rho_v[it & 3] : 0.0;
  const int bad = st->bad;
  __syncthreads();
  if (stop_sh) return;
  const double rr = sums[0], bb = sums[2];
  const double rho = it > 0 ? rho_v : bb;  // (rhat, r_0) = ||b||^2
  const double alpha = rho / sums[1];
  const bool conv = isfinite(rr) && rr <= st->tol2 * bb;
  const bool fail = !conv && (!isfinite(rr) || (it > 0 && bad) || !isfinite(alpha));
  if (conv || fail) {
    if (blockIdx.x == 0 && t == 0) {
      if (fail) st->breakdown = 1;
      st->it_done = it;
      st->done = 1;
    }
    return;
  }
  if (blockIdx.x == 0 && t == 0) {
    st->alpha[it & 3] = alpha;
    if (it == 0) st->rho_v[0] = rho;
  }
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (;;) {
    if (c.in) {
      const double si = c.r - alpha * c.v;
      double ti = si;
#pragma unroll
      for (int k = 0; k < NB; ++k) ti -= c.ck[k] * ((c.nr[k] - alpha * c.nv[k]) * c.nd[k]);
      sv[c.i] = si;
      tv[c.i] = ti;
      s[0] += ti * si;
      s[1] += ti * ti;
      s[2] += c.rh * si;
      s[3] += c.rh * ti;
    }
    band += gridDim.x;
    if (band >= B.n) break;
    c = load(band);
  }
  rb_block_sum<4>(s);
  if (t == 0) {
    const int o = slot_of(st, it) + blockIdx.x;
    st->ts[o] = s[0];
    st->tt[o] = s[1];
    st->hs[o] = s[2];
    st->ht[o] = s[3];
  }
}

__global__ __launch_bounds__(kThreads) void k_lincomb(Dims d, double* out, LinComb lc) {
  const int x = blockIdx.x * kBX + threadIdx.x;
  const int y = blockIdx.y * kBY + threadIdx.y;
  const int z = blockIdx.z;
  if (x >= d.nx || y >= d.ny) return;
  const int i = x + d.nx * (y + d.ny * z);
  double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int m = 0; m < 4; ++m)
    if (m < lc.n) a[m] = lc.in[m][i];
  double s = lc.w[0] * a[0];
#pragma unroll
  for (int m = 1; m < 4; ++m)
    if (m < lc.n) s += lc.w[m] * a[m];
  out[i] = s;
}

}  // namespace

hipError_t launch_bicg_reset(BicgState* st, double tol2, hipStream_t s) {
  hipLaunchKernelGGL(k_bicg_reset, dim3(1), dim3(256), 0, s, st, tol2);
  return hipGetLastError();
}

int bicg_blocks(const Dims& d) { return std::min(cell_bands(d), kBicgBlocks); }

hipError_t launch_bicg_start(const Dims& d, double sigma, const double* coef, const double* b, double* x,
                             const BicgBufs& B, BicgState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_bicg_start, dim3(bicg_blocks(d)), dim3(kThreads), 0, s, d, sigma, coef, b, x, B.r, B.rhat,
                     B.dinv, st);
  return hipGetLastError();
}

template <int NB>
static hipError_t bicg_iteration(const Dims& d, const double* coef, double* x, const BicgBufs& B, BicgState* st,
                                 int it, hipStream_t s, const hipEvent_t* e) {
  const hipEvent_t n = nullptr;
  const double* pold = B.p[(it + 1) & 1];
  const double* vold = B.v[(it + 1) & 1];
  const dim3 g(bicg_blocks(d)), b(kThreads);
  launch_timed(k_bicg_pv<NB>, g, b, 0, s, e ? e[0] : n, e ? e[1] : n, d, coef, B.r,
               static_cast<const double*>(B.s), static_cast<const double*>(B.t), pold, vold, B.p[it & 1], B.v[it & 1],
               static_cast<const double*>(B.rhat), static_cast<const double*>(B.dinv), x, st, it);
  launch_timed(k_bicg_st<NB>, g, b, 0, s, e ? e[2] : n, e ? e[3] : n, d, coef, static_cast<const double*>(B.r),
               static_cast<const double*>(B.v[it & 1]), static_cast<const double*>(B.rhat),
               static_cast<const double*>(B.dinv), B.s, B.t, st, it);
  return hipGetLastError();
}

hipError_t launch_bicg_iteration(const Dims& d, const double* coef, double* x, const BicgBufs& B, BicgState* st,
                                 int it, hipStream_t s, const hipEvent_t* e) {
  return d.dim == 3 ? bicg_iteration<6>(d, coef, x, B, st, it, s, e) : bicg_iteration<4>(d, coef, x, B, st, it, s, e);
}

hipError_t launch_lincomb(const Dims& d, double* out, const LinComb& lc, hipStream_t s) {
  hipLaunchKernelGGL(k_lincomb, cell_grid(d), cell_block(), 0, s, d, out, lc);
  return hipGetLastError();
}

}  // namespace erem
