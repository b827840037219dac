// Aggregation multigrid preconditioner for the TPFA pressure operator.
//
// Levels: cells aggregated 2 x 2 (x 2 in 3D).  With piecewise-constant
// prolongation P the Galerkin operator P^T A P of a two-point-flux matrix is
// again a two-point-flux matrix whose face transmissibility is the sum of the
// fine transmissibilities crossing the coarse face (Dirichlet faces included),
// so every level keeps the same face-array layout as the fine grid.
// Smoother: on the 2D grid levels three Jacobi-type sweeps weighted by the
// reciprocals of the Chebyshev points of [2/3, 2] (the degree-3 Chebyshev
// polynomial in D^-1 A, whose spectrum these diagonally dominant M-matrices
// keep inside (0, 2]); on the 3D grid levels and the LDS-resident levels two
// damped-Jacobi sweeps (omega 0.8); the same sweeps before and after the
// coarse correction, which is over-relaxed by omega_c.  The bottom level (at
// most kMgBottomCells cells) is solved exactly with a dense inverse formed
// once per setup.  The cycle is symmetric, so it is a valid
// conjugate-gradient preconditioner.  Each grid level runs two kernels: the
// down leg (sweeps from zero + restricted residual) and the up leg (coarse
// correction + sweeps), each recomputing its neighbours' intermediate sweeps
// on shrinking halos instead of waiting for a grid-wide pass; the levels with
// at most kMgLdsCells cells run inside one workgroup with everything in LDS.
#include "device.h"
#include "lds_grant.h"
#include "mg.h"

namespace erem {

namespace {

constexpr double kOmega = 0.8;

// Weights of the sweeps on the 2D grid levels: the reciprocals of the
// Chebyshev points of [lmax / 3, lmax] for lmax = 2 (the Gershgorin bound of
// D^-1 A for these operators), so the smoother is the degree-NU Chebyshev
// polynomial in D^-1 A.  Any order gives the same polynomial, so the cycle
// stays symmetric.
template <int NU>
__device__ inline double sweep_weight(int k) {
  const double lmax = 2.0, lmin = lmax / 3.0;
  const double z = 0.5 * (lmax + lmin) + 0.5 * (lmax - lmin) * cos(M_PI * (2 * k + 1) / (2.0 * NU));
  return 1.0 / z;
}

__device__ inline int fxi(int nx, int ny, int x, int y, int z) { return (z * ny + y) * (nx + 1) + x; }
__device__ inline int fyi(int nx, int ny, int x, int y, int z) { return (z * (ny + 1) + y) * nx + x; }
__device__ inline int fzi(int nx, int ny, int x, int y, int z) { return (z * ny + y) * nx + x; }

__device__ inline bool pcg_done(const PcgState* st) { return st && *(volatile const int*)&st->done; }


// ---------------------------------------------------------------------------
// Setup: coarse faces and diagonal from the fine faces.
// ---------------------------------------------------------------------------
__device__ inline void coarsen_cell(const MgLevelDev& F, const MgLevelDev& C, int X, int Y, int Z) {
  const int fnx = F.nx, fny = F.ny, fnz = F.nz;
  const int y0 = 2 * Y, y1 = min(2 * Y + 1, fny - 1);
  const int x0 = 2 * X, x1 = min(2 * X + 1, fnx - 1);
  const int z0 = fnz > 1 ? 2 * Z : 0;
  const int z1 = fnz > 1 ? min(2 * Z + 1, fnz - 1) : 0;
  auto sum_x = [&](int xf) {
    double s = 0.0;
    for (int z = z0; z <= z1; ++z)
      for (int y = y0; y <= y1; ++y) s += F.tx[fxi(fnx, fny, xf, y, z)];
    return s;
  };
  auto sum_y = [&](int yf) {
    double s = 0.0;
    for (int z = z0; z <= z1; ++z)
      for (int x = x0; x <= x1; ++x) s += F.ty[fyi(fnx, fny, x, yf, z)];
    return s;
  };
  auto sum_z = [&](int zf) {
    double s = 0.0;
    for (int y = y0; y <= y1; ++y)
      for (int x = x0; x <= x1; ++x) s += F.tz[fzi(fnx, fny, x, y, zf)];
    return s;
  };
  const double w = sum_x(2 * X);
  const double e = sum_x(min(2 * X + 2, fnx));
  const double s = sum_y(2 * Y);
  const double n = sum_y(min(2 * Y + 2, fny));
  double b = 0.0, t = 0.0;
  if (fnz > 1) {
    b = sum_z(2 * Z);
    t = sum_z(min(2 * Z + 2, fnz));
  }
  const int cnx = C.nx, cny = C.ny;
  C.tx[fxi(cnx, cny, X + 1, Y, Z)] = e;
  if (X == 0) C.tx[fxi(cnx, cny, 0, Y, Z)] = w;
  C.ty[fyi(cnx, cny, X, Y + 1, Z)] = n;
  if (Y == 0) C.ty[fyi(cnx, cny, X, 0, Z)] = s;
  C.tz[fzi(cnx, cny, X, Y, Z + 1)] = t;
  if (Z == 0) C.tz[fzi(cnx, cny, X, Y, 0)] = b;
  C.diag[X + cnx * (Y + cny * Z)] = w + e + s + n + b + t;
}

__global__ __launch_bounds__(kThreads) void k_mg_coarsen(MgLevelDev F, MgLevelDev C) {
  const int X = blockIdx.x * kBX + threadIdx.x;
  const int Y = blockIdx.y * kBY + threadIdx.y;
  if (X < C.nx && Y < C.ny) coarsen_cell(F, C, X, Y, blockIdx.z);
}

// The tail of the setup in one workgroup of 1024 threads: the coarse levels of
// the one-workgroup solve (a.lev[1] .. from a.lev[0] on; too small to be worth a
// launch each), then the dense inverse of the bottom operator by Gauss-Jordan
// (SPD, diagonally dominant, so it is stable without pivoting), the matrix in
// registers: thread t keeps row t / 16, columns 4 (t % 16) .. + 3; the new pivot
// row and the pivot column go through LDS, double buffered, a barrier per pivot.
// The chain of pivots is what it costs, 0.5 us each.  Only the wavefront that owns
// the pivot row divides and scales it.  Tail and inverse together take 41 us, what
// the inverse alone took when all sixteen wavefronts divided, four to a SIMD; the
// three launches of the tail are saved.  Rows and columns past n carry values that
// are never stored.
static_assert(kMgBottomCells <= 64, "the bottom inverse maps 64 rows x 16 column groups of 4 onto 1024 threads");
__global__ __launch_bounds__(1024) void k_mg_bottom_inverse(MgCoarseArgs a, double* __restrict__ inv) {
  __shared__ double M[64 * 64];
  __shared__ double prow[2][64];
  __shared__ double pcol[2][64];
  for (int l = 0; l + 1 < a.nlev; ++l) {
    const MgLevelDev &F = a.lev[l], &C = a.lev[l + 1];
    for (int c = threadIdx.x; c < C.nx * C.ny * C.nz; c += 1024)
      coarsen_cell(F, C, c % C.nx, (c / C.nx) % C.ny, c / (C.nx * C.ny));
    __syncthreads();
  }
  const MgLevelDev& L = a.lev[a.nlev - 1];
  const int n = L.nx * L.ny * L.nz;
  for (int j = threadIdx.x; j < 64 * 64; j += 1024) M[j] = 0.0;
  __syncthreads();
  if (static_cast<int>(threadIdx.x) < n) {
    const int c = threadIdx.x;
    const int x = c % L.nx, y = (c / L.nx) % L.ny, z = c / (L.nx * L.ny);
    // diagonal = sum of the cell's face transmissibilities (Dirichlet faces
    // included), formed here so that the finest level needs no other setup
    double dg = L.tx[fxi(L.nx, L.ny, x, y, z)] + L.tx[fxi(L.nx, L.ny, x + 1, y, z)] +
                L.ty[fyi(L.nx, L.ny, x, y, z)] + L.ty[fyi(L.nx, L.ny, x, y + 1, z)];
    if (L.nz > 1) dg += L.tz[fzi(L.nx, L.ny, x, y, z)] + L.tz[fzi(L.nx, L.ny, x, y, z + 1)];
    double* row = M + c * 64 + c;
    row[0] = dg;
    if (x > 0) row[-1] = -L.tx[fxi(L.nx, L.ny, x, y, z)];
    if (x + 1 < L.nx) row[1] = -L.tx[fxi(L.nx, L.ny, x + 1, y, z)];
    if (y > 0) row[-L.nx] = -L.ty[fyi(L.nx, L.ny, x, y, z)];
    if (y + 1 < L.ny) row[L.nx] = -L.ty[fyi(L.nx, L.ny, x, y + 1, z)];
    if (z > 0) row[-L.nx * L.ny] = -L.tz[fzi(L.nx, L.ny, x, y, z)];
    if (z + 1 < L.nz) row[L.nx * L.ny] = -L.tz[fzi(L.nx, L.ny, x, y, z + 1)];
  }
  __syncthreads();
  const int t = threadIdx.x;
  const int i = t >> 4, g = t & 15, j0 = 4 * g;
  double m[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) m[u] = M[i * 64 + j0 + u];
  for (int k = 0; k < n; ++k) {
    const int b = k & 1, u = k & 3;
    if (i >> 2 == k >> 2) {
      // this wavefront has row k, its pivot in lane 16 (k % 4) + k / 4
      const double piv = 1.0 / lane_of(u == 0 ? m[0] : u == 1 ? m[1] : u == 2 ? m[2] : m[3], 16 * u + (k >> 2));
      if (i == k) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          m[v] = j0 + v == k ? piv : m[v] * piv;
          prow[b][j0 + v] = m[v];
        }
      }
    }
    if (g == k >> 2) pcol[b][i] = u == 0 ? m[0] : u == 1 ? m[1] : u == 2 ? m[2] : m[3];
    __syncthreads();
    const double ci = pcol[b][i];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double pr = prow[b][j0 + v];
      const double upd = j0 + v == k ? -ci * pr : m[v] - ci * pr;
      m[v] = i == k ? m[v] : upd;
    }
  }
  if (i < n) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j0 + u < n) inv[i * n + j0 + u] = m[u];
  }
}

// Cell index and the neighbour sum of one level; the neighbour order (-x, +x,
// -y, +y, -z, +z) is the same everywhere, so fused and unfused forms of a
// sweep round identically.
__device__ inline int cidx(const MgLevelDev& L, int x, int y, int z) { return x + L.nx * (y + L.ny * z); }

template <class F>
__device__ inline double nb_sum(const MgLevelDev& L, int x, int y, int z, F&& v) {
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  double s = 0.0;
  if (x > 0) s += L.tx[fxi(nx, ny, x, y, z)] * v(x - 1, y, z);
  if (x + 1 < nx) s += L.tx[fxi(nx, ny, x + 1, y, z)] * v(x + 1, y, z);
  if (y > 0) s += L.ty[fyi(nx, ny, x, y, z)] * v(x, y - 1, z);
  if (y + 1 < ny) s += L.ty[fyi(nx, ny, x, y + 1, z)] * v(x, y + 1, z);
  if (z > 0) s += L.tz[fzi(nx, ny, x, y, z)] * v(x, y, z - 1);
  if (z + 1 < nz) s += L.tz[fzi(nx, ny, x, y, z + 1)] * v(x, y, z + 1);
  return s;
}

// Two damped-Jacobi sweeps from zero at one cell: x1 = w b / D,
// x2 = x1 + w (b - A x1) / D.
__device__ inline double sweep2_from_zero(const MgLevelDev& L, const double* __restrict__ b, int x, int y, int z) {
  auto x1 = [&](int xx, int yy, int zz) {
    const int j = cidx(L, xx, yy, zz);
    return kOmega * b[j] / L.diag[j];
  };
  const int i = cidx(L, x, y, z);
  const double D = L.diag[i];
  const double xi = kOmega * b[i] / D;
  return xi + kOmega * (b[i] - D * xi + nb_sum(L, x, y, z, x1)) / D;
}

// Down leg of one level, fused: the two pre-smoothing sweeps (x written for
// the up leg) and the restricted residual b - A x summed over each 2 x 2
// (x 2) aggregate.  One thread per fine cell of a column pair in z; the
// neighbours' sweeps are recomputed, so no grid-wide dependency remains.
// x pairs are adjacent lanes, y pairs adjacent rows of the 64 x 4 block.
__global__ __launch_bounds__(kThreads) void k_mg_down_restrict(MgLevelDev F, MgLevelDev C,
                                                     const double* __restrict__ b, double* __restrict__ xout,
                                                     double* __restrict__ bc, const PcgState* st) {
  if (pcg_done(st)) return;
  const int x = blockIdx.x * kBX + threadIdx.x;
  const int y = blockIdx.y * kBY + threadIdx.y;
  const int Z = blockIdx.z;
  const int z0 = F.nz > 1 ? 2 * Z : 0, z1 = F.nz > 1 ? min(2 * Z + 1, F.nz - 1) : 0;
  double acc = 0.0;
  if (x < F.nx && y < F.ny) {
    auto x2 = [&](int xx, int yy, int zz) { return sweep2_from_zero(F, b, xx, yy, zz); };
    for (int z = z0; z <= z1; ++z) {
      const int i = cidx(F, x, y, z);
      const double xi = x2(x, y, z);
      xout[i] = xi;
      acc += b[i] - F.diag[i] * xi + nb_sum(F, x, y, z, x2);
    }
  }
  acc += __shfl_xor(acc, 1, 64);
  __shared__ double sh[kBY][kBX];
  sh[threadIdx.y][threadIdx.x] = acc;
  __syncthreads();
  if ((threadIdx.x & 1) == 0 && (threadIdx.y & 1) == 0 && x < F.nx && y < F.ny) {
    const int X = x >> 1, Y = y >> 1;
    bc[X + C.nx * (Y + C.ny * Z)] = acc + sh[threadIdx.y + 1][threadIdx.x];
  }
}

// Up leg of one level, fused: coarse correction xc = x + omega_c e[parent],
// one damped-Jacobi sweep y = xc + w (b - A xc) / D, and the last sweep
// out = y + w (b - A y) / D, with the neighbours' y recomputed.  With
// rz_slot >= 0 (the finest level, b = r) also accumulates r . out into the
// CG ring slot.
__global__ __launch_bounds__(kThreads) void k_mg_up_smooth(MgLevelDev F, MgLevelDev C, const double* __restrict__ b,
                                                 const double* __restrict__ xv, const double* __restrict__ ec,
                                                 double omega_c, double* __restrict__ out, PcgState* st,
                                                 int rz_slot) {
  if (pcg_done(st)) return;
  const int x = blockIdx.x * kBX + threadIdx.x;
  const int y = blockIdx.y * kBY + threadIdx.y;
  const int z = blockIdx.z;
  const int cz = F.nz > 1 ? 1 : 0;
  double part = 0.0;
  if (x < F.nx && y < F.ny) {
    auto xc = [&](int xx, int yy, int zz) {
      return xv[cidx(F, xx, yy, zz)] + omega_c * ec[(xx >> 1) + C.nx * ((yy >> 1) + C.ny * (zz >> cz))];
    };
    auto ys = [&](int xx, int yy, int zz) {
      const int j = cidx(F, xx, yy, zz);
      const double D = F.diag[j];
      const double v = xc(xx, yy, zz);
      return v + kOmega * (b[j] - D * v + nb_sum(F, xx, yy, zz, xc)) / D;
    };
    const int i = cidx(F, x, y, z);
    const double D = F.diag[i];
    const double yi = ys(x, y, z);
    const double v = yi + kOmega * (b[i] - D * yi + nb_sum(F, x, y, z, ys)) / D;
    out[i] = v;
    part = b[i] * v;
  }
  if (rz_slot < 0) return;
  part = wave_sum(part);
  __shared__ double sh[kThreads / 64];
  const int t = threadIdx.x + threadIdx.y * kBX;
  if ((t & 63) == 0) sh[t >> 6] = part;
  __syncthreads();
  if (t == 0) {
    const int bid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);  // the block's band
    st->rz[rz_slot * st->nb + bid] = sh[0] + sh[1] + sh[2] + sh[3];
  }
}

constexpr int kTY = 8;  // tile rows of the finest 2D legs

// A 64 x kTY tile covers the 64 x 4 bands (bx, 2 by) and (bx, 2 by + 1) of
// the finest grid: its partial goes to the first, zero to the second.
__device__ inline void tile_band_store(double* slots, int nx, int ny, double v) {
  const int gx = (nx + kBX - 1) / kBX, gyb = (ny + kBY - 1) / kBY;
  const int b0 = blockIdx.x + gx * (2 * blockIdx.y);
  slots[b0] = v;
  if (2 * static_cast<int>(blockIdx.y) + 1 < gyb) slots[b0 + gx] = 0.0;
}

// Operator of a cell: the transmissibilities to its neighbours (0 toward a missing
// one) and the diagonal (1 outside the grid).
struct BoxCell {
  double tw, te, ts, tn, D;
  __device__ inline void load(const MgLevelDev& L, int gx, int gy, bool in) {
    const int nx = L.nx, ny = L.ny;
    tw = in && gx > 0 ? L.tx[fxi(nx, ny, gx, gy, 0)] : 0.0;
    te = in && gx + 1 < nx ? L.tx[fxi(nx, ny, gx + 1, gy, 0)] : 0.0;
    ts = in && gy > 0 ? L.ty[fyi(nx, ny, gx, gy, 0)] : 0.0;
    tn = in && gy + 1 < ny ? L.ty[fyi(nx, ny, gx, gy + 1, 0)] : 0.0;
    D = in ? L.diag[gx + nx * gy] : 1.0;
  }
  __device__ inline double nb(double w, double e, double s, double n) const {
    double v = tw * w;
    v = fma(te, e, v);
    v = fma(ts, s, v);
    return fma(tn, n, v);
  }
};

// ---------------------------------------------------------------------------
// The legs of the finest 2D level, with an iteration of conjugate gradients folded
// in.  A workgroup owns a tile of 64 x 8 cells (one partial of each sum) and holds
// it with a halo of H cells, K cells per thread: operands and iterates in
// registers, the neighbours' iterates from LDS (with a ring of zeros around, double
// buffered: a barrier per sweep; each sweep's outer ring goes wrong by one cell).
//
// On grids of up to 512 x 512 the legs are chains of latencies: launch, one round of
// loads, the sums of the CG step (each on a wavefront of its own), a barrier and a
// division per sweep.  Down / up on 512 x 512: 12.1 / 7.9 us; with four cells a thread on
// 256 threads, the operands in LDS and all sums on one wavefront 15.8 / 11.3.
// ---------------------------------------------------------------------------
template <int H, int NTH>
struct CgBox {
  static constexpr int W = kBX + 2 * H, R = kTY + 2 * H, N = W * R, K = (N + NTH - 1) / NTH;
  typedef double Lds[R + 2][W + 2];
  int lx[K], ly[K], j[K];
  bool in[K], own[K];
  BoxCell q[K];
  __device__ inline void place(const MgLevelDev& F, int x0, int y0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int c = threadIdx.x + k * NTH;
      ly[k] = c / W;
      lx[k] = c - ly[k] * W;
      const int gx = x0 - H + lx[k], gy = y0 - H + ly[k];
      in[k] = c < N && gx >= 0 && gx < F.nx && gy >= 0 && gy < F.ny;
      own[k] = in[k] && lx[k] >= H && lx[k] < H + kBX && ly[k] >= H && ly[k] < H + kTY;
      j[k] = gx + F.nx * gy;
      q[k].load(F, gx, gy, in[k]);
    }
  }
  __device__ inline bool cell(int k) const { return (k + 1) * NTH <= N || static_cast<int>(threadIdx.x) + k * NTH < N; }
  __device__ static inline void ring(Lds& e) {
    for (int i = threadIdx.x; i < W + 2; i += NTH) e[0][i] = e[R + 1][i] = 0.0;
    for (int i = threadIdx.x; i < R + 2; i += NTH) e[i][0] = e[i][W + 1] = 0.0;
  }
  __device__ inline void put(Lds& e, int k, double v) const {
    if (cell(k)) e[ly[k] + 1][lx[k] + 1] = v;
  }
  __device__ inline double nb(const Lds& e, int k) const {
    const int y = cell(k) ? ly[k] + 1 : 1, x = cell(k) ? lx[k] + 1 : 1;
    return q[k].nb(e[y][x - 1], e[y][x + 1], e[y - 1][x], e[y + 1][x]);
  }
  // one sweep: x + om (b - A x) / D
  __device__ inline double sweep(const Lds& e, int k, double b, double x, double om) const {
    return x + om * (fma(-q[k].D, x, b) + nb(e, k)) / q[k].D;
  }
};

// Down leg: NU weighted Jacobi sweeps from zero (the first, x1 = w b / D, needs no
// neighbours), then the restricted residual of the tile's aggregates.  In front,
// iteration it of Chronopoulos-Gear conjugate gradients (one reduction phase per
// iteration): from the slot sums of the previous leg pair the stop test on ||r_it||,
// then beta = g_it / g_{it-1}, alpha = g_it / (d_it - beta g_it / alpha_{it-1}) with
// g = r.z, d = w.z, w = A z (alpha = g_0 / d_0, beta = 0 at it = 0); s = w + beta
// s_old and r_new = r - alpha s on the box (the halo values recomputed, the tile's
// written); p = z + beta p and x += alpha p on the tile; the partial sum of
// r_new . r_new.
template <int NU>
__global__ __launch_bounds__(1024) void k_mg_down_cg(MgLevelDev F, MgLevelDev C, const double* __restrict__ b,
                                           double* __restrict__ xout, double* __restrict__ bc, PcgState* st,
                                           CgFuse cg) {
  static_assert(NU >= 2, "two sweeps at least");
  typedef CgBox<NU, 1024> Box;
  static_assert(Box::K == 1, "a cell per thread");
  const bool stop = pcg_done(st);
  __shared__ typename Box::Lds e[2];
  __shared__ double srn[kTY][kBX];
  __shared__ double sums[5], alpha_sh, beta_sh, sh[kTY / 2];
  __shared__ int stop_sh;
  const int nx = F.nx, ny = F.ny;
  const int tile = xcd_tile_id();  // 2D grid: tile = bx + gridDim.x * by
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int it = cg.it;
  // every load first
  Box B;
  B.place(F, (tile % gridDim.x) * kBX, (tile / gridDim.x) * kTY);
  const int j = B.j[0];
  const bool in = B.in[0], own = B.own[0];
  const double rb = in ? b[j] : 0.0, rw = in ? cg.w[j] : 0.0, rs = in && it > 0 ? cg.s_old[j] : 0.0;
  const double xo = own ? cg.x[j] : 0.0, zo = own ? cg.z[j] : 0.0, po = own && it > 0 ? cg.p[j] : 0.0;
  Box::ring(e[0]);
  Box::ring(e[1]);
  if (wave < 5) {
    const int nb = st->nb;
    const double* src = wave == 0   ? st->rr + (it & 3) * nb
                        : wave == 1 ? st->bb_sl
                        : wave == 2 ? st->rz + (it & 3) * nb
                        : wave == 3 ? st->wz + (it & 3) * nb
                                    : st->rz + ((it - 1) & 3) * nb;
    const double v = wave == 4 && it == 0 ? 1.0 : wave_part_sum(src, nb);
    if (lane == 0) sums[wave] = v;
  }
  if (tid < kTY * kBX) srn[tid / kBX][tid % kBX] = 0.0;
  __syncthreads();
  if (tid < 64) {  // the first wavefront decides for the block
    int halt = stop ? 1 : 0;
    double alpha = 0.0, beta = 0.0;
    const double rr = sums[0], bb = sums[1], g1 = sums[2], d1 = sums[3], g0 = sums[4];
    const bool lead = tile == 0;
    if (halt) {
      // an earlier iteration converged
    } else if (!isfinite(rr)) {
      halt = 1;
      if (lead && tid == 0) { st->nonfinite = 1; st->done = 1; st->it_done = it; }
    } else if (rr <= st->tol2 * bb) {
      halt = 1;
      if (lead && tid == 0) { st->done = 1; st->it_done = it; st->bb = bb; }
    } else if (it > 0) {
      beta = g1 / g0;
      alpha = g1 / (d1 - beta * g1 / st->alpha[(it - 1) & 3]);
    } else {
      alpha = g1 / d1;
    }
    if (tid == 0) {
      stop_sh = halt;
      alpha_sh = alpha;
      beta_sh = beta;
    }
    if (!halt && lead && tid == 0) st->alpha[it & 3] = alpha;
  }
  // the first tile may set the stop flag while this kernel runs, so every
  // wavefront follows the first one's decision, not its own read
  __syncthreads();
  if (stop_sh) return;
  const double alpha = alpha_sh, beta = beta_sh;
  const double sv = fma(beta, rs, rw);  // zero outside the grid stays zero
  const double rn = fma(-alpha, sv, rb);
  double x = sweep_weight<NU>(0) * rn / B.q[0].D;  // first sweep from zero
  B.put(e[0], 0, x);
  if (own) {
    const double pn = fma(beta, po, zo);
    cg.r_new[j] = rn;
    cg.s_new[j] = sv;
    cg.p[j] = pn;
    cg.x[j] = fma(alpha, pn, xo);
    srn[B.ly[0] - NU][B.lx[0] - NU] = rn;
  }
  __syncthreads();
  if (wave < kTY / 2) {
    const double r0 = srn[2 * wave][lane], r1 = srn[2 * wave + 1][lane];
    const double v = wave_sum(fma(r1, r1, r0 * r0));
    if (lane == 0) sh[wave] = v;
  }
#pragma unroll
  for (int k = 2; k <= NU; ++k) {
    x = B.sweep(e[k & 1], 0, rn, x, sweep_weight<NU>(k - 1));
    B.put(e[(k - 1) & 1], 0, x);
    __syncthreads();
  }
  if (tid == 0) tile_band_store(st->rr + ((it + 1) & 3) * st->nb, nx, ny, sh[0] + sh[1] + sh[2] + sh[3]);
  const double res = fma(-B.q[0].D, x, rn) + B.nb(e[(NU - 1) & 1], 0);
  if (own) xout[j] = x;
  typename Box::Lds& er = e[NU & 1];
  B.put(er, 0, own ? res : 0.0);
  __syncthreads();
  const int lx = B.lx[0], ly = B.ly[0];
  if (own && ((lx - NU) & 1) == 0 && ((ly - NU) & 1) == 0) {
    const int gx = (tile % gridDim.x) * kBX + lx - NU, gy = (tile / gridDim.x) * kTY + ly - NU;
    bc[(gx >> 1) + C.nx * (gy >> 1)] =
        (res + er[ly + 2][lx + 1]) + (er[ly + 1][lx + 2] + er[ly + 2][lx + 2]);
  }
}

// Up leg: the coarse correction v = x + w_c e[parent] on the box, then NU weighted
// Jacobi sweeps; the last covers the tile (out = z) and the ring around it, so that
// w = A z follows on the tile (w_out); the partial sums of r.z and w.z go to the
// ring slot.
template <int NU>
__global__ __launch_bounds__(576) void k_mg_up_cg(MgLevelDev F, MgLevelDev C, const double* __restrict__ b,
                                        const double* __restrict__ xv, const double* __restrict__ ec,
                                        double omega_c, double* __restrict__ out, double* __restrict__ w_out,
                                        PcgState* st, int rz_slot) {
  typedef CgBox<NU + 1, 576> Box;
  constexpr int K = Box::K, H = NU + 1;
  const bool stop = pcg_done(st);
  __shared__ typename Box::Lds e[2];
  __shared__ double sb[kTY][kBX], sz[kTY][kBX], sw[kTY][kBX], sh[2][kTY / 2];
  const int nx = F.nx, ny = F.ny;
  const int tile = xcd_tile_id();  // 2D grid: tile = bx + gridDim.x * by
  const int x0 = (tile % gridDim.x) * kBX, y0 = (tile / gridDim.x) * kTY;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Box B;
  B.place(F, x0, y0);
  double x[K], rb[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int gx = x0 - H + B.lx[k], gy = y0 - H + B.ly[k];
    const double xi = B.in[k] ? xv[B.j[k]] : 0.0, ei = B.in[k] ? ec[(gx >> 1) + C.nx * (gy >> 1)] : 0.0;
    rb[k] = B.in[k] ? b[B.j[k]] : 0.0;
    x[k] = fma(omega_c, ei, xi);
  }
  Box::ring(e[0]);
  Box::ring(e[1]);
  for (int i = tid; i < kTY * kBX; i += 576) (&sb[0][0])[i] = (&sz[0][0])[i] = (&sw[0][0])[i] = 0.0;
  if (stop) return;
#pragma unroll
  for (int k = 0; k < K; ++k) B.put(e[0], k, x[k]);
  __syncthreads();
#pragma unroll
  for (int t = 1; t <= NU; ++t) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      x[k] = B.sweep(e[(t - 1) & 1], k, rb[k], x[k], sweep_weight<NU>(NU - t));
      B.put(e[t & 1], k, x[k]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double w = fma(B.q[k].D, x[k], -B.nb(e[NU & 1], k));
    if (!B.own[k]) continue;
    out[B.j[k]] = x[k];
    w_out[B.j[k]] = w;
    const int y = B.ly[k] - H, c = B.lx[k] - H;
    sb[y][c] = rb[k];
    sz[y][c] = x[k];
    sw[y][c] = w;
  }
  __syncthreads();
  if (wave < kTY / 2) {
    const int y = 2 * wave;
    const double z0 = sz[y][lane], z1 = sz[y + 1][lane];
    const double g = wave_sum(fma(sb[y + 1][lane], z1, sb[y][lane] * z0));
    const double dz = wave_sum(fma(sw[y + 1][lane], z1, sw[y][lane] * z0));
    if (lane == 0) {
      sh[0][wave] = g;
      sh[1][wave] = dz;
    }
  }
  __syncthreads();
  if (tid == 0) {
    tile_band_store(st->rz + rz_slot * st->nb, nx, ny, sh[0][0] + sh[0][1] + sh[0][2] + sh[0][3]);
    tile_band_store(st->wz + rz_slot * st->nb, nx, ny, sh[1][0] + sh[1][1] + sh[1][2] + sh[1][3]);
  }
}

// ---------------------------------------------------------------------------
// The legs of 2D levels without conjugate-gradient work: a workgroup of 1024
// threads holds a box of 64 x 16 cells, one per thread, a wavefront per row: its
// tile plus a halo of H = NU cells, so that every sweep needs only what the box
// holds (each sweep's outer ring goes wrong by one cell).  Operands and iterate
// stay in registers, the x neighbours come from the next lanes by DPP, the y
// neighbours from LDS (double buffered: a barrier per sweep).  The operations are
// those of the finest legs, one by one and in their order.
//
// On such levels a leg is a chain of latencies (launch, one round of loads, a
// barrier and a division per sweep): a down / up leg of 256 x 256 and 128 x 128
// takes 4.0 / 4.2 us where tiles of 64 x 8 on 256 threads, four cells a thread with
// their operands in LDS, took 6.7 / 7.1.
// ---------------------------------------------------------------------------
constexpr int kBoxR = 16;           // box rows (64 columns wide)
constexpr int kBoxT = kBX * kBoxR;  // threads

// West / east neighbour's value (0 past the wavefront's ends): wavefront shifts.
__device__ inline double box_w(double v) { return dpp<0x138>(v); }
__device__ inline double box_e(double v) { return dpp<0x130>(v); }

// b - A v at the thread's cell; col: the LDS rows, stored one down.
__device__ inline double box_residual(const BoxCell& q, double b, double v, const double (*col)[kBX], int row, int lane) {
  return fma(-q.D, v, b) + q.nb(box_w(v), box_e(v), col[row][lane], col[row + 2][lane]);
}

// Down leg: NU weighted Jacobi sweeps from zero, then the restricted residual of
// the tile's aggregates.
template <int NU>
__global__ __launch_bounds__(kBoxT) void k_mg_down_box(MgLevelDev F, MgLevelDev C, const double* __restrict__ b,
                                            double* __restrict__ xout, double* __restrict__ bc, const PcgState* st) {
  constexpr int H = NU, TX = kBX - 2 * H, TR = kBoxR - 2 * H;
  static_assert(TX % 2 == 0 && TR % 2 == 0, "whole aggregates");
  const bool stop = pcg_done(st);
  __shared__ double e[2][kBoxR + 2][kBX];
  const int nx = F.nx, ny = F.ny;
  const int lane = threadIdx.x & 63, row = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_x = (nx + TX - 1) / TX;
  const int tile = xcd_tile_id();
  const int gx = (tile % tiles_x) * TX - H + lane, gy = (tile / tiles_x) * TR - H + row;
  const bool in = gx >= 0 && gx < nx && gy >= 0 && gy < ny;
  const bool own = in && lane >= H && lane < H + TX && row >= H && row < H + TR;
  const int j = gx + nx * gy;
  const double bi = in ? b[j] : 0.0;
  BoxCell q;
  q.load(F, gx, gy, in);
  if (row == 0 || row == kBoxR - 1) {  // rows beside the box
    const int r = row == 0 ? 0 : kBoxR + 1;
    e[0][r][lane] = e[1][r][lane] = 0.0;
  }
  if (stop) return;
  double x = sweep_weight<NU>(0) * bi / q.D;  // first sweep from zero
  e[0][row + 1][lane] = x;
  __syncthreads();
#pragma unroll
  for (int k = 1; k < NU; ++k) {
    x = x + sweep_weight<NU>(k) * box_residual(q, bi, x, e[(k - 1) & 1], row, lane) / q.D;
    e[k & 1][row + 1][lane] = x;
    __syncthreads();
  }
  double res = box_residual(q, bi, x, e[(NU - 1) & 1], row, lane);
  if (own) xout[j] = x;
  else res = 0.0;
  e[NU & 1][row + 1][lane] = res;
  __syncthreads();
  // aggregates start at even cells: lanes and rows at an even distance from H
  const double pair = res + e[NU & 1][row + 2][lane];
  const double sum = pair + box_e(pair);
  if (own && ((lane - H) & 1) == 0 && ((row - H) & 1) == 0) bc[(gx >> 1) + C.nx * (gy >> 1)] = sum;
}

// Up leg: the coarse correction v = x + w_c e[parent] on the box, then NU weighted
// Jacobi sweeps.
template <int NU>
__global__ __launch_bounds__(kBoxT) void k_mg_up_box(MgLevelDev F, MgLevelDev C, const double* __restrict__ b,
                                          const double* __restrict__ xv, const double* __restrict__ ec,
                                          double omega_c, double* __restrict__ out, const PcgState* st) {
  constexpr int H = NU, TX = kBX - 2 * H, TR = kBoxR - 2 * H;
  const bool stop = pcg_done(st);
  __shared__ double e[2][kBoxR + 2][kBX];
  const int nx = F.nx, ny = F.ny;
  const int lane = threadIdx.x & 63, row = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_x = (nx + TX - 1) / TX;
  const int tile = xcd_tile_id();
  const int gx = (tile % tiles_x) * TX - H + lane, gy = (tile / tiles_x) * TR - H + row;
  const bool in = gx >= 0 && gx < nx && gy >= 0 && gy < ny;
  const bool own = in && lane >= H && lane < H + TX && row >= H && row < H + TR;
  const int j = gx + nx * gy;
  const double xi = in ? xv[j] : 0.0, ei = in ? ec[(gx >> 1) + C.nx * (gy >> 1)] : 0.0;
  const double bi = in ? b[j] : 0.0;
  BoxCell q;
  q.load(F, gx, gy, in);
  if (row == 0 || row == kBoxR - 1) {
    const int r = row == 0 ? 0 : kBoxR + 1;
    e[0][r][lane] = e[1][r][lane] = 0.0;
  }
  double x = fma(omega_c, ei, xi);
  e[0][row + 1][lane] = x;
  if (stop) return;
  __syncthreads();
#pragma unroll
  for (int k = 1; k <= NU; ++k) {
    x = x + sweep_weight<NU>(NU - k) * box_residual(q, bi, x, e[(k - 1) & 1], row, lane) / q.D;
    if (k < NU) {
      e[k & 1][row + 1][lane] = x;
      __syncthreads();
    }
  }
  if (own) out[j] = x;
}

// Workgroups of the box legs.
dim3 box_grid(const MgLevelDev& L) {
  const int tx = kBX - 2 * kMgSweeps, tr = kBoxR - 2 * kMgSweeps;
  return dim3(((L.nx + tx - 1) / tx) * ((L.ny + tr - 1) / tr));
}

// ---------------------------------------------------------------------------
// Coarse levels in one workgroup, everything in LDS: a.ncyc V-cycles over
// the levels first..bottom-1 with the exact dense solve on the bottom level,
// from x = 0, on rhs b (global).  Writes x to out; with rz_slot >= 0 also
// b . out into the CG ring.  LDS per smoothed level: faces, diagonal, its
// inverse and three vectors; bottom: two vectors, the partial products of
// the dense solve and the inverse.
// ---------------------------------------------------------------------------
struct LdsLevel {
  double *tx, *ty, *tz, *diag, *B, *E, *T, *dinv;
};

__device__ inline void lds_level(const MgCoarseArgs& a, double* smem, int l, LdsLevel& S) {
  S.tx = smem + a.off[l][0];
  S.ty = smem + a.off[l][1];
  S.tz = smem + a.off[l][2];
  S.diag = smem + a.off[l][3];
  S.B = smem + a.off[l][4];
  S.E = smem + a.off[l][5];
  S.T = smem + a.off[l][6];
  S.dinv = smem + a.off[l][7];
}

// (x, y, z) of cell c of a level
__device__ inline void cell_xyz(const MgLevelDev& L, int c, int& x, int& y, int& z) {
  if (L.nz == 1) {
    y = c / L.nx;
    x = c - y * L.nx;
    z = 0;
  } else {
    const int pl = L.nx * L.ny;
    z = c / pl;
    const int r = c - z * pl;
    y = r / L.nx;
    x = r - y * L.nx;
  }
}

// Neighbour sum of cell c of an LDS level with values v(j, x, y, z) of the
// neighbour j at (x, y, z).  Every face index is valid (boundary faces are
// stored); a missing neighbour is replaced by the cell itself and its term
// dropped by a select, so all loads issue without branches and wait once.
template <class V>
__device__ inline double lds_nb_sum(const MgLevelDev& L, const LdsLevel& S, int x, int y, int z, int c, V&& v) {
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  const bool hw = x > 0, he = x + 1 < nx, hs = y > 0, hn = y + 1 < ny;
  const double tw = S.tx[fxi(nx, ny, x, y, z)], te = S.tx[fxi(nx, ny, x + 1, y, z)];
  const double ts = S.ty[fyi(nx, ny, x, y, z)], tn = S.ty[fyi(nx, ny, x, y + 1, z)];
  const double vw = v(hw ? c - 1 : c, hw ? x - 1 : x, y, z);
  const double ve = v(he ? c + 1 : c, he ? x + 1 : x, y, z);
  const double vs = v(hs ? c - nx : c, x, hs ? y - 1 : y, z);
  const double vn = v(hn ? c + nx : c, x, hn ? y + 1 : y, z);
  double s = (hw ? tw * vw : 0.0) + (he ? te * ve : 0.0) + (hs ? ts * vs : 0.0) + (hn ? tn * vn : 0.0);
  if (nz > 1) {  // uniform: 2D levels keep no z faces in LDS
    const bool hb = z > 0, ht = z + 1 < nz;
    const double tb = S.tz[fzi(nx, ny, x, y, z)], tt = S.tz[fzi(nx, ny, x, y, z + 1)];
    const double vb = v(hb ? c - nx * ny : c, x, y, hb ? z - 1 : z);
    const double vt = v(ht ? c + nx * ny : c, x, y, ht ? z + 1 : z);
    s += (hb ? tb * vb : 0.0) + (ht ? tt * vt : 0.0);
  }
  return s;
}

// One smoothed level's faces and diagonal (and 1/diagonal) into LDS, every
// load issued before the first store.  Two face values and one diagonal
// value per thread cover the level: it has at most blockDim cells and at
// most twice as many faces per direction.
__device__ inline void lds_load_level(const MgLevelDev& L, const LdsLevel& S) {
  const int bd = blockDim.x, t = threadIdx.x;
  const int n = L.nx * L.ny * L.nz;
  const int nfx = (L.nx + 1) * L.ny * L.nz, nfy = L.nx * (L.ny + 1) * L.nz;
  const int nfz = L.nz > 1 ? L.nx * L.ny * (L.nz + 1) : 0;  // 2D: z faces never read
  double fx[2], fy[2], fz[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int j = t + u * bd;
    fx[u] = j < nfx ? L.tx[j] : 0.0;
    fy[u] = j < nfy ? L.ty[j] : 0.0;
    fz[u] = j < nfz ? L.tz[j] : 0.0;
  }
  const double dg = t < n ? L.diag[t] : 1.0;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int j = t + u * bd;
    if (j < nfx) S.tx[j] = fx[u];
    if (j < nfy) S.ty[j] = fy[u];
    if (j < nfz) S.tz[j] = fz[u];
  }
  if (t < n) {
    S.diag[t] = dg;
    S.dinv[t] = 1.0 / dg;  // the sweeps multiply; one division per cell here
  }
}

// Phases of the LDS levels; each ends with a barrier.
// Down leg of level l: two damped-Jacobi sweeps from zero in one pass (E = x2,
// the first sweep's x1 = w B / D recomputed at the neighbours), then the
// restricted residual into the B of level l + 1: the sum over the (up to)
// 2 x 2 (x 2) fine cells of each coarse cell, a fine index past the edge
// clamped and its term dropped.
// One damped-Jacobi sweep of an LDS level from xin into xo (different arrays).
__device__ inline void lds_sweep(const MgLevelDev& F, const LdsLevel& S, const double* xin, double* xo) {
  const int bd = blockDim.x, t = threadIdx.x;
  const int n = F.nx * F.ny * F.nz;
  auto xv = [&](int j, int, int, int) { return xin[j]; };
  for (int c = t; c < n; c += bd) {
    int x, y, z;
    cell_xyz(F, c, x, y, z);
    const double di = S.dinv[c];
    const double v = xin[c];
    xo[c] = v + kOmega * ((S.B[c] + lds_nb_sum(F, S, x, y, z, c, xv)) * di - v);
  }
  __syncthreads();
}

__device__ inline void lds_down(const MgCoarseArgs& a, double* smem, int l) {
  const int bd = blockDim.x, t = threadIdx.x;
  const MgLevelDev& F = a.lev[l];
  const MgLevelDev& C = a.lev[l + 1];
  LdsLevel S, SC;
  lds_level(a, smem, l, S);
  lds_level(a, smem, l + 1, SC);
  {
    const int n = F.nx * F.ny * F.nz;
    auto x1 = [&](int j, int, int, int) { return kOmega * S.B[j] * S.dinv[j]; };
    for (int c = t; c < n; c += bd) {
      int x, y, z;
      cell_xyz(F, c, x, y, z);
      const double di = S.dinv[c];
      const double bi = S.B[c];
      const double xi = kOmega * bi * di;
      S.E[c] = xi + kOmega * ((bi + lds_nb_sum(F, S, x, y, z, c, x1)) * di - xi);
    }
    __syncthreads();
  }
  for (int k = 2; k < kMgLdsSweeps; k += 2) {  // further sweeps in pairs, ending in E
    lds_sweep(F, S, S.E, S.T);
    lds_sweep(F, S, S.T, S.E);
  }
  const int nc = C.nx * C.ny * C.nz;
  auto ev = [&](int j, int, int, int) { return S.E[j]; };
  auto res = [&](int x, int y, int z) {
    const int i = x + F.nx * (y + F.ny * z);
    return S.B[i] - S.diag[i] * S.E[i] + lds_nb_sum(F, S, x, y, z, i, ev);
  };
  for (int c = t; c < nc; c += bd) {
    int X0, Y0, Z0;
    cell_xyz(C, c, X0, Y0, Z0);
    const int x0 = 2 * X0, y0 = 2 * Y0;
    const bool hx = x0 + 1 < F.nx, hy = y0 + 1 < F.ny;
    const int x1 = hx ? x0 + 1 : x0, y1 = hy ? y0 + 1 : y0;
    double acc;
    if (F.nz > 1) {
      const int z0 = 2 * Z0;
      const bool hz = z0 + 1 < F.nz;
      const int z1 = hz ? z0 + 1 : z0;
      const double r000 = res(x0, y0, z0), r100 = res(x1, y0, z0), r010 = res(x0, y1, z0), r110 = res(x1, y1, z0);
      const double r001 = res(x0, y0, z1), r101 = res(x1, y0, z1), r011 = res(x0, y1, z1), r111 = res(x1, y1, z1);
      acc = r000 + (hx ? r100 : 0.0) + (hy ? r010 : 0.0) + (hx && hy ? r110 : 0.0);
      if (hz) acc += r001 + (hx ? r101 : 0.0) + (hy ? r011 : 0.0) + (hx && hy ? r111 : 0.0);
    } else {
      const double r00 = res(x0, y0, 0), r10 = res(x1, y0, 0), r01 = res(x0, y1, 0), r11 = res(x1, y1, 0);
      acc = r00 + (hx ? r10 : 0.0) + (hy ? r01 : 0.0) + (hx && hy ? r11 : 0.0);
    }
    SC.B[c] = acc;
  }
  __syncthreads();
}

// Up leg of level l: coarse correction folded into the first sweep,
// T = y(E + w_c e[parent]), then E = T + w (B - A T) / D.
__device__ inline void lds_up(const MgCoarseArgs& a, double* smem, int l) {
  const int bd = blockDim.x, t = threadIdx.x;
  const MgLevelDev& F = a.lev[l];
  const MgLevelDev& C = a.lev[l + 1];
  LdsLevel S, SC;
  lds_level(a, smem, l, S);
  lds_level(a, smem, l + 1, SC);
  const int n = F.nx * F.ny * F.nz;
  const int cz = F.nz > 1 ? 1 : 0;
  auto xc = [&](int j, int x, int y, int z) {
    return S.E[j] + a.omega_c * SC.E[(x >> 1) + C.nx * ((y >> 1) + C.ny * (z >> cz))];
  };
  for (int c = t; c < n; c += bd) {
    int x, y, z;
    cell_xyz(F, c, x, y, z);
    const double di = S.dinv[c];
    const double v = xc(c, x, y, z);
    S.T[c] = v + kOmega * ((S.B[c] + lds_nb_sum(F, S, x, y, z, c, xc)) * di - v);
  }
  __syncthreads();
  lds_sweep(F, S, S.T, S.E);
  for (int k = 2; k < kMgLdsSweeps; k += 2) {  // further sweeps in pairs, ending in E
    lds_sweep(F, S, S.E, S.T);
    lds_sweep(F, S, S.T, S.E);
  }
}

// Bottom: E = inverse * B, the columns split over the wavefronts (partial
// products in T), then summed per row.  The inverse of the symmetric bottom
// operator is symmetric: it is read by columns so that consecutive threads
// hit consecutive banks.
__device__ inline void lds_bottom(const MgCoarseArgs& a, double* smem, const double* Binv, int nb) {
  const int bd = blockDim.x, t = threadIdx.x;
  LdsLevel S;
  lds_level(a, smem, a.nlev - 1, S);
  const int groups = (bd + 63) >> 6;
  const int chunk = (nb + groups - 1) / groups;
  const int r = t & 63, g = t >> 6;
  if (r < nb) {
    const int j0 = g * chunk, j1 = min(nb, j0 + chunk);
    double acc = 0.0;
    for (int j = j0; j < j1; ++j) acc += Binv[j * nb + r] * S.B[j];
    S.T[g * nb + r] = acc;
  }
  __syncthreads();
  if (t < nb) {
    double acc = 0.0;
    for (int k = 0; k < groups; ++k) acc += S.T[k * nb + t];
    S.E[t] = acc;
  }
  __syncthreads();
}

// Residual of level l for the correction so far: B <- B - A E (in place: a
// cell writes only its own B, the neighbours' E are only read).  Thread t
// owns cell t (the level has at most blockDim cells); returns E of that cell.
__device__ inline double lds_residual(const MgCoarseArgs& a, double* smem, int l) {
  const int t = threadIdx.x;
  const MgLevelDev& F = a.lev[l];
  LdsLevel S;
  lds_level(a, smem, l, S);
  const int n = F.nx * F.ny * F.nz;
  double e = 0.0;
  if (t < n) {
    auto ev = [&](int j, int, int, int) { return S.E[j]; };
    int x, y, z;
    cell_xyz(F, t, x, y, z);
    e = S.E[t];
    S.B[t] += lds_nb_sum(F, S, x, y, z, t, ev) - S.diag[t] * e;
  }
  __syncthreads();
  return e;
}

// Coarse levels in one workgroup, everything in LDS: a.ncyc cycles on the
// first level; inside each, the coarse problem of the second level is solved
// by a.ncyc1 V-cycles over the levels below it (a W-shaped cycle with two
// visits under the first level), with the exact dense solve on the bottom
// level.  Later cycles on a level start from the residual the earlier ones
// left, and the corrections add up.  From x = 0, on rhs b (global); writes x
// to out; with rz_slot >= 0 also b . out into the CG ring.
__global__ __launch_bounds__(1024) void k_mg_coarse_lds(MgCoarseArgs a, const double* __restrict__ bglob,
                                              const double* __restrict__ binv, double* __restrict__ out,
                                              PcgState* st, int rz_slot) {
  const bool stop = pcg_done(st);  // checked once the level loads are in flight
  extern __shared__ double smem[];
  const int nl = a.nlev;          // levels in LDS, the last one is the bottom
  const int bd = blockDim.x, t = threadIdx.x;
  LdsLevel S0;
  lds_level(a, smem, 0, S0);
  const int n0 = a.n0;
  const double b0 = t < n0 ? bglob[t] : 0.0;
  // faces / diagonals of the smoothed levels, the bottom inverse, the rhs
  for (int l = 0; l + 1 < nl; ++l) {
    LdsLevel S;
    lds_level(a, smem, l, S);
    lds_load_level(a.lev[l], S);
  }
  const MgLevelDev& Lb = a.lev[nl - 1];
  const int nb = Lb.nx * Lb.ny * Lb.nz;
  double* Binv = smem + a.inv_off;
  for (int j0 = 0; j0 < nb * nb; j0 += 4 * bd) {
    double r[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + t + u * bd;
      r[u] = j < nb * nb ? binv[j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + t + u * bd;
      if (j < nb * nb) Binv[j] = r[u];
    }
  }
  if (t < n0) S0.B[t] = b0;
  if (stop) return;
  __syncthreads();
  double x0 = 0.0;  // accumulated correction of the first level, cell t
  for (int cyc = 0; cyc < a.ncyc; ++cyc) {
    if (cyc > 0) x0 += lds_residual(a, smem, 0);
    if (nl == 1) {
      lds_bottom(a, smem, Binv, nb);
      continue;
    }
    lds_down(a, smem, 0);
    double x1 = 0.0;  // accumulated correction of the second level, cell t
    for (int c1 = 0; c1 < a.ncyc1; ++c1) {
      if (c1 > 0) x1 += lds_residual(a, smem, 1);
      for (int l = 1; l + 1 < nl; ++l) lds_down(a, smem, l);
      lds_bottom(a, smem, Binv, nb);
      for (int l = nl - 2; l >= 1; --l) lds_up(a, smem, l);
    }
    if (a.ncyc1 > 1) {
      LdsLevel S1;
      lds_level(a, smem, 1, S1);
      const MgLevelDev& L1 = a.lev[1];
      if (t < L1.nx * L1.ny * L1.nz) S1.E[t] += x1;
      __syncthreads();
    }
    lds_up(a, smem, 0);
  }
  double part = 0.0;
  if (t < n0) {
    const double v = x0 + S0.E[t];
    out[t] = v;
    part = b0 * v;
  }
  if (rz_slot < 0) return;
  part = wave_sum(part);
  __shared__ double sh[16];
  if ((t & 63) == 0) sh[t >> 6] = part;
  __syncthreads();
  // the whole grid is this workgroup's: its sum in the first band's slot,
  // zeros in the others
  double* slots = st->rz + rz_slot * st->nb;
  for (int k = t + 1; k < st->nb; k += bd) slots[k] = 0.0;
  if (t == 0) {
    double s = 0.0;
    for (int w = 0; w < (bd + 63) / 64; ++w) s += sh[w];
    slots[0] = s;
  }
}

// ---------------------------------------------------------------------------
// The coarse solve of 2D hierarchies with two smoothed LDS levels above the
// bottom: the cycles of k_mg_coarse_lds, the
// same operations in the same order, with the operands in registers.  A thread owns
// cell t of each level; only the iterates that neighbours read go through LDS, so a
// sweep is four LDS reads, some ten operations, one LDS write and a barrier, with no
// division of the cell index.
//
// Bound by its chain of some 50 barriered phases: 11.8 us for 32 x 32 and two levels
// below, where k_mg_coarse_lds takes 23.8.  Grids whose halving passes the 1024
// cells high and the 64 low (33 x 29, 17 x 15, 9 x 8, 5 x 4: some 5% of the
// rectangles of 48 to 512 cells a side, 300 x 200 and 600 x 400 among them) have
// three smoothed levels and keep k_mg_coarse_lds, as thin strips do.
// ---------------------------------------------------------------------------
struct CoarseCell {
  double tw, te, ts, tn;  // transmissibilities, zero toward a missing neighbour
  double D, di;           // diagonal, its inverse
  double B, e;            // right-hand side, iterate
};

// Cell c of a level (a cell past its end: all zero, D = 1).
__device__ inline void coarse_load(const MgLevelDev& L, int c, CoarseCell& q) {
  const int nx = L.nx, ny = L.ny;
  const bool in = c < nx * ny;
  const int cc = in ? c : 0;
  const int y = cc / nx, x = cc - y * nx;
  const double tw = L.tx[fxi(nx, ny, x, y, 0)], te = L.tx[fxi(nx, ny, x + 1, y, 0)];
  const double ts = L.ty[fyi(nx, ny, x, y, 0)], tn = L.ty[fyi(nx, ny, x, y + 1, 0)];
  const double D = L.diag[cc];
  q.D = in ? D : 1.0;
  q.tw = in && x > 0 ? tw : 0.0;
  q.te = in && x + 1 < nx ? te : 0.0;
  q.ts = in && y > 0 ? ts : 0.0;
  q.tn = in && y + 1 < ny ? tn : 0.0;
  q.B = q.e = 0.0;
}

__device__ inline int coarse_parent(const MgLevelDev& F, const MgLevelDev& C, int c) {
  const int y = c / F.nx, x = c - y * F.nx;
  return (x >> 1) + C.nx * (y >> 1);
}

// sum t v_nb, v at the cell in a padded LDS array: a missing neighbour reads some
// other entry or the padding and multiplies it by zero.  Each product is rounded
// before the sum, as in lds_nb_sum.
__device__ inline double coarse_nb(const CoarseCell& q, const double* v, int nx) {
#pragma clang fp contract(off)
  const double w = q.tw * v[-1], e = q.te * v[1], s = q.ts * v[-nx], n = q.tn * v[nx];
  return w + e + s + n;
}

// One sweep, and B - A v.
__device__ inline double coarse_sweep(const CoarseCell& q, const double* v, int nx) {
  return fma(kOmega, fma(q.B + coarse_nb(q, v, nx), q.di, -q.e), q.e);
}
__device__ inline double coarse_res(const CoarseCell& q, const double* v, int nx) {
  return fma(-q.D, q.e, q.B) + coarse_nb(q, v, nx);
}

// Sum of the residuals of the (up to) 2 x 2 children of coarse cell (X, Y).
__device__ inline double coarse_children(const double* r, int fnx, int fny, int X, int Y) {
  const int x0 = 2 * X, y0 = 2 * Y;
  const bool hx = x0 + 1 < fnx, hy = y0 + 1 < fny;
  const int i = x0 + fnx * y0;
  const double r00 = r[i], r10 = r[hx ? i + 1 : i], r01 = r[hy ? i + fnx : i], r11 = r[hx && hy ? i + fnx + 1 : i];
  return r00 + (hx ? r10 : 0.0) + (hy ? r01 : 0.0) + (hx && hy ? r11 : 0.0);
}

// One double-buffered iterate of a level in LDS: a phase reads cur and writes
// oth; turn() makes the written one current.
struct CoarseBuf {
  double *cur, *oth;
  __device__ inline void turn() {
    __syncthreads();
    double* t = cur;
    cur = oth;
    oth = t;
  }
};

__global__ __launch_bounds__(kMgLdsCells) void k_mg_coarse_2d(MgCoarseArgs a, const double* __restrict__ bglob,
                                                    const double* __restrict__ binv, double* __restrict__ out,
                                                    PcgState* st, int rz_slot) {
  constexpr int S = kMgLdsCells;
  static_assert(kMgLdsSweeps == 2, "two sweeps each way");
  const bool stop = pcg_done(st);
  extern __shared__ double smem[];
  const int t = threadIdx.x;
  const MgLevelDev &L0 = a.lev[0], &L1 = a.lev[1], &L2 = a.lev[2];
  const int n0 = L0.nx * L0.ny, n1 = L1.nx * L1.ny, n2 = L2.nx * L2.ny;
  const bool on0 = t < n0, on1 = t < n1, on2 = t < n2;
  const int nx0 = L0.nx, nx1 = L1.nx;
  // LDS: the buffers (pointers to the thread's own cell), the residuals of level 0
  // and then of level 1, the bottom's right-hand side, solution, partial products
  // and inverse
  CoarseBuf b0, b1;
  double* p = smem;
  auto take = [&](int cells, int pad) {
    double* r = p + pad + t;
    p += cells + 2 * pad;
    return r;
  };
  b0.cur = take(S, kMgPad0);
  b0.oth = take(S, kMgPad0);
  b1.cur = take(S, kMgPad0);
  b1.oth = take(S, kMgPad0);
  double* rc = take(S, 0) - t;
  double* bc = take(kMgBottomCells, 0) - t;
  double* ebot = take(kMgBottomCells, 0) - t;
  double* parts = take(S, 0) - t;
  const double* zeroed = p;
  double* inv = take(kMgBottomCells * kMgBottomCells, 0) - t;
  // loads first
  CoarseCell c0, c1;
  coarse_load(L0, t, c0);
  coarse_load(L1, t, c1);
  constexpr int NI = kMgBottomCells * kMgBottomCells / S;
  double vi[NI];
#pragma unroll
  for (int k = 0; k < NI; ++k) vi[k] = t + k * S < n2 * n2 ? binv[t + k * S] : 0.0;
  const double bin = on0 ? bglob[t] : 0.0;
  const int par0 = on0 ? coarse_parent(L0, L1, t) : 0, par1 = on1 ? coarse_parent(L1, L2, t) : 0;
  for (double* q = smem + t; q < zeroed; q += S) *q = 0.0;  // padding and cells past a level's end
#pragma unroll
  for (int k = 0; k < NI; ++k) inv[t + k * S] = vi[k];
  c0.di = 1.0 / c0.D;
  c1.di = 1.0 / c1.D;
  c0.B = bin;
  if (stop) return;
  __syncthreads();
  // the bottom's columns go to as many wavefronts as level 0 fills
  const int groups = (n0 + 63) >> 6, chunk = (n2 + groups - 1) / groups;
  const int br = t & 63, bg = t >> 6, j0 = bg * chunk, j1 = min(n2, j0 + chunk);
  double x0 = 0.0;
#pragma unroll 1
  for (int cyc = 0; cyc < a.ncyc; ++cyc) {
    if (cyc > 0) {  // continue from the residual the cycle before left
      x0 += c0.e;
      c0.B += fma(-c0.D, c0.e, coarse_nb(c0, b0.cur, nx0));
    }
    c0.e = kOmega * c0.B * c0.di;
    *b0.oth = c0.e;
    b0.turn();
    c0.e = coarse_sweep(c0, b0.cur, nx0);
    *b0.oth = c0.e;
    b0.turn();
    rc[t] = coarse_res(c0, b0.cur, nx0);
    __syncthreads();
    double x1 = 0.0;
#pragma unroll 1
    for (int v = 0; v < a.ncyc1; ++v) {
      if (on1) {
        if (v == 0) {
          c1.B = coarse_children(rc, L0.nx, L0.ny, t % nx1, t / nx1);
        } else {
          x1 += c1.e;
          c1.B += fma(-c1.D, c1.e, coarse_nb(c1, b1.cur, nx1));
        }
        c1.e = kOmega * c1.B * c1.di;
        *b1.oth = c1.e;
      }
      b1.turn();
      if (on1) {
        c1.e = coarse_sweep(c1, b1.cur, nx1);
        *b1.oth = c1.e;
      }
      b1.turn();
      if (on1) rc[t] = coarse_res(c1, b1.cur, nx1);
      __syncthreads();
      if (on2) bc[t] = coarse_children(rc, L1.nx, L1.ny, t % L2.nx, t / L2.nx);
      __syncthreads();
      if (br < n2 && bg < groups) {
        double s = 0.0;
        for (int j = j0; j < j1; ++j) s += inv[j * n2 + br] * bc[j];
        parts[bg * n2 + br] = s;
      }
      __syncthreads();
      if (on2) {
        double s = 0.0;
        for (int k = 0; k < groups; ++k) s += parts[k * n2 + t];
        ebot[t] = s;
      }
      __syncthreads();
      if (on1) {
        c1.e = fma(a.omega_c, ebot[par1], c1.e);
        *b1.oth = c1.e;
      }
      b1.turn();
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (on1) {
          c1.e = coarse_sweep(c1, b1.cur, nx1);
          // the last value is the level's whole correction, for level 0
          *b1.oth = s == 1 && v + 1 == a.ncyc1 ? c1.e + x1 : c1.e;
        }
        b1.turn();
      }
    }
    c0.e = fma(a.omega_c, (b1.cur - t)[par0], c0.e);
    *b0.oth = c0.e;
    b0.turn();
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      c0.e = coarse_sweep(c0, b0.cur, nx0);
      *b0.oth = c0.e;
      b0.turn();
    }
  }
  double part = 0.0;
  if (on0) {
    const double v = x0 + c0.e;
    out[t] = v;
    part = bin * v;
  }
  if (rz_slot < 0) return;
  part = wave_sum(part);
  __shared__ double sh[kMgLdsCells / 64];
  if ((t & 63) == 0) sh[t >> 6] = part;
  __syncthreads();
  double* slots = st->rz + rz_slot * st->nb;
  for (int k = t + 1; k < st->nb; k += S) slots[k] = 0.0;
  if (t == 0) {
    double s = 0.0;
    for (int w = 0; w < groups; ++w) s += sh[w];
    slots[0] = s;
  }
}

}  // namespace

hipError_t mg_setup(const MgHierarchy& h, hipStream_t s) {
  // the levels down to the first LDS level one by one, the rest with the bottom
  // inverse
  for (int l = 1; l <= h.lc; ++l) {
    const MgLevelDev& F = h.lev[l - 1];
    const MgLevelDev& C = h.lev[l];
    const dim3 grid((C.nx + kBX - 1) / kBX, (C.ny + kBY - 1) / kBY, C.nz);
    hipLaunchKernelGGL(k_mg_coarsen, grid, cell_block(), 0, s, F, C);
  }
  hipLaunchKernelGGL(k_mg_bottom_inverse, dim3(1), dim3(1024), 0, s, h.coarse, h.binv);
  return hipGetLastError();
}

// z = M^{-1} r on the finest level; with rz_slot >= 0 also accumulates r . z
// into the CG ring.
hipError_t mg_apply(const MgHierarchy& h, const double* r, double* z, PcgState* st, int rz_slot, hipStream_t s,
                    const CgFuse* cg) {
  if (cg && !mg_fuses_cg(h)) return hipErrorInvalidValue;
  const int lc = h.lc;
  auto grid_of = [](const MgLevelDev& L) {
    return dim3((L.nx + kBX - 1) / kBX, (L.ny + kBY - 1) / kBY, L.nz);
  };
  for (int l = 0; l < lc; ++l) {
    const MgLevelDev& F = h.lev[l];
    const MgLevelDev& C = h.lev[l + 1];
    const double* b = l == 0 ? r : F.b;
    if (F.nz == 1) {
      const dim3 g((F.nx + kBX - 1) / kBX, (F.ny + kTY - 1) / kTY, 1);
      if (l == 0 && cg && cg->update)
        hipLaunchKernelGGL(k_mg_down_cg<kMgSweeps>, g, dim3(1024), 0, s, F, C, b, F.x, C.b, st, *cg);
      else
        hipLaunchKernelGGL(k_mg_down_box<kMgSweeps>, box_grid(F), dim3(kBoxT), 0, s, F, C, b, F.x, C.b, st);
    } else {
      const dim3 g((F.nx + kBX - 1) / kBX, (F.ny + kBY - 1) / kBY, C.nz);
      hipLaunchKernelGGL(k_mg_down_restrict, g, cell_block(), 0, s, F, C, b, F.x, C.b, st);
    }
  }
  {
    const double* b = lc == 0 ? r : h.lev[lc].b;
    double* out = lc == 0 ? z : h.lev[lc].x;
    if (h.reg2d)
      hipLaunchKernelGGL(k_mg_coarse_2d, dim3(1), dim3(kMgLdsCells), h.lds_bytes, s, h.coarse, b, h.binv, out, st,
                         lc == 0 ? rz_slot : -1);
    else
      hipLaunchKernelGGL(k_mg_coarse_lds, dim3(1), dim3(h.coarse_threads), h.lds_bytes, s, h.coarse, b, h.binv,
                         out, st, lc == 0 ? rz_slot : -1);
  }
  // The up leg reads its level's x at the neighbours, so it writes its result
  // to y (z on the finest level); the LDS solve leaves its result in x.
  for (int l = lc - 1; l >= 0; --l) {
    const MgLevelDev& F = h.lev[l];
    const MgLevelDev& C = h.lev[l + 1];
    const double* b = l == 0 ? (cg && cg->update ? cg->r_new : r) : F.b;
    const double* ec = l + 1 == lc ? C.x : C.y;
    double* out = l == 0 ? z : F.y;
    if (F.nz == 1) {
      const dim3 g((F.nx + kBX - 1) / kBX, (F.ny + kTY - 1) / kTY, 1);
      if (l == 0 && cg)
        hipLaunchKernelGGL(k_mg_up_cg<kMgSweeps>, g, dim3(576), 0, s, F, C, b, F.x, ec, h.omega_c, out, cg->w_out, st,
                           rz_slot);
      else
        hipLaunchKernelGGL(k_mg_up_box<kMgSweeps>, box_grid(F), dim3(kBoxT), 0, s, F, C, b, F.x, ec, h.omega_c, out,
                           st);
    } else {
      hipLaunchKernelGGL(k_mg_up_smooth, grid_of(F), cell_block(), 0, s, F, C, b, F.x, ec, h.omega_c, out, st,
                         l == 0 ? rz_slot : -1);
    }
  }
  return hipGetLastError();
}

hipError_t mg_set_lds_limit(int bytes, bool reg2d) {
  return lds_grant(reg2d ? reinterpret_cast<const void*>(&k_mg_coarse_2d)
                         : reinterpret_cast<const void*>(&k_mg_coarse_lds), bytes);
}

}  // namespace erem
