// Arnoldi process on the device for the Krylov evaluation of phi1 (Sec. 4.1,
// Alg. alg:al2).  Each new column is orthogonalised against the basis by
// classical Gram-Schmidt applied twice (CGS2) rather than by the algorithm's
// modified Gram-Schmidt: both give the same Hessenberg matrix in exact
// arithmetic, and the second pass keeps the computed basis orthogonal to
// working precision, while each projection becomes one pass over the basis
// with all its inner products at once.  Column j therefore costs three
// streaming passes and three reductions whatever j is:
//   1. w = J v_j, with the partial sums of v_i . w (i <= j);
//   2. w -= sum_i g_i v_i, with the partial sums of v_i . w again;
//   3. w -= sum_i g'_i v_i, with the partial sum of w . w.
// Each pass first adds up the partials of the pass before it, every workgroup
// all of them alike and in a fixed order, and its first workgroup writes the
// Hessenberg entries h_ij = g_i + g'_i and h_{j+1,j} = ||w|| into device memory;
// v_{j+1} = w / h_{j+1,j} is formed inside pass 1 of the next column.  A column
// is thus three launches; on grids of more than kKryDirect workgroups a fold
// (one wavefront per value) sits between the passes, since adding that many
// partials in every workgroup would cost more than the launch.  The host does
// not sync inside the process and reads H once at the end.
//
// On small grids the passes are bound by latency (launch, one round of loads, the
// sums): on 37 x 29 x 41, m = 10, a substep takes 33 launches and 135 us of kernel
// time, where a reduction launch after every pass and the basis read twice per pass
// took 62 launches and 237 us.
#include "device.h"
#include "krylov.h"

namespace erem {

namespace {

constexpr int kRedThreads = 64;  // one wavefront per reduced value
constexpr int kKryWaves = kThreads / 64;

// Sums of n partial arrays (nb values each, one after the other) into gs, by the
// whole workgroup; wavefront w takes the values w, w + 4, ..., four at a time so
// that their loads and shuffle trees overlap.
__device__ inline void take_sums(const double* __restrict__ part, int nb, int n, double* gs) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int k0 = wave; k0 < n; k0 += 4 * kKryWaves) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int b = lane; b < nb; b += 64) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u * kKryWaves;
        acc[u] += k < n ? part[static_cast<size_t>(k) * nb + b] : 0.0;
      }
    }
    const double s = sum4(acc, lane);
    if (lane < 4 && k0 + lane * kKryWaves < n) gs[k0 + lane * kKryWaves] = s;
  }
  __syncthreads();
}

// The first kKryRegs basis vectors at cell i, loaded together (ahead of the sums
// that a pass needs first); the others are read where they are used.
constexpr int kKryRegs = 12;
struct KryRow {
  double v[kKryRegs];
  __device__ inline void load(const double* __restrict__ V, size_t N, int i, bool in, int n) {
#pragma unroll
    for (int k = 0; k < kKryRegs; ++k) v[k] = in && k < n ? V[k * N + i] : 0.0;
  }
};

// V_k[i] * a for k < n summed over each wavefront, wavefront w's share of value k
// to sh[k * kKryWaves + w]; four values to a reduction.
__device__ inline void wave_dots(const KryRow& row, const double* __restrict__ V, size_t N, int i, bool in, double a,
                                 int n, double* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k0 = 0; k0 < kKryRegs; k0 += 4) {
    if (k0 >= n) break;
    const double t[4] = {row.v[k0] * a, row.v[k0 + 1] * a, row.v[k0 + 2] * a, row.v[k0 + 3] * a};
    const double s = sum4(t, lane);
    if (lane < 4 && k0 + lane < n) sh[(k0 + lane) * kKryWaves + wave] = s;
  }
  for (int k0 = kKryRegs; k0 < n; k0 += 4) {
    double t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = in && k0 + u < n ? V[(k0 + u) * N + i] * a : 0.0;
    const double s = sum4(t, lane);
    if (lane < 4 && k0 + lane < n) sh[(k0 + lane) * kKryWaves + wave] = s;
  }
}

__device__ inline void wave_value(double v, double* sh, int k) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[k * kKryWaves + (threadIdx.x >> 6)] = v;
}

// The workgroup's partials of n values, the wavefronts added in order.
__device__ inline void block_flush(const double* sh, int n, double* __restrict__ part) {
  __syncthreads();
  for (int k = threadIdx.x; k < n; k += kThreads) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kKryWaves; ++w) s += sh[k * kKryWaves + w];
    part[static_cast<size_t>(k) * gridDim.x + blockIdx.x] = s;
  }
}

// Operands of J v at cell i: the cell's stencil, and v there and at its
// neighbours (the cell itself where one is missing: its coefficient is zero).
struct KryStencil {
  double c[7], v[7];
  int n;
  __device__ inline void load(const Dims& d, const double* __restrict__ coef, const double* __restrict__ src, int i) {
    const int pl = d.nx * d.ny, z = i / pl, r = i - z * pl, y = r / d.nx, x = r - y * d.nx;
    const size_t N = d.N;
    n = d.dim == 3 ? 7 : 5;
    const int j[7] = {i, x > 0 ? i - 1 : i, x + 1 < d.nx ? i + 1 : i, y > 0 ? i - d.nx : i,
                      y + 1 < d.ny ? i + d.nx : i, z > 0 ? i - pl : i, z + 1 < d.nz ? i + pl : i};
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      c[k] = k < n ? coef[k * N + i] : 0.0;
      v[k] = k < n ? src[j[k]] : 0.0;
    }
  }
  // J (s v)
  __device__ inline double apply(double s) const {
    double jv = c[0] * (v[0] * s);
#pragma unroll
    for (int k = 1; k < 7; ++k)
      if (k < n) jv += c[k] * (v[k] * s);
    return jv;
  }
};

// Start vector w = v + J u (u null: w = v) with the partials of w . w.
__global__ __launch_bounds__(kThreads) void k_kry_start(Dims d, const double* __restrict__ coef,
                                                        const double* __restrict__ v, const double* __restrict__ u,
                                                        double* __restrict__ w, double* __restrict__ part) {
  __shared__ double sh[kKryWaves];
  const int i = blockIdx.x * kThreads + threadIdx.x;
  double a = 0.0;
  if (i < d.N) {
    a = v[i];
    if (u) {
      KryStencil q;
      q.load(d, coef, u, i);
      a += q.apply(1.0);
    }
    w[i] = a;
  }
  wave_value(a * a, sh, 0);
  block_flush(sh, 1, part);
}

// Pass 1 of column j: the norm of src from its partials (to *nrm), v_j = src /
// norm to vj, w = J v_j (the neighbours of v_j read from src and scaled), and the
// partials of v_i . w for i = 0..j (V holds v_0..v_{j-1}; v_j comes from
// registers).  src and w are different buffers: the neighbour reads of src must
// not see this pass's stores; likewise the partials read and written.
__global__ __launch_bounds__(kThreads) void k_kry_spmv(Dims d, const double* __restrict__ coef,
                                                       const double* __restrict__ src,
                                                       const double* __restrict__ pin, int nin,
                                                       double* __restrict__ nrm, double* __restrict__ vj,
                                                       double* __restrict__ w, const double* __restrict__ V, int j,
                                                       double* __restrict__ part) {
  __shared__ double sh[(kMaxKrylov + 1) * kKryWaves];
  __shared__ double gs[1];
  const int i = blockIdx.x * kThreads + threadIdx.x;
  const bool in = i < d.N;
  KryStencil q;
  KryRow row;
  q.load(d, coef, src, in ? i : 0);  // in flight while the sums are added up
  row.load(V, d.N, i, in, j);
  take_sums(pin, nin, 1, gs);
  const double h = sqrt(gs[0]);
  if (blockIdx.x == 0 && threadIdx.x == 0) *nrm = h;
  const double inv = h > 0.0 ? 1.0 / h : 0.0;  // zero: happy breakdown, the host truncates there
  double vc = 0.0, jv = 0.0;
  if (in) {
    vc = q.v[0] * inv;
    jv = q.apply(inv);
    vj[i] = vc;
    w[i] = jv;
  }
  wave_dots(row, V, d.N, in ? i : 0, in, jv, j, sh);
  wave_value(vc * jv, sh, j);
  block_flush(sh, j + 1, part);
}

// Passes 2 and 3: g from the partials of the pass before, into column H (row
// stride hs; pass 3, NORM, adds), w -= sum_{k < nv} g_k v_k, then the partials of
// v_k . w for k < nv (pass 2) or of w . w (pass 3).
template <bool NORM>
__global__ __launch_bounds__(kThreads) void k_kry_update(int N, double* __restrict__ w,
                                                         const double* __restrict__ V, int nv,
                                                         const double* __restrict__ pin, int nin,
                                                         double* __restrict__ H, int hs, double* __restrict__ part) {
  __shared__ double sh[(kMaxKrylov + 1) * kKryWaves];
  __shared__ double gs[kMaxKrylov + 1];
  const int i = blockIdx.x * kThreads + threadIdx.x;
  const bool in = i < N;
  KryRow row;
  row.load(V, N, i, in, nv);  // in flight while the sums are added up
  double acc = in ? w[i] : 0.0;
  take_sums(pin, nin, nv, gs);
  if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < nv) {
    double* h = H + static_cast<size_t>(threadIdx.x) * hs;
    *h = NORM ? *h + gs[threadIdx.x] : gs[threadIdx.x];
  }
#pragma unroll
  for (int k = 0; k < kKryRegs; ++k)
    if (k < nv) acc -= gs[k] * row.v[k];
  if (in) {
    for (int k = kKryRegs; k < nv; ++k) acc -= gs[k] * V[k * static_cast<size_t>(N) + i];
    w[i] = acc;
  }
  if (NORM) {
    wave_value(acc * acc, sh, 0);
    block_flush(sh, 1, part);
  } else {
    wave_dots(row, V, N, in ? i : 0, in, acc, nv, sh);
    block_flush(sh, nv, part);
  }
}

// Workgroup k sums the nb partials part[k * nb ..] in a fixed order into g[k], or
// their root (ROOT).
template <bool ROOT>
__global__ __launch_bounds__(kRedThreads) void k_kry_reduce(const double* __restrict__ part, int nb,
                                                            double* __restrict__ g) {
  const double s = wave_part_sum(part + static_cast<size_t>(blockIdx.x) * nb, nb);
  if (threadIdx.x == 0) g[blockIdx.x] = ROOT ? sqrt(s) : s;
}

// u = (first ? 0 : u) + sum_k c_k v_k, the last v unnormalised in w when it is
// among them (its coefficient then holds the norm's reciprocal).
__global__ __launch_bounds__(kThreads) void k_combine(int N, const double* __restrict__ V,
                                                      const double* __restrict__ w, KryCoef c,
                                                      double* __restrict__ u, int first) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= N) return;
  double acc = first ? 0.0 : u[i];
  for (int k = 0; k < c.nv; ++k) acc += c.c[k] * V[k * static_cast<size_t>(N) + i];
  if (c.last) acc += c.clast * w[i];
  u[i] = acc;
}

int kry_blocks(const Dims& d) { return (d.N + kThreads - 1) / kThreads; }

// What a pass reads as the sums of the pass before: its partials, or (many
// workgroups) their fold in g.
hipError_t kry_sums(const double* part, int nb, int n, double* g, const double** src, int* cnt, hipStream_t s) {
  *src = part;
  *cnt = nb;
  if (nb <= kKryDirect) return hipSuccess;
  hipLaunchKernelGGL(k_kry_reduce<false>, dim3(n), dim3(kRedThreads), 0, s, part, nb, g);
  *src = g;
  *cnt = 1;
  return hipGetLastError();
}

}  // namespace

size_t kry_part_words(const Dims& d, int m) { return 3 * static_cast<size_t>(m + 1) * kry_blocks(d); }

hipError_t krylov_start(const Dims& d, const double* coef, const double* v, const double* u, double* w, double* part,
                        int m, hipStream_t s) {
  const int nb = kry_blocks(d);
  hipLaunchKernelGGL(k_kry_start, dim3(nb), dim3(kThreads), 0, s, d, coef, v, u, w,
                     part + 2 * static_cast<size_t>(m + 1) * nb);
  return hipGetLastError();
}

hipError_t arnoldi_cgs2(const Dims& d, const double* coef, double* V, double* w, double* H, double* beta,
                        double* g, double* part, int m, hipStream_t s) {
  const size_t N = d.N;
  const int nb = kry_blocks(d);
  const dim3 gr(nb), b(kThreads);
  // the partials of pass 1, pass 2 and pass 3 in turn: a pass reads one region
  // and writes the next
  double* p1 = part;
  double* p2 = part + static_cast<size_t>(m + 1) * nb;
  double* p3 = part + 2 * static_cast<size_t>(m + 1) * nb;
  double* nrm = beta;
  const double* src = nullptr;
  int cnt = 0;
  hipError_t e;
  for (int j = 0; j < m; ++j) {
    double* wi = w + (j & 1) * N;
    double* wj = w + ((j + 1) & 1) * N;
    if ((e = kry_sums(p3, nb, 1, g, &src, &cnt, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_kry_spmv, gr, b, 0, s, d, coef, wi, src, cnt, nrm, V + j * N, wj, V, j, p1);
    if ((e = kry_sums(p1, nb, j + 1, g, &src, &cnt, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_kry_update<false>, gr, b, 0, s, d.N, wj, V, j + 1, src, cnt, H + j, m, p2);
    if ((e = kry_sums(p2, nb, j + 1, g, &src, &cnt, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_kry_update<true>, gr, b, 0, s, d.N, wj, V, j + 1, src, cnt, H + j, m, p3);
    nrm = H + static_cast<size_t>(j + 1) * m + j;
  }
  hipLaunchKernelGGL(k_kry_reduce<true>, dim3(1), dim3(kRedThreads), 0, s, p3, nb, nrm);
  return hipGetLastError();
}

hipError_t krylov_combine(const Dims& d, const double* V, const double* w, const KryCoef& c, double* u, int first,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_combine, dim3(kry_blocks(d)), dim3(kThreads), 0, s, d.N, V, w, c, u, first);
  return hipGetLastError();
}

}  // namespace erem
