// Newton-Leja evaluation of phi1(h J) v on a small grid by one workgroup, in
// one launch: all substeps, all terms and their stop tests (Sec. 4.2).
//
// On at most kSmallCells cells a pass over the grid takes less than the launch
// that starts it, so the passes of leja.hip cost what their launches and their
// memory round trips cost (7.5 us per four terms on 32 x 32).  Here a thread
// owns C cells for the whole evaluation: their stencil, q, p and u stay in
// registers, the neighbours' q goes through LDS (double buffered, a barrier per
// term), the coefficients wait in LDS, and the stop test of a group of four
// terms is one more barrier.  The operations on a cell are those of the passes,
// in their order, so the results are the same bits as long as the stop test
// (whose sums are formed in another order) passes at the same term.  One step on
// 32 x 32: 718 -> 140 us.
#include "device.h"
#include "lds_grant.h"
#include "leja.h"

namespace erem {

namespace {

template <class V>
__device__ inline V to_v(double x) { return static_cast<V>(x); }

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;

// LDS: two vectors of C cells per thread in double (the q buffers, and u between
// substeps), shift, dk and estf, the wavefronts' sums.
template <int C>
constexpr size_t small_lds_bytes(int K) {
  return sizeof(double) * (2 * static_cast<size_t>(C) * kSmallThreads + 3 * static_cast<size_t>(K + 1) +
                           8 * kSmallWaves);
}

template <int DIM, int C, class V>
__global__ __launch_bounds__(kSmallThreads) void k_leja_small(Dims d, const LejaCoef* __restrict__ cf,
                                                              const double* __restrict__ coef64,
                                                              const V* __restrict__ coef,
                                                              const double* __restrict__ v,
                                                              const double* __restrict__ g,
                                                              const double* __restrict__ zt,
                                                              double* __restrict__ out, LejaState* st, double delta,
                                                              int s, int K) {
  constexpr int NB = 2 * DIM;
  if (st->stopped >= 0) return;  // the device's coefficients were refused: the host evaluates again
  extern __shared__ double smem[];
  double* ub = smem;
  V* qb[2] = {reinterpret_cast<V*>(smem), reinterpret_cast<V*>(smem + C * kSmallThreads)};
  double* shf = smem + 2 * C * kSmallThreads;
  double* dks = shf + K + 1;
  double* est = dks + K + 1;
  double* red = est + K + 1;          // [kSmallWaves][4]: the group's sums
  double* red0 = red + 4 * kSmallWaves;  // term 0's
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int N = d.N, pl = d.nx * d.ny;
  int has[C];  // bit k: neighbour k exists
  V c[C][NB + 1];
#pragma unroll
  for (int r = 0; r < C; ++r) {
    const int i = t + r * kSmallThreads;
    const bool in = i < N;
    const int j = in ? i : 0;
    const int z = j / pl, y = (j - z * pl) / d.nx, x = j - z * pl - y * d.nx;
    has[r] = (x > 0 ? 1 : 0) | (x + 1 < d.nx ? 2 : 0) | (y > 0 ? 4 : 0) | (y + 1 < d.ny ? 8 : 0) |
             (DIM == 3 && z > 0 ? 16 : 0) | (DIM == 3 && z + 1 < d.nz ? 32 : 0);
    if (!in) has[r] = 0;  // a slot past the grid holds zeros and reads itself
#pragma unroll
    for (int k = 0; k <= NB; ++k) c[r][k] = in ? coef[static_cast<size_t>(k) * N + j] : V(0);
  }
  // index of neighbour k of cell r: the cell itself where it is missing
  auto nb = [&](int r, int k) {
    const int i = t + r * kSmallThreads;
    const int o = k < 2 ? 1 : (k < 4 ? d.nx : pl);
    const int h = (has[r] >> k) & 1;
    return (k & 1) ? i + h * o : i - h * o;
  };
  for (int k = t; k <= K; k += kSmallThreads) {
    shf[k] = cf->shift[k];
    dks[k] = cf->dk[k];
    est[k] = cf->estf[k];
  }
  const V ig = to_v<V>(cf->inv_g);
  const double thresh = cf->thresh;
  __shared__ int stop_sh;
  for (int j = 0; j < s; ++j) {
    V q[C], p[C];
    double sum[4];
    // start: q_0 = v + t_j g + J u, p = d_0 q_0
    // (u, the sum of the substeps so far, waits in ub, and in out)
    double src[C];
#pragma unroll
    for (int r = 0; r < C; ++r) {
      int i = t + r * kSmallThreads;
      asm volatile("" : "+v"(i));  // the addresses are formed here, not kept in registers all along
      const bool in = i < N;
      src[r] = in ? v[i] : 0.0;
      if (j > 0 && in) {
        if (g) src[r] += (j * delta) * g[i];
        double a = coef64[i] * ub[i];
#pragma unroll
        for (int k = 0; k < NB; ++k) a += coef64[static_cast<size_t>(k + 1) * N + i] * ub[nb(r, k)];
        src[r] += a;
      }
      if (C > 2) __builtin_amdgcn_sched_barrier(0);  // one cell's loads at a time: registers
    }
    __syncthreads();
    const V d0 = to_v<V>(dks[0]);
    double s0 = 0.0;
#pragma unroll
    for (int r = 0; r < C; ++r) {
      q[r] = to_v<V>(src[r]);
      p[r] = d0 * q[r];
      qb[0][t + r * kSmallThreads] = q[r];
      s0 += static_cast<double>(q[r]) * static_cast<double>(q[r]);
    }
    {
      const double z4[4] = {s0, 0.0, 0.0, 0.0};
      const double w0 = sum4(z4, lane);
      if (lane < 4) red0[4 * wave + lane] = w0;
    }
    __syncthreads();
    // the first wavefront's own: lane l < 4 holds the estimate of term k0 - 4 + l
    double eprev = 0.0;
    int stop = -1;
    for (int k0 = 1; k0 <= K && stop < 0; k0 += 4) {
      const int n = min(4, K - k0 + 1);
#pragma unroll
      for (int tt = 0; tt < 4; ++tt) {
        sum[tt] = 0.0;
        if (tt < n) {
          const int k = k0 + tt;
          const V* qc = qb[(k + 1) & 1];  // term k - 1: buffer (k - 1) & 1
          V* qo = qb[k & 1];
          const V sh = to_v<V>(shf[k]), dk = to_v<V>(dks[k]);
#pragma unroll
          for (int r = 0; r < C; ++r) {
            V jq;
            if (C > 2) asm volatile("" : "+v"(has[r]));  // the neighbours' addresses likewise
            if (DIM == 2) {
              jq = c[r][1] * qc[nb(r, 0)];
              jq = fma(c[r][0], q[r], jq);
            } else {
              jq = c[r][0] * q[r];
              jq = fma(c[r][1], qc[nb(r, 0)], jq);
            }
#pragma unroll
            for (int m = 1; m < NB; ++m) jq = fma(c[r][m + 1], qc[nb(r, m)], jq);
            const V w = fma(jq, ig, -(sh * q[r]));
            q[r] = w;
            p[r] = fma(dk, w, p[r]);
            qo[t + r * kSmallThreads] = w;
            sum[tt] += static_cast<double>(w) * static_cast<double>(w);
            if (C > 2 && (r & 1)) __builtin_amdgcn_sched_barrier(0);
          }
          __syncthreads();
        }
      }
      // stop test of the group (and of term 0 with the first) by the first
      // wavefront: lanes l < 4 take the terms k0 + l
      const double w4 = sum4(sum, lane);
      if (lane < 4) red[4 * wave + lane] = w4;
      __syncthreads();
      if (wave == 0) {
        const double S = sum_quads(red[lane]);  // 16 wavefronts x 4 values are 64 entries
        const int k = k0 + (lane & 3);
        const bool mine = lane < n;
        const double e = mine ? est[k] * sqrt(S) : 0.0;
        if (k0 == 1) {  // term 0, where term k0 - 1 is kept
          const double S0 = __shfl(sum_quads(red0[lane]), 0, 64);
          eprev = lane == 3 ? est[0] * sqrt(S0) : 0.0;
          if (lane == 0) st[j].sums[0] = S0;
          if (!isfinite(S0)) stop = 0;
        }
        // mean of the five estimates k - 4 .. k: of the group before from lane
        // l on, of this group up to lane l
        double mean = 0.0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const double v = __shfl(eprev, m, 64);
          mean += m >= lane ? v : 0.0;
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const double v = __shfl(e, m, 64);
          mean += m <= lane ? v : 0.0;
        }
        const bool bad = mine && !isfinite(S);
        const unsigned long long hit = __ballot(bad || (mine && k >= 4 && 0.2 * mean < thresh));
        const int last = stop == 0 ? -1 : (hit ? __ffsll(hit) - 1 : n - 1);  // the last term tested
        if (lane <= last) st[j].sums[k] = S;
        const unsigned long long nf = __ballot(bad && lane == last) | (stop == 0 ? 1ull : 0ull);
        if (stop < 0 && hit) stop = k0 + last;
        if (lane == 0) {
          st[j].checked = stop == 0 ? 0 : k0 + last;
          if (nf) st[j].nonfinite = 1;
          if (stop >= 0) st[j].stopped = stop;
          stop_sh = stop;
        }
        eprev = e;
      }
      __syncthreads();
      stop = stop_sh;
    }
#pragma unroll
    for (int r = 0; r < C; ++r) {
      int i = t + r * kSmallThreads;
      asm volatile("" : "+v"(i));
      const double pi = static_cast<double>(p[r]);
      if (i < N) {
        double w = j == 0 ? delta * pi : out[i] + delta * pi;
        if (zt) w += zt[i];
        out[i] = w;
        if (j + 1 < s) ub[i] = w;
      }
    }
    __syncthreads();
  }
}

template <int DIM, int C, class V>
hipError_t launch_small(const Dims& d, const LejaCoef* cf, const double* coef64, const V* coef, const double* v,
                        const double* g, const double* zt, double* out, LejaState* st, double delta, int s, int K,
                        hipStream_t q, hipEvent_t e0, hipEvent_t e1) {
  const size_t bytes = small_lds_bytes<C>(K);
  // the largest size any K needs
  const hipError_t e = lds_grant(reinterpret_cast<const void*>(&k_leja_small<DIM, C, V>),
                                 static_cast<int>(small_lds_bytes<C>(kMaxTerms)));
  if (e != hipSuccess) return e;
  launch_timed(k_leja_small<DIM, C, V>, dim3(1), dim3(kSmallThreads), static_cast<unsigned>(bytes), q, e0, e1, d, cf,
               coef64, coef, v, g, zt, out, st, delta, s, K);
  return hipGetLastError();
}

}  // namespace

bool leja_small_fits(const Dims& d) { return d.N <= (d.dim == 3 ? kSmallCells3 : kSmallCells); }

template <class V>
hipError_t leja_small(const Dims& d, const LejaCoef* cf, const double* coef64, const V* coef, const double* v,
                      const double* g, const double* zt, double* out, LejaState* st, double delta, int s, int K,
                      hipStream_t q, hipEvent_t e0, hipEvent_t e1) {
#define EREM_SMALL(DIM, C) launch_small<DIM, C, V>(d, cf, coef64, coef, v, g, zt, out, st, delta, s, K, q, e0, e1)
  if (!leja_small_fits(d)) return hipErrorInvalidValue;
  if (d.dim == 3)
    return d.N <= kSmallThreads ? EREM_SMALL(3, 1) : EREM_SMALL(3, 2);
  return d.N <= kSmallThreads ? EREM_SMALL(2, 1) : (d.N <= 2 * kSmallThreads ? EREM_SMALL(2, 2) : EREM_SMALL(2, 4));
#undef EREM_SMALL
}

template hipError_t leja_small<double>(const Dims&, const LejaCoef*, const double*, const double*, const double*,
                                       const double*, const double*, double*, LejaState*, double, int, int,
                                       hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t leja_small<float>(const Dims&, const LejaCoef*, const double*, const float*, const double*,
                                      const double*, const double*, double*, LejaState*, double, int, int,
                                      hipStream_t, hipEvent_t, hipEvent_t);

}  // namespace erem
