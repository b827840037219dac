// Batched EREM for many independent linear problems.
//
// Every problem p (its own n_x x n_y grid, packed one after the other) has a
// constant Jacobian J_p and G_p(T) = J_p T + g_p (fixed fluxes, constant
// capacity), so one EREM step is T <- T + h phi1(h J_p)(J_p T + g_p)
// (Eq. EERM) with a Gershgorin interval, substep count and divided
// differences fixed for the whole run (Sec. 4.2).
//
// MI355X mapping.  The problems are cut into tiles - strips of at most 64
// columns by a chunk of rows, one wavefront each (march.h) - and all tiles of
// all problems form one list.  A run is a sequence of phases; in each
// phase ONE work launch covers the whole tile list and advances every
// problem that is not done by one step of its own schedule:
//
//   start pass  q_0 = v + J u, p = d_0 q_0 (with the end of the previous
//               substep, u += delta p, or of the previous step,
//               T += u + delta p, folded in: a cell's neighbours' values are
//               formed from their own u, p, T, so no extra pass is needed);
//   term pass   NT = 4 or 8 Newton terms
//               q_k = ((J - cI)/gamma - xi_{k-1}) q_{k-1}, p += d_k q_k
//               (Eq. newt) on the tile, computed over the tile plus the halo
//               that NT stencil applications need; the intermediate terms
//               stay in registers;
//   finish pass T += u + delta p of the last step.
//
// Each tile stores its partial sums (sum q_k^2 per term, in FP64); at the start
// of the next pass every tile's wavefront adds up its problem's partials (those
// of a problem of many tiles from a fold between the passes) in a fixed order,
// applies the scaled-norm stop test of Sec. 4.2 to the pass's NT estimates in
// order, and so knows the problem's next phase.
// Problems of every size and substep count thus share every launch, the
// work spreads over all CUs whatever the mix, and the whole run is a fixed
// sequence of launches with no grid-wide synchronisation and no waiting
// inside a kernel, which a hipGraph captures.  Tiles of problems that are
// done return at entry.  Buffers the start pass reads with a halo and
// rewrites (T, u, p) are ping-ponged so that no tile reads a neighbour's
// updated value.
#include "batch.h"
#include "march.h"

#include <cmath>

namespace erem {

namespace {

// Rows loaded ahead: four keep 14 KB per wavefront in flight and still fit 256
// registers with eight FP64 terms (two: 71.2 ms a run, four: 70.4).
constexpr int kBatchAhead = 4;

template <class V>
__device__ inline V cv(double x) { return static_cast<V>(x); }

// Maximum over the wavefront, valid in lane 0.
__device__ inline double march_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
  return v;
}

// Start pass of substep S.sub of step S.step on one strip's chunk of rows:
// the vector w whose J w enters q_0 (T^n, or the substep sum u, both formed
// here from the arrays the previous pass left), q_0 = v + J u or G = J T + g,
// p = d_0 q_0.  Marches like the term pass (row r of w arrives, row r - 1 of
// q_0 leaves); an array that this kind of pass does not read or write gets an
// empty descriptor, so its loads give zero and its stores are dropped.
template <class V>
__device__ inline void batch_start(const BatchArgs& a, const BProb& P, const BState& S, MarchStrip st, int y0, int y1,
                                   double* part) {
  constexpr int PD = 6, U = 8;
  const int nx = P.nx, ny = P.ny, lane = threadIdx.x & 63;
  const int r0 = max(0, y0 - 1), rend = min(ny, y1 + 1);
  const long long org = P.off + static_cast<long long>(nx) * r0;
  const unsigned rb = static_cast<unsigned>(nx) * 8u, rv = static_cast<unsigned>(nx) * sizeof(V);
  const unsigned bytes = rb * static_cast<unsigned>(rend - r0), bytv = rv * static_cast<unsigned>(rend - r0);
  const bool first = S.kind == kInitFirst, sub = S.kind == kInitSub;
  const bool use_u = sub ? S.sub > 1 : (!first && P.s > 1);
  const double delta = first ? 0.0 : P.delta;
  const __amdgpu_buffer_rsrc_t rT = march_rsrc((S.tpar ? a.T1 : a.T0) + org, sub ? 0u : bytes);
  const __amdgpu_buffer_rsrc_t ru = march_rsrc((S.upar ? a.u1 : a.u0) + org, use_u ? bytes : 0u);
  const __amdgpu_buffer_rsrc_t rp =
      march_rsrc(reinterpret_cast<const V*>(S.ppar ? a.p1 : a.p0) + org, first ? 0u : bytv);
  const __amdgpu_buffer_rsrc_t ra = march_rsrc((sub ? a.v : a.g) + org, bytes);
  __amdgpu_buffer_rsrc_t rc[5];
#pragma unroll
  for (int d = 0; d < 5; ++d) rc[d] = march_rsrc(a.coef64 + d * a.ntot + org, bytes);
  // outputs: the strip's own columns, rows y0 .. y1 - 1
  const long long oout = P.off + static_cast<long long>(nx) * y0;
  const unsigned rows = static_cast<unsigned>(y1 - y0);
  double* wdst = sub ? (S.upar ? a.u0 : a.u1) : (S.tpar ? a.T0 : a.T1);
  const __amdgpu_buffer_rsrc_t ow = march_rsrc(wdst + oout, first ? 0u : rb * rows);
  const __amdgpu_buffer_rsrc_t ov = march_rsrc(a.v + oout, sub ? 0u : rb * rows);
  const __amdgpu_buffer_rsrc_t oq = march_rsrc(reinterpret_cast<V*>(a.q0) + oout, rv * rows);
  const __amdgpu_buffer_rsrc_t op = march_rsrc(reinterpret_cast<V*>(S.ppar ? a.p0 : a.p1) + oout, rv * rows);
  const V d0 = cv<V>(a.dk[P.coef_off]);
  const int gx = st.xs + lane;
  const bool in = gx < nx, out = gx >= st.x0 && gx < st.x1;
  const unsigned base = in ? static_cast<unsigned>(gx) * 8u : kMarchOut;
  const unsigned basv = in ? static_cast<unsigned>(gx) * static_cast<unsigned>(sizeof(V)) : kMarchOut;
  const unsigned bo = out ? static_cast<unsigned>(gx) * 8u : kMarchOut;
  const unsigned bov = out ? static_cast<unsigned>(gx) * static_cast<unsigned>(sizeof(V)) : kMarchOut;
  double T[U], uu[U], c[U][5], ad[U], w[2] = {0.0, 0.0};
  V pp[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    T[i] = uu[i] = ad[i] = 0.0;
    pp[i] = V(0);
#pragma unroll
    for (int d = 0; d < 5; ++d) c[i][d] = 0.0;
  }
#pragma unroll
  for (int i = 0; i < PD; ++i) {
    const unsigned o = base + static_cast<unsigned>(i) * rb;
    march_load(rT, o, T[i]);
    march_load(ru, o, uu[i]);
    march_load(rp, basv + static_cast<unsigned>(i) * rv, pp[i]);
    if (i + 1 < PD) {
#pragma unroll
      for (int d = 0; d < 5; ++d) march_load(rc[d], o, c[i][d]);
      march_load(ra, o, ad[i]);
    }
  }
  double s0 = 0.0, mx = 0.0;
  int r = r0;
  unsigned offl = base + PD * rb, ofpl = basv + PD * rv;
  unsigned offo = bo + static_cast<unsigned>(r0 - 1 - y0) * rb, ofvo = bov + static_cast<unsigned>(r0 - 1 - y0) * rv;
  for (;;) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      march_load(rT, offl, T[(k + PD) % U]);
      march_load(ru, offl, uu[(k + PD) % U]);
      march_load(rp, ofpl, pp[(k + PD) % U]);
#pragma unroll
      for (int d = 0; d < 5; ++d) march_load(rc[d], offl - rb, c[(k + PD + U - 1) % U][d]);
      march_load(ra, offl - rb, ad[(k + PD + U - 1) % U]);
      __builtin_amdgcn_sched_barrier(0);
      const double wn = T[k] + uu[k] + delta * static_cast<double>(pp[k]);  // row r
      const double wc = w[(k + 1) & 1], ws = w[k & 1];                      // rows r - 1, r - 2
      const int s = (k + U - 1) % U;
      double jw = c[s][0] * wc;
      jw += c[s][1] * west(wc);
      jw += c[s][2] * east(wc);
      jw += c[s][3] * ws;
      jw += c[s][4] * wn;
      const double q = jw + ad[s];
      const V qv = cv<V>(q);
      march_store(ow, offo, wc);
      march_store(ov, offo, q);
      march_store(oq, ofvo, qv);
      march_store(op, ofvo, d0 * qv);
      const bool row = r - 1 >= y0;
      const double qm = march_mask(row, static_cast<double>(qv));
      s0 += qm * qm;
      mx = fmax(mx, row ? fabs(wc) : 0.0);
      w[k & 1] = wn;
      if (r == y1) goto done;
      ++r;
      offl += rb;
      ofpl += rv;
      offo += rb;
      ofvo += rv;
    }
  }
done:
  s0 = wave_sum(out ? s0 : 0.0);
  mx = march_max(out && !sub ? mx : 0.0);
  if (lane == 0) {
    part[0] = s0;
    part[1] = mx;
  }
}

// Finish pass: T^N = T^{N-1} + u + delta p into the caller's array (a failed
// problem keeps its last step's T).
template <class V>
__device__ inline void batch_finish(const BatchArgs& a, const BProb& P, const BState& S, MarchStrip st, int y0,
                                    int y1) {
  constexpr int U = 8;
  const int nx = P.nx, lane = threadIdx.x & 63;
  const long long org = P.off + static_cast<long long>(nx) * y0;
  const unsigned rb = static_cast<unsigned>(nx) * 8u, rv = static_cast<unsigned>(nx) * sizeof(V);
  const unsigned rows = static_cast<unsigned>(y1 - y0);
  const bool ok = S.flags == 0;
  const double delta = ok ? P.delta : 0.0;
  const __amdgpu_buffer_rsrc_t rT = march_rsrc((S.tpar ? a.T1 : a.T0) + org, rb * rows);
  const __amdgpu_buffer_rsrc_t ru = march_rsrc((S.upar ? a.u1 : a.u0) + org, ok && P.s > 1 ? rb * rows : 0u);
  const __amdgpu_buffer_rsrc_t rp =
      march_rsrc(reinterpret_cast<const V*>(S.ppar ? a.p1 : a.p0) + org, ok ? rv * rows : 0u);
  const __amdgpu_buffer_rsrc_t ro = march_rsrc(a.T0 + org, rb * rows);
  const int gx = st.xs + lane;
  const bool out = gx >= st.x0 && gx < st.x1;
  unsigned o = out ? static_cast<unsigned>(gx) * 8u : kMarchOut;
  unsigned ov = out ? static_cast<unsigned>(gx) * static_cast<unsigned>(sizeof(V)) : kMarchOut;
  for (int y = y0; y < y1; y += U, o += U * rb, ov += U * rv) {
    double T[U], u[U];
    V p[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      march_load(rT, o + k * rb, T[k]);
      march_load(ru, o + k * rb, u[k]);
      march_load(rp, ov + k * rv, p[k]);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) march_store(ro, o + k * rb, T[k] + (u[k] + delta * static_cast<double>(p[k])));
  }
}

// Tile of this workgroup: each XCD takes one contiguous range of the list (as
// xcd_tile_id does), front to back on even passes and back to front on odd
// ones, so that a pass begins with what the pass before left in the caches.
__device__ inline int batch_tile(int back) {
  const int n = gridDim.x, b = blockIdx.x;
  const int q = n / kXcds, r = n % kXcds, x = b % kXcds, k = b / kXcds;
  const int size = q + (x < r ? 1 : 0);
  return x * q + (x < r ? x : r) + (back ? size - 1 - k : k);
}

// Reductions over the lanes that agree in lane & 7; every such lane gets them.
__device__ inline void sum_max_octets(double& s, double& m) {
  s += dpp<0x128>(s);
  m = fmax(m, dpp<0x128>(m));
  s = add_xor32(add_xor16(s));
  const auto l16 = __builtin_amdgcn_permlane16_swap(__double2loint(m), __double2loint(m), false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap(__double2hiint(m), __double2hiint(m), false, false);
  m = fmax(__hiloint2double(h16[0], l16[0]), __hiloint2double(h16[1], l16[1]));
  const auto l32 = __builtin_amdgcn_permlane32_swap(__double2loint(m), __double2loint(m), false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap(__double2hiint(m), __double2hiint(m), false, false);
  m = fmax(__hiloint2double(h32[0], l32[0]), __hiloint2double(h32[1], l32[1]));
}

// Lane l's share of the sums and maxima of partial l & 7 over n slots.
__device__ inline void batch_sums(const double* __restrict__ pp, int n, double& s, double& mx) {
  n *= kBatchPartStride;
  for (int b = threadIdx.x; b < n; b += 4 * 64) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = b + 64 * u < n ? pp[b + 64 * u] : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      s += v[u];
      mx = fmax(mx, v[u]);
    }
  }
}

// The problem's next phase, from the partials that its tiles left in the pass
// before (lane l of every wavefront holds term k + (l & 7)'s sum in `s`, and in
// `mx` the maximum of a start pass's second partial in the lanes of term 1; dk:
// the lane's divided difference): the stop test of Sec. 4.2 on the pass's
// estimates in order.  Every wavefront of the problem comes to the same state.
__device__ inline void batch_next(const BatchArgs& a, const BProb& P, BState& S, double s, double mx, double dk) {
  const int lane = threadIdx.x & 63, nt = a.nt;
  const bool init = S.phase == kPhInit;
  ++S.phases;
  if (init && S.kind != kInitSub) S.scal = a.tol_a + a.tol_r * lane_of(mx, 1);
  const double est = fabs(P.delta * dk) * sqrt(s) / (P.rootN * S.scal);
  bool stop = false;  // no further Newton work for this problem
  if (init) {
    if (S.kind == kInitStep) S.tpar ^= 1;
    if (S.kind == kInitSub) S.upar ^= 1;
    S.ppar ^= 1;
    const double s0 = lane_of(s, 0), m0 = lane_of(mx, 1);
    if (!isfinite(s0) || (S.kind != kInitSub && !isfinite(m0))) {
      S.flags |= 2;
      stop = true;
    } else if (!(S.scal > 0.0)) {
      S.flags |= 4;
      stop = true;
    } else if (nt > a.m_max) {
      S.flags |= 1;  // not even one pass fits the term budget
      stop = true;
    } else {
      S.prev[0] = S.prev[1] = S.prev[2] = 0.0;
      S.prev[3] = lane_of(est, 0);
      S.k = 1;
      S.phase = kPhTerms;
    }
  } else {
    // lanes 0 .. 3: the four estimates before the pass; lanes 4 .. nt + 3: the
    // pass's; each of the latter tests the mean of its own and the four below
    const double p01 = lane == 0 ? S.prev[0] : S.prev[1], p23 = lane == 2 ? S.prev[2] : S.prev[3];
    const double up = __shfl_up(est, 4, 64);
    const double z = lane < 4 ? (lane < 2 ? p01 : p23) : up;
    double mean = __shfl_up(z, 4, 64);
    mean += __shfl_up(z, 3, 64);
    mean += __shfl_up(z, 2, 64);
    mean += __shfl_up(z, 1, 64);
    mean = 0.2 * (mean + z);
    const int j = lane - 4;
    const bool mine = j >= 0 && j < nt;
    const double sj = __shfl_up(s, 4, 64);
    const unsigned long long bad = __ballot(mine && !isfinite(sj));
    const unsigned long long hit = __ballot(mine && S.k + j >= 4 && mean < a.thresh);
    const int fb = bad ? __ffsll(bad) : 65, fh = hit ? __ffsll(hit) : 65;
    S.terms += nt;  // all terms of the pass are kept
#pragma unroll
    for (int m = 0; m < 4; ++m) S.prev[m] = lane_of(est, nt - 4 + m);
    if (fb <= fh && fb < 65) {
      S.flags |= 2;
      stop = true;
    } else if (fh < 65) {
      if (S.sub + 1 < P.s) {
        ++S.sub;
        S.kind = kInitSub;
        S.phase = kPhInit;
      } else {
        ++S.step;
        S.sub = 0;
        if (S.step == a.nsteps) {
          S.phase = kPhFinish;
        } else {
          S.kind = kInitStep;
          S.phase = kPhInit;
        }
      }
    } else if (S.k + 2 * nt - 1 > a.m_max) {
      S.flags |= 1;
      stop = true;
    } else {
      S.k += nt;
    }
  }
  // a failed problem still takes the finish pass, which copies the T of its
  // last completed step into the caller's array
  if (stop) S.phase = kPhFinish;
}

// One phase of every unfinished problem: a wavefront per tile (a strip of
// columns by a chunk of rows).  It first makes the problem's control step -
// every tile's wavefront alike, from the state and the partials of the pass
// before, which this pass does not overwrite (both alternate between two
// buffers) - and then the phase that comes out of it; the problem's first tile
// records the state.
//
// While most problems are unfinished the pass is bound by memory: eight FP64
// terms of 7.2 M cells read 554 MB from beyond the L2s (5 stencil words, q and p,
// plus halos) and write 115 MB in about 119 us, 5.6 TB/s where a large copy
// reaches 4.8: taking every second pass back to front finds the end of the pass
// before in the Infinity Cache (a run of 50 steps 70.4 -> 65.9 ms).  The 64 x 16
// LDS tiles on 512 threads that this replaces took 215 us for the same pass (two
// workgroups' loads per CU in flight, then eight barriered terms) and 92 ms for
// the run.  When only the longest problems are left, a pass costs what one
// wavefront takes to issue its rows (about 500 cycles a row of eight terms).  A
// control launch of its own after every pass cost 6 us and a launch gap (65.9 ->
// 57.1 ms).
template <int NT, class V>
__global__ __launch_bounds__(kMarchLanes) __attribute__((amdgpu_waves_per_eu(2))) void k_bt_ctrl_work(BatchArgs a) {
  static_assert(NT <= kBatchPartStride && NT % 4 == 0, "terms per pass");
  const int t = batch_tile(a.pass & 1);
  const int lane = threadIdx.x;
  const BTile tl = a.tile[t];
  if (tl.done) return;  // the tiles of a finished problem stop here, before its state is read
  BState S = a.state[(a.pass & 1) * a.nprob + tl.pid];
  const BProb P = a.prob[tl.pid];
  const long long pcap = static_cast<long long>(kBatchPartStride) * a.part_cap;
  {
    // the partials of the pass before and the next coefficients' addresses need
    // the tile record only: their loads go out beside the state's
    double s = 0.0, mx = 0.0;
    if (S.phases >= 0)
      batch_sums(a.part + (a.pass & 1) * pcap + static_cast<long long>(kBatchPartStride) * tl.src, tl.nsrc, s, mx);
    if (S.phase == kPhDone) {
      if (lane == 0) a.tile[t].done = 1;
      return;
    }
    if (S.phases < 0) {
      S.phases = 0;  // the first pass: nothing to test yet
    } else if (S.phase == kPhFinish) {
      // the finish pass is done: the problem's tiles return at entry from now on.
      // Both copies of the state say so: a wavefront of this pass that already
      // reads it returns likewise.
      S.phase = kPhDone;
      ++S.phases;
      if (lane == 0) {
        a.tile[t].done = 1;
        if (t == tl.tile0) {
          a.state[tl.pid] = S;
          a.state[a.nprob + tl.pid] = S;
          atomicAdd(a.ndone, 1);
        }
      }
      return;
    } else {
      const int k = S.phase == kPhInit ? 0 : S.k;
      sum_max_octets(s, mx);
      batch_next(a, P, S, s, mx, a.dk[P.coef_off + min(k + (lane & 7), a.m_max)]);
    }
    if (t == tl.tile0 && lane == 0) a.state[((a.pass & 1) ^ 1) * a.nprob + tl.pid] = S;
  }
  const MarchStrip st = march_strip(P.nx, NT, tl.strip);
  const int y0 = tl.y0, y1 = min(tl.y0 + a.rows, P.ny);
  double* part = a.part + ((a.pass & 1) ^ 1) * pcap + static_cast<long long>(kBatchPartStride) * t;
  if (S.phase == kPhFinish) {
    batch_finish<V>(a, P, S, st, y0, y1);
    return;
  }
  if (S.phase == kPhInit) {
    batch_start<V>(a, P, S, st, y0, y1, part);
    return;
  }
  const int grp = (S.k - 1) / NT;
  const V* qin = reinterpret_cast<const V*>((grp & 1) ? a.q1 : a.q0) + P.off;
  V* qout = reinterpret_cast<V*>((grp & 1) ? a.q0 : a.q1) + P.off;
  V* p = reinterpret_cast<V*>(S.ppar ? a.p1 : a.p0) + P.off;
  V shift[NT], dk[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    shift[j] = march_uniform(cv<V>(a.shift[P.coef_off + S.k + j]));
    dk[j] = march_uniform(cv<V>(a.dk[P.coef_off + S.k + j]));
  }
  double sum[NT];
  march_terms<NT, kBatchAhead, V>(reinterpret_cast<const V*>(a.coef) + P.off, a.ntot, qin, qout, p, P.nx, P.ny, st, y0, y1,
                        cv<V>(P.inv_g), shift, dk, sum, [] { return false; });
#pragma unroll
  for (int j = 0; j < NT; j += 4) {
    const double s4[4] = {sum[j], sum[j + 1], sum[j + 2], sum[j + 3]};
    const double v = sum4(s4, lane);
    if (lane < 4) part[j + lane] = v;
  }
}

// Partials of the problems of more than kBatchGate tiles, folded after the pass
// that left them: every tile of a problem adds up all of its partials, so without
// a fold the reads grow with the square of the tiles.  Bound by its launch.  Two
// steps of one 2048 x 2048 problem, 8 terms x 32 rows (1344 tiles): 1.22 -> 0.78
// ms, 4096 x 4096 9.1 -> 2.65, with tiles of 8 rows 6.8 -> 1.12 and 90 -> 4.0.
__global__ __launch_bounds__(kMarchLanes) void k_bt_fold(BatchArgs a) {
  const BFold f = a.fold[blockIdx.x];
  const int lane = threadIdx.x, copy = (a.pass & 1) ^ 1;  // the copy that the pass wrote
  const int phase = a.state[copy * a.nprob + f.pid].phase;
  if (phase >= kPhFinish) return;  // no next phase to find
  double* part = a.part + static_cast<long long>(kBatchPartStride) * copy * a.part_cap;
  double s = 0.0, mx = 0.0;
  batch_sums(part + static_cast<long long>(kBatchPartStride) * f.tile0, f.n, s, mx);
  sum_max_octets(s, mx);
  if (lane < kBatchPartStride)
    part[static_cast<long long>(kBatchPartStride) * f.slot + lane] = phase == kPhInit && lane == 1 ? mx : s;
}

__global__ void k_bt_reset(BatchArgs a) {
  const int pid = blockIdx.x * blockDim.x + threadIdx.x;
  if (pid == 0) *a.ndone = 0;
  if (pid < a.ntiles) a.tile[pid].done = 0;
  if (pid >= a.nprob) return;
  BState S{};
  S.phase = kPhInit;
  S.kind = kInitFirst;
  S.k = 1;
  S.phases = -1;
  a.state[pid] = S;
  a.state[a.nprob + pid] = S;
}

// Pack one problem's stencil (SoA, stride N) into the batch layout (SoA,
// stride ntot, offset off) and form g = F - J T0 (so that G(T) = J T + g).
__global__ __launch_bounds__(256) void k_batch_pack(int nx, int ny, const double* __restrict__ coef,
                                                    const double* __restrict__ F, const double* __restrict__ T0,
                                                    double* __restrict__ bcoef, double* __restrict__ g,
                                                    long long ntot, long long off) {
  const int N = nx * ny;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
    const int x = i % nx, y = i / nx;
    double jt = coef[i] * T0[i];
    if (x > 0) jt += coef[N + i] * T0[i - 1];
    if (x + 1 < nx) jt += coef[2 * N + i] * T0[i + 1];
    if (y > 0) jt += coef[3 * N + i] * T0[i - nx];
    if (y + 1 < ny) jt += coef[4 * N + i] * T0[i + nx];
    for (int d = 0; d < 5; ++d) bcoef[d * ntot + off + i] = coef[d * N + i];
    g[off + i] = F[i] - jt;
  }
}

template <class V>
hipError_t launch_work(const BatchArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.nt == 8)
    launch_timed(k_bt_ctrl_work<8, V>, dim3(a.ntiles), dim3(kMarchLanes), 0, s, e0, e1, a);
  else
    launch_timed(k_bt_ctrl_work<4, V>, dim3(a.ntiles), dim3(kMarchLanes), 0, s, e0, e1, a);
  return hipGetLastError();
}

}  // namespace

hipError_t batch_pack(int nx, int ny, const double* coef, const double* F, const double* T0, double* bcoef,
                      double* g, long long ntot, long long off, hipStream_t s) {
  const int N = nx * ny;
  int blocks = (N + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_batch_pack, dim3(blocks), dim3(256), 0, s, nx, ny, coef, F, T0, bcoef, g, ntot, off);
  return hipGetLastError();
}

hipError_t batch_reset(const BatchArgs& a, hipStream_t s) {
  const int n = a.nprob > a.ntiles ? a.nprob : a.ntiles;  // a thread per problem state and per tile
  hipLaunchKernelGGL(k_bt_reset, dim3((n + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t batch_phase(BatchArgs a, long long pass, int fp32, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  a.pass = static_cast<int>(pass & 1);
  const hipError_t e = fp32 ? launch_work<float>(a, s, e0, e1) : launch_work<double>(a, s, e0, e1);
  if (e != hipSuccess || a.nfold == 0) return e;
  hipLaunchKernelGGL(k_bt_fold, dim3(a.nfold), dim3(kMarchLanes), 0, s, a);
  return hipGetLastError();
}

}  // namespace erem
