// Newton-Leja evaluation of phi1(delta J) v on the device (Sec. 4.2):
//
//   q_0 = v,  p_0 = d_0 q_0,
//   q_k = ((J - c I)/gamma - xi_{k-1} I) q_{k-1},  p_k = p_{k-1} + d_k q_k   (Eq. newt)
//
// One pass advances four terms (2D, k_leja_terms) or two (3D, k_leja_zmarch):
// it reads the stencil of J, q_{k-1} and p, and writes p and the last q; every
// workgroup also stores its partial sums of q_k^2 (in FP64 in both
// precisions).  The stop test of the terms so far is made at the start of the
// next pass by every workgroup alike, while its first loads are in flight
// (leja_gate): the partials are added in a fixed order (so results are
// reproducible bit for bit), the scaled error estimates ||delta d_k q_k|| =
// |delta d_k| ||q_k||_2 / (sqrt(N) scal) formed, and 10^p * mean(last five
// estimates) < 1 tested (Sec. 4.2), after every kCheckEvery terms.  Once it
// holds, the first workgroup records it, and later passes write nothing: they
// still issue their first loads (the box passes those of their whole box), which
// are on their way before the flag is known, and add up the partials.
//
// Value type V is double (FP64 path) or float (mixed path: FP32 stencil,
// vectors and accumulation; FP64 divided differences, norms and update).
#include "device.h"
#include "leja.h"
#include "march.h"

#include <algorithm>
#include <cmath>

namespace erem {

namespace {

template <class V>
__device__ inline V to_v(double x) { return static_cast<V>(x); }

// Sum of one double over the 256-thread cell block; valid in thread 0.
__device__ inline double block_sum256(double v) {
  __shared__ double sh[kThreads / 64];
  v = wave_sum(v);
  const int t = threadIdx.x + threadIdx.y * kBX;
  if ((t & 63) == 0) sh[t >> 6] = v;
  __syncthreads();
  return t == 0 ? sh[0] + sh[1] + sh[2] + sh[3] : 0.0;
}

// Rows of tile j of k_leja_box, H to a box: as march_strip's columns.
template <int H>
__host__ __device__ inline MarchStrip box_rows(int ny, int j) {
  constexpr int inner = H - 2 * kTermsPerPass2;
  MarchStrip s;
  s.xs = j * inner;
  s.x0 = j == 0 ? 0 : s.xs + kTermsPerPass2;
  s.x1 = s.xs + H >= ny ? ny : s.xs + H - kTermsPerPass2;
  return s;
}

// Tiles of k_leja_cube along a direction of n cells, W to a box, and tile j.
__host__ __device__ inline int cube_tiles(int n, int W) { return n <= W ? 1 : 1 + (n - W + W - 5) / (W - 4); }
__host__ __device__ inline MarchStrip cube_tile(int n, int W, int j) {
  MarchStrip s;
  s.xs = j * (W - 4);
  s.x0 = j == 0 ? 0 : s.xs + 2;
  s.x1 = s.xs + W >= n ? n : s.xs + W - 2;
  return s;
}

__device__ inline int block_id() { return blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z); }

__global__ void k_leja_reset(LejaState* st, int nslots, int nterms) {
  for (int s = blockIdx.x; s < nslots; s += gridDim.x) {
    LejaState* t = st + s;
    for (int j = threadIdx.x; j <= nterms; j += blockDim.x) t->sums[j] = 0.0;
    if (threadIdx.x == 0) {
      t->stopped = -1;
      t->nonfinite = 0;
      t->checked = -1;
    }
  }
}

// q_0 = v, p_0 = d_0 q_0: a copy, at most kInitBlocks workgroups so that term
// 0 has few partials.
template <class V>
__global__ __launch_bounds__(kThreads) void k_leja_init(int N, const LejaCoef* __restrict__ cf,
                                              const double* __restrict__ v, V* __restrict__ q0,
                                              V* __restrict__ p, double* __restrict__ part) {
  const V d0 = to_v<V>(cf->dk[0]);
  double s = 0.0;
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < N; i += gridDim.x * kThreads) {
    const V vi = to_v<V>(v[i]);
    q0[i] = vi;
    p[i] = d0 * vi;
    s += static_cast<double>(vi) * static_cast<double>(vi);
  }
  s = block_sum256(s);
  if (threadIdx.x == 0) part[blockIdx.x] = s;  // ring slot 0
}

// The stop test of terms g.k1 .. g.k2 (none when g.k2 < g.k1), made by the
// whole workgroup (NW wavefronts): true when the evaluation has stopped, now or
// before.  Wavefront w adds the partials of the terms k1 + w, k1 + w + NW, ...;
// the estimates of the last nine terms are formed one per lane.  The leading
// workgroup records the sums and the outcome; another workgroup of the same
// launch that already reads the new flag comes to the same outcome by itself.
template <int NW>
__device__ inline bool leja_gate(const LejaCoef* __restrict__ cf, LejaState* st, const LejaGate& g, bool lead) {
  const bool was = *(volatile const int*)&st->stopped >= 0;
  if (g.k2 < g.k1) return was;
  __shared__ double sh[kGateTerms];
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = g.k2 - g.k1 + 1;
  const int j = g.k1 - 4 + lane;  // the lane's term (lanes 0 .. n + 3)
  double old = 0.0, ef = 0.0;
  if (lane < n + 4 && j >= 0) {
    ef = cf->estf[j];
    if (j < g.k1) old = st->sums[j];
  }
  for (int i = wave; i < n; i += NW) {
    const double s = wave_part_sum(g.src[i], g.cnt[i]);
    if (lane == 0) sh[i] = s;
  }
  __syncthreads();
  if (was) return true;
  // lanes 0 .. 3: the terms before k1; lanes 4 .. n + 3: the new ones, each
  // testing the mean of its own and the four lanes below
  const bool mine = lane >= 4 && lane < n + 4;
  const double S = mine ? sh[lane - 4] : old;
  const double est = ef * sqrt(S);
  double mean = __shfl_up(est, 4, 64);
  mean += __shfl_up(est, 3, 64);
  mean += __shfl_up(est, 2, 64);
  mean += __shfl_up(est, 1, 64);
  mean += est;
  const bool bad = mine && !isfinite(S);
  const unsigned long long hit = __ballot(bad || (mine && j >= 4 && 0.2 * mean < cf->thresh));
  const int stop = hit ? g.k1 - 4 + __ffsll(hit) - 1 : -1;  // the first term that passes
  if (lead && tid < 64) {
    const int last = stop >= 0 ? stop : g.k2;
    if (mine && j <= last) st->sums[j] = S;
    if (bad && j == stop) st->nonfinite = 1;
    if (lane == 0) {
      st->checked = last;
      if (stop >= 0) st->stopped = stop;
    }
  }
  return stop >= 0;
}

template <int DIM, class V>
__global__ __launch_bounds__(kThreads) void k_leja_term(Dims d, const LejaCoef* __restrict__ cf,
                                              const V* __restrict__ coef, const V* __restrict__ qin,
                                              V* __restrict__ qout, V* __restrict__ p,
                                              const LejaState* __restrict__ st, double* __restrict__ part,
                                              int nb, int k) {
  // the stop flag is read while the operand loads are in flight; nothing is
  // written before it is known
  const bool stopped = *(volatile const int*)&st->stopped >= 0;
  const int tile = xcd_tile_id();
  const int tx = tile % gridDim.x, ty = (tile / gridDim.x) % gridDim.y;
  const int x = tx * kBX + threadIdx.x;
  const int y = ty * kBY + threadIdx.y;
  const int z = tile / (gridDim.x * gridDim.y);
  double s = 0.0;
  if (x < d.nx && y < d.ny) {
    const int N = d.N;
    const int i = x + d.nx * (y + d.ny * z);
    const V qi = qin[i];
    V jq = coef[i] * qi;
    jq += coef[N + i] * qin[x > 0 ? i - 1 : i];
    jq += coef[2 * N + i] * qin[x + 1 < d.nx ? i + 1 : i];
    jq += coef[3 * N + i] * qin[y > 0 ? i - d.nx : i];
    jq += coef[4 * N + i] * qin[y + 1 < d.ny ? i + d.nx : i];
    if (DIM == 3) {
      const int pl = d.nx * d.ny;
      jq += coef[5 * N + i] * qin[z > 0 ? i - pl : i];
      jq += coef[6 * N + i] * qin[z + 1 < d.nz ? i + pl : i];
    }
    const V r = jq * to_v<V>(cf->inv_g) - to_v<V>(cf->shift[k]) * qi;
    const V pi = p[i];
    if (stopped) return;
    p[i] = pi + to_v<V>(cf->dk[k]) * r;
    qout[i] = r;
    s = static_cast<double>(r) * static_cast<double>(r);
  } else if (stopped) {
    return;
  }
  s = block_sum256(s);
  if (threadIdx.x == 0 && threadIdx.y == 0) part[(k % kLejaRing) * nb + tile] = s;  // slot of the tile
}

// Four Newton terms in one pass on large 2D grids (march.h): a workgroup's four
// wavefronts take four consecutive chunks of rows of one strip, and leave one
// partial per term.  At 640 x 640 a pass is still half latencies (launch, first
// rows, stop test, 16 rows): 10 us with its stop test, where a pass with LDS tiles
// and a stop-test launch took 16 and two launch gaps.
template <int NT, class V>
__global__ __launch_bounds__(kThreads) void k_leja_terms(Dims d, const LejaCoef* __restrict__ cf,
                                               const V* __restrict__ coef, const V* __restrict__ qin,
                                               V* __restrict__ qout, V* __restrict__ p, LejaState* st,
                                               double* __restrict__ part, LejaGate g, int stride, int rows, int k) {
  constexpr int NW = kThreads / 64;
  const int tile = xcd_tile_id();
  const int strips = march_strips(d.nx, NT);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int y0 = ((tile / strips) * NW + wave) * rows, y1 = min(y0 + rows, d.ny);
  V shift[NT], dk[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    shift[t] = march_uniform(to_v<V>(cf->shift[k + t]));
    dk[t] = march_uniform(to_v<V>(cf->dk[k + t]));
  }
  double sum[NT];
  bool stop;
  if (y0 < d.ny) {
    stop = !march_terms<NT, 4, V>(coef, d.N, qin, qout, p, d.nx, d.ny, march_strip(d.nx, NT, tile % strips), y0, y1,
                                  to_v<V>(cf->inv_g), shift, dk, sum, [&] { return leja_gate<NW>(cf, st, g, tile == 0); });
  } else {
    stop = leja_gate<NW>(cf, st, g, false);
#pragma unroll
    for (int t = 0; t < NT; ++t) sum[t] = 0.0;
  }
  if (stop) return;  // every wavefront of the workgroup alike
  __shared__ double red[NT][NW];
  static_assert(NT == 4, "the sums of a pass are reduced together");
  const double s4 = sum4(sum, lane);
  if (lane < 4) red[lane][wave] = s4;
  __syncthreads();
  if (threadIdx.x < NT) {
    const int t = threadIdx.x;
    part[((k + t) % kLejaRing) * stride + tile] = red[t][0] + red[t][1] + red[t][2] + red[t][3];
  }
}

// Four Newton terms in one pass on small 2D grids: a workgroup of sixteen
// wavefronts holds a box of 64 columns x 16 R rows, R cells of a column per thread,
// and forms the four terms on a box that shrinks by a cell a side per term.  q's
// east and west neighbours come from the neighbouring lanes, the rows above and
// below from LDS (double buffered, a barrier per term).  The first pass of a
// substep (FIRST) also sets q_0 = src and p_0 = d_0 q_0 and has a fifth partial, of
// term 0.
//
// On a grid that does not fill the chip a pass is a chain of latencies.  All loads
// of the box go out at once, ahead of the stop test, where k_leja_terms waits for
// its rows in turn: 333 x 77 8.1 -> 5.5 us a pass and a phi1 action, with the start
// pass gone, 168 -> 141 us; 512 x 512 9.1 -> 6.8 us.  Past one box per CU the rows
// loaded twice (16 R for 16 R - 8) and the second round cost more than that.
template <int R, bool FIRST, class V>
__global__ __launch_bounds__(1024) void k_leja_box(Dims d, const LejaCoef* __restrict__ cf,
                                         const V* __restrict__ coef, const double* __restrict__ src,
                                         const V* __restrict__ qin, V* __restrict__ qout, V* __restrict__ p,
                                         LejaState* st, double* __restrict__ part, LejaGate g, int stride, int k) {
  constexpr int NT = kTermsPerPass2, NW = 16, H = NW * R;
  __shared__ V sq[2][H + 2][kMarchLanes];  // a row of zeros below and above the box
  __shared__ double red[NT + 1][NW];
  const int tile = xcd_tile_id();
  const int strips = march_strips(d.nx, NT);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const MarchStrip sx = march_strip(d.nx, NT, tile % strips), sy = box_rows<H>(d.ny, tile / strips);
  const int gx = sx.xs + lane;
  const bool xout = gx >= sx.x0 && gx < sx.x1;
  V c[R][5], q[R], pv[R];
  int cell[R];
  bool in[R], out[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int gy = sy.xs + wave * R + r;
    in[r] = gx < d.nx && gy < d.ny;
    out[r] = xout && gy >= sy.x0 && gy < sy.x1;
    cell[r] = min(gx, d.nx - 1) + d.nx * min(gy, d.ny - 1);  // every load is valid
    q[r] = FIRST ? to_v<V>(src[cell[r]]) : qin[cell[r]];
    if (!FIRST) pv[r] = p[cell[r]];
#pragma unroll
    for (int e = 0; e < 5; ++e) c[r][e] = coef[static_cast<long long>(e) * d.N + cell[r]];
  }
  const V ig = to_v<V>(cf->inv_g);
  V shift[NT], dk[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    shift[t] = to_v<V>(cf->shift[k + t]);
    dk[t] = to_v<V>(cf->dk[k + t]);
  }
  const V d0 = FIRST ? to_v<V>(cf->dk[0]) : V(0);
  __builtin_amdgcn_sched_barrier(0);
  if (wave == 0 || wave == NW - 1) {
    sq[0][wave == 0 ? 0 : H + 1][lane] = V(0);
    sq[1][wave == 0 ? 0 : H + 1][lane] = V(0);
  }
  if (leja_gate<NW>(cf, st, g, tile == 0)) return;
  double sum[NT], s0 = 0.0;
#pragma unroll
  for (int t = 0; t < NT; ++t) sum[t] = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    q[r] = in[r] ? q[r] : V(0);
#pragma unroll
    for (int e = 0; e < 5; ++e) c[r][e] = in[r] ? c[r][e] : V(0);
    if (FIRST) {
      pv[r] = d0 * q[r];
      const double v = out[r] ? static_cast<double>(q[r]) : 0.0;
      s0 += v * v;
    }
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int y = wave * R + 1;  // LDS row of the thread's first cell
#pragma unroll
    for (int r = 0; r < R; ++r) sq[t & 1][y + r][lane] = q[r];
    __syncthreads();
    V qo[R];
    const V below = sq[t & 1][y - 1][lane], above = sq[t & 1][y + R][lane];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      V jq = c[r][1] * west(q[r]);
      jq = fma(c[r][0], q[r], jq);
      jq = fma(c[r][2], east(q[r]), jq);
      jq = fma(c[r][3], r > 0 ? q[r > 0 ? r - 1 : 0] : below, jq);
      jq = fma(c[r][4], r + 1 < R ? q[r + 1 < R ? r + 1 : 0] : above, jq);
      qo[r] = fma(jq, ig, -(shift[t] * q[r]));
      pv[r] = fma(dk[t], qo[r], pv[r]);
      const double v = out[r] ? static_cast<double>(qo[r]) : 0.0;
      sum[t] += v * v;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) q[r] = qo[r];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (!out[r]) continue;
    p[cell[r]] = pv[r];
    qout[cell[r]] = q[r];
  }
  static_assert(NT == 4, "the sums of a pass are reduced together");
  const double s4 = sum4(sum, lane);
  if (lane < NT) red[lane][wave] = s4;
  if (FIRST) {
    s0 = wave_sum(s0);
    if (lane == 0) red[NT][wave] = s0;
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < NT + (FIRST ? 1 : 0)) {
    double s = red[t][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[t][w];
    part[(t < NT ? (k + t) % kLejaRing : 0) * stride + tile] = s;
  }
}

// Two Newton terms in one pass on 3D grids.  A workgroup holds a tile of 64 x
// TY columns plus a halo of one (the box) and marches through a chunk of
// planes: on the step that has plane z + 1 of q_{k-1}, term k is formed on
// plane z of the box and term k + 1 on plane z - 1 of the tile.  A thread owns
// SH cells of one box column and keeps their q, term-k values and stencil of
// the planes it needs in registers; the x and y neighbours come from LDS (one
// plane of q_{k-1} with a further halo, one plane of term k, each double
// buffered, so a step has one barrier).  Loads of a plane are issued one step
// ahead.  The multiply-adds are spelled out so that the terms round as in the
// one-term pass whatever the compiler contracts.
//
// Bound by memory: per cell and pair of terms the seven stencil words, q_{k-1},
// p in and out and the last q, 88 B where two one-term passes move 176.  Turned
// passes (zmarch_turns) find some of it in the Infinity Cache.  On 256^3 (FP64) a
// pass reads 1.34 GB from beyond the L2s (planes at the ends of chunks and halos
// twice) and writes 0.27 in 300 us, 5.4 TB/s: 248 -> 150 us per term; on 128^3 0.22
// GB in 35.5 us, 28 -> 18 us per term.
template <int TY, int SH, int NTH, bool FLIP, class V>
__global__ __launch_bounds__(NTH) void k_leja_zmarch(Dims d, const LejaCoef* __restrict__ cf,
                                           const V* __restrict__ coef, const V* __restrict__ qin,
                                           V* __restrict__ qout, V* __restrict__ p, LejaState* st,
                                           double* __restrict__ part, LejaGate g, int stride, int zc, int k) {
  constexpr int WB = kBX + 2, HB = TY + 2;   // box
  constexpr int NW = NTH / 64;
  constexpr int NS = (HB + SH - 1) / SH;     // strips of SH cells per box column
  static_assert(NS * WB <= NTH && 2 * (WB + HB) <= NTH, "a thread per strip, a thread per ring cell");
  constexpr int WQ = WB + 2, HQ = NS * SH + 2;  // q_{k-1}: one more cell around (strips may pass the box's top)
  __shared__ V sq[2][HQ][WQ], s1[2][HQ][WQ];
  const int tid = threadIdx.x;
  const int nx = d.nx, ny = d.ny, nz = d.nz, N = d.N;
  const int pl = nx * ny;
  const int tx = (nx + kBX - 1) / kBX, ty = (ny + TY - 1) / TY;
  const int tile = xcd_tile_id();
  const int x0 = (tile % tx) * kBX, y0 = ((tile / tx) % ty) * TY;
  const int z0 = (tile / (tx * ty)) * zc, z1 = min(z0 + zc, nz);
  const bool act = tid < NS * WB;
  const int bx = act ? tid % WB : 0, b0 = act ? (tid / WB) * SH : 0;  // box column, first box row
  const int gx = x0 - 1 + bx;
  const bool xin = act && gx >= 0 && gx < nx, xout = xin && bx >= 1 && bx <= kBX;
  int cell[SH];          // clamped plane offset of each cell: every load is valid
  bool in[SH], out[SH];  // in the grid; an output
#pragma unroll
  for (int r = 0; r < SH; ++r) {
    const int by = b0 + r, gy = y0 - 1 + by;
    in[r] = xin && by < HB && gy >= 0 && gy < ny;
    out[r] = in[r] && xout && by >= 1 && by <= TY;
    cell[r] = min(max(gx, 0), nx - 1) + nx * min(max(gy, 0), ny - 1);
  }
  // the ring around the box, one cell per thread: bottom, top, left, right
  int rx = 0, ry = 0;
  bool ring = false;
  {
    int e = tid;
    if (e < 2 * WB) {
      rx = e % WB + 1;
      ry = e < WB ? 0 : HB + 1;
      ring = true;
    } else if (e < 2 * (WB + HB)) {
      e -= 2 * WB;
      ry = e % HB + 1;
      rx = e < HB ? 0 : WB + 1;
      ring = true;
    }
  }
  const int rgx = x0 - 2 + rx, rgy = y0 - 2 + ry;
  const bool rin = ring && rgx >= 0 && rgx < nx && rgy >= 0 && rgy < ny;
  const int rcell = min(max(rgx, 0), nx - 1) + nx * min(max(rgy, 0), ny - 1);
  auto plane = [&](int z) {  // FLIP: counted from the top
    const int zz = min(max(z, 0), nz - 1);
    return static_cast<long long>(FLIP ? nz - 1 - zz : zz) * pl;
  };

  V c0[SH][7], c1[SH][7];              // stencil of planes z - 1 and z (then z + 1)
  V qm[SH], qc[SH], qp[SH], qr;        // q_{k-1} on planes z - 1, z, z + 1; the ring cell of z + 1
  V tm[SH], tc[SH];                    // term k on planes z - 2, z - 1
  V pc[SH], pn[SH];                    // p on planes z - 1, z
  const int zs = z0 - 1;               // first plane of term k
  {
    const long long o0 = plane(zs - 1), o1 = plane(zs), o2 = plane(zs + 1);
#pragma unroll
    for (int r = 0; r < SH; ++r) {
      qm[r] = qin[o0 + cell[r]];
      qc[r] = qin[o1 + cell[r]];
      qp[r] = qin[o2 + cell[r]];
#pragma unroll
      for (int e = 0; e < 7; ++e) c1[r][e] = coef[static_cast<long long>(e) * N + o1 + cell[r]];
      pn[r] = tm[r] = tc[r] = pc[r] = V(0);  // plane z0 - 1 has no outputs
#pragma unroll
      for (int e = 0; e < 7; ++e) c0[r][e] = V(0);
    }
    const V q1 = rin ? qin[o1 + rcell] : V(0);
    qr = rin ? qin[o2 + rcell] : V(0);
#pragma unroll
    for (int r = 0; r < SH; ++r) {
      qm[r] = in[r] && zs >= 1 ? qm[r] : V(0);
      qc[r] = in[r] && zs >= 0 ? qc[r] : V(0);
      qp[r] = in[r] ? qp[r] : V(0);
    }
    if (leja_gate<NW>(cf, st, g, tile == 0)) return;
    if (act) {
#pragma unroll
      for (int r = 0; r < SH; ++r) {
        sq[zs & 1][b0 + r + 1][bx + 1] = qc[r];
        s1[(zs & 1) ^ 1][b0 + r + 1][bx + 1] = V(0);
      }
    }
    if (ring) {
      sq[zs & 1][ry][rx] = zs >= 0 ? q1 : V(0);
      s1[0][ry][rx] = s1[1][ry][rx] = V(0);
    }
    __syncthreads();
  }
  const V ig = to_v<V>(cf->inv_g);
  const V sh0 = to_v<V>(cf->shift[k]), sh1 = to_v<V>(cf->shift[k + 1]);
  const V d0 = to_v<V>(cf->dk[k]), d1 = to_v<V>(cf->dk[k + 1]);
  double a0 = 0.0, a1 = 0.0;
  for (int z = zs; z <= z1; ++z) {
    const int par = z & 1;
    // the next plane's loads
    V cn[SH][7], qn[SH], pf[SH], qrn = V(0);
    const long long oq = plane(z + 2), oc = plane(z + 1);
#pragma unroll
    for (int r = 0; r < SH; ++r) {
      qn[r] = pf[r] = V(0);
#pragma unroll
      for (int e = 0; e < 7; ++e) cn[r][e] = V(0);
    }
    if (z < z1) {
#pragma unroll
      for (int r = 0; r < SH; ++r) {
        qn[r] = qin[oq + cell[r]];
#pragma unroll
        for (int e = 0; e < 7; ++e) cn[r][e] = coef[static_cast<long long>(e) * N + oc + cell[r]];
        if (out[r] && z + 1 < z1) pf[r] = p[oc + cell[r]];
      }
      qrn = qin[oq + rcell];
    }
    __builtin_amdgcn_sched_barrier(0);
    const bool zin = z >= 0 && z < nz, wr = z - 1 >= z0;
    V t1[SH];
#pragma unroll
    for (int r = 0; r < SH; ++r) {
      // term k on plane z
      const int ly = b0 + r + 1, lx = bx + 1;
      V jq = c1[r][0] * qc[r];
      jq = fma(c1[r][1], sq[par][ly][lx - 1], jq);
      jq = fma(c1[r][2], sq[par][ly][lx + 1], jq);
      jq = fma(c1[r][3], (r > 0 ? qc[r > 0 ? r - 1 : 0] : sq[par][ly - 1][lx]), jq);
      jq = fma(c1[r][4], (r + 1 < SH ? qc[r + 1 < SH ? r + 1 : 0] : sq[par][ly + 1][lx]), jq);
      jq = fma(c1[r][5], FLIP ? qp[r] : qm[r], jq);
      jq = fma(c1[r][6], FLIP ? qm[r] : qp[r], jq);
      const V v = fma(jq, ig, -(sh0 * qc[r]));
      t1[r] = in[r] && zin ? v : V(0);
    }
    if (wr) {
#pragma unroll
      for (int r = 0; r < SH; ++r) {
        // term k + 1 on plane z - 1
        const int ly = b0 + r + 1, lx = bx + 1;
        V jq = c0[r][0] * tc[r];
        jq = fma(c0[r][1], s1[par ^ 1][ly][lx - 1], jq);
        jq = fma(c0[r][2], s1[par ^ 1][ly][lx + 1], jq);
        jq = fma(c0[r][3], (r > 0 ? tc[r > 0 ? r - 1 : 0] : s1[par ^ 1][ly - 1][lx]), jq);
        jq = fma(c0[r][4], (r + 1 < SH ? tc[r + 1 < SH ? r + 1 : 0] : s1[par ^ 1][ly + 1][lx]), jq);
        jq = fma(c0[r][5], FLIP ? t1[r] : tm[r], jq);
        jq = fma(c0[r][6], FLIP ? tm[r] : t1[r], jq);
        const V v = fma(jq, ig, -(sh1 * tc[r]));
        if (out[r]) {
          const long long o = plane(z - 1) + cell[r];
          p[o] = fma(d1, v, fma(d0, tc[r], pc[r]));
          qout[o] = v;
          a0 += static_cast<double>(tc[r]) * static_cast<double>(tc[r]);
          a1 += static_cast<double>(v) * static_cast<double>(v);
        }
      }
    }
    if (act) {
#pragma unroll
      for (int r = 0; r < SH; ++r) {
        s1[par][b0 + r + 1][bx + 1] = t1[r];
        sq[par ^ 1][b0 + r + 1][bx + 1] = qp[r];
      }
    }
    if (ring) sq[par ^ 1][ry][rx] = qr;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SH; ++r) {
      qm[r] = qc[r];
      qc[r] = qp[r];
      qp[r] = in[r] && z + 2 < nz ? qn[r] : V(0);
      tm[r] = tc[r];
      tc[r] = t1[r];
      pc[r] = pn[r];
      pn[r] = pf[r];
#pragma unroll
      for (int e = 0; e < 7; ++e) {
        c0[r][e] = c1[r][e];
        c1[r][e] = cn[r][e];
      }
    }
    qr = rin && z + 2 < nz ? qrn : V(0);
  }
  __shared__ double red[2][NW];
  a0 = wave_sum(a0);
  a1 = wave_sum(a1);
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = a0;
    red[1][tid >> 6] = a1;
  }
  __syncthreads();
  if (tid < 2) {
    double s = red[tid][0];
    for (int w = 1; w < NW; ++w) s += red[tid][w];
    part[((k + tid) % kLejaRing) * stride + tile] = s;
  }
}

// Two Newton terms in one pass on small 3D grids: a workgroup of eight wavefronts
// holds a box of 32 x 16 columns, a thread a column of ZC planes and two more on
// either side, and forms term k on ZC + 2 planes and term k + 1 on the ZC of the
// output, 28 x 12 columns.  East and west neighbours come from the neighbouring
// lanes (a row's first and last take a wrong one, in the halo or against a
// coefficient of 0), north and south ones from LDS, above and below are the
// thread's own.  FIRST as in k_leja_box.
template <int ZC, bool FIRST, class V>
__global__ __launch_bounds__(kCubeX * kCubeY) void k_leja_cube(Dims d, const LejaCoef* __restrict__ cf,
                                                     const V* __restrict__ coef, const double* __restrict__ src,
                                                     const V* __restrict__ qin, V* __restrict__ qout,
                                                     V* __restrict__ p, LejaState* st, double* __restrict__ part,
                                                     LejaGate g, int stride, int k) {
  constexpr int NW = kCubeX * kCubeY / 64, NZ = ZC + 2;  // planes of term k
  __shared__ V sq[NZ][kCubeY + 2][kCubeX], s1[ZC][kCubeY + 2][kCubeX];
  __shared__ double red[3][NW];
  const int nx = d.nx, ny = d.ny, nz = d.nz, N = d.N;
  const int tile = xcd_tile_id();
  const int tx = cube_tiles(nx, kCubeX), ty = cube_tiles(ny, kCubeY);
  const MarchStrip bx = cube_tile(nx, kCubeX, tile % tx), by = cube_tile(ny, kCubeY, (tile / tx) % ty);
  const int z0 = tile / (tx * ty) * ZC;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lx = tid % kCubeX, ly = tid / kCubeX;
  const int gx = bx.xs + lx, gy = by.xs + ly;
  const bool in = gx < nx && gy < ny;
  const bool out = gx >= bx.x0 && gx < bx.x1 && gy >= by.x0 && gy < by.x1;
  const int cell = min(gx, nx - 1) + nx * min(gy, ny - 1);  // every load is valid
  auto plane = [&](int z) { return nx * ny * min(max(z, 0), nz - 1); };
  V c[NZ][7], q[ZC + 4], pv[ZC];
#pragma unroll
  for (int u = 0; u < ZC + 4; ++u) {
    const int o = plane(z0 - 2 + u);
    q[u] = FIRST ? to_v<V>((src + o)[cell]) : (qin + o)[cell];
  }
#pragma unroll
  for (int u = 0; u < NZ; ++u) {
    const int o = plane(z0 - 1 + u);
#pragma unroll
    for (int e = 0; e < 7; ++e) c[u][e] = (coef + e * N + o)[cell];
  }
  if (!FIRST) {
#pragma unroll
    for (int u = 0; u < ZC; ++u) pv[u] = (p + plane(z0 + u))[cell];
  }
  const V ig = to_v<V>(cf->inv_g);
  const V sh0 = to_v<V>(cf->shift[k]), sh1 = to_v<V>(cf->shift[k + 1]);
  const V d0 = to_v<V>(cf->dk[k]), d1 = to_v<V>(cf->dk[k + 1]);
  const V dz = FIRST ? to_v<V>(cf->dk[0]) : V(0);
  __builtin_amdgcn_sched_barrier(0);
  if (ly == 0 || ly == kCubeY - 1) {  // rows of zeros below and above the box
    const int y = ly == 0 ? 0 : kCubeY + 1;
#pragma unroll
    for (int u = 0; u < NZ; ++u) sq[u][y][lx] = V(0);
#pragma unroll
    for (int u = 0; u < ZC; ++u) s1[u][y][lx] = V(0);
  }
  if (leja_gate<NW>(cf, st, g, tile == 0)) return;
  double a0 = 0.0, a1 = 0.0, s0 = 0.0;
#pragma unroll
  for (int u = 0; u < ZC + 4; ++u) {
    const int z = z0 - 2 + u;
    q[u] = in && z >= 0 && z < nz ? q[u] : V(0);
    if (u >= 1 && u <= NZ) sq[u - 1][ly + 1][lx] = q[u];
  }
  if (FIRST) {
#pragma unroll
    for (int u = 0; u < ZC; ++u) {
      pv[u] = dz * q[u + 2];
      const double v = out && z0 + u < nz ? static_cast<double>(q[u + 2]) : 0.0;
      s0 += v * v;
    }
  }
  __syncthreads();
  V t[NZ];
#pragma unroll
  for (int u = 0; u < NZ; ++u) {
    const int z = z0 - 1 + u;
    const V qc = q[u + 1];
    V jq = c[u][0] * qc;
    jq = fma(c[u][1], west(qc), jq);
    jq = fma(c[u][2], east(qc), jq);
    jq = fma(c[u][3], sq[u][ly][lx], jq);
    jq = fma(c[u][4], sq[u][ly + 2][lx], jq);
    jq = fma(c[u][5], q[u], jq);
    jq = fma(c[u][6], q[u + 2], jq);
    const V v = fma(jq, ig, -(sh0 * qc));
    t[u] = in && z >= 0 && z < nz ? v : V(0);
    if (u >= 1 && u <= ZC) s1[u - 1][ly + 1][lx] = t[u];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < ZC; ++u) {
    const V qc = t[u + 1];
    V jq = c[u + 1][0] * qc;
    jq = fma(c[u + 1][1], west(qc), jq);
    jq = fma(c[u + 1][2], east(qc), jq);
    jq = fma(c[u + 1][3], s1[u][ly][lx], jq);
    jq = fma(c[u + 1][4], s1[u][ly + 2][lx], jq);
    jq = fma(c[u + 1][5], t[u], jq);
    jq = fma(c[u + 1][6], t[u + 2], jq);
    const V v = fma(jq, ig, -(sh1 * qc));
    if (out && z0 + u < nz) {
      const int o = plane(z0 + u);
      (p + o)[cell] = fma(d1, v, fma(d0, qc, pv[u]));
      (qout + o)[cell] = v;
      a0 += static_cast<double>(qc) * static_cast<double>(qc);
      a1 += static_cast<double>(v) * static_cast<double>(v);
    }
  }
  const double s4[4] = {a0, a1, s0, 0.0};
  const double s = sum4(s4, lane);
  if (lane < 3) red[lane][wave] = s;
  __syncthreads();
  if (tid < (FIRST ? 3 : 2)) {
    double v = red[tid][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[tid][w];
    part[(tid < 2 ? (k + tid) % kLejaRing : 0) * stride + tile] = v;
  }
}

// Partials of up to kGateTerms terms folded to kFoldParts each, for launches
// with more workgroups than the gate should add up.
__global__ __launch_bounds__(64) void k_leja_fold(const LejaState* st, LejaGate g, double* __restrict__ dst) {
  if (*(volatile const int*)&st->stopped >= 0) return;
  const int i = blockIdx.y, n = g.cnt[i];
  const int per = (n + kFoldParts - 1) / kFoldParts;
  const int b0 = min(n, static_cast<int>(blockIdx.x) * per);
  const double s = wave_part_sum(g.src[i] + b0, min(per, n - b0));
  if (threadIdx.x == 0) dst[i * kFoldParts + blockIdx.x] = s;
}

// The stop test on its own (one workgroup), where no pass follows that makes it.
__global__ __launch_bounds__(kThreads) void k_leja_check(const LejaCoef* __restrict__ cf, LejaState* st, LejaGate g) {
  (void)leja_gate<kThreads / 64>(cf, st, g, true);
}

// u = (first ? 0 : u) + delta * p (+ zt)  (FP64 update of the substep
// increment; zt, when not null, is a fixed vector added on every substep).  The
// last workgroup makes the stop test of the substep's last terms instead.
template <class V>
__global__ __launch_bounds__(kThreads) void k_substep_update(int N, double* __restrict__ u, const V* __restrict__ p,
                                                   double delta, int first, const double* __restrict__ zt,
                                                   const LejaCoef* __restrict__ cf, LejaState* st, LejaGate g) {
  if (blockIdx.x + 1 == gridDim.x) {
    (void)leja_gate<kThreads / 64>(cf, st, g, true);
    return;
  }
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= N) return;
  const double pi = static_cast<double>(p[i]);
  double r = first ? delta * pi : u[i] + delta * pi;
  if (zt) r += zt[i];
  u[i] = r;
}

__global__ void k_cast_f32(const double* __restrict__ a, float* __restrict__ b, long long n) {
  for (long long i = blockIdx.x * static_cast<long long>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<long long>(gridDim.x) * blockDim.x)
    b[i] = static_cast<float>(a[i]);
}

constexpr int kCoefM = kCoefMaxN + 1;  // largest order of the augmented matrix
constexpr int kCoefLd = kCoefM + 1;     // row stride of the LDS matrices (rows on distinct banks)
constexpr int kTaylorDegree = 20;

// Coefficients of one phi1 evaluation from the reduction slots (one
// workgroup of 16 x 16 threads; launch_leja_coef).  Thread (ty, tx) owns the
// entries (ty + 16 a, tx + 16 b), a, b < RB, of the lower triangle of the two
// LDS matrices; RB = ceil((n + 1) / 16) blocks of 16 rows cover the matrix.
template <int RB>
__global__ __launch_bounds__(kCoefThreads) void k_leja_coef(LejaCoefArgs a) {
  // every operation rounded on its own, in the host routine's order, so the
  // coefficients equal the host's bit for bit
#pragma clang fp contract(off)
  __shared__ double sA[kCoefM * kCoefLd], sB[kCoefM * kCoefLd];
  __shared__ double dg[kCoefM], sd[kCoefM], dd[kCoefM], inv[kTaylorDegree + 1];
  __shared__ double bc[6];
  __shared__ double wmax[kCoefThreads / 64];
  __shared__ int okf, hit;
  const int t = threadIdx.x;
  const int tx = t & 15, ty = t >> 4;
  if (t < 64) {
    // fold the 64 slots of each target (the encodings order like the values)
    unsigned long long lo = a.red->lo[t], hi = a.red->hi[t];
    unsigned long long sm = a.red->tmax[t];
    for (int off = 32; off > 0; off >>= 1) {
      const unsigned long long l2 = __shfl_xor(lo, off, 64);
      const unsigned long long h2 = __shfl_xor(hi, off, 64);
      const unsigned long long s2 = __shfl_xor(sm, off, 64);
      lo = l2 < lo ? l2 : lo;
      hi = h2 > hi ? h2 : hi;
      sm = s2 > sm ? s2 : sm;
    }
    if (t == 0) {
      const double alpha = ord_decode(lo), beta = ord_decode(hi), tm = ord_decode(sm);
      const double width = beta - alpha;
      const double mag = fmax(fabs(alpha), fabs(beta));
      const double scal = a.tol_a + a.tol_r * tm;
      bool ok = isfinite(tm) && scal > 0.0 && isfinite(width) && !(width <= 1e-14 * mag || width == 0.0);
      if (ok) {
        int s = 1;
        if (a.rho > 0.0) {
          const double q = ceil(a.h * width / a.rho);
          s = q >= a.smax ? a.smax : (q > 1.0 ? static_cast<int>(q) : 1);
        }
        ok = s == a.s;
      }
      const double cc = 0.5 * (alpha + beta), gg = 0.25 * (beta - alpha);
      const double delta = a.h / a.s;
      bc[0] = cc;
      bc[1] = gg;
      bc[2] = delta;
      bc[3] = delta * cc;
      bc[4] = delta * gg;
      bc[5] = scal;
      okf = ok;
      hit = ok && a.cache->n >= a.n && a.cache->hc == bc[3] && a.cache->hg == bc[4];
    }
  }
  __syncthreads();
  if (!okf) {
    for (int j = t; j < a.s; j += kCoefThreads) {
      a.st[j].stopped = 0;
      a.st[j].checked = -2;  // refused: the host evaluates again
    }
    return;
  }
  const int n = a.n, M = n + 1;
  if (hit) {
    if (t < n) dd[t] = a.cache->d[t];
  } else {
    // Augmented lower-bidiagonal matrix: diagonal (0, hc + hg xi_0, ...,
    // hc + hg xi_{n-1}), subdiagonal A[1][0] = 1, A[i][i-1] = hg (i >= 2).
    // The first column of its exponential is (1, phi1(hc I + hg L) e_1), the
    // divided differences of phi1(hc + hg xi).  Scaling by 2^-q brings its
    // 1-norm (the largest column sum) to at most 1/2.
    const double hc = bc[3], hg = bc[4];
    double nrm = 0.0;
    if (t < M) {
      const double dj = t == 0 ? 0.0 : hc + hg * a.xi[t - 1];
      const double below = t + 1 < M ? (t == 0 ? 1.0 : fabs(hg)) : 0.0;
      nrm = fabs(dj) + below;
    }
    for (int off = 32; off > 0; off >>= 1) nrm = fmax(nrm, __shfl_xor(nrm, off, 64));
    if ((t & 63) == 0) wmax[t >> 6] = nrm;
    // E = I on the leading M x M block, zero elsewhere (rows and columns past
    // M and the upper triangle stay zero throughout)
    for (int e = t; e < kCoefM * kCoefLd; e += kCoefThreads) {
      const int i = e / kCoefLd;
      sA[e] = (e - i * kCoefLd == i && i < M) ? 1.0 : 0.0;
      sB[e] = 0.0;
    }
    if (t >= 1 && t <= kTaylorDegree) inv[t] = 1.0 / t;
    __syncthreads();
    nrm = wmax[0];
    for (int w = 1; w < kCoefThreads / 64; ++w) nrm = fmax(nrm, wmax[w]);
    int nsq = 0;  // ceil(log2(nrm / 0.5)) exactly, as on the host
    if (nrm > 0.5) {
      int ex = 0;
      const double f = frexp(nrm / 0.5, &ex);
      nsq = f == 0.5 ? ex - 1 : ex;
    }
    const double scale = ldexp(1.0, -nsq);
    if (t < M) {
      dg[t] = (t == 0 ? 0.0 : hc + hg * a.xi[t - 1]) * scale;
      sd[t] = (t == 0 ? 0.0 : (t == 1 ? 1.0 : hg)) * scale;
    }
    __syncthreads();
    double* E = sA;
    double* T = sB;
    // Taylor polynomial by Horner's rule, E <- I + X E / k, on the lower
    // triangle
    for (int k = kTaylorDegree; k >= 1; --k) {
      const double ik = inv[k];
#pragma unroll
      for (int ra = 0; ra < RB; ++ra) {
        const int i = ty + 16 * ra;
        if (i >= M) break;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const int j = tx + 16 * rb;
          if (j > i) break;
          double v = i == 0 ? dg[0] * E[0] * ik
                            : (dg[i] * E[i * kCoefLd + j] + sd[i] * E[(i - 1) * kCoefLd + j]) * ik;
          if (i == j) v += 1.0;
          T[i * kCoefLd + j] = v;
        }
      }
      __syncthreads();
      double* x = E;
      E = T;
      T = x;
    }
    // Squaring; the last square forms the first column only.  A thread's
    // sums run over every k < 16 RB in order: the products outside
    // j <= k <= i hold a zero of the upper triangle or of the rows and
    // columns past M and add nothing, so each sum equals the host's over
    // k = j .. i.
    for (int q = 0; q < nsq; ++q) {
      if (q + 1 == nsq) {
        if (t < M) {
          double acc = 0.0;
          for (int k = 0; k <= t; ++k) acc += E[t * kCoefLd + k] * E[k * kCoefLd];
          T[t * kCoefLd] = acc;
        }
      } else {
        double acc[RB][RB];
#pragma unroll
        for (int ra = 0; ra < RB; ++ra)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) acc[ra][rb] = 0.0;
#pragma unroll
        for (int k = 0; k < 16 * RB; ++k) {
          double ar[RB], br[RB];
#pragma unroll
          for (int ra = 0; ra < RB; ++ra) ar[ra] = E[(ty + 16 * ra) * kCoefLd + k];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) br[rb] = E[k * kCoefLd + tx + 16 * rb];
#pragma unroll
          for (int ra = 0; ra < RB; ++ra)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[ra][rb] += ar[ra] * br[rb];
        }
#pragma unroll
        for (int ra = 0; ra < RB; ++ra) {
          const int i = ty + 16 * ra;
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            const int j = tx + 16 * rb;
            if (i < M && j <= i) T[i * kCoefLd + j] = acc[ra][rb];
          }
        }
      }
      __syncthreads();
      double* x = E;
      E = T;
      T = x;
    }
    if (t < n) {
      const double v = E[(t + 1) * kCoefLd];
      dd[t] = v;
      a.cache->d[t] = v;
    }
    if (t == 0) {
      a.cache->hc = hc;
      a.cache->hg = hg;
      a.cache->n = n;
    }
  }
  __syncthreads();
  const double cc = bc[0], gg = bc[1], delta = bc[2], scal = bc[5];
  if (t < n) {
    const double d = dd[t];
    a.cf->dk[t] = d;
    a.cf->shift[t] = t > 0 ? cc / gg + a.xi[t - 1] : 0.0;
    a.cf->estf[t] = fabs(delta * d) / (a.rootN * scal);
  }
  if (t == 0) {
    a.cf->inv_g = 1.0 / gg;
    a.cf->thresh = a.thresh;
  }
}

}  // namespace

namespace {

// Rows per chunk of the 2D marching pass: longer chunks once the workgroups (and so
// the partials that every workgroup adds up) would pass kGateMax.
int terms_rows(const Dims& d) {
  const long long strips = march_strips(d.nx, kTermsPerPass2);
  int rows = kTermRows;
  while (strips * ((d.ny + 4ll * rows - 1) / (4ll * rows)) > kGateMax && rows < d.ny &&
         static_cast<long long>(d.nx) * (2 * rows + 2 * kTermsPerPass2) < (1ll << 27))
    rows *= 2;
  return rows;
}

// Rows of the 3D pass's tile, and planes per chunk: about kZmarchBlocks workgroups.
int zmarch_rows(const Dims& d) { return d.ny <= kSliceRows ? kSliceRows : kZmarchRows; }
int zmarch_planes(const Dims& d) {
  const int rows = zmarch_rows(d);
  const long long xy = static_cast<long long>((d.nx + kBX - 1) / kBX) * ((d.ny + rows - 1) / rows);
  const long long chunks =
      std::max(1ll, std::min<long long>(d.nz, (rows == kSliceRows ? kSliceBlocks : kZmarchBlocks) / xy));
  return static_cast<int>((d.nz + chunks - 1) / chunks);
}

// Boxes of 16 R rows, and the rule: rows per thread of the box pass, 0 where a grid
// has more boxes than CUs even with two.
int box_blocks(const Dims& d, int R) {
  const int H = 16 * R, inner = H - 2 * kTermsPerPass2;
  const long long rows = d.ny <= H ? 1 : 1 + (d.ny - H + inner - 1) / inner;
  return static_cast<int>(std::min<long long>(march_strips(d.nx, kTermsPerPass2) * rows, 1 << 30));
}
int box_cells(const Dims& d) {
  if (d.dim != 2) return 0;
  return box_blocks(d, 1) <= kBoxOne ? 1 : box_blocks(d, 2) <= kBoxTwo ? 2 : 0;
}

// Boxes of the 3D box pass; 0 where a grid has too many for it.
int cube_blocks(const Dims& d) {
  if (d.dim != 3) return 0;
  const long long n = static_cast<long long>(cube_tiles(d.nx, kCubeX)) * cube_tiles(d.ny, kCubeY) *
                      ((d.nz + kCubeZ - 1) / kCubeZ);
  return n <= kCubeMax ? static_cast<int>(n) : 0;
}

// Every second 3D pass marches from the top down when a pass moves more than the
// Infinity Cache holds (ten words a cell): it then begins on what the pass before
// touched last.  256^3, FP64 phi1 action of 36 terms 6.16 -> 5.73 ms, 256 x 256 x 128
// 3.24 -> 2.94; on 150 x 131 x 97 in FP32 (76 MB) no difference.
bool zmarch_turns(const Dims& d, size_t word) { return 10ll * d.N * static_cast<long long>(word) > (256ll << 20); }

int terms_blocks(const Dims& d) {
  if (d.dim == 2) {
    if (const int R = box_cells(d)) return box_blocks(d, R);
    const long long rows = terms_rows(d);
    return static_cast<int>(march_strips(d.nx, kTermsPerPass2) * ((d.ny + 4 * rows - 1) / (4 * rows)));
  }
  if (const int n = cube_blocks(d)) return n;
  const int zc = zmarch_planes(d), rows = zmarch_rows(d);
  return static_cast<int>(((d.nx + kBX - 1) / kBX) * ((d.ny + rows - 1) / rows) *
                          ((d.nz + zc - 1) / zc));
}

int init_blocks(const Dims& d) { return std::min(kInitBlocks, (d.N + kThreads - 1) / kThreads); }

}  // namespace

int leja_terms_per_launch(const Dims& d, int k, int K) {
  if (d.dim == 2) {
    // the 2D pass addresses a chunk's rows with 31-bit byte offsets
    return k + kTermsPerPass2 - 1 <= K && d.nx <= (1 << 22) ? kTermsPerPass2 : 1;
  }
  return k + 1 <= K ? 2 : 1;
}

int leja_slots(const Dims& d) { return std::max(cell_bands(d), std::max(terms_blocks(d), kInitBlocks)); }

hipError_t launch_leja_reset(LejaState* st, int nslots, int nterms, hipStream_t s) {
  hipLaunchKernelGGL(k_leja_reset, dim3(nslots < 64 ? nslots : 64), dim3(256), 0, s, st, nslots, nterms);
  return hipGetLastError();
}

template <class V>
hipError_t launch_leja_init(const Dims& d, const LejaCoef* cf, const double* v, V* q0, V* p, double* part,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_leja_init<V>, dim3(init_blocks(d)), dim3(kThreads), 0, s, d.N, cf, v, q0, p, part);
  return hipGetLastError();
}

template <class V>
hipError_t launch_leja_term(const Dims& d, const LejaCoef* cf, const V* coef, const V* qin, V* qout, V* p,
                            const LejaState* st, double* part, int k, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const int nb = leja_slots(d);
  if (d.dim == 3)
    launch_timed(k_leja_term<3, V>, cell_grid(d), cell_block(), 0, s, e0, e1, d, cf, coef, qin, qout, p, st, part,
                 nb, k);
  else
    launch_timed(k_leja_term<2, V>, cell_grid(d), cell_block(), 0, s, e0, e1, d, cf, coef, qin, qout, p, st, part,
                 nb, k);
  return hipGetLastError();
}

namespace {

// src (or null): the first pass of a substep, on a grid of a box pass.
template <class V>
hipError_t launch_terms(const Dims& d, const LejaCoef* cf, const V* coef, const double* src, const V* qin, V* qout, V* p,
                        LejaState* st, double* part, const LejaGate& g, int k, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1) {
  const int nb = leja_slots(d);
  const dim3 grid(terms_blocks(d));
  if (const int R = box_cells(d)) {
    const auto kernel = src ? (R == 1 ? k_leja_box<1, true, V> : k_leja_box<2, true, V>)
                            : (R == 1 ? k_leja_box<1, false, V> : k_leja_box<2, false, V>);
    launch_timed(kernel, grid, dim3(1024), 0, s, e0, e1, d, cf, coef, src, qin, qout, p, st, part, g, nb, k);
  } else if (cube_blocks(d)) {
    launch_timed(src ? k_leja_cube<kCubeZ, true, V> : k_leja_cube<kCubeZ, false, V>, grid, dim3(kCubeX * kCubeY), 0, s,
                 e0, e1, d, cf, coef, src, qin, qout, p, st, part, g, nb, k);
  } else if (d.dim == 2) {
    launch_timed(k_leja_terms<kTermsPerPass2, V>, grid, dim3(kThreads), 0, s, e0, e1, d, cf, coef, qin, qout, p, st,
                 part, g, nb, terms_rows(d), k);
  } else {
    const bool flip = zmarch_turns(d, sizeof(V)) && (k >> 1) & 1, slice = zmarch_rows(d) == kSliceRows;
    const auto kernel = slice ? (flip ? k_leja_zmarch<kSliceRows, kSliceStrip, kSliceThreads, true, V>
                                      : k_leja_zmarch<kSliceRows, kSliceStrip, kSliceThreads, false, V>)
                              : (flip ? k_leja_zmarch<kZmarchRows, kZmarchStrip, kZmarchThreads, true, V>
                                      : k_leja_zmarch<kZmarchRows, kZmarchStrip, kZmarchThreads, false, V>);
    launch_timed(kernel, grid, dim3(slice ? kSliceThreads : kZmarchThreads), 0, s, e0, e1, d, cf, coef, qin, qout, p, st,
                 part, g, nb, zmarch_planes(d), k);
  }
  return hipGetLastError();
}

// Gate of terms k1 .. k2 whose partials the launches of leja_substep left; a
// fold first when they are too many to be added by every workgroup.
hipError_t make_gate(const Dims& d, LejaState* st, double* part, int k1, int k2, const int* cnt, LejaGate* g,
                     hipStream_t s) {
  const int nb = leja_slots(d);
  g->k1 = k1;
  g->k2 = k2;
  int most = 0;
  for (int i = 0; i <= k2 - k1; ++i) {
    const int k = k1 + i;
    g->src[i] = part + static_cast<size_t>(k % kLejaRing) * nb;
    g->cnt[i] = cnt[k % kLejaRing];
    most = std::max(most, g->cnt[i]);
  }
  if (most <= kGateMax) return hipSuccess;
  double* dst = part + static_cast<size_t>(kLejaRing) * nb;
  hipLaunchKernelGGL(k_leja_fold, dim3(kFoldParts, k2 - k1 + 1), dim3(64), 0, s, st, *g, dst);
  for (int i = 0; i <= k2 - k1; ++i) {
    g->src[i] = dst + i * kFoldParts;
    g->cnt[i] = kFoldParts;
  }
  return hipGetLastError();
}

}  // namespace

template <class V>
hipError_t leja_substep(const Dims& d, const LejaCoef* cf, const LejaVecs<V>& B, const double* src, LejaState* st,
                        double* part, int K, double* out, double delta, int first, const double* zt, hipStream_t s,
                        hipEvent_t* ev, int prof) {
  const int nterms = terms_blocks(d), nterm = cell_bands(d);
  int cnt[kLejaRing] = {};  // partials of the terms in the ring
  // the box passes make the start vectors themselves
  const bool fused = (box_cells(d) || cube_blocks(d)) && leja_terms_per_launch(d, 1, K) > 1;
  cnt[0] = fused ? nterms : init_blocks(d);
  hipError_t e = fused ? hipSuccess : launch_leja_init<V>(d, cf, src, B.qa, B.p, part, s);
  if (e != hipSuccess) return e;
  V* cur = B.qa;
  V* oth = B.qb;
  int prev = -1;  // last term already tested
  for (int k = 1, launch = 0; k <= K; ++launch) {
    const int nt = leja_terms_per_launch(d, k, K);
    const bool timed = ev && launch % prof == 0;
    hipEvent_t e0 = timed ? ev[2 * (k - 1)] : nullptr, e1 = timed ? ev[2 * (k - 1) + 1] : nullptr;
    LejaGate g{};
    g.k1 = 0;
    g.k2 = -1;
    if (k > 1 && (k - 1) % kCheckEvery == 0) {
      e = make_gate(d, st, part, prev + 1, k - 1, cnt, &g, s);
      if (e != hipSuccess) return e;
      prev = k - 1;
    }
    if (nt > 1) {
      e = launch_terms<V>(d, cf, B.coef, fused && k == 1 ? src : nullptr, cur, oth, B.p, st, part, g, k, s, e0, e1);
    } else {
      // the one-term pass only reads the flag: the test is made before it
      if (g.k2 >= g.k1) {
        hipLaunchKernelGGL(k_leja_check, dim3(1), dim3(kThreads), 0, s, cf, st, g);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      e = launch_leja_term<V>(d, cf, B.coef, cur, oth, B.p, st, part, k, s, e0, e1);
    }
    if (e != hipSuccess) return e;
    for (int t = 0; t < nt; ++t) cnt[(k + t) % kLejaRing] = nt > 1 ? nterms : nterm;
    std::swap(cur, oth);
    k += nt;
  }
  LejaGate g{};
  e = make_gate(d, st, part, prev + 1, K, cnt, &g, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_substep_update<V>, dim3((d.N + kThreads - 1) / kThreads + 1), dim3(kThreads), 0, s, d.N, out,
                     B.p, delta, first, zt, cf, st, g);
  return hipGetLastError();
}

template <class V>
hipError_t launch_substep_update(const Dims& d, double* u, const V* p, double delta, int first, hipStream_t s,
                                 LejaState* st) {
  LejaGate g{};
  g.k2 = -1;
  hipLaunchKernelGGL(k_substep_update<V>, dim3((d.N + kThreads - 1) / kThreads + 1), dim3(kThreads), 0, s, d.N, u, p,
                     delta, first, nullptr, nullptr, st, g);
  return hipGetLastError();
}

hipError_t launch_leja_coef(const LejaCoefArgs& a, hipStream_t s) {
  if (a.n < 1 || a.n > kCoefMaxN || a.s < 1 || a.s > a.smax) return hipErrorInvalidValue;
  if (a.n + 1 <= 16)  // 16-row blocks of the order n + 1 matrix
    hipLaunchKernelGGL(k_leja_coef<1>, dim3(1), dim3(kCoefThreads), 0, s, a);
  else
    hipLaunchKernelGGL(k_leja_coef<2>, dim3(1), dim3(kCoefThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_cast_f32(const double* a, float* b, long long n, hipStream_t s) {
  long long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_cast_f32, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a, b, n);
  return hipGetLastError();
}

template hipError_t launch_leja_init<double>(const Dims&, const LejaCoef*, const double*, double*, double*,
                                             double*, hipStream_t);
template hipError_t launch_leja_init<float>(const Dims&, const LejaCoef*, const double*, float*, float*, double*,
                                            hipStream_t);
template hipError_t launch_leja_term<double>(const Dims&, const LejaCoef*, const double*, const double*, double*,
                                             double*, const LejaState*, double*, int, hipStream_t, hipEvent_t,
                                             hipEvent_t);
template hipError_t launch_leja_term<float>(const Dims&, const LejaCoef*, const float*, const float*, float*, float*,
                                            const LejaState*, double*, int, hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t launch_substep_update<double>(const Dims&, double*, const double*, double, int, hipStream_t,
                                                  LejaState*);
template hipError_t leja_substep<double>(const Dims&, const LejaCoef*, const LejaVecs<double>&, const double*,
                                         LejaState*, double*, int, double*, double, int, const double*, hipStream_t,
                                         hipEvent_t*, int);
template hipError_t leja_substep<float>(const Dims&, const LejaCoef*, const LejaVecs<float>&, const double*,
                                        LejaState*, double*, int, double*, double, int, const double*, hipStream_t,
                                        hipEvent_t*, int);

}  // namespace erem
