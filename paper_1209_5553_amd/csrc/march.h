// Row-marching Newton-Leja pass on 2D grids: one wavefront advances a strip of
// 64 columns by NT terms in one sweep over its rows.
//
// Lane l holds column xs + l.  When row r of q_{k-1} arrives, term 1 is formed
// on row r - 1, term 2 on row r - 2, ..., term NT on row r - NT: every term
// needs the rows above, at and below it of the term before, and all of them
// are in registers of the same lane; the west and east neighbours are the
// next lanes', moved by DPP wavefront shifts.  So a pass needs neither LDS nor
// barriers, reads the stencil, q and p once per strip and writes p and the
// last q once.  At a strip's inner edge one column per term goes wrong (the
// next lane is missing), so a strip overlaps its neighbours by 2 NT columns;
// at the grid's own edge nothing is missing (the stencil is zero there).  The
// same holds for the NT rows above and below a chunk of rows.
//
// What bounds it: the strip's loads.  Rows are fetched PD ahead into a ring of
// NT + PD rows of registers (the row loop is unrolled by the ring, so every
// ring index is a constant), through buffer descriptors whose range check
// gives zero outside the chunk's rows and the grid's columns, so no load is
// conditional.  The dependent chain of a row is short: the part of a term that
// does not use the newest row of the term before is formed first.
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace erem {

constexpr int kMarchLanes = 64;

// Columns of strip j when NT terms are advanced: lanes start at xs, the
// outputs are [x0, x1).
struct MarchStrip {
  int xs, x0, x1;
};
__host__ __device__ inline int march_strips(int nx, int nt) {
  const int inner = kMarchLanes - 2 * nt;
  return nx <= kMarchLanes ? 1 : 1 + (nx - kMarchLanes + inner - 1) / inner;
}
__host__ __device__ inline MarchStrip march_strip(int nx, int nt, int j) {
  const int inner = kMarchLanes - 2 * nt;
  MarchStrip s;
  s.xs = j * inner;
  s.x0 = j == 0 ? 0 : s.xs + nt;
  s.x1 = s.xs + kMarchLanes >= nx ? nx : s.xs + kMarchLanes - nt;
  return s;
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Largest byte offset a descriptor can reach; lanes without a column use it as
// their base, which the range check refuses (loads give 0, stores are dropped).
constexpr unsigned kMarchOut = 0x80000000u;

__device__ inline __amdgpu_buffer_rsrc_t march_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

__device__ inline void march_load(__amdgpu_buffer_rsrc_t r, unsigned off, double& v) {
  const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  v = __hiloint2double(static_cast<int>(w.y), static_cast<int>(w.x));
}
__device__ inline void march_load(__amdgpu_buffer_rsrc_t r, unsigned off, float& v) {
  v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ inline void march_store(__amdgpu_buffer_rsrc_t r, unsigned off, double v) {
  u32x2 w;
  w.x = static_cast<unsigned>(__double2loint(v));
  w.y = static_cast<unsigned>(__double2hiint(v));
  __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, 0);
}
__device__ inline void march_store(__amdgpu_buffer_rsrc_t r, unsigned off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, 0, 0);
}

// Lane l's value of lane l - 1 (west) or l + 1 (east); 0 past the ends.
__device__ inline int dpp_west(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ inline int dpp_east(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ inline float west(float v) { return __int_as_float(dpp_west(__float_as_int(v))); }
__device__ inline float east(float v) { return __int_as_float(dpp_east(__float_as_int(v))); }
__device__ inline double west(double v) { return dpp<0x138>(v); }
__device__ inline double east(double v) { return dpp<0x130>(v); }

// A value every lane holds alike, in scalar registers.
__device__ inline double march_uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ inline float march_uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ inline int march_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// v where keep holds, else a value whose square is 0 (one select: only the
// high word goes, a denormal stays).
__device__ inline double march_mask(bool keep, double v) {
  return __hiloint2double(keep ? __double2hiint(v) : 0, __double2loint(v));
}

// One strip's chunk of rows [y0, y1) by NT terms.  coef (five arrays, stride
// cs), qin, qout and p start at the grid's first cell; shift[t], dk[t] belong
// to term t + 1 of the pass.  sum[t] gets the lane's share of sum q^2 over the
// outputs.  gate() runs once the first rows' loads are in flight; when it
// returns true the pass ends there, with nothing written.
template <int NT, int PD, class V, class Gate>
__device__ inline bool march_terms(const V* __restrict__ coef, long long cs, const V* __restrict__ qin,
                                   V* __restrict__ qout, V* __restrict__ p, int nx, int ny, MarchStrip st, int y0,
                                   int y1, V ig, const V (&shift)[NT], const V (&dk)[NT], double (&sum)[NT], Gate&& gate) {
  constexpr int U = (NT + PD + 1) / 2 * 2;  // ring rows (even: the terms keep their last two rows by row parity)
  static_assert(PD >= 2 && NT >= 2, "rows ahead, terms");
  const int lane = threadIdx.x & 63;
  const int r0 = max(0, y0 - NT), rend = min(ny, y1 + NT);  // rows loaded
  const int steps = y1 - 1 + NT - r0 + 1;
  const long long org = static_cast<long long>(nx) * r0;
  const unsigned rowb = static_cast<unsigned>(nx) * sizeof(V);
  const unsigned bytes = rowb * static_cast<unsigned>(rend - r0);
  const __amdgpu_buffer_rsrc_t rq = march_rsrc(qin + org, bytes);
  // p and the last q: the outputs' rows and columns only
  const long long oout = static_cast<long long>(nx) * y0;
  const unsigned bout = rowb * static_cast<unsigned>(y1 - y0);
  const __amdgpu_buffer_rsrc_t rp = march_rsrc(p + oout, bout), ro = march_rsrc(qout + oout, bout);
  __amdgpu_buffer_rsrc_t rc[5];
#pragma unroll
  for (int d = 0; d < 5; ++d) rc[d] = march_rsrc(coef + d * cs + org, bytes);
  const int gx = st.xs + lane;
  const unsigned col = static_cast<unsigned>(gx) * sizeof(V);
  const unsigned base = gx < nx ? col : kMarchOut;
  const bool out = gx >= st.x0 && gx < st.x1;
  const unsigned bo = (out ? col : kMarchOut) + static_cast<unsigned>(r0 - y0) * rowb;  // row r0 of the outputs
  unsigned offs = bo - static_cast<unsigned>(NT) * rowb;    // row r - NT
  unsigned offl = base + static_cast<unsigned>(PD) * rowb;  // row r + PD of q

  V c[U][5], pr[U], q0[U], Q[NT][2];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    q0[u] = V(0);
    pr[u] = V(0);
#pragma unroll
    for (int d = 0; d < 5; ++d) c[u][d] = V(0);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    Q[t][0] = Q[t][1] = V(0);
    sum[t] = 0.0;
  }
#pragma unroll
  for (int i = 0; i < PD; ++i) {
    const unsigned o = base + static_cast<unsigned>(i) * rowb;
    march_load(rq, o, q0[i]);
    if (i + 1 < PD) {
#pragma unroll
      for (int d = 0; d < 5; ++d) march_load(rc[d], o, c[i][d]);
      march_load(rp, bo + static_cast<unsigned>(i) * rowb, pr[i]);
    }
  }
  if (gate()) return false;
  int r = r0;
  const int rlast = r0 + steps - 1;
  for (;;) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      {
        // q of row r + PD, the stencil and p of row r - 1 + PD
        constexpr int kq = PD, kc = PD + U - 1;
        march_load(rq, offl, q0[(u + kq) % U]);
        const unsigned oc = offl - rowb;
#pragma unroll
        for (int d = 0; d < 5; ++d) march_load(rc[d], oc, c[(u + kc) % U][d]);
        march_load(rp, offs + static_cast<unsigned>(NT + PD - 1) * rowb, pr[(u + kc) % U]);
        // the loads stay PD rows ahead of their use (the scheduler would sink them)
        __builtin_amdgcn_sched_barrier(0);
      }
      V nv[NT];
#pragma unroll
      for (int t = 1; t <= NT; ++t) {
        const int s = (u + U - t) % U;  // ring slot of row r - t
        const V qc = t == 1 ? q0[(u + U - 1) % U] : Q[t - 2][(u + 1) & 1];
        const V qs = t == 1 ? q0[(u + U - 2) % U] : Q[t - 2][u & 1];
        const V qn = t == 1 ? q0[u] : nv[t - 2];
        V jq = c[s][1] * west(qc);
        jq = fma(c[s][0], qc, jq);
        jq = fma(c[s][2], east(qc), jq);
        jq = fma(c[s][3], qs, jq);
        jq = fma(c[s][4], qn, jq);
        const V qo = fma(jq, ig, -(shift[t - 1] * qc));
        nv[t - 1] = qo;
        pr[s] = fma(dk[t - 1], qo, pr[s]);
        const int row = r - t;
        const double qm = march_mask(row >= y0 && row < y1, static_cast<double>(qo));
        sum[t - 1] += qm * qm;
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) Q[t][u & 1] = nv[t];
      march_store(rp, offs, pr[(u + U - NT) % U]);  // rows before y0 are dropped by the range check
      march_store(ro, offs, nv[NT - 1]);
      if (r == rlast) goto done;
      ++r;
      offl += rowb;
      offs += rowb;
    }
  }
done:
#pragma unroll
  for (int t = 0; t < NT; ++t) sum[t] = out ? sum[t] : 0.0;
  return true;
}

}  // namespace erem
