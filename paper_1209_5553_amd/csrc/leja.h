// Device Newton-Leja evaluation: launchers (leja.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace erem {

constexpr int kLejaRing = 16;       // terms whose block partials are kept
constexpr int kCheckEvery = 4;      // terms between stop tests
constexpr int kTermsPerPass2 = 4;   // terms per pass on 2D grids: one stop-test group
// Most boxes of the 2D box pass with one and with two rows per thread: one box a
// CU.  An FP64 phi1 action of 32 terms, one row / two rows / rows marched: 256 x 256
// (155 / 55 boxes) 107 / 117 / 144 us; 512 x 512 (630 / 210) 185 / 129 / 154; 640 x
// 640 (960 / 324) 226 / 175 / 161.
constexpr int kBoxOne = 256, kBoxTwo = 256;
// Rows per wavefront of the 2D marching pass, more once the workgroups would pass
// kGateMax (512 x 512: four rows 1.16 times the time, sixteen 1.09 times).
constexpr int kTermRows = 8;
// Box of the 3D box pass, planes of its output, and most boxes: one a CU.  An FP64
// phi1 action of 36 terms, boxes / planes marched: 50^3 (200 boxes) 189 / 250 us,
// 64^3 (480) 268 / 257, 80^3 (1120) 455 / 381.  On 50^3 one plane a box took 209 us,
// three 200; boxes of 32 x 8 columns 215, of 64 x 16 246.
constexpr int kCubeX = 32, kCubeY = 16, kCubeZ = 2, kCubeMax = 256;
constexpr int kZmarchRows = 16;     // rows of the 3D pass's tile (64 wide)
constexpr int kZmarchStrip = 2;     // cells per thread of its box
constexpr int kZmarchThreads = 640;
// Workgroups aimed at by the 3D pass: one per CU.  A chunk reads two planes of
// the stencil and four of q more than it advances, so more, shorter chunks cost
// what they hide (128^3: 3.50 ms a step against 4.33 with 512 workgroups; 256^3
// 38.2 against 40.7 ms).
constexpr int kZmarchBlocks = 256;
// Its tile on grids of at most four rows (a vertical slice), where sixteen would be
// padding: a cell per thread, two workgroups a CU.  One FP64 step, tile of 16 / 4
// rows: 512 x 1 x 512 2.24 / 1.18 ms, 512 x 4 x 512 2.61 / 1.53, 4 x 4 x 4000 89 / 47
// (one term per pass on 64 x 4 tiles took 1.25, 2.43 and 77); two cells a thread
// 1.30, 1.62 and 53; with 768 workgroups 1.44, 1.84 and 57.
constexpr int kSliceRows = 4, kSliceStrip = 1, kSliceThreads = 448, kSliceBlocks = 512;
constexpr int kInitBlocks = 2048;    // most workgroups of the start pass
constexpr int kGateTerms = 5;       // most terms of one stop test (the first: terms 0 .. 4)
constexpr int kGateMax = 2048;      // most partials per term that every workgroup adds up by itself
constexpr int kFoldParts = 512;     // partials per term after a fold

// Stop test of terms k1 .. k2: the partials of term k1 + i are src[i][0 .. cnt[i]).
struct LejaGate {
  const double* src[kGateTerms];
  int cnt[kGateTerms];
  int k1, k2;
};

// Device vectors of the Newton passes in one precision: the stencil of J, the
// two q buffers and the accumulated polynomial p.
template <class V>
struct LejaVecs {
  const V* coef;
  V *qa, *qb, *p;
};

// Newton terms computed by the launch that starts at term k of at most K.
int leja_terms_per_launch(const Dims& d, int k, int K);
// Partial slots of one term, and the words of a partial array.
int leja_slots(const Dims& d);
inline size_t leja_part_words(const Dims& d) {
  return static_cast<size_t>(kLejaRing) * leja_slots(d) + kGateTerms * kFoldParts;
}

hipError_t launch_leja_reset(LejaState* st, int nslots, int nterms, hipStream_t s);
template <class V>
hipError_t launch_leja_init(const Dims& d, const LejaCoef* cf, const double* v, V* q0, V* p,
                            double* part, hipStream_t s);
// One term, without a stop test (the adjoint's replay; the terms left over when
// a budget is no multiple of a pass).
template <class V>
hipError_t launch_leja_term(const Dims& d, const LejaCoef* cf, const V* coef, const V* qin, V* qout,
                            V* p, const LejaState* st, double* part, int k, hipStream_t s,
                            hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// One substep of at most K terms from src, with its stop tests into st:
// out = (first ? 0 : out) + delta p (+ zt when zt is not null).  part:
// leja_part_words(d).  ev, when not null: 2 K events, every prof-th launch
// timed with the pair of its first term.
template <class V>
hipError_t leja_substep(const Dims& d, const LejaCoef* cf, const LejaVecs<V>& B, const double* src, LejaState* st,
                        double* part, int K, double* out, double delta, int first, const double* zt, hipStream_t s,
                        hipEvent_t* ev, int prof);
// A whole evaluation of s substeps on a small grid in one launch (leja_small.hip): out = sum of the substeps' increments, source v + t_j g
// (g null: v), zt (or null) added per substep; the stop states st[0 .. s) as
// leja_substep leaves them.  coef64: the stencil in FP64; coef: in the passes'
// precision.
constexpr int kSmallCells = 4096, kSmallCells3 = 2048;  // 2D, 3D
bool leja_small_fits(const Dims& d);
template <class V>
hipError_t leja_small(const Dims& d, const LejaCoef* cf, const double* coef64, const V* coef, const double* v,
                      const double* g, const double* zt, double* out, LejaState* st, double delta, int s, int K,
                      hipStream_t q, hipEvent_t e0, hipEvent_t e1);
// u = (first ? 0 : u) + delta p
template <class V>
hipError_t launch_substep_update(const Dims& d, double* u, const V* p, double delta, int first,
                                 hipStream_t s, LejaState* st);
hipError_t launch_cast_f32(const double* a, float* b, long long n, hipStream_t s);

// Coefficients of one Newton-Leja phi1 evaluation formed on the device from
// the assembly's reduction slots, so that the evaluation can be enqueued
// before the host has read the interval.  The kernel folds the slots into
// the Gershgorin interval [alpha, beta] and the largest |T|, forms
// scal = tol_a + tol_r max|T|, and, when the interval is finite and not
// degenerate and its substep count ceil(h (beta - alpha) / rho) (at least 1,
// at most smax) equals the count s the evaluation was enqueued with, fills
// cf for substeps of delta = h / s: the divided differences of
// phi1(delta (c + gamma xi)) (Sec. 4.2; the augmented bidiagonal
// exponential by Taylor scaling and squaring, as on the host), the shifts
// c / gamma + xi_{k-1} and the stop-test factors |delta d_k| / (sqrt(N) scal).
// Otherwise it marks the s stop states as stopped, so that the evaluation's
// term launches return at entry, and the host, which reads the same slots
// afterwards, evaluates again with the interval it has read.
struct LejaCoefArgs {
  const AsmReduce* red;
  int n;            // coefficients d_0 .. d_{n-1}, 1 <= n <= kCoefMaxN
  int s, smax;      // substeps enqueued; cap of the substep count
  double h, rho;    // step; widest substep interval (rho <= 0: one substep)
  double tol_a, tol_r, thresh, rootN;
  const double* xi;  // device copy of the Leja points (n values)
  DdCache* cache;
  LejaCoef* cf;
  LejaState* st;
};
constexpr int kCoefThreads = 256;
// Most coefficients the kernel forms: the augmented matrix (order n + 1 <=
// 32) and its square stay in LDS.  Past that its dependent phases (20 Taylor
// steps and up to 8 squarings) take longer than the host round trip they
// replace.
constexpr int kCoefMaxN = 31;
hipError_t launch_leja_coef(const LejaCoefArgs& a, hipStream_t s);

}  // namespace erem
