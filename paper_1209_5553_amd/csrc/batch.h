// Batched EREM over many independent linear problems (batch.hip): shared
// structures and launchers.
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace erem {

// Tile shapes of the work pass: a tile is a strip of columns (march.h) by
// kBatchTileRows[shape] rows, advanced by kBatchPassTerms[shape] Newton terms
// per pass by one wavefront.  Eight terms halve the bytes per term; short
// tiles re-read more rows (2 NT per tile) but shorten a pass whose problems do
// not fill the chip.  Two FP64 steps, us, for the shapes 0 .. 7:
//   one of 256 x 256          420   389   510   718  1117   471   381   343
//   20 of 40 .. 256 a side    954   994  1183  1671  2688  1070   857   867
//   64 of 256 x 256          2020  2395  1812  1772  1956  1315  1471  1943
//   one of 4096 x 4096       3709  4168  3707  3858  4161  2645  2990  3958
// Of 14 such sets in both precisions each ran fastest with eight terms (7: few
// small problems, then 6, 5: the chip filled).  Four terms stay for the callers
// that name such a shape, and shape 0 is what a batch has before one is chosen:
// its applied degrees are multiples of four, as a single grid's.
constexpr int kNumTileShapes = 8;
constexpr int kBatchTileRows[kNumTileShapes] = {16, 8, 32, 64, 128, 32, 16, 8};
constexpr int kBatchPassTerms[kNumTileShapes] = {4, 4, 4, 4, 4, 8, 8, 8};
constexpr int kBatchPartStride = 8;  // partials per tile (one per term of a pass)
// Most tiles whose partials every wavefront of their problem adds up by itself,
// and the slots that a larger problem's are folded into between two passes.  One
// problem, every wavefront all of them / folded: 512 x 512 (288 tiles of 16 rows)
// 397 / 421 us a run of two steps, 768 x 768 (384 of 32 rows) 408 / 405, 640 x 640
// (480 of 16 rows) 473 / 445.
constexpr int kBatchGate = 384;
constexpr int kBatchFoldParts = 64;

// Static description of one problem of the batch.
struct BProb {
  int nx, ny;
  int s;          // substeps per step
  int coef_off;   // first divided difference / shift of this problem
  long long off;  // first cell in the packed vectors
  double inv_g;   // 1 / gamma
  double delta;   // substep length h / s
  double rootN;   // sqrt(nx ny)
  int tile0;      // first tile of the problem in the tile list
  int ntiles;     // its tiles
};

// Tile list entry: the problem, the strip of columns and the first row.
struct BTile {
  int pid, strip, y0;
  int done;       // set by the tile once its problem is done: it returns at entry
  int tile0;      // the problem's first tile
  int src, nsrc;  // partial slots that add up to the problem's: its tiles', or their fold
  int pad;
};

// One wavefront of the fold: the partials of n tiles of problem pid into a slot.
struct BFold {
  int pid, tile0, n, slot;
};

// Phases of a problem; every launch picks each unfinished problem's next phase
// from what the launch before left, and advances it by that phase.
enum BPhase : int {
  kPhInit = 0,    // start of a substep: q_0, p = d_0 q_0 (and the end of the previous substep or step)
  kPhTerms = 1,   // Newton terms k .. k + nt - 1
  kPhFinish = 2,  // the last step's T update
  kPhDone = 3,
};

// Kinds of start pass.
enum BInit : int {
  kInitFirst = 0,  // first step: T^0 as given
  kInitSub = 1,    // substep j >= 1: u += delta p of substep j - 1
  kInitStep = 2,   // next step: T += u + delta p of the last substep
};

// Dynamic state of one problem (two copies, written by turns).
struct BState {
  int phase, kind;
  int step;   // steps completed
  int sub;    // current substep
  int k;      // first term of the next pass
  int terms;  // Newton terms applied
  int flags;  // 1: no convergence within m_max, 2: non-finite norm
  int tpar;   // buffer holding T^n: 0 the caller's array, 1 the internal copy
  int upar;   // buffer holding u (sum of the finished substeps' increments)
  int ppar;   // buffer holding p (the current substep's Newton sum)
  int phases; // work passes taken; -1: before the first
  int pad;
  double scal;     // error scale tol_a + tol_r max|T^n|
  double prev[4];  // the scaled error estimates of the four terms before term k
};

struct BatchArgs {
  const BProb* prob;
  BTile* tile;
  BState* state;         // two copies of nprob states
  int* ndone;            // problems done
  const double* coef64;  // 5-point stencil, SoA with stride ntot (FP64)
  const void* coef;      // stencil of the Newton terms (FP64 or FP32)
  const double* g;       // G(T) = J T + g
  double* T0;            // the caller's temperatures
  double* T1;            // internal temperature buffer
  double *u0, *u1;       // substep increment sums (ping-pong)
  double* v;             // G(T^n) of the current step
  void *q0, *q1;         // Newton vectors (FP64 or FP32)
  void *p0, *p1;         // Newton sums (ping-pong over substeps)
  const double* dk;      // divided differences, (m_max + 1) per problem
  const double* shift;   // c/gamma + xi_{k-1}, (m_max + 1) per problem
  double* part;          // kBatchPartStride partials per slot, two copies of part_cap slots (tiles, then folds)
  long long part_cap;
  const BFold* fold;
  int nfold;
  long long ntot;
  int nprob, ntiles, nsteps, m_max;
  int nt, rows;          // Newton terms per pass and rows per tile of the tile shape
  int pass;              // parity of the pass (the order in which the tiles are taken)
  double tol_a, tol_r, thresh;
};

hipError_t batch_pack(int nx, int ny, const double* coef, const double* F, const double* T0,
                      double* bcoef, double* g, long long ntot, long long off, hipStream_t s);
hipError_t batch_reset(const BatchArgs& a, hipStream_t s);
// One phase of every problem: pass number `pass` over all tiles, then the fold of
// its partials where a problem needs one.  e0 / e1 (optional) time the pass.
hipError_t batch_phase(BatchArgs a, long long pass, int fp32, hipStream_t s, hipEvent_t e0 = nullptr,
                       hipEvent_t e1 = nullptr);

}  // namespace erem
