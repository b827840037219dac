// Device Arnoldi process for the Krylov evaluation of phi1 (krylov.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace erem {

constexpr int kMaxKrylov = 64;
constexpr int kKryDirect = 1024;  // most workgroups whose partials every workgroup adds up by itself

// Coefficients of the basis vectors v_0 .. v_{nv-1} (in V), and of the last one
// while it is still unnormalised in w (clast: with the norm's reciprocal).
struct KryCoef {
  double c[kMaxKrylov];
  double clast;
  int nv, last;
};

// Words of the partial array.
size_t kry_part_words(const Dims& d, int m);
// Start vector v + J u (u null: v) into w[0, N) with the partials of its norm.
hipError_t krylov_start(const Dims& d, const double* coef, const double* v, const double* u, double* w, double* part,
                        int m, hipStream_t s);
// Arnoldi (CGS2) on the start vector that krylov_start left: beta = ||w||, then
// the columns j = 0..m-1; v_m stays unnormalised in w + (m & 1) N.  w holds 2 N
// doubles, V m N, H (row-major) (m + 1) m, g m + 1, part kry_part_words.  H and
// beta stay on the device.
hipError_t arnoldi_cgs2(const Dims& d, const double* coef, double* V, double* w, double* H, double* beta,
                        double* g, double* part, int m, hipStream_t s);
hipError_t krylov_combine(const Dims& d, const double* V, const double* w, const KryCoef& c, double* u, int first,
                          hipStream_t s);

}  // namespace erem
