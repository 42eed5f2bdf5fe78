// Device piece of the adjoint of one NDF_p step (eq. (ode_disc) transposed): the
// update of one coefficient's history cotangents.
#pragma once

#include "nse_internal.h"

namespace nse {

// The history update of StepAdjointArgs at degree l = m + k (k <= N - m) of
// member b from the predictor cotangent ab and the loaded rows hin[j] (j < depth),
// stored to a.hout (in place when a.hout == a.hin).
__device__ inline void step_adjoint_store(const GroupView& g, const StepAdjointArgs& a, int b,
                                          int m, int k, double2 ab, const double2* hin) {
  const int N = g.N, l = m + k;
  const int64_t S = a.state_count, slot = g.off[b] + coeff_offset(N, m) + k;
  const double lam = (double)l * (l + 1);
  const double q = 1.0 / fma(a.h * g.nu[b], lam, a.c[0]);
  double2 r = make_double2(hin[0].x * q, hin[0].y * q);  // r = hin[0] / (c_0 + h nu lambda)
  if (l == 0) r = make_double2(0.0, 0.0);
  if (m == 0) r.y = 0.0;
  // row j = hin[j+1] - c_{j+1} r + pi_j alpha_bar (terms past depth, ncoef, npi absent)
#pragma unroll
  for (int j = 0; j < kMaxStepCoef; ++j) {
    double2 v = make_double2(0.0, 0.0);
    if (j + 1 < kMaxStepCoef && j + 1 < a.depth) v = hin[j + 1 < kMaxStepCoef ? j + 1 : j];
    if (j + 1 < a.ncoef) {
      v.x = fma(-a.c[j + 1 < kMaxStepCoef ? j + 1 : j], r.x, v.x);
      v.y = fma(-a.c[j + 1 < kMaxStepCoef ? j + 1 : j], r.y, v.y);
    }
    if (j < kMaxSources && j < a.npi) {
      v.x = fma(a.pi[j < kMaxSources ? j : 0], ab.x, v.x);
      v.y = fma(a.pi[j < kMaxSources ? j : 0], ab.y, v.y);
    }
    if (j < a.depth) a.hout[(int64_t)j * S + slot] = v;
  }
}

}  // namespace nse
