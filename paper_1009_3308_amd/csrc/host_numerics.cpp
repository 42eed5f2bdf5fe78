// Host-side numerics: the Gauss-Legendre rule of the Gauss-rectangle
// quadrature (Section 3, eq. (quadrule)) and the radix plan of the
// longitude FFTs (Section 4.2, FFT in the azimuthal direction).
#include <algorithm>
#include <cmath>

#include "nse_internal.h"

namespace nse {

// Nodes mu_p of the n-point Gauss-Legendre rule in descending order (north
// pole first) and their weights. Newton's method on P_n in extended precision
// (x87 long double), P_n and P_n' from the three-term recurrence
// (j+1) P_{j+1} = (2j+1) x P_j - j P_{j-1}, started from the asymptotic
// guess cos(pi (k - 1/4) / (n + 1/2)); w = 2 / ((1 - x^2) P_n'(x)^2) with
// 1 - x^2 formed as (1 - x)(1 + x).
void gauss_legendre(int n, std::vector<double>& mu, std::vector<double>& w) {
  mu.assign(n, 0.0);
  w.assign(n, 0.0);
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int k = 1; k <= (n + 1) / 2; ++k) {
    long double x = std::cos(pi * (k - 0.25L) / (n + 0.5L));
    long double dp = 1.0L;
    for (int it = 0; it < 100; ++it) {
      long double p0 = 1.0L, p1 = x;
      for (int j = 1; j < n; ++j) {
        long double p2 = ((2 * j + 1) * x * p1 - j * p0) / (j + 1);
        p0 = p1;
        p1 = p2;
      }
      if (n == 1) p0 = 1.0L;
      const long double omx2 = (1.0L - x) * (1.0L + x);
      dp = n * (p0 - x * p1) / omx2;
      const long double dx = p1 / dp;
      x -= dx;
      if (std::fabs(dx) < 1e-19L) {
        // one more evaluation of P_n' at the converged node
        p0 = 1.0L;
        p1 = x;
        for (int j = 1; j < n; ++j) {
          long double p2 = ((2 * j + 1) * x * p1 - j * p0) / (j + 1);
          p0 = p1;
          p1 = p2;
        }
        if (n == 1) p0 = 1.0L;
        dp = n * (p0 - x * p1) / ((1.0L - x) * (1.0L + x));
        break;
      }
    }
    if (2 * k - 1 == n) x = 0.0L;  // the equator node of an odd rule
    const long double wk = 2.0L / ((1.0L - x) * (1.0L + x) * dp * dp);
    mu[k - 1] = (double)x;
    mu[n - k] = (double)(-x);
    w[k - 1] = (double)wk;
    w[n - k] = (double)wk;
  }
}

namespace {

constexpr int kRadices[] = {2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16};

// Passes that 16 lanes of 16 bytes take over the 64 LDS banks, averaged over the first
// lanes of each stage's butterflies and their first and last operands (1: no conflicts).
double lds_cost(const FftPlan& p) {
  double cost = 0;
  for (int s = 0; s < p.nstages; ++s) {
    const int J = p.J[s], R = p.radix[s], lanes = std::min(p.per[s], 32);
    int passes = 0, ideal = 0;
    for (int u0 = 0; u0 < lanes; u0 += 16)
      for (int r : {0, R - 1}) {
        int bank[16] = {0};
        for (int u = u0; u < std::min(lanes, u0 + 16); ++u) {
          const int i = u / J * J * R + u % J + r * J;
          ++bank[(i + p.pad0 * (i / p.J[0]) + p.pad1 * (i / p.J[1])) & 15];
        }
        passes += *std::max_element(bank, bank + 16);
        ++ideal;
      }
    cost += (double)passes / ideal;
  }
  return cost;
}

struct PlanSearch {
  int M, stages, cap;
  FftRadices f{};
  double best = 1e30;
  FftPlan plan{};

  void visit(int left, int n) {
    if (best < stages + 1e-9) return;  // no conflicts at all
    if (left == 1 && n == stages && f.r[n - 1] <= kMaxLastRadix) {
      for (int pad = 0; pad < 32; ++pad) {
        if (n == 2 && pad >= 16) break;
        const FftPlan p = make_plan(M, f, n, pad & 15, pad >> 4);
        const double cost = lds_cost(p);
        if (cost < best - 1e-9) {
          best = cost;
          plan = p;
        }
      }
    }
    if (n == stages || left == 1) return;
    for (int r : kRadices)
      if (r <= cap && left % r == 0) {
        f.r[n] = r;
        visit(left / r, n + 1);
      }
  }
};

}  // namespace

// True if M has no prime factor other than 2, 3 and 5: all such M up to kMaxM have a plan.
bool fft_length(int M) {
  if (M < 4) return false;
  for (int p : {2, 3, 5})
    while (M % p == 0) M /= p;
  return M == 1;
}

// The plan of fewest stages (at least two), among those one with the fewest LDS bank
// conflicts, with radices of at most M / 24 (or 6), so that two arrays have 48 butterflies
// to a stage (M = 96, one member: 16, 6 took 7.7 us, 4, 4, 6 takes 4.2).
FftPlan fft_plan(int M) {
  PlanSearch search{M, 2, std::max(6, M / 24)};
  for (; search.stages <= kMaxStages && search.best > 1e29; ++search.stages) search.visit(M, 0);
  return search.plan;
}

}  // namespace nse
