// Host-side AddressSanitizer harness for the graph bookkeeping of the C ABI (library host code
// built with -fsanitize=address, see build.sh): sequences launched, captured when they come
// back, replayed, evicted from a full cache and from the list of recent sequences, and dropped
// with the member blocks, for an ensemble on forked streams, contexts that share one stream, and
// trajectories with their adjoints. nse_graph_counts shows that each of these happened. Without
// a GPU it does nothing. The last line printed on success is "asan graphs: ok".
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "nse_sphere.h"

#define EXPECT(cond)                                                  \
  do {                                                                \
    if (!(cond)) {                                                    \
      std::fprintf(stderr, "asan graphs: check failed: %s (line %d)\n", #cond, __LINE__); \
      std::exit(2);                                                   \
    }                                                                 \
  } while (0)

static nse_params params() {
  nse_params p{};
  p.omega = 2.0 * M_PI;
  p.dt = 1e-3;
  p.order = 2;
  p.newton_iters = 1;
  p.precision = NSE_PREC_FP64;
  p.flags = NSE_FLAG_GRAPH | NSE_FLAG_CHECK_FINITE;
  return p;
}

static double* device_zeros(int64_t n) {
  double* d = nullptr;
  EXPECT(hipMalloc((void**)&d, sizeof(double) * 2 * n) == hipSuccess);
  EXPECT(hipMemset(d, 0, sizeof(double) * 2 * n) == hipSuccess);
  return d;
}

static void expect_counts(nse_ctx* c, int64_t captured, int64_t launched) {
  int64_t a = -1, b = -1;
  EXPECT(nse_graph_counts(c, &a, &b) == NSE_OK);
  if (a != captured || b != launched)
    std::fprintf(stderr, "asan graphs: captured %lld launched %lld, expected %lld and %lld\n",
                 (long long)a, (long long)b, (long long)captured, (long long)launched);
  EXPECT(a == captured && b == launched);
}

static void ensemble(hipStream_t st) {
  std::vector<nse_member> ms;
  for (int i = 0; i < 24; ++i) ms.push_back({i < 10 ? 63 : (i < 18 ? 127 : 255), 0, 1e-4});
  nse_params p = params();
  nse_ctx* c = nullptr;
  EXPECT(nse_sphere_init(ms.data(), (int)ms.size(), &p, st, &c) == NSE_OK);
  const int64_t S = nse_state_count(c);
  const int n = 11;  // more histories than graphs (8) and recent sequences (8) are kept
  std::vector<double*> hist;
  for (int k = 0; k < n; ++k) hist.push_back(device_zeros(3 * S));
  double* f = device_zeros(S);
  // short calls in turn: each has left the list of recent sequences when it comes again
  for (int round = 0; round < 2; ++round)
    for (double* h : hist) EXPECT(nse_step(c, h, f, 3, 10) == NSE_OK);
  expect_counts(c, 0, 0);
  // long calls: captured at once, the cache overflows
  for (double* h : hist) EXPECT(nse_step(c, h, f, 3, 40) == NSE_OK);
  expect_counts(c, n, 4 * n);
  // the last eight are kept, the first ones were evicted; short calls of those come back
  for (int k = n - 8; k < n; ++k) EXPECT(nse_step(c, hist[k], f, 3, 10) == NSE_OK);
  expect_counts(c, n, 4 * n + 8);
  for (int rep = 0; rep < 3; ++rep) EXPECT(nse_step(c, hist[0], f, 3, 10) == NSE_OK);
  expect_counts(c, n + 1, 4 * n + 10);
  EXPECT(nse_sync(c) == NSE_OK);
  EXPECT(nse_set_member_blocks(c, 20, 2, 4) == NSE_OK);  // drops the graphs
  for (int rep = 0; rep < 3; ++rep) EXPECT(nse_step(c, hist[1], f, 33, 20) == NSE_OK);
  expect_counts(c, n + 2, 4 * n + 14);
  EXPECT(nse_sync(c) == NSE_OK);
  EXPECT(nse_sphere_destroy(c) == NSE_OK);
  for (double* h : hist) (void)hipFree(h);
  (void)hipFree(f);
  std::printf("asan graphs: ensemble ok\n");
}

static void shared_stream(hipStream_t st) {
  std::vector<nse_ctx*> cs;
  std::vector<double*> hs;
  for (int i = 0; i < 24; ++i) {
    nse_member m = {i < 8 ? 63 : (i < 16 ? 127 : 255), 0, 1e-4};
    nse_params p = params();
    nse_ctx* c = nullptr;
    EXPECT(nse_sphere_init(&m, 1, &p, st, &c) == NSE_OK);
    cs.push_back(c);
    hs.push_back(device_zeros(3 * nse_state_count(c)));
  }
  for (int rep = 0; rep < 3; ++rep)
    for (size_t i = 0; i < cs.size(); ++i) EXPECT(nse_step(cs[i], hs[i], nullptr, 20 * rep, 23) == NSE_OK);
  for (size_t i = 0; i < cs.size(); ++i) {
    expect_counts(cs[i], 1, 4);
    EXPECT(nse_sphere_destroy(cs[i]) == NSE_OK);
    (void)hipFree(hs[i]);
  }
  std::printf("asan graphs: contexts on one stream ok\n");
}

static void trajectories(hipStream_t st) {
  nse_member m = {127, 0, 1e-4};
  nse_params p = params();
  nse_ctx* c = nullptr;
  EXPECT(nse_sphere_init(&m, 1, &p, st, &c) == NSE_OK);
  const int64_t S = nse_state_count(c);
  const int32_t nsteps = 25, depth = p.order + 1;
  double* hbar = device_zeros(depth * S);
  std::vector<double*> tr;
  for (int k = 0; k < 6; ++k) tr.push_back(device_zeros((nsteps + depth) * S));
  for (int rep = 0; rep < 3; ++rep) {  // launched, captured and replayed, replayed
    EXPECT(nse_step_trajectory(c, tr[0], nullptr, 3, nsteps) == NSE_OK);
    EXPECT(nse_step_adjoint_trajectory(c, tr[0], nullptr, 3, nsteps, hbar) == NSE_OK);
  }
  expect_counts(c, 2, 4);
  for (double* t : tr)  // twelve sequences in all: the cache overflows
    for (int rep = 0; rep < 3; ++rep) {
      EXPECT(nse_step_trajectory(c, t, nullptr, 0, nsteps) == NSE_OK);
      EXPECT(nse_step_adjoint_trajectory(c, t, nullptr, 0, nsteps, hbar) == NSE_OK);
    }
  // (from step 0 the range of fixed-coefficient steps differs from that of step 3)
  expect_counts(c, 2 + 12, 4 + 24);
  EXPECT(nse_sync(c) == NSE_OK);
  EXPECT(nse_sphere_destroy(c) == NSE_OK);
  for (double* t : tr) (void)hipFree(t);
  (void)hipFree(hbar);
  std::printf("asan graphs: trajectories ok\n");
}

int main() {
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) == hipSuccess && ndev > 0) {
    hipStream_t st = nullptr;
    EXPECT(hipStreamCreate(&st) == hipSuccess);
    ensemble(st);
    shared_stream(st);
    trajectories(st);
    EXPECT(hipStreamDestroy(st) == hipSuccess);
  } else {
    std::printf("asan graphs: no GPU, nothing run\n");
  }
  std::printf("asan graphs: ok\n");
  return 0;
}
