// Legendre contractions by degree pairs on the FP64 matrix cores (the direct sums
// in latitude of Section 4.2).
//
// For one order m let l_k = m + 2k, e(l) = sqrt((l^2 - m^2) / (4 l^2 - 1)) and
//   Q_k(mu) = Pbar[l_k + 1, m](mu) / mu,
// an even function of mu. The three-term recurrence of eq. (sph_har),
// mu Pbar[l] = e(l+1) Pbar[l+1] + e(l) Pbar[l-1], used twice, gives
//   Pbar[l_k, m]     = e(l_k + 1) Q_k + e(l_k) Q_{k-1},
//   Pbar[l_k + 1, m] = mu Q_k,
//   e(l_k+2) e(l_k+3) Q_{k+1} = (mu^2 - e(l_k+1)^2 - e(l_k+2)^2) Q_k - e(l_k) e(l_k+1) Q_{k-1},
// so a pair of degrees costs one recurrence step (the recurrence in mu^2 of K. Ishioka,
// J. Meteorol. Soc. Japan 96 (2018) 241-249). With Q_k = s_k q_k and
// s_{k+1} = s_{k-1} g_k / g_{k+1}, g_k = e(l_k) e(l_k + 1), s_0 = s_1 = 1, the step is
//   q_{k+1} = (A_k mu^2 + B_k) q_k - q_{k-1}.
// Its characteristic roots meet at +1 towards the pole (factor +2) and at -1 towards
// the equator (factor -2), where the rounding of the factor grows with the square of
// the number of steps. The kernels therefore carry a difference beside q:
//   pole     d_k = q_k - q_{k-1}:  d_{k+1} = tau q_k + d_k,  q_{k+1} = d_{k+1} + q_k,
//            tau = A_k (-sin^2) + (A_k + B_k - 2),
//   equator  d_k = q_k + q_{k-1}:  d_{k+1} = tau q_k - d_k,  q_{k+1} = d_{k+1} - q_k,
//            tau = A_k mu^2 + (B_k + 2),
// whose tau is small where the roots meet and is rounded relative to itself: three
// operations for two degrees (the degree-by-degree form takes three for one). With
// sigma = 1 at the pole, -1 at the equator, p_k = sigma^k q_k and e_k = sigma^k d_k (k from
// the start of the segment) both are the same step,
//   e_{k+1} = sigma tau p_k + e_k,  p_{k+1} = e_{k+1} + p_k,
// and the sign goes to the products of the odd rows. In between either form does; a wave
// takes the form of the half that holds its middle latitude.
// Unweighted sums of N = 511 over all orders: 4.7e-15 off (relative l2), 1.8e-14 with the
// two-operation step, 1.7e-14 with the degree-by-degree recurrence of the table.
// The even and the odd degrees of a pair share q_k, so the sums of all
// fields over both parities are one matrix product per order,
//   synthesis  C[lat][c] = sum_k q_k(mu_lat) B[k][c],   F(north/south) = E +- mu O,
//   analysis   S[k][c]   = sum_lat q_k(mu_lat) W[lat][c],
// with the columns c = (field; E.re, E.im, O.re, O.im): four columns per field,
// the width of v_mfma_f64_4x4x4_4b (73 TFLOP/s measured, against 49 for the
// 16x16x4 form and 68 for vector FMAs). The lanes that hold the matrix A run the
// recurrence themselves: the sum over k (and the set of rows k) may be taken in any
// order, so each of them walks its own segment of k from two seed values per
// latitude, stored once per group (computed in double-double), and nothing is
// exchanged between lanes.
//
// Operand layout of v_mfma_f64_4x4x4_4b (four independent 4x4x4 products, blocks
// blk; checked on gfx950): lane l supplies A[i = l%4][kk = l/16] and
// B[kk = l/16][j = l%4] of block (l/4)%4, and receives D[i = l/16][j = l%4] of it.
#include <algorithm>
#include <type_traits>

#include "adjoint_device.h"
#include "lane_ops.h"
#include "spectral_ops.h"

namespace nse {

namespace {

// Whether the latitudes p .. p + count - 1 take the polar form: their middle lies in the
// polar half.
__device__ __forceinline__ bool pair_polar(int p, int count, int nh) { return 2 * p + count <= nh; }
// The argument of sigma tau at node x, and d of a seed stored with the form of its tile.
__device__ __forceinline__ double pair_arg(bool polar, double x) {
  return -(polar ? (1.0 - x) * (1.0 + x) : x * x);
}
__device__ __forceinline__ double pair_diff(bool polar, const double2& seed, int tile, int nh) {
  return pair_polar(16 * tile, 16, nh) == polar ? seed.x : fma(2.0, seed.y, -seed.x);
}
// One step: rc = (A_k, A_k + B_k - 2) at the pole, (A_k, -B_k - 2) at the equator. SIGN -1:
// the equator's step of (d, q) themselves.
template <int SIGN = 0>
__device__ __forceinline__ void pair_step(const double2& rc, double t, double& e, double& p) {
  const double tau = fma(rc.x, t, rc.y);
  e = SIGN < 0 ? -fma(tau, p, e) : fma(tau, p, e);
  p = SIGN < 0 ? e - p : e + p;
}

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// Seeds, once per group: (d_k, q_k) at the first k of every segment, d_k of the polar form
// on the polar half of the tiles of 16 latitudes and of the other form on the rest, from
// the recurrence run in double-double from k = 0; the segments restart from values
// correct to the last place.
struct dd {
  double h, l;
};
#pragma clang fp contract(off)
__device__ __forceinline__ dd dd_fast(double a, double b) {
  const double s = a + b;
  return {s, b - (s - a)};
}
__device__ __forceinline__ dd dd_add(dd a, dd b) {
  const double s = a.h + b.h, v = s - a.h;
  const double e = (a.h - (s - v)) + (b.h - v);
  return dd_fast(s, e + (a.l + b.l));
}
__device__ __forceinline__ dd dd_mul(dd a, dd b) {
  const double p = a.h * b.h;
  const double e = __builtin_fma(a.h, b.h, -p);
  return dd_fast(p, e + (a.h * b.l + a.l * b.h));
}
__device__ __forceinline__ dd dd_scale(dd a, double s) { return {a.h * s, a.l * s}; }  // s = 2^n
__device__ __forceinline__ dd dd_sqrt(dd a) {
  if (!(a.h > 0.0)) return {0.0, 0.0};
  const double r = sqrt(a.h);
  const double p = r * r, e = __builtin_fma(r, r, -p);
  return dd_fast(r, ((a.h - p) - e + a.l) / (2.0 * r));
}
#pragma clang fp contract(fast)

// One thread per (latitude, order). pq0[m] = (-1)^m sqrt(prod (2i+1)/(2i)) / (sqrt(4 pi) e(m+1)),
// so q_0 = pq0[m] sin^m(theta); values below the double range flush to zero.
__global__ __launch_bounds__(64) void k_pair_seeds(GroupView g, int ks, const double2* rec_hi,
                                                   const double2* rec_lo, const double2* pq0,
                                                   double2* seeds) {
  const int N = g.N, nh = g.nh, m = blockIdx.y;
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nh) return;
  const int K = pair_count(N, m);
  const int64_t base = pair_slot(N, m);
  const double x = g.mu[p];
  const dd X = {x, 0.0};
  const dd y = dd_mul(X, X);
  dd q = {pq0[m].x, pq0[m].y};
  int ex = 0;  // value = q 2^ex
  {
    // sin^m(theta) by squaring, the exponent kept apart
    dd b = dd_sqrt(dd_mul(dd_add({1.0, 0.0}, {-x, 0.0}), dd_add({1.0, 0.0}, {x, 0.0})));
    int be = 0;
    for (int i = m; i > 0; i >>= 1) {
      if (i & 1) {
        q = dd_mul(q, b);
        ex += be;
      }
      b = dd_mul(b, b);
      be *= 2;
      if (b.h != 0.0) {
        const int s = ilogb(b.h);
        b = dd_scale(b, ldexp(1.0, -s));
        be += s;
      }
    }
  }
  const int len = pair_len(K, ks);
  const int64_t sbase = ((int64_t)m * ((nh + 15) / 16) + (p >> 4)) * (64 * ks) + (p & 15);
  const double sg = pair_polar(p & ~15, 16, nh) ? -1.0 : 1.0;
  dd q0 = {0.0, 0.0}, q1 = q;
  for (int k = 0; k < K; ++k) {
    if (k % len == 0) {
      const dd d = dd_add(q1, {sg * q0.h, sg * q0.l});
      seeds[sbase + (int64_t)(k / len) * 16] = make_double2(ldexp(d.h, ex), ldexp(q1.h, ex));
    }
    const double2 hi = rec_hi[base + k], lo = rec_lo[base + k];
    const dd t = dd_add(dd_mul({hi.x, lo.x}, y), {hi.y, lo.y});
    const dd z = dd_mul(t, q1);
    const dd n = dd_add(z, {-q0.h, -q0.l});
    q0 = q1;
    q1 = n;
    if (ex < 0 && fabs(q1.h) > 0x1p60) {
      const int s = min(60, -ex);
      q0 = dd_scale(q0, ldexp(1.0, -s));
      q1 = dd_scale(q1, ldexp(1.0, -s));
      ex += s;
    }
  }
}

}  // namespace

hipError_t launch_pair_seeds(const GroupView& g, int ks, const double2* rec_hi,
                             const double2* rec_lo, const double2* pq0, double2* seeds,
                             hipStream_t s) {
  dim3 grid((g.nh + 63) / 64, g.N + 1);
  hipLaunchKernelGGL(k_pair_seeds, grid, dim3(64), 0, s, g, ks, rec_hi, rec_lo, pq0, seeds);
  return hipGetLastError();
}

namespace {

// ---------------------------------------------------------------------------
// Synthesis. Workgroup of W waves per (order, TL W / KS tiles of 16 latitudes, member):
// the matrix B[k][c] of the order is built in LDS from the input state (a row of
// 16 or 20 columns followed by the two forms' coefficients), then wave w takes TL tiles and the
// (w mod KS)-th part of k, its four 16-lane groups a segment of it each.
constexpr int kPairCols = 16;

template <int NF>
constexpr int pair_row() {  // doubles per LDS row: columns, then (A, A + B - 2), (A, -B - 2)
  return (NF == 5 ? 20 : 16) + 4;
}

// Latitude of the tile that a lane supplies as row of A, and that it receives.
__device__ __forceinline__ int pair_row16(int lane) { return 4 * (lane & 3) + ((lane >> 2) & 3); }
__device__ __forceinline__ int pair_out16(int lane) { return 4 * (lane >> 4) + ((lane >> 2) & 3); }
// Item of launch position i of n: items have falling cost, and the positions of every
// other round of 256 (one workgroup per compute unit) take theirs backwards, so that
// the unit that was dealt the largest item gets the smallest of the next round.
__device__ __forceinline__ int pair_item(int i, int n) {
  const int r = i & ~255;
  return (i & 256) ? r + min(256, n - r) - 1 - (i & 255) : i;
}
// Order and member of this workgroup, false past the last one. With a member block
// (mb >= 2) mb members of one order follow each other on one XCD and share its L2 for
// the order's seeds and coefficients; without one the members follow each other.
// The latitude splits of one order (nsplit, splits of launch positions) are items
// of their own for one member.
__device__ __forceinline__ bool pair_place(const GroupView& g, int mb, int nsplit, int& m, int& b,
                                           int& split) {
  const int n = g.N + 1;
  if (g.nb == 1) {
    const int item = pair_item(blockIdx.x, n * nsplit);
    b = 0;
    // item / nsplit: exact in 16 fraction bits, item < 2^12
    m = nsplit == 1 ? item : (int)(((unsigned)item * (65536u / nsplit + 1u)) >> 16);
    split = item - m * nsplit;
    return true;
  }
  split = blockIdx.y;
  if (mb < 2) {
    b = blockIdx.x / n;
    m = blockIdx.x - b * n;
    return true;
  }
  const int item = xcd_item(blockIdx.x, mb), per = (g.nb + mb - 1) / mb * mb;
  m = item / per;
  b = item - m * per;
  return m <= g.N && b < g.nb;
}
inline dim3 pair_places(const GroupView& g, int mb, int nsplit) {
  if (g.nb == 1) return dim3((g.N + 1) * nsplit);
  if (mb < 2) return dim3((g.N + 1) * g.nb, nsplit);
  return dim3(xcd_grid((g.N + 1) * ((g.nb + mb - 1) / mb * mb), mb), nsplit);
}
// Keeps loaded values in registers from here on: every load before it is issued
// (and the arguments behind it are read) ahead of what follows, where the compiler
// would otherwise move each load into the branch that uses it.
__device__ __forceinline__ void pin(double2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)); }
template <typename T>
__device__ __forceinline__ void pin_arg(T v) {
  asm volatile("" ::"s"(v));
}
// State offset of member b (from the arguments where the members are evenly
// spaced: no dependent load ahead of the state's).
__device__ __forceinline__ int64_t member_offset(const GroupView& g, int b) {
  return g.ostride >= 0 ? g.off0 + b * g.ostride : g.off[b];
}

// MS: input sources of the instance (in.nsrc <= MS). The prologue's loads are
// unconditional (indices clamped, values masked afterwards): in one block the
// scalar loads of the arguments and the vector loads go out together, where a branch per
// load had put some twenty argument round trips in a row.
// Bound: at N = 511 the FP64 issue (products, recurrence) for 0.77 of the cycles, the rest the
// prologue and the stores: 27.5 us (25.6 with the two-operation step), 38 by single degrees on
// the vector units; five fields 34 against 82, 16 members of N = 255 64 against 95. At N = 255
// alone the chain of one workgroup: 11.2 against 11.4.
// TWO: a loop for each half of the latitudes, else one for both (see sums below).
template <int NF, int MS, int W, int TL, int KS, bool TWO>
__global__ __launch_bounds__(64 * W) void k_synthesis_pair(GroupView g, SynthInput in, int nsplit) {
  static_assert(NF >= 3 && NF <= 5 && W % KS == 0, "three (grid), four or five (adjoint) fields");
  constexpr int NT = 64 * W, RS = pair_row<NF>(), TW = TL * (W / KS);
  const int N = g.N, nh = g.nh, nlat = g.nlat;
  const int ntile = (nh + 15) / 16;
  int m, b, split;
  if (!pair_place(g, NF == 4 ? g.mb_synth : 0, nsplit, m, b, split)) return;  // uniform across the workgroup
  const int K = pair_count(N, m);  // degrees m .. N+1
  const int len = pair_len(K, KS), rows = 4 * KS * len;
  extern __shared__ double2 sh2[];
  double2* psi = sh2 + 1;                  // psi[-1 .. 2 K + 2]
  double2* zet = psi + 2 * K + 4;
  double2* fif = zet + 2 * K + 4;          // NF = 5: the fifth field's coefficients
  const int head = (NF == 5 ? 3 : 2) * (2 * K + 4);
  double* Bm = reinterpret_cast<double*>(sh2 + head);  // [rows][RS]

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kh = wave % KS;
  const int tile0 = split * TW + (wave / KS) * TL;
  const int64_t pbase = pair_slot(N, m);
  const double2 z2 = make_double2(0.0, 0.0);
  pin_arg(g.mu);
  pin_arg(g.pair_rec);
  pin_arg(g.pair_equ);
  pin_arg(g.pair_syn);
  pin_arg(g.pair_lam);
  const double2* seeds = KS == 2 ? g.seeds2 : g.seeds1;
  pin_arg(seeds);
  pin_arg(g.off0);
  pin_arg(g.ostride);
  pin_arg(g.gate);
#pragma unroll
  for (int i = 0; i < MS; ++i) {
    pin_arg(in.src[i]);
    pin_arg(in.coef[i]);
  }
  pin_arg(in.nsrc);
  // every global load of the prologue is requested before the first wait: the input
  // states (one degree per thread and pass), the pair coefficients of this
  // thread's row, the recurrence coefficients and the seeds. Waves past the last
  // degree or row load nothing: the loads' return path, 64 bytes a cycle and compute
  // unit, is what the prologue waits for.
  constexpr int NMAX = KS == 2 ? 340 : (64 * TW < kMaxM ? 64 * TW : kMaxM) / 3;  // 3 N + 2 <= M
  constexpr int SI = (NMAX + NT - 1) / NT;
  static_assert(NT >= NMAX / 2 + 2 + 8 * KS, "one row per thread");
  const int64_t abase = member_offset(g, b) + coeff_offset(N, m);
  double2 src[SI][MS], lm[SI], nb[SI];
#pragma unroll
  for (int u = 0; u < SI; ++u) {
    lm[u] = nb[u] = z2;
#pragma unroll
    for (int i = 0; i < MS; ++i) src[u][i] = z2;
    if (64 * wave + u * NT <= N - m) {
      const int kk = min((int)threadIdx.x + u * NT, N - m);
#pragma unroll
      for (int i = 0; i < MS; ++i) src[u][i] = in.src[i][abase + kk];
      lm[u] = g.pair_lam[m + kk];  // lambda^(-1/2), lambda^(1/2); zero at l = 0
      if (NF == 5) nb[u] = in.adj[abase + kk];
    }
  }
  double2 cf[4], rcv = z2, cc = z2, cs = z2;
  double rce = 0.0;
#pragma unroll
  for (int u = 0; u < 4; ++u) cf[u] = z2;
  if (64 * wave < K) {
    const int64_t k = pbase + min((int)threadIdx.x, K - 1);
    const double2* c = reinterpret_cast<const double2*>(g.pair_syn + k * 8);
#pragma unroll
    for (int u = 0; u < 4; ++u) cf[u] = c[u];
    rcv = g.pair_rec[k];
    rce = g.pair_equ[k];
    if (NF != 4) {
      cc = g.pair_con[2 * k];
      cs = g.pair_con[2 * k + 1];
    }
  }
  double2 sd[TL];
  double xa[TL], xo[TL];  // mu of the lane's latitude as A row, and of its output
#pragma unroll
  for (int t = 0; t < TL; ++t) {
    const int tile = min(tile0 + t, ntile - 1);
    sd[t] = seeds[(((int64_t)m * ntile + tile) * KS + kh) * 64 + (lane & 48) + pair_row16(lane)];
    xa[t] = g.mu[min(tile * 16 + pair_row16(lane), nh - 1)];
    xo[t] = g.mu[min(tile * 16 + pair_out16(lane), nh - 1)];
  }
#pragma unroll
  for (int u = 0; u < SI; ++u) {
#pragma unroll
    for (int i = 0; i < MS; ++i) pin(src[u][i]);
    pin(lm[u]);
    if (NF == 5) pin(nb[u]);
  }
#pragma unroll
  for (int u = 0; u < SI; ++u) {
    const int kk = threadIdx.x + u * NT, l = m + kk;
    if (kk <= N - m) {
      double2 v = z2;
#pragma unroll
      for (int i = 0; i < MS; ++i) {
        if (i < in.nsrc) {
          v.x += in.coef[i] * src[u][i].x;
          v.y += in.coef[i] * src[u][i].y;
        }
      }
      if (m == 0) v.y = 0.0;
      if (l == 0) v.x = 0.0;
      psi[kk] = make_double2(v.x * lm[u].x, v.y * lm[u].x);
      double2 zt = make_double2(v.x * lm[u].y, v.y * lm[u].y);
      if (NF != 3 && m == 0 && l == 1) zt.x += in.coriolis;
      zet[kk] = zt;
      if (NF == 5) {
        // fifth field: lambda^(-1/2) n_bar, real at m = 0 (n_bar formed here from
        // hbar_out[0] inside the step adjoint)
        double r = lm[u].x;
        if (in.adj_step) r *= -in.adj_h / (in.adj_c0 + in.adj_h * g.nu[b] * ((double)l * (l + 1)));
        fif[kk] = l == 0 ? z2 : make_double2(nb[u].x * r, m == 0 ? 0.0 : nb[u].y * r);
      }
    }
  }
  // zeros around the degrees m .. N: entries -1 and N - m + 1 .. 2 K + 2 (2 K + 2 <= N - m + 5)
  if (threadIdx.x < 8) {
    const int kk = threadIdx.x == 0 ? -1 : N - m + threadIdx.x;
    if (kk < 2 * K + 3) {
      psi[kk] = zet[kk] = z2;
      if (NF == 5) fif[kk] = z2;
    }
  }
  // an ended attempt of a device-controlled run: checked once the loads are in
  // flight (nothing is stored before this barrier), so the flag costs no wait
  if (gate_closed(g)) return;
  __syncthreads();
  // B of the rows: columns of fields 0 and 1 as [k][j][f], j = E.re, E.im, O.re, O.im, then
  // those of 2 and 3, then of 4 (16-byte pieces that the four lanes of a group read side by side)
#pragma unroll
  for (int u = 0; u < 4; ++u) pin(cf[u]);
  pin(rcv);
  pin(rce);
  if (NF != 4) {
    pin(cc);
    pin(cs);
  }
  if ((int)threadIdx.x < K) {
    const int k = threadIdx.x;
    double2* row = reinterpret_cast<double2*>(Bm + k * RS);
    // i m times the coefficients, and their colatitude derivative
    struct Cols {
      double2 mE, mO, dE, dO;
    };
    auto cols = [&](const double2* a) {
      const double2 am = a[-1], a0 = a[0], a1 = a[1], a2 = a[2], a3 = a[3];
      Cols c;
      c.mE = make_double2(-(cf[0].x * a0.y + cf[0].y * a2.y), cf[0].x * a0.x + cf[0].y * a2.x);
      c.mO = make_double2(-cf[1].x * a1.y, cf[1].x * a1.x);
      c.dE = make_double2(cf[1].y * am.x + cf[2].x * a1.x + cf[2].y * a3.x,
                          cf[1].y * am.y + cf[2].x * a1.y + cf[2].y * a3.y);
      c.dO = make_double2(cf[3].x * a0.x + cf[3].y * a2.x, cf[3].x * a0.y + cf[3].y * a2.y);
      return c;
    };
    auto plain = [&](const double2* z, double2& E, double2& O) {
      E = make_double2(cc.x * z[0].x + cc.y * z[2].x, cc.x * z[0].y + cc.y * z[2].y);
      O = make_double2(cs.x * z[1].x, cs.x * z[1].y);
    };
    const Cols p = cols(psi + 2 * k);
    row[0] = make_double2(p.mE.x, p.dE.x);
    row[1] = make_double2(p.mE.y, p.dE.y);
    row[2] = make_double2(p.mO.x, p.dO.x);
    row[3] = make_double2(p.mO.y, p.dO.y);
    if constexpr (NF == 3) {
      // grid mode: the third field is the vorticity, or Psi_N = -psi
      const double sg = in.stream ? -1.0 : 1.0;
      double2 E, O;
      plain((in.stream ? psi : zet) + 2 * k, E, O);
      row[4] = make_double2(sg * E.x, 0.0);
      row[5] = make_double2(sg * E.y, 0.0);
      row[6] = make_double2(sg * O.x, 0.0);
      row[7] = make_double2(sg * O.y, 0.0);
    } else {
      const Cols z = cols(zet + 2 * k);
      row[4] = make_double2(z.dE.x, z.mE.x);
      row[5] = make_double2(z.dE.y, z.mE.y);
      row[6] = make_double2(z.dO.x, z.mO.x);
      row[7] = make_double2(z.dO.y, z.mO.y);
    }
    if constexpr (NF == 5) plain(fif + 2 * k, row[8], row[9]);
    row[RS / 2 - 2] = rcv;
    row[RS / 2 - 1] = make_double2(rcv.x, -rce);
  } else if ((int)threadIdx.x < rows) {
    double2* row = reinterpret_cast<double2*>(Bm + threadIdx.x * RS);
#pragma unroll
    for (int j = 0; j < RS / 2; ++j) row[j] = z2;
  }
  __syncthreads();

  double acc[TL][NF];
#pragma unroll
  for (int t = 0; t < TL; ++t)
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[t][f] = 0.0;
  if (tile0 < ntile) {
    // two rows at a time; the next two rows' operands are read from LDS during
    // this pair's products (the last pair reads its own rows again)
    const double* row = Bm + (4 * kh + (lane >> 4)) * len * RS;
    const double* col = row + 2 * (lane & 3);
    const bool polar = pair_polar(16 * tile0, 16 * TL, nh);
    const double* form = row + (polar ? RS - 4 : RS - 2);
    const double sigma = polar ? 1.0 : -1.0;
    double e[TL], p[TL], tx[TL];
#pragma unroll
    for (int t = 0; t < TL; ++t) {
      e[t] = pair_diff(polar, sd[t], min(tile0 + t, ntile - 1), nh);
      p[t] = sd[t].y;
      tx[t] = pair_arg(polar, xa[t]);
    }
    // SIGN 1, -1: a loop for each half, with q itself (the signs are operand modifiers);
    // 0: one loop for both with p_k = sigma^k q_k
    auto sums = [&](auto sign) {
      constexpr int SIGN = decltype(sign)::value;
      struct Ops {
        double2 b01, b23, rc;
        double b4;
      };
      auto read = [&](int off) {
        Ops o;
        o.b01 = *reinterpret_cast<const double2*>(col + off);
        o.b23 = *reinterpret_cast<const double2*>(col + off + 8);
        o.rc = *reinterpret_cast<const double2*>(form + off);
        o.b4 = NF == 5 ? row[off + 16 + (lane & 3)] : 0.0;
        return o;
      };
      auto keep = [](Ops& o) {
        pin(o.b01);
        pin(o.b23);
        pin(o.rc);
        if constexpr (NF == 5) pin(o.b4);
      };
      auto step = [&](const Ops& o, bool odd) {
#pragma unroll
        for (int t = 0; t < TL; ++t) {
          const double q = SIGN == 0 && odd ? sigma * p[t] : p[t];
          acc[t][0] = mfma4(q, o.b01.x, acc[t][0]);
          acc[t][1] = mfma4(q, o.b01.y, acc[t][1]);
          acc[t][2] = mfma4(q, o.b23.x, acc[t][2]);
          if constexpr (NF >= 4) acc[t][3] = mfma4(q, o.b23.y, acc[t][3]);
          if constexpr (NF == 5) acc[t][4] = mfma4(q, o.b4, acc[t][4]);
          pair_step<SIGN>(o.rc, tx[t], e[t], p[t]);
        }
      };
      Ops o0 = read(0), o1 = read(RS);
      for (int j = 0; j < len; j += 2) {
        const int nx = j + 2 < len ? (j + 2) * RS : j * RS;
        Ops n0 = read(nx), n1 = read(nx + RS);
        step(o0, false);
        step(o1, true);
        keep(n0);
        keep(n1);
        o0 = n0;
        o1 = n1;
      }
    };
    if constexpr (!TWO) {
      sums(std::integral_constant<int, 0>{});
    } else if (polar) {
      sums(std::integral_constant<int, 1>{});
    } else {
      sums(std::integral_constant<int, -1>{});
    }
  }
  if constexpr (KS > 1) {
    // the parts of k meet in LDS (the matrix B is no longer needed)
    static_assert(KS == 2, "two parts");
    double* red = Bm + (wave / KS) * (TL * NF * 64) + lane;
    __syncthreads();
    if (kh) {
#pragma unroll
      for (int t = 0; t < TL; ++t)
#pragma unroll
        for (int f = 0; f < NF; ++f) red[(t * NF + f) * 64] = acc[t][f];
    }
    __syncthreads();
    if (kh) return;
#pragma unroll
    for (int t = 0; t < TL; ++t)
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[t][f] += red[(t * NF + f) * 64];
  }
  // lane: latitude 4 i + blk of the tile, column j; E and O sit two lanes apart. The four
  // fields then change places with the four blk, so that a store writes the 64 bytes
  // of a latitude's fields (the fifth field of NF = 5 lies by itself). At N = 511 this
  // costs the synthesis 1.2 us and saves the rings 4
  const int64_t fstride = (int64_t)(N + 1) * nlat;
  double* Fo = reinterpret_cast<double*>((NF == 5 ? g.Fa + b * 5 * fstride : g.F + b * 4 * fstride) +
                                         (int64_t)m * nlat * 4);
  const bool odd = (lane & 2) != 0;
#pragma unroll
  for (int t = 0; t < TL; ++t) {
    double r[NF < 4 ? 4 : NF];
    r[3] = 0.0;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const double v = acc[t][f], w = lane_dpp<kDppQuadXor2>(v);
      r[f] = odd ? fma(-xo[t], v, w) : fma(xo[t], w, v);
    }
    double r4[4] = {r[0], r[1], r[2], r[3]};
    transpose_banks(r4);
    const int p0 = (tile0 + t) * 16 + 4 * (lane >> 4), fl = (lane >> 2) & 3;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = p0 + i, q = odd ? nlat - 1 - p : p;  // southern ring, northern ring
      if (tile0 + t < ntile && p < nh && (!odd || q != p)) Fo[(q * 4 + fl) * 2 + (lane & 1)] = r4[i];
    }
    if constexpr (NF == 5) {
      const int p = (tile0 + t) * 16 + pair_out16(lane), q = odd ? nlat - 1 - p : p;
      double* F4 = reinterpret_cast<double*>(g.Fa + b * 5 * fstride + 4 * fstride + (int64_t)m * nlat);
      if (tile0 + t < ntile && p < nh && (!odd || q != p)) F4[2 * q + (lane & 1)] = r[4];
    }
  }
}

template <int NF, int W, int TL, int KS>
size_t synth_pair_lds(int N) {
  const int K = pair_count(N, 0), len = pair_len(K, KS);
  const size_t mat = sizeof(double) * (size_t)(4 * KS * len) * pair_row<NF>();
  const size_t red = KS > 1 ? sizeof(double) * (size_t)(W / KS) * TL * NF * 64 : 0;
  return sizeof(double2) * (size_t)((NF == 5 ? 3 : 2) * (2 * K + 4)) + std::max(mat, red);
}

template <int NF, int MS, int W, int TL, int KS, bool TWO = (NF < 5)>
hipError_t launch_synth_pair_as(const GroupView& g, SynthInput in, hipStream_t s) {
  constexpr int TW = TL * (W / KS);
  if (in.nsrc < 1 || in.nsrc > MS) return hipErrorInvalidValue;
  for (int i = in.nsrc; i < MS; ++i) in.src[i] = in.src[0];  // loaded, not used
  const int nsplit = ((g.nh + 15) / 16 + TW - 1) / TW;
  const size_t lds = synth_pair_lds<NF, W, TL, KS>(g.N);
  const dim3 grid = pair_places(g, NF == 4 ? g.mb_synth : 0, nsplit);
  hipLaunchKernelGGL((k_synthesis_pair<NF, MS, W, TL, KS, TWO>), grid, dim3(64 * W), lds, s, g, in, nsplit);
  return hipGetLastError();
}

// Segments per order: eight (two waves share an order's rows) for single members on grids
// below nh = 256, where the chain of a workgroup counts (N = 255: synthesis 11.1 us against
// 12.1 with four, five fields 12.9 against 14.5, adjoint 12.6 against 24.6; N = 300:
// synthesis 16.4 against 18.6); four elsewhere.
bool pair_eight(const GroupView& g, int mb) { return g.nh < 256 && mb < 2; }

template <int NF, int MS>
hipError_t launch_synth_pair_nf(const GroupView& g, const SynthInput& in, hipStream_t s) {
  // Two loops save the signs of the odd rows and take 4 to 30 VGPRs more. They pay while the
  // workgroups are resident at once: N = 511, four fields 27.1 us against 28.4, five (135
  // VGPRs, three waves per SIMD) 43 against 33.4; eight segments and two workgroups per
  // order at N = 255 11.3 against 11.7, three at N = 300 17.2 against 16.1
  if (pair_eight(g, NF == 4 ? g.mb_synth : 0)) {
    if (NF < 5 && g.nh <= 192) return launch_synth_pair_as<NF, MS, 6, 2, 2>(g, in, s);
    return launch_synth_pair_as<NF, MS, 6, 2, 2, false>(g, in, s);
  }
  if (g.nh <= 48) return launch_synth_pair_as<NF, MS, 3, 1, 1>(g, in, s);
  if (g.nh <= 96) return launch_synth_pair_as<NF, MS, 2, 3, 1>(g, in, s);
  if (g.nh <= 192) return launch_synth_pair_as<NF, MS, 4, 3, 1>(g, in, s);
  // (N = 511, measured with the two-operation step: eight waves of three tiles 25.3 us, four of
  // three 29.8, six of four 29.6)
  return launch_synth_pair_as<NF, MS, 8, 3, 1>(g, in, s);
}

}  // namespace

hipError_t launch_synthesis_pair(const GroupView& g, const SynthInput& in, int mode,
                                 hipStream_t s) {
  switch (mode) {
    case SYNTH_GRID: return launch_synth_pair_nf<3, 1>(g, in, s);
    case SYNTH_ADJ:
      return in.nsrc <= 3 ? launch_synth_pair_nf<5, 3>(g, in, s)
                          : launch_synth_pair_nf<5, kMaxSources>(g, in, s);
    default:
      return in.nsrc <= 3 ? launch_synth_pair_nf<4, 3>(g, in, s)
                          : launch_synth_pair_nf<4, kMaxSources>(g, in, s);
  }
}

namespace {

// ---------------------------------------------------------------------------
// Analysis. Workgroup of W waves per (order, member). The k range is cut into four
// segments of `len` rows; a wave holds GW groups of 16 latitudes (their
// recurrences and folded spectra in registers) and walks the rows once: row j of all
// segments is summed over the wave's latitudes by GW products into one accumulator,
// its blocks of different latitudes are added (row rotations) and the sums go to
// LDS, where the waves meet. The lane butterfly of the degree-by-degree form moved
// every sum through six exchanges. N = 511: 18.6 us against 30 by single degrees, bound by
// the FP64 issue for 0.55 of the cycles (0.8 for 16 members of N = 255) and the load phase; 16 members of N = 255 38
// against 38, 24 of N = 127 14.3 and of N = 63 7 against 9. (A conditional over whole
// double2 values at the LDS stores had put the loaded values into scratch memory: 19.6, 41.8,
// 19.3 and 9.8 us with the shorter step.)
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
  return v + lane_dpp<CTRL>(v);
}
constexpr int kDppRowRor8 = 0x128;  // lane l of a 16-lane row reads lane (l - 8) mod 16
constexpr int kDppRowRor4 = 0x124;

// Doubles per row of the sums in LDS: [seg][4], padded so that neighbouring rows
// start in different banks (the epilogue reads down the rows).
template <int KS>
constexpr int pair_sums() {
  return 16 * KS + 1;
}
// The adjoint's sums take the rows about a segment too (see EDGE) where segments are long:
// with eight segments per order and at most 22 rows the spikes are below 3e-13.
template <int KS>
constexpr bool pair_edge() {
  return KS == 1;
}
// Coefficients of n rows (segments side by side) in LDS: (A_k, A_k + B_k - 2) then
// (A_k, -B_k - 2), 16 bytes a read (N = 511: 18.6 us against 20.3 for two reads), or PACKED
// A_k, A_k + B_k - 2, -B_k - 2, where two workgroups on a compute unit need the room.
template <bool PACKED>
struct PairRec {
  static constexpr int kRow = PACKED ? 3 : 4;  // doubles per row
  const double *a, *b;
  __device__ __forceinline__ PairRec(const double* rec, int n, int r, bool polar)
      : a(PACKED ? rec + r : rec + 2 * (r + (polar ? 0 : n))), b(rec + r + (polar ? 1 : 2) * n) {}
  __device__ __forceinline__ double2 get(int r) const {
    return PACKED ? make_double2(a[r], b[r]) : *reinterpret_cast<const double2*>(a + 2 * r);
  }
  static __device__ __forceinline__ void put(double* rec, int n, int r, double A, double pole,
                                             double equ) {
    if (PACKED) {
      rec[r] = A;
      rec[n + r] = pole;
      rec[2 * n + r] = equ;
    } else {
      double2* v = reinterpret_cast<double2*>(rec);
      v[r] = make_double2(A, pole);
      v[n + r] = make_double2(A, equ);
    }
  }
};
// Rows of one wave: red[j pair_sums + seg 4 + col] = sum over the wave's latitudes of
// q_k W[lat][col], k = seg len + j. The wave's latitudes start at p0, its group i holds
// p0 + LG i .. + LG - 1 (this lane's: lo of them). w [lat][4], rec: PairRec.
// EDGE: the rows before and after the segment too, j = -1 .. len at rows 0 .. len + 1. The
// adjoint's sums over neighbouring rows cancel to 1 / l^2 near the equator; across segments,
// one continued over 66 rows and one fresh from its seed, the cancellation leaves
// 1e-12 of an order's rms at single degrees (N = 511), within one 1e-13.
template <int GW, int KS, bool EDGE = false, int FW = 1>
__device__ __forceinline__ void pair_rows(const double2 (&seed)[GW], const double (&x)[GW],
                                          const double (&w)[FW][GW], int p0, int lo, int nh, int len,
                                          const double* rec, double* red, int lane) {
  constexpr int NS = 4 * KS, LG = 16 / KS;
  const int segA = (lane & 3) + 4 * (((lane >> 2) & 3) % KS);
  const int segD = (lane >> 4) + 4 * (((lane >> 2) & 3) % KS);
  const bool polar = pair_polar(p0, GW * LG, nh);
  const double sigma = polar ? 1.0 : -1.0;
  const PairRec<EDGE> rl(rec, len * NS, segA, polar);
  const int rows = EDGE ? len + 2 : len;
  double* out = red + segD * 4 + (lane & 3);
  const bool wr = (lane & 12) < 4 * KS;
  double e[GW], p[GW], t[GW];
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    e[i] = pair_diff(polar, seed[i], min(p0 + i * LG + lo, nh - 1) >> 4, nh);
    p[i] = seed[i].y;
    t[i] = pair_arg(polar, x[i]);
  }
  auto store = [&](const double (&v0)[FW], const double (&v1)[FW], int j, bool odd) {
#pragma unroll
    for (int f = 0; f < FW; ++f) {
      double v = GW > 1 ? v0[f] + v1[f] : v0[f];
      if (odd) v *= sigma;
      if (KS <= 2) v = add_dpp<kDppRowRor8>(v);
      if (KS == 1) v = add_dpp<kDppRowRor4>(v);
      if (wr) out[(f * rows + j) * pair_sums<KS>()] = v;
    }
  };
  // back: the row before the state's; go: the state moves on to the next row
  auto row = [&](const double2& rc, int j, bool odd, bool back, bool go) {
    double v0[FW], v1[FW];
#pragma unroll
    for (int f = 0; f < FW; ++f) v0[f] = v1[f] = 0.0;
#pragma unroll
    for (int i = 0; i < GW; ++i) {
      const double q = back ? p[i] - e[i] : p[i];
#pragma unroll
      for (int f = 0; f < FW; ++f) {
        if (i & 1)
          v1[f] = mfma4(q, w[f][i], v1[f]);
        else
          v0[f] = mfma4(q, w[f][i], v0[f]);
      }
      if (go) pair_step(rc, t[i], e[i], p[i]);
    }
    store(v0, v1, j, odd);
  };
  double2 r0 = rl.get(0), r1 = rl.get(NS);
  const int j0 = EDGE ? 1 : 0;
  if (EDGE) row(r0, 0, true, true, false);
  for (int j = 0; j < len; j += 2) {
    const int nx = (j + 2 < len ? j + 2 : j) * NS;
    double2 n0 = rl.get(nx), n1 = rl.get(nx + NS);
    row(r0, j + j0, false, false, true);
    row(r1, j + 1 + j0, true, false, true);
    pin(n0);
    pin(n1);
    r0 = n0;
    r1 = n1;
  }
  if (EDGE) row(r0, len + 1, false, false, false);
}

// Segment and row of k (k < 2^9).
__device__ __forceinline__ int2 pair_seg(int k, int len, float rlen) {
  const int seg = (int)(((float)k + 0.5f) * rlen);
  return make_int2(seg, k - seg * len);
}
// Sum over the waves of columns (c, c + 1) of row j of a segment.
template <int W, int KS>
__device__ __forceinline__ double2 pair_fetch(const double* red, int seg, int j, int c, int stride) {
  const double* r = red + j * pair_sums<KS>() + seg * 4 + c;
  double2 v = make_double2(0.0, 0.0);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    v.x += r[w * stride];
    v.y += r[w * stride + 1];
  }
  return v;
}

// Inputs of the step update of one coefficient (as load_degree_inputs) with DEP >=
// out.depth history rows, loaded without branches.
template <int DEP>
__device__ __forceinline__ void load_step_inputs(const AnalOutput& out, int64_t slot, double2* in) {
  const double2 f = (out.forcing ? out.forcing : out.hist)[slot];
  in[0] = out.forcing ? f : make_double2(0.0, 0.0);
#pragma unroll
  for (int j = 0; j < kDegreeInputs - 1; ++j)
    in[1 + j] = j < DEP ? out.hist[(j < out.depth ? j : 0) * out.state_count + slot]
                        : make_double2(0.0, 0.0);
}

// The step update of degree l of order m (as finish_degree_from; n = sum lambda^(-1/2)).
template <int DEP>
__device__ __forceinline__ void finish_step(const AnalOutput& out, double nu, int l, int m,
                                            int64_t slot, double2 n, const double2* in) {
  if (l < 1) n = make_double2(0.0, 0.0);
  if (m == 0) n.y = 0.0;
  double2 rhs = make_double2(out.h * in[0].x, out.h * in[0].y);
  rhs.x -= out.h * n.x;
  rhs.y -= out.h * n.y;
#pragma unroll
  for (int j = 1; j <= DEP; ++j) {
    if (j < out.ncoef) {
      rhs.x -= out.c[j] * in[j].x;
      rhs.y -= out.c[j] * in[j].y;
    }
  }
  const double denom = out.c[0] + out.h * nu * ((double)l * (l + 1));
  double2 a = make_double2(rhs.x / denom, rhs.y / denom);
  if (l == 0) a = make_double2(0.0, 0.0);
  if (m == 0) a.y = 0.0;
  if (out.nonfinite && !(isfinite(a.x) && isfinite(a.y))) *out.nonfinite = 1;
  if (out.mode == ANAL_STEP_ITER) {
    out.iter[slot] = a;
    return;
  }
  if (out.shift) {
    out.hist[slot - out.state_count] = a;
    return;
  }
#pragma unroll
  for (int j = DEP - 1; j >= 1; --j)
    if (j < out.depth) out.hist[(int64_t)j * out.state_count + slot] = in[j];
  out.hist[slot] = a;
}

// DEP: 0 nonlinear mode, 3 or 6 step modes with that many history rows at most,
// -1 ANAL_NDF.
template <int W, int GW, int DEP>
__global__ __launch_bounds__(64 * W) void k_analysis_pair(GroupView g, AnalOutput out) {
  constexpr int NT = 64 * W, NS = 4, LG = 16;
  constexpr bool NDF = DEP < 0;
  const int N = g.N, nh = g.nh, nlat = g.nlat;
  int m, b, split;
  if (!pair_place(g, g.mb_anal, 1, m, b, split)) return;  // uniform across the workgroup
  const int K = pair_count(N, m), len = pair_len(K, 1);
  const int nhp = (nh + 15) & ~15;
  extern __shared__ double2 sh2[];
  double* rec = reinterpret_cast<double*>(sh2);        // PairRec of [len][NS]
  double* red = rec + PairRec<false>::kRow * len * NS;  // [W][len][pair_sums]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double2 z2 = make_double2(0.0, 0.0);
  const int64_t pbase = pair_slot(N, m);
  pin_arg(g.mu);
  pin_arg(g.pair_rec);
  pin_arg(g.pair_equ);
  pin_arg(g.pair_con);
  pin_arg(g.pair_lam);
  pin_arg(g.seeds1);
  pin_arg(g.W);
  pin_arg(g.gate);
  // the step's parameters are read ahead of the sums too: behind them each would
  // cost the epilogue a round trip of its own
  const double nu = DEP > 0 ? g.nu[b] : 0.0;
  if constexpr (DEP > 0) {
    pin_arg(nu);
    pin_arg(out.h);
    pin_arg(out.hist);
    pin_arg(out.iter);
    pin_arg(out.forcing);
    pin_arg(out.nonfinite);
    pin_arg(out.state_count);
    pin_arg(out.mode);
    pin_arg(out.shift);
    pin_arg(out.depth);
    pin_arg(out.ncoef);
#pragma unroll
    for (int j = 0; j <= DEP; ++j) pin_arg(out.c[j]);
  }
  // Every global load of the prologue is requested at once (indices clamped, values
  // masked afterwards): recurrence coefficients, then per latitude group of the wave
  // the seeds, the node and the lane's component (re or im) of the two rings of its
  // latitude, from which the lane forms its own column of We = Q(p) + Q(p') or
  // mu Wo = mu (Q(p) - Q(p')).
  constexpr int RI = (kMaxM / 3 / 2 + 2 + 2 * NS + NT - 1) / NT;
  double2 rcv[RI];
  double rce[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int r = threadIdx.x + i * NT;
    const int64_t k = pbase + min((r % NS) * len + r / NS, K - 1);
    rcv[i] = g.pair_rec[k];
    rce[i] = g.pair_equ[k];
  }
  double2 seed[GW];
  double x[GW], w[1][GW], qs[GW];
  const int lo = (lane >> 4) + 4 * ((lane >> 2) & 3), segA = lane & 3;
  const double* Wb = reinterpret_cast<const double*>(g.W + ((int64_t)b * (N + 1) + m) * nlat) + (lane & 1);
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    const int p = min((wave * GW + i) * LG + lo, nh - 1);
    seed[i] = g.seeds1[(((int64_t)m * (nhp >> 4) + (p >> 4)) * NS + segA) * 16 + (p & 15)];
    x[i] = g.mu[p];
    w[0][i] = Wb[2 * p];
    qs[i] = Wb[2 * (nlat - 1 - p)];
  }
  // the step update's inputs of the thread's first degree, and the pair coefficients
  const int La = N + 1 - m;  // degrees m .. N
  const int64_t sbase = member_offset(g, b) + coeff_offset(N, m);
  double2 din[kDegreeInputs], c0 = z2, c1 = z2;
  double rs = 0.0;
  auto load_inputs = [&](int k) {
    if constexpr (NDF)
      load_degree_inputs<true>(g, out, b, m, k, din);
    else if constexpr (DEP > 0)
      load_step_inputs<DEP>(out, sbase + k, din);
    const int kp = k >> 1;
    rs = g.pair_lam[m + k].x;
    c0 = g.pair_con[2 * (pbase + kp) + (k & 1)];          // (c1, c2) or (s, -)
    c1 = g.pair_con[2 * (pbase + (kp > 0 ? kp - 1 : 0))];  // of the pair before
  };
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int r = threadIdx.x + i * NT;
    pin(rcv[i]);
    pin(rce[i]);
    if (r < len * NS) {
      const bool in = (r % NS) * len + r / NS < K;
      PairRec<false>::put(rec, len * NS, r, in ? rcv[i].x : 0.0, in ? rcv[i].y : 0.0, in ? -rce[i] : 0.0);
    }
  }
  // an ended attempt of a device-controlled run: checked once the loads are in
  // flight (nothing is stored before this barrier), so the flag costs no wait
  if (NDF || DEP == 0) {
    if (gate_closed(g)) return;
  }
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    pin(seed[i]);
    pin(x[i]);
    pin(w[0][i]);
    pin(qs[i]);
    const double v = (lane & 2) ? x[i] * (w[0][i] - qs[i]) : w[0][i] + qs[i];
    w[0][i] = (wave * GW + i) * LG + lo < nh ? v : 0.0;
  }
  // (behind the loads that the sums need)
  if (!NDF && 64 * wave < La) load_inputs(min((int)threadIdx.x, La - 1));
  __syncthreads();
  pair_rows<GW, 1>(seed, x, w, wave * GW * LG, lo, nh, len, rec, red + wave * len * pair_sums<1>(), lane);
  const float rlen = 1.0f / (float)len;
  const int stride = len * pair_sums<1>();
  double nv[4] = {0.0, 0.0, 0.0, 0.0};
  if (NDF && (int)threadIdx.x < La) load_inputs(threadIdx.x);
  __syncthreads();
  for (int k = threadIdx.x; k < La; k += NT) {
    const int kp = k >> 1;
    if (k >= NT) load_inputs(k);
    const int2 at = pair_seg(kp, len, rlen);
    double2 v = pair_fetch<W, 1>(red, at.x, at.y, 2 * (k & 1), stride);
    v.x *= c0.x;
    v.y *= c0.x;
    if (!(k & 1) && kp > 0) {
      const int2 before = pair_seg(kp - 1, len, rlen);
      const double2 u = pair_fetch<W, 1>(red, before.x, before.y, 0, stride);
      v.x = fma(c1.y, u.x, v.x);
      v.y = fma(c1.y, u.y, v.y);
    }
    if constexpr (NDF) {
      double t[4] = {0.0, 0.0, 0.0, 0.0};
      finish_degree_from<true>(g, out, b, m, k, v.x, v.y, din, t, &rs);
#pragma unroll
      for (int i = 0; i < 4; ++i) nv[i] = lane_nanmax(nv[i], t[i]);
    } else if constexpr (DEP > 0) {
      finish_step<DEP>(out, nu, m + k, m, sbase + k, make_double2(v.x * rs, v.y * rs), din);
    } else {
      finish_degree_from(g, out, b, m, k, v.x, v.y, din, nullptr, &rs);
    }
  }
  if constexpr (NDF) {
    const int copy = (blockIdx.x * W + wave) % kNdfSpread;
    const double mx = lane_max4(nv);  // lane 16 q: the wave's maximum of nv[q]
    if ((lane & 15) == 0) {
      unsigned long long bits = (unsigned long long)__double_as_longlong(mx);
      if (mx != mx) bits = 0x7ff8000000000000ull;  // one positive NaN pattern
      atomicMax(out.nrow + copy * kNdfSpreadStride + (lane >> 4), bits);
    }
  }
}

template <int W>
size_t anal_pair_lds(int N) {
  const size_t len = pair_len(pair_count(N, 0), 1);
  return PairRec<false>::kRow * len * 32 + len * pair_sums<1>() * 8 * W;
}

template <int W, int GW>
hipError_t launch_anal_pair_as(const GroupView& g, const AnalOutput& out, hipStream_t s) {
  const size_t lds = anal_pair_lds<W>(g.N);
  const dim3 grid = pair_places(g, g.mb_anal, 1), block(64 * W);
  if (out.mode == ANAL_NDF)
    hipLaunchKernelGGL((k_analysis_pair<W, GW, -1>), grid, block, lds, s, g, out);
  else if (out.mode == ANAL_NONLINEAR)
    hipLaunchKernelGGL((k_analysis_pair<W, GW, 0>), grid, block, lds, s, g, out);
  else if (out.depth <= 3)
    hipLaunchKernelGGL((k_analysis_pair<W, GW, 3>), grid, block, lds, s, g, out);
  else
    hipLaunchKernelGGL((k_analysis_pair<W, GW, 6>), grid, block, lds, s, g, out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_analysis_pair(const GroupView& g, const AnalOutput& out, hipStream_t s) {
  // W GW tiles of 16 latitudes cover the nh of the size class
  if (g.nh <= 48) return launch_anal_pair_as<1, 3>(g, out, s);
  if (g.nh <= 96) return launch_anal_pair_as<1, 6>(g, out, s);
  if (g.nh <= 192) return launch_anal_pair_as<3, 4>(g, out, s);
  if (g.nh <= 320) return launch_anal_pair_as<4, 5>(g, out, s);
  return launch_anal_pair_as<4, 6>(g, out, s);
}

namespace {

// ---------------------------------------------------------------------------
// Adjoint of the synthesis and of its spectral prologue: the unweighted analysis of
// the field-spectrum cotangents Fbar[b][f][m][lat] to degree N+1 by the same row
// products, then the transposed synthesis columns (pair_syn) per degree,
//   psi_bar[2k]   = -i (mc1_k E0_k + mc2_{k-1} E0_{k-1}) + b1_k O1_k + b2_{k-1} O1_{k-1},
//   psi_bar[2k+1] = -i ms_k O0_k + a1_{k+1} E1_{k+1} + a2_k E1_k + a3_{k-1} E1_{k-1},
// zeta_bar the same from f3 and f2, and
//   alpha_bar = lambda^(-1/2) psi_bar + lambda^(1/2) zeta_bar
// (zero at l = 0, real at m = 0), stored or used in the adjoint of the NDF step. One
// workgroup holds an order, so the degrees couple through LDS and no panel
// cotangents go through memory. NFLD = 2: f0 and f1 only (the projection).
// Waves: WL groups of latitudes for every FW fields. N = 511: 41.4 us against 111 for the
// analysis from a table and 6.5 for the transpose (two fields 25); N = 255 with the step
// adjoint 13.5 against 13.7 and 4.9. Bound by the FP64 issue with the row sums, 0.8 of the
// cycles, then by the 25 MB of Fbar at its start.
// DEP: 0, or the step adjoint with that many history rows at most.
template <int NFLD, int FW, int WL, int GW, int KS, int DEP>
__global__ __launch_bounds__(64 * WL * (NFLD / FW), 4) void k_adjoint_pair(GroupView g,
                                                                      double2* alpha_bar,
                                                                      StepAdjointArgs sa) {
  constexpr int W = WL * (NFLD / FW), NT = 64 * W, NS = 4 * KS, LG = 16 / KS;
  constexpr int RSUM = pair_sums<KS>();
  constexpr bool EDGE = pair_edge<KS>();
  const int N = g.N, nh = g.nh, nlat = g.nlat;
  int m, b, split;
  if (!pair_place(g, 0, 1, m, b, split)) return;  // uniform across the workgroup
  const int K = pair_count(N, m), len = pair_len(K, KS), rows = EDGE ? len + 2 : len;
  const int nhp = (nh + 15) & ~15;
  extern __shared__ double2 sh2[];
  double* rec = reinterpret_cast<double*>(sh2);       // PairRec of [len][NS]
  double* wf = rec + PairRec<EDGE>::kRow * len * NS;  // [NFLD][nhp][4]
  double* red = wf;                                   // [W][FW][rows][RSUM], after the fold is read
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wl = wave % WL, f0 = (wave / WL) * FW;
  const double2 z2 = make_double2(0.0, 0.0);
  const int64_t pbase = pair_slot(N, m);
  pin_arg(g.mu);
  pin_arg(g.pair_rec);
  pin_arg(g.pair_equ);
  pin_arg(g.pair_syn);
  pin_arg(g.pair_lam);
  const double2* seeds = KS == 2 ? g.seeds2 : g.seeds1;
  pin_arg(seeds);
  pin_arg(g.Fbar);
  // as in the analysis: the loads of the prologue at once (but see kLate)
  constexpr int FI = (NFLD * (KS == 2 ? 256 : 16 * WL * GW) + NT - 1) / NT;
  const int64_t fstride = (int64_t)(N + 1) * nlat;
  const double2* Gb = g.Fbar + (int64_t)b * 4 * fstride + (int64_t)m * nlat;
  double2 qn[FI], qs[FI];
  double xn[FI];
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int t = min((int)threadIdx.x + i * NT, NFLD * nhp - 1);
    const int f = t / nhp, p = min(t - f * nhp, nh - 1);
    qn[i] = Gb[f * fstride + p];
    qs[i] = Gb[f * fstride + nlat - 1 - p];
    xn[i] = g.mu[p];
  }
  constexpr int RI = ((KS == 2 ? 340 : kMaxM / 3) / 2 + 2 + 2 * NS + NT - 1) / NT;
  double2 rcv[RI];
  double rce[RI];
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int r = threadIdx.x + i * NT;
    const int64_t k = pbase + min((r % NS) * len + r / NS, K - 1);
    rcv[i] = g.pair_rec[k];
    rce[i] = g.pair_equ[k];
  }
  double2 seed[GW];
  double x[GW], w[FW][GW];
  const int lo = (lane >> 4) + 4 * (((lane >> 2) & 3) / KS);
  const int segA = (lane & 3) + 4 * (((lane >> 2) & 3) % KS);
  auto load_seeds = [&] {
#pragma unroll
    for (int i = 0; i < GW; ++i) {
      const int p = min((wl * GW + i) * LG + lo, nh - 1);
      seed[i] = seeds[(((int64_t)m * (nhp >> 4) + (p >> 4)) * NS + segA) * 16 + (p & 15)];
      x[i] = g.mu[p];
    }
  };
  // With eight and twelve groups of latitudes the registers do not hold the folded
  // cotangents beside the seeds, nor the first degree's coefficients and history beside the
  // recurrence: 18 to 56 registers went through scratch memory. There the seeds are loaded
  // behind the fold and the coefficients behind the sums. N = 511 47.6 -> 41.4 us, N = 300 with
  // the step adjoint 26.0 -> 19.7 (order 5: 29.6 -> 21.1), without it 19.1 -> 18.5
  constexpr bool kLate = GW >= 8;
  if (!kLate) load_seeds();
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    pin(qn[i]);
    pin(qs[i]);
    pin(xn[i]);
  }
  // fold: We = G(p) + G(p'), Wo = G(p) - G(p') (the equator ring of an odd rule, its
  // own mirror, counted once); zero past the last latitude
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int t = threadIdx.x + i * NT;
    if (t < NFLD * nhp) {
      const int p = t - t / nhp * nhp;
      const double2 gs = 2 * p + 1 == nlat ? z2 : qs[i];
      double2* f = reinterpret_cast<double2*>(wf + 4 * t);
      f[0] = p < nh ? make_double2(qn[i].x + gs.x, qn[i].y + gs.y) : z2;
      f[1] = p < nh ? make_double2(xn[i] * (qn[i].x - gs.x), xn[i] * (qn[i].y - gs.y)) : z2;
    }
  }
#pragma unroll
  for (int i = 0; i < RI; ++i) {
    const int r = threadIdx.x + i * NT;
    pin(rcv[i]);
    pin(rce[i]);
    if (r < len * NS) {
      const bool in = (r % NS) * len + r / NS < K;
      PairRec<EDGE>::put(rec, len * NS, r, in ? rcv[i].x : 0.0, in ? rcv[i].y : 0.0, in ? -rce[i] : 0.0);
    }
  }
  if (kLate) load_seeds();
  __syncthreads();
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    const int p = (wl * GW + i) * LG + lo;
#pragma unroll
    for (int f = 0; f < FW; ++f)
      w[f][i] = p < nhp ? wf[((f0 + f) * nhp + p) * 4 + (lane & 3)] : 0.0;
  }
  __syncthreads();  // the folded cotangents make room for the sums
  // coefficients of the thread's first degree, in flight during the sums
  const int La = N + 1 - m;  // degrees m .. N
  const int64_t sbase = member_offset(g, b) + coeff_offset(N, m);
  double cf[6];
  double2 lm = z2, hin[kMaxStepCoef];
#pragma unroll
  for (int j = 0; j < kMaxStepCoef; ++j) hin[j] = z2;
  auto load_inputs = [&](int kk) {
    const int k = kk >> 1, kb = k > 0 ? k - 1 : 0, ka = k + 1 < K ? k + 1 : k;
    const double* c = g.pair_syn + pbase * 8;
    const bool odd = kk & 1;
    // even: mc1_k, mc2_{k-1}, b1_k, b2_{k-1}; odd: ms_k, a1_{k+1}, a2_k, a3_{k-1}
    cf[0] = c[8 * k + (odd ? 2 : 0)];
    cf[1] = c[odd ? 8 * ka + 3 : 8 * kb + 1];
    cf[2] = c[8 * k + (odd ? 4 : 6)];
    cf[3] = c[8 * kb + (odd ? 5 : 7)];
    if (odd && k + 1 >= K) cf[1] = 0.0;
    if (k == 0) {
      if (!odd) cf[1] = 0.0;
      cf[3] = 0.0;
    }
    lm = g.pair_lam[m + kk];
    if constexpr (DEP > 0) {
#pragma unroll
      for (int j = 0; j < DEP; ++j)
        hin[j] = sa.hin[(j < sa.depth ? j : 0) * sa.state_count + sbase + kk];
    }
  };
  if (!kLate && 64 * wave < La) load_inputs(min((int)threadIdx.x, La - 1));
  pair_rows<GW, KS, EDGE, FW>(seed, x, w, wl * GW * LG, lo, nh, len, rec, red + wave * FW * rows * RSUM,
                              lane);
  if (kLate && 64 * wave < La) load_inputs(min((int)threadIdx.x, La - 1));
  __syncthreads();
  const float rlen = 1.0f / (float)len;
  // sums of field f, columns (c, c + 1), row k; EDGE: from the segment of row k0
  auto sum = [&](int f, int c, int k, int k0) {
    const int2 at = pair_seg(EDGE ? k0 : k, len, rlen);
    return pair_fetch<WL, KS>(red + ((f / FW) * WL * FW + f % FW) * rows * RSUM, at.x,
                              EDGE ? at.y + 1 + k - k0 : at.y, c, FW * rows * RSUM);
  };
  for (int kk = threadIdx.x; kk < La; kk += NT) {
    if (kk >= NT) load_inputs(kk);
    const int k = kk >> 1, kb = k > 0 ? k - 1 : 0, ka = k + 1 < K ? k + 1 : k;
    // cotangent of a coefficient from its i m field fm and its derivative field fd
    auto cot = [&](int fm, int fd) {
      double2 v;
      if (kk & 1) {
        const double2 o = sum(fm, 2, k, k), e1 = sum(fd, 0, ka, k), e0 = sum(fd, 0, k, k),
                      eb = sum(fd, 0, kb, k);
        v.x = cf[0] * o.y + cf[1] * e1.x + cf[2] * e0.x + cf[3] * eb.x;
        v.y = -cf[0] * o.x + cf[1] * e1.y + cf[2] * e0.y + cf[3] * eb.y;
      } else {
        const double2 e0 = sum(fm, 0, k, k), eb = sum(fm, 0, kb, k), o0 = sum(fd, 2, k, k),
                      ob = sum(fd, 2, kb, k);
        v.x = cf[0] * e0.y + cf[1] * eb.y + cf[2] * o0.x + cf[3] * ob.x;
        v.y = -cf[0] * e0.x - cf[1] * eb.x + cf[2] * o0.y + cf[3] * ob.y;
      }
      return v;
    };
    double2 ab = cot(0, 1);
    ab = make_double2(lm.x * ab.x, lm.x * ab.y);
    if constexpr (NFLD == 4) {
      const double2 z = cot(3, 2);
      ab.x = fma(lm.y, z.x, ab.x);
      ab.y = fma(lm.y, z.y, ab.y);
    }
    if (m + kk == 0) ab.x = 0.0;
    if (m == 0) ab.y = 0.0;
    if constexpr (DEP > 0)
      step_adjoint_store(g, sa, b, m, kk, ab, hin);
    else
      alpha_bar[sbase + kk] = ab;
  }
}

template <int NFLD, int FW, int WL, int KS>
size_t adj_pair_lds(int N, int nh) {
  constexpr int W = WL * (NFLD / FW);
  const size_t len = pair_len(pair_count(N, 0), KS), rows = pair_edge<KS>() ? len + 2 : len;
  return PairRec<pair_edge<KS>()>::kRow * len * 32 * KS +
         std::max((size_t)NFLD * ((nh + 15) & ~15) * 32, rows * pair_sums<KS>() * 8 * W * FW);
}

template <int NFLD, int FW, int WL, int GW, int KS>
hipError_t launch_adj_pair_as(const GroupView& g, double2* alpha_bar, const StepAdjointArgs* sa,
                              hipStream_t s) {
  constexpr int W = WL * (NFLD / FW);
  const size_t lds = adj_pair_lds<NFLD, FW, WL, KS>(g.N, g.nh);
  const dim3 grid = pair_places(g, 0, 1), block(64 * W);
  if constexpr (NFLD == 4) {
    if (sa && sa->depth <= 3) {
      hipLaunchKernelGGL((k_adjoint_pair<NFLD, FW, WL, GW, KS, 3>), grid, block, lds, s, g,
                         alpha_bar, *sa);
      return hipGetLastError();
    }
    if (sa) {
      hipLaunchKernelGGL((k_adjoint_pair<NFLD, FW, WL, GW, KS, 6>), grid, block, lds, s, g,
                         alpha_bar, *sa);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_adjoint_pair<NFLD, FW, WL, GW, KS, 0>), grid, block, lds, s, g,
                     alpha_bar, StepAdjointArgs{});
  return hipGetLastError();
}

template <int NFLD>
hipError_t launch_adj_pair(const GroupView& g, double2* alpha_bar, const StepAdjointArgs* sa,
                           hipStream_t s) {
  // WL GW groups of 16 / ks latitudes cover the nh of the size class
  if (pair_eight(g, 0)) {
    if (g.nh <= 96) return launch_adj_pair_as<NFLD, 2, 4, 3, 2>(g, alpha_bar, sa, s);
    if (g.nh <= 192) return launch_adj_pair_as<NFLD, 2, 4, 6, 2>(g, alpha_bar, sa, s);
    return launch_adj_pair_as<NFLD, 2, 4, 8, 2>(g, alpha_bar, sa, s);
  }
  // nh >= 256: with a wave per field 46.5 us for the four fields of N = 511 against 50.5 with
  // two fields per wave, whose recurrence is shared but whose row sums are twice as many
  // (before the late loads); for two fields 27.0 against 25.5 (with the two-operation step)
  if constexpr (NFLD == 2)
    return launch_adj_pair_as<2, 2, 4, 6, 1>(g, alpha_bar, sa, s);
  else
    return launch_adj_pair_as<NFLD, 1, 2, 12, 1>(g, alpha_bar, sa, s);
}

}  // namespace

hipError_t launch_adjoint_pair(const GroupView& g, double2* alpha_bar, const StepAdjointArgs* sa,
                               bool projection, hipStream_t s) {
  return projection ? launch_adj_pair<2>(g, alpha_bar, nullptr, s)
                    : launch_adj_pair<4>(g, alpha_bar, sa, s);
}

// The most dynamic LDS that a launch for members of this truncation and grid asks for (the
// adjoint has more fields than the projection, and the five-field synthesis than the others).
size_t pair_lds_bytes(int N, int nh) {
  size_t v = synth_pair_lds<4, 8, 3, 1>(N);
  v = std::max(v, nh < 256 ? synth_pair_lds<5, 6, 2, 2>(N) : synth_pair_lds<5, 8, 3, 1>(N));
  v = std::max(v, nh <= 96 ? anal_pair_lds<1>(N) : nh <= 192 ? anal_pair_lds<3>(N) : anal_pair_lds<4>(N));
  return std::max(v, nh < 256 ? adj_pair_lds<4, 2, 4, 2>(N, nh) : adj_pair_lds<4, 1, 2, 1>(N, nh));
}

}  // namespace nse
