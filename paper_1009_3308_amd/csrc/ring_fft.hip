// Longitude transforms and the grid product (Section 4.2: FFT in the
// azimuthal direction at the M equispaced longitudes of eq. (quadrule)).
//
// Two real fields share one complex FFT: for fields a, b with Fourier coefficients
// G^a_m, G^b_m, m = 0..N, the length-M sequence
//   x_m = G^a_m + i G^b_m,  x_{M-m} = conj(G^a_m) + i conj(G^b_m)
// has the inverse DFT g^a_j + i g^b_j. The pairs are (f0, f1), the two
// components of the stream-function gradient, and (f2, f3), the two of the
// absolute-vorticity gradient, so that the advection term is the real part of
// one product:
//   q = (f0 f2 - f1 f3) / sin^2(theta) = Re[(f0 + i f1)(f2 + i f3)] / sin^2(theta)
//     = u . Grad(zeta + 2 Omega cos theta).
// A transform's rounding error is relative to the larger of its two fields;
// the vorticity gradient is larger than the stream-function gradient by about
// the degree squared for a spectrum with weight at high degree, so each
// transform holds two fields of one kind.
// A forward FFT of q gives its spectrum Q_m; the quadrature factor
// (2 pi / M) w_p of eq. (quadrule) is applied and Q_m, m = 0..N, is written for
// the ring (W[m][lat], latitude fastest); the analysis folds the two rings of
// each latitude pair.
//
// A workgroup holds one or two neighbouring rings in LDS. The transforms are
// mixed-radix and in place, decimated in frequency on the way to the grid and in
// time on the way back, the second the mirror image of the first: every butterfly
// reads and writes the same positions, so a stage needs one barrier, and the grid
// values lie in digit-reversed order, which the product does not mind. The last
// inverse stage, the product and the first forward stage work on the same R
// consecutive positions and are one pass in registers. With two rings the two real
// products go through one forward transform, q_a + i q_b.
// The plan (radices up to 16, three stages for most M, FftPlan) is chosen on the
// host for the fewest stages and then for LDS accesses without bank conflicts.
#include <algorithm>
#include <type_traits>

#include "nse_internal.h"

namespace nse {

namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// S i a for S = +-1
template <int S>
__device__ __forceinline__ double2 cmul_si(double2 a) {
  return S > 0 ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// cos/sin of 2 pi / 3, 2 pi / 5 and 4 pi / 5 in closed form:
// sqrt(3)/2, (sqrt(5)-1)/4, -(sqrt(5)+1)/4, sqrt(10+2 sqrt(5))/4, sqrt(10-2 sqrt(5))/4;
// of pi / 4, pi / 8 and 2 pi / 9, 4 pi / 9, 8 pi / 9.
constexpr double kS3 = 0.86602540378443864676;
constexpr double kC1 = 0.30901699437494742410;
constexpr double kC2 = -0.80901699437494742410;
constexpr double kS1 = 0.95105651629515357212;
constexpr double kS2 = 0.58778525229247312917;
constexpr double kH = 0.70710678118654752440;
constexpr double kC16 = 0.92387953251128675613, kS16 = 0.38268343236508977173;
constexpr double kC9a = 0.76604444311897803520, kS9a = 0.64278760968653932632;
constexpr double kC9b = 0.17364817766693034885, kS9b = 0.98480775301220805937;
constexpr double kC9d = -0.93969262078590838405, kS9d = 0.34202014332566873304;

constexpr int inverse_mod(int a, int m) {
  for (int x = 1; x < m; ++x)
    if (a * x % m == 1) return x;
  return 0;
}

// DFT of length R with kernel exp(S 2 pi i j k / R), in place.
template <int R, int S>
__device__ __forceinline__ void butterfly(double2* v);

// R = A B, A and B coprime (prime-factor map: no twiddles in between).
template <int A, int B, int S>
__device__ __forceinline__ void butterfly_coprime(double2* v) {
  constexpr int R = A * B, ia = B * inverse_mod(B % A, A), ib = A * inverse_mod(A % B, B);
  double2 w[A][B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    double2 t[A];
#pragma unroll
    for (int a = 0; a < A; ++a) t[a] = v[(B * a + A * b) % R];
    butterfly<A, S>(t);
#pragma unroll
    for (int a = 0; a < A; ++a) w[a][b] = t[a];
  }
#pragma unroll
  for (int a = 0; a < A; ++a) {
    butterfly<B, S>(w[a]);
#pragma unroll
    for (int b = 0; b < B; ++b) v[(ia * a + ib * b) % R] = w[a][b];
  }
}

template <int R, int S>
__device__ __forceinline__ void butterfly(double2* v) {
  if constexpr (R == 2) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 3) {
    const double2 t = cadd(v[1], v[2]);
    const double2 u = csub(v[1], v[2]);
    const double2 d = cmul_si<S>(make_double2(kS3 * u.x, kS3 * u.y));
    const double2 c = make_double2(v[0].x - 0.5 * t.x, v[0].y - 0.5 * t.y);
    v[0] = cadd(v[0], t);
    v[1] = cadd(c, d);
    v[2] = csub(c, d);
  } else if constexpr (R == 4) {
    const double2 a0 = cadd(v[0], v[2]), a1 = csub(v[0], v[2]);
    const double2 b0 = cadd(v[1], v[3]), b1 = cmul_si<S>(csub(v[1], v[3]));
    v[0] = cadd(a0, b0);
    v[2] = csub(a0, b0);
    v[1] = cadd(a1, b1);
    v[3] = csub(a1, b1);
  } else if constexpr (R == 5) {
    const double2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]);
    const double2 d1 = csub(v[1], v[4]), d2 = csub(v[2], v[3]);
    const double2 x0 = v[0];
    const double2 c1 = make_double2(x0.x + kC1 * t1.x + kC2 * t2.x, x0.y + kC1 * t1.y + kC2 * t2.y);
    const double2 c2 = make_double2(x0.x + kC2 * t1.x + kC1 * t2.x, x0.y + kC2 * t1.y + kC1 * t2.y);
    const double2 s1 = cmul_si<S>(make_double2(kS1 * d1.x + kS2 * d2.x, kS1 * d1.y + kS2 * d2.y));
    const double2 s2 = cmul_si<S>(make_double2(kS2 * d1.x - kS1 * d2.x, kS2 * d1.y - kS1 * d2.y));
    v[0] = cadd(x0, cadd(t1, t2));
    v[1] = cadd(c1, s1);
    v[4] = csub(c1, s1);
    v[2] = cadd(c2, s2);
    v[3] = csub(c2, s2);
  } else if constexpr (R == 6) {
    butterfly_coprime<2, 3, S>(v);
  } else if constexpr (R == 8) {
    // radix 8 from two radix-4 transforms of the even and odd samples
    double2 e[4] = {v[0], v[2], v[4], v[6]};
    double2 o[4] = {v[1], v[3], v[5], v[7]};
    butterfly<4, S>(e);
    butterfly<4, S>(o);
    const double2 o1 = make_double2(kH * (o[1].x - S * o[1].y), kH * (o[1].y + S * o[1].x));
    const double2 o2 = cmul_si<S>(o[2]);
    const double2 o3 = make_double2(kH * (-o[3].x - S * o[3].y), kH * (-o[3].y + S * o[3].x));
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
  } else if constexpr (R == 9) {
    // n = 3 n1 + n2, k = k1 + 3 k2, twiddles exp(S 2 pi i n2 k1 / 9)
    double2 w[3][3];  // [n2][k1]
#pragma unroll
    for (int n2 = 0; n2 < 3; ++n2) {
      double2 t[3] = {v[n2], v[3 + n2], v[6 + n2]};
      butterfly<3, S>(t);
#pragma unroll
      for (int k = 0; k < 3; ++k) w[n2][k] = t[k];
    }
    w[1][1] = cmul(w[1][1], make_double2(kC9a, S * kS9a));
    w[1][2] = cmul(w[1][2], make_double2(kC9b, S * kS9b));
    w[2][1] = cmul(w[2][1], make_double2(kC9b, S * kS9b));
    w[2][2] = cmul(w[2][2], make_double2(kC9d, S * kS9d));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double2 t[3] = {w[0][k], w[1][k], w[2][k]};
      butterfly<3, S>(t);
#pragma unroll
      for (int k2 = 0; k2 < 3; ++k2) v[k + 3 * k2] = t[k2];
    }
  } else if constexpr (R == 10) {
    butterfly_coprime<2, 5, S>(v);
  } else if constexpr (R == 12) {
    butterfly_coprime<4, 3, S>(v);
  } else if constexpr (R == 15) {
    butterfly_coprime<3, 5, S>(v);
  } else {
    static_assert(R == 16, "radices of FftPlan");
    // n = 4 n1 + n2, k = k1 + 4 k2, twiddles exp(S 2 pi i n2 k1 / 16)
    double2 w[4][4];  // [n2][k1]
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
      double2 t[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
      butterfly<4, S>(t);
#pragma unroll
      for (int k = 0; k < 4; ++k) w[n2][k] = t[k];
    }
    auto eighth = [](double2 a) { return make_double2(kH * (a.x - S * a.y), kH * (a.y + S * a.x)); };
    w[1][1] = cmul(w[1][1], make_double2(kC16, S * kS16));
    w[1][2] = eighth(w[1][2]);
    w[1][3] = cmul(w[1][3], make_double2(kS16, S * kC16));
    w[2][1] = eighth(w[2][1]);
    w[2][2] = cmul_si<S>(w[2][2]);
    w[2][3] = cmul_si<S>(eighth(w[2][3]));
    w[3][1] = cmul(w[3][1], make_double2(kS16, S * kC16));
    w[3][2] = cmul_si<S>(eighth(w[3][2]));
    w[3][3] = cmul(w[3][3], make_double2(-kC16, -S * kS16));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      double2 t[4] = {w[0][k], w[1][k], w[2][k], w[3][k]};
      butterfly<4, S>(t);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) v[k + 4 * k2] = t[k2];
    }
  }
}

// t / d for t d < 2^21, magic = 2^21 / d + 1
__device__ __forceinline__ int quot(int t, unsigned magic) { return (int)(((unsigned)t * magic) >> 21); }
// LDS slot of position i: pad0 free slots after every J[0] positions, pad1 after every J[1].
__device__ __forceinline__ int slot(const FftPlan& pl, int i) {
  int s = i + pl.pad0 * quot(i, pl.mj[0]);
  if (pl.pad1) s += pl.pad1 * quot(i, pl.mj[1]);
  return s;
}
// Slots between the positions i and i + J[st] of one block.
__device__ __forceinline__ int slot_stride(const FftPlan& pl, int st) {
  return pl.J[st] + (st == 0 ? pl.pad0 + pl.pad1 * pl.radix[1] : st == 1 ? pl.pad1 : 0);
}

// Powers w^r, w = exp(S 2 pi i e / M), r = 1 .. R-1, e R < M, times v[r]: w, w^2 and w^4
// are read from the table tw[k] = exp(-2 pi i k / M), the others are products of at
// most four of these.
template <int R, int S>
struct Twiddle {
  double2 w1, w2, w4;
  __device__ __forceinline__ Twiddle(const double2* tw, int e) {
    w1 = tw[e];
    w2 = R > 2 ? tw[2 * e] : w1;
    w4 = R > 4 ? tw[4 * e] : w1;
    if (S > 0) {
      w1.y = -w1.y;
      w2.y = -w2.y;
      w4.y = -w4.y;
    }
  }
  __device__ __forceinline__ void apply(double2* v) const {
    v[1] = cmul(v[1], w1);
    if constexpr (R > 2) v[2] = cmul(v[2], w2);
    double2 w3 = w1, wb = w4;
    if constexpr (R > 3) {
      w3 = cmul(w1, w2);
      v[3] = cmul(v[3], w3);
    }
#pragma unroll
    for (int r = 4; r < R; r += 4) {
      v[r] = cmul(v[r], wb);
      if (r + 1 < R) v[r + 1] = cmul(v[r + 1], cmul(wb, w1));
      if (r + 2 < R) v[r + 2] = cmul(v[r + 2], cmul(wb, w2));
      if (r + 3 < R) v[r + 3] = cmul(v[r + 3], cmul(wb, w3));
      if (r + 4 < R) wb = cmul(wb, w4);
    }
  }
};

// One stage of radix R over na arrays of stride PL, in place: the butterfly of block b,
// offset j works on the positions b L + j + r J, L = R J; decimation in frequency
// (S = 1, inverse: twiddles after the butterfly) or in time (S = -1: before).
template <int R, int S, int NT>
__device__ __forceinline__ void stage(double2* x, int na, int PL, const FftPlan& pl, int st,
                                      const double2* tw) {
  const int J = pl.J[st], per = pl.per[st], step = pl.step[st], d = slot_stride(pl, st);
  for (int t = threadIdx.x; t < na * per; t += NT) {
    const int a = na > 1 ? quot(t, pl.mper[st]) : 0, u = t - a * per;
    const int b = quot(u, pl.mj[st]), j = u - b * J;
    double2* y = x + (a * PL + slot(pl, b * J * R + j));
    const Twiddle<R, S> w(tw, j * step);  // (the last stage, J = 1, does not come here)
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = y[r * d];
    if (S < 0) w.apply(v);
    butterfly<R, S>(v);
    if (S > 0) w.apply(v);
#pragma unroll
    for (int r = 0; r < R; ++r) y[r * d] = v[r];
  }
}

// Compile-time plans of the default grids of N = 2^k - 1, M = 3 * 2^k, and of N = 100, M =
// 320 (160 rings 5.0 us, 6.9 at run time; any other M: the one that
// fft_plan found, a kernel argument). With every index a constant the ring takes 21.3
// us instead of 24.4 at M = 1536 (768 rings), 53 instead of 64 us at M = 768 (6144 rings; both
// before the four fields of an order lay together, as the figures below).
// Measured against these plans: 12, 16, 8 and 16, 12, 8 at M = 1536 22.8 us (their
// last pass needs more registers); 8, 8, 8, 3 over 384 threads 22.8; 16, 16, 3 at M =
// 768 8.8 against 8.2 us for 384 rings; 4, 16, 3 at M = 192 10.5 against 9.8 us for 2304.
template <int CM>
__host__ __device__ __forceinline__ FftPlan plan_of(const FftPlan& rt) {
  if constexpr (CM == 1536) return make_plan(CM, {16, 16, 6}, 3, 6, 0);
  else if constexpr (CM == 768) return make_plan(CM, {8, 16, 6}, 3, 6, 0);
  else if constexpr (CM == 384) return make_plan(CM, {8, 16, 3}, 3, 3, 0);
  else if constexpr (CM == 320) return make_plan(CM, {8, 8, 5}, 3, 0, 0);
  else if constexpr (CM == 192) return make_plan(CM, {8, 8, 3}, 3, 3, 0);
  else if constexpr (CM == 96) return make_plan(CM, {4, 4, 6}, 3, 0, 0);
  else if constexpr (CM == 48) return make_plan(CM, {2, 4, 6}, 3, 0, 0);
  else return rt;
}
// Calls f(integral_constant<R>) for the plan's radix.
template <typename F>
__device__ __forceinline__ void with_radix(int R, F&& f) {
  switch (R) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 12: f(std::integral_constant<int, 12>{}); break;
    case 15: f(std::integral_constant<int, 15>{}); break;
    default: f(std::integral_constant<int, 16>{}); break;
  }
}
// The same for the last stage's radix (at most kMaxLastRadix: its pass holds the
// butterflies of two or three arrays at once).
template <typename F>
__device__ __forceinline__ void with_last_radix(int R, F&& f) {
  switch (R) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    default: f(std::integral_constant<int, 6>{}); break;
  }
}
template <int S, int NT>
__device__ __forceinline__ void run_stage(double2* x, int na, int PL, const FftPlan& pl, int st,
                                          const double2* tw) {
  with_radix(pl.radix[st], [&](auto r) { stage<decltype(r)::value, S, NT>(x, na, PL, pl, st, tw); });
}
// The last stage alone (J = 1: no twiddles).
template <int S, int NT>
__device__ __forceinline__ void run_last(double2* x, int na, int PL, const FftPlan& pl) {
  const int last = pl.nstages - 1, per = pl.per[last];
  with_last_radix(pl.radix[last], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    for (int t = threadIdx.x; t < na * per; t += NT) {
      const int a = na > 1 ? quot(t, pl.mper[last]) : 0;
      double2* y = x + (a * PL + slot(pl, (t - a * per) * R));
      double2 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = y[r];
      butterfly<R, S>(v);
#pragma unroll
      for (int r = 0; r < R; ++r) y[r] = v[r];
    }
  });
  __syncthreads();
}
// f(st) for the stages before the last one, a barrier after each: in rising order
// (S = 1) or falling (S = -1); unrolled for a compile-time plan.
template <int S, bool CT, typename F>
__device__ __forceinline__ void for_stages(const FftPlan& pl, F&& f) {
  const int last = pl.nstages - 1;
  if constexpr (CT) {
#pragma unroll
    for (int i = 0; i < kMaxStages - 1; ++i) {
      const int st = S > 0 ? i : kMaxStages - 2 - i;
      if (st < last) {
        f(st);
        __syncthreads();
      }
    }
  } else {
#pragma unroll 1
    for (int i = 0; i < last; ++i) {
      f(S > 0 ? i : last - 1 - i);
      __syncthreads();
    }
  }
}
// Slot of grid point n in the order that the inverse stages leave.
__device__ __forceinline__ int grid_slot(const FftPlan& pl, int n) {
  int pos = 0;
  for (int s = 0; s < pl.nstages; ++s) {
    const int d = quot(n, pl.mr[s]);
    pos += (n - d * pl.radix[s]) * slot_stride(pl, s);
    n = d;
  }
  return pos;
}

// Northern node of ring `lat`.
__device__ __forceinline__ int ring_node(const GroupView& g, int lat) {
  return lat < g.nh ? lat : g.nlat - 1 - lat;
}

// LDS slots from one array to the next: congruent to 8 (4 for two rings) modulo 16, so that
// lanes that write the same order of the arrays hit different banks.
template <int NR>
__host__ __device__ __forceinline__ int array_len(const FftPlan& pl) {
  constexpr int c = NR == 2 ? 4 : 8;
  return (pl.len + 15 - c) / 16 * 16 + c;
}

// Spectra of NR neighbouring rings into LDS: array (ring rr, pair a) at x + (rr NP + a)
// PL holds x_m = G^a_m + i G^b_m and x_{M-m} = conj(G^a_m) + i conj(G^b_m), zero in
// between. Pairs 0 and 1 are the fields (0, 1) and (2, 3) of F[m][lat][4] (REAL1: the
// real field 2 twice); the third of NP = 3 pairs is the real field of spectrum F5 / 2,
// F5[m][lat]. All loads are issued, unconditionally, before the first LDS write; two
// lanes read the 64 bytes of an order, four those of two rings. (With the fields in
// planes of their own every lane took a cache line by itself: the ring at M = 1536
// needed 21.4 us instead of 17.5.)
template <int NP, int NR, int MAXM, int NT, bool REAL1>
__device__ __forceinline__ void load_spectra(double2* x, int PL, const FftPlan& pl, int N, int M,
                                             int nlat, int lat0, const double2* F,
                                             const double2* F5) {
  constexpr int kOrders = (MAXM + 1) / 3;  // N + 1 <= (M + 1) / 3
  constexpr int KI = (NR * 2 * kOrders + NT - 1) / NT;
  constexpr int KR = NP == 3 ? (NR * kOrders + NT - 1) / NT : 0;
  double2 ga[KI], gb[KI], gr[KR + 1];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int t = threadIdx.x + i * NT, a = t & 1, rr = (t >> 1) % NR, m = min((t >> 1) / NR, N);
    const double2* f = F + ((int64_t)m * nlat + min(lat0 + rr, nlat - 1)) * 4 + 2 * a;
    ga[i] = f[0];
    gb[i] = f[REAL1 && a ? 0 : 1];
  }
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    const int t = threadIdx.x + i * NT, rr = t % NR, m = min(t / NR, N);
    gr[i] = F5[(int64_t)m * nlat + min(lat0 + rr, nlat - 1)];
  }
  auto put = [&](double2* y, int m, double2 a, double2 b) {
    if (m > N) return;
    if (m == 0) {
      y[0] = make_double2(a.x, b.x);
    } else {
      y[slot(pl, m)] = make_double2(a.x - b.y, a.y + b.x);
      y[slot(pl, M - m)] = make_double2(a.x + b.y, b.x - a.y);
    }
  };
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int t = threadIdx.x + i * NT, a = t & 1, rr = (t >> 1) % NR;
    put(x + (rr * NP + a) * PL, (t >> 1) / NR, ga[i], gb[i]);
  }
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    const int t = threadIdx.x + i * NT, rr = t % NR, m = t / NR;
    const double h = m == 0 ? 1.0 : 0.5;
    put(x + (rr * NP + 2) * PL, m, make_double2(h * gr[i].x, h * gr[i].y), make_double2(0.0, 0.0));
  }
  const int zb = M - 2 * N - 1;  // N < k < M - N
  for (int a = 0; a < NR * NP; ++a)
    for (int t = threadIdx.x; t < zb; t += NT) x[a * PL + slot(pl, N + 1 + t)] = make_double2(0.0, 0.0);
}

// Nonlinear mode: NR rings per workgroup.
// Bound: at M = 1536 (768 rings, three per CU, 31 MB of spectra in and out) 17.3 us, of
// which about 6 are the FP64 instructions, 5 the LDS and 4 the reads of the spectra; the
// rings of a CU run in step, so these add up. Stockham rings with radices 8, 8, 8, 3 took
// 22.8 us; 68 us became 50 for 6144 rings of M = 768 and 37 became 23 for 4608 of M = 384,
// by fewer LDS passes without bank conflicts and one forward transform for two rings;
// 17.5 became 11.3 for 480 rings of M = 960 (run-time plan).
template <int MAXM, int NT, int NR, int CM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_ring(GroupView g, FftPlan rt) {
  const FftPlan pl = plan_of<CM>(rt);
  const int N = g.N, M = CM ? CM : g.M, nlat = CM ? CM / 2 : g.nlat;
  const int lat0 = NR * xcd_item(blockIdx.x, 8 / NR);  // XCD chunks of 8 rings share lines of F
  if (lat0 >= nlat) return;
  const int b = blockIdx.y;
  const int PL = array_len<NR>(pl);
  extern __shared__ double2 lds[];
  const double2* tw = g.tw;
  const int64_t fstride = (int64_t)(N + 1) * nlat;
  const double2* F0 = g.F + (int64_t)b * 4 * fstride;
  double inv_sin2[NR], c[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int lat = min(lat0 + r, nlat - 1), p = ring_node(g, lat);
    const double x = g.mu[p];
    inv_sin2[r] = 1.0 / ((1.0 - x) * (1.0 + x));
    // quadrature factor (2 pi / M) w_p; the equator ring of an odd rule is its
    // own mirror and is folded twice by the analysis
    c[r] = (6.283185307179586477 / M) * g.w[p] * (2 * p + 1 == nlat ? 0.5 : 1.0);
  }
  load_spectra<2, NR, MAXM, NT, false>(lds, PL, pl, N, M, nlat, lat0, F0, nullptr);
  // an ended attempt of a device-controlled run: checked once the loads are in
  // flight (nothing is stored before this barrier), so the flag costs no wait
  if (gate_closed(g)) return;
  __syncthreads();
  const int last = pl.nstages - 1;
  for_stages<1, (CM > 0)>(pl, [&](int st) { run_stage<1, NT>(lds, 2 * NR, PL, pl, st, tw); });
  with_last_radix(pl.radix[last], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    for (int u = threadIdx.x; u < pl.per[last]; u += NT) {
      const int s0 = slot(pl, u * R);
      double2 z[R];
#pragma unroll
      for (int rr = 0; rr < NR; ++rr) {
        double2 v0[R], v1[R];
        const double2* y = lds + (2 * rr * PL + s0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          v0[r] = y[r];
          v1[r] = y[PL + r];
        }
        butterfly<R, 1>(v0);
        butterfly<R, 1>(v1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double q = (v0[r].x * v1[r].x - v0[r].y * v1[r].y) * inv_sin2[rr];
          if (rr == 0)
            z[r] = make_double2(q, 0.0);
          else
            z[r].y = q;
        }
      }
      butterfly<R, -1>(z);
#pragma unroll
      for (int r = 0; r < R; ++r) lds[s0 + r] = z[r];
    }
  });
  __syncthreads();
  for_stages<-1, (CM > 0)>(pl, [&](int st) { run_stage<-1, NT>(lds, 1, PL, pl, st, tw); });
  double2* Wl = g.W + (int64_t)b * (N + 1) * nlat + lat0;  // W[b][m][lat]
  if constexpr (NR == 1) {
    for (int m = threadIdx.x; m <= N; m += NT) {
      const double2 z = lds[slot(pl, m)];
      Wl[(int64_t)m * nlat] = make_double2(c[0] * z.x, c[0] * z.y);
    }
  } else {
    // the two real sequences of one transform: A = (Z_m + conj Z_{M-m}) / 2,
    // B = (Z_m - conj Z_{M-m}) / (2 i)
    for (int t = threadIdx.x; t < 2 * (N + 1); t += NT) {
      const int m = t >> 1, rr = t & 1;
      const double2 zm = lds[slot(pl, m)], zc = lds[slot(pl, m ? M - m : 0)];
      const double h = 0.5 * (rr ? c[1] : c[0]);
      if (lat0 + rr < nlat)
        Wl[(int64_t)m * nlat + rr] = rr ? make_double2(h * (zm.y + zc.y), -h * (zm.x - zc.x))
                                       : make_double2(h * (zm.x + zc.x), h * (zm.y - zc.y));
    }
  }
}

// Grid mode: u_theta = f0 / sin, u_phi = -f1 / sin and the third field (f2). 625 rings of
// M = 1250: 34.8 -> 17.6 us.
template <int MAXM, int NT, int CM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_grid(GroupView g, FftPlan rt, double* grid_out) {
  const FftPlan pl = plan_of<CM>(rt);
  const int N = g.N, M = CM ? CM : g.M, nlat = CM ? CM / 2 : g.nlat;
  const int lat = xcd_item(blockIdx.x, 8);
  if (lat >= nlat) return;
  const int PL = array_len<1>(pl);
  extern __shared__ double2 lds[];
  const int64_t fstride = (int64_t)(N + 1) * nlat;
  const double x = g.mu[ring_node(g, lat)];
  const double rs = 1.0 / sqrt((1.0 - x) * (1.0 + x));
  load_spectra<2, 1, MAXM, NT, true>(lds, PL, pl, N, M, nlat, lat, g.F, nullptr);
  __syncthreads();
  for_stages<1, (CM > 0)>(pl, [&](int st) { run_stage<1, NT>(lds, 2, PL, pl, st, g.tw); });
  run_last<1, NT>(lds, 2, PL, pl);
  double* g0 = grid_out + (int64_t)lat * M;
  const int64_t gs = (int64_t)nlat * M;
  for (int j = threadIdx.x; j < M; j += NT) {
    const int p = grid_slot(pl, j);
    const double2 v0 = lds[p], v1 = lds[PL + p];
    g0[j] = rs * v0.x;
    g0[gs + j] = -rs * v0.y;
    g0[2 * gs + j] = v1.x;
  }
}

// Adjoint of the ring kernel (vector-Jacobian product on the real grid
// values): given the cotangent of the ring spectra Q (the fifth field of Fa,
// produced by the adjoint of the analysis), recompute the four forward grid
// fields of the ring, form
//   qbar_j = c_lat Re(Qbar_0 + sum_{m>=1} Qbar_m e^{i m phi_j})   (weighted r2c)^T
//   gbar0 = qbar g2 / s^2, gbar2 = qbar g0 / s^2, gbar1 = -qbar g3 / s^2, gbar3 = -qbar g1 / s^2
// and the cotangents of the field spectra (the c2r of the synthesis)^T:
//   Gbar_0 = sum_j gbar_j,  Gbar_m = 2 sum_j gbar_j e^{-i m phi_j}  (m >= 1),
// written to Fbar[b][f][m][lat]. c_lat = (2 pi / M) w_p. Three inverse transforms per
// ring, one pass for the cotangents (gbar0 + i gbar1, both of the vorticity-gradient
// size, and gbar2 + i gbar3), two forward transforms: 59 -> 32 us for 768 rings of M = 1536
// (384 threads against 256: 38 and 40.5 before the fields of an order lay together), 14.3 ->
// 13.7 us for 384 of M = 768.
template <int MAXM, int NT, int NR, int CM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_adj(GroupView g, FftPlan rt) {
  const FftPlan pl = plan_of<CM>(rt);
  const int N = g.N, M = CM ? CM : g.M, nlat = CM ? CM / 2 : g.nlat;
  const int lat0 = NR * xcd_item(blockIdx.x, 8 / NR);
  if (lat0 >= nlat) return;
  const int b = blockIdx.y;
  const int PL = array_len<NR>(pl);
  extern __shared__ double2 lds[];
  const double2* tw = g.tw;
  const int64_t fstride = (int64_t)(N + 1) * nlat;
  const double2* F5 = g.Fa + (int64_t)b * 5 * fstride;
  double cs[NR];  // c_lat / s^2
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int p = ring_node(g, min(lat0 + r, nlat - 1));
    const double x = g.mu[p];
    cs[r] = (6.283185307179586477 / M) * g.w[p] / ((1.0 - x) * (1.0 + x));
  }
  load_spectra<3, NR, MAXM, NT, false>(lds, PL, pl, N, M, nlat, lat0, F5, F5 + 4 * fstride);
  __syncthreads();
  const int last = pl.nstages - 1;
  for_stages<1, (CM > 0)>(pl, [&](int st) { run_stage<1, NT>(lds, 3 * NR, PL, pl, st, tw); });
  // (the cotangents take the first two of the ring's arrays)
  with_last_radix(pl.radix[last], [&](auto rc) {
    constexpr int R = decltype(rc)::value;
    const int per = pl.per[last];
    for (int t = threadIdx.x; t < NR * per; t += NT) {
      const int rr = NR == 1 || t < per ? 0 : 1, u = t - rr * per;
      double2* y = lds + (3 * rr * PL + slot(pl, u * R));
      double2 v0[R], v1[R], v2[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v0[r] = y[r];
        v1[r] = y[PL + r];
        v2[r] = y[2 * PL + r];
      }
      butterfly<R, 1>(v0);
      butterfly<R, 1>(v1);
      butterfly<R, 1>(v2);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double qb = (NR == 1 || rr == 0 ? cs[0] : cs[NR - 1]) * v2[r].x;
        const double2 z0 = make_double2(qb * v1[r].x, -qb * v1[r].y);
        v1[r] = make_double2(qb * v0[r].x, -qb * v0[r].y);
        v0[r] = z0;
      }
      butterfly<R, -1>(v0);
      butterfly<R, -1>(v1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        y[r] = v0[r];
        y[PL + r] = v1[r];
      }
    }
  });
  __syncthreads();
  for_stages<-1, (CM > 0)>(pl, [&](int st) {
#pragma unroll
    for (int rr = 0; rr < NR; ++rr) run_stage<-1, NT>(lds + 3 * rr * PL, 2, PL, pl, st, tw);
  });
  // unpack two real transforms per array: z = a + i b ->
  // A_m = (Z_m + conj Z_{M-m}) / 2, B_m = (Z_m - conj Z_{M-m}) / (2 i); times 2 for m >= 1
  double2* Fb = g.Fbar + (int64_t)b * 4 * fstride + lat0;  // Fbar[b][f][m][lat]
  for (int t = threadIdx.x; t < NR * (N + 1); t += NT) {
    const int m = t / NR, rr = t % NR;
    if (lat0 + rr >= nlat) continue;
    const double sc = (m == 0) ? 0.5 : 1.0;
    const int pm = slot(pl, m), pc = slot(pl, m ? M - m : 0);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double2 zm = lds[(3 * rr + a) * PL + pm], zc = lds[(3 * rr + a) * PL + pc];
      double2* out = Fb + (int64_t)(2 * a) * fstride + (int64_t)m * nlat + rr;
      out[0] = make_double2(sc * (zm.x + zc.x), sc * (zm.y - zc.y));
      out[fstride] = make_double2(sc * (zm.y + zc.y), -sc * (zm.x - zc.x));
    }
  }
}

// Longitude part of the projection (u, Z[l,m])_M of a grid velocity field:
// per ring, the real transforms Ut_m = sum_j u_theta e^{-i m phi_j} and
// Up_m = sum_j u_phi e^{-i m phi_j} (one complex FFT of u_theta + i u_phi),
// scaled by c = (2 pi / M) w_p / sin(theta_p) and written to
// Fbar[b][f][m][lat] as f = 0, 1: c Ut, -c Up. The latitude sums and the degree
// coupling of d/dtheta are done by the unweighted analysis and the prologue
// transpose, since conj(Z[l,m]) = lambda^(-1/2) (-i m Pbar / sin, -dPbar/dtheta) e^{-i m phi}
// and sin(theta) dPbar/dtheta couples degrees l - 1 and l + 1. 768 rings of M = 1536:
// 20.6 -> 13.3 us.
template <int MAXM, int NT, int CM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_ring_project(GroupView g, FftPlan rt,
                                                     const double* __restrict__ u_grid) {
  const FftPlan pl = plan_of<CM>(rt);
  const int N = g.N, M = CM ? CM : g.M, nlat = CM ? CM / 2 : g.nlat;
  const int lat = xcd_item(blockIdx.x, 8);
  if (lat >= nlat) return;
  const int b = blockIdx.y;
  const int p = ring_node(g, lat);
  extern __shared__ double2 lds[];
  const double* ut = u_grid + ((int64_t)(2 * b) * nlat + lat) * M;
  const double* up = ut + (int64_t)nlat * M;
  constexpr int KI = (MAXM + NT - 1) / NT;
  double2 u[KI];
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int j = min((int)threadIdx.x + i * NT, M - 1);
    u[i] = make_double2(ut[j], up[j]);
  }
#pragma unroll
  for (int i = 0; i < KI; ++i) {
    const int j = threadIdx.x + i * NT;
    if (j < M) lds[grid_slot(pl, j)] = u[i];
  }
  __syncthreads();
  run_last<-1, NT>(lds, 1, 0, pl);
  for_stages<-1, (CM > 0)>(pl, [&](int st) { run_stage<-1, NT>(lds, 1, 0, pl, st, g.tw); });
  const double x = g.mu[p];
  const double h = 0.5 * (6.283185307179586477 / M) * g.w[p] / sqrt((1.0 - x) * (1.0 + x));
  const int64_t fstride = (int64_t)(N + 1) * nlat;
  double2* Fb = g.Fbar + (int64_t)b * 4 * fstride + lat;  // Fbar[b][f][m][lat]
  for (int m = threadIdx.x; m <= N; m += NT) {
    const double2 zm = lds[slot(pl, m)], zc = lds[slot(pl, m ? M - m : 0)];
    Fb[(int64_t)m * nlat] = make_double2(h * (zm.x + zc.x), h * (zm.y - zc.y));
    Fb[fstride + (int64_t)m * nlat] = make_double2(-h * (zm.y + zc.y), h * (zm.x - zc.x));
  }
}

// Calls launch(MAXM, NT, CM) (as integral constants) for M: a compile-time plan if there
// is one, else the size class.
template <typename F>
hipError_t ring_dispatch(int M, F&& launch) {
  using std::integral_constant;
  switch (M) {
    case 48: return launch(integral_constant<int, 48>{}, integral_constant<int, 64>{}, integral_constant<int, 48>{});
    case 96: return launch(integral_constant<int, 96>{}, integral_constant<int, 64>{}, integral_constant<int, 96>{});
    case 192: return launch(integral_constant<int, 192>{}, integral_constant<int, 64>{}, integral_constant<int, 192>{});
    case 320: return launch(integral_constant<int, 384>{}, integral_constant<int, 128>{}, integral_constant<int, 320>{});
    case 384: return launch(integral_constant<int, 384>{}, integral_constant<int, 128>{}, integral_constant<int, 384>{});
    case 768: return launch(integral_constant<int, 768>{}, integral_constant<int, 256>{}, integral_constant<int, 768>{});
    case 1536: return launch(integral_constant<int, 1536>{}, integral_constant<int, 256>{}, integral_constant<int, 1536>{});
    default: break;
  }
  const integral_constant<int, 0> rt;
  if (M <= 192) return launch(integral_constant<int, 192>{}, integral_constant<int, 64>{}, rt);
  if (M <= 384) return launch(integral_constant<int, 384>{}, integral_constant<int, 128>{}, rt);
  if (M <= 768) return launch(integral_constant<int, 768>{}, integral_constant<int, 256>{}, rt);
  if (M <= 1024) return launch(integral_constant<int, 1024>{}, integral_constant<int, 256>{}, rt);
  return launch(integral_constant<int, kMaxM>{}, integral_constant<int, 256>{}, rt);
}

// LDS of na arrays, NR rings per workgroup.
template <int NR>
size_t ring_lds(const FftPlan& pl, int na) { return sizeof(double2) * (size_t)na * array_len<NR>(pl); }

}  // namespace

// Two rings per workgroup (M <= 1024, adjoint M <= 768: their LDS is at most 79 KB) when
// there are more rings than CUs: neighbouring rings share cache lines of the spectra, and one forward transform
// serves both. With run-time plans M = 768, 6144 rings: 64 us against 81 with one ring per
// workgroup; 384 rings: 10.9 against 12.6; M = 192, 2304 rings: 13.4 against 16.2; M = 960,
// 480 rings: 11.3 against 12.6. Up to 256 rings half of the CUs would idle; above M = 1024 a
// member alone has more than 256 pairs of rings, of which a CU holds one.
inline bool two_rings(const GroupView& g) { return (int64_t)g.nlat * g.nb > 256; }

// The most dynamic LDS that a ring kernel of this plan asks for.
size_t ring_lds_bytes(int M, const FftPlan& pl) {
  size_t v = 0;
  (void)ring_dispatch(M, [&](auto maxm, auto, auto cm) {
    constexpr int MAXM = decltype(maxm)::value, CM = decltype(cm)::value;
    const FftPlan p = plan_of<CM>(pl);
    v = ring_lds<1>(p, 3);
    if (MAXM <= 1024) v = std::max(v, ring_lds<2>(p, 4));
    if (MAXM <= 768) v = std::max(v, ring_lds<2>(p, 6));
    return hipSuccess;
  });
  return v;
}

hipError_t launch_ring_adjoint(const GroupView& g, const FftPlan& pl, hipStream_t s) {
  return ring_dispatch(g.M, [&](auto maxm, auto nt, auto cm) {
    constexpr int MAXM = decltype(maxm)::value, NT = decltype(nt)::value, CM = decltype(cm)::value;
    if constexpr (MAXM <= 768) {
      if (two_rings(g)) {
        dim3 grid(xcd_grid((g.nlat + 1) / 2, 4), g.nb);
        hipLaunchKernelGGL((k_ring_adj<MAXM, 2 * NT, 2, CM>), grid, dim3(2 * NT), ring_lds<2>(plan_of<CM>(pl), 6), s, g, pl);
        return hipGetLastError();
      }
    }
    dim3 grid(xcd_grid(g.nlat, 8), g.nb);
    constexpr int NT1 = MAXM > 768 ? 384 : NT;
    hipLaunchKernelGGL((k_ring_adj<MAXM, NT1, 1, CM>), grid, dim3(NT1), ring_lds<1>(plan_of<CM>(pl), 3), s, g, pl);
    return hipGetLastError();
  });
}

hipError_t launch_ring_project(const GroupView& g, const FftPlan& pl, const double* u_grid,
                               hipStream_t s) {
  dim3 grid(xcd_grid(g.nlat, 8), g.nb);
  return ring_dispatch(g.M, [&](auto maxm, auto nt, auto cm) {
    constexpr int MAXM = decltype(maxm)::value, NT = decltype(nt)::value, CM = decltype(cm)::value;
    hipLaunchKernelGGL((k_ring_project<MAXM, NT, CM>), grid, dim3(NT), ring_lds<1>(plan_of<CM>(pl), 1), s, g, pl, u_grid);
    return hipGetLastError();
  });
}

hipError_t launch_ring(const GroupView& g, const FftPlan& pl, int mode, double* grid_out,
                       hipStream_t s) {
  return ring_dispatch(g.M, [&](auto maxm, auto nt, auto cm) {
    constexpr int MAXM = decltype(maxm)::value, NT = decltype(nt)::value, CM = decltype(cm)::value;
    if (mode == SYNTH_GRID) {
      dim3 grid(xcd_grid(g.nlat, 8));
      hipLaunchKernelGGL((k_ring_grid<MAXM, NT, CM>), grid, dim3(NT), ring_lds<1>(plan_of<CM>(pl), 2), s, g, pl, grid_out);
      return hipGetLastError();
    }
    if constexpr (MAXM <= 1024) {
      if (two_rings(g)) {
        dim3 grid(xcd_grid((g.nlat + 1) / 2, 4), g.nb);
        const size_t lds = ring_lds<2>(plan_of<CM>(pl), 4);
        // M = 768: three workgroups of 256 threads per CU overlap their phases (6144 rings
        // 54 us against 58 with 512 threads); when there is one per CU, 512 threads are
        // faster (384 rings: 8.2 against 9.4 us)
        if (MAXM == 768 && (int64_t)g.nlat * g.nb > 1024)
          hipLaunchKernelGGL((k_ring<MAXM, NT, 2, CM>), grid, dim3(NT), lds, s, g, pl);
        else
          hipLaunchKernelGGL((k_ring<MAXM, 2 * NT, 2, CM>), grid, dim3(2 * NT), lds, s, g, pl);
        return hipGetLastError();
      }
    }
    dim3 grid(xcd_grid(g.nlat, 8), g.nb);
    constexpr int NT1 = MAXM == 384 ? 192 : NT;  // (192 rings of M = 384: 5.8 us, 6.2 with 128)
    hipLaunchKernelGGL((k_ring<MAXM, NT1, 1, CM>), grid, dim3(NT1), ring_lds<1>(plan_of<CM>(pl), 2), s, g, pl);
    return hipGetLastError();
  });
}

}  // namespace nse
