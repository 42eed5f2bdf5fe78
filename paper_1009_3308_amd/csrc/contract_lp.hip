// Split-bf16 Legendre contractions on MFMA (the synthesis and analysis of
// Section 4.2 with bf16 products and FP32 accumulation).
//
// The Legendre values are continued by the FP64 recurrence of eq. (sph_har) from two
// seed rows of the table T1 per 32 degrees, and rounded to FP32. Each operand x is
// split into three bf16 pieces
// x ~ x0 + x1 + x2 (each the rounded remainder of the previous ones), and the
// six products xi*yj with i + j <= 2 (relative weight >= 2^-16) run on
// v_mfma_f32_16x16x32_bf16, accumulating in FP32 over blocks of 32 terms; the
// block sums are added in FP64. The Legendre recurrences, the coefficient
// panels, the quadrature weights, the FFTs, the grid products and the time-step
// update stay in FP64.
//
// Synthesis: per (order m, 128-latitude tile) a workgroup of eight waves; wave w
// computes C[16 latitudes][16 columns] = sum_k T[k][lat] B[k][col] over the
// whole degree range, with columns 0-7 the even-degree and 8-15 the odd-degree
// panel values (4 fields x re/im). B is the same for the eight waves and is
// split once per workgroup into LDS in operand order (only the four degrees of
// each column's parity; the rest of the operand is zero). The northern value is
// E + O and the mirrored southern value E - O. The wave takes four blocks of 32 degrees
// at a time: lane (lat, q) continues the 32 degrees of block q, and lanes of one
// latitude then exchange groups of eight degrees (4 x 4, by register swaps), so that each
// holds its operand of all four blocks.
// Analysis: per (order m, tile of 64 or 128 degrees) four waves; wave w computes
// C[4 used rows][16 degrees] = sum_p A[row][p] T[p][k] for one or two tiles of 16 degrees, with
// rows We.re, We.im, Wo.re, Wo.im (the ring spectra folded over latitude pairs, split once
// per workgroup into LDS; only the four live rows are stored), then the
// epilogue of spectral_ops.h. A lane continues its latitude over the 16 or 32 degrees; the
// values pass through LDS (a wave's own, degree-major, rows of 68: free of bank
// conflicts) to the lanes that hold a degree of the operand.
//
// Bound by vector instructions: per 2048 values of a wave about 430 (recurrence and
// rounding 122, exchange 32, splits 200, FP64 sums 48), 20 us of issue at N = 511; the six
// products take a fifth of that on the matrix cores. Streaming the values from FP32
// tables (200 MB for each contraction) took 54.6 us for the synthesis and 53.6 for the
// analysis; now 42.5 and 42.
//
// MFMA operand layouts (checked on gfx950): for 16x16x32 bf16, lane l supplies
// row l%16 of A and column l%16 of B for K = 8*(l/16) .. +7, and receives C rows
// 4*(l/16) .. +3 of column l%16.
#include <type_traits>

#include "spectral_ops.h"

namespace nse {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kLpWaves = 4;
constexpr int kLpThreads = 64 * kLpWaves;
constexpr int kSynWaves = 8;                  // of 16 latitudes
constexpr int kSynThreads = 64 * kSynWaves, kSynTile = 16 * kSynWaves;
constexpr int kLpSeg = 32;                    // degrees continued from one seed pair
constexpr int kLpTile = kLpWaves * kLpSeg;    // most degrees per workgroup of the analysis
constexpr int kLpRow = 68;                    // row of 64 latitudes in the exchange

// x ~ h0 + h1 + h2 with h0 = bf16(x), h1 = bf16(x - h0), h2 = bf16(x - h0 - h1).
// For a double x the remainders are formed exactly in FP64.
__device__ __forceinline__ void split3(double x, __bf16& h0, __bf16& h1, __bf16& h2) {
  h0 = (__bf16)(float)x;
  const double r1 = x - (double)(float)h0;
  h1 = (__bf16)(float)r1;
  const double r2 = r1 - (double)(float)h1;
  h2 = (__bf16)(float)r2;
}
// For a float x the remainders x - h0 and x - h0 - h1 are exact in FP32.
__device__ __forceinline__ void split3f(float x, __bf16& h0, __bf16& h1, __bf16& h2) {
  h0 = (__bf16)x;
  const float r1 = x - (float)h0;
  h1 = (__bf16)r1;
  h2 = (__bf16)(r1 - (float)h1);
}

__device__ __forceinline__ floatx4 mfma_bf16x3(const bf16x8& a0, const bf16x8& a1,
                                               const bf16x8& a2, const bf16x8& b0,
                                               const bf16x8& b1, const bf16x8& b2) {
  floatx4 c = {0.f, 0.f, 0.f, 0.f};
  // smallest terms first
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2, b0, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b2, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b0, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b1, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, c, 0, 0, 0);
  return c;
}

// bf16x8 with the four given values at positions par, par+2, par+4, par+6 and
// zeros elsewhere.
__device__ __forceinline__ bf16x8 interleave(bf16x4 v, int par) {
  const __bf16 z = (__bf16)0.0f;
  bf16x8 r;
  if (par == 0) {
    r[0] = v[0]; r[1] = z; r[2] = v[1]; r[3] = z; r[4] = v[2]; r[5] = z; r[6] = v[3]; r[7] = z;
  } else {
    r[0] = z; r[1] = v[0]; r[2] = z; r[3] = v[1]; r[4] = z; r[5] = v[2]; r[6] = z; r[7] = v[3];
  }
  return r;
}

// Swaps lanes 16-31 (48-63) of a with lanes 0-15 (32-47) of b.
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
// Swaps lanes 32-63 of a with lanes 0-31 of b.
__device__ __forceinline__ void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// The lanes of a wave exchange values through the wave's own LDS: its accesses complete
// in order, the compiler must not move them across.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace

// LDS: the split panel [block][piece][64 lanes] with only the four degrees of
// the lane's parity stored (bf16x4; the other four of the operand are zero),
// and the recurrence pairs up to a multiple of four blocks; reused for the 8 x 256 FP64
// partial results at the end.
size_t synthesis_lp_lds_bytes(int N) {
  const int nblk = (N + 2 + 31) / 32;
  size_t split = (size_t)nblk * 3 * 64 * sizeof(bf16x4) + (size_t)((nblk + 3) / 4) * 4 * (kLpSeg + 1) * sizeof(double2);
  const size_t cst = sizeof(double) * kSynWaves * 256;
  return split > cst ? split : cst;
}

// LDS of the split-panel kernel: alpha coefficients and the four panels.
size_t split_panel_lp_lds_bytes(int N) { return sizeof(double2) * (size_t)(5 * N + 11); }

// The split B operand of the synthesis for one (order m, member), computed
// once per step and shared by every latitude tile: the four coefficient panels
// of the order are built in LDS (spectral_ops.h), then each 32-degree block is
// split into three bf16 pieces in operand order: lane column c = l%16 holds
// (parity c >> 3, field (c & 7) >> 1, re/im c & 1) for K = 8*(l/16) .. +7, of
// which only the four degrees of the column's parity are stored (bf16x4).
__global__ __launch_bounds__(kLpThreads) void k_split_panel_lp(GroupView g, SynthInput in,
                                                               int mode) {
  if (gate_closed(g)) return;  // an ended attempt of a device-controlled run
  const int N = g.N;
  const int m = blockIdx.x, b = blockIdx.y;
  const int L = N + 2 - m;
  const int nblk = (L + 31) / 32;
  extern __shared__ double2 sh[];
  double2* a = sh;              // [N + 3]
  double2* pan = sh + (N + 3);  // [L][4]
  load_order(a, g, in, b, m, L);
  __syncthreads();
  build_panel<4>(pan, a, N, m, L, mode, in.coriolis, in.stream != 0);
  __syncthreads();
  bf16x4* out = reinterpret_cast<bf16x4*>(g.lps + (int64_t)b * g.lpsoff[N + 1] + g.lpsoff[m]);
  for (int it = threadIdx.x; it < nblk * 64; it += blockDim.x) {
    const int kb = it >> 6, l = it & 63;
    const int c = l & 15, q = l >> 4;
    const int par = c >> 3, fld = (c & 7) >> 1, cmp = c & 1;
    bf16x4 h[3];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int k = kb * 32 + 8 * q + 2 * jj + par;  // the degrees of this column's parity
      double v = 0.0;
      if (k < L) {
        const double2 P = pan[4 * k + fld];
        v = cmp ? P.y : P.x;
      }
      __bf16 h0, h1, h2;
      split3(v, h0, h1, h2);
      h[0][jj] = h0;
      h[1][jj] = h1;
      h[2][jj] = h2;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) out[(kb * 3 + i) * 64 + l] = h[i];
  }
}

__global__ __launch_bounds__(kSynThreads) void k_synthesis_lp(GroupView g, SynthInput in, int mode) {
  if (gate_closed(g)) return;  // an ended attempt of a device-controlled run
  const int N = g.N, nh = g.nh, nlat = g.nlat;
  const int ntile = (nh + kSynTile - 1) / kSynTile;
  const int m = blockIdx.x / ntile;
  const int tile = blockIdx.x - m * ntile;
  const int b = blockIdx.y;
  const int L = N + 2 - m;
  const int nblk = (L + 31) / 32;
  extern __shared__ double2 sh[];
  bf16x4* bsplit = reinterpret_cast<bf16x4*>(sh);  // [nblk][3][64]
  double* cst = reinterpret_cast<double*>(sh);     // reused: [wave][16][16]
  // the order's split panel (k_split_panel_lp), copied into LDS
  const bf16x4* src =
      reinterpret_cast<const bf16x4*>(g.lps + (int64_t)b * g.lpsoff[N + 1] + g.lpsoff[m]);
  const int nsup = (nblk + 3) / 4;
  const double2* rec = g.rec_a + rec_slot(N, m, m);
  double2* rc = reinterpret_cast<double2*>(bsplit + nblk * 3 * 64);  // [4 nsup][kLpSeg + 1]: rows
  // of one slot more, so that the four q read different banks
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, q = lane >> 4;
  const int prow = tile * kSynTile + wave * 16 + r16;  // latitude row supplied to A
  const bool row_ok = prow < nh;
  const double* T = g.T1 + t1_order_offset(N, m, nh) + min(prow, nh - 1);
  const double x = row_ok ? g.mu[min(prow, nh - 1)] : 0.0;
  // seeds of the lane's block 4 s + q: degrees 32 (4 s + q) and the next
  auto seeds = [&](int s, double& p0, double& p1) {
    const int k = kLpSeg * (4 * s + q);
    p0 = T[(int64_t)min(k, L - 1) * nh];
    p1 = T[(int64_t)min(k + 1, L - 1) * nh];
    if (!row_ok || k >= L) p0 = 0.0;
    if (!row_ok || k + 1 >= L) p1 = 0.0;
  };
  double n0, n1;
  seeds(0, n0, n1);
  // the panel and the recurrence pairs: all loads before the first LDS write (one round
  // trip to memory instead of three)
  constexpr int kMaxBlk = (kMaxM / 3 + 1 + 31) / 32;  // L <= N + 2, 3 N + 2 <= M
  constexpr int KB = (kMaxBlk * 96 + kSynThreads - 1) / kSynThreads;
  constexpr int KR = ((kMaxBlk + 3) / 4 * 4 * kLpSeg + kSynThreads - 1) / kSynThreads;
  uint4 bv[KB];
  double2 rv[KR];
#pragma unroll
  for (int i = 0; i < KB; ++i)
    bv[i] = reinterpret_cast<const uint4*>(src)[min((int)threadIdx.x + i * kSynThreads, nblk * 96 - 1)];
#pragma unroll
  for (int i = 0; i < KR; ++i) rv[i] = rec[min((int)threadIdx.x + i * kSynThreads, L - 1)];
#pragma unroll
  for (int i = 0; i < KB; ++i) {
    const int it = threadIdx.x + i * kSynThreads;
    if (it < nblk * 96) reinterpret_cast<uint4*>(bsplit)[it] = bv[i];
  }
#pragma unroll
  for (int i = 0; i < KR; ++i) {
    const int k = threadIdx.x + i * kSynThreads;
    if (k < 4 * kLpSeg * nsup) rc[k + k / kLpSeg] = k < L ? rv[i] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  const int mypar = r16 >> 3;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int s = 0; s < nsup; ++s) {
    double p2 = n0, p1 = n1;
    if (s + 1 < nsup) seeds(s + 1, n0, n1);
    const double2* c = rc + (kLpSeg + 1) * (4 * s + q);
    float v[kLpSeg];
    v[0] = (float)p2;
    v[1] = (float)p1;
#pragma unroll
    for (int i = 2; i < kLpSeg; ++i) {
      const double t = fma(c[i].x * x, p1, -c[i].y * p2);
      p2 = p1;
      p1 = t;
      v[i] = (float)t;
    }
    // v[8 g + j] of lane (lat, q), group g of block q -> group q of block g
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      swap16(v[j], v[8 + j]);
      swap16(v[16 + j], v[24 + j]);
      swap32(v[j], v[16 + j]);
      swap32(v[8 + j], v[24 + j]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kb = 4 * s + i;
      if (kb < nblk) {
        bf16x8 a0, a1, a2;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          __bf16 h0, h1, h2;
          split3f(v[8 * i + j], h0, h1, h2);
          a0[j] = h0;
          a1[j] = h1;
          a2[j] = h2;
        }
        const bf16x4* B = bsplit + kb * 3 * 64 + lane;
        const floatx4 cc = mfma_bf16x3(a0, a1, a2, interleave(B[0], mypar), interleave(B[64], mypar),
                                       interleave(B[128], mypar));
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] += (double)cc[r];
      }
    }
  }
  __syncthreads();  // the split panel is no longer needed: reuse it
  // C rows 4q+i (latitudes of this wave), column r16
#pragma unroll
  for (int i = 0; i < 4; ++i) cst[(wave * 16 + 4 * q + i) * 16 + r16] = acc[i];
  __syncthreads();
  // one (field, latitude) per thread: E = columns 2f, 2f+1; O = columns 8+2f, 9+2f
  const int f = threadIdx.x & 3, latl = threadIdx.x >> 2;
  const int p = tile * kSynTile + latl;
  const int nf = (mode == SYNTH_NONLINEAR) ? 4 : 3;
  if (f >= nf || p >= nh) return;
  const double* row = cst + latl * 16;
  const double er = row[2 * f], ei = row[2 * f + 1], orr = row[8 + 2 * f], oi = row[9 + 2 * f];
  double2* out = g.F + ((int64_t)b * (N + 1) + m) * nlat * 4 + f;
  out[4 * p] = make_double2(er + orr, ei + oi);
  const int ps = nlat - 1 - p;
  if (ps != p) out[4 * ps] = make_double2(er - orr, ei - oi);
}

// LDS: the split A operand [block][piece][4 K-slices][4 live rows] (rows 4..15 of A are
// zero), the tile's recurrence pairs, then the folded spectra We, Wo [2][nh] and in
// their place the waves' exchange rows (at most 28 KB: five workgroups per CU, so that
// the orders of N = 511 are resident at once).
size_t analysis_lp_lds_bytes(int nh) {
  const int nblk = (nh + 31) / 32;
  const size_t fold = 2 * sizeof(double2) * (size_t)nh;
  const size_t ex = (size_t)kLpWaves * 16 * kLpRow * sizeof(float);
  return (size_t)nblk * 3 * 16 * sizeof(bf16x8) + kLpTile * sizeof(double2) + (fold > ex ? fold : ex);
}

// H: tiles of 16 degrees per wave, one or two.
template <int H>
__global__ __launch_bounds__(kLpThreads) __attribute__((amdgpu_waves_per_eu(5))) void k_analysis_lp(
    GroupView g, AnalOutput out) {
  constexpr int kSeg = 16 * H, kTile = kLpWaves * kSeg;  // degrees per wave, per workgroup
  if (gate_closed(g)) return;  // an ended attempt of a device-controlled run
  const int N = g.N, nh = g.nh;
  const int ntile = (N + kTile) / kTile;
  const int item = xcd_item(blockIdx.x, 4 * ntile);
  const int m = item / ntile;
  // tiles of high degree have less to do or nothing, so the tile that a CU's successive
  // workgroups take changes (as does the wave with the last, partial segment): 55 -> 42 us
  // at N = 511, where the CUs were busy 36 us on average
  const int tile = (item - m * ntile + (m >> 6)) % ntile;
  if (m > N || tile * kTile > N - m) return;  // uniform across the workgroup
  const int b = blockIdx.y;
  const int nblk = (nh + 31) / 32;
  extern __shared__ double2 sh[];
  bf16x8* asplit = reinterpret_cast<bf16x8*>(sh);  // [nblk][3][16]
  double2* rc = reinterpret_cast<double2*>(asplit + nblk * 3 * 16);
  double2* wsh = rc + kTile;  // We [nh], Wo [nh]; then the waves' exchange rows
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int seg = (wave + m) % kLpWaves;
  const int kw = tile * kTile + seg * kSeg;  // the wave's first degree offset
  const bool active = kw <= N - m;
  const double* T = g.T1 + t1_order_offset(N, m, nh) + (int64_t)min(kw, N - m) * nh;
  // the lane's latitude 64 s + lane, and its seeds: degrees kw and kw + 1
  auto seeds = [&](int s, double& p0, double& p1, double& x) {
    const int p = min(64 * s + lane, nh - 1);
    p0 = T[p];
    p1 = T[nh + p];
    x = g.mu[p];
    if (64 * s + lane >= nh) p0 = p1 = 0.0;
  };
  double n0, n1, nx;
  seeds(0, n0, n1, nx);
  // the tile's recurrence pairs and the ring spectra: all loads before the first LDS write
  const int kr = tile * kTile + (int)threadIdx.x;
  const double2 rv = g.rec_a[rec_slot(N, m, m) + min(kr, N + 1 - m)];
  constexpr int KW = (kMaxM / 4 + kLpThreads - 1) / kLpThreads;  // nh <= kMaxM / 4
  const double2* Wb = g.W + ((int64_t)b * (N + 1) + m) * g.nlat;
  double2 qn[KW], qs[KW];
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    const int p = min((int)threadIdx.x + i * kLpThreads, nh - 1);
    qn[i] = Wb[p];
    qs[i] = Wb[g.nlat - 1 - p];
  }
  if ((int)threadIdx.x < kTile) rc[threadIdx.x] = kr <= N + 1 - m ? rv : make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    const int p = threadIdx.x + i * kLpThreads;
    if (p < nh) {
      wsh[p] = make_double2(qn[i].x + qs[i].x, qn[i].y + qs[i].y);
      wsh[nh + p] = make_double2(qn[i].x - qs[i].x, qn[i].y - qs[i].y);
    }
  }
  __syncthreads();
  // A operand of every 32-latitude block, split once: lane row r = l%16 holds
  // We.re, We.im, Wo.re, Wo.im for r < 4 (zero otherwise), K = 8*(l/16) .. +7
  for (int it = threadIdx.x; it < nblk * 16; it += blockDim.x) {
    const int pb = it >> 4, r = it & 3, q = (it >> 2) & 3;
    bf16x8 h[3];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int p = pb * 32 + 8 * q + j;
      double v = 0.0;
      if (p < nh) {
        const double2 w = wsh[((r >> 1) ? nh : 0) + p];
        v = (r & 1) ? w.y : w.x;
      }
      __bf16 h0, h1, h2;
      split3(v, h0, h1, h2);
      h[0][j] = h0;
      h[1][j] = h1;
      h[2][j] = h2;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) asplit[(pb * 3 + i) * 16 + q * 4 + r] = h[i];
  }
  __syncthreads();

  if (!active) return;
  const bool two = kw + 16 <= N - m;  // the second tile has a degree
  const int r16 = lane & 15, q = lane >> 4;
  float* ex = reinterpret_cast<float*>(wsh) + wave * 16 * kLpRow;  // [16 degrees][kLpRow]
  bf16x8 zero8;
#pragma unroll
  for (int j = 0; j < 8; ++j) zero8[j] = (__bf16)0.0f;
  double acc0[4] = {0.0, 0.0, 0.0, 0.0}, acc1[4] = {0.0, 0.0, 0.0, 0.0};
  const double2* c = rc + seg * kSeg;
  for (int s = 0; 2 * s < nblk; ++s) {
    double p2 = n0, p1 = n1;
    const double x = nx;
    if (2 * s + 2 < nblk) seeds(s + 1, n0, n1, nx);
    bf16x8 a[2][3];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int pb = min(2 * s + i, nblk - 1);
      const bf16x8* A = asplit + pb * 3 * 16 + q * 4 + (r16 & 3);
#pragma unroll
      for (int r = 0; r < 3; ++r) a[i][r] = r16 < 4 ? A[16 * r] : zero8;
    }
    auto half = [&](auto hc, double(&ac)[4]) {
      constexpr int h = decltype(hc)::value;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int d = 16 * h + i;
        double t = d == 0 ? p2 : p1;
        if (d >= 2) {
          t = fma(c[d].x * x, p1, -c[d].y * p2);
          p2 = p1;
          p1 = t;
        }
        ex[i * kLpRow + lane] = (float)t;
      }
      wave_fence();
      floatx4 v[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          v[i][j] = *reinterpret_cast<const floatx4*>(ex + r16 * kLpRow + 32 * i + 8 * q + 4 * j);
      wave_fence();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (2 * s + i < nblk) {
          bf16x8 b0, b1, b2;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            __bf16 h0, h1, h2;
            split3f(v[i][j >> 2][j & 3], h0, h1, h2);
            b0[j] = h0;
            b1[j] = h1;
            b2[j] = h2;
          }
          const floatx4 cc = mfma_bf16x3(a[i][0], a[i][1], a[i][2], b0, b1, b2);
#pragma unroll
          for (int r = 0; r < 4; ++r) ac[r] += (double)cc[r];
        }
      }
    };
    half(std::integral_constant<int, 0>{}, acc0);
    if constexpr (H == 2) {
      if (two) half(std::integral_constant<int, 1>{}, acc1);
    }
  }
  // lanes 0..15 hold rows 0..3 (We.re, We.im, Wo.re, Wo.im) of the degrees kw + 16 h + r16
  if (q != 0) return;
  auto finish = [&](int k, const double(&ac)[4]) {
    const bool odd = k & 1;
    if (k <= N - m) finish_degree(g, out, b, m, k, odd ? ac[2] : ac[0], odd ? ac[3] : ac[1]);
  };
  finish(kw + r16, acc0);
  if constexpr (H == 2) finish(kw + 16 + r16, acc1);
}

hipError_t launch_synthesis_lp(const GroupView& g, const SynthInput& in, int mode, int prec,
                               hipStream_t s) {
  if (prec != NSE_PREC_BF16X3) return hipErrorInvalidValue;
  if (!g.lps) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_split_panel_lp, dim3(g.N + 1, g.nb), dim3(kLpThreads),
                     split_panel_lp_lds_bytes(g.N), s, g, in, mode);
  const int ntile = (g.nh + kSynTile - 1) / kSynTile;
  dim3 grid((g.N + 1) * ntile, g.nb);
  hipLaunchKernelGGL(k_synthesis_lp, grid, dim3(kSynThreads), synthesis_lp_lds_bytes(g.N), s, g,
                     in, mode);
  return hipGetLastError();
}

hipError_t launch_analysis_lp(const GroupView& g, const AnalOutput& out, int prec, hipStream_t s) {
  if (prec != NSE_PREC_BF16X3) return hipErrorInvalidValue;
  // One tile of 16 degrees per wave has the shorter chain, two share the seeds, the fold
  // and the split of the ring spectra: the line lies where the workgroups of two tiles fill
  // the chip. One and two tiles: N = 127 6.2 and 8.5 us, N = 255 10.8 and 13.6, N = 340 19.8
  // and 22.2, N = 420 31.0 and 29.3, N = 511 45.7 and 41.6, 16 members of N = 127 28.3 and
  // 25.2, 4 of N = 255 33.2 and 31.3.
  auto launch = [&](auto hc) {
    constexpr int H = decltype(hc)::value, kTile = kLpWaves * 16 * H;
    const int ntile = (g.N + kTile) / kTile;
    dim3 grid(xcd_grid((g.N + 1) * ntile, 4 * ntile), g.nb);
    hipLaunchKernelGGL(k_analysis_lp<H>, grid, dim3(kLpThreads), analysis_lp_lds_bytes(g.nh), s, g,
                       out);
  };
  if ((int64_t)(g.N + 1) * (g.N + 1) * g.nb < 160000)
    launch(std::integral_constant<int, 1>{});
  else
    launch(std::integral_constant<int, 2>{});
  return hipGetLastError();
}

}  // namespace nse
