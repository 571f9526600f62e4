// Small Hessenberg exponential F = exp(tau Hbar) e_1 in one workgroup, float64.
//
// Hbar = [[H_m, 0], [h_{m+1,m} e_m^T, 0]] is n x n with n = m + 1 <= 65; the
// last entry of F is the error estimate of the Krylov projection (eq. kryexp).
// The method is the degree-19 Taylor polynomial with scaling and squaring:
// X = tau Hbar / 2^s with ||X||_1 <= theta_19, T_19(X) evaluated by the
// Paterson-Stockmeyer scheme in powers of X^4 (X^2, X^3, X^4, then four
// Horner steps T <- X^4 T + C_i with C_i = sum_{r<4} X^r / (4i + r)!: seven
// products and no linear solve), then s squarings.  theta_19 = 1.26038 is the
// largest 1-norm for which the backward-error bound of the truncated series
// (Al-Mohy and Higham, SIAM J. Matrix Anal. Appl. 31 (2009), Section 3:
// sum_{k>19} |c_k| theta^{k-1} <= 2^-53 for the coefficients c_k of
// log(e^{-x} T_19(x))) holds; the value was computed with exact rational
// series arithmetic.  Only the first column is returned, so the last squaring
// is a matrix-vector product.
//
// Hbar's last column is zero, so every matrix of the evaluation has the form
// [[P, 0], [p', c]]: P (m x m, at most 64 x 64 = 4 x 4 tiles, two per wave) goes
// through the matrix cores, and the row p of a product P Q is p Q + c q, a
// vector-matrix product on the side.  As one 65 x 65 matrix it took 5 x 5
// tiles (four rounds of the 8 waves instead of two) with k padded to 68.
//
// Layout: the operands of every product live in LDS (two 64 x 64 row-major
// tiles of stride kNmPad, zero past m).  A product is computed with the float64
// matrix cores (v_mfma_f64_16x16x4f64) and kept in registers until a barrier,
// after which every output element is written by the one lane that holds it
// (with the linear combinations the Horner steps need; that lane also keeps
// its elements of X, X^2 and X^3 in registers), so a product may overwrite its
// own operands.  The squarings alternate between the two tiles, one barrier
// each.  Per product about 5 us (matrix cores alone 1.7 at m = 64);
// one evaluation at m = 64 in the benchmark call 83 us, 200 with X^k in
// global scratch and 65 x 65 tiles.
#pragma once

#include "kp_internal.h"

namespace kp {

constexpr double kTheta19 = 1.2603810606426387;

// Taylor coefficients 1/k!, k <= 19.
struct Taylor19 {
  double c[20];
  constexpr Taylor19() : c() {
    c[0] = 1.0;
    for (int k = 1; k <= 19; ++k) c[k] = c[k - 1] / (double)k;
  }
};
constexpr Taylor19 kTaylor{};

// The output tiles of C = A B (A, B: LDS tiles, stride kNmPad) held by this lane:
// tile t = wave + 8 s (s < 2) of the nt^2 tiles of 16 x 16.  Operands of
// v_mfma_f64_16x16x4f64: lane l supplies A[l % 16][l / 16] and B[l / 16][l %
// 16] of the 16 x 4 and 4 x 16 slices; element v of its accumulator is
// C[l / 16 + 4 v][l % 16] (checked on the device against a host product).
constexpr int kTilesPerWave = 2;
constexpr int kExDim = 64;
typedef double kp_d4 __attribute__((ext_vector_type(4)));

struct Tiles {
  kp_d4 c[kTilesPerWave];
};

__device__ inline void mm_tiles(int nt, const double* A, const double* B, Tiles& T) {
  const int lane = kp_tid() & 63, wv = kp_tid() >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const double *ap[kTilesPerWave], *bp[kTilesPerWave];
#pragma unroll
  for (int s = 0; s < kTilesPerWave; ++s) {
    T.c[s] = (kp_d4){0.0, 0.0, 0.0, 0.0};
    // (tiles past the last one compute on a valid clamped tile and are never
    // written, so the chains run unbranched)
    const int t = min(wv + kWaves * s, nt * nt - 1);
    const int ti = t / nt, tj = t - ti * nt;
    ap[s] = A + (16 * ti + lr) * kNmPad + lk;
    bp[s] = B + lk * kNmPad + 16 * tj + lr;
  }
  // four steps of k at a time: their operands are loaded before the first
  // product, and the next group's behind it
  double av[kTilesPerWave][4], bv[kTilesPerWave][4];
#pragma unroll
  for (int s = 0; s < kTilesPerWave; ++s)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      av[s][q] = ap[s][4 * q];
      bv[s][q] = bp[s][4 * q * kNmPad];
    }
  for (int g = 0; g < nt; ++g) {
    double an[kTilesPerWave][4], bn[kTilesPerWave][4];
    const int go = min(g + 1, nt - 1) * 16;
#pragma unroll
    for (int s = 0; s < kTilesPerWave; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        an[s][q] = ap[s][go + 4 * q];
        bn[s][q] = bp[s][(go + 4 * q) * kNmPad];
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int s = 0; s < kTilesPerWave; ++s)
        T.c[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s][q], bv[s][q], T.c[s], 0, 0, 0);
#pragma unroll
    for (int s = 0; s < kTilesPerWave; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        av[s][q] = an[s][q];
        bv[s][q] = bn[s][q];
      }
  }
}

// Calls f(s, v, offset, diagonal) for every element of the tiles this lane
// holds (element v of tile s at row * kNmPad + column).
template <typename F>
__device__ inline void tiles_for_each(int nt, F f) {
  const int lane = kp_tid() & 63, wv = kp_tid() >> 6;
#pragma unroll
  for (int s = 0; s < kTilesPerWave; ++s) {
    const int t = wv + kWaves * s;
    if (t >= nt * nt) continue;
    const int ti = t / nt, tj = t - ti * nt;
    const int k = 16 * tj + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * ti + (lane >> 4) + 4 * v;
      f(s, v, i * kNmPad + k, i == k);
    }
  }
}

// The row p M of a product on the side: wave g sums k = 8 g .. 8 g + 7 for
// column l into part[g][l] (before the product's barrier); row_sum adds the
// eight parts (after it).
__device__ inline void row_parts(const double* p, const double* M, double* part) {
  const int l = kp_tid() & 63, g = kp_tid() >> 6;
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kExDim / kWaves; ++q)
    s = __builtin_fma(p[8 * g + q], M[(8 * g + q) * kNmPad + l], s);
  part[kExDim * g + l] = s;
}
__device__ inline double row_sum(const double* part, int l) {
  double s = 0.0;
#pragma unroll
  for (int g = 0; g < kWaves; ++g) s += part[kExDim * g + l];
  return s;
}

// Entry (i, k) of a column-major Hessenberg matrix.
struct HessCol {
  const double* p;
  int ld;
  __device__ double operator()(int i, int k) const { return p[(int64_t)k * ld + i]; }
};

// F[0..m] = exp(tau Hbar) e_1 for the Hessenberg H (entries H(i, k)) of size
// (m+1) x m; zero_sub drops h_{m+1,m} (lucky breakdown).  Whole workgroup; lds
// holds at least kExDoubles doubles.
constexpr int kExDoubles = 2 * kExDim * kNmPad + 5 * kExDim + kWaves * kExDim;

template <typename HT>
__device__ inline void expm_hbar(const HT& H, int m, double tau, bool zero_sub, double* F, double* lds) {
  __shared__ double s_red[kWaves];
  __shared__ int s_s;
  double* sA = lds;
  double* sB = lds + kExDim * kNmPad;
  double* r1 = sB + kExDim * kNmPad;     // last rows of X, X^2, X^3, X^4, T
  double* r2 = r1 + kExDim;
  double* r3 = r2 + kExDim;
  double* r4 = r3 + kExDim;
  double* rt = r4 + kExDim;
  double* part = rt + kExDim;
  const int tid = kp_tid(), nt = (m + 15) >> 4;
  const double* c = kTaylor.c;
  // X = tau H into sA (zero past m); its last row into r1; 1-norm of X
  for (int idx = tid; idx < kExDim * kExDim; idx += kThreads) {
    const int i = idx & 63, k = idx >> 6;
    sA[i * kNmPad + k] = (k < m && i < m && i <= k + 1) ? tau * H(i, k) : 0.0;
  }
  if (tid < kExDim) r1[tid] = (tid == m - 1 && !zero_sub) ? tau * H(m, m - 1) : 0.0;
  __syncthreads();
  double cs = tid < kExDim ? fabs(r1[tid]) : 0.0;
  {
    // column l of wave g's eight rows
    const int l = tid & 63, g = tid >> 6;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kExDim / kWaves; ++q) s += fabs(sA[(8 * g + q) * kNmPad + l]);
    part[kExDim * g + l] = s;
  }
  __syncthreads();
  if (tid < kExDim) cs += row_sum(part, tid);
  const double cmax = block_max(tid < kExDim ? cs : 0.0, s_red);
  if (tid == 0) {
    int s = 0;
    if (isfinite(cmax) && cmax > kTheta19) {
      int e;
      const double r = frexp(cmax / kTheta19, &e);   // cmax/theta = r 2^e, r in [0.5,1)
      s = (r == 0.5) ? e - 1 : e;                    // smallest s: ratio <= 2^s
    }
    s_s = s;
  }
  __syncthreads();
  const int s = s_s;
  const double sc = ldexp(1.0, -s);
  for (int idx = tid; idx < kExDim * kExDim; idx += kThreads) sA[(idx >> 6) * kNmPad + (idx & 63)] *= sc;
  if (tid < kExDim) r1[tid] *= sc;
  __syncthreads();
  Tiles T;
  double x1[kTilesPerWave][4], x2[kTilesPerWave][4], x3[kTilesPerWave][4];
  // X2 = X X -> sB
  mm_tiles(nt, sA, sA, T);
  row_parts(r1, sA, part);
  tiles_for_each(nt, [&](int q, int v, int o, bool) {
    x1[q][v] = sA[o];
    x2[q][v] = T.c[q][v];
    sB[o] = T.c[q][v];
  });
  if (nt * 16 < kExDim)   // (zero past the tiles: row_parts reads all 64 rows)
    for (int idx = tid; idx < kExDim * kExDim; idx += kThreads)
      if ((idx >> 6) >= 16 * nt || (idx & 63) >= 16 * nt) sB[(idx >> 6) * kNmPad + (idx & 63)] = 0.0;
  __syncthreads();
  if (tid < kExDim) r2[tid] = row_sum(part, tid);
  __syncthreads();
  // X3 = X2 X
  mm_tiles(nt, sB, sA, T);
  row_parts(r2, sA, part);
  tiles_for_each(nt, [&](int q, int v, int, bool) { x3[q][v] = T.c[q][v]; });
  __syncthreads();
  if (tid < kExDim) r3[tid] = row_sum(part, tid);
  // X4 = X2 X2 -> sA; sB <- C_4 = I/16! + X/17! + X^2/18! + X^3/19!
  mm_tiles(nt, sB, sB, T);
  __syncthreads();
  row_parts(r2, sB, part);
  __syncthreads();
  tiles_for_each(nt, [&](int q, int v, int o, bool d) {
    sA[o] = T.c[q][v];
    sB[o] = (d ? c[16] : 0.0) + c[17] * x1[q][v] + c[18] * x2[q][v] + c[19] * x3[q][v];
  });
  if (tid < kExDim) {
    r4[tid] = row_sum(part, tid);
    rt[tid] = c[17] * r1[tid] + c[18] * r2[tid] + c[19] * r3[tid];
  }
  __syncthreads();
  // Horner in X^4: T <- X^4 T + C_i, i = 3, 2, 1, 0 (T in sB; its corner is the
  // constant of C_i)
  for (int i4 = 12; i4 >= 0; i4 -= 4) {
    mm_tiles(nt, sA, sB, T);
    row_parts(r4, sB, part);
    __syncthreads();
    tiles_for_each(nt, [&](int q, int v, int o, bool d) {
      sB[o] = T.c[q][v] + ((d ? c[i4] : 0.0) + c[i4 + 1] * x1[q][v] + c[i4 + 2] * x2[q][v] +
                           c[i4 + 3] * x3[q][v]);
    });
    if (tid < kExDim)
      rt[tid] = row_sum(part, tid) + (c[i4 + 1] * r1[tid] + c[i4 + 2] * r2[tid] + c[i4 + 3] * r3[tid]);
    __syncthreads();
  }
  // s - 1 squarings, alternating between the tiles (corner 1: p <- p T + p)
  double* src = sB;
  double* dst = sA;
  for (int it = 1; it < s; ++it) {
    mm_tiles(nt, src, src, T);
    row_parts(rt, src, part);
    tiles_for_each(nt, [&](int q, int v, int o, bool) { dst[o] = T.c[q][v]; });
    __syncthreads();
    if (tid < kExDim) rt[tid] += row_sum(part, tid);
    __syncthreads();
    double* t = src;
    src = dst;
    dst = t;
  }
  // F = R (R e_1) if s >= 1, else R e_1 (R = src)
  if (s == 0) {
    if (tid < m) F[tid] = src[tid * kNmPad];
    if (tid == m) F[m] = rt[0];
  } else {
    // 8 lanes per row
    const int r = tid >> 3, l = tid & 7;
    double v = 0.0, p = 0.0;
#pragma unroll
    for (int q = 0; q < kExDim / 8; ++q) {
      const int k = l + 8 * q;
      const double x = src[k * kNmPad];
      v = __builtin_fma(src[r * kNmPad + k], x, v);
      p = __builtin_fma(rt[k], x, p);
    }
    v += dpp_mov<0xB1>(v);
    p += dpp_mov<0xB1>(p);
    v += dpp_mov<0x4E>(v);
    p += dpp_mov<0x4E>(p);
    v += dpp_mov<0x141>(v);
    p += dpp_mov<0x141>(p);
    if (l == 0 && r < m) F[r] = v;
    if (tid == 0) F[m] = p + rt[0];
  }
  __syncthreads();
}

// ---- the evaluation as one 65 x 65 matrix (float basis) ------------------------
//
// The kernels with a float basis keep it: with the tolerance at float32's
// resolution their step control answers the last bits of the error estimate,
// and the other evaluation's rounding moved the 2 x 2048^2 result by 3e-9
// relative (float64: 1e-13), for 0.1 % of that call.
__device__ inline double* slot(const Args& a, int s) {
  return a.ex + (int64_t)s * kNmPad * kNmPad;
}

// The output tiles of C = A B (A, B: LDS tiles, stride kNmPad, n <= 65)
// held by this lane: tile t = wave + 8 s (s < kTilesPerWave65) of the
// ceil(n/16)^2 tiles of 16 x 16.  Operands of v_mfma_f64_16x16x4f64: lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16] of the 16 x 4 and 4 x 16
// slices; element v of its accumulator is C[l / 16 + 4 v][l % 16] (checked on
// the device against a host product).
constexpr int kTilesPerWave65 = 4;

struct Tiles65 {
  int nt;                       // tiles per side
  kp_d4 c[kTilesPerWave65];
};

__device__ inline void mm_tiles65(int n, const double* A, const double* B, Tiles65& T) {
  const int lane = kp_tid() & 63, wv = kp_tid() >> 6;
  T.nt = (n + 15) >> 4;
  const int ntile = T.nt * T.nt;
  const int lr = lane & 15, lk = lane >> 4;
  int arow[kTilesPerWave65], bcol[kTilesPerWave65];
#pragma unroll
  for (int s = 0; s < kTilesPerWave65; ++s) {
    T.c[s] = (kp_d4){0.0, 0.0, 0.0, 0.0};
    // tiles past the last one compute on a valid clamped tile and are never
    // written (tiles_for_each skips them), so the four chains run unbranched
    const int t = min(wv + kWaves * s, ntile - 1);
    const int ti = t / T.nt, tj = t - ti * T.nt;
    arow[s] = min(16 * ti + lr, kNmPad - 1);    // A operand: A[row][k]
    bcol[s] = min(16 * tj + lr, kNmPad - 1);    // B operand: B[k][col]
  }
  // the four accumulation chains are interleaved; the operands of step k0 + 4
  // are loaded while step k0 multiplies; entries past n enter as zeros
  double av[kTilesPerWave65], bv[kTilesPerWave65];
#pragma unroll
  for (int s = 0; s < kTilesPerWave65; ++s) {
    const double ta = A[arow[s] * kNmPad + lk], tb = B[lk * kNmPad + bcol[s]];
    av[s] = (lk < n) ? ta : 0.0;
    bv[s] = (lk < n) ? tb : 0.0;
  }
  for (int k0 = 0; k0 < n; k0 += 4) {
    const int k = k0 + 4 + lk;
    const int kc = min(k, kNmPad - 1);
    double an[kTilesPerWave65], bn[kTilesPerWave65];
#pragma unroll
    for (int s = 0; s < kTilesPerWave65; ++s) {
      an[s] = A[arow[s] * kNmPad + kc];
      bn[s] = B[kc * kNmPad + bcol[s]];
    }
#pragma unroll
    for (int s = 0; s < kTilesPerWave65; ++s)
      T.c[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s], bv[s], T.c[s], 0, 0, 0);
#pragma unroll
    for (int s = 0; s < kTilesPerWave65; ++s) {
      av[s] = (k < n) ? an[s] : 0.0;
      bv[s] = (k < n) ? bn[s] : 0.0;
    }
  }
}

// Calls f(i, k, value) for every element of C = A B inside the n x n matrix
// that this lane holds.
template <typename F>
__device__ inline void tiles_for_each65(int n, const Tiles65& T, F f) {
  const int lane = kp_tid() & 63, wv = kp_tid() >> 6;
  const int ntile = T.nt * T.nt;
#pragma unroll
  for (int s = 0; s < kTilesPerWave65; ++s) {
    const int t = wv + kWaves * s;
    if (t >= ntile) continue;
    const int ti = t / T.nt, tj = t - ti * T.nt;
    const int k = 16 * tj + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * ti + (lane >> 4) + 4 * v;
      if (i < n && k < n) f(i, k, T.c[s][v]);
    }
  }
}

// F[0..m] = exp(tau Hbar) e_1 for the Hessenberg H (entries H(i, k)) of size
// (m+1) x m; zero_sub drops h_{m+1,m} (lucky
// breakdown).  Whole workgroup; lds holds at least 2 kNmPad^2 doubles.
template <typename HT>
__device__ inline void expm_hbar65(const Args& a, const HT& H, int m, double tau, bool zero_sub, double* F, double* lds) {
  __shared__ double s_red[kWaves];
  __shared__ int s_s;
  double* sA = lds;
  double* sB = lds + kNmPad * kNmPad;
  const int n = m + 1;
  const int tid = kp_tid();
  const double* c = kTaylor.c;
  // X = tau * Hbar into sA (zero outside n x n); sB zeroed; 1-norm of X
  for (int idx = tid; idx < kNmPad * kNmPad; idx += kThreads) {
    const int i = idx / kNmPad, k = idx - i * kNmPad;
    double v = 0.0;
    if (k < m && i <= k + 1 && i < n) {
      v = H(i, k);
      if (zero_sub && k == m - 1 && i == m) v = 0.0;
    }
    sA[idx] = tau * v;
    sB[idx] = 0.0;
  }
  __syncthreads();
  double cmax = 0.0;
  for (int k = tid; k < n; k += kThreads) {
    double cs = 0.0;
    for (int i = 0; i < n; ++i) cs += fabs(sA[i * kNmPad + k]);
    cmax = fmax(cmax, cs);
  }
  cmax = block_max(cmax, s_red);
  if (tid == 0) {
    int s = 0;
    if (isfinite(cmax) && cmax > kTheta19) {
      int e;
      const double r = frexp(cmax / kTheta19, &e);   // cmax/theta = r 2^e, r in [0.5,1)
      s = (r == 0.5) ? e - 1 : e;                    // smallest s: ratio <= 2^s
    }
    s_s = s;
  }
  __syncthreads();
  const int s = s_s;
  const double sc = ldexp(1.0, -s);
  double* gX = slot(a, 0);
  double* gX2 = slot(a, 1);
  double* gX3 = slot(a, 2);
  for (int idx = tid; idx < kNmPad * kNmPad; idx += kThreads) {
    const double v = sA[idx] * sc;
    sA[idx] = v;
    gX[idx] = v;
  }
  __syncthreads();
  Tiles65 T;
  // X2 = X X -> sB and scratch
  mm_tiles65(n, sA, sA, T);
  __syncthreads();
  tiles_for_each65(n, T, [&](int i, int k, double v) {
    sB[i * kNmPad + k] = v;
    gX2[i * kNmPad + k] = v;
  });
  __syncthreads();
  // X3 = X2 X -> scratch
  mm_tiles65(n, sB, sA, T);
  __syncthreads();
  tiles_for_each65(n, T, [&](int i, int k, double v) { gX3[i * kNmPad + k] = v; });
  __syncthreads();
  // X4 = X2 X2 -> sA; sB <- C_4 = I/16! + X/17! + X^2/18! + X^3/19!
  mm_tiles65(n, sB, sB, T);
  __syncthreads();
  tiles_for_each65(n, T, [&](int i, int k, double v) {
    const int o = i * kNmPad + k;
    sA[o] = v;
    sB[o] = ((i == k) ? c[16] : 0.0) + c[17] * gX[o] + c[18] * gX2[o] + c[19] * gX3[o];
  });
  __syncthreads();
  // Horner in X^4: T <- X^4 T + C_i, i = 3, 2, 1, 0 (T in sB)
  for (int i4 = 12; i4 >= 0; i4 -= 4) {
    mm_tiles65(n, sA, sB, T);
    __syncthreads();
    tiles_for_each65(n, T, [&](int i, int k, double v) {
      const int o = i * kNmPad + k;
      sB[o] = v + (((i == k) ? c[i4] : 0.0) + c[i4 + 1] * gX[o] + c[i4 + 2] * gX2[o] +
                   c[i4 + 3] * gX3[o]);
    });
    __syncthreads();
  }
  // s - 1 squarings in place in sB
  for (int it = 1; it < s; ++it) {
    mm_tiles65(n, sB, sB, T);
    __syncthreads();
    tiles_for_each65(n, T, [&](int i, int k, double v) { sB[i * kNmPad + k] = v; });
    __syncthreads();
  }
  // F = R (R e_1) if s >= 1, else R e_1 (R = sB)
  if (s == 0) {
    for (int i = tid; i < n; i += kThreads) F[i] = sB[i * kNmPad];
  } else {
    double* col = sA;
    for (int i = tid; i < n; i += kThreads) col[i] = sB[i * kNmPad];
    __syncthreads();
    for (int i = tid; i < n; i += kThreads) {
      double v = 0.0;
      for (int k = 0; k < n; ++k) v += sB[i * kNmPad + k] * col[k];
      F[i] = v;
    }
  }
  __syncthreads();
}

}  // namespace kp
