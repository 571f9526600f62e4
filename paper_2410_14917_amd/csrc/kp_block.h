// The one-reduction Arnoldi process with a float64 basis, two steps per
// grid-wide reduction (block steps): streaming passes and the leader's scalar
// work of kernels k_blk and k_batch<double, false>.
//
// A step of Algorithm 4 reads the basis twice (inner products, then the
// projection) and synchronises the grid once.  Both costs are halved by taking
// two Krylov vectors from one reduction: with x the newest column,
//     w1 = Atilde x,  w2 = Atilde w1,
// one pass over the basis forms the inner products of every column with the
// unmeasured columns and with w1 and w2, and one pass forms the two new
// columns
//     y1 = w1 - U h,  y2 = w2 - U q,          h = T U'w1, q = T U'w2,
//     x_{j+1} = y1 / g1,  x_{j+2} = (y2 - e y1) / g2,
//     e = <y1, y2> / <y1, y1>,  g2^2 = <y2, y2> - e <y1, y2>,
// with T the GSMGS correction of Algorithm 7 over all measured columns and
// the products of the y formed from those of the w (<y1, y2> = <w1, w2> -
// (U'w1)' q).  With A U_{<j} = U H_{<j} (the columns made before), the two
// new columns of the Hessenberg matrix are exact combinations,
//     A u_j     = U h + g1 x_{j+1},
//     A x_{j+1} = [U (q - H_{<j} h_{<j} - h_j h) + (e - h_j) y1 + g2 x_{j+2}] / g1,
// the same H as two single steps to rounding (Krylov dimension 64 on the
// benchmark operators: 3e-14 against 2e-14 relative, both against modified
// Gram-Schmidt).  The two new columns are unmeasured: their norms and
// products with the older columns come with the next reduction (the lagged
// norms of Algorithm 4, for two columns).  Where w1 or w2 lies almost inside
// the span already there (guard kGuard on the squared norms), only x_{j+1} is
// made and the process goes on in single steps.  The forms H-CWY and H-NCWY
// always take single steps: their one-sided corrections do not remove the
// measured loss of orthogonality to first order, which a pair needs.
//
// What bounds it: HBM (or Infinity Cache) bytes of the basis at large grids,
// the latency chain of a step (release, coefficients, halo flags, partial
// sums, scalar work) at small ones.  R element pairs per thread and sub-tile:
// a workgroup of few elements takes R = 1, with more columns in flight per
// thread for the same registers, instead of lanes that repeat the last pair.
//
// Measured against single steps on the partition of >= 4096 elements per
// workgroup (one call): 64 x 64, m = 40 fixed 1576 -> 708 us; 256^2 adaptive
// (tol 1e-8, m <= 48) 10.48 -> 5.16 ms; 1024^2 Allen-Cahn benchmark call 93.7 ->
// 59.5 ms; 2 x 1000 x 1200 Brusselator 102.3 -> 66.8 ms; 512 uneven problems in
// one launch 1333 -> 841 ms.  H-CWY, which takes single steps here, gains from
// the partition alone (501 x 300: 13.4 -> 9.6 ms).
#pragma once

#include "kp_leader.h"
#include "kp_passes.h"

namespace kp {

constexpr int kBSlots = 4 * kMMax + 8;   // LDS stride of a wave's sums: 4 per column, 10 products of the new vectors
constexpr double kGuard = 1e-4;          // a pair needs ||y||^2 > kGuard ||w||^2 for both vectors
constexpr int kCoefLd = kMMax + 4;       // coefficients of one new column: basis columns, then w1, w2
// Workgroups whose partial rows the leader reads itself; above, each quad of
// slots is summed over the rows by one workgroup first (reduce_quads).
constexpr int kDirectRows = 16;

// What the leader's serial work reads, in LDS for the whole launch.
struct LeadB {
  // (row r, column k) of M^{-1} = (I + L)^{-1} at tab[k * kTabLd + r], r >= k,
  // and of L at tab[r * kTabLd + k], r > k: the two triangles of one table
  double tab[kMMax * kTabLd + 8];
  double H[kLdh * kMMax + 8];      // Hessenberg, column-major
  double sigma[kMMax + 8];         // unit scale of column i
  double gamma[kMMax + 8];         // divisor applied to column i + 1
  double wn2[kMMax + 8];           // ||A u_j||^2
  double h[kMMax + 8], q[kMMax + 8];   // projections of w1, w2 (last block step)
  double rp[kMMax + 8];            // raw second Hessenberg column of the last pair
  double beta, e, g1;
  int fallback_cur, m_target, breakdown, n_fallback, arnoldi_steps, onchip;
  int nopair, pend, post;
};

__device__ inline void load_tables_b(const Args& a, LeadB& L, bool resume) {
  const State* st = a.st;
  if (resume) {
    for (int idx = kp_tid(); idx < kMMax * kMMax; idx += kThreads) {
      const int k = idx / kMMax, r = idx - k * kMMax;
      if (r >= k) L.tab[k * kTabLd + r] = st->Minv[(int64_t)k * kLdt + r];
      if (r > k) L.tab[r * kTabLd + k] = st->Lm[(int64_t)k * kLdt + r];
    }
    for (int idx = kp_tid(); idx < kLdh * kMMax; idx += kThreads) L.H[idx] = st->H[idx];
    for (int i = kp_tid(); i < kMMax + 2; i += kThreads) {
      L.sigma[i] = st->sigma[i];
      L.gamma[i] = st->gamma[i];
      L.wn2[i] = st->wn2[i];
    }
  }
  if (kp_tid() == 0) {
    L.beta = st->beta;
    L.fallback_cur = st->fallback_cur;
    L.m_target = st->m_target;
    L.breakdown = st->breakdown;
    L.n_fallback = st->n_fallback;
    L.arnoldi_steps = st->arnoldi_steps;
    L.onchip = st->onchip;
    L.nopair = st->nopair;
    L.pend = 0;
    L.post = 0;
  }
  __syncthreads();
}

// The leader's LDS back to the State: counters at the phases a call can end
// after, the tables too when the launch pauses for the step-by-step entry.
// Columns and rows past the j made so far hold nothing and read as zero.
__device__ inline void store_tables_b(const Args& a, const LeadB& L, bool all, int j) {
  State* st = a.st;
  if (all) {
    for (int idx = kp_tid(); idx < kMMax * kMMax; idx += kThreads) {
      const int k = idx / kMMax, r = idx - k * kMMax;
      st->Minv[(int64_t)k * kLdt + r] = (r >= k && r <= j) ? L.tab[k * kTabLd + r] : 0.0;
      st->Lm[(int64_t)k * kLdt + r] = (r > k && r <= j) ? L.tab[r * kTabLd + k] : 0.0;
    }
    for (int idx = kp_tid(); idx < kLdh * kMMax; idx += kThreads) {
      const int k = idx / kLdh, r = idx - k * kLdh;
      st->H[idx] = (k < j && r <= k + 1) ? L.H[idx] : 0.0;
    }
    for (int i = kp_tid(); i < kMMax + 2; i += kThreads) {
      st->sigma[i] = L.sigma[i];
      st->gamma[i] = L.gamma[i];
      st->wn2[i] = L.wn2[i];
    }
  }
  if (kp_tid() == 0) {
    st->beta = L.beta;
    st->fallback_cur = L.fallback_cur;
    st->breakdown = L.breakdown;
    st->n_fallback = L.n_fallback;
    st->arnoldi_steps = L.arnoldi_steps;
    st->onchip = L.onchip;
    st->nopair = L.nopair;
  }
}

// Whether the step phase that nx opens makes two steps.
__device__ inline int pair_ok(const Args& a, const LeadB& L, int j) {
  return (a.pairs && !L.nopair && j + 2 <= min(L.m_target, a.stop_j)) ? 1 : 0;
}

__device__ inline void new_process(LeadB& L) { L.nopair = 0; }
__device__ inline double beta_of(const Args&, const LeadB& L) { return L.beta; }
__device__ inline const double* hess_of(const Args&, const LeadB& L) { return L.H; }

// ---- reductions of four values ------------------------------------------------

// Sums of four values over the 64 lanes of a wave: lane l gets the total of
// value l & 3.  The first two levels pair the values (a lane keeps the value
// of its index bits and passes the other on), so four sums cost little more
// than one; fixed order.
__device__ inline double add_perm16(double v) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ inline double add_perm32(double v) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ inline double wave_sum4(double v0, double v1, double v2, double v3) {
  const bool b0 = kp_tid() & 1, b1 = kp_tid() & 2;
  const double k01 = b0 ? v1 : v0, p01 = b0 ? v0 : v1;
  const double k23 = b0 ? v3 : v2, p23 = b0 ? v2 : v3;
  const double s01 = k01 + dpp_mov<0xB1>(p01);   // quad_perm [1,0,3,2]
  const double s23 = k23 + dpp_mov<0xB1>(p23);
  const double k = b1 ? s23 : s01, p = b1 ? s01 : s23;
  double s = k + dpp_mov<0x4E>(p);               // quad_perm [2,3,0,1]
  s += dpp_mov<0x124>(s);                        // row_ror:4
  s += dpp_mov<0x128>(s);                        // row_ror:8
  return add_perm32(add_perm16(s));
}

// ---- passes ------------------------------------------------------------------

template <int R>
__device__ inline void tile_pairs_r(int64_t q0, int64_t pend, uint32_t* lo, bool* ok) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t q = q0 + (int64_t)r * kThreads + kp_tid();
    ok[r] = q < pend;
    lo[r] = (uint32_t)(2 * ((ok[r] ? q : pend - 1) - q0));
  }
}

// Basis columns per chunk: the linear combinations keep about 20 pair loads
// in flight per thread, the inner products two chunks of 8.
template <int R> constexpr int kUpdCols = R == 4 ? 5 : (R == 2 ? 10 : 16);
template <int R> constexpr int kDotCols = 8 / R;

// acc1 += sum_i c1[i] V_i, acc2 += sum_i c2[i] V_i over the columns i0, i0 +
// step, ... (nc of them; the columns past nc repeat the last one with
// coefficient 0, so that all loads issue before the first multiply-add).
// The coefficients are in LDS.
template <int R, int C, int U>
__device__ inline void axpy_block(const double* V, int64_t ld, int64_t t0, int i0, int step, int nc,
                                  const double* c1, const double* c2, const uint32_t* lo,
                                  double2* acc1, double2* acc2) {
  double2 v[C][R];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const double* vc = uniform_ptr(V + (int64_t)(i0 + min(c, nc - 1) * step) * ld + t0);
#pragma unroll
    for (int r = 0; r < R; ++r) v[c][r] = load_at(vc, lo[r] * 8u);
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int i = i0 + min(c, nc - 1) * step;
    const double a1 = (c < nc) ? c1[i] : 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      acc1[r].x = __builtin_fma(a1, v[c][r].x, acc1[r].x);
      acc1[r].y = __builtin_fma(a1, v[c][r].y, acc1[r].y);
    }
    if constexpr (U == 2) {
      const double a2 = (c < nc) ? c2[i] : 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        acc2[r].x = __builtin_fma(a2, v[c][r].x, acc2[r].x);
        acc2[r].y = __builtin_fma(a2, v[c][r].y, acc2[r].y);
      }
    }
  }
}

// Published coefficients to LDS (one coherent round trip).
__device__ inline void load_coefs(const Args& a, double* cf) {
  const int t = kp_tid();
  if (t < kCoefLd) cf[t] = cload(&a.pub->coef[min(t, kMMax + 1)]);
  if (t >= 128 && t < 128 + kCoefLd) cf[kCoefLd + t - 128] = cload(&a.pub->coef2[min(t - 128, kMMax + 1)]);
  __syncthreads();
}

// The tails (p <= 8 entries per column) of the U new columns: lane i of wave
// 0 of workgroup 0 takes column i; the newest one is published.
template <int U>
__device__ inline void tail_update_b(const Args& a, double* V, int base, const double* cf,
                                     double& ss1, double& ss2) {
  const int t = kp_tid();
  if (t >= 64) return;
  const int64_t T0 = a.tail_off, ld = a.ld;
  const int nc = base + 1;
  double p1[kPMax], p2[kPMax];
#pragma unroll
  for (int k = 0; k < kPMax; ++k) p1[k] = p2[k] = 0.0;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int i = t + 64 * hh;
    const bool on = i < nc + U;
    const double c1 = (i <= nc) ? cf[min(i, kCoefLd - 1)] : 0.0;
    const double c2 = (U == 2 && on) ? cf[kCoefLd + min(i, kCoefLd - 1)] : 0.0;
    const double* vc = V + (int64_t)(on ? i : 0) * ld + T0;
#pragma unroll
    for (int k = 0; k < kPMax; ++k)
      if (k < a.p && on) {
        const double v = vc[k];
        p1[k] += c1 * v;
        if (U == 2) p2[k] += c2 * v;
      }
  }
#pragma unroll
  for (int k = 0; k < kPMax; ++k) {
    if (k < a.p) {
      const double y1 = wave_sum(p1[k]);
      const double y2 = U == 2 ? wave_sum(p2[k]) : 0.0;
      if (t == 0) {
        V[(int64_t)nc * ld + T0 + k] = y1;
        if (U == 2) V[(int64_t)(nc + 1) * ld + T0 + k] = y2;
        cstore(a.tx + k, U == 2 ? y2 : y1);
        ss1 += y1 * y1;
        ss2 += y2 * y2;
      }
    }
  }
}

// The U pending columns (newest: column j) from the columns 0 .. j - U and
// w1 (and w2), which sit in LDS (keep_xw) or in the columns they become.
// cf: coefficients in LDS.  keep_xw also leaves x_j in the A half of the LDS
// region.  The halo rows of x_j are published.  want_norm: partial slot 0 =
// ||x_j||^2, slot 1 = ||x_{j-1}||^2 (U == 2).
template <int R, int U>
__device__ __attribute__((always_inline)) inline void update_block(const Args& a, int j, const double* cf,
                                                                   double* hl, double* red, bool want_norm) {
  double* V = reinterpret_cast<double*>(a.V);
  const int64_t ld = a.ld;
  const int base = j - U, nc = base + 1;
  double* w1col = V + (int64_t)nc * ld;
  double* w2col = V + (int64_t)(nc + 1) * ld;
  const double* c1 = cf;
  const double* c2 = cf + kCoefLd;
  const double c1w = c1[nc], c2w1 = U == 2 ? c2[nc] : 0.0, c2w2 = U == 2 ? c2[nc + 1] : 0.0;
  const bool keep = a.keep_xw != 0;
  double2* A2 = reinterpret_cast<double2*>(hl);                       // w2, then x_j
  const double2* B2 = reinterpret_cast<const double2*>(hl) + kR * kThreads;   // w1
  const Rows o = own_rows(a);
  double ss1 = 0.0, ss2 = 0.0;
  constexpr int C = kUpdCols<R>;
  for (int si = 0; si < num_segs(a); ++si) {
    const Seg sg = seg_at(a, o, si);
    const int64_t pend = (sg.end + 1) >> 1;
    for (int64_t q0 = sg.beg >> 1; q0 < pend; q0 += (int64_t)kThreads * R) {
      const int64_t t0 = 2 * q0;
      uint32_t lo[R];
      bool ok[R];
      tile_pairs_r<R>(q0, pend, lo, ok);
      double2 acc1[R], acc2[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double2 w1 = keep ? B2[r * kThreads + kp_tid()] : Pair<double>::load(w1col + t0 + lo[r]);
        acc1[r] = make_double2(c1w * w1.x, c1w * w1.y);
        if constexpr (U == 2) {
          const double2 w2 = keep ? A2[r * kThreads + kp_tid()] : Pair<double>::load(w2col + t0 + lo[r]);
          acc2[r] = make_double2(__builtin_fma(c2w2, w2.x, c2w1 * w1.x),
                                 __builtin_fma(c2w2, w2.y, c2w1 * w1.y));
        }
      }
      for (int i1 = nc - 1; i1 >= 0; i1 -= C)
        axpy_block<R, C, U>(V, ld, t0, i1, -1, min(C, i1 + 1), c1, c2, lo, acc1, acc2);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (ok[r]) {
          Pair<double>::store(w1col + t0 + lo[r], acc1[r].x, acc1[r].y);
          ss1 += acc1[r].x * acc1[r].x + acc1[r].y * acc1[r].y;
          double2 x = acc1[r];
          if constexpr (U == 2) {
            Pair<double>::store(w2col + t0 + lo[r], acc2[r].x, acc2[r].y);
            ss2 += acc2[r].x * acc2[r].x + acc2[r].y * acc2[r].y;
            x = acc2[r];
          }
          if (keep) A2[r * kThreads + kp_tid()] = x;
          publish_pair(a, a.hx, sg, t0 + lo[r], x.x, x.y);
        }
      }
    }
  }
  if (wg_rank(a) == 0) tail_update_b<U>(a, V, base, cf, ss1, ss2);
  if (want_norm) {
    ss1 = block_sum(ss1, red);
    if constexpr (U == 2) ss2 = block_sum(ss2, red);
    if (kp_tid() == 0) {
      double* pr = a.part + (int64_t)wg_rank(a) * kCStride;
      cstore(pr, U == 2 ? ss2 : ss1);
      cstore(pr + 1, U == 2 ? ss1 : 0.0);
    }
  }
}

// Products of C columns with xa, x, w1, w2: four sums per column, added to
// the wave's row of sacc.
template <int R, int C>
__device__ inline void dots_block(const double2 (&v)[C][R], const double2* xa, const double2* xv,
                                  const double2* w1, const double2* w2, int i0, int nc, double* sacc) {
  const int lane = kp_tid() & 63, wv = kp_tid() >> 6;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double vx = v[c][r].x, vy = v[c][r].y;
      s0 = __builtin_fma(vy, xa[r].y, __builtin_fma(vx, xa[r].x, s0));
      s1 = __builtin_fma(vy, xv[r].y, __builtin_fma(vx, xv[r].x, s1));
      s2 = __builtin_fma(vy, w1[r].y, __builtin_fma(vx, w1[r].x, s2));
      s3 = __builtin_fma(vy, w2[r].y, __builtin_fma(vx, w2[r].x, s3));
    }
    if (c < nc) {
      const double s = wave_sum4(s0, s1, s2, s3);
      if (lane < 4) sacc[wv * kBSlots + 4 * (i0 + c) + lane] += s;
    }
  }
}

template <int R, int C>
__device__ inline void load_block(const double* V, int64_t ld, int64_t t0, int i0, int nc,
                                  const uint32_t* lo, double2 (&v)[C][R]) {
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const double* vc = uniform_ptr(V + (int64_t)(i0 + min(c, nc - 1)) * ld + t0);
#pragma unroll
    for (int r = 0; r < R; ++r) v[c][r] = load_at(vc, lo[r] * 8u);
  }
}

// The older columns of one sub-tile (double-buffered chunks; the first one is
// in flight in va already) and the products of the new vectors.
template <int R>
__device__ __attribute__((always_inline)) inline void tile_dots(
    const double* V, int64_t ld, int64_t t0, int jo, const uint32_t* lo, const double2* xa,
    const double2* xv, const double2* w1, const double2* w2, double2 (&va)[kDotCols<R>][R], double* sacc) {
  constexpr int C = kDotCols<R>;
  const int lane = kp_tid() & 63, wv = kp_tid() >> 6;
  double g[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) g[k] = 0.0;
  auto acc = [](double s, const double2& p, const double2& q) {
    return __builtin_fma(p.y, q.y, __builtin_fma(p.x, q.x, s));
  };
#pragma unroll
  for (int r = 0; r < R; ++r) {
    g[0] = acc(g[0], xa[r], xa[r]);
    g[1] = acc(g[1], xa[r], xv[r]);
    g[2] = acc(g[2], xa[r], w1[r]);
    g[3] = acc(g[3], xa[r], w2[r]);
    g[4] = acc(g[4], xv[r], xv[r]);
    g[5] = acc(g[5], xv[r], w1[r]);
    g[6] = acc(g[6], xv[r], w2[r]);
    g[7] = acc(g[7], w1[r], w1[r]);
    g[8] = acc(g[8], w1[r], w2[r]);
    g[9] = acc(g[9], w2[r], w2[r]);
  }
  {
    double* srow = sacc + wv * kBSlots + 4 * jo;
    const double s0 = wave_sum4(g[0], g[1], g[2], g[3]);
    const double s1 = wave_sum4(g[4], g[5], g[6], g[7]);
    const double s2 = wave_sum4(g[8], g[9], 0.0, 0.0);
    if (lane < 4) {
      srow[lane] += s0;
      srow[4 + lane] += s1;
      if (lane < 2) srow[8 + lane] += s2;
    }
  }
  double2 vb[C][R];
  for (int i0 = 0; i0 < jo; i0 += 2 * C) {
    const int i1 = i0 + C;
    if (i1 < jo) load_block<R, C>(V, ld, t0, i1, min(C, jo - i1), lo, vb);
    dots_block<R, C>(va, xa, xv, w1, w2, i0, min(C, jo - i0), sacc);
    if (i1 >= jo) break;
    const int i2 = i1 + C;
    if (i2 < jo) load_block<R, C>(V, ld, t0, i2, min(C, jo - i2), lo, va);
    dots_block<R, C>(vb, xa, xv, w1, w2, i1, min(C, jo - i1), sacc);
  }
}

// Tail rows of the block step (wave 0 of workgroup 0): w1 = K x, w2 = K w1
// (upward shifts within each block of pb entries), stored, and their share of
// the products (column t by lane t; those of the new vectors by lane 0).
__device__ inline void tail_block(const Args& a, int j, int na, int two, double* V, double* sacc) {
  const int t = kp_tid();
  if (t >= 64) return;
  const int64_t T0 = a.tail_off, ld = a.ld;
  const int p = a.p, jo = j - na;
  const double* xs = j == 0 ? a.u + T0 : V + (int64_t)j * ld + T0;
  const double* as = V + (int64_t)(na ? j - 1 : 0) * ld + T0;
  double xt[kPMax + 2], at[kPMax], w1[kPMax + 1], w2[kPMax];
#pragma unroll
  for (int k = 0; k < kPMax + 2; ++k) xt[k] = (k < p) ? xs[k] : 0.0;
#pragma unroll
  for (int k = 0; k < kPMax; ++k) at[k] = (na && k < p) ? as[k] : 0.0;
#pragma unroll
  for (int k = 0; k < kPMax + 1; ++k) w1[k] = (k < kPMax && tail_shift_in(a, k)) ? xt[k + 1] : 0.0;
#pragma unroll
  for (int k = 0; k < kPMax; ++k) w2[k] = (two && tail_shift_in(a, k)) ? w1[k + 1] : 0.0;
  if (t == 0) {
#pragma unroll
    for (int k = 0; k < kPMax; ++k) {
      if (k < p) {
        if (j == 0) V[T0 + k] = xt[k];
        V[(int64_t)(j + 1) * ld + T0 + k] = w1[k];
        if (two) V[(int64_t)(j + 2) * ld + T0 + k] = w2[k];
      }
    }
  }
  if (t < jo) {
    const double* vc = V + (int64_t)t * ld + T0;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int k = 0; k < kPMax; ++k) {
      if (k < p) {
        const double v = vc[k];
        s0 += v * at[k];
        s1 += v * xt[k];
        s2 += v * w1[k];
        s3 += v * w2[k];
      }
    }
    sacc[4 * t] += s0;
    sacc[4 * t + 1] += s1;
    sacc[4 * t + 2] += s2;
    sacc[4 * t + 3] += s3;
  }
  if (t == 0) {
    double* s = sacc + 4 * jo;
#pragma unroll
    for (int k = 0; k < kPMax; ++k) {
      s[0] += at[k] * at[k];
      s[1] += at[k] * xt[k];
      s[2] += at[k] * w1[k];
      s[3] += at[k] * w2[k];
      s[4] += xt[k] * xt[k];
      s[5] += xt[k] * w1[k];
      s[6] += xt[k] * w2[k];
      s[7] += w1[k] * w1[k];
      s[8] += w1[k] * w2[k];
      s[9] += w2[k] * w2[k];
    }
  }
}

// tc[c] = entry c + sh of the tail block of plane `plane`, over mu (zero past
// the block): the weights of b_{pb-c} in A w for w = K^sh x.
__device__ inline void tail_weights(const Args& a, int plane, int sh, double inv_mu, double* tc) {
  const int toff = (a.tangent && plane == 1) ? a.pb : 0;
#pragma unroll
  for (int c = 0; c < kPMax; ++c)
    tc[c] = (c + sh < a.pb) ? cload(a.tx + toff + c + sh) * inv_mu : 0.0;
}

// Block step j: w1 = Atilde x_j, w2 = Atilde w1 (two) and the partial sums of
// the reduction.  na: column j - 1 is unmeasured too.  upd: the update of this
// phase has left x_j in LDS (keep_xw).  The rows of w1 the neighbours need
// go through a second halo buffer and the same flags (value 2k + 1; the
// update published 2k).  KEEP (keep_xw): one sub-tile; the LDS region holds
// x_j in its A half while w1 is formed (the halo rows in B), then w1 in B (the
// halo rows in A), and w2 in A at the end, for the next update.
template <int R, bool KEEP, bool HL>
__device__ __attribute__((always_inline)) inline void matvec_block(const Args& a, int j, int na, int two,
                                                                   bool upd, double* sacc, double* hl,
                                                                   unsigned k) {
  double* V = reinterpret_cast<double*>(a.V);
  const int64_t ld = a.ld;
  const Rows o = own_rows(a);
  const int jo = j - na;
  constexpr int C = kDotCols<R>;
  for (int t = kp_tid(); t < kWaves * kBSlots; t += kThreads) sacc[t] = 0.0;
  const double inv_mu = cload(&a.pub->inv_mu);
  double* xcol = V + (int64_t)j * ld;
  double* acol = V + (int64_t)(na ? j - 1 : 0) * ld;
  double* w1col = V + (int64_t)(j + 1) * ld;
  double* w2col = V + (int64_t)(j + 2) * ld;
  double2 va[C][R];
  if constexpr (KEEP) {
    double* lA = hl;
    double* lB = hl + 2 * kR * kThreads;
    double2* A2 = reinterpret_cast<double2*>(lA);
    double2* B2 = reinterpret_cast<double2*>(lB);
    const Seg sg = seg_at(a, o, 0);
    const int64_t pend = (sg.end + 1) >> 1, q0 = sg.beg >> 1, t0 = 2 * q0;
    uint32_t lo[R];
    bool ok[R];
    tile_pairs_r<R>(q0, pend, lo, ok);
    double2 xa[R], xv[R], w1[R], w2[R];
    if (!upd) {
      const double* src = j == 0 ? a.u : xcol;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double2 v = Pair<double>::load(src + t0 + lo[r]);
        if (ok[r]) {
          A2[r * kThreads + kp_tid()] = v;
          if (j == 0) Pair<double>::store(xcol + t0 + lo[r], v.x, v.y);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
      xa[r] = na ? Pair<double>::load(acol + t0 + lo[r]) : make_double2(0.0, 0.0);
    stage_halo<double>(a, a.hx, o, lB);
    double tc[kPMax];
    tail_weights(a, 0, 0, inv_mu, tc);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) xv[r] = *reinterpret_cast<const double2*>(lA + lo[r]);
    aug_tile<double, true, LdsX, R>(a, a.hx, o, sg, LdsX{lA, t0}, lB, t0, lo, tc, w1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!ok[r]) xa[r] = xv[r] = w1[r] = make_double2(0.0, 0.0);
      w2[r] = make_double2(0.0, 0.0);
    }
    if (two) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < R; ++r) {
        B2[r * kThreads + kp_tid()] = w1[r];
        if (ok[r]) publish_pair(a, a.hx2, sg, t0 + lo[r], w1[r].x, w1[r].y);
      }
      flag_publish(a, 2 * k + 1);
      if (jo > 0) load_block<R, C>(V, ld, t0, 0, min(C, jo), lo, va);
      tail_weights(a, 0, 1, inv_mu, tc);
      flag_wait_neighbours(a, 2 * k + 1);
      stage_halo<double>(a, a.hx2, o, lA);
      __syncthreads();
      aug_tile<double, true, LdsX, R>(a, a.hx2, o, sg, LdsX{lB, t0}, lA, t0, lo, tc, w2);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (!ok[r]) w2[r] = make_double2(0.0, 0.0);
    } else if (jo > 0) {
      load_block<R, C>(V, ld, t0, 0, min(C, jo), lo, va);
    }
    tile_dots<R>(V, ld, t0, jo, lo, xa, xv, w1, w2, va, sacc);
    if (wg_rank(a) == 0) tail_block(a, j, na, two, V, sacc);
    __syncthreads();
    // (every stencil read of the halo rows is done: the new vectors' pairs)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (two)
        A2[r * kThreads + kp_tid()] = w2[r];
      else
        B2[r * kThreads + kp_tid()] = w1[r];
    }
  } else {
    if (j == 0) copy_state<double>(a, o, xcol);
    if (HL) stage_halo<double>(a, a.hx, o, hl);
    __syncthreads();
    if (two) {
      for (int si = 0; si < num_segs(a); ++si) {
        const Seg sg = seg_at(a, o, si);
        const int64_t pend = (sg.end + 1) >> 1;
        double tc[kPMax];
        tail_weights(a, sg.plane, 0, inv_mu, tc);
        for (int64_t q0 = sg.beg >> 1; q0 < pend; q0 += (int64_t)kThreads * R) {
          const int64_t t0 = 2 * q0;
          uint32_t lo[R];
          bool ok[R];
          tile_pairs_r<R>(q0, pend, lo, ok);
          double2 w[R];
          aug_tile<double, HL, Col<double>, R>(a, a.hx, o, sg, Col<double>{xcol}, hl, t0, lo, tc, w);
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (ok[r]) {
              Pair<double>::store(w1col + t0 + lo[r], w[r].x, w[r].y);
              publish_pair(a, a.hx2, sg, t0 + lo[r], w[r].x, w[r].y);
            }
        }
      }
      flag_publish(a, 2 * k + 1);
      flag_wait_neighbours(a, 2 * k + 1);
      if (HL) {
        stage_halo<double>(a, a.hx2, o, hl);
        __syncthreads();
      }
    }
    const double* hxs = two ? a.hx2 : a.hx;
    const Col<double> xc{two ? w1col : xcol};
    double* dst = two ? w2col : w1col;
    for (int si = 0; si < num_segs(a); ++si) {
      const Seg sg = seg_at(a, o, si);
      const int64_t pend = (sg.end + 1) >> 1;
      double tc[kPMax];
      tail_weights(a, sg.plane, two, inv_mu, tc);
      for (int64_t q0 = sg.beg >> 1; q0 < pend; q0 += (int64_t)kThreads * R) {
        const int64_t t0 = 2 * q0;
        uint32_t lo[R];
        bool ok[R];
        tile_pairs_r<R>(q0, pend, lo, ok);
        double2 xa[R], xv[R], w1[R], w2[R], t[R];
        if (jo > 0) load_block<R, C>(V, ld, t0, 0, min(C, jo), lo, va);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          xv[r] = Pair<double>::load(xcol + t0 + lo[r]);
          xa[r] = na ? Pair<double>::load(acol + t0 + lo[r]) : make_double2(0.0, 0.0);
          w1[r] = two ? Pair<double>::load(w1col + t0 + lo[r]) : make_double2(0.0, 0.0);
        }
        aug_tile<double, HL, Col<double>, R>(a, hxs, o, sg, xc, hl, t0, lo, tc, t);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (ok[r]) {
            Pair<double>::store(dst + t0 + lo[r], t[r].x, t[r].y);
            w2[r] = two ? t[r] : make_double2(0.0, 0.0);
            w1[r] = two ? w1[r] : t[r];
          } else {
            xa[r] = xv[r] = w1[r] = w2[r] = make_double2(0.0, 0.0);
          }
        }
        tile_dots<R>(V, ld, t0, jo, lo, xa, xv, w1, w2, va, sacc);
      }
    }
    if (wg_rank(a) == 0) tail_block(a, j, na, two, V, sacc);
    __syncthreads();
  }
}

// u = sum_{i<m} cf[i] x_i (coefficients in LDS); the last substep also writes
// out.
template <int R>
__device__ __attribute__((always_inline)) inline void combine_block(const Args& a, int m, const double* cf,
                                                                    bool last) {
  const double* V = reinterpret_cast<const double*>(a.V);
  const int64_t ld = a.ld;
  const Rows o = own_rows(a);
  constexpr int C = kUpdCols<R>;
  for (int si = 0; si < num_segs(a); ++si) {
    const Seg sg = seg_at(a, o, si);
    const int64_t pend = (sg.end + 1) >> 1;
    double* const outp = out_plane(a, sg.plane) - (int64_t)sg.plane * a.npt_pad;
    for (int64_t q0 = sg.beg >> 1; q0 < pend; q0 += (int64_t)kThreads * R) {
      const int64_t t0 = 2 * q0;
      uint32_t lo[R];
      bool ok[R];
      tile_pairs_r<R>(q0, pend, lo, ok);
      double2 acc[R];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = make_double2(0.0, 0.0);
      for (int i0 = 0; i0 < m; i0 += C)
        axpy_block<R, C, 1>(V, ld, t0, i0, 1, min(C, m - i0), cf, cf, lo, acc, acc);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (ok[r]) {
          const int64_t e = t0 + lo[r];
          *reinterpret_cast<double2*>(a.u + e) = acc[r];
          if (!last) publish_pair(a, a.hx, sg, e, acc[r].x, acc[r].y);
          if (last) {
            if (e < sg.end) outp[e] = acc[r].x;
            if (e + 1 < sg.end) outp[e + 1] = acc[r].y;
          }
        }
      }
    }
  }
  if (wg_rank(a) == 0) tail_combine_cols<double, double>(a, V, m, a.pub->coef, -1, 0.0, a.u, !last);
}

// ---- the grid-wide reduction ---------------------------------------------------
//
// Every workgroup stores its row of partial sums; slots that nobody has
// written since they were consumed hold kPartEmpty, so a reader takes the
// data in the load that first sees them (see gather_step_partials).  Up to
// kDirectRows rows are read by the leader.  Above, the rows are summed by
// slot quads first: workgroup q of the first nq reads quad q of every row (one
// 16-byte load per thread at 256 rows) and stores four sums, and the leader
// reads those: one workgroup reading 256 rows of 260 slots took 6 to 11 us
// per step on its share of the coherent path, the two hops about 4.

__device__ inline double* block_part(const Args& a, unsigned k) {
  return a.part + (int64_t)a.part_rows * kCStride + (int64_t)(k & 1u) * a.part_rows * a.bstride;
}
__device__ inline double* block_sums(const Args& a, unsigned k) {
  return a.part + (int64_t)a.part_rows * kCStride + (int64_t)2 * a.part_rows * a.bstride +
         (int64_t)(k & 1u) * a.bstride;
}

// Marks this workgroup's row and sum quads of barrier k + 1's buffers empty
// (consumed at k - 1).
__device__ inline void block_reset(const Args& a, unsigned k) {
  const int t = kp_tid(), w = wg_rank(a);
  const double empty = __builtin_bit_cast(double, kPartEmpty);
  if (t < a.bstride) cstore(block_part(a, k + 1) + (int64_t)w * a.bstride + t, empty);
  if (a.nwg > kDirectRows) {
    const int s = 4 * (w + a.nwg * (t >> 2)) + (t & 3);
    if (s < a.bstride) cstore(block_sums(a, k + 1) + s, empty);
  }
}

__device__ inline bool is_empty(unsigned lo, unsigned hi) {
  return lo == (unsigned)kPartEmpty && hi == (unsigned)(kPartEmpty >> 32);
}

typedef unsigned kp_u4 __attribute__((ext_vector_type(4)));

// One 16-byte slot pair, reloaded until it has been written (bounded).
__device__ inline kp_u4 poll_pair(const Args& a, __amdgpu_buffer_rsrc_t rs, int byte, int* ok) {
  kp_u4 v;
  int64_t t0 = 0;
  for (unsigned it = 0;; ++it) {
    v = __builtin_amdgcn_raw_buffer_load_b128(rs, byte, 0, kCoherentAux);
    if (!is_empty(v[0], v[1]) && !is_empty(v[2], v[3])) break;
    if (it == 0) t0 = wall_clock64();
    __builtin_amdgcn_s_sleep(1);
    if ((it & 15u) == 15u && (aborted(a) || wait_expired(a, t0))) {
      *ok = 0;
      break;
    }
  }
  return v;
}

// First hop (workgroups w < nwg): the sums over all rows of the slot quads w,
// w + nwg, ...; rq: 4 * kWaves doubles of LDS.
__device__ __attribute__((always_inline)) inline void reduce_quads(const Args& a, const double* buf,
                                                                   double* sums, int nslot, double* rq, int* ok) {
  const int half = kp_tid() & 1, lane = kp_tid() & 63, wv = kp_tid() >> 6;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<double*>(buf), (short)0, a.nwg * a.bstride * (int)sizeof(double), kBufWord3);
  for (int q = wg_rank(a); 4 * q < nslot; q += a.nwg) {
    double sx = 0.0, sy = 0.0;
    const int s = 4 * q + 2 * half;   // (nslot is even: a pair is written whole or not at all)
    if (s < nslot)
      for (int row = kp_tid() >> 1; row < a.nwg; row += kThreads / 2) {
        const kp_u4 v = poll_pair(a, rs, (row * a.bstride + s) * (int)sizeof(double), ok);
        sx += lo_double(v[0], v[1]);
        sy += lo_double(v[2], v[3]);
      }
    // over the 32 lanes of one half
    sx += dpp_mov<0x4E>(sx);
    sy += dpp_mov<0x4E>(sy);
    sx += dpp_mov<0x124>(sx);
    sy += dpp_mov<0x124>(sy);
    sx += dpp_mov<0x128>(sx);
    sy += dpp_mov<0x128>(sy);
    sx = add_perm32(add_perm16(sx));
    sy = add_perm32(add_perm16(sy));
    __syncthreads();
    if (lane < 2) {
      rq[wv * 4 + 2 * lane] = sx;
      rq[wv * 4 + 2 * lane + 1] = sy;
    }
    __syncthreads();
    if (kp_tid() < 4 && 4 * q + kp_tid() < nslot) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) t += rq[w * 4 + kp_tid()];
      cstore(sums + 4 * q + kp_tid(), t);
    }
  }
}

// The leader's part: tv[0 .. nslot) = the reduced sums of barrier k.
// own: its own row (LDS; tv itself when it is the only workgroup).
__device__ __attribute__((always_inline)) inline void block_gather(const Args& a, unsigned k, int nslot,
                                                                   const double* own, double* tv, int* ok) {
  const int s = 2 * kp_tid();
  if (a.nwg > kDirectRows) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        block_sums(a, k), (short)0, a.bstride * (int)sizeof(double), kBufWord3);
    if (s < nslot) {
      const kp_u4 v = poll_pair(a, rs, s * (int)sizeof(double), ok);
      tv[s] = lo_double(v[0], v[1]);
      tv[s + 1] = lo_double(v[2], v[3]);
    }
  } else if (s < nslot) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        block_part(a, k), (short)0, a.nwg * a.bstride * (int)sizeof(double), kBufWord3);
    double sx = own[s], sy = own[s + 1];
    if (a.nwg > 1) {
      kp_u4 v[kDirectRows];
      int64_t t0 = 0;
      for (unsigned it = 0;; ++it) {
        bool empty = false;
#pragma unroll
        for (int w = 1; w < kDirectRows; ++w)   // (rows past nwg lie outside the descriptor and read as zero)
          v[w] = __builtin_amdgcn_raw_buffer_load_b128(rs, (w * a.bstride + s) * (int)sizeof(double), 0,
                                                       kCoherentAux);
#pragma unroll
        for (int w = 1; w < kDirectRows; ++w)
          empty |= is_empty(v[w][0], v[w][1]) || is_empty(v[w][2], v[w][3]);
        if (!empty) break;
        if (it == 0) t0 = wall_clock64();
        __builtin_amdgcn_s_sleep(1);
        if ((it & 15u) == 15u && (aborted(a) || wait_expired(a, t0))) {
          *ok = 0;
          break;
        }
      }
#pragma unroll
      for (int w = 1; w < kDirectRows; ++w) {
        sx += lo_double(v[w][0], v[w][1]);
        sy += lo_double(v[w][2], v[w][3]);
      }
    }
    tv[s] = sx;
    tv[s + 1] = sy;
  }
  __syncthreads();
}

// ---- scalar work of the leader ---------------------------------------------------

// Row r of a table times two vectors (as row_mv, for two right-hand sides).
template <int MODE, bool TR>
__device__ inline void row_mv2(int hi, const double* tab, const double* v, const double* w, int r,
                               double& ov, double& ow) {
  const int s = kp_tid() & 7;
  double av = 0.0, aw = 0.0;
#pragma unroll
  for (int t = 0; t < kMMax / 8; ++t) {
    if (8 * t > hi) break;                     // uniform
    const int k = s + 8 * t;
    const double x = TR ? tab[r * kTabLd + k] : tab[k * kTabLd + r];
    const double xv = x * v[k], xw = x * w[k];
    const bool in = (k <= hi) && ((MODE == 0) ? (k <= r) : (MODE == 1 ? (k < r) : (k > r)));
    if (in) {
      av += xv;
      aw += xw;
    }
  }
  av += dpp_mov<0xB1>(av);
  aw += dpp_mov<0xB1>(aw);
  av += dpp_mov<0x4E>(av);
  aw += dpp_mov<0x4E>(aw);
  av += dpp_mov<0x141>(av);
  aw += dpp_mov<0x141>(aw);
  ov = av;
  ow = aw;
}

// Row c of M^{-1} (compact-WY recursion) and of L from the measured products
// sl of column c with the older ones, appended to the table.
__device__ inline void append_row(LeadB& L, int c, const double* sl, int r, bool row_lead) {
  const double mr = -row_mv<2, true>(c - 1, L.tab, sl, r);
  if (row_lead) {
    if (r < c) {
      L.tab[r * kTabLd + c] = mr - sl[r];
      L.tab[c * kTabLd + r] = sl[r];
    } else if (r == c) {
      L.tab[c * kTabLd + c] = 1.0;
    }
  }
}

// The second Hessenberg column of a pair (column c, subdiagonal divisor
// gamma[c]) and the subdiagonal of the first, once the norms alpha_c and
// alpha_{c+1} are known; lanes i <= c.
__device__ inline void finish_pair_column(LeadB& L, int c, double alc, double aln, int i) {
  const double sc = 1.0 / alc;
  if (i < c) L.H[c * kLdh + i] = sc * L.rp[i];
  if (i == c) {
    L.H[c * kLdh + c] = L.rp[c];
    L.H[c * kLdh + c + 1] = sc * L.gamma[c] * aln;
    L.H[(c - 1) * kLdh + c] = L.gamma[c - 1] * alc;
  }
}

// tv: the reduced sums of step j (four per measured column i < j - na: xa.x_i,
// x.x_i, w1.x_i, w2.x_i with xa = column j - 1, x = column j; then the ten
// products of xa, x, w1, w2).  Stored columns carry unit scales sigma_i as in
// scalar_step; the single-step rules (lagged norm, norm estimate, fallback,
// breakdown) are those of scalar_step.
__device__ __attribute__((always_inline)) inline void block_scalar(const Args& a, int j, int na, int two,
                                                                   const double* tv, LeadB& L, double* wk,
                                                                   Ctl& nx) {
  State* st = a.st;
  Pub* pb = a.pub;
  double* sla = wk;
  double* slj = wk + 72;
  double* sb = wk + 2 * 72;
  double* sq = wk + 3 * 72;
  double* sy = wk + 4 * 72;
  double* syq = wk + 5 * 72;
  double* sp = wk + 6 * 72;
  double* spq = wk + 7 * 72;
  const int i = kp_tid();
  const bool w0 = i < 64;
  const int jo = j - na, ja = j - 1;
  const double* G = tv + 4 * jo;
  const double al = sqrt(G[4]), ala = na ? sqrt(G[0]) : 1.0, cww = G[7];
  if (na && (!(ala > 0.0) || !isfinite(ala))) {
    if (i == 0) {
      nx.status = (int)KP_STATUS_NONFINITE;
      nx.phase = (int)PH_FINISH;
    }
    return;
  }
  if (na && L.pend && w0) finish_pair_column(L, ja, ala, al, i);
  if (!(al > 0.0) || !isfinite(al) || !isfinite(cww)) {
    if (i == 0) {
      if (na) L.sigma[ja] = 1.0 / ala;
      if (j == 0 && al == 0.0) {            // zero start vector: result is zero
        st->zero = 1;
        L.beta = 0.0;
        nx.phase = (int)PH_FINISH;
      } else if (al == 0.0) {               // exact invariance already reached
        L.breakdown = 1;
        nx.m_eff = j;
        nx.upd = 0;
        L.H[(j - 1) * kLdh + j] = 0.0;
        nx.phase = (int)PH_EXPM;
      } else {
        nx.status = (int)KP_STATUS_NONFINITE;
        nx.phase = (int)PH_FINISH;
      }
    }
    return;
  }
  if (j > 0 && L.fallback_cur && al <= a.eps_bd * sqrt(L.wn2[j - 1])) {
    // the exact norm of the vector produced with the fallback is negligible:
    // lucky breakdown at the previous step (this step's products are unused)
    if (i == 0) {
      L.breakdown = 1;
      L.H[(j - 1) * kLdh + j] = 0.0;
      nx.j = j;
      nx.m_eff = j;
      nx.upd = 0;
      nx.phase = (int)PH_EXPM;
    }
    return;
  }
  const double sj = 1.0 / al, sa = 1.0 / ala;
  const double sig = (w0 && i < jo) ? L.sigma[i] : (i == j ? sj : (na && i == ja ? sa : 0.0));
  if (w0) {
    const bool act = i < jo, ia = na && i == ja, ij = i == j;
    const double s = sig * sj;
    sla[i] = act ? sig * sa * tv[4 * i] : 0.0;
    slj[i] = act ? s * tv[4 * i + 1] : (ia ? s * G[1] : 0.0);
    sb[i] = act ? s * tv[4 * i + 2] : (ia ? s * G[2] : (ij ? s * G[5] : 0.0));
    sq[i] = act ? s * tv[4 * i + 3] : (ia ? s * G[3] : (ij ? s * G[6] : 0.0));
  }
  __syncthreads();
  const int r = (kp_tid() >> 6) * 8 + ((kp_tid() & 63) >> 3);
  const bool row_lead = (kp_tid() & 7) == 0;
  if (na) {
    append_row(L, ja, sla, r, row_lead);
    __syncthreads();
  }
  append_row(L, j, slj, r, row_lead);
  __syncthreads();
  double h, q = 0.0;
  if (a.orth == KP_ORTH_H_NCWY) {
    h = sb[r] - row_mv<1, true>(j, L.tab, sb, r);      // T = I - L
  } else {
    double y, yq;
    row_mv2<0, false>(j, L.tab, sb, sq, r, y, yq);     // M^{-1} b (CWY: H)
    h = y;
    if (a.orth == KP_ORTH_H_GSMGS) {
      // p = b - L^T y, then M^{-1} p (Algorithm 7's second sweep)
      if (row_lead) {
        sy[r] = y;
        syq[r] = yq;
      }
      __syncthreads();
      double p, pq;
      row_mv2<2, false>(j, L.tab, sy, syq, r, p, pq);
      if (row_lead) {
        sp[r] = sb[r] - p;
        spq[r] = sq[r] - pq;
      }
      __syncthreads();
      row_mv2<0, false>(j, L.tab, sp, spq, r, h, q);
    }
  }
  if (row_lead) {
    L.h[r] = h;
    L.q[r] = q;
  }
  __syncthreads();
  if (!w0) return;
  const bool in = i <= j;
  const double hi = in ? L.h[i] : 0.0, qi = in ? L.q[i] : 0.0;
  const double b = in ? sb[i] : 0.0, bq = in ? sq[i] : 0.0;
  const double wn2 = cww * sj * sj;
  const double sums = wave_sum4(b * b, b * hi, b * qi, bq * qi);
  const double ss = readlane_d(sums, 0);
  const double est2 = wn2 - ss;
  const int fallback = (est2 <= a.delta * wn2) ? 1 : 0;
  const double gam = fallback ? 1.0 : sqrt(est2);
  const int bd = (!fallback && gam <= a.eps_bd * sqrt(wn2)) ? 1 : 0;
  const bool bad = !isfinite(wave_sum(hi));
  // the second vector of a pair
  int done = 1;
  double e = 0.0, g2 = 1.0;
  if (two) {
    const double n1 = wn2 - readlane_d(sums, 1), n12 = G[8] * sj * sj - readlane_d(sums, 2);
    const double nw2 = G[9] * sj * sj, n22 = nw2 - readlane_d(sums, 3);
    e = n12 / n1;
    const double d2 = n22 - e * n12;
    const bool qok = isfinite(wave_sum(qi));
    if (!bad && !fallback && !bd && est2 > kGuard * wn2 && n1 > 0.0 && qok && isfinite(d2) &&
        d2 > kGuard * nw2) {
      done = 2;
      g2 = sqrt(d2);
    }
  }
  if (in) {
    L.H[j * kLdh + i] = hi;
    cstore(&pb->coef[i], -hi * sig / gam);
    if (done == 2) cstore(&pb->coef2[i], (e * hi - qi) * sig / g2);
  }
  if (i == 0) {
    if (na) L.sigma[ja] = sa;
    L.sigma[j] = sj;
    cstore(&pb->coef[j + 1], sj / gam);
    if (done == 2) {
      cstore(&pb->coef2[j + 1], -e * sj / g2);
      cstore(&pb->coef2[j + 2], sj / g2);
    }
    if (j > 0 && !na) L.H[(j - 1) * kLdh + j] = L.gamma[j - 1] * al;
    L.gamma[j] = gam;
    L.wn2[j] = wn2;
    if (j == 0) L.beta = al;
    L.fallback_cur = fallback;
    L.n_fallback += fallback;
    L.pend = 0;
    if (bad) {
      nx.status = (int)KP_STATUS_NONFINITE;
      nx.phase = (int)PH_FINISH;
    } else if (bd) {
      L.H[j * kLdh + j + 1] = 0.0;
      L.breakdown = 1;
      ++L.arnoldi_steps;
      nx.j = j + 1;
      nx.m_eff = j + 1;
      nx.upd = 0;
      nx.na = 0;
      nx.phase = (int)PH_EXPM;
    } else {
      if (done == 2) {
        L.post = 1;
        L.e = e;
        L.g1 = gam;
        L.gamma[j + 1] = g2 / gam;
        L.wn2[j + 1] = 0.0;   // (read only after a fallback, which ends a pair)
      } else if (two) {
        L.nopair = 1;
      }
      L.arnoldi_steps += done;
      nx.j = j + done;
      nx.m_eff = nx.j;
      nx.upd = done;
      nx.na = done - 1;
      nx.phase = (int)((nx.j >= L.m_target || nx.j >= a.stop_j) ? PH_CLOSE : PH_STEP);
      nx.two = nx.phase == PH_STEP ? pair_ok(a, L, nx.j) : 0;
    }
  }
}

// After the release of a pair's barrier: the raw second Hessenberg column,
// rp = (q - H_{<j} h_{<j} - h_j h) / g1 and rp_{j+1} = e - h_j, needed at the
// next reduction only (finish_pair_column).
__device__ __attribute__((always_inline)) inline void block_post(int j, LeadB& L) {
  if (!L.post) return;   // (uniform: set before the release's barrier)
  const int s = kp_tid() & 7;
  const int r = (kp_tid() >> 6) * 8 + ((kp_tid() & 63) >> 3);
  double acc = 0.0;
#pragma unroll
  for (int t = 0; t < kMMax / 8; ++t) {
    if (8 * t >= j) break;
    const int k = s + 8 * t;
    const double x = L.H[k * kLdh + r] * L.h[k];
    if (k < j && k >= r - 1) acc += x;
  }
  acc += dpp_mov<0xB1>(acc);
  acc += dpp_mov<0x4E>(acc);
  acc += dpp_mov<0x141>(acc);
  const double hj = L.h[j];
  if (s == 0 && r <= j) L.rp[r] = (L.q[r] - acc - hj * L.h[r]) / L.g1;
  if (kp_tid() == 0) L.rp[j + 1] = L.e - hj;
  __syncthreads();
  if (kp_tid() == 0) {
    L.post = 0;
    L.pend = 1;
  }
}

// Close of the Arnoldi process: exact norms of the newest column (nrm2) and,
// after a pair, of the one before it (nrm2a), which complete H.
__device__ __attribute__((always_inline)) inline void block_close(const Args& a, double nrm2, double nrm2a,
                                                                  LeadB& L, Ctl& nx) {
  State* st = a.st;
  const int j = nx.j, c = j - 1;
  const double nrm = sqrt(nrm2), nra = sqrt(nrm2a);
  const bool pair = L.pend != 0;
  __syncthreads();
  if (pair && kp_tid() < 64) finish_pair_column(L, c, nra, nrm, kp_tid());
  if (kp_tid() != 0) return;
  if (pair)
    L.sigma[c] = 1.0 / nra;
  else
    L.H[c * kLdh + j] = L.gamma[c] * nrm;
  L.pend = 0;
  st->last_nrm2 = nrm2;
  nx.upd = 0;
  if (!isfinite(nrm2) || (pair && !(nra > 0.0 && isfinite(nrm2a)))) {
    nx.status = (int)KP_STATUS_NONFINITE;
    nx.phase = (int)PH_FINISH;
    return;
  }
  if (L.fallback_cur && nrm <= a.eps_bd * sqrt(L.wn2[c])) {
    L.H[c * kLdh + j] = 0.0;
    L.breakdown = 1;
  }
  nx.phase = (int)((L.breakdown || j >= L.m_target) ? PH_EXPM : PH_STEP);
  nx.two = nx.phase == PH_STEP ? pair_ok(a, L, j) : 0;
}

}  // namespace kp
