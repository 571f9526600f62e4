// The one-reduction Arnoldi process with a float64 basis, up to kS = 3 steps per
// grid-wide reduction (block steps): streaming passes and the leader's scalar
// work of kernels k_blk and k_batch<double, false, true>.
//
// A step of Algorithm 4 reads the basis twice (inner products, then the
// projection) and synchronises the grid once.  Both costs are shared by kS
// Krylov vectors from one reduction: with x_j the newest column and theta a
// shift (the last diagonal entry of H, which keeps the w_k apart),
//     w_1 = (Atilde - theta) x_j,  w_{k+1} = (Atilde - theta) w_k,
// one pass over the basis forms the inner products of every column with the
// unmeasured columns and with the w_k, and one pass forms the new columns
//     [x_{j+1} .. x_{j+s}] = (W - U C) R^{-1},  C = T U'W,  R'R = W'W - (U'W)'C
// (R upper triangular), with T the GSMGS correction of Algorithm 7 over all
// measured columns.  The Hessenberg columns are exact combinations: with
// Atilde w_k = w_{k+1} + theta w_k and Atilde U_{<j} = U H_{<j} (the columns
// made before),
//     Atilde u_j = U h_j + X R e_1,  h_j = c_1 + theta e_j,
//     Atilde (W - U C)_k = U (c_{k+1} + theta c_k - H_{<j} c_k - c_{kj} h_j)
//                          + X (R_{k+1} + theta R_k - c_{kj} R_1),
// times R^{-1}: the same H as single steps to rounding.  The new columns are
// unmeasured: their norms and products come with the next reduction (the
// lagged norms of Algorithm 4, for s columns).
// Where a w_k lies almost inside the span already there (guard kGuard on the
// squared norms), the columns before it are made and the next block starts
// there; kMaxShort blocks in a row that made one step end the attempts.  The
// forms H-CWY and H-NCWY always take single steps (theta = 0): their one-sided
// corrections do not remove the measured loss of orthogonality to first order,
// which a block needs.
//
// What a block loses: a vector whose norm falls by rho in the projection passes
// 1 / rho of the rounding to the new column, and three of them in a row multiply
// from block to block.  The shift of every product, the first one too, keeps rho
// near the spread of the spectrum whatever its distance from zero; the guard
// bounds what is left (the first block of a process, which has no shift yet,
// smooth start vectors, operators that the tail couples).  Loss of orthogonality on the device, a diagonal at -50 (1 +- 0.05), p = 1,
// 24 columns: 3.7e-14, single steps 2.1e-14, without the shift of the first product
// 8.7e-8.  Error of the 64 x 64 call, 40 steps, against the closed form (mean of 30
// inputs): 1.2e-15, single steps 1.1e-15; 2.1e-15 without that shift and with a
// whole block first.  In a model in numpy,
// 40 random operators with reaction terms up to -500 and 36 columns: at most
// 4.4e-12, 1.6e-13 in the geometric mean; residual ||A V - V H|| / ||H|| on
// diffusion operators, 64 columns, 1e-15 to 2e-15 (single steps 2e-16).  A guard of 1e-3
// takes the mean to 8e-14 and costs a seventeenth block in some processes of 48
// steps (256^2 call 3.05 -> 3.11 ms).  Four steps lose 4e-12 on diffusion operators.
//
// What bounds it: HBM (or Infinity Cache) bytes of the basis at large grids,
// the latency chain of a phase (release, coefficients, halo flags, partial
// sums, scalar work) at small ones.  A sub-tile is R element pairs per thread:
// a workgroup of few elements takes R = 1, with more columns in flight per
// thread for the same registers, instead of lanes that repeat the last pair.
//
// Measured (one call; single steps on workgroups of >= 4096 elements, then two
// steps per reduction, then three): 64 x 64, m = 40 fixed 1576, 708, 622 us;
// 256^2 adaptive (tol 1e-8, m <= 48) 10.48, 5.16, 4.40 ms; 1024^2 Allen-Cahn
// benchmark call 93.7, 59.5, 51.3 ms; 2 x 1000 x 1200 Brusselator 102.3, 66.8,
// 49.8 ms; 512 uneven problems in one launch 1333, 841, 603 ms.  With the
// stencil from LDS and small_dots: 64 x 64 519 us, 256^2 3.75 ms, 512^2 forward
// and backward 39.9 -> 34.6 ms.  With the sections below and the partition of
// krylov_phi.hip: 64 x 64 443 us, 256^2 3.04 ms, 1024^2 44.8, the Brusselator 48.0,
// the 512 problems 595 to 630 (boxes).
#pragma once

#include "kp_leader.h"
#include "kp_passes.h"

namespace kp {

constexpr int kS = 3;                        // steps per reduction at most
constexpr int kNv = 2 * kS;                  // vectors of its products: kS - 1 unmeasured columns, x, kS new ones
constexpr int kGram = kNv * (kNv + 1) / 2;   // products among them
constexpr int kBSlots = kNv * kMMax + 24;    // LDS stride of a wave's sums
constexpr double kGuard = 1e-4;              // a new vector needs ||y||^2 > kGuard ||w||^2
constexpr int kMaxShort = 3;                 // blocks in a row that made one step: then single steps
constexpr double kSmallL = 1e-9;             // below it the correction's second order is under rounding
constexpr int kCoefLd = kMMax + 4;           // coefficients of one new column: basis columns, then the w_k
// Workgroups whose partial rows the leader reads itself; above, each quad of
// slots is summed over the rows by one workgroup first (reduce_quads).
constexpr int kDirectRows = 16;

// Slot of the product of block vectors p <= q (0 .. kS-2 unmeasured columns,
// kS-1 x, then w_1 ..) after the column slots.
__device__ constexpr int gram_at(int p, int q) { return p * kNv - p * (p - 1) / 2 + (q - p); }
__device__ inline int block_slots(int jo) { return kNv * jo + kGram + 1; }   // (even)

// Packed upper Hessenberg matrix: column k holds its k + 2 entries.
__device__ inline int hcol(int k) { return k * (k + 3) / 2; }
struct HessPacked {
  const double* p;
  __device__ double operator()(int i, int k) const { return p[hcol(k) + i]; }
};

// What the leader's serial work reads, in LDS for the whole launch.
struct alignas(16) LeadB {
  double tab[kMMax * kTabLd];      // <u_r, u_k> at [r * kTabLd + k], r != k (L + L')
  double H[kMMax * (kMMax + 3) / 2 + 8];   // Hessenberg, packed (hcol)
  double sigma[kMMax + 8];         // unit scale of column i
  double c[kS][kMMax + 8];         // projections C of the last block
  double rp[kS - 1][kMMax + 8];    // raw Hessenberg columns of its later vectors: rows of U,
  double hx[kS - 1][kS + 1];       // and rows of X
  double rr[6], ri[6];             // R and R^{-1}: 00 01 02 11 12 22
  double beta, wn2, theta, theta_used;
  int fallback_cur, m_target, breakdown, n_fallback, arnoldi_steps, onchip;
  int nopair, big, pend, post;
};

__device__ inline void load_tables_b(const Args& a, LeadB& L, bool resume) {
  const State* st = a.st;
  if (resume) {
    for (int idx = kp_tid(); idx < kMMax * kMMax; idx += kThreads) {
      const int k = idx / kMMax, r = idx - k * kMMax;
      if (r > k) L.tab[k * kTabLd + r] = L.tab[r * kTabLd + k] = st->Lm[(int64_t)k * kLdt + r];
    }
    for (int idx = kp_tid(); idx < kLdh * kMMax; idx += kThreads) {
      const int k = idx / kLdh, r = idx - k * kLdh;
      if (r <= k + 1) L.H[hcol(k) + r] = st->H[idx];
    }
    for (int i = kp_tid(); i < kMMax + 2; i += kThreads) L.sigma[i] = st->sigma[i];
  }
  if (kp_tid() == 0) {
    L.beta = st->beta;
    L.wn2 = st->wn2[0];
    L.rr[0] = st->gamma[0];
    L.theta = st->theta;
    L.fallback_cur = st->fallback_cur;
    L.m_target = st->m_target;
    L.breakdown = st->breakdown;
    L.n_fallback = st->n_fallback;
    L.arnoldi_steps = st->arnoldi_steps;
    L.onchip = st->onchip;
    L.nopair = st->nopair >> 1;
    L.big = st->nopair & 1;
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
      st->Lm[(int64_t)k * kLdt + r] = (r > k && r <= j) ? L.tab[r * kTabLd + k] : 0.0;
    }
    for (int idx = kp_tid(); idx < kLdh * kMMax; idx += kThreads) {
      const int k = idx / kLdh, r = idx - k * kLdh;
      st->H[idx] = (k < j && r <= k + 1) ? L.H[hcol(k) + r] : 0.0;
    }
    for (int i = kp_tid(); i < kMMax + 2; i += kThreads) st->sigma[i] = L.sigma[i];
  }
  if (kp_tid() == 0) {
    st->beta = L.beta;
    st->wn2[0] = L.wn2;
    st->gamma[0] = L.rr[0];
    st->theta = L.theta;
    st->fallback_cur = L.fallback_cur;
    st->breakdown = L.breakdown;
    st->n_fallback = L.n_fallback;
    st->arnoldi_steps = L.arnoldi_steps;
    st->onchip = L.onchip;
    st->nopair = (L.nopair << 1) | L.big;
  }
}

// Steps the phase that continues from column j makes.
__device__ inline int block_steps(const Args& a, const LeadB& L, int j) {
  if (!a.pairs || L.nopair >= kMaxShort) return 1;
  return max(1, min(kS, min(L.m_target, a.stop_j) - j));
}
// ... and the first phase of a run of steps from column j (no update pending): two
// where the run is no multiple of three (16 = 2 + 3 + 3 + 3 + 3 + 2, as many phases
// as whole blocks first).  The first block of a process has no shift yet, and a
// smooth start vector often lets it make only two; the last block's free place
// takes a step that the guard puts off on the way.  All of the remainder first
// reads 2 % fewer columns and has no such place: 1024^2 call 44.5 ms against
// 44.8, but EPI4 steps of Allen-Cahn at 100^2 to 256^2 6 % longer (a phase more).
__device__ inline int first_steps(const Args& a, const LeadB& L, int j) {
  const int n = block_steps(a, L, j), left = min(L.m_target, a.stop_j) - j;
  return (n == kS && left % kS) ? kS - 1 : n;
}
// (The shift starts from 0: the last one of the substep before belongs to the
// end of its process, and the first vectors of this one are smooth.)
__device__ inline void new_process(const Args& a, LeadB& L) {
  L.nopair = L.big = 0;
  L.theta = 0.0;
  cstore(&a.pub->shift, 0.0);
}
__device__ inline double beta_of(const Args&, const LeadB& L) { return L.beta; }
__device__ inline HessPacked hess_of(const Args&, const LeadB& L) { return HessPacked{L.H}; }

// ---- passes ------------------------------------------------------------------
//
// On chip (keep_xw; one plane, at most kKeepMax elements per workgroup): the
// vector the next product multiplies (x_j, then the w_k but the last) sits in
// LDS between its two halo rows, so the stencil is five LDS reads at fixed
// offsets for every product of a phase.  Afterwards the last w takes its place.
// Up to 1024 elements (R = 1) the other vectors of the block sit in LDS too
// (kSmallVec each, after the halo row: x_{j-2}, x_{j-1}, x_j, w_1, w_2).  Above, the w
// before the last one takes the space of the leader's tables, which the other
// workgroups do not use (the leader keeps it in memory), and the first of three
// is in memory.
constexpr int kSmallVec = 2 * kThreads;
// (first of the five vectors: R = 1 has n <= kSmallVec and so nx <= kSmallVec)
__device__ inline double* small_vec(double* hl, int q) { return hl + kHaloCap - (5 - q) * kSmallVec; }

// ---- tagged exchange (ll) ---------------------------------------------------------
//
// Between small workgroups an exchange of halo rows is all latency: the rows are
// stored, the stores awaited, the flag stored, the flags polled, the rows loaded.
// Where rows are short (at most 256, and 1024 elements per workgroup) every double
// of a halo row, and of the tail, goes as two 8-byte words that carry half of it
// and a 32-bit tag each, and the reader polls the words themselves (8-byte
// accesses are single).  64 x 64 call 466 -> 446 us, 256^2 3.10 -> 3.05 ms; at rows
// of 512 the doubled bytes cost 3 %.  The tag is 4k + e for vector e of phase k;
// the buffers are cleared before each call.  Vector e goes through buffer e & 1:
// a neighbour that has sent vector e + 1 has read e, and the barrier separates
// the phases.  Phases without an update read the plain rows, which the stage,
// close and combine phases publish.

__device__ inline int64_t ll_doubles(const Args& a) { return (int64_t)a.nwg * 4 * a.nx; }   // one buffer, one plane
__device__ inline unsigned long long* ll_at(const Args& a, int e, int64_t i) {
  return reinterpret_cast<unsigned long long*>(a.hx2) + (e & 1) * ll_doubles(a) + 2 * i;
}
__device__ inline unsigned long long* ll_tail(const Args& a) {
  return reinterpret_cast<unsigned long long*>(a.hx2) + 2 * ll_doubles(a);
}
__device__ inline void ll_store(unsigned long long* p, double v, unsigned tag) {
  const unsigned long long t = (unsigned long long)tag << 32;
  cstore(p, t | (unsigned)__double2loint(v));
  cstore(p + 1, t | (unsigned)__double2hiint(v));
}
// Two values (the rows above and below), polled together until both are there.
__device__ inline void ll_load2(const Args& a, const unsigned long long* p, const unsigned long long* q,
                                unsigned tag, double& u, double& v) {
  int64_t t0 = 0;
  for (unsigned it = 0;; ++it) {
    const unsigned long long p0 = cload(p), p1 = cload(p + 1), q0 = cload(q), q1 = cload(q + 1);
    if ((unsigned)(p0 >> 32) == tag && (unsigned)(p1 >> 32) == tag && (unsigned)(q0 >> 32) == tag &&
        (unsigned)(q1 >> 32) == tag) {
      u = __hiloint2double((int)(unsigned)p1, (int)(unsigned)p0);
      v = __hiloint2double((int)(unsigned)q1, (int)(unsigned)q0);
      return;
    }
    if (it == 0) t0 = wall_clock64();
    if ((it & 31u) == 31u && (aborted(a) || wait_expired(a, t0))) {
      u = v = 0.0;
      return;
    }
  }
}
// The pair (e, e + 1) of the one plane, as publish_pair.
__device__ inline void ll_publish_pair(const Args& a, const Seg& sg, int64_t e, double v0, double v1, int ev,
                                       unsigned tag) {
  const int64_t n = sg.end - sg.beg;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t off = e - sg.beg + h;
    const double v = h ? v1 : v0;
    if (off >= n) continue;
    if (off < a.nx) ll_store(ll_at(a, ev, halo_at(a, wg_rank(a), 0, 0, (int)off)), v, tag);
    if (off >= n - a.nx) ll_store(ll_at(a, ev, halo_at(a, wg_rank(a), 0, 1, (int)(off - (n - a.nx)))), v, tag);
  }
}

template <int R>
__device__ inline void tile_pairs_r(int64_t q0, int64_t pend, uint32_t* lo, bool* ok) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t q = q0 + (int64_t)r * kThreads + kp_tid();
    ok[r] = q < pend;
    lo[r] = (uint32_t)(2 * ((ok[r] ? q : pend - 1) - q0));
  }
}
// Whether this wave has a pair in the sub-tile (a wave without one skips it).
__device__ inline bool wave_in_tile(int64_t q0, int64_t pend) {
  return __builtin_amdgcn_readfirstlane((int)(q0 + (kp_tid() & ~63) < pend)) != 0;
}

// Basis columns per chunk: the linear combinations keep 16 to 20 pair loads
// in flight per thread, the inner products two chunks of 8.
template <int R> constexpr int kUpdCols = R == 1 ? 16 : 20 / R;
template <int R> constexpr int kDotCols = 8 / R;

// acc[l] += sum_i cf[l][i] V_i over the columns i0, i0 + step, ... (nc of
// them; the columns past nc repeat the last one with coefficient 0, so that
// all loads issue before the first multiply-add); cf in LDS, stride kCoefLd.
template <int R, int C, int U>
__device__ inline void axpy_block(const double* V, int64_t ld, int64_t t0, int i0, int step, int nc,
                                  const double* cf, const uint32_t* lo, double2 (&acc)[U][R]) {
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
#pragma unroll
    for (int l = 0; l < U; ++l) {
      const double w = (c < nc) ? cf[l * kCoefLd + i] : 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        acc[l][r].x = __builtin_fma(w, v[c][r].x, acc[l][r].x);
        acc[l][r].y = __builtin_fma(w, v[c][r].y, acc[l][r].y);
      }
    }
  }
}

// Published coefficients (kS columns) and the shift to LDS: one coherent round
// trip.
__device__ inline void load_coefs(const Args& a, double* cf) {
  const int t = kp_tid();
  if (t < kS * kCoefLd) {
    const int l = t / kCoefLd, i = t - l * kCoefLd;
    cf[t] = cload(&a.pub->coefs[l][min(i, kMMax + 1)]);
  } else if (t == kS * kCoefLd) {
    cf[t] = cload(&a.pub->shift);
  }
  __syncthreads();
}

// The tails (p <= 8 entries per column) of the U new columns: lane i of the
// last wave of workgroup 0 takes column i; the newest one is published.
template <int U>
__device__ inline void tail_update_b(const Args& a, double* V, int nc, const double* cf, unsigned tag, double (&ss)[U]) {
  const int t = kp_tid() & 63;
  const int64_t T0 = a.tail_off, ld = a.ld;
  double p[U][kPMax];
#pragma unroll
  for (int l = 0; l < U; ++l)
#pragma unroll
    for (int k = 0; k < kPMax; ++k) p[l][k] = 0.0;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int i = t + 64 * hh;
    const bool on = i < nc + U;
    const double* vc = V + (int64_t)(on ? i : 0) * ld + T0;
    double w[U];
#pragma unroll
    for (int l = 0; l < U; ++l) w[l] = (i <= nc + l) ? cf[l * kCoefLd + min(i, kCoefLd - 1)] : 0.0;
#pragma unroll
    for (int k = 0; k < kPMax; ++k)
      if (k < a.p && on) {
        const double v = vc[k];
#pragma unroll
        for (int l = 0; l < U; ++l) p[l][k] += w[l] * v;
      }
  }
#pragma unroll
  for (int k = 0; k < kPMax; ++k) {
    if (k < a.p) {
#pragma unroll
      for (int l = 0; l < U; ++l) {
        const double y = wave_sum(p[l][k]);
        if (t == 0) {
          V[(int64_t)(nc + l) * ld + T0 + k] = y;
          if (l == U - 1) {
            cstore(a.tx + k, y);
            if (tag) ll_store(ll_tail(a) + 2 * k, y, tag);
          }
          ss[l] += y * y;
        }
      }
    }
  }
}

// The U pending columns j - U + 1 .. j (column l: weights cf[l] on the columns
// 0 .. j - U, then on w_1 .. w_{l+1}), in place of the w_k.  pns: vectors the
// previous phase made (>= U), which says where keep_xw left them (wbuf: the
// workgroup's second buffer, null in the leader).  keep_xw also leaves x_j in
// LDS.  tag: of the tagged exchange, 0 for plain halo rows.  The halo rows of x_j are published.  want_norm:
// partial slot l = the squared norm of new column l.
template <int R, int U>
__device__ __attribute__((always_inline)) inline void update_block(const Args& a, int j, int pns, const double* cf,
                                                                   double* hl, const double* wbuf, double* red,
                                                                   bool want_norm, unsigned tag) {
  double* V = reinterpret_cast<double*>(a.V);
  const int64_t ld = a.ld;
  const int nc = j - U + 1;
  const bool keep = a.keep_xw != 0;
  const bool small = R == 1 && keep;   // (every vector of the block in LDS)
  double2* X2 = reinterpret_cast<double2*>(hl + keep_off(a));
  const double2* W2 = reinterpret_cast<const double2*>(wbuf);
  const Rows o = own_rows(a);
  double ss[U];
#pragma unroll
  for (int l = 0; l < U; ++l) ss[l] = 0.0;
  if (wg_rank(a) == 0 && kp_tid() >= kThreads - 64) tail_update_b<U>(a, V, nc, cf, tag, ss);
  constexpr int C = kUpdCols<R>;
  for (int si = 0; si < num_segs(a); ++si) {
    const Seg sg = seg_at(a, o, si);
    const int64_t pbeg = sg.beg >> 1, pend = (sg.end + 1) >> 1;
    for (int64_t q0 = pbeg; q0 < pend; q0 += (int64_t)kThreads * R) {
      if (!wave_in_tile(q0, pend)) break;
      const int64_t t0 = 2 * q0;
      uint32_t lo[R];
      bool ok[R];
      tile_pairs_r<R>(q0, pend, lo, ok);
      double2 acc[U][R];
#pragma unroll
      for (int l = 0; l < U; ++l)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[l][r] = make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const double* wcol = V + (int64_t)(nc + k) * ld + t0;
        const int slot = (int)(q0 - pbeg) + kp_tid();
#pragma unroll
        for (int r = 0; r < R; ++r) {
          double2 w;
          if (keep && k == pns - 1) {
            w = X2[slot + r * kThreads];
            if (t0 + lo[r] + 1 >= sg.end) w.y = 0.0;   // (a halo row follows an odd end)
          } else if (small) {
            w = reinterpret_cast<const double2*>(small_vec(hl, kS + k))[slot + r * kThreads];
          } else if (keep && k == pns - 2 && wbuf) {
            w = W2[slot + r * kThreads];
          } else {
            w = Pair<double>::load(wcol + lo[r]);
          }
#pragma unroll
          for (int l = k; l < U; ++l) {
            const double c = cf[l * kCoefLd + nc + k];
            acc[l][r].x = __builtin_fma(c, w.x, acc[l][r].x);
            acc[l][r].y = __builtin_fma(c, w.y, acc[l][r].y);
          }
        }
      }
      for (int i1 = nc - 1; i1 >= 0; i1 -= C)
        axpy_block<R, C, U>(V, ld, t0, i1, -1, min(C, i1 + 1), cf, lo, acc);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (ok[r]) {
#pragma unroll
          for (int l = 0; l < U; ++l) {
            Pair<double>::store(V + (int64_t)(nc + l) * ld + t0 + lo[r], acc[l][r].x, acc[l][r].y);
            ss[l] += acc[l][r].x * acc[l][r].x + acc[l][r].y * acc[l][r].y;
          }
          const double2 x = acc[U - 1][r];
          if (keep) X2[(int)(q0 - pbeg) + kp_tid() + r * kThreads] = x;
          if (small)
#pragma unroll
            for (int l = 0; l < U; ++l)
              reinterpret_cast<double2*>(small_vec(hl, kS - U + l))[kp_tid()] = acc[l][r];
          if (R == 1 && tag)
            ll_publish_pair(a, sg, t0 + lo[r], x.x, x.y, 0, tag);
          else
            publish_pair(a, a.hx, sg, t0 + lo[r], x.x, x.y);
        }
      }
    }
  }
  if (want_norm) {
    double* pr = a.part + (int64_t)wg_rank(a) * kCStride;
#pragma unroll
    for (int l = 0; l < U; ++l) {
      const double s = block_sum(ss[l], red);
      if (kp_tid() == 0) cstore(pr + l, s);
    }
  }
}

// Products of C columns with the block's vectors, put into (ACC: added to) the
// wave's row of sacc.  FULL: all kNv; else only x and w_1 (a single step after a
// single step), in the same slots.  A whole chunk is one straight line, so that
// the reductions of its columns overlap.
template <int R, int C, bool FULL, bool ACC>
__device__ inline void dots_block(const double2 (&v)[C][R], const double2 (&b)[kNv][R], int i0, int nc,
                                  double* sacc) {
  const int lane = kp_tid() & 63;
  double* srow = sacc + (kp_tid() >> 6) * kBSlots + kNv * i0;
  auto put = [](double* p, double x) { *p = ACC ? *p + x : x; };
  auto column = [&](int c) {
    double s[kNv];
#pragma unroll
    for (int q = 0; q < kNv; ++q) {
      s[q] = 0.0;
      if (FULL || q == kS - 1 || q == kS) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          s[q] = __builtin_fma(v[c][r].y, b[q][r].y, __builtin_fma(v[c][r].x, b[q][r].x, s[q]));
      }
    }
    if constexpr (FULL) {
      const double s4 = wave_sum4(s[0], s[1], s[2], s[3]), s2 = wave_sum2(s[4], s[5]);
      if (lane < 4) put(srow + kNv * c + lane, s4);
      if (lane < 2) put(srow + kNv * c + 4 + lane, s2);
    } else {
      const double s2 = wave_sum2(s[kS - 1], s[kS]);
      if (lane < 2) put(srow + kNv * c + kS - 1 + lane, s2);
    }
  };
  if (nc == C) {
#pragma unroll
    for (int c = 0; c < C; ++c) column(c);
  } else {
#pragma unroll
    for (int c = 0; c < C - 1; ++c)
      if (c < nc) column(c);
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

// The older columns of one sub-tile, double-buffered chunks (the first one is
// in flight in va already).
template <int R, bool FULL, bool ACC>
__device__ __attribute__((always_inline)) inline void columns_block(
    const double* V, int64_t ld, int64_t t0, int jo, const uint32_t* lo, const double2 (&b)[kNv][R],
    double2 (&va)[kDotCols<R>][R], double* sacc) {
  constexpr int C = kDotCols<R>;
  double2 vb[C][R];
  for (int i0 = 0; i0 < jo; i0 += 2 * C) {
    const int i1 = i0 + C;
    if (i1 < jo) load_block<R, C>(V, ld, t0, i1, min(C, jo - i1), lo, vb);
    dots_block<R, C, FULL, ACC>(va, b, i0, min(C, jo - i0), sacc);
    if (i1 >= jo) break;
    const int i2 = i1 + C;
    if (i2 < jo) load_block<R, C>(V, ld, t0, i2, min(C, jo - i2), lo, va);
    dots_block<R, C, FULL, ACC>(vb, b, i1, min(C, jo - i1), sacc);
  }
}

// The same products where all vectors of the block sit in LDS (R = 1, n <=
// kSmallVec elements): wave by wave a column of its own, 4 pairs per lane, so
// each column is reduced by one wave once (twice above 512 elements) instead
// of by every wave: the reductions, about 70 instructions each on a lone wave
// per SIMD, were what these workgroups spent their time on (64 x 64, 512
// elements: 0.33 us per column before, 0.1 after).  The loads of
// two columns are in flight while two are reduced.
__device__ __attribute__((always_inline)) inline void small_dots(const Args& a, int64_t beg, int n, int j, int jo,
                                                                 int ns, bool full, double* hl, double* srow) {
  const double* V = reinterpret_cast<const double*>(a.V) + beg;
  const int64_t ld = a.ld;
  const int lane = kp_tid() & 63, wv = __builtin_amdgcn_readfirstlane(kp_tid() >> 6);
  const int np = (n + 1) >> 1;
  const double* xl = hl + keep_off(a);
  for (int h = 0; h * 256 < np; ++h) {
    int e[4];
    bool ok[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = h * 256 + r * 64 + lane;
      ok[r] = q < np;
      e[r] = 2 * min(q, np - 1);
    }
    auto load = [&](int i, double2 (&v)[2][4]) {   // columns i, i + kWaves
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double* vc = uniform_ptr(V + (int64_t)min(i + c * kWaves, max(jo - 1, 0)) * ld);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[c][r] = load_at(vc, (uint32_t)e[r] * 8u);
      }
    };
    double2 va[2][4], vb[2][4];
    if (wv < jo) load(wv, va);
    double2 b[kNv][4];
#pragma unroll
    for (int q = 0; q < kNv; ++q) {
      const bool on = q < kS ? (q == kS - 1 || j - (kS - 1) + q >= jo) : (q - kS < ns);
      const bool last = q - kS == ns - 1;
      const double* src = last ? xl : small_vec(hl, min(q, 4));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 x = on ? *reinterpret_cast<const double2*>(src + e[r]) : make_double2(0.0, 0.0);
        b[q][r] = make_double2(ok[r] ? x.x : 0.0, (ok[r] && e[r] + 1 < n) ? x.y : 0.0);
      }
    }
    // products among the block's vectors: four per wave
    if (wv * 4 < kGram) {
      double g[4] = {0.0, 0.0, 0.0, 0.0};
      int id = 0;
#pragma unroll
      for (int p = 0; p < kNv; ++p)
#pragma unroll
        for (int q = p; q < kNv; ++q, ++id)
          if ((id >> 2) == wv) {
            double s = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) s = __builtin_fma(b[p][r].y, b[q][r].y, __builtin_fma(b[p][r].x, b[q][r].x, s));
            g[id & 3] = s;
          }
      const double s = wave_sum4(g[0], g[1], g[2], g[3]);
      if (lane < 4 && wv * 4 + lane < kGram) srow[kNv * jo + wv * 4 + lane] += s;
    }
    auto dots = [&](int i, const double2 (&v)[2][4]) {
      if (!full) {   // x and w_1 alone (a single step after a single step)
        double s[2][2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            s[c][q] = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r)
              s[c][q] = __builtin_fma(v[c][r].y, b[kS - 1 + q][r].y,
                                      __builtin_fma(v[c][r].x, b[kS - 1 + q][r].x, s[c][q]));
          }
        const double t = wave_sum4(s[0][0], s[0][1], s[1][0], s[1][1]);
        if (lane < 2 || (lane < 4 && i + kWaves < jo))
          srow[kNv * (i + (lane >> 1) * kWaves) + kS - 1 + (lane & 1)] += t;
        return;
      }
      double s[2][kNv];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < kNv; ++q) {
          s[c][q] = 0.0;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            s[c][q] = __builtin_fma(v[c][r].y, b[q][r].y, __builtin_fma(v[c][r].x, b[q][r].x, s[c][q]));
        }
      const double t0 = wave_sum4(s[0][0], s[0][1], s[0][2], s[0][3]);
      const double t1 = wave_sum4(s[1][0], s[1][1], s[1][2], s[1][3]);
      const double t2 = wave_sum4(s[0][4], s[0][5], s[1][4], s[1][5]);
      if (lane < 4) {
        const bool two = i + kWaves < jo;
        srow[kNv * i + lane] += t0;
        if (two) srow[kNv * (i + kWaves) + lane] += t1;
        if (lane < 2)
          srow[kNv * i + 4 + lane] += t2;
        else if (two)
          srow[kNv * (i + kWaves) + 2 + lane] += t2;
      }
    };
    for (int i = wv; i < jo; i += 4 * kWaves) {
      if (i + 2 * kWaves < jo) load(i + 2 * kWaves, vb);
      dots(i, va);
      if (i + 2 * kWaves >= jo) break;
      if (i + 4 * kWaves < jo) load(i + 4 * kWaves, va);
      dots(i + 2 * kWaves, vb);
    }
  }
}

// All products of one sub-tile.
template <int R, bool ACC>
__device__ __attribute__((always_inline)) inline void tile_dots(const double* V, int64_t ld, int64_t t0, int jo,
                                                                bool full, const uint32_t* lo,
                                                                const double2 (&b)[kNv][R],
                                                                double2 (&va)[kDotCols<R>][R], double* sacc) {
  const int lane = kp_tid() & 63;
  {
    double* srow = sacc + (kp_tid() >> 6) * kBSlots + kNv * jo;
    double g[kGram + 3];
#pragma unroll
    for (int p = 0; p < kNv; ++p)
#pragma unroll
      for (int q = p; q < kNv; ++q) {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r)
          s = __builtin_fma(b[p][r].y, b[q][r].y, __builtin_fma(b[p][r].x, b[q][r].x, s));
        g[gram_at(p, q)] = s;
      }
#pragma unroll
    for (int k = kGram; k < kGram + 3; ++k) g[k] = 0.0;
#pragma unroll
    for (int k = 0; k < kGram; k += 4) {
      const double s = wave_sum4(g[k], g[k + 1], g[k + 2], g[k + 3]);
      if (lane < 4 && k + lane < kGram) srow[k + lane] = ACC ? srow[k + lane] + s : s;
    }
  }
  if (full)
    columns_block<R, true, ACC>(V, ld, t0, jo, lo, b, va, sacc);
  else
    columns_block<R, false, ACC>(V, ld, t0, jo, lo, b, va, sacc);
}

// Tail rows of a block step (the last wave of workgroup 0, while the others
// wait for their neighbours' halo rows): t_{k+1} = (K - theta) t_k from t_0 = x
// (upward shift within each block of pb entries), stored, and their products
// (column t by lane t; those of the block's vectors by lane 0), in ts.
__device__ inline void tail_block(const Args& a, int j, int na, int ns, double theta, double* ts) {
  const int t = kp_tid() & 63;
  double* V = reinterpret_cast<double*>(a.V);
  const int64_t T0 = a.tail_off, ld = a.ld;
  const int p = a.p, jo = j - na;
  double b[kNv][kPMax];
#pragma unroll
  for (int q = 0; q < kS; ++q) {
    const int col = j - (kS - 1) + q;        // column of vector q; x is q = kS - 1
    const bool on = q == kS - 1 || col >= jo;
    const double* src = (j == 0 ? a.u : V + (int64_t)max(col, 0) * ld) + T0;
#pragma unroll
    for (int k = 0; k < kPMax; ++k) b[q][k] = (on && k < p) ? src[k] : 0.0;
  }
#pragma unroll
  for (int s = 0; s < kS; ++s) {
#pragma unroll
    for (int k = 0; k < kPMax; ++k) {
      const double up = (k + 1 < kPMax && tail_shift_in(a, k)) ? b[kS - 1 + s][(k + 1) % kPMax] : 0.0;
      b[kS + s][k] = (s < ns) ? up - theta * b[kS - 1 + s][k] : 0.0;
      if (t == 0 && k < p && s < ns) V[(int64_t)(j + 1 + s) * ld + T0 + k] = b[kS + s][k];
    }
  }
  if (t == 0 && j == 0)
#pragma unroll
    for (int k = 0; k < kPMax; ++k)
      if (k < p) V[T0 + k] = b[kS - 1][k];
  if (t < jo) {
    const double* vc = V + (int64_t)t * ld + T0;
    double s[kNv];
#pragma unroll
    for (int q = 0; q < kNv; ++q) s[q] = 0.0;
#pragma unroll
    for (int k = 0; k < kPMax; ++k)
      if (k < p) {
        const double v = vc[k];
#pragma unroll
        for (int q = 0; q < kNv; ++q) s[q] += v * b[q][k];
      }
#pragma unroll
    for (int q = 0; q < kNv; ++q) ts[kNv * t + q] = s[q];
  }
  if (t == 0) {
#pragma unroll
    for (int g = 0; g < kNv; ++g)
#pragma unroll
      for (int q = g; q < kNv; ++q) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < kPMax; ++k) s += b[g][k] * b[q][k];
        ts[kNv * jo + gram_at(g, q)] = s;
      }
    ts[kNv * jo + kGram] = 0.0;
  }
}

// Tail entries of x over mu, then of the next products: tt[c] multiplies
// b_{pb-c} in Atilde v for the vector v whose tail it is.
__device__ inline void tail_of_x(const Args& a, int plane, double inv_mu, double* tt) {
  const int toff = (a.tangent && plane == 1) ? a.pb : 0;
#pragma unroll
  for (int c = 0; c < kPMax; ++c) tt[c] = (c < a.pb) ? cload(a.tx + toff + c) * inv_mu : 0.0;
}
__device__ inline void tail_next(const Args& a, double shift, double* tt) {
#pragma unroll
  for (int c = 0; c < kPMax; ++c)
    tt[c] = ((c + 1 < kPMax && c + 1 < a.pb) ? tt[(c + 1) % kPMax] : 0.0) - shift * tt[c];
}

// The block step from column j: w_1 .. w_ns and the partial sums of the
// reduction.  na: unmeasured columns before x_j.  upd: the update of this
// phase has left x_j in LDS and published its halo rows.  The rows of w_k the
// neighbours need go through the two halo buffers in turn (a neighbour has read
// the rows of w_{k-1} before it publishes w_k, which this workgroup has seen
// before it publishes w_{k+1}) and the same flags (value 4k + e; the update
// published 4k).
//
// On chip.  What a product costs here is latency, not bytes: the fields, the
// neighbour offsets and the first columns of B are read once per phase, before
// the wait for the halo rows, and kept in registers.
template <int R>
__device__ __attribute__((always_inline)) inline void matvec_keep(const Args& a, int j, int na, int ns, bool upd,
                                                                  double theta, double inv_mu, double* sacc,
                                                                  double* hl, double* wbuf, unsigned k) {
  double* V = reinterpret_cast<double*>(a.V);
  const int64_t ld = a.ld;
  const Rows o = own_rows(a);
  const int jo = j - na, nx = a.nx;
  constexpr int C = kDotCols<R>;
  constexpr int kBc = R == 1 ? 4 : 2;          // columns of B kept in registers
  double* xcol = V + (int64_t)j * ld;
  const Seg sg = seg_at(a, o, 0);
  const int64_t pend = (sg.end + 1) >> 1, pbeg = sg.beg >> 1;
  const int n = (int)(sg.end - sg.beg);
  double* X = hl + keep_off(a);                // own elements; row r0 - 1 before, row r1 after
  if (!upd) {
    const double* src = j == 0 ? a.u : xcol;
    for (int64_t q = pbeg + kp_tid(); q < pend; q += kThreads) {
      const double2 v = Pair<double>::load(src + 2 * q);
      X[2 * (q - pbeg)] = v.x;
      if (2 * q + 1 < sg.end) X[2 * (q - pbeg) + 1] = v.y;
      if (j == 0) Pair<double>::store(xcol + 2 * q, v.x, v.y);
    }
  }
  // per pair: own offset (-1: none), wrapped east / west offsets of both
  // elements, diagonal factor, columns of B
  int e0[R], off[R][4];
  double2 dg[R], bc[kBc][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int e = 2 * (r * kThreads + kp_tid());
      const int c = min(e, n - 1);             // (a lane without a pair repeats the last element)
      const int64_t g = sg.beg + c;
      const bool v1 = c + 1 < n;
      const int64_t g1 = v1 ? g + 1 : g;
      e0[r] = e < n ? c : -1;
      const int row = (int)((unsigned)c / (unsigned)nx), ix = c - row * nx;
      const bool last = ix == nx - 1;
      const int c1 = v1 ? c + 1 : c, ix1 = v1 ? (last ? 0 : ix + 1) : ix;
      off[r][0] = last ? c - ix : c + 1;
      off[r][1] = ix == 0 ? c + nx - 1 : c - 1;
      off[r][2] = ix1 == nx - 1 ? c1 - ix1 : c1 + 1;
      off[r][3] = ix1 == 0 ? c1 + nx - 1 : c1 - 1;
      const double u0 = a.f0 ? a.f0[g] : 0.0, u1 = a.f0 ? a.f0[g1] : 0.0;
      if (a.kind == KP_OP_ADR)
        dg[r] = make_double2(a.react + u0, a.react + u1);
      else
        dg[r] = make_double2(__builtin_fma(-3.0 * u0, u0, 1.0), __builtin_fma(-3.0 * u1, u1, 1.0));
#pragma unroll
      for (int b = 0; b < kBc; ++b)
        if (b < a.pb) {
          const double* col = a.B + (int64_t)(a.pb - b) * a.ldb;
          bc[b][r] = make_double2(col[g], col[g1]);
        }
    }
  double tt[kPMax];
  const bool ll = R == 1 && a.ll;
  if (upd && !ll) {
    flag_wait_neighbours(a, 4 * k);
    KP_TS(a, k, 2);
  }
  const int bb = wg_rank(a);
  const int wn = (o.r1 == a.ny) ? 0 : bb + 1, ws = (o.r0 == 0) ? a.nwg - 1 : bb - 1;
  auto stage = [&](const double* hx) {
    for (int ix = kp_tid(); ix < nx; ix += kThreads) {
      const double vn = cload(hx + halo_at(a, wn, 0, 0, ix)), vs = cload(hx + halo_at(a, ws, 0, 1, ix));
      X[n + ix] = vn;
      X[ix - nx] = vs;
    }
    __syncthreads();
  };
  auto stage_ll = [&](int e) {
    for (int ix = kp_tid(); ix < nx; ix += kThreads) {
      double vn, vs;
      ll_load2(a, ll_at(a, e, halo_at(a, wn, 0, 0, ix)), ll_at(a, e, halo_at(a, ws, 0, 1, ix)), 4 * k + e, vn, vs);
      X[n + ix] = vn;
      X[ix - nx] = vs;
    }
    __syncthreads();
  };
  if (ll && upd) {
    stage_ll(0);
    KP_TS(a, k, 2);
    // (lane c polls entry c; the wave takes it from there)
    double t = 0.0, t2;
    const int c0 = kp_tid() & 63;
    if (c0 < a.pb) ll_load2(a, ll_tail(a) + 2 * c0, ll_tail(a) + 2 * c0, 4 * k, t, t2);
#pragma unroll
    for (int c = 0; c < kPMax; ++c) tt[c] = (c < a.pb) ? readlane_d(t, c) * inv_mu : 0.0;
  } else {
    tail_of_x(a, 0, inv_mu, tt);
    stage(a.hx);
  }
  for (int s = 0; s < ns; ++s) {
    const bool last = s + 1 == ns;
    double2 w[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int c = max(e0[r], 0);
        const bool v1 = e0[r] >= 0 && c + 1 < n;
        const int c1 = v1 ? c + 1 : c;
        auto at = [&](int cc, int ie, int iw, double d) {
          const double x = X[cc], xe = X[ie], xw = X[iw], xn = X[cc + nx], xs = X[cc - nx];
          const double lap = __builtin_fma(a.cx, __builtin_fma(-2.0, x, xe + xw),
                                           a.cy * __builtin_fma(-2.0, x, xn + xs));
          const double adv = __builtin_fma(a.adx, xe - xw, a.ady * (xn - xs));
          return __builtin_fma(d - theta, x, a.kind == KP_OP_ADR ? lap + (a.transpose ? adv : -adv) : lap);
        };
        double y0 = at(c, off[r][0], off[r][1], dg[r].x);
        double y1 = at(c1, off[r][2], off[r][3], dg[r].y);
#pragma unroll
        for (int b = 0; b < kBc; ++b)
          if (b < a.pb) {
            y0 = __builtin_fma(tt[b], bc[b][r].x, y0);
            y1 = __builtin_fma(tt[b], bc[b][r].y, y1);
          }
        for (int b = kBc; b < a.pb; ++b) {
          const double* col = a.B + (int64_t)(a.pb - b) * a.ldb + sg.beg;
          double tb = tt[kPMax - 1];
#pragma unroll
          for (int q = kBc; q < kPMax - 1; ++q) tb = b == q ? tt[q] : tb;
          y0 = __builtin_fma(tb, col[c], y0);
          y1 = __builtin_fma(tb, col[c1], y1);
        }
        w[r] = make_double2(e0[r] >= 0 ? y0 : 0.0, v1 ? y1 : 0.0);
      }
    __syncthreads();   // every read of X is done
    double* const hxs = (s & 1) ? a.hx : a.hx2;
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (e0[r] >= 0) {
          const int c = e0[r];
          X[c] = w[r].x;
          if (c + 1 < n) X[c + 1] = w[r].y;
          if (!last) {
            if (ll)
              ll_publish_pair(a, sg, sg.beg + c, w[r].x, w[r].y, s + 1, 4 * k + 1 + s);
            else
              publish_pair(a, hxs, sg, sg.beg + c, w[r].x, w[r].y);
            // its place for the inner products and the next update
            if (R == 1)
              *reinterpret_cast<double2*>(small_vec(hl, kS + s) + c) = w[r];
            else if (s + 2 == ns && wbuf)
              *reinterpret_cast<double2*>(wbuf + c) = w[r];
            else
              Pair<double>::store(V + (int64_t)(j + 1 + s) * ld + sg.beg + c, w[r].x, w[r].y);
          }
        }
    if (!last) {
      tail_next(a, theta, tt);
      if (ll) {
        stage_ll(s + 1);
      } else {
        flag_publish(a, 4 * k + 1 + s);
        flag_wait_neighbours(a, 4 * k + 1 + s);
        stage(hxs);
      }
    }
  }
  if (R == 1 && !upd)
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (e0[r] >= 0)
#pragma unroll
        for (int q = 0; q < kS; ++q) {
          const int col = j - (kS - 1) + q;
          if (q == kS - 1 || col >= jo)
            *reinterpret_cast<double2*>(small_vec(hl, q) + e0[r]) =
                Pair<double>::load(V + (int64_t)max(col, 0) * ld + sg.beg + e0[r]);
        }
  if constexpr (R == 1) {
    __syncthreads();
    small_dots(a, sg.beg, n, j, jo, ns, na + ns > 1, hl, sacc);
    return;
  }
  {
    const int64_t q0 = pbeg, t0 = 2 * q0;
    if (!wave_in_tile(q0, pend)) return;
    uint32_t lo[R];
    bool ok[R];
    tile_pairs_r<R>(q0, pend, lo, ok);
    double2 va[C][R], b[kNv][R];
    if (jo > 0) load_block<R, C>(V, ld, t0, 0, min(C, jo), lo, va);
    // (own pairs, as this thread left them)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = 2 * (r * kThreads + kp_tid());
#pragma unroll
      for (int q = 0; q < kNv; ++q) {
        const int col = j - (kS - 1) + q;
        double2 v = make_double2(0.0, 0.0);
        if (ok[r]) {
          if (q - kS == ns - 1)
            v = make_double2(X[c], c + 1 < n ? X[c + 1] : 0.0);
          else if (q - kS == ns - 2 && q >= kS && wbuf)
            v = *reinterpret_cast<const double2*>(wbuf + c);
          else if (q < kS ? (q == kS - 1 || col >= jo) : (q - kS < ns))
            v = Pair<double>::load(V + (int64_t)max(col, 0) * ld + t0 + lo[r]);
        }
        b[q][r] = v;
      }
    }
    tile_dots<R, false>(V, ld, t0, jo, na + ns > 1, lo, b, va, sacc);
  }
}

// The same with every vector in memory (several sub-tiles or planes).
template <int R, bool HL>
__device__ __attribute__((always_inline)) inline void matvec_stream(const Args& a, int j, int na, int ns,
                                                                    double theta, double inv_mu, double* sacc,
                                                                    double* hl, unsigned k) {
  double* V = reinterpret_cast<double*>(a.V);
  const int64_t ld = a.ld;
  const Rows o = own_rows(a);
  const int jo = j - na;
  constexpr int C = kDotCols<R>;
  if (j == 0) copy_state<double>(a, o, V);
  const double* hxs = a.hx;
  for (int s = 0; s < ns; ++s) {
    const bool last = s + 1 == ns;
    if (HL) stage_halo<double>(a, hxs, o, hl);
    __syncthreads();
    const Col<double> xc{V + (int64_t)(j + s) * ld};
    double* wcol = V + (int64_t)(j + s + 1) * ld;
    double* const hxn = (s & 1) ? a.hx : a.hx2;
    for (int si = 0; si < num_segs(a); ++si) {
      const Seg sg = seg_at(a, o, si);
      const int64_t pend = (sg.end + 1) >> 1;
      double tt[kPMax];
      tail_of_x(a, sg.plane, inv_mu, tt);
      for (int e = 0; e < s; ++e) tail_next(a, theta, tt);
      for (int64_t q0 = sg.beg >> 1; q0 < pend; q0 += (int64_t)kThreads * R) {
        if (!wave_in_tile(q0, pend)) break;
        const int64_t t0 = 2 * q0;
        uint32_t lo[R];
        bool ok[R];
        tile_pairs_r<R>(q0, pend, lo, ok);
        double2 va[C][R], w[R];
        if (last && jo > 0) load_block<R, C>(V, ld, t0, 0, min(C, jo), lo, va);
        aug_tile<double, HL, Col<double>, R>(a, hxs, o, sg, xc, hl, t0, lo, tt, w);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double2 c = xc.pair(t0 + lo[r]);
          w[r].x = __builtin_fma(-theta, c.x, w[r].x);
          w[r].y = __builtin_fma(-theta, c.y, w[r].y);
          if (ok[r]) {
            Pair<double>::store(wcol + t0 + lo[r], w[r].x, w[r].y);
            if (!last) publish_pair(a, hxn, sg, t0 + lo[r], w[r].x, w[r].y);
          }
        }
        if (last) {
          double2 b[kNv][R];
#pragma unroll
          for (int q = 0; q < kNv; ++q) {
            const int col = j - (kS - 1) + q;
            const bool on = q < kS ? (q == kS - 1 || col >= jo) : (q - kS + 1 < ns);
            const bool isw = q - kS + 1 == ns;
#pragma unroll
            for (int r = 0; r < R; ++r)
              b[q][r] = !ok[r] ? make_double2(0.0, 0.0)
                               : (isw ? w[r] : (on ? Pair<double>::load(V + (int64_t)max(col, 0) * ld + t0 + lo[r])
                                                   : make_double2(0.0, 0.0)));
          }
          tile_dots<R, true>(V, ld, t0, jo, na + ns > 1, lo, b, va, sacc);
        }
      }
    }
    if (!last) {
      flag_publish(a, 4 * k + 1 + s);
      flag_wait_neighbours(a, 4 * k + 1 + s);
      hxs = hxn;
    }
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
      if (!wave_in_tile(q0, pend)) break;
      const int64_t t0 = 2 * q0;
      uint32_t lo[R];
      bool ok[R];
      tile_pairs_r<R>(q0, pend, lo, ok);
      double2 acc[1][R];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[0][r] = make_double2(0.0, 0.0);
      for (int i0 = 0; i0 < m; i0 += C)
        axpy_block<R, C, 1>(V, ld, t0, i0, 1, min(C, m - i0), cf, lo, acc);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (ok[r]) {
          const int64_t e = t0 + lo[r];
          *reinterpret_cast<double2*>(a.u + e) = acc[0][r];
          if (!last) publish_pair(a, a.hx, sg, e, acc[0][r].x, acc[0][r].y);
          if (last) {
            if (e < sg.end) outp[e] = acc[0][r].x;
            if (e + 1 < sg.end) outp[e + 1] = acc[0][r].y;
          }
        }
      }
    }
  }
  if (wg_rank(a) == 0) tail_combine_cols<double, double>(a, V, m, a.pub->coefs[0], -1, 0.0, a.u, !last);
}

// ---- the grid-wide reduction ---------------------------------------------------
//
// Every workgroup stores its row of partial sums; slots that nobody has
// written since they were consumed hold kPartEmpty, so a reader takes the
// data in the load that first sees them (see gather_step_partials).  Up to
// kDirectRows rows are read by the leader.  Above, the rows are summed by
// slot quads first: workgroup q of the first nq reads quad q of every row (one
// 16-byte load per thread at 256 rows) and stores four sums, and the leader
// reads those: one workgroup reading 256 rows of 130 slots took 5 to 6 us
// per step on its share of the coherent path; the two hops take 5 for 260.

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
//
// With measured products below kSmallL the GSMGS correction is T = I - L - L'
// (its second order is under rounding), so C = B - (L + L') B is one product
// with the symmetric table: two workgroup barriers between the reduced sums
// and the coefficients, against five for M^{-1} kept row by row (serial part
// of a three-step phase at 64 x 64 5.4 us, of a two-step phase that way 5.9 us).  Above it, one wave
// solves with M = I + L by substitution, exactly Algorithm 7's two sweeps.

// Row r of the table times the kS columns of b (stride 72): sum over k <= hi, k
// != r (lower: k < r); 8 lanes per row as in row_mv.
__device__ inline void row_mvs(int hi, const double* tab, const double* b, int r, bool lower, double (&out)[kS]) {
  const int s = kp_tid() & 7;
#pragma unroll
  for (int l = 0; l < kS; ++l) out[l] = 0.0;
#pragma unroll
  for (int t = 0; t < kMMax / 8; ++t) {
    if (8 * t > hi) break;                     // uniform
    const int k = s + 8 * t;
    const double x = tab[r * kTabLd + k];
    const bool in = k <= hi && k != r && r <= hi && !(lower && k > r);
#pragma unroll
    for (int l = 0; l < kS; ++l) {
      const double v = x * b[72 * l + k];
      out[l] += in ? v : 0.0;
    }
  }
#pragma unroll
  for (int l = 0; l < kS; ++l) {
    out[l] += dpp_mov<0xB1>(out[l]);
    out[l] += dpp_mov<0x4E>(out[l]);
    out[l] += dpp_mov<0x141>(out[l]);
  }
}

// C = T B by substitution in one wave (row i = lane): M y = b, p = b - L' y, M c
// = p (H-CWY: c = y).  Only where the measured products are not small.
__device__ inline void solve_exact(const Args& a, int j, const double* tab, double (&v)[kS]) {
  const int i = kp_tid() & 63;
  double y[kS], p[kS];
  auto forward = [&](double (&x)[kS]) {
    for (int k = 0; k < j; ++k) {
      const double l = (i > k && i <= j) ? tab[i * kTabLd + k] : 0.0;
#pragma unroll
      for (int q = 0; q < kS; ++q) x[q] -= l * __shfl(x[q], k, 64);
    }
  };
#pragma unroll
  for (int q = 0; q < kS; ++q) y[q] = v[q];
  forward(y);
  if (a.orth == KP_ORTH_H_CWY) {
#pragma unroll
    for (int q = 0; q < kS; ++q) v[q] = y[q];
    return;
  }
#pragma unroll
  for (int q = 0; q < kS; ++q) p[q] = v[q];
  for (int k = 1; k <= j; ++k) {
    const double l = (i < k) ? tab[k * kTabLd + i] : 0.0;
#pragma unroll
    for (int q = 0; q < kS; ++q) p[q] -= l * __shfl(y[q], k, 64);
  }
  forward(p);
#pragma unroll
  for (int q = 0; q < kS; ++q) v[q] = p[q];
}

// The Hessenberg columns of the last block once the norms al[0 .. n) of its
// new columns base + 1 .. base + n are known: column base + k takes the factor
// 1 / al[k-1] (its vector's unit scale) and row base + 1 + l the factor al[l].
__device__ inline void finish_block_columns(LeadB& L, int base, int n, const double* al, int i) {
  if (i == 0) L.H[hcol(base) + base + 1] = L.rr[0] * al[0];
  for (int k = 1; k < n; ++k) {
    const double s = 1.0 / al[k - 1];
    if (i <= base) L.H[hcol(base + k) + i] = s * L.rp[k - 1][i];
    if (i <= k) L.H[hcol(base + k) + base + 1 + i] = s * L.hx[k - 1][i] * al[i];
  }
}

// 1 / sqrt(x), x > 0 and normal: the hardware estimate and two Newton steps
// (within 2 ulp; a tenth of the dependent instructions of sqrt and divide).
__device__ inline double inv_sqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int t = 0; t < 2; ++t) y = __builtin_fma(0.5 * y, __builtin_fma(-x * y, y, 1.0), y);
  return y;
}

// tv: the reduced sums of the step from column j (slots: block_slots).
// Stored columns carry unit scales sigma_i as in scalar_step; the single-step
// rules (lagged norm, norm estimate, fallback, breakdown) are those of
// scalar_step.
__device__ __attribute__((always_inline)) inline void block_scalar(const Args& a, int j, int na, int ns,
                                                                   const double* tv, LeadB& L, double* sb,
                                                                   Ctl& nx) {
  State* st = a.st;
  Pub* pb = a.pub;
  const int i = kp_tid();
  const bool w0 = i < 64;
  const int jo = j - na;
  const double* G = tv + kNv * jo;
  // norms of the columns jo .. j (vectors kS - 1 - na .. kS - 1)
  double al[kS], ial[kS];
  bool okn = true;
#pragma unroll
  for (int q = 0; q < kS; ++q) {
    const double g = (q >= kS - 1 - na) ? G[gram_at(q, q)] : 1.0;
    // (tiny norms, whose squares leave the normal range, take the slow way)
    const bool fast = g > 1e-290 && g < 1e290;
    ial[q] = fast ? inv_sqrt(g) : 1.0 / sqrt(g);
    al[q] = fast ? g * ial[q] : sqrt(g);
    if (q < kS - 1) okn = okn && al[q] > 0.0 && isfinite(al[q]);
  }
  const double alj = al[kS - 1], cww = G[gram_at(kS, kS)];
  if (!okn) {
    if (i == 0) {
      nx.status = (int)KP_STATUS_NONFINITE;
      nx.phase = (int)PH_FINISH;
    }
    return;
  }
  if (na && L.pend && w0) {
    double an[kS];
#pragma unroll
    for (int q = 0; q < kS; ++q) an[q] = (na == 2) ? al[q] : (q + 1 < kS ? al[(q + 1) % kS] : 1.0);
    finish_block_columns(L, j - na - 1, na + 1, an, i);
  }
  if (!(alj > 0.0) || !isfinite(alj) || !isfinite(cww)) {
    if (i == 0) {
#pragma unroll
      for (int q = 0; q < kS - 1; ++q)
        if (q >= kS - 1 - na) L.sigma[j - (kS - 1) + q] = 1.0 / al[q];
      if (j == 0 && alj == 0.0) {            // zero start vector: result is zero
        st->zero = 1;
        L.beta = 0.0;
        nx.phase = (int)PH_FINISH;
      } else if (alj == 0.0) {               // exact invariance already reached
        L.breakdown = 1;
        nx.m_eff = j;
        nx.upd = 0;
        L.H[hcol(j - 1) + j] = 0.0;
        nx.phase = (int)PH_EXPM;
      } else {
        nx.status = (int)KP_STATUS_NONFINITE;
        nx.phase = (int)PH_FINISH;
      }
    }
    return;
  }
  if (j > 0 && L.fallback_cur && alj <= a.eps_bd * sqrt(L.wn2)) {
    // the exact norm of the vector produced with the fallback is negligible:
    // lucky breakdown at the previous step (this step's products are unused)
    if (i == 0) {
      L.breakdown = 1;
      L.H[hcol(j - 1) + j] = 0.0;
      nx.j = j;
      nx.m_eff = j;
      nx.upd = 0;
      nx.phase = (int)PH_EXPM;
    }
    return;
  }
  // Vector q (< kS) is column j - (kS - 1) + q.  A measured column's lane reads
  // its kNv sums, a new column's lane (vector p) the products of its row.
  double sig = 0.0;
  if (w0) {
    const double sj = ial[kS - 1];
    const int p = i - (j - (kS - 1));
    const bool old = i < jo, in = i <= j;
    sig = old ? L.sigma[i] : (p == 0 ? ial[0] : (p == 1 ? ial[1] : sj));
    // slot of the product with vector q: column slots, or the Gram rows
    const double* row = old ? tv + kNv * i : G + (in ? p * kNv - p * (p + 1) / 2 : 0);
    int big = 0;
#pragma unroll
    for (int q = 0; q < kS; ++q) {
      const int col = j - (kS - 1) + q;
      if (in && col >= jo && (old || q > p)) {
        const double l = sig * ial[q] * row[q];
        L.tab[i * kTabLd + col] = L.tab[col * kTabLd + i] = l;
        big |= !(fabs(l) <= kSmallL);
      }
    }
#pragma unroll
    for (int q = 0; q < kS; ++q) sb[72 * q + i] = in ? sig * row[kS + q] * sj : 0.0;
    if (big) L.big = 1;
  }
  __syncthreads();
  const bool ncwy = a.orth == KP_ORTH_H_NCWY, gs = a.orth == KP_ORTH_H_GSMGS;
  if (!L.big || ncwy) {
    const int r = (kp_tid() >> 6) * 8 + ((kp_tid() & 63) >> 3);
    double s[kS];
    row_mvs(j, L.tab, sb, r, !gs, s);
    if ((kp_tid() & 7) == 0)
#pragma unroll
      for (int q = 0; q < kS; ++q) L.c[q][r] = sb[72 * q + r] - s[q];
  } else if (w0) {
    double v[kS];
#pragma unroll
    for (int q = 0; q < kS; ++q) v[q] = sb[72 * q + i];
    solve_exact(a, j, L.tab, v);
#pragma unroll
    for (int q = 0; q < kS; ++q) L.c[q][i] = v[q];
  }
  __syncthreads();
  if (!w0) return;
  const bool in = i <= j;
  // (products are scaled by s_j twice, not by its square, which overflows where
  // ||x_j||^2 is subnormal)
  const double sj = ial[kS - 1];
  double b[kS], c[kS];
#pragma unroll
  for (int q = 0; q < kS; ++q) {
    b[q] = in ? sb[72 * q + i] : 0.0;
    c[q] = in ? L.c[q][i] : 0.0;
  }
  // ||A u_j||^2 = ||w_1 + theta u_j||^2 for the fallback and breakdown rules
  // (block_steps' theta is 0 for the forms without blocks)
  const double th = L.theta, ws2 = cww * sj * sj;
  const double wn2 = fmax(__builtin_fma(th, __builtin_fma(2.0, readlane_d(b[0], j), th), ws2), 0.0);
  const double t4 = wave_sum4(b[0] * b[0], b[0] * c[0], b[0] * c[1], b[0] * c[2]);
  const double ss = readlane_d(t4, 0);
  const double est2 = ws2 - ss;
  const int fallback = (est2 <= a.delta * wn2) ? 1 : 0;
  const double gam = fallback ? 1.0 : sqrt(est2);
  const int bd = (!fallback && gam <= a.eps_bd * sqrt(wn2)) ? 1 : 0;
  const bool bad = !isfinite(readlane_d(t4, 1));
  // R'R = W'W - B'C, as far as the guard lets it
  int done = 1;
  double r00 = gam, r01 = 0.0, r02 = 0.0, r11 = 1.0, r12 = 0.0, r22 = 1.0;
  double i00 = 0.0, i11 = 1.0, i22 = 1.0;
  if (ns > 1 && !bad && !fallback && !bd && est2 > kGuard * ws2) {
    const double u4 = wave_sum4(b[1] * c[1], b[1] * c[2], b[2] * c[2], 0.0);
    const double n00 = ws2 - readlane_d(t4, 1), n01 = G[gram_at(kS, kS + 1)] * sj * sj - readlane_d(t4, 2);
    const double g11 = G[gram_at(kS + 1, kS + 1)] * sj * sj, n11 = g11 - readlane_d(u4, 0);
    const double q00 = inv_sqrt(n00), q01 = n01 * q00, d1 = n11 - q01 * q01;
    if (n00 > 1e-290 && n00 < 1e290 && g11 < 1e290 && d1 > kGuard * g11 && d1 > 1e-290) {
      done = 2;
      i00 = q00;
      r00 = n00 * q00;
      r01 = q01;
      i11 = inv_sqrt(d1);
      r11 = d1 * i11;
      if (ns > 2) {
        const double g22 = G[gram_at(kS + 2, kS + 2)] * sj * sj, n22 = g22 - readlane_d(u4, 2);
        const double n02 = G[gram_at(kS, kS + 2)] * sj * sj - readlane_d(t4, 3);
        const double n12 = G[gram_at(kS + 1, kS + 2)] * sj * sj - readlane_d(u4, 1);
        const double q02 = n02 * i00, q12 = (n12 - r01 * q02) * i11, d2 = n22 - q02 * q02 - q12 * q12;
        if (g22 < 1e290 && d2 > kGuard * g22 && d2 > 1e-290) {
          done = 3;
          r02 = q02;
          r12 = q12;
          i22 = inv_sqrt(d2);
          r22 = d2 * i22;
        }
      }
    }
  }
  if (done == 1) i00 = 1.0 / r00;
  const double i01 = -r01 * i00 * i11, i12 = -r12 * i11 * i22, i02 = -(r01 * i12 + r02 * i22) * i00;
  if (in) {
    L.H[hcol(j) + i] = i == j ? c[0] + th : c[0];
    cstore(&pb->coefs[0][i], -c[0] * i00 * sig);
    if (done > 1) cstore(&pb->coefs[1][i], -(c[0] * i01 + c[1] * i11) * sig);
    if (done > 2) cstore(&pb->coefs[2][i], -(c[0] * i02 + c[1] * i12 + c[2] * i22) * sig);
  }
  // the unit scales of the columns measured here
  if (in && i >= jo) L.sigma[i] = sig;
  if (i == j && a.pairs) cstore(&pb->shift, c[0] + th);   // theta of the next block: H_jj
  if (i == 0) {
    cstore(&pb->coefs[0][j + 1], i00 * sj);
    if (done > 1) {
      cstore(&pb->coefs[1][j + 1], i01 * sj);
      cstore(&pb->coefs[1][j + 2], i11 * sj);
    }
    if (done > 2) {
      cstore(&pb->coefs[2][j + 1], i02 * sj);
      cstore(&pb->coefs[2][j + 2], i12 * sj);
      cstore(&pb->coefs[2][j + 3], i22 * sj);
    }
    if (j > 0 && !na) L.H[hcol(j - 1) + j] = L.rr[0] * alj;
    L.rr[0] = r00;
    L.rr[1] = r01;
    L.rr[2] = r02;
    L.rr[3] = r11;
    L.rr[4] = r12;
    L.rr[5] = r22;
    L.ri[0] = i00;
    L.ri[1] = i01;
    L.ri[3] = i11;
    L.wn2 = wn2;
    L.theta_used = th;
    if (a.pairs) L.theta = L.c[0][j] + th;
    if (j == 0) L.beta = alj;
    L.fallback_cur = fallback;
    L.n_fallback += fallback;
    L.pend = 0;
    if (bad) {
      nx.status = (int)KP_STATUS_NONFINITE;
      nx.phase = (int)PH_FINISH;
    } else if (bd) {
      L.H[hcol(j) + j + 1] = 0.0;
      L.breakdown = 1;
      ++L.arnoldi_steps;
      nx.j = j + 1;
      nx.m_eff = j + 1;
      nx.upd = 0;
      nx.na = 0;
      nx.phase = (int)PH_EXPM;
    } else {
      L.post = done - 1;
      L.nopair = (ns > 1 && done == 1) ? L.nopair + 1 : 0;
      L.arnoldi_steps += done;
      nx.j = j + done;
      nx.m_eff = nx.j;
      nx.upd = done;
      nx.na = done - 1;
      nx.pns = ns;
      nx.phase = (int)((nx.j >= L.m_target || nx.j >= a.stop_j) ? PH_CLOSE : PH_STEP);
      nx.ns = block_steps(a, L, nx.j);
    }
  }
}

// After the release of a block's barrier: the raw Hessenberg columns of its
// later vectors (see the top of this file), needed at the next reduction only.
__device__ __attribute__((always_inline)) inline void block_post(int j, LeadB& L) {
  const int n = L.post;   // (uniform: set before the release's barrier)
  if (n == 0) return;
  const int s = kp_tid() & 7;
  const int r = (kp_tid() >> 6) * 8 + ((kp_tid() & 63) >> 3);
  double g[kS - 1];
#pragma unroll
  for (int l = 0; l < kS - 1; ++l) g[l] = 0.0;
#pragma unroll
  for (int t = 0; t < kMMax / 8; ++t) {
    if (8 * t >= j) break;
    const int k = s + 8 * t;
    const bool on = k < j && k >= r - 1;
    const double x = on ? L.H[hcol(k) + r] : 0.0;
#pragma unroll
    for (int l = 0; l < kS - 1; ++l) g[l] += on ? x * L.c[l][k] : 0.0;
  }
#pragma unroll
  for (int l = 0; l < kS - 1; ++l) {
    g[l] += dpp_mov<0xB1>(g[l]);
    g[l] += dpp_mov<0x4E>(g[l]);
    g[l] += dpp_mov<0x141>(g[l]);
  }
  const double th = L.theta_used, c0j = L.c[0][j], c1j = L.c[1][j];
  if (s == 0 && r <= j) {
    const double c0 = L.c[0][r], c1 = L.c[1][r], hj = r == j ? c0 + th : c0;
    const double u0 = c1 + th * c0 - g[0] - hj * c0j;
    const double u1 = L.c[2][r] + th * c1 - g[1] - hj * c1j;
    L.rp[0][r] = u0 * L.ri[0];
    L.rp[1][r] = u0 * L.ri[1] + u1 * L.ri[3];
  }
  if (kp_tid() == 0) {
    const double *R = L.rr, *I = L.ri;
    const double x00 = R[1] + th * R[0] - R[0] * c0j, x01 = R[3];
    const double x10 = R[2] + th * R[1] - R[0] * c1j, x11 = R[4] + th * R[3], x12 = R[5];
    L.hx[0][0] = x00 * I[0];
    L.hx[0][1] = x01 * I[0];
    L.hx[1][0] = x00 * I[1] + x10 * I[3];
    L.hx[1][1] = x01 * I[1] + x11 * I[3];
    L.hx[1][2] = x12 * I[3];
  }
  __syncthreads();
  if (kp_tid() == 0) {
    L.post = 0;
    L.pend = 1;
  }
}

// Close of the Arnoldi process: the exact norms of the pending columns (nrm2[l]
// of new column l of upd) complete H.
__device__ __attribute__((always_inline)) inline void block_close(const Args& a, const double* nrm2, LeadB& L,
                                                                  Ctl& nx) {
  State* st = a.st;
  const int j = nx.j, n = nx.upd;
  double al[kS];
  bool fin = true;
#pragma unroll
  for (int l = 0; l < kS; ++l) {
    al[l] = l < n ? sqrt(nrm2[l]) : 1.0;
    fin = fin && isfinite(al[l]) && (l + 1 >= n || al[l] > 0.0);
  }
  __syncthreads();
  if (kp_tid() < 64) finish_block_columns(L, j - n, n, al, kp_tid());
  if (kp_tid() != 0) return;
#pragma unroll
  for (int l = 0; l < kS - 1; ++l)
    if (l + 1 < n) L.sigma[j - n + 1 + l] = 1.0 / al[l];
  L.pend = 0;
  const double last2 = nrm2[n - 1];
  st->last_nrm2 = last2;
  nx.upd = 0;
  if (!fin) {
    nx.status = (int)KP_STATUS_NONFINITE;
    nx.phase = (int)PH_FINISH;
    return;
  }
  if (L.fallback_cur && sqrt(last2) <= a.eps_bd * sqrt(L.wn2)) {
    L.H[hcol(j - 1) + j] = 0.0;
    L.breakdown = 1;
  }
  nx.phase = (int)((L.breakdown || j >= L.m_target) ? PH_EXPM : PH_STEP);
  nx.ns = block_steps(a, L, j);
}

}  // namespace kp
