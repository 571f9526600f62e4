// libkrylov_phi: kernels and the C ABI declared in include/krylov_phi.h.
//
// Execution model (one MI355X, gfx950).  A whole phi_combo call is ONE
// cooperative launch of k_blk (the one-reduction forms with a float64 basis; above
// 2^18 elements those with block steps) or k_run (the others, a float basis, MGS,
// ioCGS): every workgroup loops over the phases published
// by workgroup 0 (stage, Arnoldi step = matvec+dots then update+norm, small
// exponential + controller, combine, finish) and meets the others at
// grid-wide barriers.  The grid-wide reduction of an Arnoldi step is the
// paper's single global synchronisation (Algorithm 4): every workgroup
// publishes its partial inner products, workgroup 0 reduces them and runs the
// O(m^2) scalar step, then releases the grid.  The adaptive substep controller
// runs on the device; nothing returns to the host until the call is done.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "kp_block.h"
#include "kp_internal.h"
#include "kp_leader.h"
#include "kp_passes.h"
#include "kp_plan.h"

namespace kp {

// Carve-up of the shared phase buffer (doubles).  Streaming phases: per-wave
// partial sums (sacc), coefficients, block-reduction scratch and the LDS copy
// of the stencil halo rows (hl).  Leader work, after sacc is dead: group sums
// of the partial reduction (grp), then the scalar-step work arrays (wk), and
// the reduced inner products tv.  The small exponential uses the whole buffer
// (it runs in a phase of its own).  The correction-matrix tables of the leader
// live in a separate buffer for the whole launch.
constexpr int kOffSacc = 0;
constexpr int kOffGrp = 0;
constexpr int kOffWk = 0;
constexpr int kOffCoef = kWaves * kKStride;
constexpr int kOffRed = kOffCoef + kMMax + 8;
constexpr int kOffTv = kOffRed + kWaves;
constexpr int kOffOwn = kOffTv + kKStride;   // the leader's own step sums
constexpr int kOffHl = 1536;
constexpr int kLdsDoubles = (2 * kNmPad * kNmPad > kOffHl + kHaloCap) ? 2 * kNmPad * kNmPad
                                                                      : kOffHl + kHaloCap;
static_assert(kOffGrp + kRg * kKStride <= kOffCoef, "grp overlaps coef");
static_assert(kOffWk + kWkDoubles <= kOffCoef, "wk overlaps coef");
static_assert(kOffOwn + kKStride <= kOffHl, "tv / own overlap the halo copy");
static_assert(sizeof(((LeadLds*)0)->Mi) >= kKeepMax * sizeof(double), "w of ioCGS on chip");
static_assert(kLdsDoubles >= kExDoubles, "the small exponential does not fit the phase buffer");

// One phase of the call for this workgroup.  MS: the processes with one
// reduction per inner product (MGS) or per window (ioCGS), else the
// one-reduction forms with a float basis; each kind is compiled without the
// other's phases (the registers of the update and dot passes cost the MS kernels
// 459 scalar and 38 vector spills: 355 and 2 without).  cur: control of the
// phase (LDS, identical in every workgroup); nxt: the leader's control of the
// next phase; ok: cleared when a bounded wait gives up (the launch is
// aborting).  On return cur holds the control of the next phase.
// The Brusselator's matvec pass takes both species of a grid point together
// (joint sub-tiles) with a float basis; with a float64 one the joint tile's
// extra registers spill and cost what the shared loads save (measured), so it
// keeps one plane at a time.
template <typename TB> constexpr bool kJointBr = sizeof(TB) == 4;

template <typename TB, bool MS>
__device__ __attribute__((always_inline)) inline void run_phase(const Args& a, double* lds, LeadLds& L, Ctl& cur, Ctl& nxt, int& ok,
                          int& kept, unsigned k) {
  double* sacc = lds + kOffSacc;
  double* grp = lds + kOffGrp;
  double* wk = lds + kOffWk;
  double* red = lds + kOffRed;
  double* tv = lds + kOffTv;
  double* own = lds + kOffOwn;
  double* hl = lds + kOffHl;
  const bool lead = wg_rank(a) == 0;
  const Ctl c = cur;
  // ioCGS on chip: its phases' sums go through the polled step buffers
  const bool keep_ms = MS && sizeof(TB) == 8 && a.keep_ms;
  const bool polled = (!MS && c.phase == PH_STEP) || (keep_ms && (c.phase == PH_MVEC || c.phase == PH_PROJ));
  // the matvec pass of the previous phase left x_{j-1} and w in LDS
  const bool xl = !MS && a.keep_xw && kept == c.j - 1;
  KP_TS(a, k, 0);
  if (lead) KP_TSV(a, k, 4, c.phase * 1000 + c.j);
  // this workgroup's row of the step buffer of barrier k + 1 is free again
  // (consumed at barrier k - 1): mark it unwritten before anything of this
  // phase is stored
  if (wg_rank(a) < a.nwg && kp_tid() < kKStride)
    cstore(step_part(a, k + 1) + (int64_t)wg_rank(a) * kKStride + kp_tid(),
           __builtin_bit_cast(double, kPartEmpty));
  // streaming part of the phase (every workgroup that owns rows; the others
  // of a team larger than the row count only meet the barriers)
  if (wg_rank(a) < a.nwg) switch (c.phase) {
    case PH_STAGE:
      stage_pass(a, red);
      break;
    case PH_STEP:
      if constexpr (MS) break;
      // the update that produces x_j (coefficients of the previous scalar
      // step), then the matvec + grouped dots of step j: one grid-wide sync
      // (flag_publish also completes the reset above before the partial
      // sums are stored; without an update the wait is explicit)
      // (with keep_xw, x_{j-1} and w are in LDS from the matvec pass of the
      // previous phase, and the update leaves x_j there for this one: every
      // update directly follows the matvec pass of the same Arnoldi process
      // in the same launch, since a launch pauses only after a close)
      if (c.upd) {
        update_pass<TB>(a, c.j - 1, a.pub->coefs[0], red, false, xl ? hl : nullptr);
        flag_publish(a, k);
        KP_TS(a, k, 1);
        flag_wait_neighbours(a, k);
        KP_TS(a, k, 2);
      } else {
        wait_all_stores();
      }
      {
        double* prow = step_part(a, k) + (int64_t)wg_rank(a) * kKStride;
        double* mine = lead ? own : nullptr;
        if (a.keep_xw && c.upd && xl)   // (keep_xw implies halo_lds)
          matvec_dots_pass<TB, true, true, true>(a, c.j, sacc, hl, prow, mine);
        else if (a.keep_xw)
          matvec_dots_pass<TB, true, true, false>(a, c.j, sacc, hl, prow, mine);
        else if (kJointBr<TB> && a.kind == KP_OP_BRUSSELATOR && !a.tangent && a.halo_lds)
          matvec_dots_pass<TB, true, false, false, kJointBr<TB>>(a, c.j, sacc, hl, prow, mine);
        else if (kJointBr<TB> && a.kind == KP_OP_BRUSSELATOR && !a.tangent)
          matvec_dots_pass<TB, false, false, false, kJointBr<TB>>(a, c.j, sacc, hl, prow, mine);
        else if (a.halo_lds)
          matvec_dots_pass<TB, true, false, false>(a, c.j, sacc, hl, prow, mine);
        else
          matvec_dots_pass<TB, false, false, false>(a, c.j, sacc, hl, prow, mine);
        // x_j and w stay in LDS (keep_xw) for the update of the next phase,
        // which the leader always makes an update of column j + 1
        if (a.keep_xw && kp_tid() == 0) kept = c.j;
      }
      break;
    case PH_CLOSE:
      if constexpr (MS) break;
      update_pass<TB>(a, c.j - 1, a.pub->coefs[0], red, true, xl ? hl : nullptr);
      break;
    case PH_MVEC:
      if constexpr (MS) {
        // MGS multiplies and takes v_1 . w; ioCGS takes v_{j-1} . w and v_j . w
        const int acol = c.j == 0 ? -1 : (a.orth == KP_ORTH_MGS ? 0 : c.j - 1);
        if (keep_ms) {
          if constexpr (sizeof(TB) == 8)
            iocgs_mvec(a, c.j, acol, kept == c.j, sacc, hl, L.Mi,
                       step_part(a, k) + (int64_t)wg_rank(a) * kKStride, lead ? own : nullptr);
        } else if (a.halo_lds)
          mvec_pass<TB, true>(a, c.j, acol, sacc, hl);
        else
          mvec_pass<TB, false>(a, c.j, acol, sacc, hl);
      }
      break;
    case PH_PROJ:
      if constexpr (MS) {
        // MGS: subtract the projection on v_{i-1}, then v_i . w (or the
        // norm); ioCGS: subtract both projections of the window, then the norm
        if (keep_ms) {
          if constexpr (sizeof(TB) == 8)
            iocgs_proj(a, c.j, max(0, c.j - 1), a.pub->coefs[0], red, hl, L.Mi,
                       step_part(a, k) + (int64_t)wg_rank(a) * kKStride, lead ? own : nullptr);
          if (kp_tid() == 0) kept = c.j + 1;   // (column in LDS)
        } else if (a.orth == KP_ORTH_MGS)
          proj_pass<TB>(a, c.j, c.i - 1, c.i - 1, a.pub->coefs[0], c.i <= c.j ? c.i : -1, c.i > c.j,
                        red);
        else
          proj_pass<TB>(a, c.j, max(0, c.j - 1), c.j, a.pub->coefs[0], -1, true, red);
      }
      break;
    case PH_COMBINE:
      combine_pass<TB>(a, c.m_eff, a.pub->coefs[0], c.last != 0);
      break;
    case PH_FINISH:
      finish_pass(a, c.status == KP_STATUS_NONFINITE);
      break;
    default:
      break;
  }
  KP_TS(a, k, 3);
  // (the leader counts its arrival at a step barrier after the release, so
  // that the atomic is not outstanding while it polls)
  if (!polled)
    bar_arrive(a);
  else if (!lead)
    bar_count(a);
  if (!lead) {
    bar_wait(a, k, &cur, &ok);
    KP_TS(a, k, 4);
    return;
  }
  // serial part (workgroup 0)
  if (!polled) {
    bar_gather(a, k, &ok);
    if (!ok) return;
  }
  if (kp_tid() == 0) nxt = cur;   // (re-read: c need not stay live through the pass)
  if (!MS && a.keep_xw && kp_tid() == 0 && (c.phase == PH_STEP || c.phase == PH_CLOSE)) {
    // vector passes of the two-pass count that stayed in LDS: the update's
    // x_{j-1} and w, the matvec's x_j, and the w it did not store
    const bool upd = (c.phase == PH_CLOSE || c.upd) && xl;
    L.onchip += (upd ? 2 : 0) + (c.phase == PH_STEP ? (upd ? 2 : 1) : 0);
    a.st->onchip = L.onchip;
  }
  switch (c.phase) {
    case PH_STAGE:
      leader_stage(a, red, L, nxt);
      break;
    case PH_STEP:
      if constexpr (MS) break;
      gather_step_partials(a, step_part(a, k), 2 * c.j + 3, own, tv, grp, &ok);
      if (!ok) return;
      KP_TS(a, k, 5);
      scalar_step(a, c.j, tv, L, wk, nxt);
      break;
    case PH_CLOSE:
      if constexpr (MS) break;
      reduce_partials(a, 1, tv, grp);
      leader_close(a, tv[0], L, nxt);
      break;
    case PH_MVEC:
      if constexpr (MS) {
        if (keep_ms)
          gather_few(a, step_part(a, k), kMvSlots, own, tv, grp, &ok);
        else
          reduce_partials(a, kMvSlots, tv, grp);
        if (!ok) return;
        leader_mvec(a, c.j, tv, L, nxt);
      }
      break;
    case PH_PROJ:
      if constexpr (MS) {
        if (keep_ms)
          gather_few(a, step_part(a, k), 1, own, tv, grp, &ok);
        else
          reduce_partials(a, 1, tv, grp);
        if (!ok) return;
        leader_proj(a, c.j, c.i, tv[0], L, nxt);
      }
      break;
    case PH_EXPM:
      if (keep_ms && kp_tid() == 0) kept = -1;   // (it uses the whole buffer)
      expm_phase<sizeof(TB) == 4>(a, lds, L, nxt);
      break;
    case PH_COMBINE:
      leader_combine(a, L, nxt);
      break;
    case PH_FINISH:
      if (kp_tid() == 0) nxt.phase = PH_DONE;
      break;
    default:
      break;
  }
  KP_TS(a, k, 6);
  bar_release(a, k, nxt, a.pub);
  KP_TS(a, k, 7);
  if (polled) bar_count(a);
  if (kp_tid() == 0) cur = nxt;
}

// ---- block steps (the one-reduction forms with a float64 basis) ---------------
// LDS carve-up (doubles): per-wave sums (the leader's serial work reuses
// them), block-reduction scratch, reduced sums (the workgroup's own row
// first), the tail's sums, the coefficients of the pending columns, and the
// two buffers of the on-chip region (or the halo rows).  The small
// exponential uses the whole buffer.
constexpr int kOffBRed = kWaves * kBSlots;
constexpr int kOffBTv = kOffBRed + 4 * kWaves;
constexpr int kOffBTs = kOffBTv + kBSlots;
constexpr int kOffBCf = kOffBTs + kBSlots;
constexpr int kOffBHl = (kOffBCf + kS * kCoefLd + 1 + 15) / 16 * 16;
constexpr int kLdsDoublesB = kOffBHl + kHaloCap;
static_assert(kLdsDoublesB >= kExDoubles, "the small exponential does not fit the phase buffer");
static_assert(kS * 72 <= kWaves * kBSlots && kRg * kKStride <= kWaves * kBSlots, "leader scratch");
static_assert(kBSlots <= kThreads && kS * kCoefLd < kThreads, "one thread per slot");
static_assert(kS == 3 && kS <= kCStride, "coefficient arrays, projections and norms of three columns");

// Element pairs per thread of a batched problem's tiles (single calls choose
// 1, 2 or 4 by their partition, see geometry).
constexpr int kRBatch = 4;

template <int R>
__device__ __attribute__((always_inline)) inline void update_pending(const Args& a, const Ctl& c, const double* cf,
                                                                     double* hl, const double* wbuf, double* red,
                                                                     bool want_norm, unsigned tag) {
  if (c.upd == 3)
    update_block<R, 3>(a, c.j, c.pns, cf, hl, wbuf, red, want_norm, tag);
  else if (c.upd == 2)
    update_block<R, 2>(a, c.j, c.pns, cf, hl, wbuf, red, want_norm, tag);
  else
    update_block<R, 1>(a, c.j, c.pns, cf, hl, wbuf, red, want_norm, tag);
}

// One phase of the call for this workgroup (as run_phase).
template <int R>
__device__ __attribute__((always_inline)) inline void run_phase_block(const Args& a, double* lds, LeadB& L,
                                                                      Ctl& cur, Ctl& nxt, int& ok, unsigned k) {
  double* sacc = lds;
  double* red = lds + kOffBRed;
  double* tv = lds + kOffBTv;
  double* ts = lds + kOffBTs;
  double* cf = lds + kOffBCf;
  double* hl = lds + kOffBHl;
  const bool lead = wg_rank(a) == 0, owner = wg_rank(a) < a.nwg;
  double* wbuf = lead ? nullptr : reinterpret_cast<double*>(&L);   // (keep_xw; only the leader uses its tables)
  const Ctl c = cur;
  const int nslot = block_slots(c.j - c.na);
  KP_TS(a, k, 0);
  if (lead) KP_TSV(a, k, 4, c.phase * 1000 + c.j);
  if (owner) block_reset(a, k);
  if (owner) switch (c.phase) {
    case PH_STAGE:
      stage_pass(a, red);
      break;
    case PH_STEP: {
      for (int t = kp_tid(); t < kWaves * kBSlots; t += kThreads) sacc[t] = 0.0;
      const double inv_mu = cload(&a.pub->inv_mu);
      load_coefs(a, cf);
      const double theta = cf[kS * kCoefLd];
      if (c.upd) {
        update_pending<R>(a, c, cf, hl, wbuf, red, false, a.ll ? 4 * k : 0u);
        if (a.ll)
          __syncthreads();
        else
          flag_publish(a, 4 * k);
        KP_TS(a, k, 1);
      } else {
        wait_all_stores();   // (the resets, before the partial sums)
      }
      if (lead && kp_tid() >= kThreads - 64) tail_block(a, c.j, c.na, c.ns, theta, ts);
      if (a.keep_xw) {
        matvec_keep<R>(a, c.j, c.na, c.ns, c.upd != 0, theta, inv_mu, sacc, hl, wbuf, k);
      } else {
        if (c.upd) {
          flag_wait_neighbours(a, 4 * k);
          KP_TS(a, k, 2);
        }
        if (a.halo_lds)
          matvec_stream<R, true>(a, c.j, c.na, c.ns, theta, inv_mu, sacc, hl, k);
        else
          matvec_stream<R, false>(a, c.j, c.na, c.ns, theta, inv_mu, sacc, hl, k);
      }
      if (a.ll) wait_all_stores();   // (the resets; nothing above waited for them)
      __syncthreads();
      if (kp_tid() < nslot) {
        double s = lead ? ts[kp_tid()] : 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) s += sacc[w * kBSlots + kp_tid()];
        if (lead) tv[kp_tid()] = s;
        if (a.nwg > kDirectRows || !lead)
          cstore(block_part(a, k) + (int64_t)wg_rank(a) * a.bstride + kp_tid(), s);
      }
      break;
    }
    case PH_CLOSE:
      load_coefs(a, cf);
      update_pending<R>(a, c, cf, hl, wbuf, red, true, 0u);
      break;
    case PH_COMBINE:
      load_coefs(a, cf);
      combine_block<R>(a, c.m_eff, cf, c.last != 0);
      break;
    case PH_FINISH:
      finish_pass(a, c.status == KP_STATUS_NONFINITE);
      break;
    default:
      break;
  }
  KP_TS(a, k, 3);
  if (c.phase != PH_STEP) {
    bar_arrive(a);
  } else {
    if (owner && a.nwg > kDirectRows)
      reduce_quads(a, block_part(a, k), block_sums(a, k), nslot, red, &ok);
    if (!lead) bar_count(a);
  }
  if (!lead) {
    bar_wait(a, k, &cur, &ok);
    KP_TS(a, k, 4);
    return;
  }
  if (c.phase != PH_STEP) {
    bar_gather(a, k, &ok);
    if (!ok) return;
  }
  if (kp_tid() == 0) nxt = cur;   // (re-read: c need not stay live through the pass)
  if (a.keep_xw && kp_tid() == 0 && c.phase == PH_CLOSE) L.onchip += 2;
  switch (c.phase) {
    case PH_STAGE:
      leader_stage(a, red, L, nxt);
      break;
    case PH_STEP: {
      __syncthreads();   // (tv: its own row, and nxt)
      const int steps0 = L.arnoldi_steps;
      block_gather(a, k, nslot, tv, tv, &ok);
      if (!ok) return;
      KP_TS(a, k, 5);
      block_scalar(a, c.j, c.na, c.ns, tv, L, sacc, nxt);
      // vector passes of Algorithm 4's count that stayed in LDS: 4 per step
      // (x_j and w in the update, x_j in the matvec, the store of w), but 1
      // where the step starts without an update
      if (a.keep_xw && kp_tid() == 0)
        L.onchip += 4 * max(1, L.arnoldi_steps - steps0) - (c.upd ? 0 : 3);
      break;
    }
    case PH_CLOSE:
      reduce_partials(a, kS, tv, sacc);
      block_close(a, tv, L, nxt);
      break;
    case PH_EXPM:
      store_tables_b(a, L, false, c.j);
      expm_phase<false>(a, lds, L, nxt);
      break;
    case PH_COMBINE:
      leader_combine(a, L, nxt);
      break;
    case PH_FINISH:
      store_tables_b(a, L, false, c.j);
      if (kp_tid() == 0) nxt.phase = PH_DONE;
      break;
    default:
      break;
  }
  KP_TS(a, k, 6);
  bar_release(a, k, nxt, a.pub);
  KP_TS(a, k, 7);
  if (c.phase == PH_STEP) {
    bar_count(a);
    block_post(c.j, L);
  }
  if (kp_tid() == 0) cur = nxt;
}

template <int R>
__global__ __launch_bounds__(kThreads) void k_blk(Args a, int arnoldi_only) {
  __shared__ __attribute__((aligned(16))) double lds[kLdsDoublesB];
  __shared__ LeadB lead;
  __shared__ Ctl cur, nxt;
  __shared__ int ok;
  __shared__ unsigned s_k;
  if (kp_tid() == 0) {
    const unsigned long long w = cload(release_word(a));
    s_k = (unsigned)(w >> 32);
    cur = ctl_unpack((unsigned)w, a.block != 0);
    ok = aborted(a) ? 0 : 1;
  }
  if (wg_rank(a) == 0) load_tables_b(a, lead, arnoldi_only != 0);
  __syncthreads();
  unsigned k = s_k;
  for (;;) {
    __syncthreads();
    if (!ok || cur.phase == PH_DONE) break;
    if (arnoldi_only && (cur.phase == PH_EXPM || cur.phase == PH_COMBINE || cur.phase == PH_FINISH ||
                         (cur.phase == PH_STEP && cur.j >= a.stop_j)))
      break;
    ++k;
    run_phase_block<R>(a, lds, lead, cur, nxt, ok, k);
  }
  if (arnoldi_only && wg_rank(a) == 0) store_tables_b(a, lead, true, cur.j);
}

static_assert(sizeof(LeadB) >= kKeepMax * sizeof(double) && kHaloCap >= 2 * kKeepMax, "on-chip buffers");

// The whole call (or, for the step-by-step entry, the steps up to stop_j).
template <typename TB, bool MS>
__global__ __launch_bounds__(kThreads) void k_run(Args a, int arnoldi_only) {
  __shared__ __attribute__((aligned(16))) double lds[kLdsDoubles];
  __shared__ LeadLds lead;
  __shared__ Ctl cur, nxt;
  __shared__ int ok;
  __shared__ int kept;
  __shared__ unsigned s_k;
  if (kp_tid() == 0) {
    kept = -1;
    // barriers released by earlier launches, and the control they announced
    const unsigned long long w = cload(release_word(a));
    s_k = (unsigned)(w >> 32);
    cur = ctl_unpack((unsigned)w, a.block != 0);
    ok = aborted(a) ? 0 : 1;
  }
  if (wg_rank(a) == 0) load_tables(a, lead);
  __syncthreads();
  unsigned k = s_k;
  for (;;) {
    __syncthreads();
    if (!ok || cur.phase == PH_DONE) break;
    if (arnoldi_only &&
        (cur.phase == PH_EXPM || cur.phase == PH_COMBINE || cur.phase == PH_FINISH ||
         ((cur.phase == PH_STEP || cur.phase == PH_MVEC) && cur.j >= a.stop_j)))
      break;
    ++k;
    run_phase<TB, MS>(a, lds, lead, cur, nxt, ok, kept, k);
  }
}

// Reset of the call state by nb workgroups of any size, this one being number
// b, before the launch that solves the problem: the step buffers are marked
// empty; the Hessenberg and correction matrices are zeroed so that entries
// outside their triangles read as zero (block steps keep them in LDS and
// mask instead).
__device__ inline void init_problem(const Args& a, int m_target, int nflags, int b, int nb) {
  State* st = a.st;
  {
    double* sp = a.part + (int64_t)a.part_rows * kCStride;
    const int n = a.block ? 2 * (a.part_rows + 1) * a.bstride : 2 * a.part_rows * kKStride;
    const double empty = __builtin_bit_cast(double, kPartEmpty);
    for (int i = b * (int)blockDim.x + kp_tid(); i < n; i += nb * (int)blockDim.x) sp[i] = empty;
  }
  if (a.ll) {
    const int64_t n = 2 * ll_doubles(a) + 2 * kPMax;
    for (int64_t i = b * (int)blockDim.x + kp_tid(); i < n; i += nb * (int)blockDim.x) a.hx2[i] = 0.0;
  }
  if (b != 0) return;
  for (int i = kp_tid(); i < kMMax + 2; i += blockDim.x) a.pub->coefs[0][i] = a.pub->coefs[1][i] = a.pub->coefs[2][i] = 0.0;
  for (int i = kp_tid(); i < nflags; i += blockDim.x) a.flags[i] = 0u;
  if (!a.block) for (int i = kp_tid(); i < kLdh * kMMax; i += blockDim.x) st->H[i] = 0.0;
  if (!a.block)
    for (int i = kp_tid(); i < kLdt * kMMax; i += blockDim.x) {
      st->Lm[i] = 0.0;
      st->Minv[i] = 0.0;
    }
  if (kp_tid() != 0) return;
  for (int i = 0; i < 16; ++i) a.sync[i] = 0u;   // counters, release word (STAGE), abort
  Pub* pb = a.pub;
  pb->phase = PH_STAGE;
  pb->upd = 0;
  pb->j = 0;
  pb->m_eff = 0;
  pb->last = 0;
  pb->status = KP_STATUS_OK;
  pb->inv_mu = 1.0;
  pb->xscale = 1.0;
  pb->shift = 0.0;
  st->m_target = m_target;
  st->m_cur = m_target;
  st->breakdown = 0;
  st->fallback_cur = 0;
  st->substeps = st->rejected = st->arnoldi_steps = st->expm_evals = 0;
  st->n_fallback = st->breakdowns = st->nlog = st->zero = 0;
  st->m_last = 0;
  st->onchip = 0;
  st->nopair = 0;
  st->theta = 0.0;
  st->t = 0.0;
  st->tau = a.tau0;
  st->beta = 0.0;
  st->mu = 1.0;
  st->err_max = st->omega = st->err = st->last_nrm2 = st->omega_prev = 0.0;
}

// The main call's kernel is instantiated first, so that it leads the code
// object and its placement does not move when the other kernels change size
// (its run time varied by about 1 % with placement alone, with identical
// instructions).
template __global__ void k_blk<4>(Args, int);
template __global__ void k_run<float, false>(Args, int);
template __global__ void k_blk<2>(Args, int);
template __global__ void k_blk<1>(Args, int);
template __global__ void k_run<double, true>(Args, int);
template __global__ void k_run<float, true>(Args, int);
template __global__ void k_run<double, false>(Args, int);

__global__ __launch_bounds__(256) void k_init(Args a, int m_target) {
  init_problem(a, m_target, a.nwg * kFlagStride, (int)blockIdx.x, (int)gridDim.x);
}

// ---- batched call ------------------------------------------------------------
//
// Many independent problems in one cooperative launch.  The grid is split into
// teams of consecutive workgroups; the teams of one size form a class and
// occupy a consecutive run of the grid.  Each class has a queue of problems,
// heaviest first (the host planner's assignment).  A team's leader takes the
// next problem from the front of its class's queue and, once that is empty,
// the lightest remaining problem from the back of the queue of a class of
// smaller teams, and hands it to the team's other workgroups through the
// team's slot.  The team
// then solves it exactly as a single call would (its own Args with the
// class's geometry, State, control block and barrier words), so the phases,
// barriers and coherence rules are those of k_run inside each team.  Every
// buffer a problem writes is its own (basis, state vector, partial sums, halo
// rows, tail values, small-exponential scratch): a team never takes over
// memory another workgroup wrote with plain stores in the same launch (the
// L2s of different XCDs are not coherent for plain stores).  A problem's last
// barrier (FINISH -> DONE) is passed by the whole team before its leader
// takes the next one.
//
// The Args records are read through the constant address space: they are not
// written during the launch and every access has a uniform address, so their
// fields are fetched with scalar loads, as kernel arguments are.
typedef __attribute__((address_space(4))) const Args CArgs;

struct BatchDesc {
  const CArgs* args;       // [nclass][nprob], not written during the launch
  const int* order;        // problems of class c, heaviest first: order[class_first[c] ..)
  const int* class_first;  // [nclass + 1]
  const int* team_of_wg;   // [grid] (-1: no team)
  const int* team_class;   // [nteams]
  const int* team_wg0;     // [nteams]
  unsigned long long* queue;   // [nclass]: front (low 32 bits), back (high) (coherent)
  unsigned long long* slot;    // [nteams * 8]: (sequence << 32) | (problem + 1) (coherent)
  int nprob, nclass, nteams;
  int64_t wait_ticks;      // bound of a team member's wait for its next problem
};

__device__ inline const Args& batch_args(const CArgs* base, int i) {
  return *(const Args*)(base + i);
}

// Problem of class c's queue taken from the front (heavy end) or the back
// (light end); -1 when the queue is empty.
__device__ inline int queue_take(const BatchDesc& d, int c, bool front) {
  unsigned long long* q = d.queue + c;
  unsigned long long w = cload(q);
  for (;;) {
    const unsigned f = (unsigned)w, b = (unsigned)(w >> 32);
    if (f >= b) return -1;
    const unsigned long long nw = front ? (w + 1ull) : (w - (1ull << 32));
    if (__hip_atomic_compare_exchange_strong(q, &w, nw, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT))
      return d.order[d.class_first[c] + (int)(front ? f : b - 1)];
  }
}

// Reset of every problem (one workgroup each) and, by workgroup 0, of the
// class queues and the team slots.
__global__ __launch_bounds__(256) void k_batch_init(BatchDesc d) {
  const int i = (int)blockIdx.x;
  const Args& a = batch_args(d.args, i);
  int nflags = 0;
  for (int c = 0; c < d.nclass; ++c)
    nflags = max(nflags, batch_args(d.args, c * d.nprob + i).nwg * kFlagStride);
  init_problem(a, a.m0, nflags, 0, 1);
  if (i == 0) {
    for (int c = kp_tid(); c < d.nclass; c += blockDim.x)
      d.queue[c] = (unsigned long long)(d.class_first[c + 1] - d.class_first[c]) << 32;
    for (int t = kp_tid(); t < d.nteams * 8; t += blockDim.x) d.slot[t] = 0ull;
  }
}

// BLK: block steps, as in k_blk; else the phases of k_run.
template <typename TB, bool MS, bool BLK = false>
__global__ __launch_bounds__(kThreads) void k_batch(BatchDesc d) {
  __shared__ __attribute__((aligned(16))) double lds[BLK ? kLdsDoublesB : kLdsDoubles];
  __shared__ std::conditional_t<BLK, LeadB, LeadLds> lead;
  __shared__ Ctl cur, nxt;
  __shared__ int ok, s_pi;
  __shared__ int kept;   // keep_xw is off in batched calls; never set
  __shared__ unsigned s_k;
  const int t = __builtin_amdgcn_readfirstlane(d.team_of_wg[blockIdx.x]);
  if (t < 0) return;
  if (kp_tid() == 0) kept = -1;
  const int c = __builtin_amdgcn_readfirstlane(d.team_class[t]);
  const bool lead_wg = (int)blockIdx.x == __builtin_amdgcn_readfirstlane(d.team_wg0[t]);
  unsigned long long* slot = d.slot + 8 * (size_t)t;
  for (unsigned seq = 1;; ++seq) {
    // the team's next problem: chosen by the leader, handed to the others
    if (kp_tid() == 0) {
      int pi = -1;
      if (lead_wg) {
        // own class first; then the light end of the classes of smaller
        // teams (classes are ordered by decreasing team size), solved with
        // its planned row partition (the Args of such a (class, problem)
        // pair), so its result is the same whichever team takes it
        pi = queue_take(d, c, true);
        for (int cc = c + 1; pi < 0 && cc < d.nclass; ++cc) pi = queue_take(d, cc, false);
        cstore(slot, ((unsigned long long)seq << 32) | (unsigned)(pi + 1));
      } else {
        // bounded wait on the leader (it publishes as soon as the previous
        // problem's last barrier is released)
        const int64_t t0 = wall_clock64();
        unsigned long long w = cload(slot);
        while ((unsigned)(w >> 32) < seq) {
          __builtin_amdgcn_s_sleep(1);
          w = cload(slot);
          if (wall_clock64() - t0 > d.wait_ticks) break;
        }
        pi = ((unsigned)(w >> 32) >= seq) ? (int)(unsigned)w - 1 : -1;
      }
      s_pi = pi;
    }
    __syncthreads();
    const int pi = __builtin_amdgcn_readfirstlane(s_pi);
    if (pi < 0) break;
    const Args& a = batch_args(d.args, c * d.nprob + pi);
    if (kp_tid() == 0) {
      const unsigned long long w = cload(release_word(a));
      s_k = (unsigned)(w >> 32);
      cur = ctl_unpack((unsigned)w, a.block != 0);
      ok = aborted(a) ? 0 : 1;
    }
    if (wg_rank(a) == 0) {
      if constexpr (BLK)
        load_tables_b(a, lead, false);
      else
        load_tables(a, lead);
    }
    __syncthreads();
    unsigned k = s_k;
    for (;;) {
      __syncthreads();
      if (!ok || cur.phase == PH_DONE) break;
      ++k;
      if constexpr (BLK)
        run_phase_block<kRBatch>(a, lds, lead, cur, nxt, ok, k);
      else
        run_phase<TB, MS>(a, lds, lead, cur, nxt, ok, kept, k);
    }
    __syncthreads();
    if (!ok) break;   // a bounded wait gave up: this team stops
  }
}

// Outcome of every problem of a batched call (one thread per problem, after
// the batched kernel has finished).  A problem whose team stopped before
// finishing it reports KP_STATUS_ABORTED.
__global__ __launch_bounds__(64) void k_batch_info(BatchDesc d, kp_info* out) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= d.nprob) return;
  const Args& a = batch_args(d.args, i);
  const State* st = a.st;
  const Pub* pb = a.pub;
  kp_info r;
  r.status = (a.sync[kSyncAbort] != 0u || pb->phase != PH_DONE) ? (int)KP_STATUS_ABORTED
                                                                  : pb->status;
  r.substeps = st->substeps;
  r.rejected = st->rejected;
  r.arnoldi_steps = st->arnoldi_steps;
  r.expm_evals = st->expm_evals;
  r.m_last = st->m_last;
  r.n_fallback = st->n_fallback;
  r.breakdowns = st->breakdowns;
  r.schedule_len = min(st->nlog, kLogMax);
  r.onchip_passes = st->onchip;   // (0: batched problems keep nothing in LDS)
  r.err_max = st->err_max;
  r.mu = st->mu;
  r.t_end = st->t;
  out[i] = r;
}

// Right-hand sides of the derivative of the phi combination along a
// constant-coefficient stencil direction L that commutes with A (periodic
// constant-coefficient ADR: both are circulant):
//   d/dtheta sum_k h^k phi_k(hA) b_k = sum_{j=0}^{p+1} h^j phi_j(hA) c_j,
//   c_j = h L b_j - (j - 1) L b_{j-1}   (b_{p+1} = b_{-1} = 0),
// from d/dtheta phi_k(hA) = h L phi_k'(hA) and phi_k' = phi_k - k phi_{k+1}.
// L = lc (Lap) - la.(Dx, Dy) (sign flipped when transposed) + lr I on the
// nx x ny periodic grid.  One thread per grid point and column; C is
// N x (p+2) with leading dimension N.
__global__ __launch_bounds__(256) void k_dir_rhs(const double* B, int64_t ldb, int p, int nx,
                                                 int ny, double cx, double cy, double adx,
                                                 double ady, double lr, int transpose, double h,
                                                 double* C) {
  const int64_t npt = (int64_t)nx * ny;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= npt * (p + 2)) return;
  const int j = (int)(t / npt);
  const int64_t e = t - (int64_t)j * npt;
  const int row = (int)(e / nx), ix = (int)(e - (int64_t)row * nx);
  const int64_t ie = row * (int64_t)nx + (ix + 1 == nx ? 0 : ix + 1);
  const int64_t iw = row * (int64_t)nx + (ix == 0 ? nx - 1 : ix - 1);
  const int64_t in = (row + 1 == ny ? 0 : row + 1) * (int64_t)nx + ix;
  const int64_t is = (row == 0 ? ny - 1 : row - 1) * (int64_t)nx + ix;
  auto Lb = [&](int k) {
    const double* b = B + (int64_t)k * ldb;
    const double c = b[e];
    const double adv = adx * (b[ie] - b[iw]) + ady * (b[in] - b[is]);
    return cx * (b[ie] + b[iw] - 2.0 * c) + cy * (b[in] + b[is] - 2.0 * c) +
           (transpose ? adv : -adv) + lr * c;
  };
  double v = 0.0;
  if (j <= p) v += h * Lb(j);
  if (j >= 1) v -= (double)(j - 1) * Lb(j - 1);
  C[t] = v;
}

// <x, y> in a fixed order (the gradient of the loss in an operator
// coefficient): 256 workgroups each reduce one contiguous chunk, then one
// workgroup sums the 256 partials.
constexpr int kDotBlocks = 256;

__global__ __launch_bounds__(256) void k_dot_partial(const double* x, const double* y, int64_t n,
                                                     double* part) {
  __shared__ double red[4];
  const int64_t chunk = (n + kDotBlocks - 1) / kDotBlocks;
  const int64_t lo = (int64_t)blockIdx.x * chunk, hi = min(n, lo + chunk);
  double s = 0.0;
  for (int64_t e = lo + threadIdx.x; e < hi; e += 256) s += x[e] * y[e];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void k_dot_final(const double* part, double* out) {
  __shared__ double red[4];
  double s = part[threadIdx.x];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *out = (red[0] + red[1]) + (red[2] + red[3]);
}

// Zero fill of n doubles (a kernel rather than a memset node, so that a
// caller may capture the enqueuing call in a graph and replay it).
__global__ __launch_bounds__(256) void k_zero(double* x, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += stride) x[e] = 0.0;
}

// ---- exponential integrators (Section 4.1): right-hand side and remainders --
// One thread per grid point of an nx x ny periodic grid; the linear part is
// nu Lap v - ax Dx v - ay Dy v with the operators' second-order differences.

struct RhsK {
  int kind, nx, ny;
  double cx, cy;      // nu / dx^2, nu / dy^2
  double adx, ady;    // ax / (2 dx), ay / (2 dy)
  double gamma;
};

struct Nbr {
  int64_t e, ie, iw, in, is;
};

__device__ inline Nbr nbr_at(const RhsK& r, int64_t e) {
  const int iy = (int)(e / r.nx), ix = (int)(e - (int64_t)iy * r.nx);
  Nbr b;
  b.e = e;
  b.ie = (int64_t)iy * r.nx + (ix + 1 == r.nx ? 0 : ix + 1);
  b.iw = (int64_t)iy * r.nx + (ix == 0 ? r.nx - 1 : ix - 1);
  b.in = (int64_t)(iy + 1 == r.ny ? 0 : iy + 1) * r.nx + ix;
  b.is = (int64_t)(iy == 0 ? r.ny - 1 : iy - 1) * r.nx + ix;
  return b;
}

// (nu Lap - ax Dx - ay Dy) of the grid function d(.) at b.e
template <typename F>
__device__ inline double lin_at(const RhsK& r, const Nbr& b, F d) {
  const double c = d(b.e), ve = d(b.ie), vw = d(b.iw), vn = d(b.in), vs = d(b.is);
  return r.cx * (ve + vw - 2.0 * c) + r.cy * (vn + vs - 2.0 * c) -
         (r.adx * (ve - vw) + r.ady * (vn - vs));
}

// The nonlinear term and its derivative at a point value x.
__device__ inline double nl_term(const RhsK& r, double x) {
  return r.kind == KP_RHS_ALLEN_CAHN ? x - x * x * x : r.gamma * x * (x - 0.5) * (1.0 - x);
}
__device__ inline double nl_deriv(const RhsK& r, double x) {
  return r.kind == KP_RHS_ALLEN_CAHN ? 1.0 - 3.0 * x * x : r.gamma * (-3.0 * x * x + 3.0 * x - 0.5);
}

// f = f(u); jd (when non-null) = the Jacobian's diagonal field at u (the
// ADR kind's KP_OP_ADR field); B (when non-null) = [0, f] (N x 2, ld ldb).
__global__ __launch_bounds__(256) void k_rhs(RhsK r, const double* u, double* f, double* jd,
                                             double* B, int64_t ldb) {
  const int64_t n = (int64_t)r.nx * r.ny;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const Nbr b = nbr_at(r, e);
  const double x = u[e];
  const double v = lin_at(r, b, [&](int64_t i) { return u[i]; }) + nl_term(r, x);
  f[e] = v;
  if (jd) jd[e] = nl_deriv(r, x);
  if (B) {
    B[e] = 0.0;
    B[ldb + e] = v;
  }
}

// The remainder R(w) = f(w) - f(u_n) - J_n (w - u_n) at b.e.
__device__ inline double remainder_at(const RhsK& r, const Nbr& b, const double* un,
                                      const double* fn, const double* w, const double* fw) {
  const auto d = [&](int64_t i) { return w[i] - un[i]; };
  const double jd = lin_at(r, b, d) + nl_deriv(r, un[b.e]) * d(b.e);
  return fw[b.e] - fn[b.e] - jd;
}

// EPI columns of step n: B = [0, f_n, b_2, .., b_M] with
// b_m = sum_i alpha_{m,i} R(u_{n-i}) / h^{m-1} (v_m = h sum_i alpha_{m,i} R_i,
// b_m = v_m / h^m).  u[k], f[k] = u_{n-k}, f(u_{n-k}).
struct EpiK {
  const double* u[4];
  const double* f[4];
  double alpha[4][3];   // alpha[m-1][i-1]
  double hinv[4];       // hinv[m-1] = 1 / h^{m-1}
  int M, P;
};

__global__ __launch_bounds__(256) void k_epi_cols(RhsK r, EpiK q, double* B, int64_t ldb) {
  const int64_t n = (int64_t)r.nx * r.ny;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const Nbr b = nbr_at(r, e);
  double R[3] = {0.0, 0.0, 0.0};
  for (int i = 1; i <= q.P; ++i) R[i - 1] = remainder_at(r, b, q.u[0], q.f[0], q.u[i], q.f[i]);
  B[e] = 0.0;
  B[ldb + e] = q.f[0][e];
  for (int m = 2; m <= q.M; ++m) {
    double s = 0.0;
    for (int i = 1; i <= q.P; ++i) s += q.alpha[m - 1][i - 1] * R[i - 1];
    B[(int64_t)m * ldb + e] = s * q.hinv[m - 1];
  }
}

// SRERK3 second stage: B = [0, f_n, 0, c3 R(z)] with c3 = 32/9 / h^2.
__global__ __launch_bounds__(256) void k_srerk_cols(RhsK r, const double* un, const double* fn,
                                                    const double* z, const double* fz, double c3,
                                                    double* B, int64_t ldb) {
  const int64_t n = (int64_t)r.nx * r.ny;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const Nbr b = nbr_at(r, e);
  B[e] = 0.0;
  B[ldb + e] = fn[e];
  B[2 * ldb + e] = 0.0;
  B[3 * ldb + e] = c3 * remainder_at(r, b, un, fn, z, fz);
}

// out = a + y.
__global__ __launch_bounds__(256) void k_axpy(double* out, const double* a, const double* y,
                                              int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += stride) out[e] = a[e] + y[e];
}

// A deterministic non-degenerate right-hand side for the calibration solves.
__global__ __launch_bounds__(256) void k_fill_pattern(double* x, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += stride)
    x[e] = sin(0.37 * (double)(e + 1)) + 0.5 * cos(0.0101 * (double)e);
}

// Plain streaming read (kp_read_bandwidth): each thread sums its 16-byte
// elements of x, four loads in flight per round, and one lane per wave
// stores its sum (so the loads are not dead); the practical HBM read rate.
__global__ __launch_bounds__(kThreads) void k_read_probe(const double2* x, int64_t n2,
                                                         double* sink) {
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  double s = 0.0;
  for (; e + 3 * stride < n2; e += 4 * stride) {
    const double2 v0 = x[e], v1 = x[e + stride], v2 = x[e + 2 * stride], v3 = x[e + 3 * stride];
    s += (v0.x + v0.y) + (v1.x + v1.y) + (v2.x + v2.y) + (v3.x + v3.y);
  }
  for (; e < n2; e += stride) s += x[e].x + x[e].y;
  if ((threadIdx.x & 63) == 0) sink[(int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6)] = s;
}

// Small exponential alone (test entry): F = exp(tau Hbar_m) e_1.  H and F are in
// the small exponential's scratch, not in the State: a paused Arnoldi process
// resumes from the H there (block steps make their columns from it).
__global__ __launch_bounds__(kThreads) void k_expm_test(const double* H, double* F, int m, double tau) {
  __shared__ __attribute__((aligned(16))) double lds[kLdsDoubles];
  expm_hbar(HessCol{H, kLdh}, m, tau, false, F, lds);
}
static_assert(kLdh * kMMax + kNmPad <= kExSlots * kNmPad * kNmPad, "H and F of the test entry");

// Workspace of the allocation-free entry point (kp_phi_combo_noalloc): one
// array per GPU, 32 MiB above KP_NOALLOC_BYTES for the halo rows and partial
// sums of the block steps' finer partition (noalloc_need), held by the loaded code object until the process ends.  Host
// code reaches it only through the address hipGetSymbolAddress returns for
// the current device (the array's name in host code is a host-side stand-in).
constexpr size_t kScratchBytes = (size_t)KP_NOALLOC_BYTES + ((size_t)32 << 20);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

}  // namespace kp

// ============================================================================
// Host side
// ============================================================================

using kp::Args;
using kp::Pub;
using kp::State;

struct BatchCache;

struct kp_ctx {
  kp_config cfg;
  hipStream_t stream = nullptr;
  int device = 0;
  int ncu = 0;
  int64_t wait_ticks = 0;
  void* V = nullptr;
  size_t v_bytes = 0;
  double* u = nullptr;
  size_t u_bytes = 0;
  double* part = nullptr;
  size_t part_bytes = 0;
  double* hx = nullptr;
  size_t hx_bytes = 0;
  unsigned* flags = nullptr;
  size_t flags_bytes = 0;
  unsigned* sync = nullptr;
  State* st = nullptr;
  Pub* pub = nullptr;
  double* ex = nullptr;
  double* tx = nullptr;
  double* aux = nullptr;           // backward: [0...0 g] matrix, tangent outputs, dot partials
  size_t aux_bytes = 0;
  double* integ = nullptr;         // integrators: state and right-hand-side history, columns
  size_t integ_bytes = 0;
  int occ[7] = {-1, -1, -1, -1, -1, -1, -1};
  Args last{};
  int have_begin = 0;
  int arn_target = 0;
  BatchCache* batch = nullptr;   // plan, workspace and graph of the last batched call
  State* st_last = nullptr;      // State of the last single call
  kp::PlanModel model;           // the batched planner's cost model (kp_calibrate)
  int model_gen = 0;             // bumped when the model changes (part of the plan key)
  long long* ts = nullptr;       // device timeline of single calls (KP_TIMELINE builds)
  int ts_kmax = 0;
  char err[512] = {0};
};

namespace {

int hip_fail(kp_ctx* c, hipError_t e, const char* what) {
  if (c) snprintf(c->err, sizeof(c->err), "%s: %s", what, hipGetErrorString(e));
  return KP_EHIP;
}

#define KP_HIP(ctx, call)                                   \
  do {                                                      \
    hipError_t e_ = (call);                                 \
    if (e_ != hipSuccess) return hip_fail(ctx, e_, #call);  \
  } while (0)

int check_config(const kp_config* c) {
  if (c->orth < 0 || c->orth > KP_ORTH_IOCGS) return KP_EINVAL;
  if (c->controller != KP_CTRL_POWER && c->controller != KP_CTRL_PI) return KP_EINVAL;
  if (c->rows_per_wg < 0) return KP_EINVAL;
  if (c->basis_dtype != KP_BASIS_F64 && c->basis_dtype != KP_BASIS_F32) return KP_EINVAL;
  if (c->m_init < 0 || c->m_init > KP_MMAX) return KP_EINVAL;
  if (!std::isfinite(c->tau_init) || c->tau_init < 0.0) return KP_EINVAL;
  if (c->max_substeps < 0 || c->fixed_m < 0 || c->fixed_m > KP_MMAX) return KP_EINVAL;
  if (c->fixed_m > 0 && c->fixed_substeps < 1) return KP_EINVAL;
  if (c->fixed_substeps < 0) return KP_EINVAL;
  if (!std::isfinite(c->fallback_delta) || !std::isfinite(c->breakdown_eps)) return KP_EINVAL;
  if (c->breakdown_eps < 0.0) return KP_EINVAL;
  return KP_OK;
}

bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  if (!a || !b || na == 0 || nb == 0) return false;
  const char* pa = static_cast<const char*>(a);
  const char* pb = static_cast<const char*>(b);
  return pa < pb + nb && pb < pa + na;
}

// Validate the operator and problem; fill the problem part of Args.
// No HIP call happens here.
int build_args(const kp_ctx* ctx, const kp_op* A, const double* B, int p, int64_t ldb,
               double h, double tol, int m_max, double* out, bool need_out, Args* a) {
  if (!ctx || !A || !B) return KP_EINVAL;
  if (need_out && !out) return KP_EINVAL;
  if (A->kind < KP_OP_ADR || A->kind > KP_OP_BRUSSELATOR) return KP_EINVAL;
  if (A->nx < 1 || A->ny < 1) return KP_EINVAL;
  if (!(A->dx > 0.0) || !(A->dy > 0.0) || !std::isfinite(A->dx) || !std::isfinite(A->dy))
    return KP_EINVAL;
  const double coefs[] = {A->nu, A->nu2, A->ax, A->ay, A->react, A->brus_a, A->brus_b};
  for (double v : coefs)
    if (!std::isfinite(v)) return KP_EINVAL;
  if (A->kind == KP_OP_ALLEN_CAHN && !A->field0) return KP_EINVAL;
  if (A->kind == KP_OP_BRUSSELATOR && (!A->field0 || !A->field1)) return KP_EINVAL;
  const int nplanes = A->kind == KP_OP_BRUSSELATOR ? 2 : 1;
  const int64_t npt = (int64_t)A->nx * A->ny;
  const int64_t N = npt * nplanes;
  if (N > (int64_t)1 << 30) return KP_EINVAL;
  if (p < 0 || p > KP_PMAX) return KP_EINVAL;
  if (ldb < N) return KP_EINVAL;
  if (m_max < 1 || m_max > KP_MMAX) return KP_EINVAL;
  if (!(h >= 0.0) || !std::isfinite(h)) return KP_EINVAL;
  const kp_config& cfg = ctx->cfg;
  if (cfg.fixed_m == 0 && !(tol > 0.0 && std::isfinite(tol))) return KP_EINVAL;
  if (cfg.fixed_m > m_max) return KP_EINVAL;
  if (need_out) {
    const size_t ob = (size_t)N * sizeof(double);
    const size_t bb = (size_t)ldb * (p + 1) * sizeof(double);
    if (overlaps(out, ob, B, bb)) return KP_EINVAL;
    if (overlaps(out, ob, A->field0, (size_t)npt * sizeof(double))) return KP_EINVAL;
    if (overlaps(out, ob, A->field1, (size_t)npt * sizeof(double))) return KP_EINVAL;
  }
  Args r{};
  r.B = B;
  r.ldb = ldb;
  r.f0 = A->field0;
  r.f1 = A->field1;
  r.out = out;
  r.N = (int)N;
  r.p = p;
  r.pb = p;
  r.tangent = 0;
  r.dout = nullptr;
  r.wg0 = 0;
  r.npt = (int)npt;
  r.nx = A->nx;
  r.ny = A->ny;
  r.nplanes = nplanes;
  r.npt_pad = (npt + kp::kPlaneAlign - 1) / kp::kPlaneAlign * kp::kPlaneAlign;
  if (nplanes == 2) r.npt_pad += kp::kPlaneSkew;
  r.tail_off = r.npt_pad * nplanes;
  r.ld = r.tail_off + kp::kTailPad;
  r.kind = A->kind;
  r.transpose = A->transpose ? 1 : 0;
  r.cx = A->nu / (A->dx * A->dx);
  r.cy = A->nu / (A->dy * A->dy);
  r.cx2 = A->nu2 / (A->dx * A->dx);
  r.cy2 = A->nu2 / (A->dy * A->dy);
  r.inv_nx = 1.0 / (double)A->nx;
  r.halo_lds = (2 * nplanes * (int64_t)A->nx <= kp::kHaloCap) ? 1 : 0;
  r.adx = A->ax / (2.0 * A->dx);
  r.ady = A->ay / (2.0 * A->dy);
  r.react = A->react;
  r.ba = A->brus_a;
  r.bb = A->brus_b;
  r.orth = cfg.orth;
  r.controller = cfg.controller;
  r.fixed_m = cfg.fixed_m;
  r.fixed_substeps = cfg.fixed_m > 0 ? cfg.fixed_substeps : 0;
  r.max_substeps = cfg.max_substeps > 0 ? cfg.max_substeps : 2000;
  r.m_max = m_max;
  r.m0 = cfg.fixed_m > 0 ? cfg.fixed_m : std::min(cfg.m_init > 0 ? cfg.m_init : 16, m_max);
  r.tau0 = cfg.fixed_m > 0 ? h / (double)std::max(1, cfg.fixed_substeps)
                           : (cfg.tau_init > 0.0 ? std::min(cfg.tau_init, h) : h);
  r.stop_j = INT_MAX;
  r.basis_f32 = cfg.basis_dtype == KP_BASIS_F32 ? 1 : 0;
  r.block = (!r.basis_f32 && !kp::orth_multi_sync(r.orth)) ? 1 : 0;
  r.bstride = kp::kNv * m_max + 24;
  r.tile_r = kp::kRBatch;
  r.h = h;
  r.tol = tol > 0.0 ? tol : 1.0;
  r.delta = cfg.fallback_delta == 0.0 ? 1e-10 : (cfg.fallback_delta < 0.0 ? 0.0 : cfg.fallback_delta);
  r.eps_bd = cfg.breakdown_eps == 0.0 ? 1e-12 : cfg.breakdown_eps;
  // several steps per reduction: H-GSMGS only (see kp_block.h).  A fallback
  // threshold above the guard takes the exact norm at every step, so there is
  // no estimate to divide a first vector by.  The later vectors of a block are
  // held against the guard alone (0.01 of a norm), so a breakdown threshold
  // that comes near it (default 1e-12) is tested step by step.
  r.pairs = (r.block && r.orth == KP_ORTH_H_GSMGS && r.delta <= kp::kGuard && r.eps_bd <= kp::kGuard) ? 1 : 0;
  *a = r;
  return KP_OK;
}

int occupancy(kp_ctx* ctx, const void* kernel, int which) {
  if (ctx->occ[which] < 0) {
    int occ = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, kp::kThreads, 0);
    if (e != hipSuccess) return -1;
    ctx->occ[which] = occ;
  }
  return ctx->occ[which];
}

// The persistent kernel that runs a's process.
const void* run_kernel(const Args& a) {
  if (a.block)
    return a.tile_r == 1   ? reinterpret_cast<const void*>(&kp::k_blk<1>)
           : a.tile_r == 2 ? reinterpret_cast<const void*>(&kp::k_blk<2>)
                           : reinterpret_cast<const void*>(&kp::k_blk<4>);
  if (kp::orth_multi_sync(a.orth))
    return a.basis_f32 ? reinterpret_cast<const void*>(&kp::k_run<float, true>)
                       : reinterpret_cast<const void*>(&kp::k_run<double, true>);
  return a.basis_f32 ? reinterpret_cast<const void*>(&kp::k_run<float, false>)
                     : reinterpret_cast<const void*>(&kp::k_run<double, false>);
}

// Single calls of the forms without block steps on large grids: k_blk holds six
// vectors' registers for their two and streams with shorter chunks, which costs
// more there than its shorter latencies save (H-CWY, one substep of 64 steps:
// 1024^2 7.57 ms, 6.50 in k_run; 700^2 4.29, 3.92; 634 x 348 adaptive 2.75, 3.55).
constexpr int64_t kSinglesMax = 1 << 18;   // elements up to which k_blk runs single steps
void choose_kernel(Args* a) {
  if (a->block && !a->pairs && (int64_t)a->npt * a->nplanes > kSinglesMax) a->block = 0;
}

// Co-resident workgroups per CU of that kernel (block steps: of every tile
// size, since the geometry, which needs it, chooses among them).
int kernel_occupancy(kp_ctx* ctx, const Args& a) {
  if (!a.block)
    return occupancy(ctx, run_kernel(a),
                     kp::orth_multi_sync(a.orth) ? (a.basis_f32 ? 3 : 2) : (a.basis_f32 ? 1 : 6));
  return std::min({occupancy(ctx, reinterpret_cast<const void*>(&kp::k_blk<4>), 0),
                   occupancy(ctx, reinterpret_cast<const void*>(&kp::k_blk<2>), 4),
                   occupancy(ctx, reinterpret_cast<const void*>(&kp::k_blk<1>), 5)});
}

int device_setup(kp_ctx* ctx) {
  if (ctx->ncu > 0) return KP_OK;
  KP_HIP(ctx, hipGetDevice(&ctx->device));
  int ncu = 0, rate_khz = 0;
  KP_HIP(ctx, hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, ctx->device));
  KP_HIP(ctx, hipDeviceGetAttribute(&rate_khz, hipDeviceAttributeWallClockRate, ctx->device));
  ctx->ncu = ncu;
  if (rate_khz <= 0) rate_khz = 100000;
  // bound of every device-wide wait: 4 s, or KP_WAIT_LIMIT_US microseconds
  // (read when the context first touches the device; for failure tests)
  double limit_s = 4.0;
  if (const char* e = std::getenv("KP_WAIT_LIMIT_US")) {
    const double us = std::atof(e);
    if (us > 0.0 && us < 4.0e6) limit_s = us * 1e-6;
  }
  ctx->wait_ticks = std::max<int64_t>(1, (int64_t)((double)rate_khz * 1000.0 * limit_s));
  return KP_OK;
}

int grow(kp_ctx* ctx, void** p, size_t* have, size_t need) {
  if (*have >= need) return KP_OK;
  if (*p) {
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipStreamSynchronize");
    hipFree(*p);
    *p = nullptr;
    *have = 0;
  }
  hipError_t e = hipMalloc(p, need);
  if (e != hipSuccess) {
    *p = nullptr;
    snprintf(ctx->err, sizeof(ctx->err), "hipMalloc(%zu): %s", need, hipGetErrorString(e));
    return KP_ENOMEM;
  }
  *have = need;
  return KP_OK;
}

// Grid geometry: workgroup b owns rows [b*rows, (b+1)*rows) of every plane.
// At least one full sub-tile (kThreads * kR pairs) of elements per workgroup
// (or the configured rows_per_wg), at most one workgroup per co-resident slot;
// an even row count when nx is odd keeps every segment start even (pair
// alignment).  Where a one-reduction form runs on one plane, the largest row
// count whose rows fit one sub-tile is taken instead when the co-resident
// workgroups still cover the grid with it: x_j and w then stay on chip
// between the passes (keep_xw below).
//
// Block steps (kp_block.h) spread a grid further: down to kSpreadFew elements per
// workgroup while there are at most kFewWgs of them, else to kSpread: a finer
// split takes the streaming time down and adds partial rows to the reduction
// (one call, elements per workgroup: 97 x 61 584 449 us, 388 409; 64 x 64 512
// 444, 256 437, 128 458; 128^2 512 1.76 ms, 256 1.71, 128 1.80; 256^2 1024 3.44 ms,
// 512 3.04, 256 3.56).
// ioCGS (float64 basis) also starts at kSpreadFew, but keeps to kFewWgs workgroups up
// to the 4096 elements its window on chip allows: its phases are short, and every
// arrival costs the leader's gather (two substeps of 40 steps, us by elements per
// workgroup: 64^2 256 1200, 1024 1219, 4096 1398; 256^2 512 1382, 1024 1284, 4096
// 1572; 512^2 1024 2058, 2048 1592, 4096 1687; with 4096 elements, the counted
// barriers and nothing on chip 2015, 2207 and 2438).
// spread = false: the partition without these rules (kp_phi_combo_noalloc's
// capacity is stated for it).
constexpr int64_t kSpread = 512, kSpreadFew = 256;
constexpr int kFewWgs = 64;
constexpr int kLlMax = 256;   // widest rows of the tagged exchange (kp_block.h)

void geometry(int ncu_slots, int rows_cfg, Args* a, bool spread = true) {
  const int64_t per_wg_min = (int64_t)kp::kThreads * kp::kR * 2;
  int64_t rows = (per_wg_min + (int64_t)a->nx * a->nplanes - 1) / ((int64_t)a->nx * a->nplanes);
  if (rows_cfg <= 0 && a->nplanes == 1 && 2 * (int64_t)a->nx <= per_wg_min &&
      !kp::orth_multi_sync(a->orth)) {
    int64_t rk = per_wg_min / a->nx;
    if ((a->nx & 1) && (rk & 1) && rk < a->ny) --rk;
    if (rk >= 1 && rk < rows && (a->ny + rk - 1) / rk <= ncu_slots) rows = rk;
  }
  if (rows_cfg <= 0 && spread && a->orth == KP_ORTH_IOCGS && !a->basis_f32) {
    const int64_t row = (int64_t)a->nx * a->nplanes;
    for (int64_t e = kSpreadFew; e <= kp::kKeepMax; e *= 2) {
      rows = (e + row - 1) / row;
      if ((a->ny + rows - 1) / rows <= kFewWgs) break;
    }
    int64_t cap = kp::kKeepMax / row;          // (whole rows, even ones when nx is odd)
    if (a->nx & 1) cap &= ~(int64_t)1;
    if (cap >= 1) rows = std::min(rows, cap);
  }
  if (rows_cfg <= 0 && spread && a->block) {
    const int64_t row = (int64_t)a->nx * a->nplanes;
    rows = (kSpreadFew + row - 1) / row;
    if ((a->ny + rows - 1) / rows > kFewWgs) rows = (kSpread + row - 1) / row;
  }
  if (rows_cfg > 0) rows = rows_cfg;
  rows = std::max<int64_t>(rows, (a->ny + ncu_slots - 1) / ncu_slots);
  rows = std::max<int64_t>(1, std::min<int64_t>(rows, a->ny));
  if ((a->nx & 1) && (rows & 1) && rows < a->ny) ++rows;
  a->rows_per_wg = (int)rows;
  a->nwg = (int)((a->ny + rows - 1) / rows);
  a->nteam = a->nwg;
  a->part_rows = a->nwg;
  // one plane whose rows per workgroup fit one sub-tile (kThreads * kR
  // pairs): the products read x_j in LDS, where the update before left it, and
  // leave w there for the next update (kp_block.h; with a float basis
  // matvec_dots_pass; ioCGS: iocgs_mvec)
  a->keep_ms = (a->orth == KP_ORTH_IOCGS && !a->basis_f32 && a->nplanes == 1 && spread &&
                rows * a->nx <= kp::kKeepMax && 2 * (int64_t)a->nx <= kp::kKeepMax)
                   ? 1 : 0;
  a->keep_xw = (a->nplanes == 1 && rows * a->nx <= 2 * (int64_t)kp::kThreads * kp::kR &&
                2 * (int64_t)a->nx <= 2 * (int64_t)kp::kThreads * kp::kR &&
                !kp::orth_multi_sync(a->orth) && 4 * kp::kR * kp::kThreads <= kp::kHaloCap)
                   ? 1 : 0;
  if (a->block) {
    // on chip, the smallest tile that holds the rows; otherwise the fewest
    // pairs per thread, counting a tile's reductions as 0.7 of a pair: the fastest
    // of the three on 14 of 15 partitions of 256 to 16384 elements per plane, one
    // and two planes, and 2 % from it at 2100 (one substep of 48 steps, us with 1, 2
    // and 4 pairs: two planes of 1024 1740, 1941, 2434; 2100 3081, 2965, 3022; 4096
    // 5357, 4780, 4659; 5000 6396, 6014, 6313; 8400 10604, 9645, 9749; one plane of
    // 6000 3914, 3461, 3570).  It does not rank the slower two
    double best = 0.0;
    for (int r : {4, 2, 1}) {
      const int64_t tile = (int64_t)2 * kp::kThreads * r, tiles = (rows * a->nx + tile - 1) / tile;
      const double cost = (double)tiles * (r + 0.7);
      if (a->keep_xw && tiles > 1) continue;
      if (best == 0.0 || cost < best) {
        best = cost;
        a->tile_r = r;
      }
    }
    a->ll = (a->keep_xw && a->tile_r == 1 && a->nx <= kLlMax) ? 1 : 0;
  }
}

// Partial sums (doubles) of nwg workgroups: the counted buffer, the two step
// buffers and, for block steps, the two buffers of their sums.
size_t part_doubles(const Args& a, int nwg) {
  return (size_t)nwg * kp::kCStride +
         2 * (a.block ? (size_t)(nwg + 1) * a.bstride : (size_t)nwg * kp::kKStride);
}

// Halo rows (doubles) of nwg workgroups, one buffer; pairs need a second one.
size_t halo_doubles(const Args& a, int nwg) { return (size_t)nwg * a.nplanes * 2 * a.nx; }
// Doubles of the halo area: the plain rows, then the second buffer or the
// tagged ones with the tail's words.
size_t halo_area(const Args& a, int nwg) {
  return halo_doubles(a, nwg) * (a.ll ? 5 : (a.pairs ? 2 : 1)) + (a.ll ? 2 * kp::kPMax : 0);
}

// Workspace that a context keeps beside the basis and the state vector, sized so
// that a call whose coarse partition (geometry without spread) and vectors are
// no larger than those of an earlier call never grows it: the finer partitions
// give a smaller grid more workgroups, tags or halo rows than a larger one, and
// growing stops the stream, is refused under capture and frees what captured
// graphs of earlier calls use.  Partial sums and flags: every slot of the chip at
// the largest stride (1.7 MB).  Halo rows: with nx * planes of 4096 or more both
// partitions are the same, so twice the coarse count; below, two buffers take at
// most 4 N doubles (a row per workgroup) and 4 * 4096 per workgroup slot, the
// tagged exchange's five at most 10 N and 10 kLlMax per slot.
size_t part_kept(int slots) {
  return (size_t)slots * kp::kCStride + 2 * (size_t)(slots + 1) * (kp::kNv * kp::kMMax + 24);
}
static_assert(kp::kNv * kp::kMMax + 24 >= kp::kKStride, "the larger stride of a step buffer");
size_t halo_kept(int slots, int rows_cfg, const Args& a, size_t u_doubles) {
  Args g = a;
  geometry(slots, rows_cfg, &g, false);
  return std::max({halo_area(a, a.nwg), 2 * halo_doubles(g, g.nwg),
                   std::min(4 * u_doubles, (size_t)slots * 4 * 4096),
                   std::min(10 * u_doubles, (size_t)slots * 2 * kLlMax * 5) + 2 * kp::kPMax});
}

// Allocate the workspace for a problem and finish Args.
int prepare(kp_ctx* ctx, Args* a) {
  int rc = device_setup(ctx);
  if (rc) return rc;
  const size_t esz = a->basis_f32 ? sizeof(float) : sizeof(double);
  const size_t vneed = (size_t)a->ld * (size_t)(a->m_max + 2) * esz;
  if ((rc = grow(ctx, &ctx->V, &ctx->v_bytes, vneed))) return rc;
  if ((rc = grow(ctx, reinterpret_cast<void**>(&ctx->u), &ctx->u_bytes,
                 (size_t)a->ld * sizeof(double))))
    return rc;
  choose_kernel(a);
  const int occ = kernel_occupancy(ctx, *a);
  if (occ <= 0) {
    snprintf(ctx->err, sizeof(ctx->err), "the persistent kernel does not fit on a CU");
    return KP_EHIP;
  }
  const int slots = ctx->ncu * occ;
  geometry(slots, ctx->cfg.rows_per_wg, a);
  if ((rc = grow(ctx, reinterpret_cast<void**>(&ctx->part), &ctx->part_bytes,
                 part_kept(slots) * sizeof(double))))
    return rc;
  if ((rc = grow(ctx, reinterpret_cast<void**>(&ctx->hx), &ctx->hx_bytes,
                 halo_kept(slots, ctx->cfg.rows_per_wg, *a, ctx->u_bytes / sizeof(double)) *
                     sizeof(double))))
    return rc;
  if ((rc = grow(ctx, reinterpret_cast<void**>(&ctx->flags), &ctx->flags_bytes,
                 (size_t)slots * kp::kFlagStride * sizeof(unsigned))))
    return rc;
  if (!ctx->st) {
    KP_HIP(ctx, hipMalloc(&ctx->st, sizeof(State)));
    KP_HIP(ctx, hipMalloc(&ctx->pub, sizeof(Pub)));
    KP_HIP(ctx, hipMalloc(&ctx->sync, 64));
    KP_HIP(ctx, hipMalloc(&ctx->ex, sizeof(double) * kp::kExSlots * kp::kNmPad * kp::kNmPad));
    KP_HIP(ctx, hipMalloc(&ctx->tx, sizeof(double) * kp::kTailPad));
  }
  a->V = ctx->V;
  a->u = ctx->u;
  a->part = ctx->part;
  a->hx = ctx->hx;
  a->hx2 = ctx->hx + halo_doubles(*a, a->nwg);
  a->tx = ctx->tx;
  a->flags = ctx->flags;
  a->sync = ctx->sync;
  a->st = ctx->st;
  a->pub = ctx->pub;
  a->ex = ctx->ex;
  a->wait_ticks = ctx->wait_ticks;
#ifdef KP_TIMELINE
  a->ts = ctx->ts;
  a->ts_kmax = ctx->ts_kmax;
#endif
  return KP_OK;
}

// The buffers prepare() allocates, carved 256-byte aligned from one region
// at base (nullptr: only the size).  Returns the bytes the problem needs.
size_t carve(Args* a, char* base) {
  const size_t esz = a->basis_f32 ? sizeof(float) : sizeof(double);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  char* st = take(sizeof(State));
  char* pub = take(sizeof(Pub));
  char* sync = take(64);
  char* ex = take(sizeof(double) * kp::kExSlots * kp::kNmPad * kp::kNmPad);
  char* tx = take(sizeof(double) * kp::kTailPad);
  char* part = take(part_doubles(*a, a->nwg) * sizeof(double));
  char* hx = take(halo_area(*a, a->nwg) * sizeof(double));
  char* flags = take((size_t)a->nwg * kp::kFlagStride * sizeof(unsigned));
  char* u = take((size_t)a->ld * sizeof(double));
  char* V = take((size_t)a->ld * (size_t)(a->m_max + 2) * esz);
  if (base) {
    a->st = reinterpret_cast<State*>(st);
    a->pub = reinterpret_cast<Pub*>(pub);
    a->sync = reinterpret_cast<unsigned*>(sync);
    a->ex = reinterpret_cast<double*>(ex);
    a->tx = reinterpret_cast<double*>(tx);
    a->part = reinterpret_cast<double*>(part);
    a->hx = reinterpret_cast<double*>(hx);
    a->hx2 = a->hx + halo_doubles(*a, a->nwg);
    a->flags = reinterpret_cast<unsigned*>(flags);
    a->u = reinterpret_cast<double*>(u);
    a->V = V;
  }
  return off;
}

// Bytes by which kp_phi_combo_noalloc's capacity is counted: the workspace on
// the partition of at least 4096 elements per workgroup, with three partial
// rows, one halo buffer and 768 bytes for the control block, whatever the
// kernels keep there, so the problems accepted depend on neither.  What the
// finer partition takes beyond that is in the array above KP_NOALLOC_BYTES: two
// halo buffers of at most 32 N bytes (a row per workgroup), or the tagged
// exchange's five of at most 256 workgroups and 256 elements per row (5.3 MB),
// and 1.7 MB of partial sums.
constexpr size_t kCountedPub = 768;
size_t noalloc_need(int ncu_slots, int rows_cfg, const Args& a) {
  Args g = a;
  geometry(ncu_slots, rows_cfg, &g, false);
  const size_t esz = a.basis_f32 ? sizeof(float) : sizeof(double);
  const size_t parts[] = {sizeof(State), kCountedPub, 64,
                          sizeof(double) * kp::kExSlots * kp::kNmPad * kp::kNmPad,
                          sizeof(double) * kp::kTailPad,
                          (size_t)3 * g.nwg * kp::kKStride * sizeof(double),
                          halo_doubles(g, g.nwg) * sizeof(double),
                          (size_t)g.nwg * kp::kFlagStride * sizeof(unsigned),
                          (size_t)g.ld * sizeof(double),
                          (size_t)g.ld * (size_t)(g.m_max + 2) * esz};
  size_t off = 0;
  for (size_t b : parts) off += (b + 255) / 256 * 256;
  return off;
}

int launch(kp_ctx* ctx, Args a, int arnoldi_only) {
  void* args[] = {&a, &arnoldi_only};
  KP_HIP(ctx, hipLaunchCooperativeKernel(run_kernel(a), dim3(a.nwg), dim3(kp::kThreads), args, 0,
                                         ctx->stream));
  return KP_OK;
}

int launch_init(kp_ctx* ctx, const Args& a, int m_target) {
  hipLaunchKernelGGL(kp::k_init, dim3(a.ll ? a.nwg : (a.nwg + 7) / 8), dim3(256), 0, ctx->stream, a, m_target);
  KP_HIP(ctx, hipGetLastError());
  return KP_OK;
}

int fill_info_from(kp_ctx* ctx, const Args& a, kp_info* info) {
  KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  State h;
  KP_HIP(ctx, hipMemcpy(&h, a.st, offsetof(State, sigma), hipMemcpyDeviceToHost));
  Pub pb;
  KP_HIP(ctx, hipMemcpy(&pb, a.pub, sizeof(Pub), hipMemcpyDeviceToHost));
  unsigned flags[16] = {0};
  KP_HIP(ctx, hipMemcpy(flags, a.sync, sizeof(flags), hipMemcpyDeviceToHost));
  std::memset(info, 0, sizeof(*info));
  info->status = flags[kp::kSyncAbort] ? KP_STATUS_ABORTED : pb.status;
  info->substeps = h.substeps;
  info->rejected = h.rejected;
  info->arnoldi_steps = h.arnoldi_steps;
  info->expm_evals = h.expm_evals;
  info->m_last = h.m_last;
  info->n_fallback = h.n_fallback;
  info->breakdowns = h.breakdowns;
  info->schedule_len = std::min(h.nlog, kp::kLogMax);
  info->err_max = h.err_max;
  info->mu = h.mu;
  info->t_end = h.t;
  info->onchip_passes = h.onchip;
  return KP_OK;
}

int fill_info(kp_ctx* ctx, kp_info* info) { return fill_info_from(ctx, ctx->last, info); }

// ---- the allocation-free entry point: the static scratch array --------------

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's scratch array (looked up once per device, with
// that device current), or nullptr with ctx->err set.
void* scratch_address(kp_ctx* ctx) {
  if (ctx->device < 0 || ctx->device >= kMaxDevices) {
    snprintf(ctx->err, sizeof(ctx->err), "device %d beyond the scratch table", ctx->device);
    return nullptr;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[ctx->device]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(kp::scratch));
    if (e != hipSuccess || !ptr) {
      snprintf(ctx->err, sizeof(ctx->err), "hipGetSymbolAddress(scratch): %s",
               hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_ptr[ctx->device] = ptr;
  }
  return g_scratch_ptr[ctx->device];
}

// ---- batched call: plan, workspace, graph -------------------------------------

// Planner inputs of one problem: its size and a Gershgorin-type bound of
// ||A|| (the coefficient fields are not read: a pointwise term of unknown size
// counts as 1 for ADR, 2 for the Allen-Cahn factor 1 - 3u^2, b + 1 + 2a^2 for
// the Brusselator Jacobian).
kp::PlanProblem plan_problem(const kp_op& A, int p, int m_max, double h) {
  const double ix2 = 1.0 / (A.dx * A.dx), iy2 = 1.0 / (A.dy * A.dy);
  const double nu = std::max(std::fabs(A.nu), A.kind == KP_OP_BRUSSELATOR ? std::fabs(A.nu2) : 0.0);
  double rho = 4.0 * nu * (ix2 + iy2);
  if (A.kind == KP_OP_ADR)
    rho += std::fabs(A.ax) / A.dx + std::fabs(A.ay) / A.dy + std::fabs(A.react) + (A.field0 ? 1.0 : 0.0);
  else if (A.kind == KP_OP_ALLEN_CAHN)
    rho += 2.0;
  else
    rho += std::fabs(A.brus_b) + 1.0 + 2.0 * A.brus_a * A.brus_a;
  kp::PlanProblem q;
  q.nx = A.nx;
  q.ny = A.ny;
  q.n = (int64_t)A.nx * A.ny * (A.kind == KP_OP_BRUSSELATOR ? 2 : 1);
  q.p = p;
  q.c = (A.field0 ? 1 : 0) + (A.field1 ? 1 : 0);
  q.m_max = m_max;
  q.h_rho = std::fabs(h) * rho;
  return q;
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Sizes of a problem's own buffers (bytes, each 256-aligned): basis, state
// vector, partial sums, halo rows, small-exponential scratch, tail values.
struct ProbBufs {
  size_t v, u, part, hx, ex, tx;
  size_t total() const { return v + u + part + hx + ex + tx; }
};

}  // namespace

struct BatchCache {
  std::vector<long long> key;
  kp::Plan plan;
  int n_wg = 0;
  int nprob = 0;
  int nclass = 0;
  std::vector<int> class_size;        // team size of class c
  std::vector<int> class_wg0;         // first workgroup of class c's run of teams
  std::vector<size_t> prob_off;       // arena offset of each problem's buffers
  std::vector<ProbBufs> prob_buf;     // their sizes, as the arena was laid out
  std::vector<int> prob_nwg;          // largest row-owning workgroup count over the classes
  std::vector<int> prob_class;        // class the plan gave each problem
  std::vector<int64_t> flag_off;      // per problem, in unsigned
  void* arena = nullptr;              // per-problem buffers
  State* st = nullptr;                // [nprob]
  Pub* pub = nullptr;                 // [nprob]
  unsigned* sync = nullptr;           // [nprob][16]
  unsigned* flags = nullptr;
  Args* d_args = nullptr;             // [nclass][nprob]
  int* d_meta = nullptr;              // order | class_first | team_of_wg | team_class | team_wg0
  unsigned long long* d_q = nullptr;  // class queues, then team slots
  kp_info* d_info = nullptr;          // [nprob]
  std::vector<Args> hargs;
  kp::BatchDesc desc{};
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

void batch_free(BatchCache* b) {
  if (!b) return;
  if (b->exec) hipGraphExecDestroy(b->exec);
  if (b->graph) hipGraphDestroy(b->graph);
  void* bufs[] = {b->arena, b->st, b->pub, b->sync, b->flags, b->d_args, b->d_meta, b->d_q,
                  b->d_info};
  for (void* x : bufs)
    if (x) hipFree(x);
  delete b;
}

// The kernel of a batched call's problems (they share the configuration).
// The forms without block steps take k_run's phases, unless every problem has
// two planes: single steps in the block kernel, with two columns per chunk and
// the registers of six vectors, cost 5 % on 256 problems of sides 16 to 64
// (H-CWY: 4.46 ms, 4.23 in k_run's phases), 7 % on six of sides 300 to 700
// (7.37, 6.88), 0.4 to 0.8 % on sides up to 256 and 512, and gain 1 % on 128
// Brusselators of sides 32 to 256 (38.8, 39.2).
void choose_batch_kernel(std::vector<Args>& as) {
  bool two = true;
  for (const Args& a : as) two = two && a.nplanes == 2;
  if (!two && !as[0].pairs)
    for (Args& a : as) a.block = 0;
}
const void* batch_kernel(const Args& a) {
  if (a.block) return reinterpret_cast<const void*>(&kp::k_batch<double, false, true>);
  if (kp::orth_multi_sync(a.orth))
    return a.basis_f32 ? reinterpret_cast<const void*>(&kp::k_batch<float, true>)
                       : reinterpret_cast<const void*>(&kp::k_batch<double, true>);
  return a.basis_f32 ? reinterpret_cast<const void*>(&kp::k_batch<float, false>)
                     : reinterpret_cast<const void*>(&kp::k_batch<double, false>);
}

// Geometry of a problem on the teams of one class (team size g, first
// workgroup of the class's run of teams wg0).
void batch_geometry(int g, int wg0, Args* a) {
  int rows, nw;
  kp::plan_rows(a->nx, a->ny, g, &rows, &nw);
  a->rows_per_wg = rows;
  a->nwg = nw;
  a->nteam = g;
  a->wg0 = wg0;
}

ProbBufs prob_bufs(const Args& a, int nwg_max) {
  const size_t esz = a.basis_f32 ? sizeof(float) : sizeof(double);
  ProbBufs r;
  r.v = align256((size_t)a.ld * (a.m_max + 2) * esz);
  r.u = align256((size_t)a.ld * sizeof(double));
  r.part = align256(part_doubles(a, nwg_max) * sizeof(double));
  r.hx = align256(halo_area(a, nwg_max) * sizeof(double));
  r.ex = align256(sizeof(double) * kp::kExSlots * kp::kNmPad * kp::kNmPad);
  r.tx = align256(sizeof(double) * kp::kTailPad);
  return r;
}

// New plan, allocations and graph for the problem set of `as` (validated).
// (forced: this plan instead of the planner's).
int batch_create(kp_ctx* ctx, const std::vector<Args>& as, const std::vector<kp::PlanProblem>& qs,
                 std::vector<long long>&& key, BatchCache** out, const kp::Plan* forced = nullptr) {
  BatchCache* b = new BatchCache();
  b->key = std::move(key);
  const int np = (int)as.size();
  b->nprob = np;
  const void* kernel = batch_kernel(as[0]);
  int occ = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, kp::kThreads, 0);
  if (e != hipSuccess || occ < 1) {
    batch_free(b);
    if (e != hipSuccess) return hip_fail(ctx, e, "batched occupancy");
    snprintf(ctx->err, sizeof(ctx->err), "the batched kernel does not fit on a CU");
    return KP_EHIP;
  }
  b->n_wg = ctx->ncu * occ;
  const kp::PlanModel model = ctx->model;
  b->plan = forced ? *forced : kp::make_plan(qs, b->n_wg, model);
  const kp::Plan& pl = b->plan;
  const int nt = (int)pl.team_size.size();
  // classes: the runs of equal-size teams (the plan lays them out big, mid,
  // single), each with the problems the plan gave its teams, heaviest first
  std::vector<int> team_class(nt);
  for (int t = 0; t < nt; ++t) {
    if (t == 0 || pl.team_size[t] != pl.team_size[t - 1]) {
      b->class_size.push_back(pl.team_size[t]);
      b->class_wg0.push_back(pl.team_wg0[t]);
    }
    team_class[t] = (int)b->class_size.size() - 1;
  }
  const int nc = (int)b->class_size.size();
  b->nclass = nc;
  std::vector<std::vector<int>> lists(nc);
  for (int t = 0; t < nt; ++t)
    for (int q = pl.team_first[t]; q < pl.team_first[t + 1]; ++q)
      lists[team_class[t]].push_back(pl.order[q]);
  std::vector<int> order, class_first(1, 0);
  for (int c = 0; c < nc; ++c) {
    const int g = b->class_size[c];
    std::stable_sort(lists[c].begin(), lists[c].end(), [&](int x, int y) {
      return kp::plan_time(qs[x], g, model) > kp::plan_time(qs[y], g, model);
    });
    order.insert(order.end(), lists[c].begin(), lists[c].end());
    class_first.push_back((int)order.size());
  }
  b->prob_class.assign(np, 0);
  for (int c = 0; c < nc; ++c)
    for (int i : lists[c]) b->prob_class[i] = c;
  // per-problem buffers, sized for the class that spreads the problem widest
  b->prob_nwg.assign(np, 1);
  for (int i = 0; i < np; ++i)
    for (int c = 0; c < nc; ++c) {
      Args g = as[i];
      batch_geometry(b->class_size[c], b->class_wg0[c], &g);
      b->prob_nwg[i] = std::max(b->prob_nwg[i], g.nwg);
    }
  size_t off = 0;
  b->prob_off.assign(np, 0);
  b->flag_off.assign(np, 0);
  int64_t nflags = 0;
  for (int i = 0; i < np; ++i) {
    b->prob_off[i] = off;
    b->prob_buf.push_back(prob_bufs(as[i], b->prob_nwg[i]));
    off += b->prob_buf[i].total();
    b->flag_off[i] = nflags;
    nflags += (int64_t)b->prob_nwg[i] * kp::kFlagStride;
  }
  e = hipMalloc(&b->arena, std::max<size_t>(off, 256));
  if (e == hipSuccess) e = hipMalloc(&b->st, sizeof(State) * np);
  if (e == hipSuccess) e = hipMalloc(&b->pub, sizeof(Pub) * np);
  if (e == hipSuccess) e = hipMalloc(&b->sync, 64 * (size_t)np);
  if (e == hipSuccess) e = hipMalloc(&b->flags, sizeof(unsigned) * (size_t)std::max<int64_t>(nflags, 1));
  if (e == hipSuccess) e = hipMalloc(&b->d_args, sizeof(Args) * (size_t)nc * np);
  const size_t nmeta = (size_t)np + (nc + 1) + b->n_wg + 2 * (size_t)nt;
  if (e == hipSuccess) e = hipMalloc(&b->d_meta, sizeof(int) * nmeta);
  if (e == hipSuccess) e = hipMalloc(&b->d_q, sizeof(unsigned long long) * (nc + 8 * (size_t)nt));
  if (e == hipSuccess) e = hipMalloc(&b->d_info, sizeof(kp_info) * np);
  if (e != hipSuccess) {
    snprintf(ctx->err, sizeof(ctx->err), "batched workspace: %s", hipGetErrorString(e));
    batch_free(b);
    return KP_ENOMEM;
  }
  // every team takes part, also one the plan left without problems: it
  // takes problems from the other classes' queues
  std::vector<int> team_of_wg(b->n_wg, -1);
  for (int t = 0; t < nt; ++t)
    for (int w = 0; w < pl.team_size[t]; ++w) team_of_wg[pl.team_wg0[t] + w] = t;
  std::vector<int> meta;
  meta.reserve(nmeta);
  meta.insert(meta.end(), order.begin(), order.end());
  meta.insert(meta.end(), class_first.begin(), class_first.end());
  meta.insert(meta.end(), team_of_wg.begin(), team_of_wg.end());
  meta.insert(meta.end(), team_class.begin(), team_class.end());
  meta.insert(meta.end(), pl.team_wg0.begin(), pl.team_wg0.end());
  e = hipMemcpy(b->d_meta, meta.data(), sizeof(int) * nmeta, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    batch_free(b);
    return hip_fail(ctx, e, "hipMemcpy(plan)");
  }
  b->desc.args = (const kp::CArgs*)(b->d_args);
  b->desc.order = b->d_meta;
  b->desc.class_first = b->d_meta + np;
  b->desc.team_of_wg = b->d_meta + np + (nc + 1);
  b->desc.team_class = b->d_meta + np + (nc + 1) + b->n_wg;
  b->desc.team_wg0 = b->d_meta + np + (nc + 1) + b->n_wg + nt;
  b->desc.queue = b->d_q;
  b->desc.slot = b->d_q + nc;
  b->desc.nprob = np;
  b->desc.nclass = nc;
  b->desc.nteams = nt;
  b->desc.wait_ticks = ctx->wait_ticks;
  // the graph: reset of every problem, the queues and the team slots -> the
  // persistent batched kernel (cooperative) -> the per-problem outcome records
  hipGraphNode_t n1, n2, n3;
  void* a1[] = {&b->desc};
  void* a2[] = {&b->desc};
  void* a3[] = {&b->desc, &b->d_info};
  hipKernelNodeParams p1{}, p2{}, p3{};
  p1.func = reinterpret_cast<void*>(&kp::k_batch_init);
  p1.gridDim = dim3(np);
  p1.blockDim = dim3(256);
  p1.kernelParams = a1;
  p2.func = const_cast<void*>(kernel);
  p2.gridDim = dim3(b->n_wg);
  p2.blockDim = dim3(kp::kThreads);
  p2.kernelParams = a2;
  p3.func = reinterpret_cast<void*>(&kp::k_batch_info);
  p3.gridDim = dim3((np + 63) / 64);
  p3.blockDim = dim3(64);
  p3.kernelParams = a3;
  hipLaunchAttributeValue coop{};
  coop.cooperative = 1;
  e = hipGraphCreate(&b->graph, 0);
  if (e == hipSuccess) e = hipGraphAddKernelNode(&n1, b->graph, nullptr, 0, &p1);
  if (e == hipSuccess) e = hipGraphAddKernelNode(&n2, b->graph, &n1, 1, &p2);
  if (e == hipSuccess) e = hipGraphKernelNodeSetAttribute(n2, hipKernelNodeAttributeCooperative, &coop);
  if (e == hipSuccess) e = hipGraphAddKernelNode(&n3, b->graph, &n2, 1, &p3);
  if (e == hipSuccess) e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    batch_free(b);
    return hip_fail(ctx, e, "batched graph");
  }
  *out = b;
  return KP_OK;
}

// Per-call Args of every (class, problem): the caller's pointers and
// coefficients, the class's team geometry and the problem's own buffers.
void batch_fill_args(BatchCache* b, const std::vector<Args>& as, int64_t wait_ticks) {
  const int np = b->nprob;
  b->hargs.resize((size_t)b->nclass * np);
  for (int i = 0; i < np; ++i) {
    Args a = as[i];
    const ProbBufs& z = b->prob_buf[i];
    char* base = static_cast<char*>(b->arena) + b->prob_off[i];
    a.V = base;
    a.u = reinterpret_cast<double*>(base + z.v);
    a.part = reinterpret_cast<double*>(base + z.v + z.u);
    a.hx = reinterpret_cast<double*>(base + z.v + z.u + z.part);
    a.hx2 = a.hx + halo_doubles(a, b->prob_nwg[i]);
    a.ex = reinterpret_cast<double*>(base + z.v + z.u + z.part + z.hx);
    a.tx = reinterpret_cast<double*>(base + z.v + z.u + z.part + z.hx + z.ex);
    a.st = b->st + i;
    a.pub = b->pub + i;
    a.sync = b->sync + 16 * (size_t)i;
    a.flags = b->flags + b->flag_off[i];
    a.wait_ticks = wait_ticks;
    a.part_rows = b->prob_nwg[i];
    // a team of a larger class that takes the problem (from the light end of
    // its planned class's queue) keeps the planned row partition, its extra
    // workgroups only meeting the barriers: the partial sums, and so the
    // result, do not depend on which team solves the problem
    const int pc = b->prob_class[i];
    Args planned = a;
    batch_geometry(b->class_size[pc], b->class_wg0[pc], &planned);
    for (int c = 0; c < b->nclass; ++c) {
      Args& r = b->hargs[(size_t)c * np + i];
      r = a;
      batch_geometry(b->class_size[c], b->class_wg0[c], &r);
      if (b->class_size[c] > b->class_size[pc]) {
        r.rows_per_wg = planned.rows_per_wg;
        r.nwg = planned.nwg;
      }
    }
  }
}

}  // namespace

extern "C" {

int kp_version(void) { return 10300; }

int kp_read_bandwidth(kp_ctx* ctx, int64_t bytes, int32_t reps, double* gbps_host) {
  if (!ctx || !gbps_host || reps < 1 || reps > 1000 || bytes < (int64_t)1 << 20 ||
      bytes > (int64_t)1 << 36)
    return KP_EINVAL;
  int rc = device_setup(ctx);
  if (rc) return rc;
  const int64_t n2 = bytes / 16;
  const int nblk = ctx->ncu;                       // the persistent kernels' launch shape
  double2* x = nullptr;
  double* sink = nullptr;
  if (hipMalloc(&x, (size_t)n2 * 16) != hipSuccess) return KP_ENOMEM;
  if (hipMalloc(&sink, sizeof(double) * (size_t)nblk * (kp::kThreads / 64)) != hipSuccess) {
    hipFree(x);
    return KP_ENOMEM;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  std::vector<float> ms;
  rc = KP_OK;
  hipLaunchKernelGGL(kp::k_zero, dim3(4096), dim3(256), 0, ctx->stream, (double*)x, 2 * n2);
  if (hipGetLastError() != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
      hipEventCreate(&e1) != hipSuccess)
    rc = KP_EHIP;
  for (int r = 0; r <= reps && rc == KP_OK; ++r) {  // the first launch warms up
    if (hipEventRecord(e0, ctx->stream) != hipSuccess) { rc = KP_EHIP; break; }
    hipLaunchKernelGGL(kp::k_read_probe, dim3(nblk), dim3(kp::kThreads), 0, ctx->stream,
                       (const double2*)x, n2, sink);
    float t = 0.f;
    if (hipGetLastError() != hipSuccess || hipEventRecord(e1, ctx->stream) != hipSuccess ||
        hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&t, e0, e1) != hipSuccess) {
      rc = KP_EHIP;
      break;
    }
    if (r) ms.push_back(t);
  }
  if (e0) hipEventDestroy(e0);
  if (e1) hipEventDestroy(e1);
  hipFree(sink);
  hipFree(x);
  if (rc) {
    snprintf(ctx->err, sizeof(ctx->err), "kp_read_bandwidth: HIP error");
    return rc;
  }
  std::sort(ms.begin(), ms.end());
  *gbps_host = (double)n2 * 16.0 / (1e-3 * ms[ms.size() / 2]) * 1e-9;
  return KP_OK;
}

int kp_set_timeline(kp_ctx* ctx, long long* ts, int32_t kmax) {
  if (!ctx || kmax < 0 || (kmax > 0 && !ts)) return KP_EINVAL;
#ifdef KP_TIMELINE
  ctx->ts = kmax > 0 ? ts : nullptr;
  ctx->ts_kmax = kmax;
  return KP_OK;
#else
  return KP_EUNSUPPORTED;
#endif
}

int kp_timeline_layout(int32_t* slots_host, int32_t* workgroups_host) {
  if (!slots_host || !workgroups_host) return KP_EINVAL;
  *slots_host = kp::kTsSlots;
  *workgroups_host = kp::kTsWgs;
#ifdef KP_TIMELINE
  return 1;
#else
  return 0;
#endif
}

int kp_runtime_version(int32_t* runtime_host, int32_t* driver_host) {
  int rv = 0, dv = 0;
  if (hipRuntimeGetVersion(&rv) != hipSuccess) return KP_EHIP;
  if (hipDriverGetVersion(&dv) != hipSuccess) return KP_EHIP;
  if (runtime_host) *runtime_host = rv;
  if (driver_host) *driver_host = dv;
  return KP_OK;
}

const char* kp_strerror(int code) {
  switch (code) {
    case KP_OK: return "ok";
    case KP_EINVAL: return "invalid argument";
    case KP_ENOMEM: return "device allocation failed";
    case KP_EHIP: return "HIP runtime error";
    case KP_EUNSUPPORTED: return "unsupported combination of options";
    case KP_ESTATE: return "call out of order";
    case KP_ETOOLARGE: return "problem exceeds a fixed capacity";
    default: return "unknown error";
  }
}

const char* kp_last_error(kp_ctx* ctx) { return ctx ? ctx->err : ""; }

int kp_create(kp_ctx** out, const kp_config* cfg) {
  if (!out) return KP_EINVAL;
  kp_config c{};
  if (cfg) c = *cfg;
  int rc = check_config(&c);
  if (rc) return rc;
  kp_ctx* ctx = new (std::nothrow) kp_ctx();
  if (!ctx) return KP_ENOMEM;
  ctx->cfg = c;
  ctx->stream = static_cast<hipStream_t>(c.stream);
  *out = ctx;
  return KP_OK;
}

int kp_set_config(kp_ctx* ctx, const kp_config* cfg) {
  if (!ctx || !cfg) return KP_EINVAL;
  int rc = check_config(cfg);
  if (rc) return rc;
  ctx->cfg = *cfg;
  ctx->stream = static_cast<hipStream_t>(cfg->stream);
  ctx->have_begin = 0;
  return KP_OK;
}

int kp_destroy(kp_ctx* ctx) {
  if (!ctx) return KP_EINVAL;
  if (ctx->ncu > 0) hipStreamSynchronize(ctx->stream);
  batch_free(ctx->batch);
  void* bufs[] = {ctx->V,  ctx->u,    ctx->part, ctx->hx, ctx->flags, ctx->st,
                  ctx->pub, ctx->sync, ctx->ex, ctx->tx, ctx->aux, ctx->integ};
  for (void* b : bufs)
    if (b) hipFree(b);
  delete ctx;
  return KP_OK;
}

int kp_phi_combo(kp_ctx* ctx, const kp_op* A, const double* B, int32_t p, int64_t ldb,
                 double h, double tol, int32_t m_max, double* out, kp_info* info) {
  Args a;
  int rc = build_args(ctx, A, B, p, ldb, h, tol, m_max, out, true, &a);
  if (rc) return rc;
  if ((rc = prepare(ctx, &a))) return rc;
  const int m0 = a.m0;
  if ((rc = launch_init(ctx, a, m0))) return rc;
  if ((rc = launch(ctx, a, 0))) return rc;
  ctx->last = a;
  ctx->st_last = a.st;
  ctx->have_begin = 0;
  if (info) return fill_info(ctx, info);
  return KP_OK;
}

int kp_phi_combo_noalloc(kp_ctx* ctx, const kp_op* A, const double* B, int32_t p, int64_t ldb,
                         double h, double tol, int32_t m_max, double* out, kp_info* info) {
  Args a;
  int rc = build_args(ctx, A, B, p, ldb, h, tol, m_max, out, true, &a);
  if (rc) return rc;
  if ((rc = device_setup(ctx))) return rc;
  int cur = -1;
  KP_HIP(ctx, hipGetDevice(&cur));
  if (cur != ctx->device) {
    snprintf(ctx->err, sizeof(ctx->err), "context bound to device %d, device %d is current",
             ctx->device, cur);
    return KP_EINVAL;
  }
  choose_kernel(&a);
  const int occ = kernel_occupancy(ctx, a);
  if (occ <= 0) {
    snprintf(ctx->err, sizeof(ctx->err), "the persistent kernel does not fit on a CU");
    return KP_EHIP;
  }
  geometry(ctx->ncu * occ, ctx->cfg.rows_per_wg, &a);
  const size_t need = noalloc_need(ctx->ncu * occ, ctx->cfg.rows_per_wg, a);
  if (need > (size_t)KP_NOALLOC_BYTES || carve(&a, nullptr) > kp::kScratchBytes) {
    snprintf(ctx->err, sizeof(ctx->err),
             "workspace of %zu bytes exceeds the static scratch of %zu bytes", need,
             (size_t)KP_NOALLOC_BYTES);
    return KP_ETOOLARGE;
  }
  char* base = static_cast<char*>(scratch_address(ctx));
  if (!base) return KP_EHIP;
  carve(&a, base);
  a.wait_ticks = ctx->wait_ticks;
  if ((rc = launch_init(ctx, a, a.m0))) return rc;
  if ((rc = launch(ctx, a, 0))) return rc;
  ctx->last = a;
  ctx->st_last = a.st;
  ctx->have_begin = 0;
  if (info) return fill_info(ctx, info);
  return KP_OK;
}

int kp_phi_combo_tangent(kp_ctx* ctx, const kp_op* A, const kp_op* dA, const double* B,
                         int32_t p, int64_t ldb, double h, double tol, int32_t m_max,
                         double* out, double* dout, kp_info* info) {
  if (!ctx || !A || !dA || !dout) return KP_EINVAL;
  if (A->kind != KP_OP_ADR && A->kind != KP_OP_ALLEN_CAHN) return KP_EUNSUPPORTED;
  if (dA->kind != A->kind || dA->nx != A->nx || dA->ny != A->ny || dA->dx != A->dx ||
      dA->dy != A->dy || (dA->transpose != 0) != (A->transpose != 0))
    return KP_EINVAL;
  if (dA->field0 || dA->field1) return KP_EUNSUPPORTED;
  const double dc[] = {dA->nu, dA->ax, dA->ay, dA->react};
  for (double v : dc)
    if (!std::isfinite(v)) return KP_EINVAL;
  if (p < 0 || 2 * p > KP_PMAX) return KP_EUNSUPPORTED;
  Args a;
  int rc = build_args(ctx, A, B, p, ldb, h, tol, m_max, out, true, &a);
  if (rc) return rc;
  const size_t ob = (size_t)a.N * sizeof(double);
  if (overlaps(dout, ob, out, ob) || overlaps(dout, ob, B, (size_t)ldb * (p + 1) * sizeof(double)) ||
      overlaps(dout, ob, A->field0, ob))
    return KP_EINVAL;
  // the pair [a; c] of augmented vectors: two planes, tail of 2p entries
  a.tangent = 1;
  a.dout = dout;
  a.nplanes = 2;
  a.pb = p;
  a.p = 2 * p;
  a.tail_off = a.npt_pad * 2;
  a.ld = a.tail_off + kp::kTailPad;
  a.halo_lds = (2 * 2 * (int64_t)A->nx <= kp::kHaloCap) ? 1 : 0;
  a.dcx = dA->nu / (A->dx * A->dx);
  a.dcy = dA->nu / (A->dy * A->dy);
  a.dadx = dA->ax / (2.0 * A->dx);
  a.dady = dA->ay / (2.0 * A->dy);
  a.dreact = dA->react;
  if ((rc = prepare(ctx, &a))) return rc;
  const int m0 = a.m0;
  if ((rc = launch_init(ctx, a, m0))) return rc;
  if ((rc = launch(ctx, a, 0))) return rc;
  ctx->last = a;
  ctx->st_last = a.st;
  ctx->have_begin = 0;
  if (info) return fill_info(ctx, info);
  return KP_OK;
}

int kp_phi_combo_backward(kp_ctx* ctx, const kp_op* A, const double* B, int32_t p,
                          int64_t ldb, double h, double tol, int32_t m_max, const double* g,
                          double* grad_B, int64_t ldgb, int32_t coef_mask, double* grad_coef,
                          kp_info* info) {
  if (!ctx || !A || !B || !g) return KP_EINVAL;
  if (coef_mask < 0 || coef_mask > 15 || (coef_mask && !grad_coef)) return KP_EINVAL;
  if (!grad_B && !coef_mask) return KP_EINVAL;
  Args a;
  int rc = build_args(ctx, A, B, p, ldb, h, tol, m_max, nullptr, false, &a);
  if (rc) return rc;
  const int64_t N = a.N;
  if (grad_B && ldgb < N) return KP_EINVAL;
  if (coef_mask && ((A->kind != KP_OP_ADR && A->kind != KP_OP_ALLEN_CAHN) ||
                    (A->kind == KP_OP_ADR && !A->field0 ? p + 1 : 2 * p) > KP_PMAX))
    return KP_EUNSUPPORTED;   // refused before any work is enqueued
  if ((rc = device_setup(ctx))) return rc;
  // Coefficient directions commute with a constant-coefficient ADR operator
  // (all are circulant): the derivative is then one plain solve with the
  // p + 2 right-hand sides of k_dir_rhs; otherwise a tangent solve.
  const bool commuting = A->kind == KP_OP_ADR && !A->field0;
  // aux: W = [0_1 .. 0_p | g] (N x (p+1)), then y, dy (N each), dot partials,
  // then C (N x (p+2)) for the commuting directions
  const size_t need =
      sizeof(double) * ((size_t)(p + 3) * N + kp::kDotBlocks + (commuting ? (size_t)(p + 2) * N : 0));
  if ((rc = grow(ctx, reinterpret_cast<void**>(&ctx->aux), &ctx->aux_bytes, need))) return rc;
  double* W = ctx->aux;
  double* y = W + (size_t)(p + 1) * N;
  double* dy = y + N;
  double* part = dy + N;
  double* C = part + kp::kDotBlocks;
  if (grad_B && (overlaps(grad_B, (size_t)ldgb * (p + 1) * sizeof(double), g, N * sizeof(double)) ||
                 overlaps(grad_B, (size_t)ldgb * (p + 1) * sizeof(double), B,
                          (size_t)ldb * (p + 1) * sizeof(double))))
    return KP_EINVAL;
  int worst = KP_STATUS_OK;
  auto track = [&](const kp_info* r) {   // worst status, summed work
    if (r->status > worst) worst = r->status;
    info->substeps += r->substeps;
    info->rejected += r->rejected;
    info->arnoldi_steps += r->arnoldi_steps;
    info->expm_evals += r->expm_evals;
    info->n_fallback += r->n_fallback;
    info->breakdowns += r->breakdowns;
    info->err_max = std::max(info->err_max, r->err_max);
    info->t_end = r->t_end;
  };
  kp_info tmp;
  kp_info* ip = info ? &tmp : nullptr;
  if (info) std::memset(info, 0, sizeof(*info));
  if (grad_B) {
    // dL/db_k = h^k phi_k(h A^T) g: the phi combination of A^T with
    // B_k = [0, ..., 0, g] (k zero columns), a view of W from column p - k
    kp_op At = *A;
    At.transpose = A->transpose ? 0 : 1;
    if (p > 0) {
      const int64_t nz = (int64_t)p * N;
      hipLaunchKernelGGL(kp::k_zero, dim3((unsigned)std::min<int64_t>((nz + 255) / 256, 4096)),
                         dim3(256), 0, ctx->stream, W, nz);
      KP_HIP(ctx, hipGetLastError());
    }
    KP_HIP(ctx, hipMemcpyAsync(W + (size_t)p * N, g, sizeof(double) * N, hipMemcpyDeviceToDevice,
                               ctx->stream));
    for (int k = 0; k <= p; ++k) {
      if ((rc = kp_phi_combo(ctx, &At, W + (size_t)(p - k) * N, k, N, h, tol, m_max,
                             grad_B + (size_t)k * ldgb, ip)))
        return rc;
      if (info) track(ip);
    }
  }
  // dL/dtheta = <g, dy/dtheta>: one tangent solve per requested coefficient
  for (int c = 0; c < 4; ++c) {
    if (!(coef_mask & (1 << c))) continue;
    kp_op dA = *A;
    dA.field0 = dA.field1 = nullptr;
    dA.nu = c == 0 ? 1.0 : 0.0;
    dA.ax = c == 1 ? 1.0 : 0.0;
    dA.ay = c == 2 ? 1.0 : 0.0;
    dA.react = c == 3 ? 1.0 : 0.0;
    if (commuting) {
      const int64_t tot = N * (p + 2);
      hipLaunchKernelGGL(kp::k_dir_rhs, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0,
                         ctx->stream, B, ldb, p, A->nx, A->ny, dA.nu / (A->dx * A->dx),
                         dA.nu / (A->dy * A->dy), dA.ax / (2.0 * A->dx), dA.ay / (2.0 * A->dy),
                         dA.react, A->transpose ? 1 : 0, h, C);
      KP_HIP(ctx, hipGetLastError());
      if ((rc = kp_phi_combo(ctx, A, C, p + 1, N, h, tol, m_max, dy, ip))) return rc;
    } else if ((rc = kp_phi_combo_tangent(ctx, A, &dA, B, p, ldb, h, tol, m_max, y, dy, ip))) {
      return rc;
    }
    if (info) track(ip);
    hipLaunchKernelGGL(kp::k_dot_partial, dim3(kp::kDotBlocks), dim3(256), 0, ctx->stream, g, dy,
                       N, part);
    hipLaunchKernelGGL(kp::k_dot_final, dim3(1), dim3(256), 0, ctx->stream, part, grad_coef + c);
    KP_HIP(ctx, hipGetLastError());
  }
  if (info) {
    KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
    info->status = worst;
  }
  return KP_OK;
}

// ---- exponential integrators ---------------------------------------------------

namespace {

// Coefficient matrices alpha_{m,i} of Section 4.1 (rows m = 1..M, columns
// i = 1..P; the first row is zero).
const double kEpi4[3][2] = {{0.0, 0.0}, {-3.0 / 10.0, 3.0 / 40.0}, {32.0 / 5.0, -11.0 / 10.0}};
const double kEpi5[4][3] = {{0.0, 0.0, 0.0},
                            {-4.0 / 5.0, 2.0 / 5.0, -4.0 / 45.0},
                            {12.0, -9.0 / 2.0, 8.0 / 9.0},
                            {3.0, 0.0, -1.0 / 3.0}};

struct Integ {
  kp_ctx* ctx;
  kp::RhsK rk;
  kp_rhs rhs;
  int64_t n;
  double tol;
  int m_max;
  kp_info* info;
  int worst = KP_STATUS_OK;
  double *fn, *jd, *B, *y, *z, *fz;

  unsigned grid() const { return (unsigned)((n + 255) / 256); }

  // the Jacobian of f at un (its ADR field is jd, computed with f(un))
  kp_op jac(const double* un) const {
    kp_op J{};
    J.nx = rhs.nx;
    J.ny = rhs.ny;
    J.dx = rhs.dx;
    J.dy = rhs.dy;
    J.nu = rhs.nu;
    J.brus_a = 1.0;
    J.brus_b = 3.0;
    if (rhs.kind == KP_RHS_ALLEN_CAHN) {
      J.kind = KP_OP_ALLEN_CAHN;
      J.field0 = un;
    } else {
      J.kind = KP_OP_ADR;
      J.ax = rhs.ax;
      J.ay = rhs.ay;
      J.field0 = jd;
    }
    return J;
  }

  int phi(const kp_op& J, int p, double h) {
    kp_info r;
    const int rc = kp_phi_combo(ctx, &J, B, p, n, h, tol, m_max, y, info ? &r : nullptr);
    if (rc || !info) return rc;
    worst = std::max(worst, (int)r.status);
    info->substeps += r.substeps;
    info->rejected += r.rejected;
    info->arnoldi_steps += r.arnoldi_steps;
    info->expm_evals += r.expm_evals;
    info->n_fallback += r.n_fallback;
    info->breakdowns += r.breakdowns;
    info->m_last = r.m_last;
    info->err_max = std::max(info->err_max, r.err_max);
    return KP_OK;
  }

  int launched() {
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? KP_OK : hip_fail(ctx, e, "integrator kernel");
  }

  // f(u) into f (and the ADR Jacobian field into jd when want_jd)
  int rhs_at(const double* u, double* f, bool want_jd, double* Bcols) {
    hipLaunchKernelGGL(kp::k_rhs, dim3(grid()), dim3(256), 0, ctx->stream, rk, u, f,
                       want_jd ? jd : nullptr, Bcols, (int64_t)n);
    return launched();
  }

  int axpy(double* out, const double* a) {
    hipLaunchKernelGGL(kp::k_axpy, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)),
                       dim3(256), 0, ctx->stream, out, a, (const double*)y, (int64_t)n);
    return launched();
  }

  // one SRERK3 step of size h from u_in to u_out (u_out may equal u_in)
  int srerk3(const double* u_in, double* u_out, double h) {
    int rc;
    if ((rc = rhs_at(u_in, fn, true, B))) return rc;      // B = [0, f_n]
    const kp_op J = jac(u_in);
    if ((rc = phi(J, 1, 0.75 * h))) return rc;
    if ((rc = axpy(z, u_in))) return rc;                  // z = u_n + y
    if ((rc = rhs_at(z, fz, false, nullptr))) return rc;
    hipLaunchKernelGGL(kp::k_srerk_cols, dim3(grid()), dim3(256), 0, ctx->stream, rk, u_in,
                       (const double*)fn, (const double*)z, (const double*)fz,
                       (32.0 / 9.0) / (h * h), B, (int64_t)n);
    if ((rc = launched())) return rc;
    if ((rc = phi(J, 3, h))) return rc;
    return axpy(u_out, u_in);
  }
};

}  // namespace

int kp_integrate(kp_ctx* ctx, const kp_rhs* f, int32_t method, double dt, int32_t nsteps,
                 int32_t start_substeps, double* u, double tol, int32_t m_max, kp_info* info) {
  if (!ctx || !f || !u) return KP_EINVAL;
  if (f->kind != KP_RHS_ALLEN_CAHN && f->kind != KP_RHS_ADR) return KP_EINVAL;
  if (f->nx < 1 || f->ny < 1 || (int64_t)f->nx * f->ny > ((int64_t)1 << 30)) return KP_EINVAL;
  const double vals[] = {f->dx, f->dy, f->nu, f->ax, f->ay, f->gamma, dt};
  for (double v : vals)
    if (!std::isfinite(v)) return KP_EINVAL;
  if (!(f->dx > 0.0) || !(f->dy > 0.0) || !(dt > 0.0) || nsteps < 0) return KP_EINVAL;
  if (method != KP_EPI4 && method != KP_EPI5 && method != KP_SRERK3) return KP_EINVAL;
  if (method != KP_SRERK3 && start_substeps < 1) return KP_EINVAL;
  if (m_max < 1 || m_max > KP_MMAX) return KP_EINVAL;
  if (ctx->cfg.fixed_m == 0 && !(tol > 0.0 && std::isfinite(tol))) return KP_EINVAL;
  int rc = device_setup(ctx);
  if (rc) return rc;
  const int P = method == KP_EPI4 ? 2 : (method == KP_EPI5 ? 3 : 0);
  const int M = method == KP_EPI4 ? 3 : 4;      // SRERK3 uses p = 3
  const int64_t n = (int64_t)f->nx * f->ny;
  // workspace: states u_{n-k} and f(u_{n-k}) (k <= P), B (M + 1 columns),
  // y, z, f(z), the ADR Jacobian field
  const size_t need = sizeof(double) * (size_t)n * (2 * (P + 1) + (M + 1) + 4);
  if ((rc = grow(ctx, reinterpret_cast<void**>(&ctx->integ), &ctx->integ_bytes, need))) return rc;
  double* ws = ctx->integ;
  double* ru = ws;                                   // ring of states, P + 1 slots
  double* rf = ru + (size_t)(P + 1) * n;             // ring of f values
  Integ g;
  g.ctx = ctx;
  g.rhs = *f;
  g.rk.kind = f->kind;
  g.rk.nx = f->nx;
  g.rk.ny = f->ny;
  g.rk.cx = f->nu / (f->dx * f->dx);
  g.rk.cy = f->nu / (f->dy * f->dy);
  g.rk.adx = f->ax / (2.0 * f->dx);
  g.rk.ady = f->ay / (2.0 * f->dy);
  g.rk.gamma = f->gamma;
  g.n = n;
  g.tol = tol;
  g.m_max = m_max;
  g.info = info;
  g.B = rf + (size_t)(P + 1) * n;
  g.y = g.B + (size_t)(M + 1) * n;
  g.z = g.y + n;
  g.fz = g.z + n;
  g.jd = g.fz + n;
  g.fn = rf;                                         // SRERK3: f_n in ring slot 0
  if (info) std::memset(info, 0, sizeof(*info));
  if (method == KP_SRERK3) {
    for (int s = 0; s < nsteps; ++s)
      if ((rc = g.srerk3(u, u, dt))) return rc;
  } else {
    // slot (cur - k) mod (P + 1) holds u_{n-k}
    KP_HIP(ctx, hipMemcpyAsync(ru, u, sizeof(double) * n, hipMemcpyDeviceToDevice, ctx->stream));
    int cur = 0;
    auto slot_u = [&](int k) { return ru + (size_t)((cur - k + (P + 1)) % (P + 1)) * n; };
    auto slot_f = [&](int k) { return rf + (size_t)((cur - k + (P + 1)) % (P + 1)) * n; };
    // the first P states by SRERK3 substeps (the f ring, filled after, is
    // their scratch meanwhile: g.fn is its slot 0)
    const int nstart = std::min(P, (int)nsteps);
    for (int k = 0; k < nstart; ++k) {
      double* nxt = ru + (size_t)((cur + 1) % (P + 1)) * n;
      KP_HIP(ctx, hipMemcpyAsync(nxt, slot_u(0), sizeof(double) * n, hipMemcpyDeviceToDevice,
                                 ctx->stream));
      for (int s = 0; s < start_substeps; ++s)
        if ((rc = g.srerk3(nxt, nxt, dt / start_substeps))) return rc;
      cur = (cur + 1) % (P + 1);
    }
    const double* Ep = method == KP_EPI4 ? &kEpi4[0][0] : &kEpi5[0][0];
    kp::EpiK q{};
    q.M = M;
    q.P = P;
    for (int m = 0; m < M; ++m) {
      for (int i = 0; i < P; ++i) q.alpha[m][i] = Ep[m * P + i];
      q.hinv[m] = 1.0 / std::pow(dt, (double)m);
    }
    if (nsteps > nstart) {
      // f of the states in the ring (and, for the newest, the Jacobian field)
      for (int k = nstart; k >= 0; --k)
        if ((rc = g.rhs_at(slot_u(k), slot_f(k), k == 0, nullptr))) return rc;
    }
    for (int s = nstart; s < nsteps; ++s) {
      for (int k = 0; k <= P; ++k) {
        q.u[k] = slot_u(k);
        q.f[k] = slot_f(k);
      }
      hipLaunchKernelGGL(kp::k_epi_cols, dim3(g.grid()), dim3(256), 0, ctx->stream, g.rk, q,
                         g.B, (int64_t)n);
      if ((rc = g.launched())) return rc;
      if ((rc = g.phi(g.jac(slot_u(0)), M, dt))) return rc;
      double* nxt = slot_u(P);                       // the oldest state is no longer read
      if ((rc = g.axpy(nxt, slot_u(0)))) return rc;
      cur = (cur + 1) % (P + 1);
      if ((rc = g.rhs_at(slot_u(0), slot_f(0), true, nullptr))) return rc;
    }
    KP_HIP(ctx, hipMemcpyAsync(u, slot_u(0), sizeof(double) * n, hipMemcpyDeviceToDevice,
                               ctx->stream));
  }
  if (info) {
    KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
    info->status = g.worst;
    info->t_end = dt * nsteps;
  }
  return KP_OK;
}

int kp_get_schedule(kp_ctx* ctx, double* tau_host, int32_t* m_host, int32_t cap) {
  if (!ctx || cap < 0 || (cap > 0 && (!tau_host || !m_host))) return KP_EINVAL;
  const State* st = ctx->st_last;
  if (!st) return KP_ESTATE;
  KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  int nlog = 0;
  KP_HIP(ctx, hipMemcpy(&nlog, &st->nlog, sizeof(int), hipMemcpyDeviceToHost));
  const int n = std::min(std::min(nlog, kp::kLogMax), cap);
  if (n > 0) {
    KP_HIP(ctx, hipMemcpy(tau_host, st->log_tau, n * sizeof(double), hipMemcpyDeviceToHost));
    KP_HIP(ctx, hipMemcpy(m_host, st->log_m, n * sizeof(int32_t), hipMemcpyDeviceToHost));
  }
  return n;
}

int kp_arnoldi_begin(kp_ctx* ctx, const kp_op* A, const double* B, int32_t p, int64_t ldb,
                     int32_t m_max) {
  if (!ctx) return KP_EINVAL;
  Args a;
  kp_config saved = ctx->cfg;
  ctx->cfg.fixed_m = 0;
  int rc = build_args(ctx, A, B, p, ldb, 1.0, 1.0, m_max, nullptr, false, &a);
  ctx->cfg = saved;
  if (rc) return rc;
  if ((rc = prepare(ctx, &a))) return rc;
  a.stop_j = 0;
  if ((rc = launch_init(ctx, a, m_max))) return rc;
  if ((rc = launch(ctx, a, 1))) return rc;
  ctx->last = a;
  ctx->have_begin = 1;
  ctx->arn_target = 0;
  return KP_OK;
}

int kp_arnoldi_step(kp_ctx* ctx, int32_t nsteps) {
  if (!ctx || nsteps < 0) return KP_EINVAL;
  if (!ctx->have_begin) return KP_ESTATE;
  ctx->arn_target = std::min(ctx->arn_target + nsteps, ctx->last.m_max);
  Args a = ctx->last;
  a.stop_j = ctx->arn_target;
  return launch(ctx, a, 1);
}

int kp_arnoldi_read(kp_ctx* ctx, double* H_host, double* V_host, int32_t* j_host,
                    double* beta_host, int32_t* flags_host) {
  if (!ctx) return KP_EINVAL;
  if (!ctx->have_begin) return KP_ESTATE;
  const Args& a = ctx->last;
  KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  std::vector<char> buf(sizeof(State));
  State* h = reinterpret_cast<State*>(buf.data());
  KP_HIP(ctx, hipMemcpy(h, ctx->st, sizeof(State), hipMemcpyDeviceToHost));
  Pub pb;
  KP_HIP(ctx, hipMemcpy(&pb, ctx->pub, sizeof(Pub), hipMemcpyDeviceToHost));
  const int j = pb.j;
  if (j_host) *j_host = j;
  if (beta_host) *beta_host = h->beta;
  if (flags_host) {
    flags_host[0] = h->breakdown;
    flags_host[1] = h->n_fallback;
  }
  if (H_host) {
    const int mm = a.m_max;
    for (int c = 0; c < mm; ++c)
      for (int r = 0; r <= mm; ++r) H_host[(size_t)c * (mm + 1) + r] = h->H[(size_t)c * kp::kLdh + r];
  }
  if (V_host) {
    const int ncol = j + 1;
    const size_t L = (size_t)a.N + a.p;
    const size_t esz = a.basis_f32 ? sizeof(float) : sizeof(double);
    std::vector<char> raw((size_t)a.ld * ncol * esz);
    KP_HIP(ctx, hipMemcpy(raw.data(), ctx->V, raw.size(), hipMemcpyDeviceToHost));
    for (int c = 0; c < ncol; ++c) {
      double scale;
      if (c < j) scale = h->sigma[c];
      else scale = (h->last_nrm2 > 0.0 && !h->breakdown) ? 1.0 / std::sqrt(h->last_nrm2) : 0.0;
      auto at = [&](int64_t e) {
        return a.basis_f32 ? (double)reinterpret_cast<float*>(raw.data())[(size_t)c * a.ld + e]
                           : reinterpret_cast<double*>(raw.data())[(size_t)c * a.ld + e];
      };
      for (int s = 0; s < a.nplanes; ++s)
        for (int64_t q = 0; q < a.npt; ++q)
          V_host[(size_t)c * L + (size_t)s * a.npt + q] = at(s * a.npt_pad + q) * scale;
      for (int k = 0; k < a.p; ++k)
        V_host[(size_t)c * L + a.N + k] = at(a.tail_off + k) * scale;
    }
  }
  return KP_OK;
}

int kp_phi_combo_batched(kp_ctx* ctx, int32_t nprob, const kp_op* ops, const double* const* B,
                         const int32_t* p, const int64_t* ldb, const double* h, double tol,
                         int32_t m_max, double* const* out, kp_info* infos) {
  if (!ctx || nprob < 1 || !ops || !B || !p || !ldb || !h || !out) return KP_EINVAL;
  int rc = device_setup(ctx);
  if (rc) return rc;
  std::vector<Args> as(nprob);
  std::vector<kp::PlanProblem> qs(nprob);
  std::vector<std::pair<uintptr_t, uintptr_t>> spans(nprob);
  for (int i = 0; i < nprob; ++i) {
    if ((rc = build_args(ctx, &ops[i], B[i], p[i], ldb[i], h[i], tol, m_max, out[i], true, &as[i])))
      return rc;
    qs[i] = plan_problem(ops[i], p[i], m_max, h[i]);
    const uintptr_t o = reinterpret_cast<uintptr_t>(out[i]);
    spans[i] = {o, o + (uintptr_t)as[i].N * sizeof(double)};
  }
  // outputs of different problems must not overlap (each team writes its own)
  std::sort(spans.begin(), spans.end());
  for (int i = 1; i < nprob; ++i)
    if (spans[i].first < spans[i - 1].second) return KP_EINVAL;
  choose_batch_kernel(as);
  std::vector<long long> key = {nprob, m_max, ctx->cfg.basis_dtype, ctx->cfg.orth,
                                ctx->cfg.fixed_m, ctx->cfg.fixed_substeps, ctx->model_gen,
                                // the workspace's layout (prob_bufs) also depends on what
                                // build_args derives from the rest of the configuration
                                as[0].block, as[0].pairs, as[0].bstride, as[0].ll};
  for (int i = 0; i < nprob; ++i) {
    key.push_back(ops[i].kind);
    key.push_back(ops[i].nx);
    key.push_back(ops[i].ny);
    key.push_back(p[i]);
  }
  if (!ctx->batch || ctx->batch->key != key) {
    if (ctx->batch) {
      KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
      batch_free(ctx->batch);
      ctx->batch = nullptr;
    }
    if ((rc = batch_create(ctx, as, qs, std::move(key), &ctx->batch))) return rc;
  }
  BatchCache* b = ctx->batch;
  batch_fill_args(b, as, ctx->wait_ticks);
  KP_HIP(ctx, hipMemcpyAsync(b->d_args, b->hargs.data(), sizeof(Args) * b->hargs.size(),
                             hipMemcpyHostToDevice, ctx->stream));
  KP_HIP(ctx, hipGraphLaunch(b->exec, ctx->stream));
  ctx->have_begin = 0;
  if (infos) {
    KP_HIP(ctx, hipMemcpyAsync(infos, b->d_info, sizeof(kp_info) * nprob, hipMemcpyDeviceToHost,
                               ctx->stream));
    KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  }
  return KP_OK;
}

int kp_get_batch_schedule(kp_ctx* ctx, int32_t i, double* tau_host, int32_t* m_host,
                          int32_t cap) {
  if (!ctx || cap < 0 || (cap > 0 && (!tau_host || !m_host))) return KP_EINVAL;
  if (!ctx->batch) return KP_ESTATE;
  if (i < 0 || i >= ctx->batch->nprob) return KP_EINVAL;
  KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  const State* st = ctx->batch->st + i;
  int nlog = 0;
  KP_HIP(ctx, hipMemcpy(&nlog, &st->nlog, sizeof(int), hipMemcpyDeviceToHost));
  const int n = std::min(std::min(nlog, kp::kLogMax), cap);
  if (n > 0) {
    KP_HIP(ctx, hipMemcpy(tau_host, st->log_tau, n * sizeof(double), hipMemcpyDeviceToHost));
    KP_HIP(ctx, hipMemcpy(m_host, st->log_m, n * sizeof(int32_t), hipMemcpyDeviceToHost));
  }
  return n;
}

int kp_batch_plan(int32_t nprob, const kp_op* ops, const int32_t* p, const double* h,
                  int32_t m_max, int32_t n_wg, int32_t* team_of_problem, int32_t* team_wg0,
                  int32_t* team_size, int32_t* nteams, double* makespan, double* work) {
  if (nprob < 1 || !ops || !p || !h || n_wg < 1 || !team_of_problem || !team_wg0 ||
      !team_size || !nteams)
    return KP_EINVAL;
  if (m_max < 1 || m_max > KP_MMAX) return KP_EINVAL;
  std::vector<kp::PlanProblem> qs(nprob);
  for (int i = 0; i < nprob; ++i) {
    const kp_op& A = ops[i];
    if (A.nx < 1 || A.ny < 1 || !(A.dx > 0.0) || !(A.dy > 0.0) || p[i] < 0 || p[i] > KP_PMAX ||
        !std::isfinite(h[i]) || A.kind < KP_OP_ADR || A.kind > KP_OP_BRUSSELATOR)
      return KP_EINVAL;
    qs[i] = plan_problem(A, p[i], m_max, h[i]);
  }
  const kp::Plan pl = kp::make_plan(qs, n_wg, kp::PlanModel());
  const int nt = (int)pl.team_size.size();
  for (int t = 0; t < nt; ++t) {
    team_wg0[t] = pl.team_wg0[t];
    team_size[t] = pl.team_size[t];
    for (int q = pl.team_first[t]; q < pl.team_first[t + 1]; ++q) team_of_problem[pl.order[q]] = t;
  }
  *nteams = nt;
  if (makespan) *makespan = pl.makespan;
  if (work) *work = pl.work;
  return KP_OK;
}

// ---- calibration of the batched planner's cost model --------------------------

namespace {

// Solve the n x n system A x = b (row-major, n <= 8) by Gaussian elimination
// with partial pivoting; false when singular.
bool solve_small(int n, double* A, double* b, double* x) {
  for (int c = 0; c < n; ++c) {
    int piv = c;
    for (int r = c + 1; r < n; ++r)
      if (std::fabs(A[r * n + c]) > std::fabs(A[piv * n + c])) piv = r;
    if (A[piv * n + c] == 0.0) return false;
    for (int k = 0; k < n; ++k) std::swap(A[c * n + k], A[piv * n + k]);
    std::swap(b[c], b[piv]);
    for (int r = c + 1; r < n; ++r) {
      const double f = A[r * n + c] / A[c * n + c];
      for (int k = c; k < n; ++k) A[r * n + k] -= f * A[c * n + k];
      b[r] -= f * b[c];
    }
  }
  for (int r = n - 1; r >= 0; --r) {
    double v = b[r];
    for (int k = r + 1; k < n; ++k) v -= A[r * n + k] * x[k];
    x[r] = v / A[r * n + r];
  }
  return true;
}

bool cache_read(const char* path, const std::string& key, kp::PlanModel* md) {
  FILE* f = std::fopen(path, "r");
  if (!f) return false;
  char line[512];
  bool found = false;
  while (std::fgets(line, sizeof(line), f)) {
    char k[256];
    double v[5];
    if (std::sscanf(line, "%255s %lf %lf %lf %lf %lf", k, &v[0], &v[1], &v[2], &v[3], &v[4]) == 6 &&
        key == k && v[0] > 0.0) {
      md->bw_wg = v[0];
      md->t_step = v[1];
      md->t_team = v[2];
      md->t_log = v[3];
      md->t_expm64 = v[4];
      found = true;   // the last entry of the key wins
    }
  }
  std::fclose(f);
  return found;
}

void cache_write(const char* path, const std::string& key, const kp::PlanModel& md) {
  std::vector<std::string> keep;
  if (FILE* f = std::fopen(path, "r")) {
    char line[512];
    while (std::fgets(line, sizeof(line), f)) {
      char k[256];
      if (std::sscanf(line, "%255s", k) == 1 && key != k) keep.push_back(line);
    }
    std::fclose(f);
  }
  const std::string tmp = std::string(path) + ".tmp";
  FILE* f = std::fopen(tmp.c_str(), "w");
  if (!f) return;
  for (const auto& l : keep) std::fputs(l.c_str(), f);
  std::fprintf(f, "%s %.9g %.9g %.9g %.9g %.9g\n", key.c_str(), md.bw_wg, md.t_step, md.t_team,
               md.t_log, md.t_expm64);
  std::fclose(f);
  std::rename(tmp.c_str(), path);
}

}  // namespace

int kp_calibrate(kp_ctx* ctx, int32_t force, double* model_host) {
  if (!ctx) return KP_EINVAL;
  int rc = device_setup(ctx);
  if (rc) return rc;
  hipDeviceProp_t prop;
  KP_HIP(ctx, hipGetDeviceProperties(&prop, ctx->device));
  char kbuf[256];
  // (the steps per reduction and "batch" name the kernels that the fit is of)
  snprintf(kbuf, sizeof(kbuf), "%s/cu%d/lib%d/batch%d", prop.gcnArchName, ctx->ncu, kp_version(), kp::kS);
  const std::string key(kbuf);
  const char* path = std::getenv("KP_AUTOTUNE_CACHE");
  kp::PlanModel md;
  auto finish = [&](int code) {
    ctx->model = md;
    ctx->model_gen += 1;
    if (model_host) {
      model_host[0] = md.bw_wg;
      model_host[1] = md.t_step;
      model_host[2] = md.t_team;
      model_host[3] = md.t_log;
      model_host[4] = md.t_expm64;
    }
    return code;
  };
  if (!force && path && *path && cache_read(path, key, &md)) return finish(1);

  // the small exponential at m = 64: device time of the test kernel
  if (!ctx->st) {
    KP_HIP(ctx, hipMalloc(&ctx->st, sizeof(State)));
    KP_HIP(ctx, hipMalloc(&ctx->pub, sizeof(Pub)));
    KP_HIP(ctx, hipMalloc(&ctx->sync, 64));
    KP_HIP(ctx, hipMalloc(&ctx->ex, sizeof(double) * kp::kExSlots * kp::kNmPad * kp::kNmPad));
    KP_HIP(ctx, hipMalloc(&ctx->tx, sizeof(double) * kp::kTailPad));
  }
  hipEvent_t e0, e1;
  KP_HIP(ctx, hipEventCreate(&e0));
  KP_HIP(ctx, hipEventCreate(&e1));
  auto timed = [&](auto&& fn, int reps, double* med_s) -> int {
    std::vector<float> ms;
    for (int r = 0; r <= reps; ++r) {           // the first call warms up
      KP_HIP(ctx, hipEventRecord(e0, ctx->stream));
      const int c = fn();
      if (c) return c;
      KP_HIP(ctx, hipEventRecord(e1, ctx->stream));
      KP_HIP(ctx, hipEventSynchronize(e1));
      float t = 0.f;
      KP_HIP(ctx, hipEventElapsedTime(&t, e0, e1));
      if (r) ms.push_back(t);
    }
    std::sort(ms.begin(), ms.end());
    *med_s = 1e-3 * ms[ms.size() / 2];
    return KP_OK;
  };
  {
    const int m = 64;
    std::vector<double> Hs((size_t)kp::kLdh * kp::kMMax, 0.0);
    for (int c = 0; c < m; ++c)
      for (int r = 0; r <= c + 1; ++r)
        Hs[(size_t)c * kp::kLdh + r] = (r == c) ? -2.0 - 0.05 * c : 0.3 * std::sin(1.0 + r + 7.0 * c);
    KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
    KP_HIP(ctx, hipMemcpy(ctx->ex, Hs.data(), Hs.size() * sizeof(double), hipMemcpyHostToDevice));
    double t = 0.0;
    rc = timed([&]() {
      hipLaunchKernelGGL(kp::k_expm_test, dim3(1), dim3(kp::kThreads), 0, ctx->stream, ctx->ex,
                         ctx->ex + Hs.size(), m, 1.0);
      return hipGetLastError() == hipSuccess ? KP_OK : KP_EHIP;
    }, 5, &t);
    if (rc) return rc;
    md.t_expm64 = t;
  }
  // fixed-schedule sets (one substep of m steps, advection-diffusion, p = 1) through
  // the batched kernel itself, identical problems on uniform teams that fill the
  // grid: teams of one and of more workgroups, 4096 and more elements each, so
  // that the four columns of the fit are independent
  struct Cal { int side, g, m; };
  const Cal cals[] = {{128, 1, 48}, {64, 1, 48}, {128, 2, 48}, {128, 4, 48}, {256, 16, 48}, {512, 16, 24}, {512, 64, 48}};
  const int ncal = (int)(sizeof(cals) / sizeof(cals[0]));
  const int p = 1, n_wg = ctx->ncu;            // (one workgroup per CU at least is resident)
  size_t nb = 0, ny = 0;
  for (const Cal& c : cals) {
    const size_t n = (size_t)c.side * c.side;
    nb = std::max(nb, n * (p + 1));
    ny = std::max(ny, n * (size_t)std::max(1, n_wg / c.g));
  }
  double* Bd = nullptr;
  double* yd = nullptr;
  KP_HIP(ctx, hipMalloc(&Bd, sizeof(double) * nb));
  if (hipMalloc(&yd, sizeof(double) * ny) != hipSuccess) {
    hipFree(Bd);
    return KP_ENOMEM;
  }
  hipLaunchKernelGGL(kp::k_fill_pattern, dim3(4096), dim3(256), 0, ctx->stream, Bd, (int64_t)nb);
  const kp_config saved = ctx->cfg;
  ctx->cfg = kp_config{};                      // H-GSMGS, float64, the default controller
  ctx->cfg.stream = saved.stream;
  double A[ncal][4], y[ncal];
  int used = 0;
  for (int i = 0; i < ncal && rc == KP_OK; ++i) {
    const Cal& c = cals[i];
    if (c.g > n_wg) continue;
    const int np = n_wg / c.g;
    kp_op op{};
    op.kind = KP_OP_ADR;
    op.nx = op.ny = c.side;
    op.dx = op.dy = 1.0 / c.side;
    op.nu = 0.01;
    op.ax = 1.0;
    op.ay = 0.5;
    ctx->cfg.fixed_m = c.m;
    ctx->cfg.fixed_substeps = 1;
    const int64_t n = (int64_t)c.side * c.side;
    std::vector<Args> as(np);
    std::vector<kp::PlanProblem> qs(np, plan_problem(op, p, c.m, 1e-4));
    for (int q = 0; q < np && rc == KP_OK; ++q)
      rc = build_args(ctx, &op, Bd, p, n, 1e-4, 1.0, c.m, yd + q * n, true, &as[q]);
    if (rc) break;
    choose_batch_kernel(as);
    const kp::Plan plan = kp::uniform_plan(np, n_wg, c.g);
    BatchCache* b = nullptr;
    if ((rc = batch_create(ctx, as, qs, {}, &b, &plan))) break;
    batch_fill_args(b, as, ctx->wait_ticks);
    double t = 0.0;
    rc = timed([&]() -> int {
      KP_HIP(ctx, hipMemcpyAsync(b->d_args, b->hargs.data(), sizeof(Args) * b->hargs.size(),
                                 hipMemcpyHostToDevice, ctx->stream));
      KP_HIP(ctx, hipGraphLaunch(b->exec, ctx->stream));
      return KP_OK;
    }, 3, &t);
    hipStreamSynchronize(ctx->stream);
    batch_free(b);
    const double S = c.m;
    y[used] = t - md.t_expm64 * (S * S) / (64.0 * 64.0);
    A[used][0] = kp::plan_bytes(qs[0], S, S, c.g, md);
    A[used][1] = S;
    A[used][2] = c.g > 1 ? S : 0.0;
    A[used][3] = S * std::log2((double)c.g);
    ++used;
  }
  ctx->cfg = saved;
  ctx->have_begin = 0;
  hipFree(Bd);
  hipFree(yd);
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  if (rc) return rc;
  // least squares of the relative errors, the coefficients not negative: the most
  // negative of a solution is left out and the rest fitted again
  double x[4] = {0};
  bool in[4] = {true, true, true, true}, ok = false;
  for (int round = 0; round < 4; ++round) {
    double AtA[16], Atb[4], z[4];
    for (int r = 0; r < 4; ++r) {
      Atb[r] = 0.0;
      for (int k = 0; k < 4; ++k) AtA[r * 4 + k] = (r == k && !in[r]) ? 1.0 : 0.0;
      for (int i = 0; i < used && in[r]; ++i) {
        Atb[r] += A[i][r] / y[i];
        for (int k = 0; k < 4; ++k)
          if (in[k]) AtA[r * 4 + k] += A[i][r] * A[i][k] / (y[i] * y[i]);
      }
    }
    if (!solve_small(4, AtA, Atb, z)) break;
    int worst = -1;
    for (int k = 1; k < 4; ++k)
      if (in[k] && z[k] < 0.0 && (worst < 0 || z[k] * A[used - 1][k] < z[worst] * A[used - 1][worst])) worst = k;
    if (worst < 0) {
      std::copy(z, z + 4, x);
      ok = x[0] > 0.0;
      break;
    }
    in[worst] = false;
  }
  if (!ok) {   // no usable fit: the built-in constants, and nothing cached
    md = kp::PlanModel();
    return finish(2);
  }
  md.bw_wg = 1.0 / x[0];
  md.t_step = std::max(x[1], 1e-7);
  md.t_team = x[2];
  md.t_log = x[3];
  if (path && *path) cache_write(path, key, md);
  return finish(0);
}

int kp_expm_hbar(kp_ctx* ctx, const double* H_host, int32_t ldh, int32_t m, double tau,
                 double* F_host) {
  if (!ctx || !H_host || !F_host || m < 1 || m > KP_MMAX || ldh < m + 1 || !std::isfinite(tau))
    return KP_EINVAL;
  int rc = device_setup(ctx);
  if (rc) return rc;
  if (!ctx->st) {
    KP_HIP(ctx, hipMalloc(&ctx->st, sizeof(State)));
    KP_HIP(ctx, hipMalloc(&ctx->pub, sizeof(Pub)));
    KP_HIP(ctx, hipMalloc(&ctx->sync, 64));
    KP_HIP(ctx, hipMalloc(&ctx->ex, sizeof(double) * kp::kExSlots * kp::kNmPad * kp::kNmPad));
    KP_HIP(ctx, hipMalloc(&ctx->tx, sizeof(double) * kp::kTailPad));
  }
  std::vector<double> Hs((size_t)kp::kLdh * kp::kMMax, 0.0);
  for (int c = 0; c < m; ++c)
    for (int r = 0; r <= m; ++r) Hs[(size_t)c * kp::kLdh + r] = H_host[(size_t)c * ldh + r];
  KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  double* F = ctx->ex + Hs.size();
  KP_HIP(ctx, hipMemcpy(ctx->ex, Hs.data(), Hs.size() * sizeof(double), hipMemcpyHostToDevice));
  hipLaunchKernelGGL(kp::k_expm_test, dim3(1), dim3(kp::kThreads), 0, ctx->stream, ctx->ex, F, m, tau);
  KP_HIP(ctx, hipGetLastError());
  KP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  KP_HIP(ctx, hipMemcpy(F_host, F, (m + 1) * sizeof(double), hipMemcpyDeviceToHost));
  return KP_OK;
}

}  // extern "C"
