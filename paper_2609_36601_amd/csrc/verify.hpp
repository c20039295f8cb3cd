// The speculative verification kernel.
#pragma once

#include "common.hpp"

namespace saki {

// ---------------------------------------------------------------------------
// Speculative verification.  A work item is one position; items are taken
// position-major (position 0 of every block, then position 1, ...), so a
// block's positions run on different workgroups and, in a small batch, at the
// same time.  Positions are independent given their rows, and the first
// stopping one decides: each block keeps its smallest stopping position with
// its outcome in one word (atomicMin on accepted_len[b]; stop_word), items
// after it are skipped, and a short second kernel turns the words into the
// outputs.  A position whose rejection is certain from the row statistics says
// so before it has its lambda* and correction (the smallest such position of a
// block, atomicMin on correction[b]): positions behind it are skipped too.  In a batch large enough to fill the chip, position j of a block is
// taken long after its position j - 1 has ended, so few positions are
// evaluated in vain; in a small batch the idle workgroups evaluate them ahead
// instead of the block's positions running one after another.
// Measured on one MI355X, V = 151,936 bf16, against one workgroup per block
// that took its positions in order: 64 blocks of 8 with every output 789 ->
// 206 us (all 512 positions at once), 1,024 blocks of 8 without per-position
// outputs 1,177 -> 928 us (the last blocks' remaining positions no longer run
// one after another at the end).
// ---------------------------------------------------------------------------
struct VerifyParams {
  const void* s;
  const void* t;
  int64_t n_blocks;
  int64_t stride;
  int64_t row_offset;
  int V;
  int k;
  const int32_t* draft;
  double eps;
  float lam_mid;  // mid_lambda(eps)
  uint64_t seed;
  int eos;
  int32_t* accepted_len;  // the blocks' words until verify_end_kernel
  int32_t* correction;    // the blocks' first position known to reject until then (k: none)
  saki_couple_out pp;  // per-position outputs (fields may be NULL)
  int has_pp;
  unsigned long long* next_item;  // work counter in the caller's workspace, zero at launch
};

// A block's outcome: the position j at which it stops, whether it stops behind
// an accepted EOS draft, and the correction (-1: none).  Smaller j is smaller,
// so atomicMin keeps the first stop; j = k without a stop.  6 + 1 bits of j
// (k <= 64), one of EOS, 22 of the correction (vocab <= 2^21).
__host__ __device__ inline int32_t stop_word(int j, bool eos, int corr) {
  return (j << 23) | (eos ? 1 << 22 : 0) | (corr + 1);
}
__host__ __device__ inline int stop_pos(int32_t w) { return w >> 23; }
static_assert(SAKI_MAX_BLOCK_K <= 64 && SAKI_MAX_VOCAB <= (1 << 21), "stop_word holds k and the vocabulary");

// An upper bound of log q(z) - log p(z) = g(lambda*), g(lam) = lam x_z - A(lam),
// from the row statistics: g is concave, so it lies below its tangents at
// lambda = 0 and at the middle node lm, whose largest values over a bracket of
// lambda* are at its ends.  KL(lm) against eps tells on which side of lm lambda*
// lies (both, when too close to tell); below, KL(lam) = int_0^lam l A''(l) dl <=
// lam (A'(lm) - A'(0)), so lambda* is at least eps / (A'(lm) - A'(0)).  `slack`
// covers the float sums: the moments of d to 1e-5 of its range (ten times their
// rounding), A to 1e-4.
__device__ __forceinline__ double log_ratio_bound(const RowStats& R, double eps, float s, float t) {
  if (!(R.lam_mid > 0.0)) return 0.0;
  const double lm = R.lam_mid, c = static_cast<double>(R.c);
  const double slack = 1e-5 * (static_cast<double>(R.dmax) - static_cast<double>(R.dmin));
  const double xz = static_cast<double>(t) - static_cast<double>(s) - c;
  const double klm = lm * R.mid_A1 - R.mid_A, rise = R.mid_A1 - (R.mean_p - c) + slack;
  const double low = eps < lm * rise ? eps / rise : lm;
  const double la = klm < eps * (1.0 - 1e-3) - slack ? lm : low, lb = klm > eps * (1.0 + 1e-3) + slack ? lm : 1.0;
  const double k0 = xz - (R.mean_p - c), km = xz - R.mid_A1;
  const double u0 = fmax(k0 * la, k0 * lb);
  const double um = lm * xz - R.mid_A + fmax(km * (la - lm), km * (lb - lm));
  const double b = fmin(u0, um) + 1e-4 + slack;
  return b < 0.0 ? b : 0.0;  // (NaN: no bound)
}

// o: the per-position outputs, in the argument segment or elsewhere (the
// proposals are written by verify_begin_kernel)
template <typename O>
__device__ __forceinline__ void write_skipped(const O* o, int64_t r, uint8_t status) {
  if (o->lambda) o->lambda[r] = nanf_();
  if (o->kl) o->kl[r] = nanf_();
  if (o->tv) o->tv[r] = nanf_();
  if (o->accept_prob) o->accept_prob[r] = nanf_();
  if (o->margin) o->margin[r] = nanf_();
  if (o->logp_token) o->logp_token[r] = nanf_();
  if (o->logt_token) o->logt_token[r] = nanf_();
  if (o->logq_token) o->logq_token[r] = nanf_();
  if (o->token) o->token[r] = -1;
  if (o->teacher_argmax) o->teacher_argmax[r] = -1;
  if (o->target) o->target[r] = -1;
  if (o->corrected) o->corrected[r] = 0;
  if (o->row_status) o->row_status[r] = status;
}

// VNT threads per workgroup: 256 (two workgroups per CU), or 512 (one per CU)
// when a call has no more blocks than CUs: each position's sweeps are spread
// over eight waves, nothing shares its CU, and about CUs / n_blocks positions
// of a block run ahead of the first stop.  (Two workgroups per CU from more
// positions than CUs on take the average batch faster, 64 / 256 blocks of 8 x
// 151,936 with every output in 190 / 415 instead of 206 / 470 us, but a batch
// whose blocks stop early slower, its positions sharing the chip with twice as
// many evaluated in vain: 64 / 128 / 256 blocks stopped at position 0 309 / 370 /
// 460 us, 169 / 192 / 269 now.)
template <typename T, int KC, int VNT, bool K34>
__global__ __launch_bounds__(VNT, VNT == 256 ? 2 : 1) void verify_kernel(VerifyParams) {
  using SH = RowShared<VNT, (KC > 0 ? CACHED_MAXC : MAX_CHUNKS), KC>;
  __shared__ SH sh;
  __shared__ RowPlan plan;
  Block<VNT, SH> B(sh);
  const auto* P = kernel_args<VerifyParams>();
  const int V = P->V;
  const int nch = (V + CHUNK - 1) / CHUNK;
  const bool need_tv = P->has_pp && P->pp.tv != nullptr;
  // outputs that need lambda* at an accepted position
  const bool need_lam = P->has_pp && (P->pp.lambda || P->pp.kl || P->pp.tv || P->pp.accept_prob || P->pp.margin || P->pp.logq_token);
  // Thread 0 takes the next item that its block does not rule out and posts it
  // in LDS; readfirstlane makes it, and so the loop's exit, uniform in every
  // wave, so all threads reach the same barriers.  The counter only grows, so
  // every thread 0 reaches n_items and every loop ends.
  __shared__ long long next_i;
  const long long n_items = P->n_blocks * P->k;
  const unsigned int nb = static_cast<unsigned int>(P->n_blocks);
  auto look = [](const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  for (;;) {
    P = kernel_args<VerifyParams>();
    if (B.tid == 0) {
      long long i;
      for (;;) {
        i = static_cast<long long>(take_index(P->next_item));
        if (i >= n_items) break;
        // a stale word only costs a position evaluated in vain
        const int32_t w = look(P->accepted_len + i % nb), rj = look(P->correction + i % nb);
        if (stop_pos(w) >= static_cast<int>(i / nb) && rj >= static_cast<int>(i / nb)) break;
      }
      next_i = i;
    }
    __syncthreads();
    const unsigned int i_lo = static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(next_i)));
    const unsigned int i_hi = static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(next_i >> 32)));
    __syncthreads();
    const long long item = static_cast<long long>((static_cast<unsigned long long>(i_hi) << 32) | i_lo);
    if (item >= n_items) break;
    const int j = static_cast<int>(item / nb);
    const int64_t b = item % nb;
    const int64_t r = b * P->k + j;
    // is this position behind its block's stop, or behind one known to reject?
    auto behind = [&](int32_t word, int32_t rj) { return stop_pos(word) < j || rj < j; };
    // a position resolved in a plain form whose TV turns out too small for
    // that form's rounding is processed again with every sweep in the expm1
    // form (rare): force_acc is all that crosses the restart
    bool force_acc = false;
    for (;;) {
      const T* srow = static_cast<const T*>(P->s) + r * P->stride;
      const T* trow = static_cast<const T*>(P->t) + r * P->stride;
      const uint64_t g = static_cast<uint64_t>(P->row_offset + r);
      const int z = P->draft[r];
      if (uniform(z < 0 || z >= V)) {
        if (B.tid == 0) {
          if (P->has_pp) write_skipped(&P->pp, r, SAKI_ROW_BAD_DRAFT);
          atomicMin(P->accepted_len + b, stop_word(j, false, -1));
        }
        break;
      }
      // while wave 0 combines the sums, a lane of the last wave draws the uniform
      auto idle = [&]() {
        if (B.tid == VNT - WAVE) sh.u = philox_uniform(P->seed, ACCEPT, g, 0);
      };
      const RowStats& R = stats_sweep<T, VNT, K34>(B, srow, trow, V, P->lam_mid, false, false, idle);
      P = kernel_args<VerifyParams>();
      if (uniform(!R.finite)) {
        if (B.tid == 0) {
          if (P->has_pp) write_skipped(&P->pp, r, SAKI_ROW_NONFINITE);
          atomicMin(P->accepted_len + b, stop_word(j, false, -1));
        }
        break;
      }
      const float sz = Loader<T>::load1(srow + z), tz = Loader<T>::load1(trow + z);
      const double u = static_cast<double>(sh.u);
      // g(lam) = lam x_z - A(lam) = log q(z) - log p(z) is concave in lam with
      // g(0) = 0, so on a bracket [la, lb] of lambda* it lies above min(g(la),
      // g(lb)): a draft with u below exp of that is accepted whatever lambda*
      // is, and when no output needs lambda* its search is skipped.  The
      // bracket is [0, 1] (g(1) = log pi(z) - log p(z)), or split at the
      // middle node by the sign of KL(lm) - eps; the middle node's values come
      // from float sums, so that bound keeps a margin of 2e-6.
      if (!need_lam) {
        const double lr1 = (static_cast<double>(tz) - R.lse_t) - (static_cast<double>(sz) - R.lse_s);
        double gmin = fmin(0.0, lr1);
        if (R.lam_mid > 0.0) {
          const double lm = R.lam_mid;
          const double xz = static_cast<double>(tz) - static_cast<double>(sz) - static_cast<double>(R.c);
          const double gm = lm * xz - R.mid_A;
          const double klm = lm * R.mid_A1 - R.mid_A;
          // Above the middle node the bracket can end below 1, where
          // convexity alone forces KL > eps.  With A and A' known at lm and 1, the
          // tangent of A at lambda lies below A at lm, so A'(lambda) >=
          // (A(lambda) - A(lm)) / (lambda - lm), and A(lambda) lies above the
          // tangent at 1; together KL(lambda) >= (lm T1(lambda) - lambda A(lm))
          // / (lambda - lm), T1 that tangent, which passes eps at lh below.
          // On [lm, lh] g lies above lambda x_z minus the chord of A from lm
          // to 1 (A is convex), a line: its smaller end value bounds g.
          // Guards keep lh away from cancellations in the float sums.
          const double A1 = R.lse_t - R.lse_s - static_cast<double>(R.c);
          const double D1 = R.mean_pi - static_cast<double>(R.c);
          const double num = R.kl1_est - P->eps, den = lm * D1 - R.mid_A - P->eps;
          double g_hi = lr1;
          if (num > 1e-2 * (fabs(R.kl1_est) + P->eps) &&
              den > 1e-2 * (fabs(lm * D1) + fabs(R.mid_A) + P->eps)) {
            const double lh = fmax(lm, lm * num / den * (1.0 + 1e-3) + 1e-6);
            if (lh < 1.0) g_hi = lh * xz - (R.mid_A + (A1 - R.mid_A) * (lh - lm) / (1.0 - lm));
          }
          const double lo_side = fmin(0.0, gm), hi_side = fmin(gm, g_hi);
          const double gb = (klm < P->eps * (1.0 - 1e-3)) ? hi_side : (klm > P->eps * (1.0 + 1e-3)) ? lo_side
                                                                     : fmin(lo_side, hi_side);
          gmin = fmax(gmin, gb - 2e-6);
        }
        if (uniform(u < exp(gmin))) {
          if (P->has_pp && B.tid == 0) {
            if (P->pp.logp_token) P->pp.logp_token[r] = static_cast<float>(static_cast<double>(sz) - R.lse_s);
            if (P->pp.logt_token) P->pp.logt_token[r] = static_cast<float>(static_cast<double>(tz) - R.lse_t);
            if (P->pp.token) P->pp.token[r] = z;
            if (P->pp.teacher_argmax) P->pp.teacher_argmax[r] = R.vstar;
            if (P->pp.target) P->pp.target[r] = z;
            if (P->pp.corrected) P->pp.corrected[r] = 0;
            if (P->pp.row_status) P->pp.row_status[r] = SAKI_ROW_OK;
          }
          if (P->eos >= 0 && z == P->eos && B.tid == 0) atomicMin(P->accepted_len + b, stop_word(j, true, -1));
          break;
        }
      }
      // Positions the interpolating start places well take the fused sweep
      // (the lambda node, and the residual chunk masses where the start
      // predicts a rejection); the others the lambda search and, when rejected
      // or when TV is asked for, the final sweep.  With one workgroup per CU
      // every position takes the search: it evaluates a node at lambda* itself,
      // where the fused sweep's node can lie 2% away (200 blocks of 8 x 5,000:
      // lambda* and TV within 6e-7 against 4e-6 and 7e-6), and the batch waits for
      // its slowest position, which the fused sweep, run in vain there, delays
      // (32 blocks of 8 x 151,936, every output: 119 us, 136 with it; one block,
      // whose positions may all settle in it: 103 us, 92 with it).
      const bool end_first = R.kl1_est <= 1.05 * P->eps + 1e-5;
      if (B.wave == 0) {
        // the block's words again, loaded while the start point is computed: the
        // position is dropped when an earlier one stops the block
        const int32_t word = look(P->accepted_len + b), rj = look(P->correction + b);
        const bool place = P->eps > 0.0 && R.dmin != R.dmax;  // lambda* is searched for
        StartPoint S0;
        S0.lam = 1.0; S0.A = R.lse_t - R.lse_s - static_cast<double>(R.c); S0.herm = true;
        if (place && !end_first) S0 = start_point(R, P->eps);
        const double top = S0.lam * (static_cast<double>(R.dmax) - static_cast<double>(R.c));
        const bool fu = VNT == 256 && !force_acc && place && S0.herm && top <= 56.0 &&
                        (top - S0.A) * static_cast<double>(LOG2E) <= 56.0;
        // rejected whatever lambda* turns out to be: the positions behind are not needed
        const bool reject = place && sh.u > fexp2(static_cast<float>(log_ratio_bound(R, P->eps, sz, tz)) * LOG2E);
        if (B.lane == 0) {
          const bool drop = behind(word, rj);
          if (reject && !drop) atomicMin(P->correction + b, j);
          plan.C = reject ? 1 : 0;
          plan.S0 = S0;
          plan.fused = drop ? -1 : fu ? 1 : 0;
        }
      }
      __syncthreads();
      const int way = __builtin_amdgcn_readfirstlane(plan.fused);
      if (way < 0) break;
      const bool fused = VNT == 256 && way != 0;
      // once said, a rejection stands (the positions behind may have been skipped)
      const bool rejected = uniform(plan.C != 0);
      LamResult L;
      FinalConst F;
      double TV = __builtin_nan("");
      bool settled = false;  // lambda*, the decision, TV (if valid) and the residual chunk from the fused sweep
      bool tv_ok = false;
      bool tv_acc = false;   // the fused sweep's form (the final sweep's is F.acc)
      int res_chunk = nch;
      bool search = true;    // lambda* by lambda sweeps
      // between the sweeps of a search: has the block stopped meanwhile?  (The
      // words as they were before the last sweep, so that nothing waits for them.)
      int32_t word = 0, rj = 0;
      int swept = 0;
      auto gone = [&]() {
        if (j == 0) return false;
        if (B.tid == 0) sh.next = behind(word, rj) ? 1u : 0u;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(static_cast<int>(sh.next)) != 0;
      };
      if (fused) {
        // the decision at the start point (in float, as in the coupling kernel)
        const float lam_g = static_cast<float>(plan.S0.lam);
        const float A_g = static_cast<float>(plan.S0.A * static_cast<double>(LOG2E));
        const bool reject_g = uniform(!(sh.u < fexp2(fminf(0.0f, fmaf(lam_g, fmaf(tz - sz, LOG2E, -R.cL), -A_g)))));
        FusedConst FC;
        FC.msL = R.ms * LOG2E;
        FC.cL = R.cL;
        FC.lam = lam_g;
        FC.AL = A_g;
        FC.gsc = 0.0f;
        FC.set_y();
        const bool facc = (end_first ? R.kl1_est < 1.01 * KL_ACCURATE : P->eps < KL_ACCURATE) || R.pmax > P_PEAKED;
        tv_acc = facc;
        FusedSums FS = fused_sweep_any<T, float, VNT, false>(B, srow, trow, nullptr, V, FC, facc, reject_g,
                                                                  0.0f, 0.0f, -1, 0.0f);
        double le0 = 0.0;
        if (B.wave == 0) {
          FC.set_node();
          word = look(P->accepted_len + b);
          rj = look(P->correction + b);
          const LamEval E0 = fused_node(R, FS, FC, end_first, facc);
          const LamResult L0 = lambda_search_with(R, P->eps, [](float, bool) { LamEval e{}; return e; },
                                                  [] { return true; }, false, 0.0f, true, E0, facc);
          int state = -1, C0 = 0;
          double alpha0 = 0.0;
          FinalConst F0{};
          FusedFinal FF0{};
          if (L0.sweeps == 0) {
            F0 = final_const(R, L0, false);
            alpha0 = exp(fmin(0.0, L0.log_ratio(sz, tz)));
            C0 = rejected || !(u < alpha0) ? 1 : 0;
            FF0 = fused_tv(R, L0, F0, FC, FS, facc);
            // settled unless the decision or TV needs the final sweep: a
            // rejection needs valid residual masses (kept only where the
            // start predicted it), TV a valid correction
            const bool need_final = (C0 != 0) ? !(FF0.ok && reject_g) : (need_tv && !FF0.ok);
            state = need_final ? 0 : 1;
          }
          if (state != 1 && behind(word, rj)) state = -2;  // more sweeps, in vain
          if (B.lane == 0) {
            plan.L = L0;
            plan.F = F0;
            plan.FF = FF0;
            plan.E0 = E0;
            plan.alpha = alpha0;
            plan.state = state;
            plan.C = C0;
          }
        } else if (reject_g) {
          le0 = res_race_begin<VNT>(B, nch, P->seed, g);
        }
        __syncthreads();
        const int state = __builtin_amdgcn_readfirstlane(plan.state);
        if (state == -2) break;
        search = state < 0;
        if (!search) {
          L = plan.L;
          F = plan.F;
          if (state == 1) {
            settled = true;
            tv_ok = plan.FF.ok;
            if (tv_ok) TV = plan.FF.TV;
            if (uniform(plan.C != 0)) {
              const double hx = plan.FF.hmax * LN2_D;  // expm1(x) <= x + x^2, as in the coupling kernel
              const double hb = hx * (1.0 + hx) * 1.02 + 2e-6;
              res_chunk = __builtin_amdgcn_readfirstlane(
                  res_race_end<VNT>(B, nch, P->seed, g, le0, hb, plan.FF.flip));
              if (res_chunk < 0) {
                settled = false;
                res_chunk = nch;
              }
            }
          }
        }
      }
      if (search) {
        const LamEval E0 = fused ? plan.E0 : LamEval{};
        L = lambda_search_with(R, P->eps, [&](float lam, bool acc) {
          ++swept;
          if (B.tid == 0) {
            word = look(P->accepted_len + b);
            rj = look(P->correction + b);
          }
          return lam_sweep<T, VNT>(B, srow, trow, V, R, lam, acc);
        }, [&] { return swept > 0 && gone(); }, force_acc, static_cast<float>(plan.S0.lam), fused, E0, tv_acc);
        if (L.sweeps < 0) break;
        F = final_const(R, L, force_acc);
      }
      const double alpha = exp(fmin(0.0, L.log_ratio(sz, tz)));
      const bool accept = u < alpha && !rejected;
      if (!settled && (need_tv || !accept)) {
        if (swept > 0 && gone()) break;
        TV = final_sweep_any<T, float, VNT, false>(B, srow, trow, nullptr, V, F, !accept, 0.0f, -1, 0.0f);
        tv_ok = true;
        if (!accept) {
          res_chunk = chunk_race<VNT>(B, nch, P->seed, RES_CHUNK, g, [&](int c) {
            const float m = sh.chunk_a[c];
            return m > 0.0f ? log(static_cast<double>(m)) : -__builtin_huge_val();
          });
        }
      }
      if (uniform((need_tv || !accept) && tv_ok && !force_acc &&
                  redo_accurate(R, L, settled ? tv_acc : F.acc, TV))) {
        force_acc = true;
        continue;
      }
      int y = z;
      float sy = sz, ty = tz;
      if (!accept) {
        const int c1 = res_chunk;
        if (c1 < nch) {
          const ElemFetch<T> fr = elem_fetch<T, VNT>(srow, trow, c1, V, B.tid);
          float sw, tw;
          const int yc = elem_pick<VNT>(B, fr, c1, V, P->seed, RES_ELEM, g, [&](float sv, float tv, int) {
            float p;
            const float w = res_weight_any(sv, tv, F, &p);
            return w > 0.0f ? flog2(w) * LN2 : -finf();
          }, &sw, &tw);
          if (yc < V) {
            y = yc;
            sy = sw;
            ty = tw;
          }
        }
      }
      P = kernel_args<VerifyParams>();
      if (P->has_pp && B.tid == 0) {
        const double logp_y = static_cast<double>(sy) - R.lse_s;
        const double logt_y = static_cast<double>(ty) - R.lse_t;
        if (P->pp.lambda) P->pp.lambda[r] = L.lam;
        if (P->pp.kl) P->pp.kl[r] = static_cast<float>(L.KL);
        if (P->pp.tv) P->pp.tv[r] = static_cast<float>(TV);
        if (P->pp.accept_prob) P->pp.accept_prob[r] = static_cast<float>(alpha);
        if (P->pp.margin) P->pp.margin[r] = static_cast<float>(fabs(u - alpha));
        if (P->pp.logp_token) P->pp.logp_token[r] = static_cast<float>(logp_y);
        if (P->pp.logt_token) P->pp.logt_token[r] = static_cast<float>(logt_y);
        if (P->pp.logq_token) P->pp.logq_token[r] = static_cast<float>(logp_y + L.log_ratio(sy, ty));
        if (P->pp.token) P->pp.token[r] = y;
        if (P->pp.teacher_argmax) P->pp.teacher_argmax[r] = R.vstar;
        if (P->pp.target) P->pp.target[r] = accept ? z : R.vstar;
        if (P->pp.corrected) P->pp.corrected[r] = accept ? 0 : 1;
        if (P->pp.row_status) P->pp.row_status[r] = SAKI_ROW_OK;
      }
      if (B.tid == 0) {
        if (!accept)
          atomicMin(P->accepted_len + b, stop_word(j, false, y));
        else if (P->eos >= 0 && z == P->eos)
          atomicMin(P->accepted_len + b, stop_word(j, true, -1));
      }
      break;
    }
  }
}

// Launches the verification kernel for one form of the stats sweep; each PART
// (K34) is compiled in its own unit (verify.hip).
template <int PART>
hipError_t launch_verify_part(const VerifyParams& P, int cus, bool bf16, hipStream_t st);

}  // namespace saki
