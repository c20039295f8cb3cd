// The speculative verification kernel.
#pragma once

#include "common.hpp"

namespace saki {

// ---------------------------------------------------------------------------
// Speculative verification: one workgroup per block, positions in order.
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
  uint64_t seed;
  int eos;
  int32_t* accepted_len;
  int32_t* correction;
  saki_couple_out pp;  // per-position outputs (fields may be NULL)
  int has_pp;
  unsigned int* next_block;  // work counter in the caller's workspace, zero at launch
};

__device__ inline void write_skipped(const saki_couple_out& o, int64_t r, int32_t draft, uint8_t status) {
  if (o.lambda) o.lambda[r] = nanf_();
  if (o.kl) o.kl[r] = nanf_();
  if (o.tv) o.tv[r] = nanf_();
  if (o.accept_prob) o.accept_prob[r] = nanf_();
  if (o.margin) o.margin[r] = nanf_();
  if (o.logp_token) o.logp_token[r] = nanf_();
  if (o.logt_token) o.logt_token[r] = nanf_();
  if (o.logq_token) o.logq_token[r] = nanf_();
  if (o.proposal) o.proposal[r] = draft;
  if (o.token) o.token[r] = -1;
  if (o.teacher_argmax) o.teacher_argmax[r] = -1;
  if (o.target) o.target[r] = -1;
  if (o.corrected) o.corrected[r] = 0;
  if (o.row_status) o.row_status[r] = status;
}

// VNT threads per workgroup: 256 (two workgroups per CU) for large batches,
// 512 (one per CU) when a call has no more blocks than CUs, as in rollouts,
// so that each position's sweeps are spread over eight waves.
template <typename T, int KC, int VNT, bool K34>
__global__ __launch_bounds__(VNT, VNT == 256 ? 2 : 1) void verify_kernel(VerifyParams P) {
  using SH = RowShared<VNT, (KC > 0 ? CACHED_MAXC : MAX_CHUNKS), KC>;
  __shared__ SH sh;
  __shared__ RowPlan plan;
  Block<VNT, SH> B(sh);
  const int V = P.V;
  const int nch = (V + CHUNK - 1) / CHUNK;
  const saki_couple_out& o = P.pp;
  const bool need_tv = P.has_pp && o.tv != nullptr;
  // outputs that need lambda* at an accepted position
  const bool need_lam = P.has_pp && (o.lambda || o.kl || o.tv || o.accept_prob || o.margin || o.logq_token);
  // Blocks cost one to k positions, so workgroups take them from a counter
  // (dynamic scheduling) rather than with a fixed stride.  Each iteration
  // takes a new block or ends the loop, so at most n_blocks + 1 iterations run.
  __shared__ unsigned int next_b;
  for (int64_t it = 0; it <= P.n_blocks; ++it) {
    const unsigned int bu = take_next(P.next_block, &next_b);
    // unsigned: n_blocks < 2^31 and the counter stays below n_blocks + grid
    if (bu >= static_cast<unsigned int>(P.n_blocks)) break;
    const int64_t b = static_cast<int64_t>(bu);
    int n = P.k;
    int corr = -1;
    int next_unwritten = P.k;  // first position whose per-position outputs are not yet written
    // a position resolved in a plain form whose TV turns out too small for
    // that form's rounding is processed again with every sweep in the expm1
    // form (rare): force_acc is all that crosses the restart
    bool force_acc = false;
    for (int j = 0; j < P.k; ++j) {
      const int64_t r = b * P.k + j;
      const T* srow = static_cast<const T*>(P.s) + r * P.stride;
      const T* trow = static_cast<const T*>(P.t) + r * P.stride;
      const uint64_t g = static_cast<uint64_t>(P.row_offset + r);
      const int z = P.draft[r];
      if (z < 0 || z >= V) {
        if (P.has_pp && B.tid == 0) write_skipped(o, r, z, SAKI_ROW_BAD_DRAFT);
        n = j;
        next_unwritten = j + 1;
        break;
      }
      const RowStats& R = stats_sweep<T, VNT, true, K34>(B, srow, trow, V, mid_lambda(P.eps), false);
      if (!R.finite) {
        if (P.has_pp && B.tid == 0) write_skipped(o, r, z, SAKI_ROW_NONFINITE);
        n = j;
        next_unwritten = j + 1;
        break;
      }
      const float sz = Loader<T>::load1(srow + z), tz = Loader<T>::load1(trow + z);
      const double u = static_cast<double>(philox_uniform(P.seed, ACCEPT, g, 0));
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
        if (R.lam_mid > 0.0f) {
          const double lm = static_cast<double>(R.lam_mid);
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
          const double num = R.kl1_est - P.eps, den = lm * D1 - R.mid_A - P.eps;
          double g_hi = lr1;
          if (num > 1e-2 * (fabs(R.kl1_est) + P.eps) &&
              den > 1e-2 * (fabs(lm * D1) + fabs(R.mid_A) + P.eps)) {
            const double lh = fmax(lm, lm * num / den * (1.0 + 1e-3) + 1e-6);
            if (lh < 1.0) g_hi = lh * xz - (R.mid_A + (A1 - R.mid_A) * (lh - lm) / (1.0 - lm));
          }
          const double lo_side = fmin(0.0, gm), hi_side = fmin(gm, g_hi);
          const double gb = (klm < P.eps * (1.0 - 1e-3)) ? hi_side : (klm > P.eps * (1.0 + 1e-3)) ? lo_side
                                                                     : fmin(lo_side, hi_side);
          gmin = fmax(gmin, gb - 2e-6);
        }
        if (u < exp(gmin)) {
          if (P.has_pp && B.tid == 0) {
            if (o.logp_token) o.logp_token[r] = static_cast<float>(static_cast<double>(sz) - R.lse_s);
            if (o.logt_token) o.logt_token[r] = static_cast<float>(static_cast<double>(tz) - R.lse_t);
            if (o.proposal) o.proposal[r] = z;
            if (o.token) o.token[r] = z;
            if (o.teacher_argmax) o.teacher_argmax[r] = R.vstar;
            if (o.target) o.target[r] = z;
            if (o.corrected) o.corrected[r] = 0;
            if (o.row_status) o.row_status[r] = SAKI_ROW_OK;
          }
          if (P.eos >= 0 && z == P.eos) {
            n = j + 1;
            next_unwritten = j + 1;
            break;
          }
          continue;
        }
      }
      // Positions the interpolating start places well take the fused sweep
      // (the lambda node, and the residual chunk masses where the start
      // predicts a rejection); the others the lambda search and, when
      // rejected or when TV is asked for, the final sweep.  With one
      // workgroup per CU (rollout waves) a position's steps are not hidden
      // behind another workgroup's, and the fused sweep's serial start and
      // settling cost more than the lambda sweep they replace: every position
      // takes the search there.
      const bool end_first = R.kl1_est <= 1.05 * P.eps + 1e-5;
      if (B.wave == 0) {
        bool fu = VNT == 256 && !force_acc && P.eps > 0.0 && R.dmin != R.dmax;
        StartPoint S0;
        S0.lam = 1.0; S0.A = R.lse_t - R.lse_s - static_cast<double>(R.c); S0.herm = true;
        if (fu) {
          if (!end_first) S0 = start_point(R, P.eps);
          const double top = S0.lam * (static_cast<double>(R.dmax) - static_cast<double>(R.c));
          fu = S0.herm && top <= 56.0 && (top - S0.A) * static_cast<double>(LOG2E) <= 56.0;
        }
        if (B.lane == 0) {
          plan.S0 = S0;
          plan.fused = fu ? 1 : 0;
        }
      }
      __syncthreads();
      LamResult L;
      FinalConst F;
      double TV = __builtin_nan("");
      bool settled = false;  // lambda*, the decision, TV (if valid) and the residual chunk from the fused sweep
      bool tv_ok = false;
      bool tv_acc = false;   // the fused sweep's form (the final sweep's is F.acc)
      int res_chunk = nch;
      auto sweep1 = [&](float lam, bool acc) { return lam_sweep<T, VNT>(B, srow, trow, V, R, lam, acc); };
      if (plan.fused != 0) {
        const double xz = (static_cast<double>(LOG2E) * (static_cast<double>(tz) - static_cast<double>(sz)) -
                           static_cast<double>(R.cL)) * LN2_D;
        const bool reject_g = !(u < exp(fmin(0.0, plan.S0.lam * xz - plan.S0.A)));
        FusedConst FC;
        FC.msL = R.ms * LOG2E;
        FC.cL = R.cL;
        FC.lam = static_cast<float>(plan.S0.lam);
        FC.AL = static_cast<float>(plan.S0.A * static_cast<double>(LOG2E));
        FC.gsc = 0.0f;
        FC.set_y();
        const bool facc = (end_first ? R.kl1_est < 1.01 * KL_ACCURATE : P.eps < KL_ACCURATE) || R.pmax > P_PEAKED;
        tv_acc = facc;
        const FusedSums FS = fused_sweep_any<T, float, VNT, false>(B, srow, trow, nullptr, V, FC, facc, reject_g,
                                                                  0.0f, 0.0f, -1, 0.0f);
        if (B.wave == 0) {
          const LamEval E0 = fused_node(R, FS, FC, end_first, facc);
          const LamResult L0 = lambda_search_with(R, P.eps, [](float, bool) { LamEval e{}; return e; }, false, 0.0f,
                                                  &E0, facc, true);
          int state = -1, C0 = 0;
          FinalConst F0{};
          FusedFinal FF0{};
          if (L0.sweeps == 0) {
            F0 = final_const(R, L0, false);
            C0 = !(u < exp(fmin(0.0, L0.log_ratio(sz, tz)))) ? 1 : 0;
            FF0 = fused_tv(R, L0, F0, FC, FS, facc);
            // settled unless the decision or TV needs the final sweep: a
            // rejection needs valid residual masses (kept only where the
            // start predicted it), TV a valid correction
            const bool need_final = (C0 != 0) ? !(FF0.ok && reject_g) : (need_tv && !FF0.ok);
            state = need_final ? 0 : 1;
          }
          if (B.lane == 0) {
            plan.L = L0;
            plan.F = F0;
            plan.FF = FF0;
            plan.state = state;
            plan.C = C0;
          }
        }
        __syncthreads();
        if (plan.state < 0) {
          const LamEval E0 = fused_node(R, FS, FC, end_first, facc);
          L = lambda_search_with(R, P.eps, sweep1, false, 0.0f, &E0, facc);
          F = final_const(R, L, false);
        } else {
          L = plan.L;
          F = plan.F;
          if (plan.state == 1) {
            settled = true;
            tv_ok = plan.FF.ok;
            if (tv_ok) TV = plan.FF.TV;
            if (plan.C != 0) {
              const double hb = expm1(plan.FF.hmax * LN2_D) * 1.02 + 2e-6;
              const double flip = plan.FF.flip;
              res_chunk = chunk_race_certain<VNT>(B, nch, P.seed, RES_CHUNK, g, [&](int c, double& m, double& bb) {
                m = fmax(static_cast<double>(sh.chunk_a[c]), 0.0);
                bb = hb * static_cast<double>(sh.chunk_b[c]) + flip;
              });
              if (res_chunk < 0) {
                settled = false;
                res_chunk = nch;
              }
            }
          }
        }
      } else {
        L = lambda_search<T, VNT>(B, srow, trow, V, R, P.eps, force_acc);
        F = final_const(R, L, force_acc);
      }
      const double alpha = exp(fmin(0.0, L.log_ratio(sz, tz)));
      const bool accept = u < alpha;
      if (!settled && (need_tv || !accept)) {
        TV = final_sweep_any<T, float, VNT, false>(B, srow, trow, nullptr, V, F, !accept, 0.0f, -1, 0.0f);
        tv_ok = true;
        if (!accept) {
          res_chunk = chunk_race<VNT>(B, nch, P.seed, RES_CHUNK, g, [&](int c) {
            const float m = sh.chunk_a[c];
            return m > 0.0f ? log(static_cast<double>(m)) : -__builtin_huge_val();
          });
        }
      }
      if ((need_tv || !accept) && tv_ok && !force_acc && redo_accurate(R, L, settled ? tv_acc : F.acc, TV)) {
        force_acc = true;
        --j;
        continue;
      }
      force_acc = false;
      int y = z;
      float sy = sz, ty = tz;
      if (!accept) {
        const int c1 = res_chunk;
        if (c1 < nch) {
          const ElemFetch<T> fr = elem_fetch<T, VNT>(srow, trow, c1, V, B.tid);
          float sw, tw;
          const int yc = elem_pick<VNT>(B, fr, c1, V, P.seed, RES_ELEM, g, [&](float sv, float tv, int) {
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
      if (P.has_pp && B.tid == 0) {
        const double logp_y = static_cast<double>(sy) - R.lse_s;
        const double logt_y = static_cast<double>(ty) - R.lse_t;
        if (o.lambda) o.lambda[r] = L.lam;
        if (o.kl) o.kl[r] = static_cast<float>(L.KL);
        if (o.tv) o.tv[r] = static_cast<float>(TV);
        if (o.accept_prob) o.accept_prob[r] = static_cast<float>(alpha);
        if (o.margin) o.margin[r] = static_cast<float>(fabs(u - alpha));
        if (o.logp_token) o.logp_token[r] = static_cast<float>(logp_y);
        if (o.logt_token) o.logt_token[r] = static_cast<float>(logt_y);
        if (o.logq_token) o.logq_token[r] = static_cast<float>(logp_y + L.log_ratio(sy, ty));
        if (o.proposal) o.proposal[r] = z;
        if (o.token) o.token[r] = y;
        if (o.teacher_argmax) o.teacher_argmax[r] = R.vstar;
        if (o.target) o.target[r] = accept ? z : R.vstar;
        if (o.corrected) o.corrected[r] = accept ? 0 : 1;
        if (o.row_status) o.row_status[r] = SAKI_ROW_OK;
      }
      if (!accept) {
        n = j;
        corr = y;
        next_unwritten = j + 1;
        break;
      }
      if (P.eos >= 0 && z == P.eos) {
        n = j + 1;
        next_unwritten = j + 1;
        break;
      }
    }
    if (B.tid == 0) {
      P.accepted_len[b] = n;
      P.correction[b] = corr;
      if (P.has_pp) {
        // positions after the end of the block's committed prefix
        for (int jj = next_unwritten; jj < P.k; ++jj) {
          const int64_t r = b * P.k + jj;
          write_skipped(o, r, P.draft[r], SAKI_ROW_SKIPPED);
        }
      }
    }
  }
}

// Launches the verification kernel for one form of the stats sweep; each PART
// (K34) is compiled in its own unit (verify.hip).
template <int PART>
hipError_t launch_verify_part(const VerifyParams& P, int cus, bool bf16, hipStream_t st);

}  // namespace saki
