// The coupling kernel (with the routed loss and gradient fused into it).
#pragma once

#include "common.hpp"

namespace saki {

struct CoupleParams {
  const void* s;
  const void* t;
  int64_t n_rows;
  int64_t stride;
  int64_t row_offset;
  int V;
  double eps;
  float lam_mid;  // mid_lambda(eps)
  uint64_t seed;
  saki_couple_out out;
  // routing
  const uint8_t* valid;
  float grad_scale;
  float* row_loss;
  double* scaled_loss;  // workspace [n_rows] or NULL
  void* grad;
  int64_t grad_stride;
  int target_mode;      // SAKI_TARGET_MODE or SAKI_TARGET_SAMPLE
  unsigned int* next_row;  // work counter in the caller's workspace, zero at launch; NULL: one row per workgroup
};

// K34: the stats sweep sums k3, k4 (radii below K34_EPS).
template <typename T, typename G, bool ROUTE, bool GRAD, int KC, bool K34>
__global__ __launch_bounds__(NT, WG_PER_CU) void couple_kernel(CoupleParams) {
  using SH = RowSharedK<KC>;
  __shared__ SH sh;
  __shared__ RowPlan plan;
  Block<NT, SH> B(sh);
  const auto* P = kernel_args<CoupleParams>();
  const int V = P->V;
  const int nch = (V + CHUNK - 1) / CHUNK;
  // Workgroups take rows from a counter: their speeds differ (the two
  // workgroups of a CU, and CUs, get unequal shares of the memory system), so
  // a fixed stride left the slowest ones finishing ~15% after the median.
  // Workgroup b starts with row b.  Far from the end of the launch a lane of an
  // idle wave takes the next index while wave 0 combines a row's sums, and
  // posts it in LDS, so that a wave that is done with a row goes on to the next
  // one without a barrier (the next row's first LDS writes are the chunk
  // masses, read last before the barriers of the races, and each wave's own
  // cache and reduction slots; plan and rs are written behind its first
  // barrier).  The last two rows per workgroup are taken when it is free for
  // them: a row taken ahead waits for the current one, and the launch ends
  // later for it (4,096 long-rollout rows, eight per workgroup: +3%).
  // readfirstlane makes the index, and so the loop's exit, uniform in every
  // wave: all threads reach the same barriers.  The indices only grow, so
  // every workgroup ends.
  unsigned int ru = blockIdx.x;
  bool taken = true;
  // a row resolved in a plain form whose TV turns out too small for that
  // form's rounding is processed again with every sweep in the expm1 form (rare)
  bool force_acc = false;
  // unsigned: n_rows < 2^31 and the counter stays below n_rows + grid
  const unsigned int n_rows = static_cast<unsigned int>(P->n_rows);
  for (;;) {
    P = kernel_args<CoupleParams>();
    if (!taken) {
      if (B.tid == 0) sh.next = gridDim.x + take_index(P->next_row);
      __syncthreads();
      ru = static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(sh.next)));
    }
    if (ru >= n_rows) break;
    const bool ahead = P->next_row == nullptr || ru + 2 * gridDim.x < n_rows;
    const bool take_now = ahead && !force_acc;
    taken = ahead;
    const int64_t r = static_cast<int64_t>(ru);
    const T* srow = static_cast<const T*>(P->s) + r * P->stride;
    const T* trow = static_cast<const T*>(P->t) + r * P->stride;
    G* grow = GRAD ? static_cast<G*>(P->grad) + r * P->grad_stride : nullptr;
    const uint64_t g = static_cast<uint64_t>(P->row_offset + r);
    const float M = (ROUTE && P->valid) ? (P->valid[r] ? 1.0f : 0.0f) : 1.0f;

    const bool sample_target = ROUTE && P->target_mode == SAKI_TARGET_SAMPLE;
    // while wave 0 combines the sums: the proposal's chunk race on the other
    // waves, the accept uniform and the next index on a lane of the last one
    auto idle = [&]() {
      constexpr int NW = SH::NW;
      const bool last = B.tid == NT - WAVE;
      const bool take = last && take_now;
      unsigned int nx = n_rows;
      if (take && P->next_row) nx = gridDim.x + take_index(P->next_row);
      double key;
      int idx;
      wave_chunk_race(nch, (B.wave - 1) * WAVE + B.lane, (NW - 1) * WAVE, P->seed, PROP_CHUNK, g, [&](int c) {
        return static_cast<double>(sh.chunk_a[c]) * LN2_D + log(static_cast<double>(sh.chunk_b[c]));
      }, &key, &idx);
      if (B.lane == 0) {
        sh.race_key[B.wave] = key;
        sh.race_idx[B.wave] = idx;
      }
      if (last) {
        if (take) sh.next = nx;
        sh.u = philox_uniform(P->seed, ACCEPT, g, 0);
      }
    };
    const RowStats& R = stats_sweep<T, NT, K34>(B, srow, trow, V, P->lam_mid, true, sample_target, idle);
    if (ahead) ru = static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(sh.next)));
    P = kernel_args<CoupleParams>();
    if (uniform(!R.finite)) {
      if (GRAD) fill_row<G, NT>(B.wave, B.lane, grow, V, M != 0.0f ? nanf_() : 0.0f);
      if (B.tid == 0) {
        const auto* Q = kernel_args<CoupleParams>();
        if (Q->out.lambda) Q->out.lambda[r] = nanf_();
        if (Q->out.kl) Q->out.kl[r] = nanf_();
        if (Q->out.tv) Q->out.tv[r] = nanf_();
        if (Q->out.accept_prob) Q->out.accept_prob[r] = nanf_();
        if (Q->out.margin) Q->out.margin[r] = nanf_();
        if (Q->out.logp_token) Q->out.logp_token[r] = nanf_();
        if (Q->out.logt_token) Q->out.logt_token[r] = nanf_();
        if (Q->out.logq_token) Q->out.logq_token[r] = nanf_();
        if (Q->out.proposal) Q->out.proposal[r] = -1;
        if (Q->out.token) Q->out.token[r] = -1;
        if (Q->out.teacher_argmax) Q->out.teacher_argmax[r] = -1;
        if (Q->out.target) Q->out.target[r] = -1;
        if (Q->out.corrected) Q->out.corrected[r] = 0;
        if (Q->out.row_status) Q->out.row_status[r] = SAKI_ROW_NONFINITE;
        if (ROUTE) {
          const float l = (M != 0.0f) ? nanf_() : 0.0f;
          if (Q->row_loss) Q->row_loss[r] = l;
          if (Q->scaled_loss) Q->scaled_loss[r] = static_cast<double>(l);
        }
      }
      force_acc = false;
      continue;
    }

    // The logit of the teacher mode (the loss and gradient at a correction) is
    // loaded early.
    const float s_vstar = Loader<T>::load1(srow + R.vstar);

    // Rows the interpolating start places well take the fused sweep (the
    // lambda node and a speculative final sweep in one pass), and so do rows
    // whose teacher end may be feasible (the node lambda = 1, where A is known
    // exactly); the others, and fused rows whose checks fail, the lambda
    // search and the final sweep.
    // The serial steps between sweeps run on one wave at a time: wave 0 the
    // start point while wave 1 draws the proposal z ~ p in the chunk that won
    // the chunk race, which leaves the other waves' issue slots to the other
    // workgroup of the CU; the results go through LDS (plan).
    const bool end_first = R.kl1_est <= 1.05 * P->eps + 1e-5;
    if (B.wave == 0) {
      bool fu = !force_acc && P->eps > 0.0 && R.dmin != R.dmax;
      StartPoint S0;
      S0.lam = 1.0; S0.A = R.lse_t - R.lse_s - static_cast<double>(R.c); S0.herm = true;
      if (fu) {
        if (!end_first) S0 = start_point(R, P->eps);
        const double top = S0.lam * (static_cast<double>(R.dmax) - static_cast<double>(R.c));
        fu = S0.herm && top <= 56.0 && (top - S0.A) * static_cast<double>(LOG2E) <= 56.0;
      }
      if (B.lane == 0) {
        plan.S0 = S0;
        plan.fused = fu ? 1 : 0;
      }
    } else if (B.wave == 1) {
      float ws, wt;
      const int pc = race_winner(sh);
      const int zz = wave_elem_race<T>(srow, trow, pc < nch ? pc : 0, V, B.lane, P->seed, PROP_ELEM, g,
                                       [](float sv, float, int) { return sv; }, &ws, &wt);
      if (B.lane == 0) {
        plan.z = zz;
        plan.sz = ws;
        plan.tz = wt;
      }
    }
    __syncthreads();
    const bool fused = uniform(plan.fused != 0);

    float sz = plan.sz, tz = plan.tz;
    int z = plan.z;
    if (z >= V) {  // unreachable for finite rows: every chunk has a winner
      z = R.vstar;
      sz = s_vstar;
      tz = Loader<T>::load1(trow + z);
    }
    const double u = static_cast<double>(sh.u);
    const double logp_z = static_cast<double>(sz) - R.lse_s;
    const double logt_z = static_cast<double>(tz) - R.lse_t;
    const double adv = logt_z - logp_z;
    auto coef_of = [&](bool corr) {
      return ROUTE ? static_cast<float>(static_cast<double>(P->grad_scale) * M * (corr ? 1.0 : adv)) : 0.0f;
    };
    // the gradient's indicator at a correction: the teacher mode, or a draw
    // from pi by the same two-level race on its own streams (teacher chunk
    // masses from the stats sweep); it does not depend on lambda
    int hot_c = R.vstar;
    float s_hot_c = s_vstar;
    bool have_hot_c = !sample_target;
    auto correction_target = [&]() {
      if (have_hot_c) return;
      have_hot_c = true;
      const int ct = chunk_race<NT>(B, nch, P->seed, TS_CHUNK, g, [&](int c) {
        return static_cast<double>(sh.chunk_c[c]) * LN2_D + log(static_cast<double>(sh.chunk_d[c]));
      });
      const int cc = ct < nch ? ct : 0;
      const ElemFetch<T> ft = elem_fetch<T, NT>(srow, trow, cc, V, B.tid);
      float sv, tv;
      const int vt = elem_pick<NT>(B, ft, cc, V, P->seed, TS_ELEM, g,
                                   [&](float, float tl, int) { return tl; }, &sv, &tv);
      if (vt < V) {
        hot_c = vt;
        s_hot_c = sv;
      }
    };

    LamResult L;
    FinalConst F;
    bool C = false;
    bool search = true;    // lambda* by lambda sweeps
    double TV = 0.0, alpha = 0.0;
    bool tv_acc = false;   // the fused sweep's form (the final sweep's is F.acc)
    bool settled = false;  // TV, the residual chunk and the gradient row come from the fused sweep
    bool redo = false;     // the row again in the expm1 forms
    int res_chunk = nch;
    if (fused) {
      // accept decision at the start point: it sets the gradient the fused
      // sweep writes, and must agree with the one at lambda*
      // (in float: a decision within its rounding of a tie may differ from the
      // one at lambda*, and then takes the final sweep)
      const float lam_g = static_cast<float>(plan.S0.lam);
      const float A_g = static_cast<float>(plan.S0.A * static_cast<double>(LOG2E));
      const bool Cg = uniform(!(sh.u < fexp2(fminf(0.0f, fmaf(lam_g, fmaf(tz - sz, LOG2E, -R.cL), -A_g)))));
      if (Cg) correction_target();
      const float coef_g = coef_of(Cg);
      FusedConst FC;
      FC.msL = R.ms * LOG2E;
      FC.cL = R.cL;
      FC.lam = lam_g;
      FC.AL = A_g;
      const float invS = static_cast<float>(R.shift * R.inv_s);
      FC.gsc = coef_g * invS;
      FC.set_y();
      // the expm1 form where the lambda sweep would take it (KL below
      // KL_ACCURATE: the radius, or KL(pi || p) at the teacher end) and on
      // peaked rows, whose TV the plain form would often leave too imprecise;
      // elsewhere a row whose TV turns out too small for the plain form is
      // processed again in the accurate forms (redo_accurate)
      const bool facc = (end_first ? R.kl1_est < 1.01 * KL_ACCURATE : P->eps < KL_ACCURATE) || R.pmax > P_PEAKED;
      tv_acc = facc;
      FusedSums FS = fused_sweep_any<T, G, NT, GRAD>(B, srow, trow, grow, V, FC, facc, Cg, coef_g, invS,
                                                          Cg ? hot_c : z, Cg ? s_hot_c : sz);
      // wave 0: lambda* from the node's model when it needs no sweep, the
      // accept decision there and TV from the fused sums; the other waves run
      // the residual's chunk race meanwhile where a correction is predicted
      double le0 = 0.0;
      if (B.wave == 0) {
        FC.set_node();
        const LamEval E0 = fused_node(R, FS, FC, end_first, facc);
        const LamResult L0 = lambda_search_with(R, P->eps, [](float, bool) { LamEval e{}; return e; },
                                                [] { return true; }, false, 0.0f, true, E0, facc);
        int state = -1, C0 = 0, redo = 0;
        double alpha0 = 0.0;
        FinalConst F0{};
        FusedFinal FF0{};
        if (L0.sweeps == 0) {
          F0 = final_const(R, L0, false);
          alpha0 = exp(fmin(0.0, L0.log_ratio(sz, tz)));
          C0 = !(u < alpha0) ? 1 : 0;
          FF0 = fused_tv(R, L0, F0, FC, FS, facc);
          state = (FF0.ok && (C0 != 0) == Cg) ? 1 : 0;
          redo = (state == 1 && redo_accurate(R, L0, facc, FF0.TV)) ? 1 : 0;
        }
        if (B.lane == 0) {
          plan.L = L0;
          plan.F = F0;
          plan.FF = FF0;
          plan.E0 = E0;
          plan.alpha = alpha0;
          plan.state = state;
          plan.C = C0;
          plan.redo = redo;
        }
      } else if (Cg) {
        le0 = res_race_begin<NT>(B, nch, P->seed, g);
      }
      __syncthreads();
      const int state = __builtin_amdgcn_readfirstlane(plan.state);
      search = state < 0;
      if (!search) {
        L = plan.L;
        F = plan.F;
        alpha = plan.alpha;
        C = uniform(plan.C != 0);
        if (state == 1) {
          TV = plan.FF.TV;
          settled = true;
          redo = uniform(plan.redo != 0);
          if (C && !redo) {
            // the residual chunk from the masses at the node, each within
            // (2^hmax - 1) of its positive mass plus the sign-change bound
            // (expm1(x) <= x + x^2 for the x <= 0.007 that fused_tv lets through)
            const double hx = plan.FF.hmax * LN2_D;
            const double hb = hx * (1.0 + hx) * 1.02 + 2e-6;
            res_chunk = __builtin_amdgcn_readfirstlane(
                res_race_end<NT>(B, nch, P->seed, g, le0, hb, plan.FF.flip));
            if (res_chunk < 0) {
              settled = false;
              res_chunk = nch;
            }
          }
        }
      }
    }
    if (search) {
      // lambda sweeps: from the fused sweep's node where its model did not
      // settle lambda*, else from the start
      const LamEval E0 = fused ? plan.E0 : LamEval{};
      L = lambda_search_with(R, P->eps, [&](float lam, bool acc) {
        return lam_sweep<T, NT>(B, srow, trow, V, R, lam, acc);
      }, [] { return false; }, force_acc, 0.0f, fused, E0, tv_acc);
      F = final_const(R, L, force_acc);
      alpha = exp(fmin(0.0, L.log_ratio(sz, tz)));
      C = uniform(!(u < alpha));
    }

    // alpha: accept test, Eq. accept in the log form exp(min(0, log q(z) - log p(z)))
    if (C && !redo) correction_target();
    const float coef = coef_of(C);
    const int hot = C ? hot_c : z;
    const float s_hot = C ? s_hot_c : sz;

    if (!settled) {
      TV = final_sweep_any<T, G, NT, GRAD>(B, srow, trow, grow, V, F, C, coef, hot, s_hot);
      if (C) {
        res_chunk = chunk_race<NT>(B, nch, P->seed, RES_CHUNK, g, [&](int c) {
          const float m = sh.chunk_a[c];
          return m > 0.0f ? log(static_cast<double>(m)) : -__builtin_huge_val();
        });
      }
    }
    if (!settled && !force_acc) redo = uniform(redo_accurate(R, L, F.acc, TV));
    if (redo) {
      // the same row again: its gradient is rewritten, its outputs written then
      force_acc = true;
      ru = static_cast<unsigned int>(r);
      taken = true;
      continue;
    }
    force_acc = false;

    int y = z;
    float sy = sz, ty = tz;
    if (C) {
      // a residual that rounds to zero everywhere in float (lambda* x within
      // rounding of A*) leaves no chunk with mass; the proposal is kept then
      const int c1 = res_chunk;
      if (c1 < nch) {
        const ElemFetch<T> fr = elem_fetch<T, NT>(srow, trow, c1, V, B.tid);
        float sw, tw;
        const int yc = elem_pick<NT>(B, fr, c1, V, P->seed, RES_ELEM, g, [&](float sv, float tv, int) {
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

    if (B.tid == 0) {
      const double logp_y = static_cast<double>(sy) - R.lse_s;
      const double logt_y = static_cast<double>(ty) - R.lse_t;
      const double logq_y = logp_y + L.log_ratio(sy, ty);
      const auto* Q = kernel_args<CoupleParams>();
      if (Q->out.lambda) Q->out.lambda[r] = L.lam;
      if (Q->out.kl) Q->out.kl[r] = static_cast<float>(L.KL);
      if (Q->out.tv) Q->out.tv[r] = static_cast<float>(TV);
      if (Q->out.accept_prob) Q->out.accept_prob[r] = static_cast<float>(alpha);
      if (Q->out.margin) Q->out.margin[r] = static_cast<float>(fabs(u - alpha));
      if (Q->out.logp_token) Q->out.logp_token[r] = static_cast<float>(logp_y);
      if (Q->out.logt_token) Q->out.logt_token[r] = static_cast<float>(logt_y);
      if (Q->out.logq_token) Q->out.logq_token[r] = static_cast<float>(logq_y);
      if (Q->out.proposal) Q->out.proposal[r] = z;
      if (Q->out.token) Q->out.token[r] = y;
      if (Q->out.teacher_argmax) Q->out.teacher_argmax[r] = R.vstar;
      if (Q->out.target) Q->out.target[r] = hot;
      if (Q->out.corrected) Q->out.corrected[r] = C ? 1 : 0;
      if (Q->out.row_status) Q->out.row_status[r] = SAKI_ROW_OK;
      if (ROUTE) {
        double l = 0.0;
        if (M != 0.0f) {
          if (C) {
            const double logp_v = static_cast<double>(s_hot) - R.lse_s;
            l = -logp_v;
          } else {
            l = -adv * logp_z;
          }
        }
        if (Q->row_loss) Q->row_loss[r] = static_cast<float>(l);
        if (Q->scaled_loss) Q->scaled_loss[r] = static_cast<double>(Q->grad_scale) * l;
      }
    }
  }
}

// Launches the coupling kernel for one logit type and one form of the stats
// sweep; each PART (bit 0: K34, bit 1: f32 logits) is compiled in its own unit
// (couple.hip), so that the build runs them in parallel.
template <int PART>
hipError_t launch_couple_part(const CoupleParams& P, bool route, bool grad, bool grad_bf16, int grid, hipStream_t st);

}  // namespace saki
