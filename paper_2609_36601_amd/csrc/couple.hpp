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
  unsigned int* next_row;  // work counter in the caller's workspace, zero at launch
  // Rows resolved in the plain forms whose TV turns out too small for their
  // rounding are listed (redo_list, redo_count, in the workspace) and processed
  // again by a second launch with every sweep in the expm1 form (redo_pass).
  unsigned int* redo_list;
  unsigned int* redo_count;
  int redo_pass;
};

// K34: the stats sweep sums k3, k4 (radii below K34_EPS).
template <typename T, typename G, bool ROUTE, bool GRAD, int KC, bool K34>
__global__ __launch_bounds__(NT, WG_PER_CU) void couple_kernel(CoupleParams P) {
  __shared__ RowSharedK<KC> sh;
  __shared__ RowPlan plan;
  Block<NT, RowSharedK<KC>> B(sh);
  const int V = P.V;
  const int nch = (V + CHUNK - 1) / CHUNK;
  // Workgroups take rows from a counter: their speeds differ (the two
  // workgroups of a CU, and CUs, get unequal shares of the memory system), so
  // a fixed stride left the slowest ones finishing ~15% after the median.
  // Each iteration takes a new row or ends the loop: at most n_rows + 1.
  __shared__ unsigned int next_r;
  // the second launch takes its rows from the list the first one made
  const unsigned int n_work = P.redo_pass
      ? static_cast<unsigned int>(__builtin_amdgcn_readfirstlane(static_cast<int>(*P.redo_count)))
      : static_cast<unsigned int>(P.n_rows);
  const bool force_acc = P.redo_pass != 0;
  for (int64_t it = 0; it <= P.n_rows; ++it) {
    const unsigned int ru = take_next(P.next_row, &next_r);
    // unsigned: n_rows < 2^31 and the counter stays below n_rows + grid
    if (ru >= n_work) break;
    const int64_t r = static_cast<int64_t>(P.redo_pass ? P.redo_list[ru] : ru);
    const T* srow = static_cast<const T*>(P.s) + r * P.stride;
    const T* trow = static_cast<const T*>(P.t) + r * P.stride;
    G* grow = GRAD ? static_cast<G*>(P.grad) + r * P.grad_stride : nullptr;
    const uint64_t g = static_cast<uint64_t>(P.row_offset + r);
    const float M = (ROUTE && P.valid) ? (P.valid[r] ? 1.0f : 0.0f) : 1.0f;

    const bool sample_target = ROUTE && P.target_mode == SAKI_TARGET_SAMPLE;
    const RowStats& R = stats_sweep<T, NT, true, K34>(B, srow, trow, V, mid_lambda(P.eps), true, sample_target);
    if (!R.finite) {
      if (GRAD) fill_row<G, NT>(B.wave, B.lane, grow, V, M != 0.0f ? nanf_() : 0.0f);
      if (B.tid == 0) {
        const saki_couple_out& o = P.out;
        if (o.lambda) o.lambda[r] = nanf_();
        if (o.kl) o.kl[r] = nanf_();
        if (o.tv) o.tv[r] = nanf_();
        if (o.accept_prob) o.accept_prob[r] = nanf_();
        if (o.margin) o.margin[r] = nanf_();
        if (o.logp_token) o.logp_token[r] = nanf_();
        if (o.logt_token) o.logt_token[r] = nanf_();
        if (o.logq_token) o.logq_token[r] = nanf_();
        if (o.proposal) o.proposal[r] = -1;
        if (o.token) o.token[r] = -1;
        if (o.teacher_argmax) o.teacher_argmax[r] = -1;
        if (o.target) o.target[r] = -1;
        if (o.corrected) o.corrected[r] = 0;
        if (o.row_status) o.row_status[r] = SAKI_ROW_NONFINITE;
        if (ROUTE) {
          const float l = (M != 0.0f) ? nanf_() : 0.0f;
          if (P.row_loss) P.row_loss[r] = l;
          if (P.scaled_loss) P.scaled_loss[r] = static_cast<double>(l);
        }
      }
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
    // start point while wave 1 draws the proposal z ~ p (the two-level race on
    // the stats sweep's chunk masses, then the entry race in the winning
    // chunk), which leaves the other waves' issue slots to the other
    // workgroup of the CU; the results go through LDS (plan).
    const bool end_first = R.kl1_est <= 1.05 * P.eps + 1e-5;
    if (B.wave == 0) {
      bool fu = !force_acc && P.eps > 0.0 && R.dmin != R.dmax;
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
    } else if (B.wave == 1) {
      float ws, wt;
      const int zz = wave_proposal<T>(srow, trow, nch, V, B.lane, P.seed, PROP_CHUNK, PROP_ELEM, g,
                                      [&](int c) {
                                        return static_cast<double>(sh.chunk_a[c]) * LN2_D +
                                               log(static_cast<double>(sh.chunk_b[c]));
                                      },
                                      [](float sv, float, int) { return sv; }, &ws, &wt);
      if (B.lane == 0) {
        plan.z = zz;
        plan.sz = ws;
        plan.tz = wt;
      }
    }
    __syncthreads();
    const bool fused = plan.fused != 0;

    float sz = plan.sz, tz = plan.tz;
    int z = plan.z;
    if (z >= V) {  // unreachable for finite rows: every chunk has a winner
      z = R.vstar;
      sz = s_vstar;
      tz = Loader<T>::load1(trow + z);
    }
    const double u = static_cast<double>(philox_uniform(P.seed, ACCEPT, g, 0));
    const double logp_z = static_cast<double>(sz) - R.lse_s;
    const double logt_z = static_cast<double>(tz) - R.lse_t;
    const double adv = logt_z - logp_z;
    auto coef_of = [&](bool corr) {
      return ROUTE ? static_cast<float>(static_cast<double>(P.grad_scale) * M * (corr ? 1.0 : adv)) : 0.0f;
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
      const int ct = chunk_race<NT>(B, nch, P.seed, TS_CHUNK, g, [&](int c) {
        return static_cast<double>(sh.chunk_c[c]) * LN2_D + log(static_cast<double>(sh.chunk_d[c]));
      });
      const int cc = ct < nch ? ct : 0;
      const ElemFetch<T> ft = elem_fetch<T, NT>(srow, trow, cc, V, B.tid);
      float sv, tv;
      const int vt = elem_pick<NT>(B, ft, cc, V, P.seed, TS_ELEM, g,
                                   [&](float, float tl, int) { return tl; }, &sv, &tv);
      if (vt < V) {
        hot_c = vt;
        s_hot_c = sv;
      }
    };
    auto sweep1 = [&](float lam, bool acc) { return lam_sweep<T, NT>(B, srow, trow, V, R, lam, acc); };

    LamResult L;
    FinalConst F;
    bool C;
    double TV = 0.0;
    bool tv_acc = false;   // the fused sweep's form (the final sweep's is F.acc)
    bool settled = false;  // TV, the residual chunk and the gradient row come from the fused sweep
    int res_chunk = nch;
    if (fused) {
      // accept decision at the start point: it sets the gradient the fused
      // sweep writes, and must agree with the one at lambda*
      const double xz = (static_cast<double>(LOG2E) * (static_cast<double>(tz) - static_cast<double>(sz)) -
                         static_cast<double>(R.cL)) * LN2_D;
      const bool Cg = !(u < exp(fmin(0.0, plan.S0.lam * xz - plan.S0.A)));
      if (Cg) correction_target();
      const float coef_g = coef_of(Cg);
      FusedConst FC;
      FC.msL = R.ms * LOG2E;
      FC.cL = R.cL;
      FC.lam = static_cast<float>(plan.S0.lam);
      FC.AL = static_cast<float>(plan.S0.A * static_cast<double>(LOG2E));
      const float invS = static_cast<float>(shift_correction(R.ms, FC.msL) / R.sum_s);
      FC.gsc = coef_g * invS;
      FC.set_y();
      // the expm1 form where the lambda sweep would take it (KL below
      // KL_ACCURATE: the radius, or KL(pi || p) at the teacher end) and on
      // peaked rows, whose TV the plain form would often leave too imprecise;
      // elsewhere a row whose TV turns out too small for the plain form is
      // listed for the accurate second launch (redo_accurate)
      const bool facc = (end_first ? R.kl1_est < 1.01 * KL_ACCURATE : P.eps < KL_ACCURATE) || R.pmax > P_PEAKED;
      tv_acc = facc;
      const FusedSums FS = fused_sweep_any<T, G, NT, GRAD>(B, srow, trow, grow, V, FC, facc, Cg, coef_g, invS,
                                                          Cg ? hot_c : z, Cg ? s_hot_c : sz);
      // wave 0: lambda* from the node's model when it needs no sweep, the
      // accept decision there and TV from the fused sums
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
          state = (FF0.ok && (C0 != 0) == Cg) ? 1 : 0;
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
        // the node's model did not settle lambda*: the search goes on with
        // lambda sweeps from that node
        const LamEval E0 = fused_node(R, FS, FC, end_first, facc);
        L = lambda_search_with(R, P.eps, sweep1, false, 0.0f, &E0, facc);
        F = final_const(R, L, false);
        C = !(u < exp(fmin(0.0, L.log_ratio(sz, tz))));
      } else {
        L = plan.L;
        F = plan.F;
        C = plan.C != 0;
        if (plan.state == 1) {
          TV = plan.FF.TV;
          settled = true;
          if (C) {
            // the residual chunk from the masses at the node, each within
            // (2^hmax - 1) of its positive mass plus the sign-change bound
            const double hb = expm1(plan.FF.hmax * LN2_D) * 1.02 + 2e-6;
            const double flip = plan.FF.flip;
            res_chunk = chunk_race_certain<NT>(B, nch, P.seed, RES_CHUNK, g, [&](int c, double& m, double& b) {
              m = fmax(static_cast<double>(sh.chunk_a[c]), 0.0);
              b = hb * static_cast<double>(sh.chunk_b[c]) + flip;
            });
            if (res_chunk < 0) {
              settled = false;
              res_chunk = nch;
            }
          }
        }
      }
    } else {
      L = lambda_search<T, NT>(B, srow, trow, V, R, P.eps, force_acc);
      F = final_const(R, L, force_acc);
      C = !(u < exp(fmin(0.0, L.log_ratio(sz, tz))));
    }

    // accept test, Eq. accept in the log form exp(min(0, log q(z) - log p(z)))
    const double alpha = exp(fmin(0.0, L.log_ratio(sz, tz)));
    if (C) correction_target();
    const float coef = coef_of(C);
    const int hot = C ? hot_c : z;
    const float s_hot = C ? s_hot_c : sz;

    if (!settled) {
      TV = final_sweep_any<T, G, NT, GRAD>(B, srow, trow, grow, V, F, C, coef, hot, s_hot);
      if (C) {
        res_chunk = chunk_race<NT>(B, nch, P.seed, RES_CHUNK, g, [&](int c) {
          const float m = sh.chunk_a[c];
          return m > 0.0f ? log(static_cast<double>(m)) : -__builtin_huge_val();
        });
      }
    }
    if (!force_acc && redo_accurate(R, L, settled ? tv_acc : F.acc, TV)) {
      // listed for the second launch, which rewrites the row's gradient and
      // writes its outputs
      if (B.tid == 0) P.redo_list[atomicAdd(P.redo_count, 1u)] = static_cast<unsigned int>(r);
      continue;
    }

    int y = z;
    float sy = sz, ty = tz;
    if (C) {
      // a residual that rounds to zero everywhere in float (lambda* x within
      // rounding of A*) leaves no chunk with mass; the proposal is kept then
      const int c1 = res_chunk;
      if (c1 < nch) {
        const ElemFetch<T> fr = elem_fetch<T, NT>(srow, trow, c1, V, B.tid);
        float sw, tw;
        const int yc = elem_pick<NT>(B, fr, c1, V, P.seed, RES_ELEM, g, [&](float sv, float tv, int) {
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
      const saki_couple_out& o = P.out;
      if (o.lambda) o.lambda[r] = L.lam;
      if (o.kl) o.kl[r] = static_cast<float>(L.KL);
      if (o.tv) o.tv[r] = static_cast<float>(TV);
      if (o.accept_prob) o.accept_prob[r] = static_cast<float>(alpha);
      if (o.margin) o.margin[r] = static_cast<float>(fabs(u - alpha));
      if (o.logp_token) o.logp_token[r] = static_cast<float>(logp_y);
      if (o.logt_token) o.logt_token[r] = static_cast<float>(logt_y);
      if (o.logq_token) o.logq_token[r] = static_cast<float>(logq_y);
      if (o.proposal) o.proposal[r] = z;
      if (o.token) o.token[r] = y;
      if (o.teacher_argmax) o.teacher_argmax[r] = R.vstar;
      if (o.target) o.target[r] = hot;
      if (o.corrected) o.corrected[r] = C ? 1 : 0;
      if (o.row_status) o.row_status[r] = SAKI_ROW_OK;
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
        if (P.row_loss) P.row_loss[r] = static_cast<float>(l);
        if (P.scaled_loss) P.scaled_loss[r] = static_cast<double>(P.grad_scale) * l;
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
