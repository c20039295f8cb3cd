// Rollout kernels: student draft sampling and the first-rejection commit of a
// speculative wave (SAKI App. I, steps 1, 7 and 8; App. F).  Included by
// saki.hip inside namespace saki, after the verification kernel.
#pragma once

// ---------------------------------------------------------------------------
// Draft sampling, z ~ p = softmax(s), by the two-level exponential race on the
// proposal streams.  One workgroup per row: one read of the row for the chunk
// masses (each wave owns whole chunks; the race compares ln W_c, and a chunk's
// shift is carried in the key), then the entry race inside the winning chunk
// re-reads one chunk.
// ---------------------------------------------------------------------------
struct SampleParams {
  const void* s;
  int64_t n_rows;
  int64_t stride;
  int64_t row_offset;
  int64_t row_step;
  int V;
  uint64_t seed;
  int32_t* token;
  uint8_t* status;
};

// What bounds it: with fewer rows than CUs the row's one CU (one exponential and
// five more VALU instructions an entry, ~7 us for 151,936 entries, and the
// races' serial steps); with more, HBM.  Eight waves per workgroup, each with
// SAMPLE_DEPTH chunks in flight, hide the load latency, and two workgroups per
// CU each other's serial steps.  Sixteen waves were no faster on long rows and
// 1-2 us slower below 32,000 entries.  Rows are not split over CUs: the call
// has no workspace to exchange partial races through.  V = 151,936 bf16, rows
// 16 / 256 / 1,000: 20.5 / 21.6 / 79 us with one chunk ahead, the maximum and
// finiteness of each chunk taken separately and one workgroup per CU, 15.1 /
// 18.5 / 56 us now; V = 32,000, 1,000 rows: 36 -> 22 us.
constexpr int SAMPLE_NT = 512;
constexpr int SAMPLE_WG_PER_CU = 2;
template <typename T>
constexpr int SAMPLE_DEPTH = sizeof(T) == 2 ? 4 : 2;

// Rows whose largest logit is below this take the exponents against the wave's
// maximum times log2 e rounded once: that rounding (a sixteenth of a power of two
// at most here) scales all of a chunk's terms alike and is part of the chunk's
// reference.  For larger logits it grows with them, past 2^127 from a few
// 10^9 on, where a chunk's terms would all become 0 or infinite: those rows take the
// per-chunk form.
constexpr float SAMPLE_MAX_TOP = 0x1p20f;

// The chunk masses of any row: every chunk against its own maximum by
// differences (chunk c keeps that maximum, in natural units, and the sum of
// e^(s - max)), every entry's finiteness taken.  Returns whether all are finite.
template <typename T, int SNT, typename BL>
__device__ __forceinline__ bool sample_masses_any(BL& B, const T* srow, int V) {
  const int nch = (V + CHUNK - 1) / CHUNK;
  bool fin = true;
  for (int c = B.wave; c < nch; c += SNT / WAVE) {
    float x[EPL];
    uint32_t vm;
    load_lane<T, true>(srow, c, B.lane, V, x, &vm);
    float m = -finf();
#pragma unroll
    for (int e = 0; e < EPL; ++e)
      if ((vm >> e) & 1u) {
        m = fmaxf(m, x[e]);
        fin = fin && (x[e] - x[e] == 0.0f);  // false for NaN and +-inf
      }
    const float cm = wave_max(m);
    float acc = 0.0f;
#pragma unroll
    for (int e = 0; e < EPL; ++e)
      if ((vm >> e) & 1u) acc += fexp2((x[e] - cm) * LOG2E);
    const float sum = wave_sum(acc);
    if (B.lane == 0) {
      B.sh.chunk_a[c] = cm;
      B.sh.chunk_b[c] = sum;
    }
  }
  return B.max(fin ? 0.0f : 1.0f) == 0.0f;
}

template <typename T>
__global__ __launch_bounds__(SAMPLE_NT, SAMPLE_WG_PER_CU) void sample_kernel(SampleParams P) {
  constexpr int SNT = SAMPLE_NT, D = SAMPLE_DEPTH<T>;
  __shared__ RowShared<SNT> sh;
  Block<SNT> B(sh);
  constexpr int NW = SNT / WAVE;
  const int V = P.V;
  const int nch = (V + CHUNK - 1) / CHUNK, nfull = V / CHUNK;
  const int nw = B.wave < nfull ? (nfull - 1 - B.wave) / NW + 1 : 0;  // this wave's full chunks
  for (int64_t r = blockIdx.x; r < P.n_rows; r += gridDim.x) {
    const T* srow = static_cast<const T*>(P.s) + r * P.stride;
    const uint64_t g = static_cast<uint64_t>(P.row_offset + r * P.row_step);
    // chunk i of the wave; past its last one the last is read again (unused),
    // so that every load is issued on every path
    auto load = [&](Frag<T>& f, int i) { frag_load<false>(f, srow, B.wave + min(i, nw - 1) * NW, B.lane); };
    Frag<T> f[D];
    if (nw > 0) {
#pragma unroll
      for (int j = 0; j < D; ++j) load(f[j], j);
    }
    // ln E of this thread's chunk, while the first loads are in flight
    double le = 0.0;
    if (B.tid < nch) le = ln_exp_race(P.seed, PROP_CHUNK, g, B.tid);
    // Exponents are relative to the wave's running maximum, as in the stats
    // sweep: chunk c keeps (MsL, sum 2^(s log2 e - MsL)).  A row whose smallest
    // entry is above -inf and whose maxima and sums are finite is finite (a NaN
    // or +inf entry makes a chunk's sum NaN or infinite); any other, and one
    // whose maximum is SAMPLE_MAX_TOP or more in size, goes through
    // sample_masses_any.  MsL stays finite on a wave that has only met entries
    // at the type's lowest value (masks): their sum is then 0.
    float Ms = -finf(), MsL = -finf(), lo = finf();
    bool fin = true;
    auto mass = [&](auto tail, const float* x, uint32_t vm, int c) {
      constexpr bool TAIL = decltype(tail)::value;
      float ls = -finf();
#pragma unroll
      for (int e = 0; e < EPL; e += 2) {
        const bool v0 = !TAIL || ((vm >> e) & 1u), v1 = !TAIL || ((vm >> (e + 1)) & 1u);
        ls = max3_raw(ls, v0 ? x[e] : -finf(), v1 ? x[e + 1] : -finf());
        lo = min3_raw(lo, v0 ? x[e] : finf(), v1 ? x[e + 1] : finf());
      }
      if (wave_any(ls > Ms)) {
        Ms = wave_max(ls);
        MsL = fmaxf(__fmul_rn(Ms, LOG2E), -FLT_MAX);
      }
      float acc = 0.0f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float es = fexp2(fmaf(x[e], LOG2E, -MsL));
        acc += (!TAIL || ((vm >> e) & 1u)) ? es : 0.0f;
      }
      fin = fin && acc < finf();  // false for NaN
      const float sum = wave_sum_last(acc);
      if (B.lane == WAVE - 1) {
        sh.chunk_a[c] = MsL;
        sh.chunk_b[c] = sum;
      }
    };
    auto full = [&](const Frag<T>& fr, int i) {
      float x[EPL];
      frag_unpack(fr, x);
      mass(std::integral_constant<bool, false>(), x, 0xffffu, B.wave + i * NW);
    };
    int i = 0;
    for (; i + D <= nw; i += D) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const Frag<T> cur = f[j];
        load(f[j], i + j + D);
        full(cur, i + j);
      }
    }
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
      if (i + j < nw) full(f[j], i + j);
    if ((V % CHUNK) != 0 && (nfull % NW) == B.wave) {
      float x[EPL];
      uint32_t vm;
      load_lane<T, true>(srow, nfull, B.lane, V, x, &vm);
      mass(std::integral_constant<bool, true>(), x, vm, nfull);
    }
    fin = fin && lo > -finf();
    // the block max is also the barrier that publishes the chunk masses
    const float top = B.max(fin ? Ms : finf());
    double unit = LN2_D;  // of the chunks' references
    bool finite = true;
    if (uniform(!(fabsf(top) < SAMPLE_MAX_TOP))) {
      unit = 1.0;
      finite = uniform(sample_masses_any<T, SNT>(B, srow, V));
    }
    int z = -1;
    if (finite) {
      double best = __builtin_huge_val();
      int bi = 0x7fffffff;
      for (int c = B.tid; c < nch; c += SNT) {
        const double e = c == B.tid ? le : ln_exp_race(P.seed, PROP_CHUNK, g, c);
        const double key = e - (static_cast<double>(sh.chunk_a[c]) * unit + log(static_cast<double>(sh.chunk_b[c])));
        if (key < best) { best = key; bi = c; }
      }
      B.argmin(best, bi);
      z = elem_race<SNT>(B, bi < nch ? bi : 0, V, P.seed, PROP_ELEM, g,
                         [&](int v) { return Loader<T>::load1(srow + v); });
      if (z >= V) z = -1;  // unreachable for finite rows: every chunk has a winner
    }
    if (B.tid == 0) {
      P.token[r] = z;
      if (P.status) P.status[r] = finite ? SAKI_ROW_OK : SAKI_ROW_NONFINITE;
    }
  }
}

// ---------------------------------------------------------------------------
// Commit of one speculative wave: for each running sequence, append the
// accepted drafts and the correction (the per-position token of the
// verification) to its trajectory, with the per-position metadata in token
// order, cut at max_len; update length and done.  One thread per sequence:
// the work is a few stores per committed token.
// ---------------------------------------------------------------------------
struct CommitParams {
  saki_traj tr;
  int k;
  int eos;
  const int32_t* accepted_len;
  const int32_t* correction;
  saki_couple_out pp;
  int32_t* n_commit;
};

__global__ __launch_bounds__(256) void commit_kernel(CommitParams P) {
  const int64_t b = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (b >= P.tr.n_seq) return;
  const saki_traj& T = P.tr;
  int32_t m = 0;
  const int32_t len = T.length[b];
  if (T.done[b] == SAKI_SEQ_RUNNING) {
    if (len < 0 || len > T.max_len) {
      T.done[b] = SAKI_SEQ_STOPPED;
    } else {
      int32_t n = P.accepted_len[b];
      n = n < 0 ? 0 : (n > P.k ? P.k : n);
      const int32_t want = n + ((n < P.k && P.correction[b] >= 0) ? 1 : 0);
      const int64_t room = T.max_len - len;
      m = static_cast<int32_t>(want < room ? want : room);
      int32_t last = -1;
      for (int32_t j = 0; j < m; ++j) {
        const int64_t r = b * P.k + j;
        const int64_t o = b * T.max_len + len + j;
        const int32_t y = P.pp.token[r];
        T.tokens[o] = y;
        if (T.corrected) T.corrected[o] = (j == n) ? 1 : 0;
        if (T.lambda) T.lambda[o] = P.pp.lambda ? P.pp.lambda[r] : nanf_();
        if (T.kl) T.kl[o] = P.pp.kl ? P.pp.kl[r] : nanf_();
        if (T.tv) T.tv[o] = P.pp.tv ? P.pp.tv[r] : nanf_();
        if (T.logp_token) T.logp_token[o] = P.pp.logp_token ? P.pp.logp_token[r] : nanf_();
        if (T.logt_token) T.logt_token[o] = P.pp.logt_token ? P.pp.logt_token[r] : nanf_();
        if (T.teacher_argmax) T.teacher_argmax[o] = P.pp.teacher_argmax ? P.pp.teacher_argmax[r] : -1;
        last = y;
      }
      T.length[b] = len + m;
      if (m == 0)
        T.done[b] = SAKI_SEQ_STOPPED;
      else if (len + m >= T.max_len || (P.eos >= 0 && last == P.eos))
        T.done[b] = SAKI_SEQ_FINISHED;
    }
  }
  if (P.n_commit) P.n_commit[b] = m;
}
