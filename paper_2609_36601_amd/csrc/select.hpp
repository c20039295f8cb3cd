// Placement controls (Random-TM, TV-Weighted-TM): per trajectory, select
// m = corrections among the valid positions.  Keys in double: ln E with
// E = -ln U (Random-TM, and the uniform fill of TV-Weighted-TM from the
// positions with TV = 0), ln E - ln TV for the positions with TV > 0.  The k
// smallest keys of a tier are found exactly, ties to the lower row.
// Included by saki.hip inside namespace saki.
#pragma once

// What bounds it: latency.  A trajectory's keys (8 B a row) are a few tens of
// KiB, so every pass runs from L2; the Philox block and the two or three
// double logarithms of a key are the only real arithmetic, and the number of
// dependent passes sets the time.  One workgroup per trajectory makes three
// coalesced passes: keys (with their count and range), a histogram over
// SEL_BINS bins linear in the key, and the marking of the rows below the bin
// that holds the k-th smallest key; the bin's own rows (a few) are ranked in
// LDS.  64 trajectories of 2,048 to 4,096 rows: 367 us for the bisection over
// the keys' 64-bit images (64 uncoalesced passes) before, 23.6 us now (one MI355X, same box).
constexpr int SEL_BINS = 2048;
// Rows of the bin that can be ranked in LDS (by counting: SEL_CAP^2 compares).
constexpr int SEL_CAP = 1024;
// Rows per trajectory (on average) from which a trajectory takes a workgroup of
// 1,024 threads; shorter ones leave most of its waves idle in every pass and
// take 256 threads, four workgroups per CU.
constexpr int64_t SEL_WIDE_ROWS = 512;

struct SelectParams {
  int mode;
  int64_t n_traj;
  int64_t n_rows;
  const int64_t* off;
  const float* tv;
  const uint8_t* corrected;
  const uint8_t* valid;
  uint64_t seed;
  int64_t row_offset;
  uint8_t* sel;   // holds each row's tier (0, 1; 2 = not valid) until it is marked
  double* keys;   // workspace [n_rows]
};

template <int SNT>
struct SelShared {
  static constexpr int NW = SNT / WAVE;
  double red_d[NW][RED_MAX];
  float red_f[NW][4];
  int red_i[NW][4];
  unsigned int hist[SEL_BINS];
  unsigned int wave_tot[NW];
  int bin;                 // the bin of the k-th smallest key
  unsigned int before, in_bin;  // rows below that bin, rows in it
  unsigned int n_cand;
  double cand_key[SEL_CAP];
  int64_t cand_row[SEL_CAP];
};

__device__ __forceinline__ uint64_t order_bits(double k) {
  const uint64_t u = __builtin_bit_cast(uint64_t, k);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Bin of a key: non-decreasing in the key (each step rounds monotonically), so
// the k-th smallest key lies in the bin that the cumulative counts give.  NaN
// (an infinite key with scale 0) goes to bin 0, as every key does there.
__device__ __forceinline__ int sel_bin(double key, double base, double scale) {
  const double x = (key - base) * scale;
  return x > 0.0 ? (x < static_cast<double>(SEL_BINS) ? static_cast<int>(x) : SEL_BINS - 1) : 0;
}

// Any set of keys (ties, infinities, more rows in one bin than LDS holds, more
// than 2^31 rows): bisection over the keys' order-preserving 64-bit images for
// the k-th smallest, ties to the lower row by a scan in row order.  The rows of
// `tier` for which in(key) holds are marked SEL_TAKEN or SEL_LEFT; others keep
// their tier.
constexpr uint8_t SEL_TAKEN = 3, SEL_LEFT = 4;
template <int SNT, typename In>
__device__ void select_bisect(Block<SNT, SelShared<SNT>>& B, const SelectParams& P, int64_t lo_r, int64_t hi_r,
                              int tier, double k, In in) {
  auto count = [&](uint64_t x, bool strict) {
    double n = 0;
    for (int64_t r = lo_r + B.tid; r < hi_r; r += SNT) {
      const double key = P.keys[r];
      if (P.sel[r] != tier || !in(key)) continue;
      const uint64_t o = order_bits(key);
      n += strict ? (o < x) : (o <= x);
    }
    double v[1] = {n};
    B.sum(v);
    return v[0];
  };
  uint64_t lo = 0, hi = ~0ull;
  while (lo < hi) {
    const uint64_t mid = lo + (hi - lo) / 2;
    if (count(mid, false) >= k) hi = mid; else lo = mid + 1;
  }
  const uint64_t T = lo;
  double need = k - count(T, true);  // rows with key image T to take, lowest rows first
  for (int64_t r0 = lo_r; r0 < hi_r; r0 += SNT) {
    const int64_t r = r0 + B.tid;
    bool mine = false, eq = false;
    if (r < hi_r) {
      const double key = P.keys[r];
      mine = P.sel[r] == tier && in(key);
      const uint64_t o = order_bits(key);
      eq = mine && o == T;
      if (mine && !eq) P.sel[r] = o < T ? SEL_TAKEN : SEL_LEFT;
    }
    const uint64_t m = __ballot(eq);
    if (B.lane == 0) B.sh.wave_tot[B.wave] = static_cast<unsigned int>(__popcll(m));
    __syncthreads();
    unsigned int before = static_cast<unsigned int>(__popcll(m & ((1ull << B.lane) - 1))), all = 0;
    for (int w = 0; w < SelShared<SNT>::NW; ++w) {
      before += w < B.wave ? B.sh.wave_tot[w] : 0u;
      all += B.sh.wave_tot[w];
    }
    if (eq) P.sel[r] = static_cast<double>(before) < need ? SEL_TAKEN : SEL_LEFT;
    need -= static_cast<double>(all);
    __syncthreads();
  }
}

// Counts the rows of `tier` with in(key) into the bins of (base, scale) and
// finds the bin of the k-th smallest: sh.bin, sh.before, sh.in_bin.
template <int SNT, typename In>
__device__ void sel_histogram(Block<SNT, SelShared<SNT>>& B, const SelectParams& P, int64_t lo_r, int64_t hi_r,
                              int tier, unsigned int k, double base, double scale, In in) {
  constexpr int PER = SEL_BINS / SNT;
  SelShared<SNT>& sh = B.sh;
#pragma unroll
  for (int i = 0; i < PER; ++i) sh.hist[B.tid + i * SNT] = 0u;
  if (B.tid == 0) {
    sh.bin = 0;
    sh.before = sh.in_bin = sh.n_cand = 0u;
  }
  __syncthreads();
  for (int64_t r = lo_r + B.tid; r < hi_r; r += SNT) {
    const double key = P.keys[r];
    if (P.sel[r] == tier && in(key)) atomicAdd(&sh.hist[sel_bin(key, base, scale)], 1u);
  }
  __syncthreads();
  // inclusive scan over the threads of each thread's PER consecutive bins
  unsigned int own[PER], tot = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    own[i] = sh.hist[B.tid * PER + i];
    tot += own[i];
  }
  unsigned int inc = tot;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const unsigned int up = __shfl_up(inc, o, WAVE);
    if (B.lane >= o) inc += up;
  }
  if (B.lane == WAVE - 1) sh.wave_tot[B.wave] = inc;
  __syncthreads();
  unsigned int cum = inc - tot;
  for (int w = 0; w < B.wave; ++w) cum += sh.wave_tot[w];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (cum < k && cum + own[i] >= k) {  // exactly one bin of one thread
      sh.bin = B.tid * PER + i;
      sh.before = cum;
      sh.in_bin = own[i];
    }
    cum += own[i];
  }
  __syncthreads();
}

template <int SNT>
__global__ __launch_bounds__(SNT) void select_kernel(SelectParams P) {
  using SH = SelShared<SNT>;
  __shared__ SH sh;
  Block<SNT, SH> B(sh);
  for (int64_t i = blockIdx.x; i < P.n_traj; i += gridDim.x) {
    const int64_t lo = P.off[i], hi = P.off[i + 1];
    if (lo < 0 || hi < lo || hi > P.n_rows) continue;  // malformed range: rows left unwritten
    // keys and tiers; each thread reads back only the rows it wrote, until the marking's LDS lists
    double cnt[3] = {0, 0, 0};  // corrections among valid rows, rows of tier 0, of tier 1
    float mn[2] = {finf(), finf()}, mx[2] = {-finf(), -finf()};
    for (int64_t r = lo + B.tid; r < hi; r += SNT) {
      const bool M = P.valid ? (P.valid[r] != 0) : true;
      uint8_t tier = 2;
      double key = __builtin_huge_val();
      if (M) {
        const double u = static_cast<double>(philox_uniform(P.seed, SELECT, static_cast<uint64_t>(P.row_offset + r), 0));
        const double lE = log(-log(u));
        const double d = static_cast<double>(P.tv[r]);
        if (P.mode == SAKI_SELECT_RANDOM) {
          tier = 0; key = lE;
        } else if (d > 0.0) {
          tier = 0; key = lE - log(d);
        } else {
          tier = 1; key = lE;
        }
        cnt[0] += (P.corrected[r] != 0);
        cnt[1] += (tier == 0);
        cnt[2] += (tier == 1);
        const float kf = static_cast<float>(key);
        if (tier == 0) {
          mn[0] = fminf(mn[0], kf);
          mx[0] = fmaxf(mx[0], kf);
        } else {
          mn[1] = fminf(mn[1], kf);
          mx[1] = fmaxf(mx[1], kf);
        }
      }
      P.keys[r] = key;
      P.sel[r] = tier;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float a = -wave_max(-mn[t]), b = wave_max(mx[t]);
      if (B.lane == 0) {
        sh.red_f[B.wave][2 * t] = a;
        sh.red_f[B.wave][2 * t + 1] = b;
      }
    }
    __syncthreads();
    B.sum(cnt);
    const double m = cnt[0], n0 = cnt[1];
    // the tier that is selected from in part, and how many of it
    const int tier = m <= n0 ? 0 : 1;
    const double k = tier == 0 ? m : m - n0, n_tier = cnt[1 + tier];
    float kmin = finf(), kmax = -finf();
    for (int w = 0; w < SH::NW; ++w) {
      kmin = fminf(kmin, sh.red_f[w][2 * tier]);
      kmax = fmaxf(kmax, sh.red_f[w][2 * tier + 1]);
    }
    // rows outside that tier: all of tier 0 when tier 1 fills up, none of tier 1 otherwise
    auto outside = [&](uint8_t t) -> uint8_t { return (tier == 1 && t == 0) ? 1 : 0; };
    if (k <= 0.0 || k >= n_tier) {
      const uint8_t all = k > 0.0 ? 1 : 0;
      for (int64_t r = lo + B.tid; r < hi; r += SNT) {
        const uint8_t t = P.sel[r];
        P.sel[r] = t == tier ? all : outside(t);
      }
      __syncthreads();  // red_f is read above by every thread before the next trajectory writes it
      continue;
    }
    // linear bins over the tier's keys (the float-rounded ends only move the
    // first and last bin); a range that is empty or infinite puts every key in bin 0
    const double range = static_cast<double>(kmax) - static_cast<double>(kmin);
    const bool wide = range > 0.0 && range < __builtin_huge_val();
    const double base = wide ? static_cast<double>(kmin) : 0.0, scale = wide ? SEL_BINS / range : 0.0;
    const bool few = hi - lo < (int64_t{1} << 31);  // the bins count in 32 bits
    bool done = false;
    unsigned int below = 0;  // rows taken below the window
    int b1 = -1, b2 = -1;
    double base2 = 0.0, scale2 = 0.0;
    if (few) {
      sel_histogram<SNT>(B, P, lo, hi, tier, static_cast<unsigned int>(k), base, scale, [](double) { return true; });
      b1 = sh.bin;
      below = sh.before;
      unsigned int n_in = sh.in_bin;
      if (n_in > SEL_CAP && wide) {
        // a second level inside the bin (trajectories of several 100,000 rows)
        base2 = base + b1 / scale;
        scale2 = scale * SEL_BINS;
        __syncthreads();
        sel_histogram<SNT>(B, P, lo, hi, tier, static_cast<unsigned int>(k) - below, base2, scale2,
                           [&](double key) { return sel_bin(key, base, scale) == b1; });
        b2 = sh.bin;
        below += sh.before;
        n_in = sh.in_bin;
      }
      done = n_in <= SEL_CAP;
    }
    // position of a key against the window: < 0 taken, 0 inside, > 0 left
    auto side = [&](double key) {
      if (b1 < 0) return 0;
      const int d1 = sel_bin(key, base, scale) - b1;
      return (d1 != 0 || b2 < 0) ? d1 : sel_bin(key, base2, scale2) - b2;
    };
    if (done) {
      // marks the rows on either side and lists the window's
      for (int64_t r = lo + B.tid; r < hi; r += SNT) {
        const uint8_t t = P.sel[r];
        uint8_t mark = 0;
        if (t != tier) {
          mark = outside(t);
        } else {
          const double key = P.keys[r];
          const int sd = side(key);
          mark = sd < 0 ? 1 : 0;
          if (sd == 0) {
            // in_bin rows <= SEL_CAP, unless malformed ranges overlap and another
            // workgroup has changed `sel` since they were counted: the list stays
            // in its bounds whatever the ranges
            const unsigned int slot = atomicAdd(&sh.n_cand, 1u);
            if (slot < SEL_CAP) {
              sh.cand_key[slot] = key;
              sh.cand_row[slot] = r;
            }
          }
        }
        P.sel[r] = mark;
      }
      __syncthreads();
      const unsigned int n = sh.n_cand < SEL_CAP ? sh.n_cand : SEL_CAP;
      const unsigned int take = static_cast<unsigned int>(k) - below;
      for (unsigned int c = B.tid; c < n; c += SNT) {
        const double key = sh.cand_key[c];
        const int64_t r = sh.cand_row[c];
        unsigned int rank = 0;
        for (unsigned int j = 0; j < n; ++j) {
          const double kj = sh.cand_key[j];
          rank += (kj < key || (kj == key && sh.cand_row[j] < r)) ? 1u : 0u;
        }
        // the row's mark was written by another thread of the workgroup, before the barrier
        P.sel[r] = rank < take ? 1 : 0;
      }
      __syncthreads();
    } else {
      select_bisect<SNT>(B, P, lo, hi, tier, k - static_cast<double>(below), [&](double key) { return side(key) == 0; });
      // from `sel` and the keys alone: the inputs may be the buffer `sel` itself
      for (int64_t r = lo + B.tid; r < hi; r += SNT) {
        const uint8_t t = P.sel[r];
        P.sel[r] = t == SEL_TAKEN ? 1 : t == SEL_LEFT ? 0 : t != tier ? outside(t) : side(P.keys[r]) < 0 ? 1 : 0;
      }
      __syncthreads();
    }
  }
}
