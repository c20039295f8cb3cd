// SAKI coupling-and-routing kernels for gfx950 and the C ABI of include/saki.h.
//
// One workgroup of NT = 256 threads (4 waves) owns one row at a time and
// walks the grid's rows persistently; two workgroups share a compute unit, so
// one row's serial steps (reductions, the lambda search, the races) overlap
// the other's streaming sweeps.  The row engine (row_engine.hpp) runs the
// stats sweep, the lambda sweeps and the final sweep over a row.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include <mutex>
#include <string>

#include "../../include/saki.h"
#include "couple.hpp"
#include "verify.hpp"

#include "probe.hpp"

namespace saki {

// Clears the work counters at the start of a workspace (a kernel rather than
// a memset node, so that a captured graph replays it correctly).
__global__ void clear_counter_kernel(unsigned int* c) {
  if (threadIdx.x < 4) c[threadIdx.x] = 0u;
}

// Verification, before: no block has stopped or is known to reject, no item is
// taken.  The proposals are copied here, before any output is written, so that
// `token` or `proposal` may share the draft's buffer.
__global__ __launch_bounds__(256) void verify_begin_kernel(unsigned long long* next_item, int64_t n_blocks, int k,
                                                           int32_t* accepted_len, int32_t* correction,
                                                           const int32_t* draft, int32_t* proposal) {
  const int64_t b = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (b == 0) *next_item = 0ull;
  if (b < n_blocks) {
    accepted_len[b] = stop_word(k, false, -1);
    correction[b] = k;
    if (proposal)
      for (int j = 0; j < k; ++j) proposal[b * k + j] = draft[b * k + j];
  }
}

// Verification, after: each block's word (its first stopping position) becomes
// its accepted length and correction; the positions behind it are skipped
// ones, also those evaluated ahead.
__global__ __launch_bounds__(256) void verify_end_kernel(VerifyParams P) {
  const int64_t b = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (b >= P.n_blocks) return;
  const int32_t w = P.accepted_len[b];
  const int j = stop_pos(w);
  P.accepted_len[b] = j + ((w >> 22) & 1);
  P.correction[b] = (w & ((1 << 22) - 1)) - 1;
  if (P.has_pp) {
    for (int jj = j + 1; jj < P.k; ++jj) {
      const int64_t r = b * P.k + jj;
      write_skipped(&P.pp, r, SAKI_ROW_SKIPPED);
    }
  }
}

#include "rollout.hpp"

// ---------------------------------------------------------------------------
// Standalone routed loss and gradient from given events.
// ---------------------------------------------------------------------------
struct RouteParams {
  const void* s;
  int64_t n_rows;
  int64_t stride;
  int V;
  const int32_t* token;
  const uint8_t* corrected;
  const int32_t* vstar;
  const float* advantage;
  const uint8_t* valid;
  float grad_scale;
  float* row_loss;
  double* scaled_loss;
  void* grad;
  int64_t grad_stride;
  unsigned int* next_row;  // work counter in the caller's workspace, zero at launch
};

// Shared state of the standalone routed loss: the block reductions and, for
// bf16 rows, a row cache of KC chunks of s per wave (the log-sum-exp sweep
// stores the wave's last KC full chunks, the gradient sweep reads them).
template <int NT_, int KC>
struct RouteShared {
  static constexpr int NW = NT_ / WAVE;
  static constexpr int CACHE_CHUNKS = KC;
  double red_d[NW][RED_MAX];
  float red_f[NW][4];
  int red_i[NW][4];
  uint4 cache[KC > 0 ? NW * KC * 2 * WAVE : 1];  // [wave][slot][half][lane]
};
// 9 chunks per wave: 72 KiB, two workgroups per CU
constexpr int ROUTE_KC = 9;

// Standalone routed loss: two sweeps over s per row (log-sum-exp, then the
// gradient), the loss from the logit of the supervised entry.  Workgroups take
// rows from a counter, as in the coupling kernel.
template <typename T, typename G, bool GRAD>
__global__ __launch_bounds__(NT, WG_PER_CU) void route_kernel(RouteParams P) {
  using SH = RouteShared<NT, (sizeof(T) == 2 ? ROUTE_KC : 0)>;
  __shared__ SH sh;
  Block<NT, SH> B(sh);
  const int V = P.V;
  __shared__ unsigned int next_r;
  for (int64_t it = 0; it <= P.n_rows; ++it) {
    const unsigned int ru = take_next(P.next_row, &next_r);
    // unsigned: n_rows < 2^31 and the counter stays below n_rows + grid
    if (ru >= static_cast<unsigned int>(P.n_rows)) break;
    const int64_t r = static_cast<int64_t>(ru);
    const T* srow = static_cast<const T*>(P.s) + r * P.stride;
    G* grow = GRAD ? static_cast<G*>(P.grad) + r * P.grad_stride : nullptr;
    const bool M = P.valid ? (P.valid[r] != 0) : true;
    const bool C = P.corrected[r] != 0;
    const int hot = C ? P.vstar[r] : P.token[r];
    const bool hot_ok = hot >= 0 && hot < V;
    // the supervised entry's logit, loaded before the sweeps
    const float s_hot = hot_ok ? Loader<T>::load1(srow + hot) : 0.0f;
    float msL;
    const double S = lse_sweep<T, NT>(B, srow, V, &msL);
    const double lse = static_cast<double>(msL) * LN2_D + log(S);
    const bool bad = M && (!hot_ok || !isfinite(lse));
    const double A = C ? 0.0 : static_cast<double>(P.advantage[r]);
    float coef = 0.0f;
    if (M && !bad) coef = static_cast<float>(static_cast<double>(P.grad_scale) * (C ? 1.0 : A));
    if (GRAD)
      route_grad_sweep<T, G, NT>(B, srow, grow, V, msL, static_cast<float>(1.0 / S), coef, hot_ok ? hot : -1,
                                 s_hot, bad);
    if (B.tid == 0) {
      double l = 0.0;
      if (bad) {
        l = __builtin_nan("");
      } else if (M) {
        const double logp_h = static_cast<double>(s_hot) - lse;
        l = C ? -logp_h : -A * logp_h;
      }
      if (P.row_loss) P.row_loss[r] = static_cast<float>(l);
      if (P.scaled_loss) P.scaled_loss[r] = static_cast<double>(P.grad_scale) * l;
    }
  }
}

// Deterministic sum of the scaled row losses: fixed per-thread strides, then a
// fixed-order tree.  What bounds it: latency, on the one workgroup that the
// fixed order leaves; each thread has LOSS_DEPTH loads in flight, and the tree
// over 1,024 partial sums (i + i + 512, + 256, ...) takes one barrier: its four
// upper levels lie in the registers of one wave, the others are lane shifts (a
// coupling call of 256 rows x 4,096: 27.6 -> 26.1 us, against one load in flight
// and a barrier a level).  The additions and their order are unchanged.
constexpr int LOSS_DEPTH = 8;
__global__ __launch_bounds__(1024) void loss_sum_kernel(const double* x, int64_t n, double* out) {
  __shared__ double part[1024];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += LOSS_DEPTH * 1024) {
    double v[LOSS_DEPTH];
#pragma unroll
    for (int e = 0; e < LOSS_DEPTH; ++e) {
      const int64_t k = i + e * 1024;
      const double y = x[k < n ? k : i];
      v[e] = k < n ? y : 0.0;
    }
#pragma unroll
    for (int e = 0; e < LOSS_DEPTH; ++e) acc += v[e];
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x >= WAVE) return;
  double p[1024 / WAVE];
#pragma unroll
  for (int e = 0; e < 1024 / WAVE; ++e) p[e] = part[threadIdx.x + e * WAVE];
#pragma unroll
  for (int w = 512 / WAVE; w > 0; w >>= 1)
#pragma unroll
    for (int e = 0; e < w; ++e) p[e] += p[e + w];
#pragma unroll
  for (int w = WAVE / 2; w > 0; w >>= 1) p[0] += __shfl_down(p[0], w);
  if (threadIdx.x == 0) *out = p[0];
}

#include "select.hpp"

}  // namespace saki

// ===========================================================================
// C ABI
// ===========================================================================
namespace {

thread_local std::string g_last_error;

saki_status fail(saki_status st, const std::string& msg) {
  g_last_error = msg;
  return st;
}

saki_status ok() {
  g_last_error.clear();
  return SAKI_OK;
}

int elem_size(int32_t dt) { return dt == SAKI_BF16 ? 2 : 4; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

saki_status device_cus(int* cus) {
  static std::mutex mu;
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return fail(SAKI_E_DEVICE, "hipGetDevice failed");
  std::lock_guard<std::mutex> lock(mu);
  if (dev < 64 && cache[dev] > 0) {
    *cus = cache[dev];
    return SAKI_OK;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    return fail(SAKI_E_DEVICE, "hipDeviceGetAttribute(MultiprocessorCount) failed");
  if (dev < 64) cache[dev] = n;
  *cus = n;
  return SAKI_OK;
}

saki_status check_rows(const saki_rows* in, bool need_teacher = true) {
  if (!in) return fail(SAKI_E_NULLPTR, "rows descriptor is NULL");
  if (in->dtype != SAKI_F32 && in->dtype != SAKI_BF16) return fail(SAKI_E_DTYPE, "unknown logits dtype");
  if (in->reserved != 0) return fail(SAKI_E_VALUE, "saki_rows.reserved must be 0");
  if (in->n_rows < 0) return fail(SAKI_E_SHAPE, "n_rows < 0");
  if (in->vocab < 1 || in->vocab > SAKI_MAX_VOCAB) return fail(SAKI_E_SHAPE, "vocab outside [1, SAKI_MAX_VOCAB]");
  if (in->row_stride < in->vocab) return fail(SAKI_E_SHAPE, "row_stride < vocab");
  if (in->row_offset < 0) return fail(SAKI_E_VALUE, "row_offset < 0");
  if (in->n_rows == 0) return SAKI_OK;
  if (!in->student || (need_teacher && !in->teacher))
    return fail(SAKI_E_NULLPTR, "student or teacher pointer is NULL");
  if (!aligned16(in->student) || (need_teacher && !aligned16(in->teacher)) ||
      (in->row_stride * elem_size(in->dtype)) % 16 != 0)
    return fail(SAKI_E_ALIGN, "logit base pointers and row pitch must be 16-byte aligned");
  return SAKI_OK;
}

saki_status check_route(const saki_route_args* rt, int64_t vocab, bool* want_loss_sum) {
  *want_loss_sum = false;
  if (!rt) return SAKI_OK;
  if (!isfinite(rt->grad_scale)) return fail(SAKI_E_VALUE, "grad_scale is not finite");
  if (rt->correction_target != SAKI_TARGET_MODE && rt->correction_target != SAKI_TARGET_SAMPLE)
    return fail(SAKI_E_VALUE, "unknown correction_target");
  if (rt->grad) {
    if (rt->grad_dtype != SAKI_F32 && rt->grad_dtype != SAKI_BF16) return fail(SAKI_E_DTYPE, "unknown grad dtype");
    if (rt->grad_stride < vocab) return fail(SAKI_E_SHAPE, "grad_stride < vocab");
    if (!aligned16(rt->grad) || (rt->grad_stride * elem_size(rt->grad_dtype)) % 16 != 0)
      return fail(SAKI_E_ALIGN, "grad base pointer and row pitch must be 16-byte aligned");
  }
  *want_loss_sum = rt->loss_sum != nullptr;
  return SAKI_OK;
}

size_t loss_ws_bytes(int64_t n_rows) {
  const size_t b = static_cast<size_t>(n_rows) * sizeof(double);
  return (b + 255) & ~static_cast<size_t>(255);
}

size_t list_ws_bytes(int64_t n_rows) {
  const size_t b = static_cast<size_t>(n_rows) * sizeof(unsigned int);
  return (b + 255) & ~static_cast<size_t>(255);
}

saki_status launched(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SAKI_E_LAUNCH, std::string(what) + ": " + hipGetErrorString(e));
  return SAKI_OK;
}

// The coupling launch for the rows' type and the radius (see couple.hpp).
saki_status launch_couple(const saki::CoupleParams& P, bool bf16, bool route, bool grad, bool grad_bf16, int grid,
                          hipStream_t st) {
  const bool k34 = saki::use_k34(P.eps);
  const auto f = bf16 ? (k34 ? saki::launch_couple_part<1> : saki::launch_couple_part<0>)
                      : (k34 ? saki::launch_couple_part<3> : saki::launch_couple_part<2>);
  const hipError_t e = f(P, route, grad, grad_bf16, grid, st);
  if (e != hipSuccess) return fail(SAKI_E_LAUNCH, std::string("couple_kernel: ") + hipGetErrorString(e));
  return SAKI_OK;
}

template <typename T, typename G, bool GRAD>
saki_status launch_route(const saki::RouteParams& P, int grid, hipStream_t st) {
  hipLaunchKernelGGL((saki::route_kernel<T, G, GRAD>), dim3(grid), dim3(saki::NT), 0, st, P);
  return launched("route_kernel");
}

}  // namespace

extern "C" {

size_t saki_workspace_bytes(int op, int64_t n_rows, int64_t vocab) {
  (void)vocab;
  if (n_rows <= 0) return 0;
  switch (op) {
    case SAKI_OP_COUPLE:
      // the counter, the scaled row losses, and four bytes a row that callers'
      // workspaces have always held (unused)
      return 256 + loss_ws_bytes(n_rows) + list_ws_bytes(n_rows);
    case SAKI_OP_ROUTE:
      return 256 + loss_ws_bytes(n_rows);  // the row counter, then the scaled row losses
    case SAKI_OP_VERIFY:
      return 256;  // the work counter
    case SAKI_OP_SELECT:
      return loss_ws_bytes(n_rows);
    default:
      return 0;
  }
}

}  // extern "C"

// The library's own scratch for saki_couple_static: a workspace for
// SAKI_STATIC_MAX_ROWS rows.  Each GPU the library runs on holds its own copy
// until the process ends.  In host code
// `scratch` names a host-side stand-in, not the device array: only the
// address from hipGetSymbolAddress (static_scratch) is passed to kernels.
static __device__ __align__(256) unsigned char scratch[256 + SAKI_STATIC_MAX_ROWS * (sizeof(double) + sizeof(unsigned int))];

namespace {

constexpr size_t STATIC_SCRATCH_BYTES =
    256 + static_cast<size_t>(SAKI_STATIC_MAX_ROWS) * (sizeof(double) + sizeof(unsigned int));

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept.
saki_status static_scratch(void** ptr) {
  static std::mutex mu;
  static void* cache[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return fail(SAKI_E_DEVICE, "hipGetDevice failed");
  if (dev >= 64) return fail(SAKI_E_DEVICE, "device index above 63");
  std::lock_guard<std::mutex> lock(mu);
  if (cache[dev] == nullptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return fail(SAKI_E_DEVICE, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
    cache[dev] = p;
  }
  *ptr = cache[dev];
  return SAKI_OK;
}

// use_static: the workspace is the static scratch (ws and ws_bytes unused),
// looked up after every argument check.
saki_status couple_impl(const saki_rows* in, double eps, uint64_t seed, const saki_couple_out* out,
                        const saki_route_args* route, void* ws, size_t ws_bytes, saki_stream_t stream,
                        bool use_static);

}  // namespace

extern "C" {

saki_status saki_couple(const saki_rows* in, double eps, uint64_t seed, const saki_couple_out* out,
                        const saki_route_args* route, void* ws, size_t ws_bytes, saki_stream_t stream) {
  return couple_impl(in, eps, seed, out, route, ws, ws_bytes, stream, false);
}

saki_status saki_couple_static(const saki_rows* in, double eps, uint64_t seed, const saki_couple_out* out,
                               const saki_route_args* route, saki_stream_t stream) {
  return couple_impl(in, eps, seed, out, route, nullptr, 0, stream, true);
}

}  // extern "C"

namespace {

saki_status couple_impl(const saki_rows* in, double eps, uint64_t seed, const saki_couple_out* out,
                        const saki_route_args* route, void* ws, size_t ws_bytes, saki_stream_t stream,
                        bool use_static) {
  saki_status st = check_rows(in);
  if (st != SAKI_OK) return st;
  if (!out) return fail(SAKI_E_NULLPTR, "out is NULL");
  if (!(eps >= 0.0) || !isfinite(eps)) return fail(SAKI_E_VALUE, "eps must be finite and >= 0");
  bool want_sum = false;
  st = check_route(route, in->vocab, &want_sum);
  if (st != SAKI_OK) return st;
  if (use_static && in->n_rows > SAKI_STATIC_MAX_ROWS)
    return fail(SAKI_E_SHAPE, "n_rows above SAKI_STATIC_MAX_ROWS (the static scratch holds one double per row)");
  if (in->n_rows == 0) return ok();
  if (in->n_rows >= (int64_t{1} << 31)) return fail(SAKI_E_SHAPE, "more than 2^31 - 1 rows in one call");
  if (use_static) {
    st = static_scratch(&ws);
    if (st != SAKI_OK) return st;
    ws_bytes = STATIC_SCRATCH_BYTES;
  }
  if (!ws) return fail(SAKI_E_WORKSPACE, "workspace is NULL");
  if (ws_bytes < saki_workspace_bytes(SAKI_OP_COUPLE, in->n_rows, in->vocab))
    return fail(SAKI_E_WORKSPACE, "workspace smaller than saki_workspace_bytes(SAKI_OP_COUPLE)");
  if ((reinterpret_cast<uintptr_t>(ws) & 7u) != 0) return fail(SAKI_E_ALIGN, "workspace must be 8-byte aligned");
  double* const row_losses = reinterpret_cast<double*>(static_cast<char*>(ws) + 256);
  int cus = 0;
  st = device_cus(&cus);
  if (st != SAKI_OK) return st;
  saki::CoupleParams P{};
  P.s = in->student;
  P.t = in->teacher;
  P.n_rows = in->n_rows;
  P.stride = in->row_stride;
  P.row_offset = in->row_offset;
  P.V = static_cast<int>(in->vocab);
  P.eps = eps;
  P.lam_mid = saki::mid_lambda(eps);
  P.seed = seed;
  P.out = *out;
  if (route) {
    P.valid = route->valid_mask;
    P.grad_scale = route->grad_scale;
    P.row_loss = route->row_loss;
    P.scaled_loss = want_sum ? row_losses : nullptr;
    P.grad = route->grad;
    P.grad_stride = route->grad_stride;
    P.target_mode = route->correction_target;
  }
  // workspace: the row counter, then (behind 256 bytes) the scaled row losses
  unsigned int* const counter = static_cast<unsigned int*>(ws);
  const int64_t slots = static_cast<int64_t>(cus) * saki::WG_PER_CU;
  const int grid = static_cast<int>(std::min<int64_t>(in->n_rows, slots));
  hipStream_t hs = static_cast<hipStream_t>(stream);
  // one row per workgroup needs no counter (nor the launch that clears it)
  if (in->n_rows > slots) {
    P.next_row = counter;
    hipLaunchKernelGGL(saki::clear_counter_kernel, dim3(1), dim3(64), 0, hs, counter);
    st = launched("clear_counter_kernel");
    if (st != SAKI_OK) return st;
  }
  st = launch_couple(P, in->dtype == SAKI_BF16, route != nullptr, route && route->grad,
                     route && route->grad_dtype == SAKI_BF16, grid, hs);
  if (st != SAKI_OK) return st;
  if (want_sum) {
    hipLaunchKernelGGL(saki::loss_sum_kernel, dim3(1), dim3(1024), 0, hs,
                       static_cast<const double*>(row_losses), in->n_rows, route->loss_sum);
    st = launched("loss_sum_kernel");
    if (st != SAKI_OK) return st;
  }
  return ok();
}

}  // namespace

extern "C" {

saki_status saki_route_loss(const void* student, int32_t dtype, int64_t n_rows, int64_t vocab,
                            int64_t row_stride, const int32_t* token, const uint8_t* corrected,
                            const int32_t* teacher_argmax, const float* advantage,
                            const saki_route_args* route, void* ws, size_t ws_bytes,
                            saki_stream_t stream) {
  if (dtype != SAKI_F32 && dtype != SAKI_BF16) return fail(SAKI_E_DTYPE, "unknown logits dtype");
  if (n_rows < 0) return fail(SAKI_E_SHAPE, "n_rows < 0");
  if (vocab < 1 || vocab > SAKI_MAX_VOCAB) return fail(SAKI_E_SHAPE, "vocab outside [1, SAKI_MAX_VOCAB]");
  if (row_stride < vocab) return fail(SAKI_E_SHAPE, "row_stride < vocab");
  if (!route) return fail(SAKI_E_NULLPTR, "route is NULL");
  bool want_sum = false;
  saki_status st = check_route(route, vocab, &want_sum);
  if (st != SAKI_OK) return st;
  if (n_rows >= (int64_t{1} << 31)) return fail(SAKI_E_SHAPE, "more than 2^31 - 1 rows in one call");
  if (n_rows == 0) return ok();
  if (!student || !token || !corrected || !teacher_argmax || !advantage)
    return fail(SAKI_E_NULLPTR, "student, token, corrected, teacher_argmax and advantage are required");
  if (!ws) return fail(SAKI_E_WORKSPACE, "workspace is NULL");
  if (ws_bytes < saki_workspace_bytes(SAKI_OP_ROUTE, n_rows, vocab)) return fail(SAKI_E_WORKSPACE, "workspace too small");
  if ((reinterpret_cast<uintptr_t>(ws) & 7u) != 0) return fail(SAKI_E_ALIGN, "workspace must be 8-byte aligned");
  double* row_losses = reinterpret_cast<double*>(static_cast<char*>(ws) + 256);
  if (!aligned16(student) || (row_stride * elem_size(dtype)) % 16 != 0)
    return fail(SAKI_E_ALIGN, "student base pointer and row pitch must be 16-byte aligned");
  int cus = 0;
  st = device_cus(&cus);
  if (st != SAKI_OK) return st;
  saki::RouteParams P{};
  P.s = student;
  P.n_rows = n_rows;
  P.stride = row_stride;
  P.V = static_cast<int>(vocab);
  P.token = token;
  P.corrected = corrected;
  P.vstar = teacher_argmax;
  P.advantage = advantage;
  P.valid = route->valid_mask;
  P.grad_scale = route->grad_scale;
  P.row_loss = route->row_loss;
  P.scaled_loss = want_sum ? row_losses : nullptr;
  P.grad = route->grad;
  P.grad_stride = route->grad_stride;
  P.next_row = static_cast<unsigned int*>(ws);
  const int grid = static_cast<int>(std::min<int64_t>(n_rows, static_cast<int64_t>(cus) * saki::WG_PER_CU));
  hipStream_t hs = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(saki::clear_counter_kernel, dim3(1), dim3(64), 0, hs, P.next_row);
  st = launched("clear_counter_kernel");
  if (st != SAKI_OK) return st;
  const bool grad = route->grad != nullptr;
  const bool gbf = route->grad_dtype == SAKI_BF16;
  if (dtype == SAKI_BF16) {
    st = !grad ? launch_route<uint16_t, float, false>(P, grid, hs)
         : gbf ? launch_route<uint16_t, uint16_t, true>(P, grid, hs)
               : launch_route<uint16_t, float, true>(P, grid, hs);
  } else {
    st = !grad ? launch_route<float, float, false>(P, grid, hs)
         : gbf ? launch_route<float, uint16_t, true>(P, grid, hs)
               : launch_route<float, float, true>(P, grid, hs);
  }
  if (st != SAKI_OK) return st;
  if (want_sum) {
    hipLaunchKernelGGL(saki::loss_sum_kernel, dim3(1), dim3(1024), 0, hs, row_losses, n_rows,
                       route->loss_sum);
    st = launched("loss_sum_kernel");
    if (st != SAKI_OK) return st;
  }
  return ok();
}

saki_status saki_spec_verify(const saki_rows* in, int32_t k, const int32_t* draft, double eps,
                             uint64_t seed, int32_t eos_id, int32_t* accepted_len,
                             int32_t* correction, const saki_couple_out* per_pos, void* ws,
                             size_t ws_bytes, saki_stream_t stream) {
  saki_status st = check_rows(in);
  if (st != SAKI_OK) return st;
  if (k < 1 || k > SAKI_MAX_BLOCK_K) return fail(SAKI_E_SHAPE, "k outside [1, SAKI_MAX_BLOCK_K]");
  if (in->n_rows % k != 0) return fail(SAKI_E_SHAPE, "n_rows is not a multiple of k");
  if (!(eps >= 0.0) || !isfinite(eps)) return fail(SAKI_E_VALUE, "eps must be finite and >= 0");
  if (in->n_rows == 0) return ok();
  if (!draft || !accepted_len || !correction)
    return fail(SAKI_E_NULLPTR, "draft, accepted_len and correction are required");
  if (in->n_rows / k >= (int64_t{1} << 31)) return fail(SAKI_E_SHAPE, "more than 2^31 - 1 blocks");
  if (!ws || ws_bytes < saki_workspace_bytes(SAKI_OP_VERIFY, in->n_rows, in->vocab))
    return fail(SAKI_E_WORKSPACE, "workspace NULL or smaller than saki_workspace_bytes(SAKI_OP_VERIFY)");
  if ((reinterpret_cast<uintptr_t>(ws) & 3u) != 0) return fail(SAKI_E_ALIGN, "workspace must be 4-byte aligned");
  int cus = 0;
  st = device_cus(&cus);
  if (st != SAKI_OK) return st;
  saki::VerifyParams P{};
  P.s = in->student;
  P.t = in->teacher;
  P.n_blocks = in->n_rows / k;
  P.stride = in->row_stride;
  P.row_offset = in->row_offset;
  P.V = static_cast<int>(in->vocab);
  P.k = k;
  P.draft = draft;
  P.eps = eps;
  P.lam_mid = saki::mid_lambda(eps);
  P.seed = seed;
  P.eos = eos_id;
  P.accepted_len = accepted_len;
  P.correction = correction;
  if (per_pos) {
    P.pp = *per_pos;
    P.has_pp = 1;
  }
  // the 64-bit counter at the first 8-byte boundary of the 256 bytes
  P.next_item = reinterpret_cast<unsigned long long*>((reinterpret_cast<uintptr_t>(ws) + 7u) & ~static_cast<uintptr_t>(7u));
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const dim3 per_block(static_cast<unsigned>((P.n_blocks + 255) / 256));
  hipLaunchKernelGGL(saki::verify_begin_kernel, per_block, dim3(256), 0, hs, P.next_item, P.n_blocks, P.k,
                     P.accepted_len, P.correction, P.draft, P.has_pp ? P.pp.proposal : nullptr);
  st = launched("verify_begin_kernel");
  if (st != SAKI_OK) return st;
  const bool bf16 = in->dtype == SAKI_BF16;
  const hipError_t e = saki::use_k34(P.eps) ? saki::launch_verify_part<1>(P, cus, bf16, hs)
                                            : saki::launch_verify_part<0>(P, cus, bf16, hs);
  if (e != hipSuccess) return fail(SAKI_E_LAUNCH, std::string("verify_kernel: ") + hipGetErrorString(e));
  hipLaunchKernelGGL(saki::verify_end_kernel, per_block, dim3(256), 0, hs, P);
  st = launched("verify_end_kernel");
  if (st != SAKI_OK) return st;
  return ok();
}

saki_status saki_sample(const saki_rows* in, int64_t row_step, uint64_t seed, int32_t* token,
                        uint8_t* row_status, saki_stream_t stream) {
  saki_status st = check_rows(in, false);
  if (st != SAKI_OK) return st;
  if (row_step < 1) return fail(SAKI_E_VALUE, "row_step < 1");
  if (in->n_rows > 0 && (in->n_rows - 1) > (INT64_MAX - in->row_offset) / row_step)
    return fail(SAKI_E_VALUE, "row_offset + (n_rows - 1) * row_step overflows");
  if (in->n_rows == 0) return ok();
  if (!token) return fail(SAKI_E_NULLPTR, "token is required");
  int cus = 0;
  st = device_cus(&cus);
  if (st != SAKI_OK) return st;
  saki::SampleParams P{};
  P.s = in->student;
  P.n_rows = in->n_rows;
  P.stride = in->row_stride;
  P.row_offset = in->row_offset;
  P.row_step = row_step;
  P.V = static_cast<int>(in->vocab);
  P.seed = seed;
  P.token = token;
  P.status = row_status;
  const int grid = static_cast<int>(std::min<int64_t>(P.n_rows, static_cast<int64_t>(cus) * saki::SAMPLE_WG_PER_CU));
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const bool bf16 = in->dtype == SAKI_BF16;
  if (bf16)
    hipLaunchKernelGGL(saki::sample_kernel<uint16_t>, dim3(grid), dim3(saki::SAMPLE_NT), 0, hs, P);
  else
    hipLaunchKernelGGL(saki::sample_kernel<float>, dim3(grid), dim3(saki::SAMPLE_NT), 0, hs, P);
  st = launched("sample_kernel");
  if (st != SAKI_OK) return st;
  return ok();
}

saki_status saki_commit(const saki_traj* traj, int32_t k, int32_t eos_id,
                        const int32_t* accepted_len, const int32_t* correction,
                        const saki_couple_out* per_pos, int32_t* n_commit, saki_stream_t stream) {
  if (!traj) return fail(SAKI_E_NULLPTR, "trajectory descriptor is NULL");
  if (k < 1 || k > SAKI_MAX_BLOCK_K) return fail(SAKI_E_SHAPE, "k outside [1, SAKI_MAX_BLOCK_K]");
  if (traj->n_seq < 0) return fail(SAKI_E_SHAPE, "n_seq < 0");
  if (traj->max_len < 0 || traj->max_len > INT32_MAX) return fail(SAKI_E_SHAPE, "max_len outside [0, 2^31 - 1]");
  if (traj->n_seq == 0) return ok();
  if (!traj->tokens || !traj->length || !traj->done)
    return fail(SAKI_E_NULLPTR, "tokens, length and done are required");
  if (!accepted_len || !correction || !per_pos || !per_pos->token)
    return fail(SAKI_E_NULLPTR, "accepted_len, correction and per_pos->token are required");
  saki::CommitParams P{};
  P.tr = *traj;
  P.k = k;
  P.eos = eos_id;
  P.accepted_len = accepted_len;
  P.correction = correction;
  P.pp = *per_pos;
  P.n_commit = n_commit;
  const int64_t grid = (traj->n_seq + 255) / 256;
  if (grid > INT32_MAX) return fail(SAKI_E_SHAPE, "n_seq too large");
  hipLaunchKernelGGL(saki::commit_kernel, dim3(static_cast<unsigned>(grid)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), P);
  saki_status st = launched("commit_kernel");
  if (st != SAKI_OK) return st;
  return ok();
}

saki_status saki_probe_metrics(const saki_rows* in, int32_t k, float* c1, float* ck, float* kl_ts,
                               float* entropy, int32_t* topk, uint8_t* row_status,
                               saki_stream_t stream) {
  saki_status st = check_rows(in);
  if (st != SAKI_OK) return st;
  if (k < 1 || k > SAKI_MAX_PROBE_K || k > in->vocab) return fail(SAKI_E_SHAPE, "k outside [1, min(SAKI_MAX_PROBE_K, vocab)]");
  if (in->n_rows == 0) return ok();
  int cus = 0;
  st = device_cus(&cus);
  if (st != SAKI_OK) return st;
  saki::ProbeParams P{};
  P.s = in->student;
  P.t = in->teacher;
  P.n_rows = in->n_rows;
  P.stride = in->row_stride;
  P.V = static_cast<int>(in->vocab);
  P.k = k;
  P.c1 = c1;
  P.ck = ck;
  P.kl_ts = kl_ts;
  P.entropy = entropy;
  P.topk = topk;
  P.row_status = row_status;
  const int grid = static_cast<int>(std::min<int64_t>(in->n_rows, static_cast<int64_t>(cus) * saki::PROBE_WG_PER_CU));
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (in->dtype == SAKI_BF16)
    hipLaunchKernelGGL(saki::probe_kernel<uint16_t>, dim3(grid), dim3(saki::NT), 0, hs, P);
  else
    hipLaunchKernelGGL(saki::probe_kernel<float>, dim3(grid), dim3(saki::NT), 0, hs, P);
  st = launched("probe_kernel");
  if (st != SAKI_OK) return st;
  return ok();
}

saki_status saki_select_positions(int32_t mode, int64_t n_traj, int64_t n_rows,
                                  const int64_t* traj_offsets, const float* tv,
                                  const uint8_t* corrected, const uint8_t* valid_mask, uint64_t seed,
                                  int64_t row_offset, uint8_t* selected, void* ws, size_t ws_bytes,
                                  saki_stream_t stream) {
  if (mode != SAKI_SELECT_RANDOM && mode != SAKI_SELECT_TV_WEIGHTED) return fail(SAKI_E_VALUE, "unknown mode");
  if (n_traj < 0 || n_rows < 0) return fail(SAKI_E_SHAPE, "n_traj < 0 or n_rows < 0");
  if (row_offset < 0) return fail(SAKI_E_VALUE, "row_offset < 0");
  if (n_traj == 0 || n_rows == 0) return ok();
  if (!traj_offsets || !tv || !corrected || !selected)
    return fail(SAKI_E_NULLPTR, "traj_offsets, tv, corrected and selected are required");
  if (!ws) return fail(SAKI_E_WORKSPACE, "workspace is NULL");
  if (ws_bytes < loss_ws_bytes(n_rows)) return fail(SAKI_E_WORKSPACE, "workspace too small");
  if ((reinterpret_cast<uintptr_t>(ws) & 7u) != 0) return fail(SAKI_E_ALIGN, "workspace must be 8-byte aligned");
  int cus = 0;
  saki_status st = device_cus(&cus);
  if (st != SAKI_OK) return st;
  saki::SelectParams P{};
  P.mode = mode;
  P.n_traj = n_traj;
  P.n_rows = n_rows;
  P.off = traj_offsets;
  P.tv = tv;
  P.corrected = corrected;
  P.valid = valid_mask;
  P.seed = seed;
  P.row_offset = row_offset;
  P.sel = selected;
  P.keys = static_cast<double*>(ws);
  // the mean length decides (the ranges themselves are device data): either
  // workgroup size takes trajectories of any length
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (n_rows / n_traj >= saki::SEL_WIDE_ROWS) {
    const int grid = static_cast<int>(std::min<int64_t>(n_traj, static_cast<int64_t>(cus) * 2));
    hipLaunchKernelGGL(saki::select_kernel<1024>, dim3(grid), dim3(1024), 0, hs, P);
  } else {
    const int grid = static_cast<int>(std::min<int64_t>(n_traj, static_cast<int64_t>(cus) * 4));
    hipLaunchKernelGGL(saki::select_kernel<256>, dim3(grid), dim3(256), 0, hs, P);
  }
  st = launched("select_kernel");
  if (st != SAKI_OK) return st;
  return ok();
}

const char* saki_status_str(saki_status s) {
  switch (s) {
    case SAKI_OK: return "ok";
    case SAKI_E_NULLPTR: return "a required pointer is NULL";
    case SAKI_E_SHAPE: return "invalid shape";
    case SAKI_E_VALUE: return "invalid value";
    case SAKI_E_DTYPE: return "unknown dtype";
    case SAKI_E_ALIGN: return "pointer or pitch not 16-byte aligned";
    case SAKI_E_WORKSPACE: return "workspace missing or too small";
    case SAKI_E_DEVICE: return "HIP device error";
    case SAKI_E_LAUNCH: return "kernel launch failed";
  }
  return "unknown status";
}

const char* saki_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
