// Adaptive drafting (Section "Online Adaptive Drafting"): the stop rule 1 - prod sigmoid(f_phi(e_i)) > gamma over the
// proposed tokens of every sequence, and the value of the weighted binary cross-entropy that trains the head
// against the acceptance ratios min(1, p/q).  The head's logits are an input.
//
//   adapt_rule_kernel   one wavefront per sequence, four per workgroup: lane i forms sigmoid(a_i) and its two
//                       log-probabilities in binary64; the running product is formed left to right (at most 63
//                       factors) so that it has one fixed order, by every lane alike from lane reads, and lane i keeps
//                       its own term; per-sequence loss partials go to the workspace.  With an arrival counter the last
//                       workgroup adds them in a fixed order: a call is bound by its launches (64 sequences of up to 10 positions 6.9 us with
//                       one, 9.2 to 10.3 with two).  The chain counts where windows are long: walked by one lane that also
//                       stored every position, 16 sequences of 63 took 13.1 us, 6.8 now (10.5 with two launches).  Above 1024 sequences the sum is a launch of its own: the arrivals, one a
//                       workgroup at one word, take longer than that (3000 sequences 13.9 / 11.1 us, 512 7.7 / 10.2).
//   adapt_total_kernel  the same sum as a launch of its own, for the entry point whose scratch overlapping calls may
//                       share: they spoil each other's values there, and must not spoil a counter for later calls.
#include <mutex>

#include "device_math.h"
#include "otv_host.h"

namespace otv {
namespace {

struct AdaptArgs {
  ot_adapt_in in;
  ot_adapt_out out;
  double* part;      // [B, 2] loss sum and token count of each sequence
  int32_t* count;    // workgroups that have delivered, 0 between launches; nullptr: the sum is a launch of its own
};

constexpr int kThreads = 256, kWaves = kThreads / 64;
constexpr int kOneLaunchB = 1024;

// Sums of the B partials in a fixed order (all kThreads threads).
__device__ inline void adapt_total(const AdaptArgs& a, double (*s_w)[kWaves], int tid) {
  const int wave = tid >> 6, lane = tid & 63;
  double total = 0.0, count = 0.0;
  constexpr int kAtOnce = kOneLaunchB / kThreads;        // sequences asked for before any of them is added
  for (int b0 = tid; b0 < a.in.B; b0 += kAtOnce * kThreads) {
    double t[kAtOnce], c[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int b = min(b0 + j * kThreads, a.in.B - 1);
      t[j] = observe(a.part + 2 * b);
      c[j] = observe(a.part + 2 * b + 1);
    }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j)
      if (b0 + j * kThreads < a.in.B) { total += t[j]; count += c[j]; }
  }
  total = wave_sum(total);
  count = wave_sum(count);
  if (lane == 0) { s_w[0][wave] = total; s_w[1][wave] = count; }
  __syncthreads();
  if (tid == 0) {
    const double t = (s_w[0][0] + s_w[0][1]) + (s_w[0][2] + s_w[0][3]);
    const double c = (s_w[1][0] + s_w[1][1]) + (s_w[1][2] + s_w[1][3]);
    a.out.bce[0] = t;
    a.out.bce[1] = c;
    a.out.bce[2] = t / fmax(1.0, c);
  }
}

__global__ __launch_bounds__(kThreads) void adapt_rule_kernel(AdaptArgs a) {
  const int tid = threadIdx.x, wave = uniform(tid >> 6), i = tid & 63;
  const int b = blockIdx.x * kWaves + wave;
  __shared__ double s_w[2][kWaves];
  __shared__ int s_last;
  const bool live = b < a.in.B;
  const int r0 = live ? a.in.row_off[b] : 0, k = live ? a.in.row_off[b + 1] - r0 - 1 : -1;
  const int n = live && a.in.n_valid ? min(k, max(a.in.n_valid[b], 0)) : k;
  double sig = 0.0, cost = 0.0;
  if (i < n) {
    const double x = (double)a.in.head_logits[r0 + i];
    sig = 1.0 / (1.0 + exp(-x));
    if (a.out.bce) {
      // ln sigmoid(x) = -(ln(1 + e^-|x|) + max(-x, 0)),  ln(1 - sigmoid(x)) = -(ln(1 + e^-|x|) + max(x, 0))
      const double t = log1p(exp(-fabs(x)));
      const double l = (double)a.in.labels[r0 + i];
      cost = (double)a.in.w_accept * l * (t + fmax(-x, 0.0)) + (double)a.in.w_reject * (1.0 - l) * (t + fmax(x, 0.0));
    }
  }
  constexpr int kAtOnce = 8;                             // lane reads in front of the steps that wait for them
  const int n_all = uniform(n);
  double alive = 1.0, mine = 1.0, total = 0.0;           // mine: the product up to and including position i
  const double factor = i < n ? sig : 1.0;               // (past the window: factors of 1 and costs of 0)
  for (int j0 = 0; j0 < n_all; j0 += kAtOnce) {
    double f[kAtOnce], c[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) { f[j] = lane_value(factor, j0 + j); c[j] = lane_value(cost, j0 + j); }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      alive *= f[j];
      total += c[j];
      if (i == j0 + j) mine = alive;
    }
  }
  const bool summed = a.count && a.out.bce;              // by the last workgroup of this launch
  if (i == 0 && live) {
    publish(a.part + 2 * b, total);
    publish(a.part + 2 * b + 1, (double)n);
  }
  if (summed) {                                          // the partials are counted in before the outputs are stored
    stores_done();
    __syncthreads();
    if (tid == 0) s_last = arrive(a.count, gridDim.x);
  }
  const double rej = i < n ? 1.0 - mine : 0.0;
  const unsigned long long stop = __ballot(i < n && rej > (double)a.in.gamma);
  if (i <= k) {                                          // the sequence's unused entries read 0
    a.out.p_accept[r0 + i] = (float)sig;
    a.out.p_any_reject[r0 + i] = (float)rej;
  }
  if (i == 0 && live) a.out.n_keep[b] = stop ? (int)__ffsll((long long)stop) : n;
  if (!summed) return;
  __syncthreads();
  if (s_last) adapt_total(a, s_w, tid);
}

__global__ __launch_bounds__(kThreads) void adapt_total_kernel(AdaptArgs a) {
  __shared__ double s_w[2][kWaves];
  adapt_total(a, s_w, threadIdx.x);
}

}  // namespace
}  // namespace otv

using namespace otv;

namespace {

// Scratch of ot_adaptive_drafting_static: the per-sequence loss partials, in an array that is part of the library's
// code object instead of an allocation.  Every GPU the library runs on holds its own copy at its own address; that
// address is looked up once per device (the array's name is only a host-side handle, never a device pointer).
static __device__ __align__(256) double scratch[2 * OT_STATIC_MAX_BATCH];

constexpr int kMaxDevices = 64;
double* g_scratch_ptr[kMaxDevices];        // device address of `scratch` on each device, nullptr until looked up
std::mutex g_scratch_mutex;

// Address of `scratch` on the current device (looked up on the first call per device), or nullptr with the error set.
double* static_scratch() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) { (void)ot_fail_hip(e, "hipGetDevice"); return nullptr; }
  if (dev < 0 || dev >= kMaxDevices) { (void)ot_fail(OT_ERR_SHAPE, "device index %d is not supported", dev); return nullptr; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) { (void)ot_fail_hip(e, "hipGetSymbolAddress(scratch)"); return nullptr; }
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  return g_scratch_ptr[dev];
}

// Validates the arguments shared by the two entry points and launches on `stream` with the loss partials in `part` and the
// arrival counter at `count` (or none).
int adaptive_drafting(const char* who, const ot_adapt_in* in, ot_adapt_out* out, int max_batch, int max_k, double* part,
                      int32_t* count, hipStream_t stream) {
  if (in->reserved != 0) return ot_fail(OT_ERR_SHAPE, "%s: reserved must be 0", who);
  if (in->B < 0 || in->B > max_batch) return ot_fail(OT_ERR_SHAPE, "%s: B = %d exceeds the limit of %d sequences", who, in->B, max_batch);
  if (!(in->gamma >= 0.f && in->gamma <= 1.f)) return ot_fail(OT_ERR_SHAPE, "%s: gamma must be in [0, 1]", who);
  if (out->bce && !in->labels) return ot_fail(OT_ERR_NULL, "%s: the loss value needs labels", who);
  if (out->bce && !(in->w_accept >= 0.f && in->w_reject >= 0.f)) return ot_fail(OT_ERR_SHAPE, "%s: weights must be non-negative", who);
  AdaptArgs a{};
  if (in->B > kOneLaunchB) count = nullptr;
  a.in = *in; a.out = *out; a.part = part; a.count = count;
  if (in->B > 0) {
    if (!in->row_off || !in->row_off_host || !in->head_logits) return ot_fail(OT_ERR_NULL, "%s: row_off, row_off_host and head_logits must not be NULL", who);
    if (!out->p_accept || !out->p_any_reject || !out->n_keep) return ot_fail(OT_ERR_NULL, "%s: p_accept, p_any_reject and n_keep are required", who);
    if (in->row_off_host[0] != 0) return ot_fail(OT_ERR_SHAPE, "%s: row_off[0] must be 0", who);
    for (int b = 0; b < in->B; ++b) {
      const int64_t rows = (int64_t)in->row_off_host[b + 1] - in->row_off_host[b];
      if (rows < 1 || rows - 1 > max_k) return ot_fail(OT_ERR_SHAPE, "%s: sequence %d owns %lld rows", who, b, (long long)rows);
    }
    hipLaunchKernelGGL(adapt_rule_kernel, dim3(ceil_div(in->B, kWaves)), dim3(kThreads), 0, stream, a);
  }
  if (out->bce && (in->B == 0 || !count)) hipLaunchKernelGGL(adapt_total_kernel, dim3(1), dim3(kThreads), 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return ot_fail_hip(e, who);
  return OT_OK;
}

}  // namespace

// Looks up the static scratch of the current device ahead of the first ot_adaptive_drafting_static call (from
// ot_verify_init, so that a caller who must not trigger any set-up later has it done).
int ot_static_scratch_prepare() { return static_scratch() ? OT_OK : OT_ERR_HIP; }

#pragma GCC visibility push(default)
extern "C" {

int ot_adaptive_drafting(ot_ctx* ctx, const ot_adapt_in* in, ot_adapt_out* out) {
  if (!ctx || !in || !out) return ot_fail(OT_ERR_NULL, "ot_adaptive_drafting: ctx, in and out must not be NULL");
  return adaptive_drafting("ot_adaptive_drafting", in, out, ctx->max_batch, ctx->max_k, ctx->adapt_part, ctx->adapt_count, ctx->stream);
}

int ot_adaptive_drafting_static(const ot_adapt_in* in, ot_adapt_out* out, void* stream) {
  if (!in || !out) return ot_fail(OT_ERR_NULL, "ot_adaptive_drafting_static: in and out must not be NULL");
  if (in->B > OT_STATIC_MAX_BATCH)
    return ot_fail(OT_ERR_SHAPE, "ot_adaptive_drafting_static: B = %d exceeds OT_STATIC_MAX_BATCH = %d, the size of the static "
                   "scratch; use ot_adaptive_drafting", in->B, OT_STATIC_MAX_BATCH);
  double* part = static_scratch();
  if (!part) return OT_ERR_HIP;
  return adaptive_drafting("ot_adaptive_drafting_static", in, out, OT_STATIC_MAX_BATCH, OT_MAX_K, part, nullptr, static_cast<hipStream_t>(stream));
}

}  // extern "C"
#pragma GCC visibility pop
