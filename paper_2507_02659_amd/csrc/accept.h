// Acceptance test of a translated proposal (Algorithm 1, rejection-sampling step) as device functions: the merge of
// softmax partials into row statistics, and the test itself, which one wavefront runs for a whole sequence.
//
// The lane at which a segment starts owns its mapped position j: it forms p_j(t_j), the ratio min(1, p/q') and its Philox uniform;
// acceptance tests at different positions are independent given (u_j, p_j(t_j), q'_j), so "stop at the first rejection" is a
// ballot and a find-first-set, not a loop.  The outcome is the FinalInfo record of the sequence: where and from what the final token
// is drawn.
#pragma once

#include "translate.h"

namespace otv {

// exp((x - mx) / T) for x <= mx, by which the sum of a part with maximum x is rescaled to the row's: through the hardware 2^x
// (exponent scale sc), or in binary64 (exact; wavefront-uniform).
__device__ __forceinline__ double rescale(float x, float mx, float sc, double invT, bool exact) {
  return exact ? exp(((double)x - (double)mx) * invT) : (double)__builtin_amdgcn_exp2f((x - mx) * sc);
}

// The scale of a target row's exponents, log2(e) / T.
__device__ __forceinline__ float row_scale(float T) { return T > 0.f ? (1.f / T) * kLog2eF : kLog2eF; }

// Lanes of a wavefront hold running statistics r of parts of one row (exponent scale sc): merges them in a fixed order; lane 0
// publishes the row's (max, 1 / sum, argmax) to LDS slot `at` and, if asked, (max, sum, argmax) to the workspace.
__device__ __forceinline__ void wave_publish_row(const RunStat& r, float sc, int row, int lane, float* s_mx, double* s_inv,
                                        int* s_arg, int at, bool to_workspace, float* g_mx, double* g_S, int32_t* g_arg,
                                        double invT = 1.0, bool exact = false) {
  const float mx = wave_max(r.mx);
  const int arg = wave_min(r.mx == mx ? r.arg : 0x7FFFFFFF);
  const double S = wave_sum(r.mx == -INFINITY ? 0.0 : r.sum * rescale(r.mx, mx, sc, invT, exact));
  if (lane == 0) {
    s_mx[at] = mx; s_inv[at] = 1.0 / S; s_arg[at] = arg;
    if (to_workspace) { g_mx[row] = mx; g_S[row] = S; g_arg[row] = arg; }
  }
}

// Merges the LM head's partials of one target row (nfine of them, one per column tile): called by a whole wavefront.
// A lane requests eight 16-byte partials at a time before it looks at any of them (one round trip to memory for up
// to 512 tiles) and keeps a running maximum with the sum rescaled to it; the lanes are then merged (wave_publish_row).  Sums
// are rescaled and added in binary64, in a fixed order.
__device__ inline void merge_fused_row(const Partial* __restrict__ part, int nfine, int row, float T, int lane,
                                       float* s_mx, double* s_inv, int* s_arg, int at, bool to_workspace, float* g_mx,
                                       double* g_S, int32_t* g_arg) {
  const uint4* p = reinterpret_cast<const uint4*>(part + (int64_t)row * nfine);
  constexpr int kAtOnce = 8;
  uint4 raw[kAtOnce];
  auto load = [&](int c0) {
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) raw[j] = p[min(c0 + j * 64 + lane, nfine - 1)];
  };
  load(0);                                             // in front of everything that waits for the temperature
  const float sc = row_scale(T);
  RunStat r;
  for (int c0 = 0; c0 < nfine; c0 += kAtOnce * 64) {
    if (c0 > 0) load(c0);
    float bm = -INFINITY;
    int bi = 0x7FFFFFFF;
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      if (c0 + j * 64 >= nfine) break;                 // wavefront-uniform
      const float m = c0 + j * 64 + lane < nfine ? __uint_as_float(raw[j].x) : -INFINITY;
      raw[j].x = __float_as_uint(m);
      const int ai = (int)raw[j].y;
      if (m > bm || (m == bm && ai < bi)) { bm = m; bi = ai; }
    }
    if (bm > r.mx || (bm == r.mx && bi < r.arg)) {
      r.sum *= (double)__builtin_amdgcn_exp2f((r.mx - bm) * sc);
      r.mx = bm; r.arg = bi;
    }
    if (r.mx != -INFINITY) {
#pragma unroll
      for (int j = 0; j < kAtOnce; ++j) {
        if (c0 + j * 64 >= nfine) break;
        const double sum = c0 + j * 64 + lane < nfine ? __hiloint2double((int)raw[j].w, (int)raw[j].z) : 0.0;
        r.sum += sum * (double)__builtin_amdgcn_exp2f((__uint_as_float(raw[j].x) - r.mx) * sc);
      }
    }
  }
  wave_publish_row(r, sc, row, lane, s_mx, s_inv, s_arg, at, to_workspace, g_mx, g_S, g_arg);
}

// The same for the chunk partials of the statistics launch (three arrays, nch entries per row): lane c takes chunks
// c, c + 64, ...  exact: as above; steps of many sequences, which no single chain of instructions bounds, ask for it.
__device__ __forceinline__ void merge_chunk_row(const float* __restrict__ pmax, const double* __restrict__ psum,
                                       const int32_t* __restrict__ parg, int nch, int row, float T, double invT, int lane,
                                       float* s_mx, double* s_inv, int* s_arg, int at, bool to_workspace, float* g_mx,
                                       double* g_S, int32_t* g_arg, bool exact) {
  const int64_t o = (int64_t)row * nch;
  const float sc = row_scale(T);
  RunStat r;
  for (int c = lane; c < nch; c += 64) {
    const float m = pmax[o + c];
    const int ai = parg[o + c];
    const double sum = psum[o + c];
    if (m > r.mx || (m == r.mx && ai < r.arg)) {
      if (r.mx != -INFINITY) r.sum *= rescale(r.mx, m, sc, invT, exact);
      r.mx = m; r.arg = ai;
    }
    if (m != -INFINITY) r.sum += sum * rescale(m, r.mx, sc, invT, exact);
  }
  wave_publish_row(r, sc, row, lane, s_mx, s_inv, s_arg, at, to_workspace, g_mx, g_S, g_arg, invT, exact);
}

// What is merged to the statistics of a draft row, as loaded (asked for before anything is known about the temperature).
// kChunks: the first chunk partials of the statistics launch; otherwise the pieces that the LM-head launch left.
constexpr int kChunksAtOnce = 4;                           // chunks asked for before any of them is looked at
template <bool kChunks> struct DraftPartials;
template <> struct DraftPartials<true> {
  float m[kChunksAtOnce];
  int arg[kChunksAtOnce];
  double sum[kChunksAtOnce];
  __device__ __forceinline__ void load(const StepArgs& a, int q, int c0 = 0) {
    const int64_t o = (int64_t)q * a.nchd;
#pragma unroll
    for (int j = 0; j < kChunksAtOnce; ++j) {
      const int c = min(c0 + j, a.nchd - 1);
      m[j] = a.dpart_max[o + c]; arg[j] = a.dpart_arg[o + c]; sum[j] = a.dpart_sum[o + c];
    }
  }
};
template <> struct DraftPartials<false> {
  DraftPiece pc[kDraftPieces];
  __device__ __forceinline__ void load(const StepArgs& a, int q) {
    const int last = a.plan.pieces(q) - 1;
    const DraftPiece* rec = a.dpiece + (int64_t)q * kDraftPieces;
#pragma unroll
    for (int j = 0; j < kDraftPieces; ++j) pc[j] = rec[min(j, last)];
  }
};

// Statistics of draft row q from the chunk partials of the statistics launch (ascending chunks): lane-local.  kWide: the row may
// have more than kChunksAtOnce chunks (compiled in where it has not, the binary64 exponential costs every step 0.3 us).
template <bool kWide>
__device__ __forceinline__ void merge_draft_chunks(const StepArgs& a, int q, float Td, double invTd, DraftPartials<true>& p, float* out_mx, double* out_S,
                                          int* out_arg, bool exact) {
  const float sc = Td > 0.f ? kLog2eF / Td : kLog2eF;
  constexpr int kAtOnce = kChunksAtOnce;
  RunStat r;
  for (int c0 = 0; c0 < a.nchd; c0 += kAtOnce) {
    if (c0 > 0) p.load(a, q, c0);
    const float before = r.mx;
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j)
      if (c0 + j < a.nchd && p.m[j] > r.mx) { r.mx = p.m[j]; r.arg = p.arg[j]; }   // ascending chunks: a later equal maximum does not replace
    // in binary64 always: a factor per group of chunks, each with the error of a binary32 2^x, would add up in the sums of the
    // first chunks, which carry one such error already
    if (kWide && before != -INFINITY && r.mx > before) r.sum *= rescale(before, r.mx, sc, invTd, true);
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j)
      if (c0 + j < a.nchd && p.m[j] != -INFINITY) r.sum += p.sum[j] * rescale(p.m[j], r.mx, sc, invTd, exact);
    if (!kWide) break;
  }
  *out_mx = r.mx; *out_S = r.sum; *out_arg = r.arg;
}

// The same from the row's pieces (ascending order).
__device__ __forceinline__ void merge_draft_pieces(const StepArgs& a, int q, float Td, const DraftPartials<false>& p, float* out_mx,
                                                   double* out_S, int* out_arg) {
  const int n = a.plan.pieces(q);
  const float scale = Td > 0.f ? kLog2eF / Td : kLog2eF;
  float bm = -INFINITY;
  int ba = 0x7FFFFFFF;
#pragma unroll
  for (int j = 0; j < kDraftPieces; ++j)
    if (j < n && p.pc[j].mx > bm) { bm = p.pc[j].mx; ba = p.pc[j].arg; }
  double total = 0.0;
#pragma unroll
  for (int j = 0; j < kDraftPieces; ++j)
    if (j < n && p.pc[j].mx != -INFINITY) total += p.pc[j].sum * (double)__builtin_amdgcn_exp2f((p.pc[j].mx - bm) * scale);
  *out_mx = bm; *out_S = total; *out_arg = ba;
}

// The acceptance test of sequence b by one wavefront, in three parts: what it needs of the drafter (walk and q'), the test, and
// the outputs of the lead group.  A lane holds the segment that starts at its draft position (Window) and the draft row there.
struct DraftLane {
  float zq, mxq;                // draft logit of the drafted id; the draft row's maximum, its lowest index, its sum
  int argq, dm;
  double Sq, invSq, q, qp;      // q(d) of the drafted id; q'(t) of the segment
};

// The outcome of the test.  n: first rejected mapped position, or m; `ratio` and `pt` of this lane's segment.
struct Outcome {
  int n, at;                    // at: draft position where the rejected segment starts (m: where the walk ended)
  double pt, ratio;
};

// s_pmx / s_pinv / s_parg: maximum, 1 / sum and argmax of the sequence's target rows; z_tok: z[row pos, t] of a reached segment; u1 its
// uniform.
__device__ __forceinline__ Outcome test_window(float T, double invT, const Window& w, const DraftLane& D, bool reached, int pos, float z_tok,
                                      double u1, const float* s_pmx, const double* s_pinv, const int* s_parg) {
  Outcome o;
  const int row = reached ? pos : 0;
  bool ok = true;               // other lanes do not veto
  o.pt = 0.0; o.ratio = 0.0;
  if (T > 0.f) {
    o.pt = exp(((double)z_tok - (double)s_pmx[row]) * invT) * s_pinv[row];
    o.ratio = D.qp > 0.0 ? fmin(1.0, o.pt / D.qp) : o.pt > 0.0 ? 1.0 : 0.0;
    ok = u1 < o.ratio;
  } else {
    ok = w.t == s_parg[row];
    o.pt = o.ratio = ok ? 1.0 : 0.0;
  }
  const unsigned long long rejected = __ballot(reached && !ok);
  o.at = rejected ? (int)__builtin_ctzll(rejected) : w.end;
  o.n = rejected ? __popcll(w.starts & bits_below(o.at)) : w.m;
  return o;
}

// The outputs of the test: p_tok, ratio and out_tokens of the sequence's rows and its counts.
__device__ __forceinline__ void write_outcome(const StepArgs& a, int b, int r0, int k, int lane, float T, const Window& w, const Outcome& o,
                                     bool reached, int pos, const int* s_parg) {
  if (reached) {
    a.out.p_tok[r0 + pos] = (float)o.pt;
    a.out.ratio[r0 + pos] = (float)o.ratio;
    if (pos < o.n) a.out.out_tokens[r0 + pos] = w.t;
  }
  if (lane <= k) {
    if (lane >= w.m) { a.out.p_tok[r0 + lane] = 0.f; a.out.ratio[r0 + lane] = 0.f; }
    // a greedy sequence's final token is the argmax of row n; otherwise entry n belongs to the draw (which may run before or
    // after this store)
    if (lane > o.n) a.out.out_tokens[r0 + lane] = -1;
    else if (lane == o.n && !(T > 0.f)) a.out.out_tokens[r0 + lane] = s_parg[lane];
  }
  const int hits = __popcll(__ballot(reached && w.L > 1 && pos < o.n));
  if (lane == 0) {
    a.out.n_accept[b] = o.n;
    a.out.n_accept_draft[b] = o.at;                       // the accepted spans end where the rejected one starts
    a.out.hits_accepted[b] = hits;
    a.out.n_emit[b] = o.n + 1;
  }
}

// The outputs of a sequence with a drafted id outside [0, V_d): it proposes and emits nothing.
__device__ __forceinline__ void write_bad_sequence(const StepArgs& a, int b, int r0, int k, int lane) {
  if (lane <= k) {
    a.out.mapped_ids[r0 + lane] = -1; a.out.span_start[r0 + lane] = -1; a.out.span_len[r0 + lane] = 0;
    a.out.q_tok[r0 + lane] = 0.f; a.out.out_tokens[r0 + lane] = -1; a.out.p_tok[r0 + lane] = 0.f; a.out.ratio[r0 + lane] = 0.f;
  }
  if (lane == 0) {
    a.out.n_mapped[b] = 0; a.out.hits_proposed[b] = 0; a.out.flags[b] = OT_FLAG_BAD_ID;
    a.out.n_accept[b] = 0; a.out.n_accept_draft[b] = 0; a.out.n_emit[b] = 0; a.out.hits_accepted[b] = 0;
  }
}

// log2(e) / T as two positive floats, its first 21 bits and the rest, so that -inf times either is -inf: split at the nearest
// float, the lower one is negative for about half of all temperatures (0.7, 0.9, ..), and a masked logit gave NaN.
struct Scale { float hi, lo; };
__device__ __forceinline__ Scale split_scale(double invT) {
  const double x = invT * 1.4426950408889634;
  Scale s;
  s.hi = (float)__hiloint2double(__double2hiint(x), 0);
  s.lo = fmaxf((float)(x - (double)s.hi), 1e-30f);
  return s;
}

// Where and from what the final token is drawn (wavefront-uniform).  u2: the uniform of row n.
__device__ __forceinline__ FinalInfo final_info(int r0, int q0, float T, float Td, Scale sc, Scale scq, const Window& w, const DraftLane& D,
                                       const Outcome& o, double u2, const float* s_pmx, const double* s_pinv) {
  FinalInfo fin{};                                      // mode 0: nothing to draw
  fin.row = r0 + o.n; fin.t_ng = -1; fin.t_pre = -1; fin.argq = -1; fin.flags = w.flags; fin.u2 = u2;
  fin.mx = s_pmx[o.n]; fin.sc_hi = sc.hi; fin.sc_lo = sc.lo; fin.invS = s_pinv[o.n]; fin.scq_hi = scq.hi; fin.scq_lo = scq.lo;
  if (!(T > 0.f)) return fin;
  if (o.n == w.m && !(w.flags & OT_FLAG_UNMAPPABLE)) {
    fin.mode = 2;                                       // everything accepted: free token ~ p
    return fin;
  }
  fin.mode = 3;                                         // correction token ~ norm(max(0, p - q'))
  fin.drow = q0 + o.at;                                 // the rejected span's first draft row, or the untranslatable id's
  fin.greedy_draft = !(Td > 0.f);
  fin.mxq = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(D.mxq), o.at));
  fin.invSq = lane_value(D.invSq, o.at);
  fin.argq = __builtin_amdgcn_readlane(D.argq, o.at);
  if (o.n < w.m && __builtin_amdgcn_readlane(w.L, o.at) > 1) {   // Eq. 2 overrides for the n-gram matched at this position
    fin.t_ng = __builtin_amdgcn_readlane(w.t, o.at);
    fin.pi = lane_value(D.qp, o.at);
    fin.t_pre = __builtin_amdgcn_readlane(D.dm, o.at);
    fin.q_pre = lane_value(D.q, o.at) - fin.pi;
  }
  return fin;
}

}  // namespace otv
