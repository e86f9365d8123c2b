// Forward values of the hybrid cross-vocabulary distillation loss (Section "Cross-vocabulary Distillation", the
// loss equation): reverse KL D_KL(q' || p) on drafted tokens that translate through the direct map, and on the
// sub-tokens of n-gram tokens either the negative log-likelihood -log q(d_i) or the approximate KL with Eq. 2's two
// overrides, weighted by lambda (a constant, or the verified target probability p(t_i)).
//
// The call follows a verification step on the same inputs and reuses what that step left behind: the translation
// (mapped ids and spans in the step's output buffers), the logits and the softmax statistics of every target and
// draft row in the workspace.  With those, ln p(v) = (z_v - max)/T - ln S costs one fused multiply-add per id and
// q'(v) one exponential; no probability row is materialised unless the caller asks for the q' rows.
//
// One launch, grid = (groups of terms) x (rows).  Every workgroup finds its row's token by itself (kind, spans); one
// wavefront forms the constants of p and q' at that position (LossRow) and, in group 0, the row's NLL and lambda, while
// the others copy the draft row to LDS; then the workgroup sums q' (ln q' - ln p) over its terms in binary64 (optionally
// writing q', Eq. 2, as fp32), publishes the sum and counts itself in at its row.  The last workgroup of a row adds the
// groups' sums in a fixed order and counts the row in; the last of all forms the totals, in a fixed order.  A row
// without a KL term is counted in by its group 0 alone.  Nothing waits for another workgroup.
//
// The terms are the mapped pairs (target id, draft id), listed once per context in ascending target id: a quarter of the
// target ids where a 32000-id drafter meets a 128256-id target, and the logits are still read in order.  With every target
// id visited the launch took 39 us at 144 rows, bound by its binary64 instructions.  Now it is bound by the chain of round
// trips in a workgroup: 60 to 100 rows of 128256 ids are 32 to 52 MB, 5 to 8 us at the rate of a large copy.
// Measured, us per call: 144 rows x 128256 ids 17.3 (20.8 before the places below, with overrides and bounds tested at every term and
// the copy shared with the wavefront that forms the constants), against 42.8 for four launches (in the kernel trace: constants 7.6, tiles
// of 1024 ids with the gather from memory 30.9, sums per row 4.8, totals 4.0); 9 rows x 100000 ids 12.6 / 19.7.
#include <algorithm>
#include <type_traits>

#include "device_math.h"
#include "otv_host.h"
#include "resid.h"

namespace otv {
namespace {

constexpr int kPerTurn = 8;                   // terms per thread and turn, a workgroup's threads apart

struct LossRow {
  int32_t t_ng, t_pre;   // Eq. 2 overrides: target id of the n-gram / direct image of its first sub-token, or -1
  double pi, q_pre, ln_pi, ln_q_pre;
  // ln p(v) = (z_v - mx) * invT - lnS at the token's target row; ln q(d) = (zq_d - mxq) * invTd - lnSq at the draft row of
  // its first sub-token
  double mx, invT, lnS, mxq, invTd, lnSq;
};

struct LossArgs {
  int32_t B, M, V_t, V_d, dtype;
  const int32_t* row_off;
  const float* temperature;
  const float* draft_temperature;
  const void* draft_logits;
  const int32_t* draft_ids;
  const int32_t* dmap;
  const int32_t* tmap;
  const int2* pairs;     // [n_pairs] (target id, draft id) of the direct map in ascending target id
  int32_t n_pairs;
  const float* Z;
  int64_t ldz;
  const float* row_max; const double* row_sum;
  const float* drow_max; const double* drow_sum;
  // translation and outcome of the verification step
  const int32_t* n_mapped; const int32_t* n_accept; const int32_t* mapped_ids; const int32_t* span_start;
  const int32_t* span_len; const float* p_tok;
  // options
  float lambda; int32_t lambda_mode, ngram_term, accepted_only;
  // workspace
  double* part;          // [M, kLossGroups] sums of a row's groups
  int32_t* count;        // [M + 1] groups of a row that have delivered, and (first entry) rows that have; 0 between launches
  // outputs
  ot_loss_out out;
};

__device__ inline float draft_logit(const LossArgs& a, int drow, int dv) {
  const int64_t at = (int64_t)drow * a.V_d + dv;
  return a.dtype == OT_BF16 ? bf16_to_f32(static_cast<const uint16_t*>(a.draft_logits)[at])
                            : static_cast<const float*>(a.draft_logits)[at];
}

// The constants of row `row` (token t of L drafted tokens from draft row drow on), by one wavefront; lane 0 holds the
// token's NLL and weight.
__device__ inline LossRow make_loss_row(const LossArgs& a, int row, int kind, int drow, int L, int t, float T, float Td, int lane,
                                        double* nll, double* weight) {
  LossRow R;
  R.t_ng = -1; R.t_pre = -1; R.pi = 0.0; R.q_pre = 0.0; R.ln_pi = 0.0; R.ln_q_pre = 0.0;
  R.invT = 1.0 / (double)T; R.invTd = 1.0 / (double)Td;
  const int dr = drow + min(lane, L - 1);               // lane l: sub-token l
  const int id = a.draft_ids[dr];
  const double mxq = (double)a.drow_max[dr], Sq = a.drow_sum[dr];
  R.mx = (double)a.row_max[row]; R.lnS = log(a.row_sum[row]);
  const double lnSq = log(Sq);
  R.mxq = __shfl(mxq, 0); R.lnSq = __shfl(lnSq, 0);
  *nll = 0.0; *weight = 0.0;
  if (kind == 2) {                                      // wavefront-uniform
    const int d1 = __shfl(id, 0);
    const int t_pre = a.dmap[d1];
    const double lq = ((double)draft_logit(a, dr, id) - mxq) * R.invTd - lnSq;
    const double lq_first = __shfl(lq, 0);
    double lq_sum = 0.0;
    for (int l = 0; l < L; ++l) lq_sum += __shfl(lq, l);
    *nll = -lq_sum;
    *weight = a.lambda_mode == OT_LAMBDA_TARGET_PROB ? (double)a.p_tok[row] : (double)a.lambda;
    // Eq. 2's overrides for this n-gram
    R.t_ng = t;
    R.pi = exp(lq_sum); R.ln_pi = lq_sum;
    R.t_pre = t_pre;
    R.q_pre = exp(lq_first) - R.pi;
    R.ln_q_pre = R.q_pre > 0.0 ? log(R.q_pre) : 0.0;
  }
  return R;
}

// Sum of x over the workgroup in a fixed order, valid in thread 0.
template <int kWaves>
__device__ inline double block_sum(double x, double* s_w, int wave, int lane) {
  x = wave_sum(x);
  if (lane == 0) s_w[wave] = x;
  __syncthreads();
  double total = 0.0;
  if (wave == 0) total = wave_sum(lane < kWaves ? s_w[lane] : 0.0);
  return total;
}

// The sums over all rows and the mean over the drafted tokens considered.  Everything about a few rows is asked for before any
// of it is looked at: one round trip to memory for four rows per thread.
template <int kWaves>
__device__ inline void loss_totals(const LossArgs& a, double (*s_term)[kWaves], int tid, int wave, int lane) {
  constexpr int kAtOnce = 4, kThreads = 64 * kWaves;
  double term[4] = {0.0, 0.0, 0.0, 0.0};                // direct, n-gram, direct tokens, n-gram sub-tokens
  double* other = a.ngram_term == OT_NGRAM_TERM_APPROX_KL ? a.out.kl : a.out.nll;
  for (int row0 = tid; row0 < a.M; row0 += kAtOnce * kThreads) {
    int kind[kAtOnce], len[kAtOnce];
    double kl[kAtOnce], x[kAtOnce], weight[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int row = min(row0 + j * kThreads, a.M - 1);
      kind[j] = observe(a.out.kind + row);
      kl[j] = observe(a.out.kl + row);
      x[j] = observe(other + row);
      weight[j] = observe(a.out.weight + row);
      len[j] = a.span_len[row];
    }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      if (row0 + j * kThreads >= a.M) break;
      if (kind[j] == 1) {
        term[0] += kl[j];
        term[2] += 1.0;
      } else if (kind[j] == 2) {
        term[1] += weight[j] * x[j];
        term[3] += (double)len[j];
      }
    }
  }
  double t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    t[i] = wave_sum(term[i]);
    if (lane == 0) s_term[i][wave] = t[i];
  }
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = wave_sum(lane < kWaves ? s_term[i][lane] : 0.0);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) a.out.totals[i] = t[i];
    a.out.totals[4] = (t[0] + t[1]) / fmax(1.0, t[2] + t[3]);
  }
}

// Terms i = first + e * kThreads of n: mapped pairs in ascending target id, or every target id with its pre-image (past the
// end the last one, masked later).
template <int kThreads>
__device__ inline void load_terms(const LossArgs& a, bool pairs, int n, int first, int2* id) {
  if (n == 0) {                                          // nothing is mapped
#pragma unroll
    for (int e = 0; e < kPerTurn; ++e) id[e] = make_int2(0, -1);
  } else if (pairs) {
#pragma unroll
    for (int e = 0; e < kPerTurn; ++e) id[e] = a.pairs[min(first + e * kThreads, n - 1)];
  } else {
#pragma unroll
    for (int e = 0; e < kPerTurn; ++e) {
      const int v = min(first + e * kThreads, n - 1);
      id[e] = make_int2(v, a.tmap[v]);
    }
  }
}

// Row offsets of a few sequences as a kernel argument (the host has them); of more they come from memory, another round trip (256 of
// them as an argument cost every call 0.3 us on the host).
constexpr int kArgumentB = 31;
struct LossRowOffsets { int32_t v[kArgumentB + 1]; };

// Grid: the workgroups of a row (`groups` of them) run on one XCD back to back, so that they meet in its L2, where a draft row that
// is gathered from memory stays while they do.  seq_rows > 0: places of seq_rows rows for every sequence, of which those past its
// window end at once; a workgroup then knows its sequence and row without a load, and everything else about them comes with one
// round trip of scalar loads, which do not wait behind the vector loads of its terms.  Most rows of a batch have no token with a KL
// term, and what their workgroups take to find that out the others wait for (6.7 us of 21 with the row's sequence looked up behind
// the first turn's loads, and what hangs on it loaded after that).  A sequence's last row never has a token: the
// place in front of it takes it along (16 windows of 8 tokens then are 512 workgroups, all on the chip at once, and not 576).
// 0: the rows one after the other: ragged windows that would leave most places empty, and where the q' rows are wanted, which
// every row's workgroups write (us per call, rows / places: 16 windows of 1 to 10 tokens x 50257 ids 20.2 / 20.9, 48 of them 35.2 / 36.7).
// n_arrivals: rows, or places with a row, that are counted in.
template <int kThreads>
__global__ __launch_bounds__(kThreads, 4) void loss_kernel(LossArgs a, LossRowOffsets ro, int seq_rows, int n_arrivals, int groups,
                                                          int group_terms, int staged) {
  constexpr int kWaves = kThreads / 64;
  __shared__ LossRow s_row;
  __shared__ double s_term[4][kWaves];
  __shared__ int s_last;
  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  const int slot = (int)blockIdx.x >> 3, place = slot / groups * 8 + ((int)blockIdx.x & 7), grp = slot % groups;
  if (a.M == 0) {                                        // an empty batch
    if (blockIdx.x == 0) loss_totals<kWaves>(a, s_term, tid, wave, lane);
    return;
  }
  int b, r0, row;
  bool free_row = false;                                 // row + 1 is the sequence's last
  if (seq_rows > 0) {
    b = place / seq_rows;
    if (b >= a.B) return;                                // padding of the id space
    const bool argument = a.B <= kArgumentB;
    r0 = argument ? ro.v[b] : a.row_off[b];
    const int rows = (argument ? ro.v[b + 1] : a.row_off[b + 1]) - r0, at = place % seq_rows;
    if (at >= max(rows - 1, 1)) return;                  // past the sequence's window
    row = r0 + at;
    free_row = at == rows - 2;
  } else {
    row = place;
    if (row >= a.M) return;
    b = find_sequence(a.row_off, a.B, row, 0, lane);
    r0 = a.row_off[b];
  }
  b = uniform(b); row = uniform(row);
  const int j = row - r0;
  const int s = a.span_start[row], L = a.span_len[row], t = a.mapped_ids[row];
  const float T = a.temperature[b];
  const float Td = a.draft_temperature ? a.draft_temperature[b] : T;
  const int n_mapped = a.n_mapped[b], n_accept = a.n_accept[b];
  const bool pairs = a.out.qprime == nullptr;            // terms: the mapped pairs, or (q' is wanted everywhere) all ids
  const int n_terms = pairs ? a.n_pairs : a.V_t;
  const int i0 = grp * group_terms, i1 = min(i0 + group_terms, n_terms);
  // the first turn's ids depend on nothing else
  const float* z = a.Z + (int64_t)row * a.ldz;
  int2 id[kPerTurn], id_next[kPerTurn] = {};             // (target id, draft id or -1)
  float zv[kPerTurn];
  load_terms<kThreads>(a, pairs, n_terms, i0 + tid, id);
  if (i0 + kPerTurn * kThreads < i1) load_terms<kThreads>(a, pairs, n_terms, i0 + tid + kPerTurn * kThreads, id_next);
  int kind = 0;
  if (j < n_mapped && T > 0.f && Td > 0.f) kind = L == 1 ? 1 : (!a.accepted_only || j < n_accept) ? 2 : 0;
  kind = uniform(kind);
  const bool need_kl = kind == 1 || (kind == 2 && a.ngram_term == OT_NGRAM_TERM_APPROX_KL);
  const bool visit = need_kl || (kind != 0 && a.out.qprime != nullptr);
  float* qprime = a.out.qprime ? a.out.qprime + (int64_t)row * a.V_t : nullptr;
  if (!visit && qprime)                                  // a row without a token exports zeros
    for (int v = i0 + tid; v < i1; v += kThreads) qprime[v] = 0.f;
  if (!visit && grp != 0) return;
#pragma unroll
  for (int e = 0; e < kPerTurn; ++e) zv[e] = z[id[e].x];
  const int drow = uniform(r0 - b + (kind != 0 ? s : 0));
  const char* zq = static_cast<const char*>(a.draft_logits) + (size_t)drow * a.V_d * (a.dtype == OT_BF16 ? 2 : 4);
  if (wave == 0) {
    double nll = 0.0, weight = 0.0;
    if (kind != 0) {
      const LossRow R = make_loss_row(a, row, kind, drow, uniform(L), t, T, Td, lane, &nll, &weight);
      if (lane == 0) s_row = R;
    }
    if (grp == 0 && lane == 0) {
      publish(a.out.kind + row, kind);
      publish(a.out.nll + row, nll);
      publish(a.out.weight + row, weight);
      if (free_row) {
        publish(a.out.kind + row + 1, 0);
        publish(a.out.nll + row + 1, 0.0);
        publish(a.out.weight + row + 1, 0.0);
        publish(a.out.kl + row + 1, 0.0);
      }
    }
  }
  double kl = 0.0;
  if (visit) {
    int lds_at = -1;
    if (staged && wave > 0) lds_at = stage_draft_row<kThreads - 64>(zq, a.dtype, a.V_d, tid - 64, 0);
    if (staged && wave == 0) lds_at = (int)(reinterpret_cast<uintptr_t>(zq) & 15);   // where that starts the copy
    __syncthreads();
    const LossRow R = s_row;
    const bool plain_row = pairs && uniform(R.t_ng & R.t_pre) < 0;   // neither override (-1 both)
    for (int at = i0 + tid; at - tid < i1; at += kPerTurn * kThreads) {
      uint32_t xq[kPerTurn];
      int dv[kPerTurn];
#pragma unroll
      for (int e = 0; e < kPerTurn; ++e) dv[e] = id[e].y;
      load_draft_logits<kPerTurn>(zq, a.dtype, lds_at, dv, xq);
      float z_next[kPerTurn] = {};                       // asked for behind what this turn waits for, its ids a turn earlier
      int2 id_after[kPerTurn] = {};
      if (at - tid + kPerTurn * kThreads < i1) {
#pragma unroll
        for (int e = 0; e < kPerTurn; ++e) z_next[e] = z[id_next[e].x];
      }
      if (at - tid + 2 * kPerTurn * kThreads < i1) load_terms<kThreads>(a, pairs, n_terms, at + 2 * kPerTurn * kThreads, id_after);
      // kPlain: mapped pairs, all of the turn's terms exist, no override among the row's ids
      auto add_terms = [&](auto plain) {
        constexpr bool kPlain = decltype(plain)::value;
#pragma unroll
        for (int e = 0; e < kPerTurn; ++e) {
          const int v = id[e].x;
          double q = 0.0, lq = 0.0;
          if (kPlain || dv[e] >= 0) {
            lq = ((double)__uint_as_float(a.dtype == OT_BF16 ? xq[e] << 16 : xq[e]) - R.mxq) * R.invTd - R.lnSq;
            q = exp_neg_fast(lq);
          }
          if (!kPlain && v == R.t_pre) { q = R.q_pre; lq = R.ln_q_pre; }
          if (!kPlain && v == R.t_ng) { q = R.pi; lq = R.ln_pi; }   // the n-gram case of Eq. 2 wins when both name the same id
          const double lp = ((double)zv[e] - R.mx) * R.invT - R.lnS;
          if ((kPlain || at + e * kThreads < i1) && q > 0.0) kl += q * (lq - lp);
          if (!kPlain && qprime && at + e * kThreads < i1) qprime[v] = (float)q;
        }
      };
      if (plain_row && at - tid + kPerTurn * kThreads <= i1) add_terms(std::true_type());   // workgroup-uniform
      else add_terms(std::false_type());
#pragma unroll
      for (int e = 0; e < kPerTurn; ++e) { id[e] = id_next[e]; id_next[e] = id_after[e]; zv[e] = z_next[e]; }
    }
    // the n-gram's target id, where it is no draft id's image and so in no pair
    if (pairs && grp == 0 && tid == 0 && R.t_ng >= 0 && a.tmap[R.t_ng] < 0 && R.pi > 0.0)
      kl += R.pi * (R.ln_pi - (((double)z[R.t_ng] - R.mx) * R.invT - R.lnS));
    kl = need_kl ? block_sum<kWaves>(kl, s_term[0], wave, lane) : 0.0;
  }
  if (wave == 0) {
    bool row_done = need_kl || grp == 0;
    if (need_kl && groups > 1) {
      double* part = a.part + (int64_t)row * groups;
      int last = 0;
      if (lane == 0) {
        publish(part + grp, kl);
        last = arrive(a.count + 1 + row, groups);
      }
      row_done = uniform(last) != 0;
      kl = row_done ? wave_sum(lane < groups ? observe(part + lane) : 0.0) : 0.0;   // a wavefront holds all groups
    }
    if (lane == 0) {
      s_last = 0;
      if (row_done) {
        publish(a.out.kl + row, need_kl ? kl : 0.0);
        s_last = arrive(a.count, n_arrivals);
      }
    }
  }
  __syncthreads();
  if (s_last) loss_totals<kWaves>(a, s_term, tid, wave, lane);
}

// How a launch is split: threads per workgroup, the draft row in LDS or gathered from memory, groups of terms per row.  A
// workgroup is a chain of about eight round trips, so a compute unit should hold several: 126 registers leave room for sixteen
// wavefronts, the copies of the draft row for as many workgroups as fit into LDS: four of 256 threads up to 40 KB, two of 512
// up to 78 KB, one of 1024 up to 150 KB.  Above that the logits are gathered, and where a row's logits lie in the order of its terms
// (`local`: one vocabulary on both sides, or nearly) already from 78 KB on: neighbouring lanes then read the same line.  Gathered
// at random, a row has to stay in the L2 of its XCD (4 MB) while its workgroups are at it: enough groups per row that the 128
// workgroups which the XCD holds work on 2 MB of rows.  Otherwise as many groups as fill the chip, and no more than eight turns
// in one where nothing was copied.
// Measured, us per call (1024 threads, at most 16 groups | four launches | now): 144 rows x 128256 ids with 32000 draft ids
// 24.3 | 42.8 | 21.5, 432 rows x 152064 53 | 100 | 45; 1024 rows x 5000 with 2000 37.5 | 25.7 | 17.9; 1200 x 32000 with 32000
// 97 | 77 | 78.5; fp32, 1024 x 32000 with 32000 in order 87 | 65 | 66; fp32, 60000 draft ids at random, 432 rows 167 | 107 | 89, 1024
// rows 477 | 276 | 282.  Still behind the four launches, whose constants were formed once a row: 1200 rows x 600 ids 43 | 20 | 23.
struct LossPlan { int threads, staged, groups, group_terms; };
LossPlan loss_plan(int M, int n_terms, int64_t row_bytes, bool local, int n_cu) {
  LossPlan p;
  p.staged = row_bytes <= (local ? 78 << 10 : (int64_t)kDrawLdsBytes);
  p.threads = !p.staged || row_bytes <= 40 << 10 ? 256 : row_bytes <= 78 << 10 ? 512 : 1024;
  const int turn = kPerTurn * p.threads;
  int want = ceil_div((int64_t)(1024 / p.threads) * n_cu, std::max(M, 1));
  if (!p.staged) want = std::max(want, ceil_div(n_terms, 8 * turn));
  if (!p.staged && !local) want = std::max(want, (int)std::min<int64_t>(kLossGroups, 128 * row_bytes / (2 << 20)));
  const int turns = std::max(1, ceil_div(n_terms, (int64_t)std::max(1, std::min({kLossGroups, ceil_div(n_terms, turn), want})) * turn));
  p.group_terms = turns * turn;
  p.groups = std::max(1, ceil_div(n_terms, p.group_terms));
  return p;
}

}  // namespace
}  // namespace otv

using namespace otv;

#pragma GCC visibility push(default)
extern "C" {

int ot_distill_loss(ot_ctx* ctx, const ot_step_in* in, const ot_step_out* step, const float* target_logits,
                    const ot_loss_config* cfg, ot_loss_out* out) {
  if (!ctx || !in || !step || !cfg || !out) return ot_fail(OT_ERR_NULL, "ot_distill_loss: ctx, in, step_out, cfg and out must not be NULL");
  if (cfg->lambda_mode != OT_LAMBDA_FIXED && cfg->lambda_mode != OT_LAMBDA_TARGET_PROB)
    return ot_fail(OT_ERR_SHAPE, "ot_distill_loss: unknown lambda_mode %d", cfg->lambda_mode);
  if (cfg->ngram_term != OT_NGRAM_TERM_NLL && cfg->ngram_term != OT_NGRAM_TERM_APPROX_KL)
    return ot_fail(OT_ERR_SHAPE, "ot_distill_loss: unknown ngram_term %d", cfg->ngram_term);
  if (in->B < 0 || in->B > ctx->max_batch) return ot_fail(OT_ERR_SHAPE, "ot_distill_loss: B = %d exceeds max_batch = %d", in->B, ctx->max_batch);
  if (!out->kind || !out->kl || !out->nll || !out->weight || !out->totals)
    return ot_fail(OT_ERR_NULL, "ot_distill_loss: kind, kl, nll, weight and totals are required");
  if (in->B > 0) {
    if (!in->row_off || !in->row_off_host || !in->temperature)
      return ot_fail(OT_ERR_NULL, "ot_distill_loss: row_off, row_off_host and temperature must not be NULL");
    if (!step->n_mapped || !step->n_accept || !step->mapped_ids || !step->span_start || !step->span_len || !step->p_tok)
      return ot_fail(OT_ERR_NULL, "ot_distill_loss: the step's n_mapped, n_accept, mapped_ids, span_start, span_len and p_tok are required");
    if (in->row_off_host[0] != 0) return ot_fail(OT_ERR_SHAPE, "ot_distill_loss: row_off[0] must be 0");
    for (int b = 0; b < in->B; ++b) {
      const int64_t rows = (int64_t)in->row_off_host[b + 1] - in->row_off_host[b];
      if (rows < 1 || rows - 1 > ctx->max_k) return ot_fail(OT_ERR_SHAPE, "ot_distill_loss: sequence %d owns %lld rows", b, (long long)rows);
    }
  }
  const int M = in->B > 0 ? in->row_off_host[in->B] : 0;
  if (M - in->B > 0 && (!in->draft_logits || !in->draft_ids)) return ot_fail(OT_ERR_NULL, "ot_distill_loss: draft_logits and draft_ids must not be NULL");

  LossArgs a{};
  a.B = in->B; a.M = M; a.V_t = ctx->V_t; a.V_d = ctx->V_d; a.dtype = ctx->dtype;
  a.row_off = in->row_off; a.temperature = in->temperature; a.draft_temperature = in->draft_temperature;
  a.draft_logits = in->draft_logits; a.draft_ids = in->draft_ids; a.dmap = ctx->dmap; a.tmap = ctx->tmap; a.pairs = ctx->pairs; a.n_pairs = ctx->n_pairs;
  a.Z = target_logits ? target_logits : ctx->Z; a.ldz = ctx->V_t;
  a.row_max = ctx->row_max; a.row_sum = ctx->row_sum; a.drow_max = ctx->drow_max; a.drow_sum = ctx->drow_sum;
  a.n_mapped = step->n_mapped; a.n_accept = step->n_accept; a.mapped_ids = step->mapped_ids;
  a.span_start = step->span_start; a.span_len = step->span_len; a.p_tok = step->p_tok;
  a.lambda = cfg->lambda; a.lambda_mode = cfg->lambda_mode; a.ngram_term = cfg->ngram_term; a.accepted_only = cfg->accepted_only != 0;
  a.part = ctx->loss_part; a.count = ctx->loss_count;
  a.out = *out;

  hipStream_t st = ctx->stream;
  const int n_terms = out->qprime ? a.V_t : a.n_pairs;
  const int64_t row_bytes = (int64_t)a.V_d * (a.dtype == OT_BF16 ? 2 : 4) + 32;
  const LossPlan p = loss_plan(M, n_terms, row_bytes, ctx->local_pairs, ctx->n_cu);
  LossRowOffsets ro{};
  int seq_rows = 0, n_places = 0;                        // of the longest window
  for (int b = 0; b < in->B; ++b) {
    const int n = std::max(1, in->row_off_host[b + 1] - in->row_off_host[b] - 1);
    seq_rows = std::max(seq_rows, n);
    n_places += n;
  }
  if (out->qprime || (int64_t)seq_rows * in->B > 2 * (int64_t)n_places) seq_rows = 0;
  const int n_arrivals = seq_rows > 0 ? n_places : M;
  for (int b = 0; b <= in->B && in->B > 0 && in->B <= kArgumentB; ++b) ro.v[b] = in->row_off_host[b];
  const int places = seq_rows > 0 ? seq_rows * in->B : std::max(M, 1);
  const dim3 grid((unsigned)(p.groups * ceil_div(places, 8) * 8)), block(p.threads);
  const size_t lds = p.staged ? row_bytes : 16;
  const auto kernel = p.threads == 1024 ? loss_kernel<1024> : p.threads == 512 ? loss_kernel<512> : loss_kernel<256>;
  hipLaunchKernelGGL(kernel, grid, block, lds, st, a, ro, seq_rows, n_arrivals, p.groups, p.group_terms, p.staged);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return ot_fail_hip(e, "ot_distill_loss: launch");
  return OT_OK;
}

}  // extern "C"
#pragma GCC visibility pop
