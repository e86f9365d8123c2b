// The launches that draw the final token of every sequence (Algorithm 1: correction token from the residual of Eq. 2,
// or free token from p), grid = (groups of units of target ids) x (sequences).
//   final_draw_kernel   the outcome records of the acceptance test are in memory (written by the launch before).
//   accept_draw_kernel  follows the launch that did the draft side and the softmax partials, the LM head's or the
//                       statistics launch: every workgroup first repeats the translation and the acceptance test of its
//                       sequence (one wavefront merges the partials of the draft rows and walks the window from the
//                       probe record while the others merge the target rows' partials, one wavefront per row; then that
//                       wavefront runs the test: a few microseconds of work on data that sits in L2, cheaper than a
//                       launch of its own: with an earlier draw 300 sequences x 32003 ids took 42 us against 10.5 + 30.6
//                       and a launch; all of it takes 21 now), then takes part in the draw.  The workgroups of
//                       a sequence reach the same outcome; only group 0 writes the outputs of the translation and the
//                       test, the draft rows' merged statistics and the cache's use statistics.
#include <algorithm>

#include "accept.h"
#include "resid.h"

namespace otv {
namespace {

template <int kPer, bool kBlocks, bool kExps>
__global__ __launch_bounds__(kDrawWaves * 64) void final_draw_kernel(StepArgs a, DrawSplit s) {
  const int b = blockIdx.y, grp = blockIdx.x, tid = threadIdx.x;
  const int wave = uniform(tid >> 6), lane = tid & 63;
  __shared__ DrawLds s_draw;
  int dv[kPer];
  const int first = draw_first_id<kPer, kBlocks>(s, grp, wave);
  load_tmap<kPer>(a.tmap, a.V_t, first + lane, 64, first + 64 * kPer <= a.V_t, dv);   // overlaps the next load
  const FinalInfo f = a.fin[b];
  if (f.mode == 0) return;                  // greedy or flagged sequence: nothing to draw
  draw_final_token<kPer, kBlocks, kDrawWaves, kExps>(a, b, grp, s, f, dv, &s_draw);
}

// Row offsets of up to kFusedMaxB sequences as a kernel argument (the host has them): the workgroup knows its rows without
// a dependent load in front of everything else.  With more sequences they come from memory.
struct RowOffsets { int32_t v[kFusedMaxB + 1]; };
constexpr int64_t kRepeatedMergeBytes = 32 << 20;

// kDraw = false: grid = (1) x (sequences); the workgroup only runs the test and leaves the outcome record in memory for
// a final_draw_kernel launch (used when repeating the test in every group of units would cost more than a launch).
// kChunks: the partials come from the statistics launch (chunk partials in three arrays per side) instead of the
// LM head's epilogue and draft-row pieces; kFused as well: only the draft rows' do.
// kMany: more than kFusedMaxB sequences: row offsets from memory, partials merged in binary64 (as a runtime flag these two
// cost a single sequence 0.7 of 13 us).
// kWide: draft rows of more than kChunksAtOnce chunks (merge_draft_chunks).
// kBlocks: units of several blocks (draw_split).
// kExps: a draw with the draft row's exponentials in LDS (launch_draw).  As a runtime flag it cost the others 0.5 to 0.9 us of 10 to 12
// (112 registers instead of 94).
template <int kPer, bool kDraw, bool kChunks, bool kMany = false, bool kWide = kMany, bool kFused = !kChunks, bool kBlocks = false,
          int kWaves = kDrawWaves, bool kExps = false>
__global__ __launch_bounds__(kWaves * 64) void accept_draw_kernel(StepArgs a, RowOffsets ro, DrawSplit split) {
  const int b = blockIdx.y, grp = blockIdx.x, tid = threadIdx.x;
  const int wave = uniform(tid >> 6), lane = tid & 63;
  __shared__ DrawLds s_draw;
  __shared__ FinalInfo s_fin;
  __shared__ float s_pmx[64];
  __shared__ double s_pinv[64];
  __shared__ int s_parg[64];
  int dv[kPer];

  const int r0 = kMany ? a.row_off[b] : ro.v[b];
  const int k = (kMany ? a.row_off[b + 1] : ro.v[b + 1]) - r0 - 1;
  const float T = a.temperature[b];
  const float Td = a.draft_temperature ? a.draft_temperature[b] : T;
  const uint64_t sid = a.seq_id[b];
  const bool lead = grp == 0;               // the group that writes the test's outputs and the row statistics

  // The LM-head launch left what the drafted ids look up (ProbeRecord) and the draft rows' statistics.  The last
  // wavefront fetches them (one load of each array per lane), walks the window (Eq. 1), asks for the logits of the
  // proposed tokens and forms q' while they are on their way, all on its own, while the other wavefronts merge the softmax
  // partials of the target rows; the translation is thus repeated by every group of the sequence, and the lead group
  // writes its outputs and the cache's use statistics.  That wavefront's chain of round trips and binary64 functions is what
  // the others wait for: its loads leave before anything is known about the temperature, the walk comes before the functions,
  // and q' is formed once as a product instead of through the logarithms of its factors (from the launch's start to the
  // outcome 5.4 -> 2.7 us for one sequence of five drafted ids).
  const int q0 = r0 - b;
  constexpr int kTestWave = kWaves - 1;   // runs the walk and the test
  Window W;
  DraftLane D;
  float z_tok = 0.f;
  bool bad = false, reached = false;
  int pos = 0;
  double u1 = 0.0;
  double invT = 1.0;
  uint32_t rnd[4] = {0, 0, 0, 0};             // of row `lane`: word 0 tests that mapped position, word 1 draws its final token
  Scale sc{}, scq{};
  if (wave == kTestWave) {
    const ProbeRecord* rec = a.probe + b;
    const unsigned long long hit = rec->hit[lane];
    D.dm = rec->dm[lane];
    bad = rec->bad != 0;                      // wavefront-uniform
    D.zq = rec->zq[lane];
    D.mxq = 0.f; D.Sq = 1.0; D.argq = -1;
    DraftPartials<kChunks> part;
    if (lane < k) part.load(a, q0 + lane);
    if (T > 0.f) philox4x32_10((uint32_t)lane, a.step, (uint32_t)sid, (uint32_t)(sid >> 32), (uint32_t)a.seed, (uint32_t)(a.seed >> 32), rnd);
    invT = T > 0.f ? 1.0 / (double)T : 1.0;
    const double invTd = Td > 0.f ? 1.0 / (double)Td : 1.0;
    sc = split_scale(invT); scq = split_scale(invTd);
    W = walk_window(k, lane, hit, D.dm);
    reached = ((W.starts >> lane) & 1ull) != 0ull;
    pos = __popcll(W.starts & bits_below(lane));
    if (reached) z_tok = a.Z[(int64_t)(r0 + pos) * a.ldz + W.t];
    u1 = u24(__shfl(rnd[0], pos));
    if (lane < k) {
      if constexpr (kChunks) merge_draft_chunks<kWide>(a, q0 + lane, Td, invTd, part, &D.mxq, &D.Sq, &D.argq, kMany);
      else merge_draft_pieces(a, q0 + lane, Td, part, &D.mxq, &D.Sq, &D.argq);
      if (lead) { a.drow_max[q0 + lane] = D.mxq; a.drow_sum[q0 + lane] = D.Sq; a.drow_arg[q0 + lane] = D.argq; }
    }
    D.invSq = 1.0 / D.Sq;
    D.q = Td > 0.f ? exp(((double)D.zq - (double)D.mxq) * invTd) * D.invSq : 0.0;
    if (!(Td > 0.f) && lane < k) D.q = a.draft_ids[q0 + lane] == D.argq ? 1.0 : 0.0;
    D.qp = segment_q(D.q, W);
  }
  if (kMany && wave != kTestWave) invT = T > 0.f ? 1.0 / (double)T : 1.0;
  for (int row = wave; row <= k; row += kWaves) {
    if (!kFused)
      merge_chunk_row(a.tpart_max, a.tpart_sum, a.tpart_arg, a.ncht, r0 + row, T, invT, lane, s_pmx, s_pinv, s_parg, row, lead,
                      a.row_max, a.row_sum, a.row_arg, kMany);
    else
      merge_fused_row(a.fused.part, a.fused.nfine, r0 + row, T, lane, s_pmx, s_pinv, s_parg, row, lead, a.row_max,
                      a.row_sum, a.row_arg);
  }
  if (!(T > 0.f) && !lead) return;            // a greedy sequence draws nothing: its other groups have nothing to do
  // The inverse map of this wavefront's ids is needed last (by the masses) and asked for here, behind the loads
  // that the test waits for: loads return in issue order, and asked for first it held those back by its own latency.
  const int first = draw_first_id<kPer, kBlocks>(split, grp, wave);
  if (kDraw) load_tmap<kPer>(a.tmap, a.V_t, first + lane, 64, first + 64 * kPer <= a.V_t, dv);
  __syncthreads();
  Outcome O;
  if (wave == kTestWave) {
    FinalInfo fin{};                          // mode 0: nothing to draw
    if (!bad) {
      O = test_window(T, invT, W, D, reached, pos, z_tok, u1, s_pmx, s_pinv, s_parg);
      fin = final_info(r0, q0, T, Td, sc, scq, W, D, O, u24((uint32_t)__builtin_amdgcn_readlane((int)rnd[1], O.n)), s_pmx, s_pinv);
    }
    if (lane == 0) s_fin = fin;
    if (!kDraw && lane == 0) a.fin[b] = fin;
  }
  if (kDraw) __syncthreads();
  if (wave == kTestWave && lead) {            // behind the barrier: nobody in this launch waits for these
    if (bad) {
      write_bad_sequence(a, b, r0, k, lane);
    } else {
      write_translation(a, b, r0, k, lane, W, reached, pos, D.qp, !(T > 0.f));
      write_outcome(a, b, r0, k, lane, T, W, O, reached, pos, s_parg);
    }
  }
  if (!kDraw) return;
  const FinalInfo f = s_fin;
  if (f.mode == 0) return;
  draw_final_token<kPer, kBlocks, kWaves, kExps>(a, b, grp, split, f, dv, &s_draw);
}

// Units of the draw and their share per workgroup.  While no more than a workgroup per compute unit is needed for one turn each,
// a wavefront takes as few ids as that allows: 128 (up to 512 units), else 256, else 512.  A
// small batch is bound by the chain of instructions and round trips in one workgroup, which fewer ids per lane shorten.  With
// more groups than compute units a sequence has as many groups as leave no more than one workgroup per compute unit (up to 112
// registers: a second of 16 wavefronts does not fit): its start, its share of the merge and its look at the masses are then paid once
// for several turns, and a turn's loads overlap the sums of the turn before.  (As many turns as brought the number of groups back
// to one per compute unit, rounded up, left 200 sequences x 128256 ids with two groups, 368 workgroups: 104 us per step from the logits
// where one group each takes 65.)
// With more sequences than compute units a sequence has one workgroup.  Two of 8 wavefronts on a compute unit then take 300
// sequences at once, where 16 wavefronts take 256 and then 44: what the 8 in a workgroup need for all turns is hardly more than what 16
// need, as the loads bound both.  Taken where half of LDS holds the draft row's exponentials: 300 / 512 / 700 sequences x 32003 ids, us per
// step from the logits with 16 / 8 wavefronts 43.7 / 38.1, 55.3 / 48.7, 75.3 / 69.1; 300 x 128256 109 / 108; with rows that do not fit
// (32000 fp32 ids) 51.7 / 88.7.
// Measured, us per step, 128 / 256 / 512 ids a wavefront: 6 rows x 32000 ids 53.9 / 54.1 / 55.2, 12 rows x 64000 (d = 1024) 39.4 /
// 40.1 / 42.6, 24 x 152064 -- / 180.8 / 182.0, 80 x 32000 66.7 / 66.2 / 68.1, 6 x 152064 (d = 1024) -- / 69.2 / 70.7.
// Above 4096 units of 512 ids a unit is as many blocks of 512 as leave no more than that, and a sequence's masses 33 KB of LDS at
// any vocabulary (a mass for every 1024 ids filled LDS at 20 million).  Against units of 1024 ids with 16 a lane, which spilled 20
// registers, us per step from the logits: 16 sequences of 2.2 million ids 116 -> 103, of 9 million 401 -> 344, one of 4.2 million
// 27.3 -> 28.1.
constexpr int kMaxUnits = 4096;
template <int kPer> DrawSplit draw_split(int V_t, int B, int n_cu, int waves = kDrawWaves) {
  DrawSplit s;
  s.n_units = ceil_div(V_t, 64 * kPer);
  s.blocks = kPer == 8 ? ceil_div(s.n_units, kMaxUnits) : 1;
  s.n_units = ceil_div(s.n_units, s.blocks);
  // as many groups a sequence as bring the workgroups to what the chip holds at once
  const int groups = std::max(1, std::max(n_cu, 1) * (kDrawWaves / waves) / std::max(B, 1));
  s.group_units = ceil_div(ceil_div(s.n_units, groups), waves) * waves;
  s.row_at = 0;
  s.exps = false;
  return s;
}

size_t draw_lds_bytes(const DrawSplit& s) { return (size_t)(draw_lds_doubles(s.n_units) + 1) / 2 * 2 * sizeof(double); }

// ids per lane, their split, wavefronts per workgroup
struct DrawPlan { int per; DrawSplit split; int waves; };
DrawPlan draw_plan(int V_t, int V_d, int B, int n_cu) {
  const DrawSplit two = draw_split<2>(V_t, B, n_cu), four = draw_split<4>(V_t, B, n_cu);
  if (two.group_units == kDrawWaves && two.n_units <= 512 && B <= kFusedMaxB) return {2, two, kDrawWaves};
  if (four.group_units == kDrawWaves && B <= kFusedMaxB) return {4, four, kDrawWaves};
  const DrawSplit eight = draw_split<8>(V_t, B, n_cu);
  if (B > n_cu && B > kFusedMaxB && eight.blocks == 1 && draw_lds_bytes(eight) + exps_bytes(V_d) <= kDrawLdsBytes / 2)
    return {8, draw_split<8>(V_t, B, n_cu, 8), 8};
  return {8, eight, kDrawWaves};
}

// Every group of units of a sequence repeats the merge of its rows' partials: M x nfine x 16 bytes per group.  Up to
// about the traffic that costs as much as a launch this is one launch; beyond it the test gets a launch of its own.  (A few chunks
// of the statistics launch per row: always one.)
bool test_has_its_launch(int hosted, int nfine, int M, const DrawSplit& s) {
  return hosted != kHostsNothing && (int64_t)M * nfine * (int64_t)sizeof(Partial) * ceil_div(s.n_units, s.group_units) > kRepeatedMergeBytes;
}

// What was left by which launch: see StepArgs::hosted.
template <int kPer, bool kBlocks, int kWaves, bool kExps>
hipError_t launch_draw_kernels(const StepArgs& a, const RowOffsets& ro, const DrawSplit& s, dim3 grid, size_t lds, hipStream_t stream) {
  const dim3 block(kWaves * 64);
  auto test_and_draw = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, stream, a, ro, s); };
  if (a.B > kFusedMaxB) {
    if (a.hosted != kHostsNothing) return hipErrorInvalidValue;
    if constexpr (kPer == 8) test_and_draw(accept_draw_kernel<kPer, true, true, true, true, false, kBlocks, kWaves, kExps>);
    else return hipErrorInvalidValue;
  } else if constexpr (kWaves != kDrawWaves) {
    return hipErrorInvalidValue;                         // see draw_plan
  } else if (a.hosted == kHostsNothing) {
    if (a.nchd > kChunksAtOnce) test_and_draw(accept_draw_kernel<kPer, true, true, false, true, false, kBlocks, kWaves, kExps>);
    else test_and_draw(accept_draw_kernel<kPer, true, true, false, false, false, kBlocks, kWaves, kExps>);
  } else if (!test_has_its_launch(a.hosted, a.fused.nfine, a.M, s)) {
    if (a.hosted == kHostsAll) test_and_draw(accept_draw_kernel<kPer, true, false, false, false, true, kBlocks, kWaves, kExps>);
    else test_and_draw(accept_draw_kernel<kPer, true, true, false, true, true, kBlocks, kWaves, kExps>);
  } else {
    const auto test = a.hosted == kHostsAll ? accept_draw_kernel<8, false, false> : accept_draw_kernel<8, false, true, false, true, true>;
    hipLaunchKernelGGL(test, dim3(1, a.B), block, 0, stream, a, ro, s);
    hipLaunchKernelGGL((final_draw_kernel<kPer, kBlocks, kExps>), grid, block, lds, stream, a, s);
  }
  return hipGetLastError();
}

// row_off_host holds the B + 1 row offsets.
template <int kPer, bool kBlocks = false, int kWaves = kDrawWaves>
hipError_t launch_draw(const StepArgs& a, const int32_t* row_off_host, const DrawSplit& split, hipStream_t stream) {
  constexpr size_t kLdsBytes = kWaves == kDrawWaves ? kDrawLdsBytes : kDrawLdsBytes / 2;
  DrawSplit s = split;
  const dim3 grid(ceil_div(s.n_units, s.group_units), a.B);
  size_t lds = draw_lds_bytes(s);
  // From two turns on the workgroup keeps the draft row in LDS where it fits: a gather from memory moves a 128-byte line
  // per id, about 2 us of a turn, the copy costs that once (128 sequences x 128256 ids: 51 us without, 39 with).  From three turns on
  // its exponentials if those fit, formed once a workgroup and not once an id: the turns then wait for the target's logits and the
  // inverse map alone.  us per step from the logits, exponentials / logits as stored, with one turn and a part of one 17.6 / 16.8
  // (200 sequences x 9000 ids, draft rows of 8000), with two 23.8 / 23.0 (128 x 32003, 32000) or even (draft rows of 1000), with two and a
  // half 20.9 / 21.2 (200 x 20011, 8000), with eight 48.3 / 52.3 (128 x 128256, 32000); workgroups of 8 wavefronts with two turns 33.2 /
  // 26.9 (700 x 6500, 4000).  Up to the largest copies (20 / 128 sequences): 50257 bf16 ids 26.0 / 60 against 26.4 / 76 gathered, 75000
  // 26.6 / 62 against 28 / 89.
  s.exps = kPer == 8 && s.group_units > 2 * kWaves && lds + exps_bytes(a.V_d) <= kLdsBytes;
  const size_t row_bytes = s.exps ? exps_bytes(a.V_d) : (size_t)a.V_d * (a.dtype == OT_BF16 ? 2 : 4) + 32;
  if (s.group_units > kWaves && lds + row_bytes <= kLdsBytes) {
    s.row_at = (int)(lds / sizeof(double));
    lds += row_bytes;
  }
  RowOffsets ro;
  for (int b = 0; b <= kFusedMaxB; ++b) ro.v[b] = row_off_host[b <= a.B ? b : a.B];
  if constexpr (kPer == 8)                               // several turns: draw_plan takes 512 ids a unit
    if (s.exps) return launch_draw_kernels<kPer, kBlocks, kWaves, true>(a, ro, s, grid, lds, stream);
  return launch_draw_kernels<kPer, kBlocks, kWaves, false>(a, ro, s, grid, lds, stream);
}

}  // namespace

hipError_t launch_final_draw(const StepArgs& a, const int32_t* row_off_host, int n_cu, hipStream_t stream) {
  if (a.B == 0) return hipSuccess;
  const DrawPlan plan = draw_plan(a.V_t, a.V_d, a.B, n_cu);
  if (plan.per == 2) return launch_draw<2>(a, row_off_host, plan.split, stream);
  if (plan.per == 4) return launch_draw<4>(a, row_off_host, plan.split, stream);
  if (plan.waves == 8) return launch_draw<8, false, 8>(a, row_off_host, plan.split, stream);
  if (plan.split.blocks == 1) return launch_draw<8>(a, row_off_host, plan.split, stream);
  return launch_draw<8, true>(a, row_off_host, plan.split, stream);
}

int final_draw_launches(int hosted, int nfine, int M, int V_t, int V_d, int B, int n_cu) {
  return test_has_its_launch(hosted, nfine, M, draw_plan(V_t, V_d, B, n_cu).split) ? 2 : 1;
}

}  // namespace otv
