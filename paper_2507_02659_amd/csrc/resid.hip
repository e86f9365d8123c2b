// The launches that draw the final token of every sequence (Algorithm 1: correction token from the residual of Eq. 2,
// or free token from p), grid = (groups of tiles of kResidTile target ids) x (sequences).
//   final_draw_kernel   the outcome records of the acceptance test are in memory (written by the launch before).
//   accept_draw_kernel  follows the launch that did the draft side and the softmax partials, the LM head's or the
//                       statistics launch: every workgroup first repeats the translation and the acceptance test of its
//                       sequence (one wavefront merges the partials of the draft rows and walks the window from the
//                       probe record while the others merge the target rows' partials, one wavefront per row; then that
//                       wavefront runs the test: a few microseconds of work on data that sits in L2, cheaper than a
//                       launch of its own: 300 sequences x 32003 ids 42 us, against 10.5 + 30.6 and a launch), then
//                       takes part in the draw.  The workgroups of a sequence reach the same outcome; only group 0
//                       writes the outputs of the translation and the test, the draft rows' merged statistics and
//                       the cache's use statistics.
#include <algorithm>

#include "accept.h"
#include "resid.h"

namespace otv {
namespace {

// row_at: where the draft row's copy starts in the dynamic LDS, in doubles (0: no copy)
__global__ __launch_bounds__(kDrawThreads) void final_draw_kernel(StepArgs a, int group_tiles, int row_at) {
  const int b = blockIdx.y, grp = blockIdx.x, tid = threadIdx.x;
  const int wave = uniform(tid >> 6), lane = tid & 63;
  __shared__ DrawLds s_draw;
  int dv[kPerLane];
  load_tmap<kPerLane>(a.tmap, a.V_t, draw_first_id(grp * group_tiles, wave, lane), 64, dv);   // overlaps the next load
  const FinalInfo f = a.fin[b];
  if (f.mode == 0) return;                  // greedy or flagged sequence: nothing to draw
  draw_final_token(a, b, grp, group_tiles, f, dv, &s_draw, row_at);
}

// Row offsets of up to kFusedMaxB sequences as a kernel argument (the host has them): the workgroup knows its rows without
// a dependent load in front of everything else.  With more sequences they come from memory.
struct RowOffsets { int32_t v[kFusedMaxB + 1]; };
constexpr int64_t kRepeatedMergeBytes = 32 << 20;

// kDraw = false: grid = (1) x (sequences); the workgroup only runs the test and leaves the outcome record in memory for
// a final_draw_kernel launch (used when repeating the test in every tile group would cost more than a launch).
// kChunks: the partials come from the statistics launch (chunk partials in three arrays per side) instead of the
// LM head's epilogue and draft-row pieces.
// kMany: more than kFusedMaxB sequences: row offsets from memory, partials merged in binary64 (as a runtime flag these two
// cost a single sequence 0.7 of 13 us).
// kWide: draft rows of more than kChunksAtOnce chunks (merge_draft_chunks).
template <bool kDraw, bool kChunks, bool kMany, bool kWide = kMany>
__global__ __launch_bounds__(kDrawThreads) void accept_draw_kernel(StepArgs a, RowOffsets ro, int group_tiles, int row_at) {
  const int b = blockIdx.y, grp = blockIdx.x, tid = threadIdx.x;
  const int wave = uniform(tid >> 6), lane = tid & 63;
  __shared__ DrawLds s_draw;
  __shared__ FinalInfo s_fin;
  __shared__ float s_pmx[64];
  __shared__ double s_pinv[64];
  __shared__ int s_parg[64];
  int dv[kPerLane];

  const int r0 = kMany ? a.row_off[b] : ro.v[b];
  const int k = (kMany ? a.row_off[b + 1] : ro.v[b + 1]) - r0 - 1;
  const float T = a.temperature[b];
  const float Td = a.draft_temperature ? a.draft_temperature[b] : T;
  const uint64_t sid = a.seq_id[b];
  const bool lead = grp == 0;               // the group that writes the test's outputs and the row statistics

  // The LM-head launch left what the drafted ids look up (ProbeRecord) and the draft rows' statistics.  The last
  // wavefront fetches them (one load of each array per lane), walks the window (Eq. 1), asks for the logits of the
  // proposed tokens and forms q' while they are on their way, all on its own, while the other wavefronts merge the softmax
  // partials of the target rows; the translation is thus repeated by every tile group of the sequence, and the lead group
  // writes its outputs and the cache's use statistics.  That wavefront's chain of round trips and binary64 functions is what
  // the others wait for: its loads leave before anything is known about the temperature, the walk comes before the functions,
  // and q' is formed once as a product instead of through the logarithms of its factors (from the launch's start to the
  // outcome 5.4 -> 3.8 us for one sequence of five drafted ids).
  const int q0 = r0 - b;
  constexpr int kTestWave = kDrawWaves - 1;   // runs the walk and the test
  Window W;
  DraftLane D;
  float z_tok = 0.f;
  bool bad = false, reached = false;
  int pos = 0;
  double u1 = 0.0;
  uint32_t rnd[4] = {0, 0, 0, 0};             // of row `lane`: word 0 tests that mapped position, word 1 draws its final token
  if (wave == kTestWave) {
    const ProbeRecord* rec = a.probe + b;
    const unsigned long long hit = rec->hit[lane];
    D.dm = rec->dm[lane];
    bad = rec->bad != 0;                      // wavefront-uniform
    D.zq = rec->zq[lane];
    D.mxq = 0.f; D.Sq = 1.0; D.argq = -1; D.q = 0.0;
    DraftPartials<kChunks> part;
    if (lane < k) part.load(a, q0 + lane);
    W = walk_window(k, lane, hit, D.dm);
    reached = ((W.starts >> lane) & 1ull) != 0ull;
    pos = __popcll(W.starts & bits_below(lane));
    if (reached) z_tok = a.Z[(int64_t)(r0 + pos) * a.ldz + W.t];
    if (lane < k) {
      if constexpr (kChunks) merge_draft_chunks<kWide>(a, q0 + lane, Td, part, &D.mxq, &D.Sq, &D.argq, kMany);
      else merge_draft_pieces(a, q0 + lane, Td, part, &D.mxq, &D.Sq, &D.argq);
      if (lead) { a.drow_max[q0 + lane] = D.mxq; a.drow_sum[q0 + lane] = D.Sq; a.drow_arg[q0 + lane] = D.argq; }
      if (Td > 0.f) D.q = exp(((double)D.zq - (double)D.mxq) * (1.0 / (double)Td)) / D.Sq;
      else D.q = a.draft_ids[q0 + lane] == D.argq ? 1.0 : 0.0;
    }
    D.qp = segment_q(D.q, W);
    if (T > 0.f) philox4x32_10((uint32_t)lane, a.step, (uint32_t)sid, (uint32_t)(sid >> 32), (uint32_t)a.seed, (uint32_t)(a.seed >> 32), rnd);
    u1 = u24(__shfl(rnd[0], pos));
  }
  const double invT = T > 0.f ? 1.0 / (double)T : 1.0;
  const double invTd = Td > 0.f ? 1.0 / (double)Td : 1.0;
  for (int row = wave; row <= k; row += kDrawWaves) {
    if (kChunks)
      merge_chunk_row(a.tpart_max, a.tpart_sum, a.tpart_arg, a.ncht, r0 + row, invT, lane, s_pmx, s_pinv, s_parg, row, lead,
                      a.row_max, a.row_sum, a.row_arg, kMany);
    else
      merge_fused_row(a.fused.part, a.fused.nfine, r0 + row, invT, lane, s_pmx, s_pinv, s_parg, row, lead, a.row_max,
                      a.row_sum, a.row_arg);
  }
  if (!(T > 0.f) && !lead) return;            // a greedy sequence draws nothing: its other groups have nothing to do
  // The inverse map of this wavefront's ids is needed last (by the tile masses) and asked for here, behind the loads
  // that the test waits for: loads return in issue order, and asked for first it held those back by its own latency.
  if (kDraw) load_tmap<kPerLane>(a.tmap, a.V_t, draw_first_id(grp * group_tiles, wave, lane), 64, dv);
  __syncthreads();
  Outcome O;
  if (wave == kTestWave) {
    FinalInfo fin{};                          // mode 0: nothing to draw
    if (!bad) {
      O = test_window(T, invT, W, D, reached, pos, z_tok, u1, s_pmx, s_pinv, s_parg);
      fin = final_info(r0, q0, T, Td, invT, invTd, W, D, O, u24((uint32_t)__builtin_amdgcn_readlane((int)rnd[1], O.n)), s_pmx, s_pinv);
    }
    if (lane == 0) s_fin = fin;
    if (!kDraw && lane == 0) a.fin[b] = fin;
  }
  if (kDraw) __syncthreads();
  if (wave == kTestWave && lead) {            // behind the barrier: nobody in this launch waits for these
    if (bad) {
      write_bad_sequence(a, b, r0, k, lane);
    } else {
      write_translation(a, b, r0, k, lane, W, reached, pos, D.qp);
      write_outcome(a, b, r0, k, lane, T, W, O, reached, pos, s_parg);
    }
  }
  if (!kDraw) return;
  const FinalInfo f = s_fin;
  if (f.mode == 0) return;
  draw_final_token(a, b, grp, group_tiles, f, dv, &s_draw, row_at);
}

}  // namespace

// Tiles per workgroup of the draw.  Eight (one turn) as long as that leaves no more than a workgroup per compute unit:
// a small batch is bound by the chain of round trips in one workgroup, which every further turn would lengthen.  With
// more, each workgroup takes as many turns as bring their number back to one per compute unit (86 registers: five
// wavefronts per SIMD, so that a workgroup of 16 fills one): its start, its share of the merge and its count at the end are then paid once for several turns,
// and a turn's loads overlap the sums of the turn before.  At most 64 turns, so that the halves' scratch stays small.
// Measured (kernel time, one turn per workgroup against this rule): 128 sequences x 128256 ids 109 + 10 us of a test
// launch against 39 us in one launch (2 us a turn), 64 x 152064 (half greedy) 39 + 10 against 30, 300 x 32003 65 against
// 30; 16 x 128256 and below stay at one turn.  Right above one workgroup per compute unit (us per step from the logits, two
// rows a sequence): 17 x 128256 27.1 against 22.4, 20: 28.9 / 22.8, 24: 31.4 / 24.2, 32: 33.8 / 26.2.  Up to 1.25, 1.5 and 2
// workgroups per compute unit were slower at 64, 128 and 300 sequences as well (128: 60, 56 and 51 against 38 us).
int draw_group_tiles(int ntiles, int B, int n_cu) {
  const int64_t groups = (int64_t)ceil_div(ntiles, kTurnTiles) * B;
  return kTurnTiles * std::min(64, std::max(1, ceil_div(groups, std::max(n_cu, 1))));
}

// hosted: the LM-head launch left its softmax partials, the draft rows' pieces and the probe records; otherwise the
// statistics launch left its chunk partials and the probe records.  row_off_host holds the B + 1 row offsets.
hipError_t launch_final_draw(const StepArgs& a, const int32_t* row_off_host, int n_cu, hipStream_t stream) {
  if (a.B == 0) return hipSuccess;
  const int group_tiles = draw_group_tiles(a.ntiles, a.B, n_cu);
  const dim3 grid(ceil_div(a.ntiles, group_tiles), a.B), block(kDrawThreads);
  size_t lds = std::max((size_t)a.ntiles, 2 * (size_t)group_tiles) * sizeof(double);
  // From two turns on the workgroup keeps the draft row in LDS where it fits: a gather from memory moves a 128-byte line
  // per id, about 2 us of a turn, the copy costs that once (128 sequences x 128256 ids: 51 us without, 39 with).  Up to the largest
// copies (us per step from the logits, 20 / 128 sequences): 50257 bf16 ids 26.0 / 60 against 26.4 / 76 gathered, 75000 26.6 / 62
// against 28 / 89, 32000 fp32 ids 24.7 / 59 against 25.6 / 71.
  int row_at = 0;
  const size_t row_bytes = (size_t)a.V_d * (a.dtype == OT_BF16 ? 2 : 4) + 32;
  if (group_tiles > kTurnTiles && lds + 16 + row_bytes <= kDrawLdsBytes) {
    row_at = (int)((lds + 15) / 16) * 2;
    lds = (size_t)row_at * sizeof(double) + row_bytes;
  }
  RowOffsets ro;
  for (int b = 0; b <= kFusedMaxB; ++b) ro.v[b] = row_off_host[b <= a.B ? b : a.B];
  if (!a.hosted) {                                         // a few chunks per row: always one launch
    if (a.B > kFusedMaxB) hipLaunchKernelGGL((accept_draw_kernel<true, true, true>), grid, block, lds, stream, a, ro, group_tiles, row_at);
    else if (a.nchd > kChunksAtOnce) hipLaunchKernelGGL((accept_draw_kernel<true, true, false, true>), grid, block, lds, stream, a, ro, group_tiles, row_at);
    else hipLaunchKernelGGL((accept_draw_kernel<true, true, false>), grid, block, lds, stream, a, ro, group_tiles, row_at);
    return hipGetLastError();
  }
  if (a.B > kFusedMaxB) return hipErrorInvalidValue;
  // Every tile group of a sequence repeats the merge of its rows' partials: M x nfine x 16 bytes per group.  Up to
  // about the traffic that costs as much as a launch this is one launch; beyond it the test gets a launch of its own.
  const int64_t repeated = (int64_t)a.M * a.fused.nfine * (int64_t)sizeof(Partial) * grid.x;
  if (repeated <= kRepeatedMergeBytes) {
    hipLaunchKernelGGL((accept_draw_kernel<true, false, false>), grid, block, lds, stream, a, ro, group_tiles, row_at);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((accept_draw_kernel<false, false, false>), dim3(1, a.B), block, 0, stream, a, ro, group_tiles, row_at);
  hipLaunchKernelGGL(final_draw_kernel, grid, block, lds, stream, a, group_tiles, row_at);
  return hipGetLastError();
}

}  // namespace otv
