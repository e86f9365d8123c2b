// LM-head projection z = h . W for the k+1 verified rows of every sequence (Algorithm 1, the target pass that
// yields p(t_t) .. p(t_{t+m}) in parallel): Z[M, V_t] (fp32) = H[M, d] (bf16) x W[d, V_t] (bf16), fp32 accumulate.
//
// At verification time M = sum_b (k_b + 1) is a few rows to a few hundred, so the product is bound by streaming
// the d x V_t weights from HBM exactly once, not by the matrix cores.  The design follows from that:
//   * W is re-tiled once at init into the register layout of v_mfma_f32_16x16x32_bf16 operands: the fragment for
//     16 vocabulary columns x 32 hidden indices is 64 lanes x 16 bytes, stored contiguously, and the four
//     fragments of 64 adjacent columns per 32-deep step are adjacent.  A wavefront streams the fragments of its
//     columns with fully coalesced 1 KB loads: no transpose anywhere.
//   * Every weight is used by exactly one wavefront, which keeps accumulators for ALL rows of the M-block
//     (up to 11 x 16 rows while the product is bound by HBM), so W is read from HBM once.  More than 176 rows run as
//     several M-blocks of up to 18 x 16 rows per column tile, scheduled so that they share W in one L2.
//   * From 17 rows on, both operands travel by direct global->LDS loads.  The hidden rows, shared by the wavefronts
//     of a workgroup, go through double-buffered slices 128 (or, for the tall M-blocks, 64) columns deep (swizzled
//     rows: conflict-free 16-byte reads); each hidden fragment read from LDS feeds NW MFMAs.  The weight fragments
//     go through a wavefront-private ring four (two) steps deep, so that the one barrier per slice never waits on
//     HBM latency.
//   * The epilogue also reduces each row's logits over the workgroup's columns to softmax partials (maximum, its
//     column, sum of exponentials at the row's temperature), so that no later pass has to read the logits for them.
//   * A workgroup owns 128 to 640 columns, so that the launch fits into few, full rounds of one workgroup per compute
//     unit (what a workgroup does outside its main loop is time its compute unit does not stream).
//   * The launch can host the draft side of the step, the work that needs no target logits (see draft-side jobs in
//     the kernel): with one M-block inside the multiplying workgroups, behind their first loads; with several, or with up
//     to 16 rows, in workgroups at the front of the launch.  With several M-blocks it may also leave the partials alone.
//   * All waits on the load counter are written by hand, by number (loads complete in issue order), and workgroup
//     barriers carry no fence: with direct-to-LDS loads in flight every wait the compiler adds itself is a full
//     drain of the counter, which would empty the weight pipeline at every slice.
// Operand roles: the weight fragment is MFMA operand A and the hidden fragment operand B, so a lane ends up with
// four consecutive vocabulary columns of one row and stores them as one float4.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "translate.h"

namespace otv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));


// Packed layout (16-byte units): unit(wt * packed_tile_units(nks) + (ks * 4 + sub) * 64 + lane) holds
//   W[ks*32 + 8*(lane/16) + e][wt*64 + sub*16 + lane%16], e = 0..7; zero outside [d, V_t].  The gap between tiles is
//   never read.
__global__ __launch_bounds__(256) void pack_w_kernel(const uint16_t* __restrict__ W, int d, int V_t,
                                                     uint4* __restrict__ Wp, int nks, int64_t n_units) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u >= n_units) return;
  const int lane = (int)(u & 63);
  const int sub = (int)((u >> 6) & 3);
  const int64_t rest = u >> 8;
  const int ks = (int)(rest % nks);
  const int wt = (int)(rest / nks);
  const int n = wt * 64 + sub * 16 + (lane & 15);
  const int kb = ks * 32 + 8 * (lane >> 4);
  uint32_t w[4] = {0, 0, 0, 0};
  if (n < V_t) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = kb + e;
      const uint32_t x = kk < d ? (uint32_t)W[(int64_t)kk * V_t + n] : 0u;
      w[e >> 1] |= x << (16 * (e & 1));
    }
  }
  Wp[(int64_t)wt * packed_tile_units(nks) + ((int64_t)ks * 4 + sub) * 64 + lane] = make_uint4(w[0], w[1], w[2], w[3]);
}

// ---------------------------------------------------------------------------------------------------------------
// Wide kernel: M-blocks of up to MT*16 rows.  WPG wavefronts per workgroup, each owning NW*16 columns over the whole
// hidden dimension.  The hidden slice (KC columns of all rows of the M-block) is double-buffered in LDS and filled
// by direct global->LDS loads (no staging registers): the next slice is requested before the current one feeds the
// MFMAs, and one barrier per slice hands the buffers over.  LDS rows are unpadded; the 16-byte chunks of a row are
// XOR-swizzled with the row index (applied on the global side of the copy, since a direct load writes consecutive
// lanes to consecutive LDS addresses) so that the 16 rows a fragment read touches fall into 16 distinct bank groups.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

// s_waitcnt immediate (gfx9 encoding) that waits until at most N vector-memory loads are outstanding and nothing else
constexpr int vmcnt_imm(int n) { return (n & 0xF) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// Workgroup barrier without the memory fence of __syncthreads().  The fence makes the compiler drain every
// outstanding vector-memory load (it cannot tell a direct-to-LDS load that must be visible from a register prefetch
// that need not be), which would empty the prefetch pipelines at every hand-over.  The kernels below wait by count for
// exactly the loads that have to be visible (s_waitcnt above) and then meet here; LDS reads of the buffer that is
// handed back have been consumed by MFMAs before a wavefront arrives.
// The empty asm statements keep the compiler from moving memory accesses across the barrier.
__device__ inline void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Barrier that publishes this wavefront's LDS writes (all LDS operations done) without touching the load counter.
__device__ inline void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), vmcnt and expcnt unconstrained
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }
// largest divisor of n that is at most `limit` (limit >= 1)
constexpr int largest_divisor_c(int n, int limit) { return n % limit == 0 ? limit : largest_divisor_c(n, limit - 1); }

template <int MT, int PF, int WPG, int KC, int NW, bool W_ONCE>
__global__ __launch_bounds__(WPG * 64) void lmhead_bf16_wide_kernel(const uint16_t* __restrict__ H, int M, int d,
                                                                    const uint4* __restrict__ Wp, int nks,
                                                                    int n_wtiles, float* __restrict__ Z, int V_t,
                                                                    int64_t ldz, int vec_store,
                                                                    const uint16_t* __restrict__ zeros, int m_blocks,
                                                                    FusedStats fs, int n_front, int n_piece_jobs,
                                                                    int helpers_look_up, StepArgs ds) {
  constexpr int kKSteps = KC / 32;                 // MFMA steps per slice
  constexpr int kCPR = KC / 8;                     // 16-byte chunks per slice row
  constexpr int kSliceChunks = MT * 16 * kCPR;
  constexpr int kDma = (kSliceChunks + WPG * 64 - 1) / (WPG * 64);
  static_assert(kSliceChunks % 64 == 0 && kSliceChunks >= 64, "a slice is a whole number of wavefront-wide loads");
  constexpr int kPatchNW = NW <= 4 ? NW : 3;        // column tiles that the epilogue turns at a time
  constexpr int kPatchRow = kPatchNW * 16 + 4;     // floats per padded row of the epilogue patch
  // steps per trip of the main loop: whole pairs of slices (buffers A, B) and whole turns of the weight ring, so
  // that both the buffer and the ring array of every step are known at compile time
  constexpr int kUnroll = 2 * kKSteps * PF / gcd_c(2 * kKSteps, PF);
  // Where the refill of the weight ring stands among the MFMAs of a step counts in the 128-column kernels, whose steps are one
  // load each: left to the compiler it moved with unrelated code, 50.5 or 51.9 us for 80 rows x 32000 columns (d = 4096).
  // Up to six row tiles it is held behind the first; with more, that is 1 to 3 % slower than where the compiler puts it.
  constexpr bool kEarlyRefill = PF == 8 && MT <= 6;
  static_assert(PF % kKSteps == 0 && PF <= 8, "a weight fetch is used a whole number of slices later");
  static_assert(kGemmKPad % KC == 0 && (kCPR == 8 || kCPR == 16), "slice geometry");
  static_assert((PF - 1) * NW + (PF / kKSteps) * kDma + NW < 64, "the load counter has 6 bits");
  static_assert(NW >= 1 && NW <= 5, "a wavefront owns 16 to 80 columns");
  __shared__ __attribute__((aligned(16))) uint16_t sA[MT * 16 * KC];
  __shared__ __attribute__((aligned(16))) uint16_t sB[MT * 16 * KC];
  // epilogue: one 16-row tile per wavefront; before the main loop: scratch of the draft-side jobs, four sequences' lookups
  constexpr int kLookupFloats = (int)(sizeof(DraftLds) * (WPG * 64 / 128) / (sizeof(float) * WPG) + 4) / 4 * 4;
  constexpr int kPatchFloats = 16 * kPatchRow > kLookupFloats ? 16 * kPatchRow : kLookupFloats;
  __shared__ __attribute__((aligned(16))) float sPatch[WPG][kPatchFloats];
  // The weight fragments travel by direct global->LDS loads as well, into a ring of PF steps: one array per step (so
  // that the compiler can tell them apart), each wavefront using its own NW KB of every array.  A register prefetch
  // next to direct-to-LDS loads would make the compiler drain the load counter at each first use of a register.
  // (Measured: fetching the weights into registers eight steps ahead instead, which doubles the bytes in flight per CU
  // and keeps them out of LDS, is no faster at 144 rows: 222 against 218 us per step.)
  constexpr int kRing = WPG * NW * 64;
  __shared__ uint4 sW0[kRing], sW1[kRing], sW2[PF > 2 ? kRing : 1], sW3[PF > 3 ? kRing : 1], sW4[PF > 4 ? kRing : 1],
      sW5[PF > 5 ? kRing : 1], sW6[PF > 6 ? kRing : 1], sW7[PF > 7 ? kRing : 1];
  // fused row statistics: row offsets and temperatures of the sequences (staged by direct loads in the prologue),
  // and the exponent scale log2(e)/T of each row of the M-block
  __shared__ int32_t sRowOff[kFusedMaxB + 1];
  __shared__ float sTemp[kFusedMaxB + 1];
  __shared__ float sTempDraft[kFusedMaxB + 1];       // the drafter's temperatures, staged only when they are given apart
  __shared__ float sScale[MT * 16];
  static_assert(WPG * 64 >= kFusedMaxB + 1, "one thread per sequence stages its row offset and temperature");
  static_assert((WPG & (WPG - 1)) == 0, "the mask below tells the compiler the range of the wavefront index");
  const int tid = threadIdx.x, wave = (tid >> 6) & (WPG - 1), lane = tid & 63;
  // The first n_front workgroups of the launch (a multiple of 8) multiply nothing: they run the draft side (see below).
  const int wg = (int)blockIdx.x - n_front;
  // Workgroup id -> (column tile, M-block).  Consecutive ids go round-robin to the 8 XCDs, each with its own L2; the
  // M-blocks of one column tile get ids that land on the same XCD back to back, so that when M needs several
  // blocks their weight streams coincide in that XCD's L2 and HBM is still read once.
  const int xcd = wg & 7, slot = wg >> 3;
  const int col_tile = (slot / m_blocks) * 8 + xcd, m_block = slot % m_blocks;
  const int n_col_tiles = (n_wtiles * 4 + WPG * NW - 1) / (WPG * NW);
  const bool hosts = n_piece_jobs > 0;               // this launch runs the draft side of the step (see below)
  // stages the sequences' row offsets and temperatures in LDS (4-byte direct loads: lane i of a wavefront fills entry
  // 64*wave + i); a wait for the loads and a barrier follow
  auto stage_sequences = [&]() {
    if (fs.part && wave * 64 <= fs.B) {
      __builtin_amdgcn_global_load_lds((glb_ptr_t)(fs.row_off + min(tid, fs.B)), (lds_ptr_t)(sRowOff + wave * 64), 4, 0,
                                       0);
      __builtin_amdgcn_global_load_lds((glb_ptr_t)(fs.temperature + min(tid, fs.B - 1)), (lds_ptr_t)(sTemp + wave * 64),
                                       4, 0, 0);
      if (hosts && ds.draft_temperature)
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(ds.draft_temperature + min(tid, fs.B - 1)),
                                         (lds_ptr_t)(sTempDraft + wave * 64), 4, 0, 0);
    }
  };
  // The draft side of the step, the part that needs none of the logits, comes in two kinds of jobs.
  // Piece job j: the softmax statistics (a3) of one piece of a draft row (see PiecePlan); at most one per multiplying
  // workgroup, which asks for it in front of its first loads and reduces it while those land.  Lookup job b: what the
  // drafted ids of sequence b look up (the drafted logit, the direct image, the n-gram table probes of every window),
  // left as a ProbeRecord for the next launch, which walks the windows.
  // All threads call a job (workgroup barriers inside).
  // Every lane holds the row offsets and the drafter's temperatures of sequences lane, lane + 64, ...: the owner of a
  // draft row (the last b with row_off[b] - b <= q, a monotone predicate) is then a count over ballots and its
  // temperature one lane read, with no chain of dependent loads.  piece_request asks for these and for the first
  // batch of the job's first row piece; piece_job (later, so that the loads overlap whatever is issued in between)
  // reduces it and goes through the rest of the chunk.
  constexpr int kSeqRegs = (kFusedMaxB + 64) / 64;
  int seq_before[kSeqRegs];
  float seq_temp[kSeqRegs];
  RowFirstBatch<uint16_t, kPieceBatch> first_batch;
  auto piece_request = [&](int job) {
    const float* temps = ds.draft_temperature ? ds.draft_temperature : fs.temperature;
#pragma unroll
    for (int j = 0; j < kSeqRegs; ++j) {
      const int b = min(64 * j + lane, fs.B - 1);
      seq_before[j] = fs.row_off[b] - b;
      seq_temp[j] = temps[b];
    }
    int q, i, e0, n;
    ds.plan.locate(job, &q, &i);
    PiecePlan::span(ds.V_d, ds.plan.pieces(q), i, &e0, &n);
    workgroup_draft_piece_request<uint16_t, WPG>(ds, q, e0, n, tid, first_batch);
  };
  auto piece_job = [&](int job) {
    float* st_mx = reinterpret_cast<float*>(&sPatch[0][0]);
    int32_t* st_arg = reinterpret_cast<int32_t*>(st_mx + WPG);
    double* st_S = reinterpret_cast<double*>(st_mx + 2 * WPG);
    int q, i, e0, n;
    ds.plan.locate(job, &q, &i);
    bool first = true;
    for (; q < ds.K; q += ds.plan.workers) {
      PiecePlan::span(ds.V_d, ds.plan.pieces(q), i, &e0, &n);
      int owner = -1;
      float Td = 1.f;
#pragma unroll
      for (int j = 0; j < kSeqRegs; ++j) {
        const bool before = 64 * j + lane < fs.B && seq_before[j] <= q;
        owner += __popcll(__ballot(before));
      }
#pragma unroll
      for (int j = 0; j < kSeqRegs; ++j) {
        const float t = __shfl(seq_temp[j], owner & 63);
        if ((owner >> 6) == j) Td = t;
      }
      DraftPiece* out = ds.dpiece + (int64_t)q * kDraftPieces + i;
      if (first) workgroup_draft_piece<uint16_t, WPG, true>(ds, q, e0, n, Td, tid, st_mx, st_arg, st_S, out, &first_batch);
      else workgroup_draft_piece<uint16_t, WPG>(ds, q, e0, n, Td, tid, st_mx, st_arg, st_S, out);
      first = false;
    }
  };
  // The same for one wavefront on its own (front workgroups: every wavefront is a worker of the plan): no workgroup
  // barriers, and 16 sixteen-byte loads in flight per lane, because a workgroup that only reads next to the other
  // workgroups' streams gets the bytes it keeps in flight once per several microseconds.
  auto wave_piece_jobs = [&](int job) {
    const float* temps = ds.draft_temperature ? ds.draft_temperature : fs.temperature;
#pragma unroll
    for (int j = 0; j < kSeqRegs; ++j) {
      const int b = min(64 * j + lane, fs.B - 1);
      seq_before[j] = fs.row_off[b] - b;
      seq_temp[j] = temps[b];
    }
    int q, i, e0, n;
    ds.plan.locate(job, &q, &i);
    for (; q < ds.K; q += ds.plan.workers) {
      PiecePlan::span(ds.V_d, ds.plan.pieces(q), i, &e0, &n);
      int owner = -1;
      float Td = 1.f;
#pragma unroll
      for (int j = 0; j < kSeqRegs; ++j) {
        const bool before = 64 * j + lane < fs.B && seq_before[j] <= q;
        owner += __popcll(__ballot(before));
      }
#pragma unroll
      for (int j = 0; j < kSeqRegs; ++j) {
        const float t = __shfl(seq_temp[j], owner & 63);
        if ((owner >> 6) == j) Td = t;
      }
      DraftPiece r; r.mx = -INFINITY; r.arg = 0x7FFFFFFF; r.sum = 0.0;
      if (n > 0) {
        wave_row_stats<uint16_t, 16>(static_cast<const uint16_t*>(ds.draft_logits) + (int64_t)q * ds.V_d + e0, n,
                                     Td > 0.f ? kLog2eF / Td : kLog2eF, lane, &r.mx, &r.arg, &r.sum);
        r.arg += e0;
      }
      if (lane == 0) ds.dpiece[(int64_t)q * kDraftPieces + i] = r;
    }
  };
  auto lookup_job = [&](int b) {               // the sequences are staged in LDS
    DraftLds* probe_lds = reinterpret_cast<DraftLds*>(&sPatch[0][0]);
    static_assert(sizeof(DraftLds) <= sizeof(sPatch), "the lookups' scratch fits into the epilogue patch");
    const int r0 = sRowOff[b], k = sRowOff[b + 1] - r0 - 1;
    draft_lds_reset(probe_lds, tid);
    __syncthreads();
    fetch_ids_and_probe(ds, r0 - b, k, tid, WPG * 64, probe_lds);
    __syncthreads();
    ProbeRecord* rec = ds.probe + b;
    if (tid < 64) { rec->hit[tid] = probe_lds->hit[tid]; rec->zq[tid] = probe_lds->zq[tid]; rec->dm[tid] = probe_lds->dm[tid]; }
    if (tid == 0) rec->bad = probe_lds->bad;
    __syncthreads();
  };
  // A workgroup with nothing to multiply takes the lookups of every n_helpers-th group of four sequences, 128 threads
  // each: next to the other workgroups' weight streams every dependent load of a lookup takes several microseconds, and
  // so the chains of loads of four sequences run side by side.  The sequences are staged first.
  auto helper_lookups = [&](int helper, int n_helpers) {
    stage_sequences();
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    wg_barrier();
    constexpr int kAtOnce = WPG * 64 / 128;
    static_assert(sizeof(DraftLds) * kAtOnce <= sizeof(sPatch), "the lookups' scratch fits into the epilogue patch");
    const int slot = tid >> 7, g = tid & 127;
    DraftLds* L = reinterpret_cast<DraftLds*>(&sPatch[0][0]) + slot;
    for (int b0 = helper; b0 < fs.B; b0 += kAtOnce * n_helpers) {
      const int b = b0 + slot * n_helpers;
      const bool valid = b < fs.B;
      const int r0 = valid ? sRowOff[b] : 0, k = valid ? sRowOff[b + 1] - r0 - 1 : 0;
      if (valid) draft_lds_reset(L, g);
      __syncthreads();
      if (valid) fetch_ids_and_probe(ds, r0 - b, k, g, 128, L);
      __syncthreads();
      if (valid && g < 64) {
        ProbeRecord* rec = ds.probe + b;
        rec->hit[g] = L->hit[g]; rec->zq[g] = L->zq[g]; rec->dm[g] = L->dm[g];
        if (g == 0) rec->bad = L->bad;
      }
      __syncthreads();
    }
  };
  if (wg < 0) {
    // Front workgroups: the whole draft side of a launch that is bound by the matrix cores (several M-blocks), where a
    // piece in front of every multiplying workgroup's loop would add its time to each of them.  They start first and
    // are done long before the launch ends; every wavefront of them is a worker of the plan, and front workgroup h takes
    // its share of the lookups.
    // The lookups come first: their chains of dependent loads are short while the launch has not yet filled the
    // memory system, and several times as long afterwards.
    const int h = (int)blockIdx.x;
    helper_lookups(h, n_front);
    if (h * WPG + wave < n_piece_jobs) wave_piece_jobs(h * WPG + wave);
    return;
  }
  if (col_tile >= n_col_tiles) {
    // Padding of the id space: a workgroup with nothing to multiply.  Where the launch has such workgroups and they can
    // finish in time (the host decides), they take the sequences' lookups, on compute units that the multiplying
    // workgroups leave idle.  (The draft rows stay with the multiplying workgroups: next to their saturating streams a
    // workgroup that only reads was measured at about 10 GB/s however many loads it keeps in flight, so five of them
    // cannot get through 8 MB of draft logits in time.)
    if (helpers_look_up && hosts) {
      const int n_pad_tiles = (n_col_tiles + 7) / 8 * 8 - n_col_tiles;
      helper_lookups((col_tile - n_col_tiles) * m_blocks + m_block, n_pad_tiles * m_blocks);
    }
    return;
  }
  const int t16_own = (col_tile * WPG + wave) * NW;   // first 16-column tile of this wavefront
  const bool active = t16_own < n_wtiles * 4;
  // A wavefront past the last tile (only in the last workgroup) multiplies the last tile again and stores nothing:
  // the main loop then has no wavefront-dependent branch and every wavefront issues the same loads in the same order.
  // (With 48 or 80 columns a wavefront can straddle the end: its surplus tiles are the last one as well, and the columns
  // they stand for lie past V_t, where nothing is counted or stored.)
  const int t16 = active ? t16_own : n_wtiles * 4 - NW;
  const int row0 = m_block * (MT * 16);
  // fragment (16-column tile t, step ks) sits at 16-byte unit (t/4) * packed_tile_units(nks) + (ks * 4 + t%4) * 64 + lane
  constexpr bool kOneTile = 4 % NW == 0;               // all fragments of a step lie in one 64-column tile, back to back
  const uint4* wp[kOneTile ? 1 : NW];
#pragma unroll
  for (int nw = 0; nw < (kOneTile ? 1 : NW); ++nw) {
    const int t = min(uniform(t16) + nw, n_wtiles * 4 - 1);
    wp[nw] = Wp + (int64_t)(t / 4) * packed_tile_units(nks) + (t % 4) * 64 + lane;
  }

  // Swizzle key of a row: the 16-byte chunks of a row are XORed with the low bits of the row index (measured: with
  // 128-byte rows, folding bit 3 of the row into the key as well stalls 46 % of the LDS cycles on bank conflicts,
  // the plain low bits 2 %).
  auto row_key = [](int row) { return row & (kCPR - 1); };
  // request slice kc (in 32-column steps) into buffer s: chunk q of the buffer holds logical chunk (q%kCPR)^key(row).
  // A request past the end of K re-reads the last slice, so that every slice issues the same number of loads and
  // the in-order load counter can be waited on by number.
  auto request = [&](int kc_want, uint16_t* s) {
    const int kc = min(kc_want, nks - kKSteps);
#pragma unroll
    for (int j = 0; j < kDma; ++j) {
      // wave-uniform.  A wavefront whose turn falls past the end loads the last 64 chunks once more (the same bytes to
      // the same place as their owner): every wavefront then issues exactly kDma loads per slice, the loop has no
      // branch, and the load counter can be waited on by number.
      const int q0 = min((j * WPG + wave) * 64, kSliceChunks - 64);
      {
        const int q = q0 + lane;
        const int row = q / kCPR, pc = q % kCPR;
        const int lc = pc ^ row_key(row);
        const int gr = min(row0 + row, M - 1);     // rows past M are never stored: any valid row will do
        const int gk = kc * 32 + lc * 8;
        const uint16_t* src = gk < d ? H + (int64_t)gr * d + gk : zeros;   // the padded tail of K must read as zero
        __builtin_amdgcn_global_load_lds((glb_ptr_t)src, (lds_ptr_t)(s + q0 * 8), 16, 0, 0);
      }
    }
  };
  auto ring = [&](int s) -> uint4* {
    return (s == 0 ? sW0 : s == 1 ? sW1 : s == 2 ? sW2 : s == 3 ? sW3 : s == 4 ? sW4 : s == 5 ? sW5 : s == 6 ? sW6 : sW7) +
           wave * (NW * 64);
  };
  // fetch the fragments of step kf into this wavefront's part of ring array s
  // With a single M-block every weight is read exactly once by the whole launch: those loads are marked nontemporal
  // (cache-policy bit 1 of the load), which a plain streaming read of the same bytes was measured to gain 12 % from
  // (7.05 against 6.3 TB/s).  With several M-blocks the later ones find the weights in L2 and the mark would not help.
  constexpr int kWeightPolicy = W_ONCE ? 2 : 0;
  auto fetch_w = [&](int kf, int s) {
#pragma unroll
    for (int nw = 0; nw < NW; ++nw)
      __builtin_amdgcn_global_load_lds((glb_ptr_t)(kOneTile ? wp[0] + ((int64_t)kf * 4 + nw) * 64 : wp[kOneTile ? 0 : nw] + (int64_t)kf * 256),
                                       (lds_ptr_t)(ring(s) + nw * 64), 16, 0, kWeightPolicy);
  };

  // This workgroup's piece of the draft rows is asked for first: it is reduced while the first weight fragments and the
  // hidden slice, asked for right behind it, land.  2 to 3 us that the launch which follows no longer has to wait for.
  const int own_job = col_tile * m_blocks + m_block;
  // (only a launch with a single M-block gives its multiplying workgroups pieces: W_ONCE says so at compile time, which
  // keeps the piece's registers out of the kernels whose accumulators leave none to spare)
  const bool has_job = W_ONCE && n_front == 0 && own_job < n_piece_jobs;
  if (has_job) piece_request(own_job);
  request(0, sA);
#pragma unroll
  for (int s = 0; s < PF; ++s) fetch_w(min(s, nks - 1), s);
  stage_sequences();
  if (has_job) piece_job(own_job);
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  wg_barrier();
  // Without idle workgroups to take them, the lookups go to the multiplying workgroups as well, from the last one down.
  if (hosts && !helpers_look_up && n_front == 0)
    for (int b = n_col_tiles * m_blocks - 1 - own_job; b < fs.B; b += n_col_tiles * m_blocks) lookup_job(b);

  f32x4 acc[MT][NW];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nw = 0; nw < NW; ++nw) acc[mt][nw] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int a_row = lane & 15, a_grp = lane >> 4;
  // one slice out of buffer hs; kc = its first step, s0 = ring array of that step (compile-time after unrolling)
  auto compute = [&](const uint16_t* hs, int kc, int s0) {
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) {
      const int kk = kc + ks;
      const int rs = (s0 + ks) % PF;
      // This step's weight fragments were requested PF steps ago; since then PF-1 refills and PF/kKSteps hidden slices
      // were requested, so they have landed once no more loads than that are outstanding.  Waiting by number here
      // (with an instruction between the wait and the read) also spares the compiler from inserting its own wait,
      // which with direct-to-LDS loads in flight is always a full drain.
      __builtin_amdgcn_s_waitcnt(vmcnt_imm((PF - 1) * NW + (PF / kKSteps) * kDma));
      asm volatile("s_nop 0");
      __builtin_amdgcn_sched_barrier(0);
      uint4 bw[NW];
#pragma unroll
      for (int nw = 0; nw < NW; ++nw) bw[nw] = ring(rs)[nw * 64 + lane];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int pc = (ks * 4 + a_grp) ^ row_key(a_row);
        const uint4 hv = *reinterpret_cast<const uint4*>(&hs[(mt * 16 + a_row) * KC + pc * 8]);
        const bf16x8 hf = __builtin_bit_cast(bf16x8, hv);
#pragma unroll
        for (int nw = 0; nw < NW; ++nw) {
          acc[mt][nw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bw[nw]), hf, acc[mt][nw],
                                                                0, 0, 0);
        }
        // The ring array is free again: refill it with the fragments PF steps ahead (past the end: the last ones again)
        if (kEarlyRefill && mt == 0) {
          __builtin_amdgcn_sched_barrier(0);
          fetch_w(min(kk + PF, nks - 1), rs);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (!kEarlyRefill) fetch_w(min(kk + PF, nks - 1), rs);
      __builtin_amdgcn_sched_barrier(0);   // keep the next step's LDS reads from being hoisted (register budget)
    }
  };
  // Loads complete in issue order, so once at most kKSteps*NW loads (the weight fragments requested during the slice)
  // are outstanding, this wavefront's part of the next hidden slice has landed in LDS.
  auto hand_over = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(kKSteps * NW));
    wg_barrier();
  };

  // Whole trips run without a branch inside (the compiler's bookkeeping of the load counter degrades to full drains at
  // the first use of a loaded register behind any control-flow merge that a shorter path could reach); the slices that
  // are left after the last whole trip follow as straight-line code behind forward branches.
  auto one_slice = [&](int kc, int p) {
    request(kc + kKSteps, (p & 1) ? sA : sB);
    __builtin_amdgcn_sched_barrier(0);
    compute((p & 1) ? sB : sA, kc, (p * kKSteps) % PF);
    hand_over();
  };
  int base = 0;
  for (; base + kUnroll <= nks; base += kUnroll) {
#pragma unroll
    for (int p = 0; p < kUnroll / kKSteps; ++p) one_slice(base + p * kKSteps, p);
  }
#pragma unroll
  for (int p = 0; p < kUnroll / kKSteps - 1; ++p)
    if (base + p * kKSteps < nks) one_slice(base + p * kKSteps, p);
  if (fs.part) {
    // Row statistics of this workgroup's column tile, from the accumulators: per row the maximum, its lowest column
    // and sum exp((z - max)/T), first per wavefront (NW*16 columns), then merged over the wavefronts; one partial per
    // row and column tile goes to memory.  All LDS buffers of the main loop are free: every wavefront has passed the
    // barrier that followed its last slice (the weight ring may still receive the surplus refills; it is not used).
    // The statistics scratch (3 x 4 bytes per lane and row tile) reuses LDS of the main loop: either both hidden
    // buffers (maxima and sums in the first, columns in the second), or, where that holds fewer row tiles at once, one
    // hidden buffer each for the maxima and the sums and the first weight-ring array for the columns (the ring is
    // drained first: the surplus refills past the end of K still land there).  Not the epilogue patch: a wavefront that
    // is done here goes on to turn its logits through its part of the patch while the merging threads still read.
    // When even that is too small for all row tiles at once the row tiles are taken in groups of kStatMT.
    constexpr int kFitHidden = MT * KC / (16 * WPG), kFitSpread = MT * KC / (8 * WPG) < 4 * NW ? MT * KC / (8 * WPG) : 4 * NW;
    // row tiles per group: the largest divisor of MT that fits, in whichever layout allows the larger one
    constexpr int kGroupHidden = largest_divisor_c(MT, kFitHidden < MT ? kFitHidden : MT);
    constexpr int kGroupSpread = largest_divisor_c(MT, kFitSpread < MT ? kFitSpread : MT);
    constexpr bool kSpread = kGroupSpread > kGroupHidden;
    constexpr int kStatMT = kSpread ? kGroupSpread : kGroupHidden;
    static_assert(kStatMT >= 1 && MT % kStatMT == 0, "row tiles split evenly into statistics groups");
    static_assert(sizeof(float) * WPG * kStatMT * 64 * (kSpread ? 1 : 2) <= sizeof(sA) &&
                  sizeof(float) * WPG * kStatMT * 64 <= (kSpread ? sizeof(sW0) : sizeof(sB)), "the scratch fits");
    float* st_max = reinterpret_cast<float*>(sA);
    float* st_sum = kSpread ? reinterpret_cast<float*>(sB) : st_max + WPG * kStatMT * 64;
    int32_t* st_arg = kSpread ? reinterpret_cast<int32_t*>(sW0) : reinterpret_cast<int32_t*>(sB);
    if (kSpread) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // before the barrier below
    for (int r = tid; r < MT * 16; r += WPG * 64) {
      const int row = min(row0 + r, M - 1);
      int lo = 0, hi = fs.B - 1;                    // sequence that owns the row: last b with row_off[b] <= row
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sRowOff[mid] <= row) lo = mid; else hi = mid - 1;
      }
      const float T_b = sTemp[lo];
      sScale[r] = T_b > 0.f ? 1.4426950408889634f / T_b : 1.4426950408889634f;
    }
    lds_barrier();
    // every lane reduces its own NW*4 values of a row (no cross-lane traffic) and parks the partial in LDS; only a
    // wavefront that reaches past column V_t (or repeats the last tile) has to mask
    const int n_valid = active ? V_t - (t16 * 16 + 4 * (lane >> 4)) : 0;   // this lane's columns n0 + 16*nw + e < V_t
    const bool all_valid = __builtin_amdgcn_readfirstlane(active && (t16 + NW) * 16 <= V_t);
#pragma unroll
    for (int h = 0; h < MT; h += kStatMT) {
#pragma unroll
      for (int ml = 0; ml < kStatMT; ++ml) {
        const int mt = h + ml;
        const float sc = sScale[mt * 16 + (lane & 15)];
        float v[NW * 4];
#pragma unroll
        for (int nw = 0; nw < NW; ++nw)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            v[nw * 4 + e] = (all_valid || nw * 16 + e < n_valid) ? acc[mt][nw][e] : -INFINITY;
        float best = v[0];
        int bi = 0;
#pragma unroll
        for (int i = 1; i < NW * 4; ++i)            // ascending columns: the first maximum is kept
          if (v[i] > best) { best = v[i]; bi = i; }
        const int barg = best == -INFINITY ? 0x7FFFFFFF : t16 * 16 + 4 * (lane >> 4) + (bi >> 2) * 16 + (bi & 3);
        // exponents v * sc + nb, one fused multiply-add each.  nb is rounded, by up to 1e-6 where the maximum is large: the
        // sum is off by that power of two as a whole and is put right as a whole.  (Added up four by four: 20 terms in a
        // row would round away more than the 8 of a narrower workgroup.)
        const float nb = best == -INFINITY ? 0.f : -best * sc;
        const float nb_off = best == -INFINITY ? 0.f : fmaf(-best, sc, -nb);
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < NW * 4; i += 4) {                                                 // masked: exp2(-inf) = 0
          float t[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = __builtin_amdgcn_exp2f(fmaf(v[i + e], sc, nb));
          sum += (t[0] + t[1]) + (t[2] + t[3]);
        }
        sum *= __builtin_amdgcn_exp2f(nb_off);
        const int at = (wave * (kStatMT * 16) + ml * 16 + (lane & 15)) * 4 + (lane >> 4);
        st_max[at] = best; st_sum[at] = sum; st_arg[at] = barg;
      }
      lds_barrier();
      // one thread per row merges the WPG x 4 partials in a fixed order and writes the tile's partial
      if (tid < kStatMT * 16 && row0 + h * 16 + tid < M) {
        const float sc = sScale[h * 16 + tid];
        float best = -INFINITY;
        int barg = 0x7FFFFFFF;
#pragma unroll
        for (int w = 0; w < WPG; ++w) {
          const f32x4 m4 = *reinterpret_cast<const f32x4*>(&st_max[(w * (kStatMT * 16) + tid) * 4]);
          const int4 a4 = *reinterpret_cast<const int4*>(&st_arg[(w * (kStatMT * 16) + tid) * 4]);
          const int a[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (m4[g] > best || (m4[g] == best && a[g] < barg)) { best = m4[g]; barg = a[g]; }
        }
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < WPG; ++w) {
          const f32x4 m4 = *reinterpret_cast<const f32x4*>(&st_max[(w * (kStatMT * 16) + tid) * 4]);
          const f32x4 s4 = *reinterpret_cast<const f32x4*>(&st_sum[(w * (kStatMT * 16) + tid) * 4]);
#pragma unroll
          for (int g = 0; g < 4; ++g)
            if (m4[g] != -INFINITY) sum += (double)s4[g] * (double)__builtin_amdgcn_exp2f((m4[g] - best) * sc);
        }
        Partial out;
        out.mx = best; out.arg = barg; out.sum = sum;
        fs.part[(int64_t)(row0 + h * 16 + tid) * fs.nfine + col_tile] = out;
      }
      if (h + kStatMT < MT) lds_barrier();         // the next group overwrites the scratch
    }
  }
  if (!active) return;
  // Epilogue.  After the MFMAs a lane holds Z[row0 + mt*16 + lane%16][(t16 + nw)*16 + 4*(lane/16) + 0..3]: 64-byte
  // pieces of 16 rows per store.  Each 16-row tile is turned through a wave-private LDS patch (padded rows) so that a
  // store instruction writes whole rows of the wavefront's columns contiguously.  With several M-blocks the logits are
  // written with nontemporal stores: they are not re-read by this kernel and should not evict the weights that the
  // other M-blocks of the column tile are about to find in L2 (measured at 160 rows: 242 against 253 us per step).  With
  // one M-block nothing in L2 is worth keeping, and plain stores were measured 1 % faster (144 rows: 205 against 207 us).
  float* patch = sPatch[wave];
  auto store_tiles = [&](auto first_tile, auto n_tiles, int mt) {
    constexpr int nw0 = decltype(first_tile)::value, kTiles = decltype(n_tiles)::value;
    constexpr int kVecPerRow = kTiles * 4;               // float4 per patch row
#pragma unroll
    for (int nw = 0; nw < kTiles; ++nw)
      *reinterpret_cast<f32x4*>(&patch[(lane & 15) * kPatchRow + nw * 16 + 4 * (lane >> 4)]) = acc[mt][nw0 + nw];
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
      const int idx = i * 64 + lane;
      const int r = idx / kVecPerRow, c4 = idx % kVecPerRow;
      const f32x4 v = *reinterpret_cast<const f32x4*>(&patch[r * kPatchRow + 4 * c4]);
      const int m = row0 + mt * 16 + r;
      const int n = (t16 + nw0) * 16 + 4 * c4;
      if (m < M) {
        float* dst = Z + (int64_t)m * ldz + n;
        if (vec_store && n + 3 < V_t) {
          if (W_ONCE) *reinterpret_cast<f32x4*>(dst) = v;
          else __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(dst));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < V_t) dst[e] = v[e];
        }
      }
    }
  };
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    store_tiles(std::integral_constant<int, 0>(), std::integral_constant<int, kPatchNW>(), mt);
    if constexpr (NW > kPatchNW)
      store_tiles(std::integral_constant<int, kPatchNW>(), std::integral_constant<int, NW - kPatchNW>(), mt);
  }
}

// ---------------------------------------------------------------------------------------------------------------
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));   // rows may start at any float

// A row's four logits from column n on.
__device__ __forceinline__ void store_logits(float* __restrict__ dst, int n, int V_t, const f32x4& z) {
  if (n + 4 <= V_t) {
    *reinterpret_cast<f32x4_u*>(dst) = z;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < V_t) dst[e] = z[e];
  }
}

// Exponent scales of an M-block's rows, for the statistics of their logits: thread b holds sequence b's rows and temperature
// (asked for in front of the first weights, at most 255 sequences) and fills in those of the block.
struct BlockScales {
  int lo = 0, hi = 0;
  float T = 0.f;
  __device__ __forceinline__ void load(const FusedStats& fs, int tid) {
    if (fs.part && tid < fs.B) { lo = fs.row_off[tid]; hi = fs.row_off[tid + 1]; T = fs.temperature[tid]; }
  }
  __device__ __forceinline__ void fill(float* s_scale, int row0, int n_rows) const {
    for (int r = max(lo - row0, 0); r < min(hi - row0, n_rows); ++r) s_scale[r] = T > 0.f ? kLog2eF / T : kLog2eF;
  }
};

// Skinny kernel: M <= 16 rows (one MFMA row tile).  A workgroup takes 64 columns at a time and splits the hidden dimension
// over its 8 wavefronts, so that even a 32000-column head yields thousands of wavefronts streaming W; the hidden
// fragments are tiny and read straight from global memory (L2 resident).  The 8 partial tiles are summed through
// LDS in a fixed order; a row's 64 logits end up in 16 lanes, which also form their softmax partial.
// The draft side of the step runs in workgroups of its own in front (n_front of them, see front_draft_side).  Two workgroups fit on
// a compute unit (94 registers, three fetches deep; 144 with four deep and branches around the refills, where 500 + 16 workgroups
// were a third round: 44.4 us for 6 rows x 32000 columns, 40.1 now and without the draft side).  Several tiles per workgroup, so
// that there are fewer partials, empty its pipeline at every tile: 190 to 211 us for 152064 columns instead of 166.
template <int PF>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void lmhead_bf16_skinny_kernel(const uint16_t* __restrict__ H, int M, int d,
                                                                 const uint4* __restrict__ Wp, int nks,
                                                                 float* __restrict__ Z, int V_t, int64_t ldz,
                                                                 const uint16_t* __restrict__ zeros, FusedStats fs, int n_front, StepArgs ds) {
  constexpr int kWaves = 8;
  constexpr int kRow = 17;                          // float4 per padded row of the reduction scratch
  __shared__ f32x4 sRed[kWaves][16 * kRow];
  __shared__ float sScale[16];
  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  const int wg = (int)blockIdx.x - n_front;
  static_assert(sizeof(sRed) >= kFrontLdsBytes, "scratch of the draft side");
  if (wg < 0) {
    front_draft_side<uint16_t, kWaves>(ds, blockIdx.x, tid, sRed);
    return;
  }
  const int wt = wg;
  const int ks0 = (int)(((int64_t)nks * wave) / kWaves), ks1 = (int)(((int64_t)nks * (wave + 1)) / kWaves);
  const int h_col = 8 * (lane >> 4);
  const uint32_t h_at = (uint32_t)(min(lane & 15, M - 1) * d + h_col);   // rows past M are never stored: any valid row will do
  BlockScales scales;
  scales.load(fs, tid);

  const uint4* wp = Wp + (int64_t)wt * packed_tile_units(nks);
  f32x4 acc[4];
#pragma unroll
  for (int nw = 0; nw < 4; ++nw) acc[nw] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 bq[PF][4];
  uint4 hq[PF];
  auto fetch = [&](int slot, int ks) {
    const uint4* w = wp + (int64_t)ks * 256;
#pragma unroll
    for (int nw = 0; nw < 4; ++nw)                 // read once by the whole launch: nontemporal (see the wide kernel)
      bq[slot][nw] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(w + nw * 64 + lane));
    // the padded tail of the hidden dimension must read as zero
    hq[slot] = *reinterpret_cast<const uint4*>(ks * 32 + h_col < d ? H + ks * 32 + h_at : zeros);
  };
  auto multiply = [&](int slot) {
    const bf16x8 hf = __builtin_bit_cast(bf16x8, hq[slot]);
#pragma unroll
    for (int nw = 0; nw < 4; ++nw)
      acc[nw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bq[slot][nw]), hf, acc[nw], 0, 0, 0);
  };
#pragma unroll
  for (int s = 0; s < PF; ++s)
    if (ks0 + s < ks1) fetch(s, ks0 + s);
  int base = ks0;
  for (; base + 2 * PF <= ks1; base += PF) {       // every refill in range: no branch inside
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      multiply(s);
      fetch(s, base + s + PF);
    }
  }
#pragma unroll
  for (int s = 0; s < 2 * PF - 1; ++s) {
    if (base + s < ks1) {
      multiply(s % PF);
      if (s < PF - 1 && base + s + PF < ks1) fetch(s % PF, base + s + PF);
    }
  }
  // acc[nw][e] = partial Z[lane%16][64*wt + 16*nw + 4*(lane/16) + e]
#pragma unroll
  for (int nw = 0; nw < 4; ++nw) sRed[wave][(lane & 15) * kRow + nw * 4 + (lane >> 4)] = acc[nw];
  scales.fill(sScale, 0, 16);
  __syncthreads();
  if (wave >= 4) return;
  const int m = tid >> 4, c = tid & 15;              // row and float4 column of the summed tile
  f32x4 sum = sRed[0][m * kRow + c];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) sum += sRed[w][m * kRow + c];
  const int n = wt * 64 + 4 * c;
  if (m < M) store_logits(Z + (int64_t)m * ldz + n, n, V_t, sum);
  if (fs.part) {
    const float z[4] = {sum[0], sum[1], sum[2], sum[3]};
    const Partial p = partial_of_64(z, n, V_t, sScale[m < M ? m : 0]);
    if (m < M && c == 0) fs.part[(int64_t)m * fs.nfine + wt] = p;
  }
}

// ---------------------------------------------------------------------------------------------------------------
// fp32 head of up to 16 rows or less than 384 hidden indices (f32_plan), on v_mfma_f32_16x16x4_f32 (binary32 products and sums, twice the
// rate of the vector units' fused multiply-adds).  Bound by the matrix cores from about 48 rows on (147 TFLOP/s is what a large fp32
// product reaches on this card), by the weight stream below.  W is re-tiled once at init so that a wavefront's loads are contiguous:
// unit(wt, kb, s, lane), one float4, holds W[16*kb + 4*(lane/16) + s][64*wt + 4*(lane%16) + 0..3], zero outside [d, V_t].
// The four floats of a lane feed four MFMAs, one per interleaved set of 16 columns {64*wt + 4*i + nw}, and a lane's
// float4 of hidden values H[row][16*kb + 4*(lane/16) + 0..3] feeds the four steps s: the hidden index that a lane group
// contributes to an MFMA may be any, as long as both operands take the same.
// A workgroup owns 64 columns and up to 48 rows and splits the hidden dimension over its wavefronts, whose partial tiles
// are summed through LDS in a fixed order: a head of 1024 columns is 16 workgroups of 8 wavefronts, one of 32000 is 500
// per row block.  The row blocks of a column tile run on the same XCD back to back and meet in its L2.
// The launch also leaves softmax partials and takes the draft side (a workgroup per job, or packed into few: f32_row_front), which
// spares the statistics launch: 17.4 -> 14.2 us per step at 5 rows, d = 256, V_t = 1024.  Its registers for that leave four workgroups
// with two row tiles on a compute unit, three with three (f32_plan counts on it).
// Measured with the draft side: 64 rows, d = 256, V_t = 32000 18.9 us; 5 rows, d = 256, V_t = 1024 4.9 to 5.4 us, where a kernel whose
// threads owned one column each over all of the hidden dimension took 68 (4 workgroups of serial chains) and its one long chain per
// logit was off by 6e-7 against 64 bits instead of 1.1e-7.
__global__ __launch_bounds__(256) void pack_w_f32_kernel(const float* __restrict__ W, int d, int V_t,
                                                         float4* __restrict__ Wp, int nkb, int64_t n_units) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u >= n_units) return;
  const int lane = (int)(u & 63), s = (int)((u >> 6) & 3);
  const int64_t rest = u >> 8;
  const int kb = (int)(rest % nkb), wt = (int)(rest / nkb);
  const int k = kb * 16 + 4 * (lane >> 4) + s, n = wt * 64 + 4 * (lane & 15);
  float w[4] = {0.f, 0.f, 0.f, 0.f};
  if (k < d)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < V_t) w[e] = W[(int64_t)k * V_t + n + e];
  Wp[(int64_t)wt * packed_f32_tile_units(nkb) + ((int64_t)kb * 4 + s) * 64 + lane] = make_float4(w[0], w[1], w[2], w[3]);
}

// kStats: partials and the draft side; a launch without them runs the kernel that does not hold their code.
template <int MT, int WAVES, int PF, bool kStats>
__global__ __launch_bounds__(WAVES * 64) void lmhead_f32_kernel(const float* __restrict__ H, int M, int d,
                                                                const f32x4* __restrict__ Wp, int nkb, int n_wtiles,
                                                                float* __restrict__ Z, int V_t, int64_t ldz, int m_blocks,
                                                                FusedStats fs, int n_front, StepArgs ds) {
  constexpr int kRow = 17;                              // float4 per padded row of the reduction scratch
  __shared__ f32x4 sRed[WAVES][MT * 16 * kRow];
  __shared__ float sScale[kStats ? MT * 16 : 1];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  static_assert(sizeof(sRed) >= kFrontLdsBytes && sizeof(sRed) >= WAVES * sizeof(DraftLds), "scratch of the draft side");
  static_assert(WAVES * 64 >= kFusedMaxB, "a thread per sequence");
  const int wg = (int)blockIdx.x - (kStats ? n_front : 0);   // n_front is a multiple of 8: the XCDs below are those of the block ids
  if (kStats && wg < 0) {
    if (ds.plan.base == kDraftPieces) front_draft_side<float, WAVES>(ds, blockIdx.x, tid, sRed);
    else front_draft_rows<float, WAVES, false>(ds, blockIdx.x, n_front, tid, sRed);
    return;
  }
  const int slot = wg >> 3;
  const int wt = (slot / m_blocks) * 8 + (wg & 7), row0 = (slot % m_blocks) * (MT * 16);
  if (wt >= n_wtiles) return;                           // padding of the id space
  BlockScales scales;
  if constexpr (kStats) scales.load(fs, tid);
  const int whole = d / 16;                             // blocks without a ragged end, split over the wavefronts
  const int kb0 = (int)(((int64_t)whole * wave) / WAVES), kb1 = (int)(((int64_t)whole * (wave + 1)) / WAVES);
  const f32x4* wp = Wp + (int64_t)wt * packed_f32_tile_units(nkb) + lane;
  const int g = lane >> 4;
  const float* hp[MT];                                  // rows past M are never stored: any valid row will do
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) hp[mt] = H + (int64_t)min(row0 + mt * 16 + (lane & 15), M - 1) * d + 4 * g;

  f32x4 acc[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nw = 0; nw < 4; ++nw) acc[mt][nw] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 wq[PF][4], hq[PF][MT];
  auto fetch = [&](int st, int kb) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const f32x4* src = wp + ((int64_t)kb * 4 + s) * 64;
      wq[st][s] = m_blocks == 1 ? __builtin_nontemporal_load(src) : *src;   // read once by the whole launch: nontemporal
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) hq[st][mt] = *reinterpret_cast<const f32x4_u*>(hp[mt] + kb * 16);
  };
  auto multiply = [&](int st) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nw = 0; nw < 4; ++nw)
          acc[mt][nw] = __builtin_amdgcn_mfma_f32_16x16x4f32(wq[st][s][nw], hq[st][mt][s], acc[mt][nw], 0, 0, 0);
  };
#pragma unroll
  for (int st = 0; st < PF; ++st)
    if (kb0 + st < kb1) fetch(st, kb0 + st);
  int base = kb0;
  for (; base + 2 * PF <= kb1; base += PF) {            // every refill in range: no branch inside
#pragma unroll
    for (int st = 0; st < PF; ++st) {
      multiply(st);
      fetch(st, base + st + PF);
    }
  }
#pragma unroll
  for (int st = 0; st < 2 * PF - 1; ++st) {
    if (base + st < kb1) {
      multiply(st % PF);
      if (st < PF - 1 && base + st + PF < kb1) fetch(st % PF, base + st + PF);
    }
  }
  if (wave == WAVES - 1 && whole < nkb) {               // the ragged end of the hidden dimension reads as zero
    const int left = d - (whole * 16 + 4 * g);
#pragma unroll
    for (int s = 0; s < 4; ++s) wq[0][s] = wp[((int64_t)whole * 4 + s) * 64];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < 4; ++e) hq[0][mt][e] = e < left ? hp[mt][whole * 16 + e] : 0.f;
    multiply(0);
  }
  // acc[mt][nw][e] = partial Z[row0 + 16*mt + lane%16][64*wt + 4*(4*(lane/16) + e) + nw]
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      sRed[wave][(mt * 16 + (lane & 15)) * kRow + 4 * g + e] = f32x4{acc[mt][0][e], acc[mt][1][e], acc[mt][2][e], acc[mt][3][e]};
  if constexpr (kStats) scales.fill(sScale, row0, MT * 16);
  __syncthreads();
  for (int i = tid; i < MT * 256; i += WAVES * 64) {
    const int r = i >> 4, c = i & 15;
    f32x4 sum = sRed[0][r * kRow + c];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) sum += sRed[w][r * kRow + c];
    const int m = row0 + r, n = wt * 64 + 4 * c;
    if (m < M) store_logits(Z + (int64_t)m * ldz + n, n, V_t, sum);
    if constexpr (kStats) {
      const float z[4] = {sum[0], sum[1], sum[2], sum[3]};
      const Partial p = partial_of_64(z, n, V_t, sScale[m < M ? r : 0]);
      if (m < M && c == 0) fs.part[(int64_t)m * fs.nfine + wt] = p;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// fp32 head of more than 16 rows and a longer hidden dimension (f32_plan), on the bf16 matrix instruction, which is sixteen times as
// fast as the binary32 one.  A binary32 value is the sum of three bf16 values, exactly: the nearest one, the nearest one to what is
// left, and the rest (24 significant bits, of which each of the first two takes eight and leaves a remainder of either sign).  Of the
// nine products of two such triples the six largest are formed (each exact, added up in binary32); what is left out is at most 2^-24 of
// a product and leans to no side.  (Parts cut off instead of rounded all have the sign of the value: up to 2^-21 left out, always
// towards zero, 4.5e-7 of the logit of a token that its hidden row lies along.)  A rounding per 32 products instead of one per 4: error
// against 64 bits at 64 rows x 32000 columns, d = 1024, eight seeds, here / with the binary32 instruction: logits 2.3e-7 / 2.9e-7 of
// their norm, probabilities of the proposed tokens 3.0e-7 / 3.2e-7, their ratios 2.4e-7 / 2.6e-7.
// Same packed weights and the same split over four wavefronts as above; a step is two blocks of 16 hidden indices.  Bound by the
// loads: of 36 us at 64 rows x 32000 columns (d = 1024; 45.8 with the binary32 instruction; 0.3 less with parts cut off) 25 are left
// without the hidden rows' traffic (one L2 read of all rows per 64 columns), the splits and half of the products, 30 with the traffic
// alone.  Tried instead: the hidden rows' thirds shared through LDS, wavefronts by columns and halves of the hidden dimension: 43 us, a
// barrier per 64 hidden indices and longer chains of sums (3.4e-7).
struct Thirds { bf16x8 part[3]; };
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Thirds split_thirds(const float (&x)[8], float& largest) {
  uint32_t w[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) largest = fmaxf(fmaxf(__builtin_fabsf(x[2 * i]), __builtin_fabsf(x[2 * i + 1])), largest);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      w[t][i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));   // to nearest
      if (t < 2) {
        a -= __uint_as_float(w[t][i] << 16);
        b -= __uint_as_float(w[t][i] & 0xFFFF0000u);
      }
    }
  }
  Thirds r;
#pragma unroll
  for (int t = 0; t < 3; ++t) r.part[t] = __builtin_bit_cast(bf16x8, make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]));
  return r;
}

template <int MT, bool kStats>
__global__ __launch_bounds__(256, MT == 2 ? 3 : 2) void lmhead_f32_thirds_kernel(const float* __restrict__ H, int M, int d,
                                                                   const f32x4* __restrict__ Wp, int nkb, int n_wtiles,
                                                                   float* __restrict__ Z, int V_t, int64_t ldz, int m_blocks,
                                                                   FusedStats fs, int n_front, StepArgs ds) {
  constexpr int kWaves = 4;
  constexpr int kRow = 17;                              // float4 per padded row of the reduction scratch
  __shared__ f32x4 sRed[kWaves][MT * 16 * kRow];
  __shared__ float sScale[kStats ? MT * 16 : 1];
  __shared__ int sBad[kWaves];
  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  static_assert(sizeof(sRed) >= kFrontLdsBytes && sizeof(sRed) >= kWaves * sizeof(DraftLds), "scratch of the draft side");
  static_assert(kWaves * 64 >= kFusedMaxB, "a thread per sequence");
  const int wg = (int)blockIdx.x - (kStats ? n_front : 0);   // n_front is a multiple of 8: the XCDs below are those of the block ids
  if (kStats && wg < 0) {
    if (ds.plan.base == kDraftPieces) front_draft_side<float, kWaves>(ds, blockIdx.x, tid, sRed);
    else front_draft_rows<float, kWaves, true, MT == 2 ? 8 : 16>(ds, blockIdx.x, n_front, tid, sRed);
    return;
  }
  const int slot = wg >> 3;
  const int wt = (slot / m_blocks) * 8 + (wg & 7), row0 = (slot % m_blocks) * (MT * 16);
  if (wt >= n_wtiles) return;                           // padding of the id space
  BlockScales scales;
  if constexpr (kStats) scales.load(fs, tid);
  // steps of two 16-deep blocks without a ragged end, split over the wavefronts; the last one takes what is left over
  const int pairs = d / 32;
  const int p0 = pairs * wave / kWaves, p1 = pairs * (wave + 1) / kWaves;
  const f32x4* wp = Wp + (int64_t)wt * packed_f32_tile_units(nkb) + lane;
  const int g = lane >> 4;
  const float* hp[MT];                                  // rows past M are never stored: any valid row will do
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) hp[mt] = H + (int64_t)min(row0 + mt * 16 + (lane & 15), M - 1) * d + 4 * g;

  f32x4 acc[MT][4];
  f32x4 wq[2][8], hq[MT][2];
  float largest = 0.f;                                  // absolute value of an operand
  auto clear = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nw = 0; nw < 4; ++nw) acc[mt][nw] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto fetch_w = [&](int st, int p) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const f32x4* src = wp + ((int64_t)p * 8 + i) * 64;
      wq[st][i] = m_blocks == 1 ? __builtin_nontemporal_load(src) : *src;   // read once by the whole launch: nontemporal
    }
  };
  auto fetch_h = [&](int p) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j) hq[mt][j] = *reinterpret_cast<const f32x4_u*>(hp[mt] + p * 32 + j * 16);
  };
  // What is left of the hidden dimension behind the whole steps (fewer than 32): reads as zero past its end.
  auto fetch_rest = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) wq[0][i] = wp[(int64_t)min(pairs * 8 + i, nkb * 4 - 1) * 64];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int k = pairs * 32 + j * 16 + 4 * g + e;
          const float x = hp[mt][min(k, d - 1) - 4 * g];
          hq[mt][j][e] = k < d ? x : 0.f;
        }
  };
  // One step out of weight slot st, which is refilled for step next_w once its values are split, the hidden values for next_h.
  auto step = [&](auto refill, int st, int next_w, int next_h) {
    constexpr bool kRefill = decltype(refill)::value;
    Thirds h[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = hq[mt][i / 4][i % 4];
      h[mt] = split_thirds(x, largest);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (kRefill) fetch_h(next_h);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int nw = 0; nw < 4; ++nw) {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = wq[st][i][nw];
      const Thirds w = split_thirds(x, largest);
      constexpr int kW[6] = {2, 0, 1, 1, 0, 0}, kH[6] = {0, 2, 1, 0, 1, 0};   // the small products first
#pragma unroll
      for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][nw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.part[kW[i]], h[mt].part[kH[i]], acc[mt][nw], 0, 0, 0);
    }
    if (kRefill) fetch_w(st, next_w);
    __builtin_amdgcn_sched_barrier(0);
  };
  clear();
  if (p0 < p1) {
    // a refill past this wavefront's last step asks for that again: no branch inside
    fetch_w(0, p0);
    fetch_h(p0);
    fetch_w(1, min(p0 + 1, p1 - 1));
    for (int p = p0;; p += 2) {
      step(std::true_type(), 0, min(p + 2, p1 - 1), min(p + 1, p1 - 1));
      if (p + 1 >= p1) break;
      step(std::true_type(), 1, min(p + 3, p1 - 1), min(p + 2, p1 - 1));
      if (p + 2 >= p1) break;
    }
  }
  const bool rest = wave == kWaves - 1 && pairs * 2 < nkb;
  if (rest) {
    fetch_rest();
    step(std::false_type(), 0, 0, 0);
  }
  // An infinite or NaN operand does not survive the split (inf - inf), and 0 times an infinite part is no longer the product.  The
  // last part of an operand below 2^-110 is rounded to a multiple of 2^-133, the least bf16 value: less than 2^-73 of a product with
  // an operand below 2^60.  A workgroup that ends up with a logit that is not finite, or met an operand of 2^60 or more, forms its tile
  // again on the binary32 matrix instruction.
  auto sound = [&]() {
    bool ok = largest < 0x1p60f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nw = 0; nw < 4; ++nw)
#pragma unroll
        for (int e = 0; e < 4; ++e) ok = ok && __builtin_fabsf(acc[mt][nw][e]) < INFINITY;
    return __ballot(!ok) == 0ull;
  };
  // acc[mt][nw][e] = partial Z[row0 + 16*mt + lane%16][64*wt + 4*(4*(lane/16) + e) + nw]
  auto park = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sRed[wave][(mt * 16 + (lane & 15)) * kRow + 4 * g + e] = f32x4{acc[mt][0][e], acc[mt][1][e], acc[mt][2][e], acc[mt][3][e]};
  };
  park();
  const bool ok = sound();
  if (lane == 0) sBad[wave] = !ok;
  if constexpr (kStats) scales.fill(sScale, row0, MT * 16);
  __syncthreads();
  if (sBad[0] | sBad[1] | sBad[2] | sBad[3]) {          // workgroup-uniform
    clear();
    auto multiply_f32 = [&]() {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int nw = 0; nw < 4; ++nw)
            acc[mt][nw] = __builtin_amdgcn_mfma_f32_16x16x4f32(wq[0][i][nw], hq[mt][i / 4][i % 4], acc[mt][nw], 0, 0, 0);
    };
    for (int p = p0; p < p1; ++p) {
      fetch_w(0, p);
      fetch_h(p);
      multiply_f32();
    }
    if (rest) {
      fetch_rest();
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (pairs * 8 + i >= nkb * 4) wq[0][i] = f32x4{0.f, 0.f, 0.f, 0.f};   // no such block: its stand-in may be infinite
      multiply_f32();
    }
    __syncthreads();
    park();
    __syncthreads();
  }
  for (int i = tid; i < MT * 256; i += kWaves * 64) {
    const int r = i >> 4, c = i & 15;
    f32x4 sum = sRed[0][r * kRow + c];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) sum += sRed[w][r * kRow + c];
    const int m = row0 + r, n = wt * 64 + 4 * c;
    if (m < M) store_logits(Z + (int64_t)m * ldz + n, n, V_t, sum);
    if constexpr (kStats) {
      const float z[4] = {sum[0], sum[1], sum[2], sum[3]};
      const Partial p = partial_of_64(z, n, V_t, sScale[m < M ? r : 0]);
      if (m < M && c == 0) fs.part[(int64_t)m * fs.nfine + wt] = p;
    }
  }
}

// Front workgroups of the kernels that give each draft-side job one: a sequence's lookups, a piece of a draft row.
int front_jobs(const StepArgs& a) { return a.B + a.plan.jobs(a.K); }
bool front_plan_fits(const StepArgs& a) {
  return a.K >= 1 && a.B >= 1 && a.plan.base >= 1 && a.plan.more >= 0 && a.plan.more <= a.K &&
         a.plan.base + (a.plan.more > 0) <= kDraftPieces &&
         (int64_t)a.plan.more * (a.plan.base + 1) + (int64_t)(a.K - a.plan.more) * a.plan.base == a.plan.workers;
}

// How more than 16 rows of an fp32 head run: row tiles per block, and the kernel.
// Below 384 hidden indices a wavefront of the thirds kernel has less than three steps, and the other one is faster or even (24 to 64 rows
// x 32000 columns, d = 256: 2 to 6 %, d = 64: 4 to 17 %); from there on the thirds are, by 9 % over 84 shapes at d = 384, 15 % over 378
// at d = 512 and 1024, 34 % at 256 rows x 32000 columns.  The other one takes two row tiles, or three where that pads less (48 rows,
// 144 rows); smaller blocks read the weights again out of L2 but put more wavefronts on a compute unit, which cover its loads.  The
// thirds kernel takes the block whose workgroups cost the fullest compute unit least, 2 + 2.5 per row tile each (us at d = 1024, measured
// at 24 to 256 rows x 1000 to 100000 columns: a step takes 19 us more than their sum): small heads fill the chip with small blocks, large
// ones split the weights less often.  64 rows x 8000 / 32000 columns, us per step with blocks of 2 / 3 / 4 tiles 25.8 / 29.0 / 31.1 and
// 47.3 / 56.8 / 46.1, 80 rows x 32000 59.3 / 56.9 / 67.3.
struct F32Plan { int tiles; bool thirds; int workgroups, at_once; };   // workgroups that multiply; that the chip holds at once
F32Plan f32_plan(int M, int d, int V_t, int n_cu) {
  const int tiles = ceil_div(M, 16), n_wtiles = ceil_div(V_t, 64);
  F32Plan p{1, false, 0, 2 * n_cu};
  if (tiles > 1 && d < 384) {
    p.tiles = ceil_div(tiles, 3) * 3 < ceil_div(tiles, 2) * 2 ? 3 : 2;
    p.at_once = n_cu * (p.tiles == 2 ? 4 : 3);
  } else if (tiles > 1) {
    p.thirds = true;
    double least = INFINITY;
    for (int mt = 2; mt <= 4; ++mt) {
      const double cost = ceil_div((int64_t)n_wtiles * ceil_div(tiles, mt), std::max(n_cu, 1)) * (2.0 + 2.5 * mt);
      if (cost < least) { least = cost; p.tiles = mt; }
    }
    p.at_once = n_cu * (p.tiles == 2 ? 3 : 2);
  }
  p.workgroups = ceil_div(n_wtiles, 8) * 8 * ceil_div(tiles, p.tiles);
  return p;
}

// Front workgroups of an fp32 launch that takes the draft side by whole rows: few, because its multiplying workgroups fill the
// chip, and no more than its last round has room for.  (64 rows, d = 1024, V_t = 32000: 1000 workgroups, four to a compute unit; a
// workgroup for each of 16 sequences' lookups and 48 rows' pieces put some of those back by a round: 50.8 us instead of 46.2.)
int f32_row_front(const F32Plan& p, int B, int K) {
  const int want = std::min(32, ceil_div(std::max(B, ceil_div(K, 4)), 8) * 8);
  if (!p.thirds) return want;
  const int room = (ceil_div(p.workgroups, std::max(p.at_once, 1)) * p.at_once - p.workgroups) / 8 * 8;
  return room >= 8 ? std::min(want, room) : want;
}

template <int MT>
hipError_t launch_f32_thirds(const float* H, int M, int d, const float* Wp, float* Z, int V_t, int64_t ldz, const FusedStats& fs,
                             const StepArgs* draft_side, const F32Plan& plan, hipStream_t stream) {
  const int nkb = ceil_div(d, 16), n_wtiles = ceil_div(V_t, 64), m_blocks = ceil_div(M, MT * 16);
  const int n_front = !draft_side ? 0 : draft_side->plan.base == kDraftPieces ? ceil_div(front_jobs(*draft_side), 8) * 8
                                                                              : f32_row_front(plan, draft_side->B, draft_side->K);
  const dim3 grid((unsigned)(n_front + ceil_div(n_wtiles, 8) * 8 * m_blocks)), block(256);
  const f32x4* wp = reinterpret_cast<const f32x4*>(Wp);
  if (fs.part)
    hipLaunchKernelGGL((lmhead_f32_thirds_kernel<MT, true>), grid, block, 0, stream, H, M, d, wp, nkb, n_wtiles, Z, V_t, ldz,
                       m_blocks, fs, n_front, draft_side ? *draft_side : StepArgs{});
  else
    hipLaunchKernelGGL((lmhead_f32_thirds_kernel<MT, false>), grid, block, 0, stream, H, M, d, wp, nkb, n_wtiles, Z, V_t, ldz,
                       m_blocks, fs, 0, StepArgs{});
  return hipGetLastError();
}

template <int MT, int WAVES, int PF>
hipError_t launch_f32(const float* H, int M, int d, const float* Wp, float* Z, int V_t, int64_t ldz, const FusedStats& fs,
                      const StepArgs* draft_side, const F32Plan& plan, hipStream_t stream) {
  const int nkb = ceil_div(d, 16), n_wtiles = ceil_div(V_t, 64), m_blocks = ceil_div(M, MT * 16);
  const int n_front = !draft_side ? 0 : draft_side->plan.base == kDraftPieces ? ceil_div(front_jobs(*draft_side), 8) * 8
                                                                              : f32_row_front(plan, draft_side->B, draft_side->K);
  const dim3 grid((unsigned)(n_front + ceil_div(n_wtiles, 8) * 8 * m_blocks)), block(WAVES * 64);
  const f32x4* wp = reinterpret_cast<const f32x4*>(Wp);
  if (fs.part)
    hipLaunchKernelGGL((lmhead_f32_kernel<MT, WAVES, PF, true>), grid, block, 0, stream, H, M, d, wp, nkb, n_wtiles, Z, V_t, ldz,
                       m_blocks, fs, n_front, draft_side ? *draft_side : StepArgs{});
  else
    hipLaunchKernelGGL((lmhead_f32_kernel<MT, WAVES, PF, false>), grid, block, 0, stream, H, M, d, wp, nkb, n_wtiles, Z, V_t, ldz,
                       m_blocks, fs, 0, StepArgs{});
  return hipGetLastError();
}

// Rows above which an M-block is split: up to 11 row tiles run as one block that streams every weight once.  Measured at
// 160 / 176 rows (d = 4096, V_t = 128256): 217 / 225 us per step as one block against 244 / 246 us as two.
constexpr int kSingleBlockRows = 176;

// Rough duration of an LM-head launch: the weights stream at 6 TB/s or the product runs at 1 PFLOP/s, whichever is longer.
double lmhead_launch_us(int M, int d, int Vp) { return std::max(2.0 * d * (double)Vp / 6.0e6, 2.0 * M * d * (double)Vp / 1.0e9); }

// How more than 176 rows run: as several M-blocks per column tile (their weight streams meet in one L2), of `tiles` row
// tiles each, by the kernel whose wavefronts own 32 columns or by the one whose wavefronts own 64 (`wide`).  That regime
// is bound by the L2 -> LDS traffic, LDS reads and the card's power, and the launch runs in rounds of one workgroup per
// compute unit, on each of the eight XCDs by itself (a column tile and its M-blocks stay on one: 99 tiles of 5 blocks are 65
// workgroups on three of them, a third round on 32 compute units).  The estimate was fitted to all eleven blocks at 247
// shapes (d = 512 to 4096, 8000 to 152064 columns, 184 to 1024 rows): a few us outside the loop plus 14 + 5.6 per row tile in
// it for 256 columns at d = 3584; with 64 columns per wavefront a hidden fragment read from LDS feeds four MFMAs instead of two
// and a column costs 17 % less, but the accumulators leave room for 11 row tiles at most.  A round that is partly empty
// costs about 0.6 of what it leaves idle (the clock of the busy part rises).  The block it takes is 0.25 % slower than the
// best one on average and 4 % at most; blocks chosen by their height alone were 13 % slower on average and up to 2.4 times
// (and better by 2 to 3 % at five shapes).  Measured, us per step, against those: 192 / 512 rows on V_t = 8000 (d = 4096)
// 52 / 62 against 99 / 145, on V_t = 33024 184 / 400 rows 97 / 142 against 97 / 142, 1024 rows on V_t = 128256 1018 against 1076.
struct TallPlan { int tiles; bool wide; int workgroups; double rounds, round_us; };
TallPlan tall_plan(int M, int d, int Vp, int n_cu) {
  TallPlan best{9, false, 0, 1.0, INFINITY};
  auto consider = [&](int mt, int cols, double outside, double per_column) {
    const int workgroups = ceil_div(ceil_div(Vp, cols), 8) * 8 * ceil_div(M, 16 * mt);   // eight times those of the fullest XCD
    const double per_cu = workgroups / std::max(1.0, (double)n_cu);
    const double rounds = per_cu < 1.0 ? 0.61 + 0.39 * per_cu : 0.42 * per_cu + 0.58 * std::ceil(per_cu);
    const TallPlan p{mt, cols == 512, workgroups, rounds, outside + d / 3584.0 * (14 + 5.6 * mt) * per_column * cols / 256};
    if (p.rounds * p.round_us < best.rounds * best.round_us) best = p;
  };
  for (int mt : {4, 6, 9, 10, 12, 14, 16, 18}) consider(mt, 256, 5.0, 1.0);
  for (int mt : {9, 10, 11}) consider(mt, 512, 9.0, 0.83);
  return best;
}

// Front workgroups of a launch that hosts the draft side with several M-blocks: one per four sequences (the lookups go
// four sequences at a time), a multiple of 8 (the XCD mapping of the multiplying workgroups holds), 8 to 64.  A
// workgroup that only reads, next to the multiplying ones, draws about 8 GB/s however much it keeps in flight (measured:
// 8 of them need 280 us for the 18.4 MB of 288 draft rows), so the compute-unit time the draft rows cost is given by
// their bytes; few front workgroups keep that time inside the slack of the last round of multiplying workgroups, many push
// some of those into a round of their own.  0: one M-block, where the multiplying workgroups take the draft side themselves.
constexpr double kFrontBytesPerUs = 8e3;     // one front workgroup, next to the multiplying ones
int lmhead_bf16_front_workgroups(int M, int B) {
  if (M <= kSingleBlockRows) return 0;
  return std::min(64, std::max(8, ceil_div(ceil_div(B, 4), 8) * 8));
}
constexpr int kWideWaves = 8;      // wavefronts per workgroup of every wide kernel: each one of a front workgroup is a worker

template <int MT, int PF, int WPG, int KC, int NW, bool W_ONCE = false>
hipError_t launch_wide(const uint16_t* H, int M, int d, const uint16_t* Wp, int Kp, int Vp, float* Z, int V_t,
                       int64_t ldz, const uint16_t* zeros, const FusedStats& fs, const StepArgs* draft_side, int n_cu,
                       hipStream_t stream) {
  const int nks = Kp / 32, n_wtiles = Vp / kGemmColsPerWave;
  const int m_blocks = ceil_div(M, MT * 16);
  const int col_tiles = ceil_div(n_wtiles * 4, WPG * NW);
  StepArgs ds{};
  int n_front = 0, n_piece_jobs = 0, helpers_look_up = 0;
  const int padded_tiles = ceil_div(col_tiles, 8) * 8;
  if (draft_side && fs.part) {
    ds = *draft_side;
    const PiecePlan& plan = ds.plan;
    static_assert(WPG == kWideWaves, "the plan of the front workgroups counts on this many wavefronts each");
    n_front = lmhead_bf16_front_workgroups(M, ds.B);
    const int workers = n_front > 0 ? n_front * WPG : col_tiles * m_blocks;
    if (ds.K < 1 || plan.workers < 1 || plan.workers > workers || plan.base < 1 ||
        plan.base + (plan.more > 0) > kDraftPieces || plan.more < 0 || plan.more > ds.K ||
        (plan.workers < ds.K && (plan.base != 1 || plan.more != 0)))
      return hipErrorInvalidValue;
    n_piece_jobs = plan.jobs(ds.K);
    // the workgroups that pad the id space take the sequences' lookups if they finish well inside the launch: about
    // 60 us per four sequences (a chain of about six dependent loads next to the saturating weight streams) against
    // the time the weights take to stream or the product to be formed
    const int helpers = (padded_tiles - col_tiles) * m_blocks;
    if (n_front == 0 && helpers > 0 && ceil_div(ds.B, 4 * helpers) * 60.0 <= 0.5 * lmhead_launch_us(M, d, Vp))
      helpers_look_up = 1;
  }
  dim3 grid(n_front + padded_tiles * m_blocks), block(WPG * 64);
  const int vec_store = (ldz % 4 == 0) && (reinterpret_cast<uintptr_t>(Z) % 16 == 0);
  if (W_ONCE && m_blocks != 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL((lmhead_bf16_wide_kernel<MT, PF, WPG, KC, NW, W_ONCE>), grid, block, 0, stream, H, M, d,
                     reinterpret_cast<const uint4*>(Wp), nks, n_wtiles, Z, V_t, ldz, vec_store, zeros, m_blocks, fs,
                     n_front, n_piece_jobs, helpers_look_up, ds);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pack_w_bf16(const uint16_t* W, int d, int V_t, uint16_t* Wp, int Kp, int Vp, hipStream_t stream) {
  const int nks = Kp / 32;
  const int64_t n_units = (int64_t)(Vp / 64) * nks * 256;
  hipLaunchKernelGGL(pack_w_kernel, dim3((unsigned)((n_units + 255) / 256)), dim3(256), 0, stream, W, d, V_t,
                     reinterpret_cast<uint4*>(Wp), nks, n_units);
  return hipGetLastError();
}

// Columns per workgroup of the wide kernels.  A single M-block streams every weight once, bound by HBM, one workgroup per
// CU: the launch runs in rounds, a round costs its stream time whether or not all CUs take part, and what a workgroup
// does outside its main loop (first loads, row statistics, stores: about 12 us) is time its CU does not stream.  So the
// width is the one whose rounds stream the fewest columns, 40 more counted per round: up to 32768 columns run as one round
// of 128-column workgroups, up to 65536 of 256, and so on.  Measured on 256 CUs, us per step at 24 / 80 / 128 rows:
//   V_t = 32000, d = 4096:  128 columns 62 / 74 / 86, 256: 75 / 87 / 100 (125 workgroups)
//   V_t = 80000, d = 4096:  384 columns 123 / 136 / 149, 256: 144 / 164 / 196 (two rounds), 512: 132 / 150 / 165
//   V_t = 152064, d = 3584: 640 columns 191 / 204 / 223, 256: 221 / 244 / 278 (three rounds), 384: 214 / 237 / 255 (two)
// 80 columns per wavefront leave accumulators for 8 row tiles (9 spill: 590 us).  Workgroups of 128 columns are taken in a
// single round only: in several they lose to every other width, and a row would have more than 256 partials.
int lmhead_bf16_tile_cols(int M, int d, int Vp, int n_cu) {
  if (M > kSingleBlockRows) return tall_plan(M, d, Vp, n_cu).wide ? 512 : 256;
  if (M <= 16 || n_cu < 1) return 256;
  constexpr int kOutsideLoop = 40;
  int best = 256, best_cost = ceil_div(ceil_div(Vp, 256), n_cu) * (256 + kOutsideLoop);
  for (int cols : {128, 384, 512, 640}) {
    if ((cols == 128 && Vp > cols * n_cu) || (cols == 640 && M > 128)) continue;
    const int cost = ceil_div(ceil_div(Vp, cols), n_cu) * (cols + kOutsideLoop);
    if (cost < best_cost) { best = cols; best_cost = cost; }
  }
  return best;
}

int lmhead_bf16_fused_partials(int M, int d, int Vp, int n_cu) {
  if (M <= 16) return Vp / kGemmColsPerWave;
  return ceil_div(Vp, lmhead_bf16_tile_cols(M, d, Vp, n_cu));
}

// Workgroups of launch_lmhead_bf16 that share the draft rows when the launch hosts the draft side: the multiplying
// ones with a single M-block (their number: one per tile of columns), workgroups of their own or front ones otherwise.
int lmhead_bf16_draft_workers(int M, int d, int Vp, int B, int K, int n_cu) {
  const int nfine = lmhead_bf16_fused_partials(M, d, Vp, n_cu);
  if (M <= 16) return kDraftPieces * K;      // workgroups of their own
  return M > kSingleBlockRows ? lmhead_bf16_front_workgroups(M, B) * kWideWaves : nfine;
}

// Partials per row of up to 16 rows beyond which these are merged by a statistics launch over the logits instead: every workgroup
// of the draw merges its sequence's rows, 512 partials a round trip.  6 rows: 500 partials (32000 columns) 49.1 us per step against
// 53.4 with a statistics launch; 2376 (152064 columns) 179.7 against 178.3, the launch that merges takes 13.4 us instead of 7.9.
constexpr int kMaxMergedPartials = 1024;
// Whether the pieces of draft rows of row_bytes each, a workgroup on each, end before a launch of head_us does, or no later than a
// statistics launch behind it would: a workgroup that only reads draws 8 KB per us next to the weight streams.
static bool front_pieces_end_in_time(double row_bytes, double head_us) {
  return row_bytes / kDraftPieces / kFrontBytesPerUs <= head_us + 5.0;
}

// Whether the LM-head launch should host the draft side (the draft rows' statistics, the drafted ids' lookups, and the
// target rows' softmax partials from its epilogue).  With a single M-block hosting spares the statistics launch and its
// pass over the logits (about 5 TB/s), and costs a workgroup its piece of a draft row and the row statistics of its tile.
// Hosted where a piece is at most half a row, or where the pass over the logits would take 9 us per row of a workgroup.
// Heads of 128-column workgroups are never hosted: their logits are few and their epilogues many.  Measured, us per step
// hosted / separate: V_t = 128256, 128 rows 82 / 92 (d = 1024); V_t = 48000, 96 rows 98 / 101, 128 rows (whole draft rows)
// 117 / 108; V_t = 60000, 168 rows 102 / 87 (d = 2048); V_t = 32000, 80 rows 74 / 72; V_t = 8000, 80 rows 64 / 58.
// With several M-blocks front workgroups take the draft side: hosted where the launch, with them in its rounds, is estimated to end
// before a launch without them and the statistics pass, over the draft rows alone if the launch still leaves the target rows'
// partials.  The row statistics cost a round of multiplying workgroups kStatsUs in either structure; the partials alone cost a launch
// more (8 us with its draft rows' chunks merged).  Both are fitted to 240 shapes (d = 1024 and 4096, 8000 to 152064 columns, 192 to 1024
// rows, draft rows of 8000 and 32000 ids), each timed in all three structures: the choice costs 0.5 % on average against the best, 15 %
// at most (400 rows x 20001, d = 1024, draft rows of 8000: separate 53.9, hosted 46.6); without the partials alone the best choice of
// the other two costs 1.9 %.  us per step, hosted / separate / partials alone: 1024 rows x 128256 1039 / -- / 1003, 512 rows x 128256
// (d = 1024) 245 / 218 / 193, 240 rows 129 / 116 / 114, 320 rows x 50000 (d = 1024) 59.7 / 67.7 / 64.5, 192 rows x 8000 (d = 1024) 41.7 / 26.0 /
// 28.5.  Front workgroups cost most where they push multiplying ones into a round more: V_t = 128256, 320 rows (502 + 16 workgroups) 412
// us hosted, 365 separate.
int lmhead_bf16_hosts(int M, int d, int Vp, int B, int K, int V_d, int n_cu) {
  if (B < 1 || B > kFusedMaxB || K < 1) return kHostsNothing;
  const int workers = lmhead_bf16_draft_workers(M, d, Vp, B, K, n_cu);
  if (M <= 16)
    return Vp / kGemmColsPerWave <= kMaxMergedPartials && front_pieces_end_in_time(2.0 * V_d, lmhead_launch_us(M, d, Vp)) ? kHostsAll
                                                                                                                         : kHostsNothing;
  if (M <= kSingleBlockRows) {
    if (lmhead_bf16_tile_cols(M, d, Vp, n_cu) < 256) return kHostsNothing;
    return 2 * K <= workers || 4.0 * M * Vp / 5.0e6 >= 9.0 * ceil_div(K, workers) ? kHostsAll : kHostsNothing;
  }
  const int n_front = workers / kWideWaves;
  const TallPlan plan = tall_plan(M, d, Vp, n_cu);
  const double front_us = 2.0 * K * (double)V_d / (n_front * kFrontBytesPerUs) + ceil_div(B, 4 * n_front) * 10.0;
  if (n_front >= n_cu) return kHostsNothing;
  // The launch ends at the first moment by which n_front compute units that come free after front_us and the others have
  // had room for all workgroups, each kStatsUs longer for the row statistics; 0.4 of what stays idle counts (0.5 sent
  // 1024 rows x 50000, d = 1024, to the partials alone, 162 us per step instead of 154).
  constexpr double kStatsUs = 7.0;
  const double t = plan.round_us + kStatsUs, n = plan.workgroups;
  const double rounds_alone = std::ceil(n / (n_cu - n_front) - 1e-9);          // the front's compute units never join
  double end = rounds_alone * t;
  for (int front_rounds = 1; front_us + front_rounds * t < end; ++front_rounds) {
    const double at = front_us + front_rounds * t;
    if ((n_cu - n_front) * std::floor(at / t) + n_front * front_rounds >= n) end = at;
  }
  for (double at = t; at < end; at += t)
    if ((n_cu - n_front) * std::round(at / t) + n_front * std::floor(std::max(0.0, at - front_us) / t) >= n) end = at;
  const double hosted = std::max(front_us, 0.4 * end + 0.6 * (n * t + n_front * front_us) / n_cu);
  const double draft_us = 2.0 * K * (double)V_d / 5.0e6;
  const double separate = plan.rounds * plan.round_us + 4.0 + 4.0 * M * Vp / 5.0e6 + draft_us;
  const double partials = plan.rounds * (plan.round_us + kStatsUs) + 8.0 + draft_us;
  return hosted < std::min(separate, partials) ? kHostsAll : partials < separate ? kHostsPartials : kHostsNothing;
}

hipError_t launch_lmhead_bf16(const uint16_t* H, int M, int d, const uint16_t* Wp, int Kp, int Vp, float* Z, int V_t,
                              int64_t ldz, const uint16_t* zeros, const FusedStats* fused, const StepArgs* draft_side,
                              int n_cu, hipStream_t stream) {
  if (M == 0) return hipSuccess;
  const int tiles = ceil_div(M, 16);
  FusedStats fs{};
  if (fused && fused->part) {
    if (fused->nfine != lmhead_bf16_fused_partials(M, d, Vp, n_cu) || fused->B < 1 || fused->B > kFusedMaxB)
      return hipErrorInvalidValue;
    fs = *fused;
  }
  if (tiles <= 1) {
    const int nks = Kp / 32, n_wtiles = Vp / kGemmColsPerWave;
    const bool hosts = draft_side && fs.part;
    if (hosts && !front_plan_fits(*draft_side)) return hipErrorInvalidValue;
    const int n_front = hosts ? front_jobs(*draft_side) : 0;
    hipLaunchKernelGGL((lmhead_bf16_skinny_kernel<3>), dim3(n_front + n_wtiles), dim3(512), 0, stream, H, M, d,
                       reinterpret_cast<const uint4*>(Wp), nks, Z, V_t, ldz, zeros, fs, n_front,
                       hosts ? *draft_side : StepArgs{});
    return hipGetLastError();
  }
  if (M <= kSingleBlockRows) {
    // 64 to 96 KB of weights in flight per workgroup at every width; hidden slices of 64 columns where LDS holds no 128
    const int tile_cols = lmhead_bf16_tile_cols(M, d, Vp, n_cu);
#define OT_WIDE(cols, mt, pf, kc)                                                                                        \
  if (tile_cols == cols && tiles <= mt)                                                                                  \
    return launch_wide<mt, pf, 8, kc, cols / 128, true>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream)
    OT_WIDE(128, 2, 8, 64); OT_WIDE(128, 4, 8, 64); OT_WIDE(128, 6, 8, 64); OT_WIDE(128, 9, 8, 64); OT_WIDE(128, 11, 8, 64);
    OT_WIDE(256, 2, 4, 128); OT_WIDE(256, 4, 4, 128); OT_WIDE(256, 6, 4, 128); OT_WIDE(256, 9, 4, 128); OT_WIDE(256, 11, 4, 64);
    OT_WIDE(384, 2, 4, 64); OT_WIDE(384, 4, 4, 64); OT_WIDE(384, 6, 4, 64); OT_WIDE(384, 9, 2, 64); OT_WIDE(384, 11, 2, 64);
    OT_WIDE(512, 2, 2, 64); OT_WIDE(512, 4, 2, 64); OT_WIDE(512, 6, 2, 64); OT_WIDE(512, 9, 2, 64); OT_WIDE(512, 10, 2, 64);
    OT_WIDE(512, 11, 2, 64);
    OT_WIDE(640, 2, 2, 64); OT_WIDE(640, 4, 2, 64); OT_WIDE(640, 6, 2, 64); OT_WIDE(640, 8, 2, 64);
#undef OT_WIDE
    return hipErrorInvalidValue;
  }
  // More than 176 rows run as several M-blocks per column tile (tall_plan).  Heights above 144 rows use hidden
  // slices of 64 columns and a weight ring two steps deep to fit in LDS.
  const TallPlan plan = tall_plan(M, d, Vp, n_cu);
  if (plan.wide) {
    switch (plan.tiles) {
      case 10: return launch_wide<10, 2, 8, 64, 4>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
      case 11: return launch_wide<11, 2, 8, 64, 4>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
      default: return launch_wide<9, 2, 8, 64, 4>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    }
  }
  const int best_mt = plan.tiles;
  switch (best_mt) {
    case 4: return launch_wide<4, 4, 8, 128, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    case 6: return launch_wide<6, 4, 8, 128, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    case 10: return launch_wide<10, 2, 8, 64, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    case 12: return launch_wide<12, 2, 8, 64, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    case 14: return launch_wide<14, 2, 8, 64, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    case 16: return launch_wide<16, 2, 8, 64, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    case 18: return launch_wide<18, 2, 8, 64, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
    default: return launch_wide<9, 4, 8, 128, 2>(H, M, d, Wp, Kp, Vp, Z, V_t, ldz, zeros, fs, draft_side, n_cu, stream);
  }
}

hipError_t launch_pack_w_f32(const float* W, int d, int V_t, float* Wp, hipStream_t stream) {
  const int nkb = ceil_div(d, 16);
  const int64_t n_units = (int64_t)ceil_div(V_t, 64) * nkb * 256;
  hipLaunchKernelGGL(pack_w_f32_kernel, dim3((unsigned)((n_units + 255) / 256)), dim3(256), 0, stream, W, d, V_t,
                     reinterpret_cast<float4*>(Wp), nkb, n_units);
  return hipGetLastError();
}

hipError_t launch_lmhead_f32(const float* H, int M, int d, const float* Wp, float* Z, int V_t, int64_t ldz,
                             const FusedStats* fused, const StepArgs* draft_side, int n_cu, hipStream_t stream) {
  if (M == 0) return hipSuccess;
  FusedStats fs{};
  if (fused && fused->part) {
    if (fused->nfine != ceil_div(V_t, 64) || fused->B < 1 || fused->B > kFusedMaxB) return hipErrorInvalidValue;
    fs = *fused;
  }
  if (!fs.part) draft_side = nullptr;
  if (draft_side && !front_plan_fits(*draft_side)) return hipErrorInvalidValue;
  const F32Plan plan = f32_plan(M, d, V_t, n_cu);
  if (plan.thirds) {
    if (plan.tiles == 4) return launch_f32_thirds<4>(H, M, d, Wp, Z, V_t, ldz, fs, draft_side, plan, stream);
    if (plan.tiles == 3) return launch_f32_thirds<3>(H, M, d, Wp, Z, V_t, ldz, fs, draft_side, plan, stream);
    return launch_f32_thirds<2>(H, M, d, Wp, Z, V_t, ldz, fs, draft_side, plan, stream);
  }
  if (plan.tiles == 1) return launch_f32<1, 8, 4>(H, M, d, Wp, Z, V_t, ldz, fs, draft_side, plan, stream);
  if (plan.tiles == 3) return launch_f32<3, 4, 2>(H, M, d, Wp, Z, V_t, ldz, fs, draft_side, plan, stream);
  return launch_f32<2, 4, 2>(H, M, d, Wp, Z, V_t, ldz, fs, draft_side, plan, stream);
}

// A launch that leaves room on the chip gives every piece of a draft row a workgroup of its own, a larger one takes whole rows, or
// halves where that leaves the busiest wavefront less (48 rows by 32 wavefronts).
int lmhead_f32_draft_workers(int M, int d, int V_t, int B, int K, int n_cu) {
  const F32Plan plan = f32_plan(M, d, V_t, n_cu);
  if (plan.workgroups + B + kDraftPieces * K <= 2 * n_cu) return kDraftPieces * K;
  const int wavefronts = 4 * f32_row_front(plan, B, K);
  return plan.thirds && ceil_div(2 * K, wavefronts) < 2 * ceil_div(K, wavefronts) ? 2 * K : K;
}
// Whether the fp32 launch should leave partials and take the draft side.  That spares the statistics launch (6 us and a pass over both
// sides' logits).  It costs the multiplying workgroups their epilogue and the launch behind it the merge of a partial per row and 64
// columns (and a launch where the test gets one of its own); where wavefronts of front workgroups take whole draft rows, the launch
// lasts as long as they do: one draws 3.5 KB per us, 1.6 with more than two rows in turn, and a fifth of that while the weights stream
// (1020 rows x 65536, d = 64, seven rows of 8000 ids each, 282 us hosted, 211 separate).  A front that pushes
// multiplying workgroups into one round more costs 0.15 of a round.
// Measured at 1296 shapes (d = 64 to 1024, 1024 to 152064 columns, 2 to 1530 rows, draft rows of 1000 to 32000 ids), before the thirds
// kernel and with the front's loads asked for one after the other: the choice costs
// 0.2 % on average against the better one, 10 % at most (16 rows x 100000, d = 256, draft rows of 8000 ids, 36.0 / 32.7).  With a draft
// row priced at 3 KB per us next to any head it was 3 % and 63 %; with the thirds kernel, at 378 shapes, 0.6 % and 12 %.  us per step, hosted / separate: 5 rows x 100000 (d = 1024), draft
// rows of 32000 ids 123 / 91, of 1000 92 / 92; 16 rows x 152064 (2376 partials a row) 138 / 137, x 32000 32.3 / 36.0; 64 rows x 32000
// with draft rows of 8000 54.9 / 58.3.
bool lmhead_f32_hosts_draft_side(int M, int d, int V_t, int B, int K, int V_d, int n_cu) {
  if (B < 1 || B > kFusedMaxB || K < 1) return false;
  const double product_us = 2.0 * M * d * (double)V_t / 1.0e8, head_us = std::max(4.0 * d * (double)V_t / 6.0e6, product_us);
  const int workers = lmhead_f32_draft_workers(M, d, V_t, B, K, n_cu);
  if (workers == kDraftPieces * K) return front_pieces_end_in_time(4.0 * V_d, head_us);
  const F32Plan plan = f32_plan(M, d, V_t, n_cu);
  const int front = f32_row_front(plan, B, K);
  const double rows_each = ceil_div(workers, 4 * front) * (double)K / workers;
  const double front_us = ceil_div(B, front) * 1.0 + rows_each * (4.0 * V_d / (rows_each <= (plan.thirds ? 3 : 2) ? 3.5e3 : 1.6e3)) + 0.8 * head_us;
  const int at_once = plan.at_once, multiplying = plan.workgroups, rounds = ceil_div(multiplying, at_once);
  const double added_us = 0.0035 * ceil_div(V_t, 64) + 0.5e-6 * M * (double)V_t + 0.06 * product_us +
                          (ceil_div(multiplying + front, at_once) > rounds ? 0.15 * product_us / rounds : 0.0) +
                          (final_draw_launches(kHostsAll, ceil_div(V_t, 64), M, V_t, V_d, B, n_cu) > 1 ? 15.0 : 0.0);
  const double statistics_us = 6.0 + (4.0 * M * (double)V_t + 4.0 * K * (double)V_d) / 5.0e6;
  return std::max(head_us + added_us, front_us) < head_us + statistics_us;
}

}  // namespace otv
