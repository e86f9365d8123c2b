// Draft side of a verification step, as device functions shared by the kernels that host it: everything that needs
// the drafter's logits and ids but nothing of the target's logits.
//   * softmax statistics of the draft rows (Notation paragraph: q = softmax(zq / T_d)): one wavefront per row, or one
//     workgroup per piece of a row with the pieces merged where they are used;
//   * translation of the drafted window into the target vocabulary (Section "Cross-vocabulary N-gram Cache", Eq. 1):
//     every window (start s, length L) of the drafted ids is probed in the n-gram table by its own thread; lane s of
//     one wavefront prepares the segment that would start at s, and the window is then walked left to right as a chase
//     through start + length: the longest cache hit at s yields one target token whose q' is the product of the L
//     sub-token probabilities, otherwise the direct image of d_s, and a draft id with neither ends the proposal.
// The lookups of a sequence (drafted logits, direct images, table probes) need memory and can run early, next to the
// LM head, which leaves them in a ProbeRecord; the walk itself is a fraction of a microsecond of one wavefront and runs where
// the acceptance test does.
#pragma once

#include "device_math.h"
#include "otv_internal.h"

namespace otv {

constexpr float kLog2eF = 1.4426950408889634f;

// LDS scratch of one sequence's lookups (k <= 63 drafted positions).
struct DraftLds {
  unsigned long long hit[64];   // (length << 60) | (slot << 32) | target of the longest cache hit starting here, 0 = none
  float zq[64];                 // draft logit of the drafted id
  int32_t dm[64];               // direct image of the drafted id, or -1
  int32_t bad;                  // a drafted id was outside [0, V_d)
};

// A walked window.  Lane s of the walking wavefront holds the segment that would start at draft position s (target id or -1,
// draft tokens covered, cache slot or -1); bit s of `starts` says that the walk reached it.  The j-th set bit is mapped
// position j and is tested against row j of the sequence.  All but the segments is wavefront-uniform.
struct Window {
  int t, L, slot;
  unsigned long long starts;
  int m, end, flags;            // mapped positions; where the walk ended (k, or the draft id that could not be translated)
};
__device__ __forceinline__ unsigned long long bits_below(int i) { return (1ull << i) - 1ull; }   // i <= 63

// Probe of one key held in registers (fully unrolled so that `ids` never has to live in scratch memory).
// Returns the slot index of the entry, or -1.
__device__ __forceinline__ int cache_lookup(const CacheTable& C, const int32_t (&ids)[OT_MAX_NGRAM_LEN], int L) {
  uint32_t h = 0x9E3779B9u ^ (uint32_t)L;                  // same mixing as hash_ngram()
#pragma unroll
  for (int i = 0; i < OT_MAX_NGRAM_LEN; ++i) {
    if (i < L) {
      h ^= (uint32_t)ids[i] + 0x7F4A7C15u + (h << 6) + (h >> 2);
      h *= 0x85EBCA6Bu;
      h ^= h >> 13;
    }
  }
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  h &= C.mask;
  for (uint32_t probe = 0; probe <= C.mask; ++probe) {     // bounded: the table is never more than half full
    const int32_t* slot = C.slots + (size_t)h * C.stride;
    const int sl = slot[0];
    if (sl == 0) return -1;
    if (sl == L) {
      bool same = true;
#pragma unroll
      for (int i = 0; i < OT_MAX_NGRAM_LEN; ++i)
        if (i < L) same = same && (slot[2 + i] == ids[i]);
      if (same) return (int)h;
    }
    h = (h + 1) & C.mask;
  }
  return -1;
}

__device__ __forceinline__ void draft_lds_reset(DraftLds* L, int g) {
  if (g == 0) L->bad = 0;
  if (g < 64) { L->hit[g] = 0ull; L->dm[g] = -1; }
}

// Thread g of n: range check, drafted logit and direct image of the drafted positions; every window (s, len) of the
// drafted ids against the n-gram table, the longest hit per start wins.  draft_lds_reset and a barrier come before,
// a barrier after.
__device__ __forceinline__ void fetch_ids_and_probe(const StepArgs& a, int q0, int k, int g, int n, DraftLds* L) {
  for (int i = g; i < k; i += n) {
    const int d = a.draft_ids[q0 + i];
    if (d < 0 || d >= a.V_d) {
      L->bad = 1;
    } else {
      const int64_t at = (int64_t)(q0 + i) * a.V_d + d;
      L->zq[i] = a.dtype == OT_BF16 ? bf16_to_f32(static_cast<const uint16_t*>(a.draft_logits)[at])
                                    : static_cast<const float*>(a.draft_logits)[at];
      L->dm[i] = a.dmap[d];
    }
  }
  if (a.cache.slots != nullptr) {
    const int nL = a.cache.max_len - 1;
    for (int w = g; w < k * nL; w += n) {
      const int s = w / nL, len = 2 + w % nL;
      if (s + len <= k) {
        int32_t ids[OT_MAX_NGRAM_LEN];
        bool in_range = true;
#pragma unroll
        for (int i = 0; i < OT_MAX_NGRAM_LEN; ++i) {
          ids[i] = i < len ? a.draft_ids[q0 + s + i] : 0;
          in_range = in_range && ids[i] >= 0 && ids[i] < a.V_d;
        }
        if (in_range) {
          const int slot = cache_lookup(a.cache, ids, len);
          if (slot >= 0) {
            const unsigned int t = (unsigned int)a.cache.slots[(size_t)slot * a.cache.stride + 1];
            atomicMax(&L->hit[s], ((unsigned long long)len << 60) | ((unsigned long long)slot << 32) | t);
          }
        }
      }
    }
  }
}

// The lookups of sequence b by a workgroup of n threads (all call it): its ProbeRecord.
__device__ __forceinline__ void lookup_sequence(const StepArgs& a, int b, int tid, int n, DraftLds* L) {
  const int r0 = a.row_off[b], k = a.row_off[b + 1] - r0 - 1;
  draft_lds_reset(L, tid);
  __syncthreads();
  fetch_ids_and_probe(a, r0 - b, k, tid, n, L);
  __syncthreads();
  ProbeRecord* rec = a.probe + b;
  if (tid < 64) { rec->hit[tid] = L->hit[tid]; rec->zq[tid] = L->zq[tid]; rec->dm[tid] = L->dm[tid]; }
  if (tid == 0) rec->bad = L->bad;
}

// The same by one wavefront on its own (L: its part of LDS).  Its LDS operations are done in order; the compiler is kept from moving
// them across the hand-overs.
__device__ __forceinline__ void wave_lookup_sequence(const StepArgs& a, int b, int lane, DraftLds* L) {
  const int r0 = a.row_off[b], k = a.row_off[b + 1] - r0 - 1;
  auto hand_over = []() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), vmcnt and expcnt unconstrained
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
  };
  draft_lds_reset(L, lane);
  hand_over();
  fetch_ids_and_probe(a, r0 - b, k, lane, 64, L);
  hand_over();
  ProbeRecord* rec = a.probe + b;
  rec->hit[lane] = L->hit[lane]; rec->zq[lane] = L->zq[lane]; rec->dm[lane] = L->dm[lane];
  if (lane == 0) rec->bad = L->bad;
  hand_over();
}

// ---------------------------------------------------------------------------------------------- draft row statistics
// 16-byte vectors of a logit row, kept as loaded until they are used (a bf16 vector unpacks to 8 floats).
template <typename T> struct RowVec;
template <> struct RowVec<float> {
  static constexpr int kVec = 4;
  typedef float4 Raw;
  __device__ static Raw load(const float* p) { return *reinterpret_cast<const float4*>(p); }
  __device__ static Raw lowest() { return make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY); }
  __device__ static void unpack(const Raw& r, float* v) { v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w; }
  __device__ static float one(const float* p) { return *p; }
};
template <> struct RowVec<uint16_t> {
  static constexpr int kVec = 8;
  typedef uint4 Raw;
  __device__ static Raw load(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
  __device__ static Raw lowest() { return make_uint4(0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u, 0xFF80FF80u); }   // -inf
  __device__ static void unpack(const Raw& r, float* v) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
  __device__ static float one(const uint16_t* p) { return bf16_to_f32(*p); }
};

// Running (maximum, lowest index of it, sum of exponentials relative to it) of one lane.
struct RunStat {
  float mx = -INFINITY;
  int arg = 0x7FFFFFFF;
  double sum = 0.0;
  // raises the maximum to (bm, bi) if that is larger; the sum is rescaled to the new maximum
  __device__ inline void raise(float bm, int bi, float scale) {
    if (bm > mx) {
      sum *= (double)__builtin_amdgcn_exp2f((mx - bm) * scale);   // mx = -inf: the sum is 0 and stays 0
      mx = bm;
      arg = bi;
    }
  }
};

// One wavefront reduces one whole logit row to (maximum, its lowest index, sum of exp((x - max) * scale / log2 e)).
// Every lane requests kBatch 16-byte vectors at a time before it touches any of them: the draft side runs next to a
// kernel that saturates the memory system, where a load takes several microseconds to return, so the bytes in flight
// decide how long a row takes.  A lane keeps a running maximum and a running sum relative to it (rescaled when the
// maximum moves); the 64 lanes are merged at the end by shuffles in a fixed order.  Sums of one vector are formed in
// binary32, everything above that in binary64.  A row may start at any element (an odd vocabulary: every row at another
// alignment): the vectors begin at its first 16-byte boundary, and the few elements before and behind them are read one by
// one, by a lane each.  (Rows off the boundary read one by one throughout take a front workgroup five times as long: 200 rows
// of 50257 ids next to a head of 50257 columns 435 us per step, 170 when the statistics run as a launch of their own.)
// All lanes return the row's statistics.
// kFirst: the first batch was requested earlier (row_first_batch_load with the same x and V) and is taken from `first`.
template <typename T, int kBatch> struct RowFirstBatch { typename RowVec<T>::Raw raw[kBatch]; };

// elements of row x (V of them) before its first 16-byte boundary
template <typename T>
__device__ __forceinline__ int row_head(const T* x, int V) {
  return min((int)((16 - (reinterpret_cast<uintptr_t>(x) & 15)) & 15) / (int)sizeof(T), V);
}

template <typename T, int kBatch>
__device__ __forceinline__ void row_first_batch_load(const T* __restrict__ x, int V, int lane,
                                                     RowFirstBatch<T, kBatch>& first) {
  constexpr int kVec = RowVec<T>::kVec;
  const int head = V > 0 ? row_head(x, V) : 0;
  const int n_vec = V > 0 ? (V - head) / kVec : 0;
  const T* xv = x + head;
#pragma unroll
  for (int j = 0; j < kBatch; ++j) {
    const int at = j * 64 + lane;
    first.raw[j] = at < n_vec ? RowVec<T>::load(xv + (int64_t)at * kVec) : RowVec<T>::lowest();
  }
}

template <typename T, int kBatch, bool kFirst = false>
__device__ __forceinline__ void wave_row_stats(const T* __restrict__ x, int V, float scale, int lane, float* out_max,
                                               int* out_arg, double* out_sum,
                                               const RowFirstBatch<T, kBatch>* first = nullptr) {
  constexpr int kVec = RowVec<T>::kVec;
  typedef typename RowVec<T>::Raw Raw;
  const int head = row_head(x, V);
  const int n_vec = (V - head) / kVec;            // whole vectors read as such
  const T* xv = x + head;
  RunStat r;
  for (int base = 0; base < n_vec; base += 64 * kBatch) {
    Raw raw[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int at = base + j * 64 + lane;
      if (kFirst && base == 0) raw[j] = first->raw[j];
      else raw[j] = at < n_vec ? RowVec<T>::load(xv + (int64_t)at * kVec) : RowVec<T>::lowest();
    }
    float bm = -INFINITY;
    int bi = 0x7FFFFFFF;
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      if (base + j * 64 >= n_vec) break;        // wavefront-uniform: the remaining vectors of the batch are empty
      float v[kVec];
      RowVec<T>::unpack(raw[j], v);
#pragma unroll
      for (int e = 0; e < kVec; ++e)
        if (v[e] > bm) { bm = v[e]; bi = (base + j * 64 + lane) * kVec + e; }   // ascending index: first maximum kept
    }
    r.raise(bm, bi, scale);
    if (r.mx != -INFINITY) {
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        if (base + j * 64 >= n_vec) break;
        // the vector is unpacked again rather than kept unpacked since the first pass (8 registers instead of 4 each)
        asm volatile("" : "+v"(raw[j].x), "+v"(raw[j].y), "+v"(raw[j].z), "+v"(raw[j].w));
        float v[kVec];
        RowVec<T>::unpack(raw[j], v);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < kVec; ++e) s += __builtin_amdgcn_exp2f((v[e] - r.mx) * scale);   // masked: exp2(-inf) = 0
        r.sum += (double)s;
      }
    }
  }
  if (r.mx != -INFINITY) r.arg += head;
  if (lane < V - n_vec * kVec) {                  // fewer than two vectors' elements are left
    const int at = lane < head ? lane : lane + n_vec * kVec;
    const float v = RowVec<T>::one(x + at);
    r.raise(v, at, scale);
    if (v == r.mx) r.arg = min(r.arg, at);        // an element in front of an equal maximum
    if (r.mx != -INFINITY) r.sum += (double)__builtin_amdgcn_exp2f((v - r.mx) * scale);   // nothing but -inf so far: no (-inf) - (-inf)
  }
  float mx = r.mx;
  int arg = r.arg;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float om = __shfl_xor(mx, off);
    const int oa = __shfl_xor(arg, off);
    if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
  }
  double s = r.mx == -INFINITY ? 0.0 : r.sum * (double)__builtin_amdgcn_exp2f((r.mx - mx) * scale);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  *out_max = mx; *out_arg = arg; *out_sum = s;
}

// ---------------------------------------------------------------------------------------------- the walk
// One wavefront walks the window of k drafted ids (Eq. 1) from what lane s looked up at draft position s: the longest cache hit
// there and the direct image.  Where no window hits the cache that is a count of leading ones, otherwise a chase through
// start + length with wavefront-uniform lane reads, a few cycles per token.
__device__ __forceinline__ Window walk_window(int k, int lane, unsigned long long hit, int dm) {
  Window w;
  const bool found = lane < k && hit != 0ull;
  w.t = lane < k ? (found ? (int)(hit & 0xFFFFFFFFull) : dm) : -1;
  w.L = found ? (int)(hit >> 60) : 1;
  w.slot = found ? (int)((hit >> 32) & 0x0FFFFFFFull) : -1;
  w.flags = 0;
  const unsigned long long can = __ballot(w.t >= 0);        // a hit or a direct image; not set from k on
  if (__ballot(found) == 0ull) {
    w.m = w.end = (int)__builtin_ctzll(~can);
    w.starts = bits_below(w.m);
  } else {
    w.m = 0; w.end = 0; w.starts = 0ull;
    while (w.end < k && ((can >> w.end) & 1ull)) {
      w.starts |= 1ull << w.end;
      w.end += __builtin_amdgcn_readlane(w.L, w.end);
      ++w.m;
    }
  }
  if (w.end < k) w.flags |= OT_FLAG_UNMAPPABLE;
  return w;
}

// q'(t) of the segment that starts at this lane from the lanes' q(d): the product over its draft tokens (Eq. 1).  Below about 1e-308
// it is 0, as the exponential of the summed logarithms would be (eight factors of 1e-45 are enough at a low draft temperature): a
// token with p > 0 is accepted then.
__device__ __forceinline__ double segment_q(double q, const Window& w) {
  double qp = q;
  if (__ballot(w.L > 1) != 0ull) {
    for (int l = 1; __ballot(w.L > l) != 0ull; ++l) {
      const double next = __shfl_down(q, l);
      if (l < w.L) qp *= next;
    }
  }
  return qp;
}

// The translation's outputs (n_mapped, hits_proposed, flags; mapped_ids, span_start, span_len, q_tok of the sequence's rows) and
// the use statistics of the cache entries, by one wavefront of the step per sequence.  pos: mapped position of a segment that
// the walk reached.  with_flags: nothing is drawn (otherwise the draw, which may add a flag, writes them).
__device__ __forceinline__ void write_translation(const StepArgs& a, int b, int r0, int k, int lane, const Window& w, bool reached,
                                                  int pos, double qp, bool with_flags) {
  const bool is_hit = reached && w.L > 1;
  if (is_hit) {
    // use statistics of the entry (Appendix, cache eviction): one more use, last used now
    atomicAdd(&a.cache.uses[w.slot], 1u);
    a.cache.last_used[w.slot] = a.cache.clock;
    const uint32_t at = atomicAdd(a.cache.log_count, 1u);        // and the host hears of it through the log
    if (at < (uint32_t)kCacheLogCap) a.cache.log[at] = make_uint2((uint32_t)w.slot + 1u, a.cache.clock);
  }
  const int hits = __popcll(__ballot(is_hit));
  if (lane == 0) {
    a.out.n_mapped[b] = w.m;
    a.out.hits_proposed[b] = hits;
    if (with_flags) a.out.flags[b] = w.flags;
  }
  if (reached) {
    a.out.mapped_ids[r0 + pos] = w.t; a.out.span_start[r0 + pos] = lane; a.out.span_len[r0 + pos] = w.L;
    a.out.q_tok[r0 + pos] = (float)qp;
  }
  if (lane >= w.m && lane <= k) {
    a.out.mapped_ids[r0 + lane] = -1; a.out.span_start[r0 + lane] = -1; a.out.span_len[r0 + lane] = 0;
    a.out.q_tok[r0 + lane] = 0.f;
  }
}

// Softmax statistics of elements [e0, e0 + n) of draft row q by one workgroup of kWaves wavefronts (all threads call it;
// it contains workgroup barriers): every wavefront takes a contiguous slice, the slices are merged through LDS in
// ascending order (of equal maxima the lowest index is kept, the sums are added in one fixed order), thread 0 writes the
// record.  s_mx / s_arg / s_S: kWaves LDS words each.
constexpr int kPieceBatch = 8;
// the slice of elements [e0, e0 + n) of draft row q that wavefront `wave` of kWaves takes: whole 16-byte vectors
template <typename TD, int kWaves>
__device__ __forceinline__ const TD* piece_wave_slice(const StepArgs& a, int q, int e0, int n, int wave, int* lo, int* n_own) {
  constexpr int kVec = RowVec<TD>::kVec;
  const int slice = ((n + kWaves - 1) / kWaves + kVec - 1) / kVec * kVec;
  *lo = wave * slice;
  *n_own = min(slice, n - *lo);
  return static_cast<const TD*>(a.draft_logits) + (int64_t)q * a.V_d + e0 + *lo;
}

// requests the first batch of this wavefront's slice, for a later workgroup_draft_piece<.., true> of the same piece
template <typename TD, int kWaves, int kBatch = kPieceBatch>
__device__ __forceinline__ void workgroup_draft_piece_request(const StepArgs& a, int q, int e0, int n, int tid,
                                                              RowFirstBatch<TD, kBatch>& first) {
  int lo, n_own;
  const TD* x = piece_wave_slice<TD, kWaves>(a, q, e0, n, tid >> 6, &lo, &n_own);
  row_first_batch_load<TD, kBatch>(x, n_own, tid & 63, first);
}

template <typename TD, int kWaves, bool kFirst = false, int kBatch = kPieceBatch>
__device__ __forceinline__ void workgroup_draft_piece(const StepArgs& a, int q, int e0, int n, float Td, int tid,
                                                      float* s_mx, int32_t* s_arg, double* s_S, DraftPiece* out,
                                                      const RowFirstBatch<TD, kBatch>* first = nullptr) {
  const int wave = tid >> 6, lane = tid & 63;
  int lo, n_own;
  const TD* x = piece_wave_slice<TD, kWaves>(a, q, e0, n, wave, &lo, &n_own);
  const float scale = Td > 0.f ? kLog2eF / Td : kLog2eF;
  float mx = -INFINITY;
  int arg = 0x7FFFFFFF;
  double S = 0.0;
  if (n_own > 0) {
    wave_row_stats<TD, kBatch, kFirst>(x, n_own, scale, lane, &mx, &arg, &S, first);
    arg += e0 + lo;
  }
  // The two barriers order LDS accesses only (all LDS operations of this wavefront done, then meet): the fence of
  // __syncthreads() would also wait for the record's store to be acknowledged, microseconds next to a saturating stream.
  auto lds_barrier = []() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0), vmcnt and expcnt unconstrained
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  if (lane == 0) { s_mx[wave] = mx; s_arg[wave] = arg; s_S[wave] = S; }
  lds_barrier();
  if (tid == 0) {
    float bm = -INFINITY;
    int ba = 0x7FFFFFFF;
    for (int w = 0; w < kWaves; ++w)
      if (s_mx[w] > bm) { bm = s_mx[w]; ba = s_arg[w]; }     // ascending slices: a later equal maximum does not replace
    double total = 0.0;
    for (int w = 0; w < kWaves; ++w)
      if (s_mx[w] != -INFINITY) total += s_S[w] * (double)__builtin_amdgcn_exp2f((s_mx[w] - bm) * scale);
    DraftPiece r; r.mx = bm; r.arg = ba; r.sum = total;
    *out = r;
  }
  lds_barrier();
}

// Draft-side job `job` of a launch with a workgroup for each of them in front of those that multiply: the lookups of sequence
// `job`, then one piece of a draft row each (a.plan with as many workers as pieces).  lds: kFrontLdsBytes.
constexpr size_t kFrontLdsBytes = sizeof(DraftLds) > 512 ? sizeof(DraftLds) : 512;
template <typename TD, int kWaves>
__device__ __forceinline__ void front_draft_side(const StepArgs& a, int job, int tid, void* lds) {
  if (job < a.B) {
    lookup_sequence(a, job, tid, kWaves * 64, static_cast<DraftLds*>(lds));
    return;
  }
  if (job - a.B >= a.plan.jobs(a.K)) return;            // padding
  int q, i, e0, n;
  a.plan.locate(job - a.B, &q, &i);
  PiecePlan::span(a.V_d, a.plan.pieces(q), i, &e0, &n);
  constexpr int kBatch = 4;                             // as many as leave the multiplying workgroups' registers alone
  RowFirstBatch<TD, kBatch> first;
  workgroup_draft_piece_request<TD, kWaves, kBatch>(a, q, e0, n, tid, first);
  const float* temps = a.draft_temperature ? a.draft_temperature : a.temperature;
  const float Td = temps[find_sequence(a.row_off, a.B, q, 1, tid & 63)];
  static_assert(kWaves * (sizeof(double) + 2 * sizeof(float)) <= kFrontLdsBytes, "the slices' statistics fit");
  double* s_S = static_cast<double*>(lds);
  float* s_mx = reinterpret_cast<float*>(s_S + kWaves);
  workgroup_draft_piece<TD, kWaves, true, kBatch>(a, q, e0, n, Td, tid, s_mx, reinterpret_cast<int32_t*>(s_mx + kWaves), s_S,
                                          a.dpiece + (int64_t)q * kDraftPieces + i, &first);
}

// The same by few workgroups: front workgroup j of n takes the lookups of sequences, then every wavefront of it whole draft rows, or
// halves (a.plan with one or two pieces per row).  Next to the other workgroups' streams a dependent load takes microseconds, so
// that the chains of loads decide how long this lasts.
// kAhead: a piece's first batch is asked for a piece ahead (the first one in front of the lookups), and the sequences' row offsets and
// temperatures are held across the lanes (at most kFusedMaxB of them).  Takes 70 registers; a kernel whose multiplying workgroups
// would lose a wavefront per SIMD to them goes without (fp32 head at d < 384: 64 rows x 32000 columns, d = 256 / 376, 26.1 -> 29.0 / 32.7
// -> 37.5 us per step with kAhead).
template <typename TD, int kWaves, bool kAhead, int kBatch = kPieceBatch>
__device__ __forceinline__ void front_draft_rows(const StepArgs& a, int j, int n, int tid, void* lds) {
  const int lane = tid & 63, wave = uniform(tid >> 6), pieces = a.plan.base, jobs = a.K * pieces;
  const float* temps = a.draft_temperature ? a.draft_temperature : a.temperature;
  constexpr int kSeqRegs = (kFusedMaxB + 64) / 64;
  int seq_before[kSeqRegs];
  float seq_temp[kSeqRegs];
  if constexpr (kAhead) {
#pragma unroll
    for (int i = 0; i < kSeqRegs; ++i) {
      const int b = min(64 * i + lane, a.B - 1);
      seq_before[i] = a.row_off[b] - b;
      seq_temp[i] = temps[b];
    }
  }
  auto temperature_of = [&](int q) {
    if constexpr (!kAhead) return temps[find_sequence(a.row_off, a.B, q, 1, lane)];
    int owner = -1;
    float Td = 1.f;
#pragma unroll
    for (int i = 0; i < kSeqRegs; ++i) owner += __popcll(__ballot(64 * i + lane < a.B && seq_before[i] <= q));
#pragma unroll
    for (int i = 0; i < kSeqRegs; ++i) {
      const float t = __shfl(seq_temp[i], owner & 63);
      if ((owner >> 6) == i) Td = t;
    }
    return Td;
  };
  int e0, len;
  auto piece = [&](int job) {
    PiecePlan::span(a.V_d, pieces, job % pieces, &e0, &len);
    return static_cast<const TD*>(a.draft_logits) + (int64_t)(job / pieces) * a.V_d + e0;
  };
  int job = n * kWaves - 1 - (j * kWaves + wave);       // from the last wavefront on: the first ones have the lookups
  RowFirstBatch<TD, kBatch> first, next;
  if constexpr (kAhead) {
    const TD* x = piece(min(job, jobs - 1));
    row_first_batch_load<TD, kBatch>(x, len, lane, next);
  }
  DraftLds* L = static_cast<DraftLds*>(lds);
  if (a.B <= n) {
    if (j < a.B) lookup_sequence(a, j, tid, kWaves * 64, L);
  } else {                                              // several sequences each: side by side, a wavefront on each
    for (int b = j * kWaves + wave; b < a.B; b += n * kWaves) wave_lookup_sequence(a, b, lane, L + wave);
  }
  for (; job < jobs; job += n * kWaves) {
    if constexpr (kAhead) {                             // past the end: the last piece again, looked at by nobody
      first = next;
      const TD* x_next = piece(min(job + n * kWaves, jobs - 1));
      row_first_batch_load<TD, kBatch>(x_next, len, lane, next);
    }
    const int q = job / pieces;
    const float Td = temperature_of(q);
    const TD* x = piece(job);
    DraftPiece r; r.mx = -INFINITY; r.arg = 0x7FFFFFFF; r.sum = 0.0;
    if (len > 0) {
      wave_row_stats<TD, kBatch, kAhead>(x, len, Td > 0.f ? kLog2eF / Td : kLog2eF, lane, &r.mx, &r.arg, &r.sum, &first);
      if (r.mx != -INFINITY) r.arg += e0;
    }
    if (lane == 0) a.dpiece[(int64_t)q * kDraftPieces + job % pieces] = r;
  }
}

// Softmax partial of 64 columns of a target row, held by a row of 16 consecutive lanes, four columns from n on each: in all of
// these lanes.  sc: exponent scale of the row.  Four exponentials are added in binary32, the rest in binary64.
__device__ __forceinline__ Partial partial_of_64(const float* z, int n, int V_t, float sc) {
  float v[4], best = -INFINITY;
  int arg = 0x7FFFFFFF;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = n + e < V_t ? z[e] : -INFINITY;
    if (v[e] > best) { best = v[e]; arg = n + e; }         // ascending columns: the first maximum is kept
  }
  Partial p;
  p.mx = row16_max(best);
  p.arg = row16_min(best == p.mx ? arg : 0x7FFFFFFF);
  float s = 0.f;
  if (p.mx != -INFINITY) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s += __builtin_amdgcn_exp2f((v[e] - p.mx) * sc);   // masked: exp2(-inf) = 0
  }
  p.sum = row16_sum((double)s);
  return p;
}

}  // namespace otv
