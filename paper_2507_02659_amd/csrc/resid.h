// Final token of every sequence (Algorithm 1: correction token from the residual, or free token from p), as device
// functions for the kernels that host the draw.
//
// At the first rejected row the token is drawn from norm(max(0, p - q')) (Notation paragraph), with q' extended over
// the whole target vocabulary by Eq. 2: q'(v) = q_s(tmap[v]) through the inverse direct map (0 where v has no
// pre-image), except that the n-gram matched at this position gets the product pi of its sub-token probabilities
// and the direct image of its first sub-token gets q_s(d_1) - pi.  When everything was accepted the draw is from p.
//
// Only the ONE row per sequence where the draw happens is touched.  A workgroup of 16 wavefronts takes a run of
// consecutive tiles of kResidTile target ids of one sequence (draw_group_tiles), eight at a time, two wavefronts per tile:
//   every workgroup  forms the masses of max(0, p - q') of its tiles in binary64, publishes them and counts itself in;
//   the workgroup that arrives last for its sequence  walks the tile masses in ascending order with a wavefront scan
//                    to the tile that holds u * total, re-forms that tile with each thread owning 4 consecutive ids,
//                    scans the running sum in ascending id order and emits the first id whose running sum exceeds the
//                    target (inverse CDF).  Which workgroup that is varies from run to run; what it computes does not.
//                    When the residual is empty (reachable only through underflow) it walks the masses of p, the
//                    fallback distribution, instead: every workgroup leaves that of a tile without residual mass in its
//                    place, negative (nothing to do in the common case; formed by the last workgroup alone, 32 such
//                    sequences of 128256 ids took 50 us, 29 now).
// Nothing waits: a workgroup that is not last simply ends.  A workgroup that has all tiles of its sequence (a small
// vocabulary, or many sequences) keeps the masses in LDS and counts nothing: three round trips to memory less.
// What bounds a small batch is the chain of instructions and round trips in one workgroup (the launch that tests and draws, in
// the kernel trace: 16 x 128256 ids 17.9 us, 26.3 before its gathers were freed and its scans and reductions moved from the LDS
// permute network to data-parallel moves; one sequence of 32000 ids 12.5 against 16.2 us).
#pragma once

#include "device_math.h"
#include "otv_internal.h"

namespace otv {

constexpr int kDrawWaves = 16;                       // wavefronts per workgroup
constexpr int kDrawThreads = kDrawWaves * 64;
constexpr int kTurnTiles = kDrawWaves / 2;           // tiles a workgroup sums at a time: two wavefronts share one
constexpr int kPerLane = kResidTile / 128;           // ids per lane while two wavefronts sum one tile
constexpr int kPickThreads = 256;
constexpr int kPer = kResidTile / kPickThreads;      // consecutive ids per thread while the chosen tile is scanned
static_assert(kPer == 4, "the fixed summation trees below are written for 4 ids per thread");

// p(v) and q'(v) of Eq. 2 at the final row of one sequence.
struct FinalRow {
  const float* z;
  float mx, sc_hi, sc_lo;        // row maximum; log2(e) / T split into two positive floats
  double invS;
  const void* zq;
  int lds_at;                    // where the draft row's copy starts in the dynamic LDS, in bytes (-1: there is none)
  int dtype;
  float mxq, scq_hi, scq_lo;     // the same for the draft row
  double invSq;
  int argq;
  bool greedy_draft;
  bool residual;
  int t_ng, t_pre;
  double pi, q_pre;

  // exp((x - max) / T) / S for x <= max.  The exponent goes through the hardware 2^x in binary32: the difference to the
  // row maximum is formed in binary32 (its rounding is random, not a bias), the scale is applied as a two-float
  // product so that its own rounding does not tilt the whole row, and the normaliser is applied in binary64.  Relative
  // error about 2e-7 per value, unbiased; the running sums over the vocabulary are binary64.
  __device__ static inline double softmax_term(float x, float mx, float sc_hi, float sc_lo, double invS) {
    const float d = x - mx;
    return (double)__builtin_amdgcn_exp2f(fmaf(d, sc_hi, d * sc_lo)) * invS;
  }
  __device__ inline double p_of(float zv) const { return softmax_term(zv, mx, sc_hi, sc_lo, invS); }
  // q'(v) given the draft id dv = tmap[v] (or -1) and, when dv >= 0 and the draft is not greedy, its logit
  __device__ inline double qprime(int v, int dv, float xq) const {
    double q = 0.0;
    if (dv >= 0) q = greedy_draft ? ((dv == argq) ? 1.0 : 0.0) : softmax_term(xq, mxq, scq_hi, scq_lo, invSq);
    if (v == t_pre) q = q_pre;
    if (v == t_ng) q = pi;       // the n-gram case of Eq. 2 wins when both name the same id
    return q;
  }
};

// A scale x > 0 as two positive floats, its first 21 bits and the rest, so that -inf times either is -inf: split at the nearest
// float, the lower one is negative for about half of all temperatures (0.7, 0.9, ..), and a masked logit gave NaN.
__device__ inline float scale_hi(double x) { return (float)__hiloint2double(__double2hiint(x), 0); }
__device__ inline float scale_lo(double x, float hi) { return fmaxf((float)(x - (double)hi), 1e-30f); }

// The record is the same for every lane: all of it goes to scalar registers.
__device__ inline FinalRow make_final_row(const StepArgs& a, const FinalInfo& f) {
  FinalRow R;
  R.z = a.Z + (int64_t)uniform(f.row) * a.ldz;
  const double sc = f.invT * 1.4426950408889634, scq = f.invTd * 1.4426950408889634;
  const float sc_hi = scale_hi(sc), scq_hi = scale_hi(scq);
  R.mx = uniform((float)f.mx); R.sc_hi = uniform(sc_hi); R.sc_lo = uniform(scale_lo(sc, sc_hi)); R.invS = uniform(f.invS);
  R.residual = uniform(f.mode) == 3;
  R.lds_at = -1;
  R.dtype = a.dtype;
  R.t_ng = uniform(f.t_ng); R.t_pre = uniform(f.t_pre); R.pi = uniform(f.pi); R.q_pre = uniform(f.q_pre);
  R.zq = static_cast<const char*>(a.draft_logits) + (size_t)uniform(f.drow) * a.V_d * (a.dtype == OT_BF16 ? 2 : 4);
  R.mxq = uniform((float)f.mxq); R.scq_hi = uniform(scq_hi); R.scq_lo = uniform(scale_lo(scq, scq_hi));
  R.invSq = uniform(f.invSq); R.argq = uniform(f.argq);
  R.greedy_draft = uniform(f.greedy_draft) != 0;
  return R;
}

// Inverse direct map of N ids v = first + e * stride (independent of which row is drawn from: issued early).  Ids past
// the vocabulary read the last entry and are masked afterwards: no branch around the loads.
template <int N>
__device__ inline void load_tmap(const int32_t* __restrict__ tmap, int V_t, int first, int stride, int* dv) {
#pragma unroll
  for (int e = 0; e < N; ++e) dv[e] = tmap[min(first + e * stride, V_t - 1)];
}

// Stand-in logit of an id that does not exist or has no pre-image: finite, so that the two-float scaling below never
// meets inf * 0, and so far below any maximum that its exponential is exactly 0.
constexpr float kFarBelow = -1e30f;

// The dynamic LDS of the draw kernels: the tiles' masses, then (where a workgroup takes several turns) the draft row.
typedef __attribute__((address_space(3))) char* lds_chars;
extern __shared__ __attribute__((aligned(16))) double s_draw_dynamic[];
__device__ inline lds_chars draw_lds() { return (lds_chars)(void __attribute__((address_space(3)))*)s_draw_dynamic; }

// Logits of draft ids dv (negative: the row's first) as stored, from the row's copy in the dynamic LDS where there is one.
template <int N>
__device__ inline void load_draft_logits(const void* zq, int dtype, int lds_at, const int* dv, uint32_t* xq) {
  if (lds_at >= 0) {
    const lds_chars s_row = draw_lds() + lds_at;
    if (dtype == OT_BF16) {
#pragma unroll
      for (int e = 0; e < N; ++e) xq[e] = *(const __attribute__((address_space(3))) uint16_t*)(s_row + 2 * max(dv[e], 0));
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) xq[e] = *(const __attribute__((address_space(3))) uint32_t*)(s_row + 4 * max(dv[e], 0));
    }
  } else if (dtype == OT_BF16) {
#pragma unroll
    for (int e = 0; e < N; ++e) xq[e] = static_cast<const uint16_t*>(zq)[max(dv[e], 0)];
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) xq[e] = static_cast<const uint32_t*>(zq)[max(dv[e], 0)];
  }
}

// What tile_values needs from memory for N ids v = first + e * stride, as loaded: the row's logits and, where the draw is
// from a residual of a sampling drafter, the logits of the ids' pre-images.
template <int N> struct TileRaw { float z[N]; uint32_t xq[N]; };

// All 2 N loads leave before anything waits: no lane is masked off (an id without a pre-image reads the row's first
// logit) and nothing is converted between two loads.  With the conversion inside a conditional block per id every
// gather was waited for by itself, eight round trips of about 1 us in a row.
template <int N>
__device__ inline void load_tile(const FinalRow& R, int V_t, int first, int stride, const int* dv, TileRaw<N>& raw) {
#pragma unroll
  for (int e = 0; e < N; ++e) raw.z[e] = R.z[min(first + e * stride, V_t - 1)];
  if (!R.residual || R.greedy_draft) {                   // wavefront-uniform
#pragma unroll
    for (int e = 0; e < N; ++e) raw.xq[e] = 0u;
  } else {
    load_draft_logits<N>(R.zq, R.dtype, R.lds_at, dv, raw.xq);
  }
}

// Mass r(v) of those ids, the N of them across the wavefront inside [lo, hi): max(0, p - q'), or p where the draw is from
// p.  The common case (all ids exist, a sampling drafter, no id of Eq. 2's two overrides among them: tested once per
// wavefront) costs an id about twenty instructions; this is what bounds a turn, not the memory.
template <int N>
__device__ inline void tile_values(const FinalRow& R, int V_t, int first, int stride, int lo, int hi, const int* dv,
                                   const TileRaw<N>& raw, double* r) {
  const bool all_exist = hi <= V_t;
#pragma unroll
  for (int e = 0; e < N; ++e)                                     // beyond V_t: 2^(-huge) = 0
    r[e] = R.p_of(all_exist || first + e * stride < V_t ? raw.z[e] : kFarBelow);
  if (!R.residual) return;
  const uint32_t shift = R.dtype == OT_BF16 ? 16u : 0u;
  float xq[N];
#pragma unroll
  for (int e = 0; e < N; ++e) xq[e] = dv[e] >= 0 ? __uint_as_float(raw.xq[e] << shift) : kFarBelow;
  const bool special = R.greedy_draft || (R.t_pre >= lo && R.t_pre < hi) || (R.t_ng >= lo && R.t_ng < hi);
  if (!special) {
#pragma unroll
    for (int e = 0; e < N; ++e)                                   // no pre-image: 2^(-huge) = 0; beyond V_t: max(0, 0 - q) = 0
      r[e] = fmax(0.0, r[e] - FinalRow::softmax_term(xq[e], R.mxq, R.scq_hi, R.scq_lo, R.invSq));
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const int v = first + e * stride;
      r[e] = v < V_t ? fmax(0.0, r[e] - R.qprime(v, dv[e], xq[e])) : 0.0;
    }
  }
}

// first id a lane sums among the eight tiles that start at `tile0`
__device__ inline int draw_first_id(int tile0, int wave, int lane) {
  return (tile0 + (wave >> 1)) * kResidTile + (wave & 1) * (kResidTile / 2) + lane;
}

// Copies the draft row to byte `at` of the dynamic LDS (all threads call it, a barrier follows): whole 16-byte chunks where
// the row covers them, element by element at its ends, each byte at its own offset within a chunk.  Returns where the row
// starts there.
template <int kThreads>
__device__ inline int stage_draft_row(const void* zq, int dtype, int V_d, int tid, int at) {
  const int esz = dtype == OT_BF16 ? 2 : 4;
  const char* row = static_cast<const char*>(zq);
  const int head = (int)(reinterpret_cast<uintptr_t>(row) & 15), bytes = V_d * esz;
  const int chunks = (head + bytes + 15) / 16;
  const int whole0 = head ? 1 : 0, whole1 = (head + bytes) / 16;     // chunks [whole0, whole1) lie inside the row
  const lds_chars s_row = draw_lds() + at;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  constexpr int kAtOnce = 4;
  for (int c0 = tid; c0 < chunks; c0 += kAtOnce * kThreads) {
    u32x4 x[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {                    // any other chunk number loads the nearest of those
      const int c = min(max(c0 + j * kThreads, whole0), whole1 - 1);
      x[j] = whole0 < whole1 ? *reinterpret_cast<const u32x4*>(row + (c * 16 - head)) : u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int c = c0 + j * kThreads, from = c * 16 - head;
      if (c >= whole0 && c < whole1) {
        *(__attribute__((address_space(3))) u32x4*)(s_row + c * 16) = x[j];
      } else if (c < chunks) {
        for (int o = max(from, 0); o < min(from + 16, bytes); o += esz) {
          if (esz == 2) *(__attribute__((address_space(3))) uint16_t*)(s_row + head + o) = *reinterpret_cast<const uint16_t*>(row + o);
          else *(__attribute__((address_space(3))) uint32_t*)(s_row + head + o) = *reinterpret_cast<const uint32_t*>(row + o);
        }
      }
    }
  }
  return at + head;
}

struct DrawLds {
  double w[kPickThreads / 64];
  double base, target;
  int first[kPickThreads / 64], lastnz[kPickThreads / 64];
  int pick, fallback, last;
};

constexpr size_t kDrawLdsBytes = 150 << 10;    // dynamic LDS of a workgroup with a copy of the draft row at most (160 KB a compute unit)

// Mass of the 512 ids from `lo` on (this lane: first + e * 64), in every lane: of the residual or, where that is zero, minus
// that of p.
__device__ inline double half_tile_mass(const FinalRow& R, int V_t, int first, int lo, const int* dv, const TileRaw<kPerLane>& raw) {
  double r[kPerLane];
  auto sum = [&](const FinalRow& S) {
    tile_values<kPerLane>(S, V_t, first, 64, lo, lo + kResidTile / 2, dv, raw, r);
    double x = 0.0;
#pragma unroll
    for (int e = 0; e < kPerLane; e += 4) x += (r[e] + r[e + 1]) + (r[e + 2] + r[e + 3]);
    return wave_sum(x);
  };
  const double mass = sum(R);
  if (!R.residual || !(mass == 0.0)) return mass;
  FinalRow P = R;
  P.residual = false;
  return -sum(P);
}
// The same of a tile from its halves.
__device__ inline double tile_mass(double a, double b) { return a <= 0.0 && b <= 0.0 ? a + b : fmax(a, 0.0) + fmax(b, 0.0); }

// Workgroup `grp` of sequence b takes tiles [grp * group_tiles, (grp + 1) * group_tiles), group_tiles a multiple of
// kTurnTiles (all kDrawThreads threads call this; f is the sequence's outcome record with f.mode != 0; dv holds tmap of
// the ids draw_first_id(grp * group_tiles, wave, lane) + e * 64, e < kPerLane).  The dynamic LDS holds
// max(ntiles, 2 * group_tiles) doubles (twice ntiles where one workgroup has all tiles) and, if row_at > 0, from double row_at on room for the draft row and 32 bytes.
__device__ inline void draw_final_token(const StepArgs& a, int b, int grp, int group_tiles, const FinalInfo& f, int* dv,
                                        DrawLds* L, int row_at) {
  double* s_tiles = s_draw_dynamic;
  const int tid = threadIdx.x, wave = uniform((int)(threadIdx.x >> 6)), lane = tid & 63;
  FinalRow R = make_final_row(a, f);
  const int tile0 = grp * group_tiles, tile1 = min(tile0 + group_tiles, a.ntiles);
  if (row_at > 0 && R.residual && !R.greedy_draft) {     // workgroup-uniform
    R.lds_at = stage_draft_row<kDrawThreads>(R.zq, R.dtype, a.V_d, tid, 8 * row_at);
    __syncthreads();
  }

  // ---- masses of this workgroup's tiles: wavefronts 2i and 2i+1 take the two halves of a tile (coalesced: consecutive
  // lanes on consecutive ids) and leave them in LDS; after the last turn one thread per tile adds the halves and publishes
  for (int t0 = tile0; t0 < tile1; t0 += kTurnTiles) {
    const int tile = t0 + (wave >> 1), first = draw_first_id(t0, wave, lane);
    if (tile >= tile1) break;
    TileRaw<kPerLane> raw;
    load_tile<kPerLane>(R, a.V_t, first, 64, dv, raw);
    int dv_next[kPerLane] = {};                          // asked for behind what this turn waits for
    if (t0 + kTurnTiles < tile1) load_tmap<kPerLane>(a.tmap, a.V_t, first + kTurnTiles * kResidTile, 64, dv_next);
    const double mass = half_tile_mass(R, a.V_t, first, draw_first_id(t0, wave, 0), dv, raw);
    if (lane == 0) s_tiles[2 * (tile - tile0) + (wave & 1)] = mass;
#pragma unroll
    for (int e = 0; e < kPerLane; ++e) dv[e] = dv_next[e];
  }
  __syncthreads();
  if (gridDim.x == 1) {                                  // all tiles are this workgroup's (at most kDrawThreads): they stay in LDS
    const double mass = tid < a.ntiles ? tile_mass(s_tiles[2 * tid], s_tiles[2 * tid + 1]) : 0.0;
    __syncthreads();
    if (tid < a.ntiles) { s_tiles[tid] = fmax(mass, 0.0); s_tiles[a.ntiles + tid] = mass; }
  } else {
    for (int i = tid; i < tile1 - tile0; i += kDrawThreads)
      publish(&a.tile_r[(int64_t)b * a.ntiles + tile0 + i], tile_mass(s_tiles[2 * i], s_tiles[2 * i + 1]));
    stores_done();                                        // before this workgroup is counted
    __syncthreads();
    if (tid == 0) L->last = arrive(&a.resid_count[b], gridDim.x);
    __syncthreads();
    if (!L->last) return;
    for (int t = tid; t < a.ntiles; t += kDrawThreads) s_tiles[t] = fmax(observe(&a.tile_r[(int64_t)b * a.ntiles + t]), 0.0);
  }
  __syncthreads();

  // ---- the last workgroup of the sequence: inverse CDF over the tile masses, then inside the tile that holds the draw
  // Wavefront 0: running mass over the tiles in ascending order, in place (a wavefront scan of 64 tiles at a time plus a
  // carry), and the tile where it crosses u * total.  The total and the crossing both come from these same sums.
  auto pick_tile = [&](bool may_fall_back) {
    double* m = s_tiles;
    double carry = 0.0;
    for (int t0 = 0; t0 < a.ntiles; t0 += 64) {
      const int t = t0 + lane;
      const double incl = wave_scan(t < a.ntiles ? m[t] : 0.0) + carry;
      if (t < a.ntiles) m[t] = incl;
      carry = __shfl(incl, 63);
    }
    const double total = carry;
    const int fallback = may_fall_back && !(total > 0.0);    // residual of zero mass: draw from p
    const double target = f.u2 * total;
    int pick = -1;
    for (int t0 = 0; t0 < a.ntiles && pick < 0; t0 += 64) {
      const int t = t0 + lane;
      const unsigned long long hit = __ballot(t < a.ntiles && m[t] > target);
      if (hit) pick = t0 + (int)__ffsll((long long)hit) - 1;
    }
    if (pick < 0) {                          // rounding pushed the target past the end: take the last tile that adds mass
      pick = 0;
      for (int t = 1; t < a.ntiles; ++t) if (m[t] > m[t - 1]) pick = t;
    }
    const double base = pick > 0 ? m[pick - 1] : 0.0;
    if (lane == 0) {
      // The word is not read back: the leading workgroup stored it in this launch, on an XCD with its own L2.  That store was
      // written through before the workgroup was counted in, so this one comes after it.
      if (fallback) publish(&a.out.flags[b], f.flags | OT_FLAG_RESID_ZERO);
      L->pick = pick; L->base = base; L->target = target; L->fallback = fallback;
    }
  };
  if (wave == 0) pick_tile(true);
  __syncthreads();
  if (L->fallback) {                         // workgroup-uniform
    R.residual = false;
    for (int t = tid; t < a.ntiles; t += kDrawThreads)
      s_tiles[t] = fabs(gridDim.x == 1 ? s_tiles[a.ntiles + t] : observe(&a.tile_r[(int64_t)b * a.ntiles + t]));
    __syncthreads();
    if (wave == 0) pick_tile(false);
    __syncthreads();
  }
  const double target = L->target;
  const bool picker = wave < kPickThreads / 64;
  const int pick = uniform(L->pick);
  const int v0 = pick * kResidTile + tid * kPer;         // a picking thread owns kPer consecutive ids: ascending running sum
  double r[kPer] = {0.0, 0.0, 0.0, 0.0};
  double excl = 0.0;
  if (picker) {
    int dvp[kPer];
    TileRaw<kPer> raw;
    load_tmap<kPer>(a.tmap, a.V_t, v0, 1, dvp);
    load_tile<kPer>(R, a.V_t, v0, 1, dvp, raw);
    tile_values<kPer>(R, a.V_t, v0, 1, pick * kResidTile, (pick + 1) * kResidTile, dvp, raw, r);
    const double incl = wave_scan(((r[0] + r[1]) + r[2]) + r[3]);
    excl = __shfl_up(incl, 1);
    if (lane == 0) excl = 0.0;
    if (lane == 63) L->w[wave] = incl;
  }
  __syncthreads();
  if (picker) {
    double before = L->base;
    for (int w = 0; w < wave; ++w) before += L->w[w];
    double c = before + excl;
    int first = 0x7FFFFFFF, last = -1;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      c += r[e];
      if (r[e] > 0.0) {
        last = v0 + e;
        if (first == 0x7FFFFFFF && c > target) first = v0 + e;
      }
    }
    // ids ascend with the lanes: the lowest lane that crossed, the highest that holds mass.  (By ballots: LDS atomics of a
    // whole wavefront on one word are unrolled lane by lane, which took 3 to 4 us here.)
    const unsigned long long crossed = __ballot(first != 0x7FFFFFFF), mass = __ballot(last >= 0);
    const int w_first = crossed ? __builtin_amdgcn_readlane(first, (int)__ffsll((long long)crossed) - 1) : -1;
    const int w_last = mass ? __builtin_amdgcn_readlane(last, 63 - (int)__clzll((long long)mass)) : -1;
    if (lane == 0) { L->first[wave] = w_first; L->lastnz[wave] = w_last; }
  }
  __syncthreads();
  if (tid == 0) {
    int token = -1;
    for (int w = 0; w < kPickThreads / 64 && token < 0; ++w) token = L->first[w];
    for (int w = kPickThreads / 64 - 1; w >= 0 && token < 0; --w) token = L->lastnz[w];
    a.out.out_tokens[f.row] = token;
  }
}

}  // namespace otv
