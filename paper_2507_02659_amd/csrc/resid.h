// Final token of every sequence (Algorithm 1: correction token from the residual, or free token from p), as device
// functions for the kernels that host the draw.
//
// At the first rejected row the token is drawn from norm(max(0, p - q')) (Notation paragraph), with q' extended over
// the whole target vocabulary by Eq. 2: q'(v) = q_s(tmap[v]) through the inverse direct map (0 where v has no
// pre-image), except that the n-gram matched at this position gets the product pi of its sub-token probabilities
// and the direct image of its first sub-token gets q_s(d_1) - pi.  When everything was accepted the draw is from p.
//
// Only the ONE row per sequence where the draw happens is touched.  A workgroup of 16 wavefronts takes a run of consecutive
// units of one sequence, a unit per wavefront and turn, of 64 * kPer target ids each (of a vast vocabulary a number of such blocks,
// draw_split):
//   every workgroup  forms the masses of max(0, p - q') of its units in binary64 and publishes them; when they have reached
//                    memory it looks at the masses of all units of its sequence, and ends if one is still missing;
//   the workgroup that finds them all  (the one whose masses arrive last does; more than one may, and they do the same)
//                    scans the masses to the unit that holds u * total, re-forms that unit with one id per thread, scans
//                    the running sum in ascending id order and emits the first id whose running sum exceeds the target
//                    (inverse CDF).  When the residual is empty (reachable only through underflow) it takes the masses of
//                    p, the fallback distribution, instead: every wavefront leaves that of a unit without residual mass in
//                    its place, negative (nothing to do in the common case).
// Nothing waits for another workgroup.  A mass that is missing reads as kNoMass, which the finder puts back for the next launch
// once it has its copy; a workgroup that looks while that happens ends, since the finder goes on.  (Counted in at one word
// per sequence instead, sixteen arrivals took 0.9 to 2.3 us next to each other and a look at the masses followed all the same.)
// A workgroup that has all units of its sequence (a small vocabulary, or many sequences) keeps the masses in LDS.
// What bounds a small batch is the chain of instructions and round trips in one workgroup, at the clock that the LM head leaves
// behind (2.4 GHz after 6 rows x 32000 ids, 1.25 after 144 x 128256): few instructions count for more than few bytes.  From its
// start to its end the launch that tests and draws takes 8.3 us there at 6 rows x 32000 ids and 17.9 at 144 x 128256; with tiles
// of 1024 ids, a counter per sequence and four ids per thread at the end it took 10.8 and 22.3 (12.1 and 24 with the test as it was).
#pragma once

#include "device_math.h"
#include "otv_internal.h"

namespace otv {

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // a row of logits may start at any float

constexpr int kDrawWaves = 16;                       // wavefronts per workgroup, unless two workgroups share a compute unit (draw_plan)

// p(v) and q'(v) of Eq. 2 at the final row of one sequence.
struct FinalRow {
  const float* z;
  float mx, sc_hi, sc_lo;        // row maximum; log2(e) / T split into two positive floats
  double invS;
  const void* zq;
  int lds_at;                    // where the draft row's copy starts in the dynamic LDS, in bytes (-1: there is none)
  bool exps;                     // the copy holds exp((x - max) / T_d) of the row's logits, in binary32, and 0 in front of the first
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
  __device__ static inline float exponential(float x, float mx, float sc_hi, float sc_lo) {
    const float d = x - mx;
    return __builtin_amdgcn_exp2f(fmaf(d, sc_hi, d * sc_lo));
  }
  __device__ static inline double softmax_term(float x, float mx, float sc_hi, float sc_lo, double invS) {
    return (double)exponential(x, mx, sc_hi, sc_lo) * invS;
  }
  __device__ inline double p_of(float zv) const { return softmax_term(zv, mx, sc_hi, sc_lo, invS); }
  // max(0, p - q') from the id's logit and the exponential of its pre-image, in units of the target's normaliser (ratio: -invSq /
  // invS): one product, rounded once.  The masses of the units and the ids of the one that is taken both come from this.
  __device__ inline double residual_of(float zv, float q_exp, double ratio) const {
    return fmax(0.0, fma((double)q_exp, ratio, (double)exponential(zv, mx, sc_hi, sc_lo)));
  }
  // q(d) of a sampling drafter from what load_tile left for the id's pre-image: a logit, or from the copy an exponential
  template <bool kExps> __device__ inline double q_of(float xq) const {
    return kExps ? (double)xq * invSq : softmax_term(xq, mxq, scq_hi, scq_lo, invSq);
  }
  // q'(v) given the draft id dv = tmap[v] (or -1) and, when dv >= 0 and the draft is not greedy, what q_of takes
  template <bool kExps> __device__ inline double qprime(int v, int dv, float xq) const {
    double q = 0.0;
    if (dv >= 0) q = greedy_draft ? ((dv == argq) ? 1.0 : 0.0) : q_of<kExps>(xq);
    if (v == t_pre) q = q_pre;
    if (v == t_ng) q = pi;       // the n-gram case of Eq. 2 wins when both name the same id
    return q;
  }
};

// The record is the same for every lane: all of it goes to scalar registers.
__device__ inline FinalRow make_final_row(const StepArgs& a, const FinalInfo& f) {
  FinalRow R;
  R.z = a.Z + (int64_t)uniform(f.row) * a.ldz;
  R.mx = uniform(f.mx); R.sc_hi = uniform(f.sc_hi); R.sc_lo = uniform(f.sc_lo); R.invS = uniform(f.invS);
  R.residual = uniform(f.mode) == 3;
  R.lds_at = -1;
  R.exps = false;
  R.dtype = a.dtype;
  R.t_ng = uniform(f.t_ng); R.t_pre = uniform(f.t_pre); R.pi = uniform(f.pi); R.q_pre = uniform(f.q_pre);
  R.zq = static_cast<const char*>(a.draft_logits) + (size_t)uniform(f.drow) * a.V_d * (a.dtype == OT_BF16 ? 2 : 4);
  R.mxq = uniform(f.mxq); R.scq_hi = uniform(f.scq_hi); R.scq_lo = uniform(f.scq_lo);
  R.invSq = uniform(f.invSq); R.argq = uniform(f.argq);
  R.greedy_draft = uniform(f.greedy_draft) != 0;
  return R;
}

// Inverse direct map of N ids v = first + e * stride (independent of which row is drawn from: issued early).  Ids past
// the vocabulary read the last entry and are masked afterwards: no branch around the loads.  all_exist (wavefront-uniform): there
// are none, and the loads share one address.
template <int N>
__device__ inline void load_tmap(const int32_t* __restrict__ tmap, int V_t, int first, int stride, bool all_exist, int* dv) {
  if (all_exist) {
    const int32_t* p = tmap + first;
#pragma unroll
    for (int e = 0; e < N; ++e) dv[e] = p[e * stride];
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) dv[e] = tmap[min(first + e * stride, V_t - 1)];
  }
}

// Stand-in logit of an id that does not exist or has no pre-image: finite, so that the two-float scaling below never
// meets inf * 0, and so far below any maximum that its exponential is exactly 0.
constexpr float kFarBelow = -1e30f;

// The dynamic LDS of the draw kernels: the units' masses, then (where a workgroup takes several turns) the draft row.
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

// The same from a copy of the row's exponentials: 0 for an id without a pre-image (dv = -1).
template <int N>
__device__ inline void load_draft_exps(int lds_at, const int* dv, uint32_t* xq) {
  const lds_chars s_row = draw_lds() + lds_at;
#pragma unroll
  for (int e = 0; e < N; ++e) xq[e] = *(const __attribute__((address_space(3))) uint32_t*)(s_row + 4 * dv[e]);
}

// What tile_values needs from memory for N ids v = first + e * stride, as loaded: the row's logits and, where the draw is
// from a residual of a sampling drafter, the logits of the ids' pre-images.
template <int N> struct TileRaw { float z[N]; uint32_t xq[N]; };

// All 2 N loads leave before anything waits: no lane is masked off (an id without a pre-image reads the row's first
// logit) and nothing is converted between two loads.  With the conversion inside a conditional block per id every
// gather was waited for by itself, eight round trips of about 1 us in a row.
template <int N>
__device__ inline void load_logits(const FinalRow& R, int V_t, int first, int stride, bool all_exist, float* z_out) {
  if (all_exist) {
    const float* z = R.z + first;
#pragma unroll
    for (int e = 0; e < N; ++e) z_out[e] = z[e * stride];
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) z_out[e] = R.z[min(first + e * stride, V_t - 1)];
  }
}
template <int N>
__device__ inline void load_tile(const FinalRow& R, int V_t, int first, int stride, bool all_exist, const int* dv, TileRaw<N>& raw) {
  load_logits<N>(R, V_t, first, stride, all_exist, raw.z);
  if (!R.residual || R.greedy_draft) {                   // wavefront-uniform
#pragma unroll
    for (int e = 0; e < N; ++e) raw.xq[e] = 0u;
  } else if (R.exps) {
    load_draft_exps<N>(R.lds_at, dv, raw.xq);
  } else {
    load_draft_logits<N>(R.zq, R.dtype, R.lds_at, dv, raw.xq);
  }
}

// Mass r(v) of those ids, the N of them across the wavefront inside [lo, hi): max(0, p - q'), or p where the draw is from
// p.  The common case (all ids exist, a sampling drafter, no id of Eq. 2's two overrides among them: tested once per
// wavefront) costs an id about twenty instructions, or fourteen where the draft row's exponentials are in LDS.
template <int N, bool kExps>
__device__ inline void subtract_draft(const FinalRow& R, int V_t, int first, int stride, int lo, int hi, const int* dv,
                                      const TileRaw<N>& raw, double* r) {
  float xq[N];
  if (kExps) {
#pragma unroll
    for (int e = 0; e < N; ++e) xq[e] = __uint_as_float(raw.xq[e]);
  } else {
    const uint32_t shift = R.dtype == OT_BF16 ? 16u : 0u;
#pragma unroll
    for (int e = 0; e < N; ++e) xq[e] = dv[e] >= 0 ? __uint_as_float(raw.xq[e] << shift) : kFarBelow;
  }
  const bool special = R.greedy_draft || (R.t_pre >= lo && R.t_pre < hi) || (R.t_ng >= lo && R.t_ng < hi);
  if (!special && kExps) {
    const double ratio = -(R.invSq / R.invS);
#pragma unroll
    for (int e = 0; e < N; ++e) r[e] = R.residual_of(hi <= V_t || first + e * stride < V_t ? raw.z[e] : kFarBelow, xq[e], ratio) * R.invS;
  } else if (!special) {
#pragma unroll
    for (int e = 0; e < N; ++e)                                   // no pre-image: 2^(-huge) = 0; beyond V_t: max(0, 0 - q) = 0
      r[e] = fmax(0.0, r[e] - R.q_of<kExps>(xq[e]));
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const int v = first + e * stride;
      r[e] = v < V_t ? fmax(0.0, r[e] - R.qprime<kExps>(v, dv[e], xq[e])) : 0.0;
    }
  }
}
template <int N>
__device__ inline void target_masses(const FinalRow& R, int V_t, int first, int stride, int hi, const float* z, double* r) {
  if (hi <= V_t) {
#pragma unroll
    for (int e = 0; e < N; ++e) r[e] = R.p_of(z[e]);
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) r[e] = R.p_of(first + e * stride < V_t ? z[e] : kFarBelow);   // beyond V_t: 2^(-huge) = 0
  }
}
template <int N>
__device__ inline void tile_values(const FinalRow& R, int V_t, int first, int stride, int lo, int hi, const int* dv,
                                   const TileRaw<N>& raw, double* r) {
  target_masses<N>(R, V_t, first, stride, hi, raw.z, r);
  if (!R.residual) return;
  if (R.exps) subtract_draft<N, true>(R, V_t, first, stride, lo, hi, dv, raw, r);
  else subtract_draft<N, false>(R, V_t, first, stride, lo, hi, dv, raw, r);
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

// Copies the draft row's exponentials exp((x - max) / T_d), as softmax_term forms them in front of the normaliser, to byte `at` of
// the dynamic LDS, a multiple of 16 with room for exps_bytes(V_d) (all threads call it, a barrier follows).  The elements of a
// 16-byte chunk of the row lie on a 16-byte boundary there; what a chunk holds of other rows counts as an id without a pre-image (0),
// and so does the element in front of the first.  Returns where the row starts.
__host__ __device__ constexpr size_t exps_bytes(int V_d) { return 4 * ((size_t)V_d + 20); }
template <int kThreads, typename T>
__device__ inline int stage_draft_exps(const FinalRow& R, int V_d, int tid, int at) {
  constexpr int kVec = 16 / sizeof(T), kAtOnce = 4;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const T* row = static_cast<const T*>(R.zq);
  const int head = (int)(reinterpret_cast<uintptr_t>(row) & 15) / (int)sizeof(T);   // elements of the first chunk in front of the row
  const int chunks = (head + V_d + kVec - 1) / kVec;
  const int whole0 = head ? 1 : 0, whole1 = (head + V_d) / kVec;     // chunks [whole0, whole1) lie inside the row
  const lds_chars s_row = draw_lds() + at + 16;                      // where the first chunk goes
  auto put = [&](int c, const float (&x)[kVec]) {
    float t[kVec];
#pragma unroll
    for (int e = 0; e < kVec; ++e) t[e] = FinalRow::exponential(x[e], R.mxq, R.scq_hi, R.scq_lo);
#pragma unroll
    for (int e = 0; e < kVec; e += 4)
      *(__attribute__((address_space(3))) f32x4*)(s_row + (c * kVec + e) * 4) = f32x4{t[e], t[e + 1], t[e + 2], t[e + 3]};
  };
  auto bits = [](const u32x4& raw, int e) {
    return sizeof(T) == 4 ? raw[e & 3] : e & 1 ? raw[(e / 2) & 3] & 0xFFFF0000u : raw[(e / 2) & 3] << 16;
  };
  for (int c0 = tid; c0 < chunks; c0 += kAtOnce * kThreads) {
    u32x4 raw[kAtOnce];
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {                    // any other chunk number loads the nearest of those
      const int c = min(max(c0 + j * kThreads, whole0), whole1 - 1);
      raw[j] = whole0 < whole1 ? *reinterpret_cast<const u32x4*>(row + (c * kVec - head)) : u32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int c = c0 + j * kThreads;
      if (c >= chunks) break;
      float x[kVec];
      if (c >= whole0 && c < whole1) {
#pragma unroll
        for (int e = 0; e < kVec; ++e) x[e] = __uint_as_float(bits(raw[j], e));
      } else {
#pragma unroll
        for (int e = 0; e < kVec; ++e) {
          const int i = c * kVec - head + e;
          x[e] = i < 0 || i >= V_d ? kFarBelow
                 : sizeof(T) == 4  ? reinterpret_cast<const float*>(row)[i]
                                   : bf16_to_f32(reinterpret_cast<const uint16_t*>(row)[i]);
        }
      }
      put(c, x);
    }
  }
  if (tid == 0)
    *(__attribute__((address_space(3))) float*)(s_row + (head - 1) * 4) = FinalRow::exponential(kFarBelow, R.mxq, R.scq_hi, R.scq_lo);
  return at + 16 + head * 4;
}

struct DrawLds {
  double w[16];                 // sums of the chosen unit's wavefronts
  int missing;
};

constexpr size_t kDrawLdsBytes = 150 << 10;    // dynamic LDS of a workgroup with a copy of the draft row at most (160 KB a compute unit)

// Mass of the unit of 64 * kPer ids from `lo` on (this lane: lo + lane + e * 64), in every lane: of the residual or, where that
// is zero, minus that of p.
template <int kPer>
__device__ inline double unit_mass(const FinalRow& R, int V_t, int lo, int lane, const int* dv, const TileRaw<kPer>& raw) {
  double r[kPer];
  auto sum = [&](const FinalRow& S) {
    tile_values<kPer>(S, V_t, lo + lane, 64, lo, lo + 64 * kPer, dv, raw, r);
    double x = r[0] + r[1];
#pragma unroll
    for (int e = 2; e < kPer; e += 2) x += r[e] + r[e + 1];
    return wave_sum(x);
  };
  const double mass = sum(R);
  if (!R.residual || !(mass == 0.0)) return mass;
  FinalRow P = R;
  P.residual = false;
  return -sum(P);
}

// In the workspace for a unit whose mass is not there (bits of a NaN that no arithmetic gives).
constexpr unsigned long long kNoMassBits = ~0ull;
__device__ inline bool no_mass(double x) { return (unsigned long long)__double_as_longlong(x) == kNoMassBits; }

// A mass as stored (the residual's or, negative, that of p) as one of the distribution that is drawn from.
__device__ inline double drawn_mass(double x, bool of_p) { return of_p ? fabs(x) : fmax(x, 0.0); }

// What the scan of the masses chooses: the unit, the mass in front of it, and the target mass u * total.
struct UnitPick { int unit; double base, target; bool empty; };

// Mass of a unit of several blocks from those of two parts of it: minus that of p where neither holds residual mass.
__device__ inline double joined_mass(double a, double b) { return a <= 0.0 && b <= 0.0 ? a + b : fmax(a, 0.0) + fmax(b, 0.0); }

// By one wavefront, from the masses of n_units units (at most 4096) in LDS and the sums of 64 of them each.  The total and the
// crossing come from the same sums; where rounding pushes the target past the end the last unit with mass is taken.  What is taken
// has mass of its own at every level: every lane of a scan adds in another order, so that a running sum can pass the target at an
// entry of zero, by a unit in the last place.
// kInside: among the blocks of a unit that was taken, `from` (its base and the target), instead.
template <bool kInside = false>
__device__ inline UnitPick pick_unit(const double* s_mass, const double* s_sums, int n_units, double u2, int lane, bool of_p,
                                     const UnitPick& from = UnitPick{0, 0.0, 0.0, false}) {
  const int n_chunks = (n_units + 63) / 64;
  UnitPick p;
  const double sum = s_sums[min(lane, n_chunks - 1)], x = lane < n_chunks ? sum : 0.0;
  const double incl = wave_scan(x) + from.base, total = lane_value(incl, 63);
  p.empty = !(total > 0.0);
  p.target = kInside ? from.target : u2 * total;
  p.base = from.base;
  int c = 0;
  const unsigned long long past = __ballot(x > 0.0 && incl > p.target), some = past ? past : __ballot(x > 0.0);
  if (some) {
    c = past ? (int)__builtin_ctzll(past) : 63 - (int)__builtin_clzll(some);
    if (c > 0) p.base = lane_value(incl, c - 1);
  }
  const double m = c * 64 + lane < n_units ? drawn_mass(s_mass[c * 64 + lane], of_p) : 0.0;
  const double run = wave_scan(m);
  const unsigned long long past1 = __ballot(m > 0.0 && p.base + run > p.target), some1 = __ballot(m > 0.0);
  const int i = past1 ? (int)__builtin_ctzll(past1) : some1 ? 63 - (int)__builtin_clzll(some1) : 0;
  p.unit = c * 64 + i;
  if (i > 0) p.base += lane_value(run, i - 1);
  return p;
}

// How the draw is split, see draw_split.  A unit is `blocks` (1 unless kBlocks) times 64 * kPer ids, at most 1024 blocks; row_at:
// where the draft row's copy starts in the dynamic LDS, in doubles (0: no copy); exps: of its exponentials (stage_draft_exps), for the
// kernels that have their code (kExps).
struct DrawSplit { int n_units, group_units, row_at, blocks; bool exps; };
template <int kPer, bool kBlocks>
__device__ inline int draw_first_id(const DrawSplit& s, int grp, int wave) {
  return (grp * s.group_units + wave) * (64 * kPer) * (kBlocks ? s.blocks : 1);
}

// Workgroup `grp` of sequence b takes units [grp * group_units, (grp + 1) * group_units) of n_units, group_units a multiple of
// kWaves (all threads call this; f is the sequence's outcome record with f.mode != 0; dv holds tmap of the ids
// draw_first_id + lane + e * 64, e < kPer).  The dynamic LDS holds 65 doubles for every 64 units begun (draw_lds_doubles) and, if
// row_at > 0, from double row_at on room for the draft row and 32 bytes.
__host__ __device__ inline int draw_lds_doubles(int n_units) { return (n_units + 63) / 64 * 65; }
template <int kPer, bool kBlocks, int kWaves, bool kExps>
__device__ inline void draw_final_token(const StepArgs& a, int b, int grp, const DrawSplit& split, const FinalInfo& f, int* dv,
                                        DrawLds* L) {
  constexpr int kThreads = 64 * kWaves;
  static_assert(kWaves >= kPer, "a wavefront for every 64 ids of a block");
  constexpr int kUnit = 64 * kPer;                        // ids of a block
  const int n_units = split.n_units, group_units = split.group_units, row_at = split.row_at, blocks = kBlocks ? split.blocks : 1;
  const int tid = threadIdx.x, wave = uniform((int)(threadIdx.x >> 6)), lane = tid & 63;
  const int n_chunks = (n_units + 63) / 64;
  double *s_mass = s_draw_dynamic, *s_sums = s_mass + n_chunks * 64;   // the masses; the sums of 64 each
  FinalRow R = make_final_row(a, f);
  const int unit0 = grp * group_units, unit1 = min(unit0 + group_units, n_units);
  const bool alone = gridDim.x == 1;
  double* masses = a.unit_mass + (int64_t)b * a.max_units;
  if (tid == 0) L->missing = 0;
  // of the units this wavefront takes, those whose ids all exist: the first one's logits and pre-images are asked for in front of the
  // copy of the draft row
  int unit = unit0 + wave;
  const int n_whole = min(unit1, a.V_t / kUnit);
  constexpr int kVecs = kPer < 4 ? 1 : kPer / 4;
  f32x4_any z4[kVecs];
  int4 d4[kVecs];
  auto fetch = [&](int u_want) {                          // past the last turn the last unit once more
    const int u = min(u_want, n_whole - 1);
    const float* z = R.z + u * kUnit;
    const int32_t* t = a.tmap + u * kUnit;
#pragma unroll
    for (int j = 0; j < kVecs; ++j) {
      z4[j] = *reinterpret_cast<const f32x4_any*>(z + 256 * j + 4 * lane);
      d4[j] = *reinterpret_cast<const int4*>(t + 256 * j + 4 * lane);
    }
  };
  if (row_at > 0 && R.residual && !R.greedy_draft) {     // workgroup-uniform
    R.exps = kExps && split.exps;
    if (R.exps && !kBlocks && n_whole > 0) fetch(unit);
    if (!R.exps) R.lds_at = stage_draft_row<kThreads>(R.zq, R.dtype, a.V_d, tid, 8 * row_at);
    else if (a.dtype == OT_BF16) R.lds_at = stage_draft_exps<kThreads, uint16_t>(R, a.V_d, tid, 8 * row_at);
    else R.lds_at = stage_draft_exps<kThreads, float>(R, a.V_d, tid, 8 * row_at);
    __syncthreads();
  }

  // ---- masses of this workgroup's units, a wavefront on each (coalesced: consecutive lanes on consecutive ids)
  auto deliver = [&](int u, double mass) {
    if (lane == 0) {
      if (alone) s_mass[u] = mass;
      else publish(masses + u, mass);
    }
  };
  auto overridden = [&](int lo) { return (R.t_pre >= lo && R.t_pre < lo + kUnit) || (R.t_ng >= lo && R.t_ng < lo + kUnit); };
  auto general_mass = [&](int u) {
    const int lo = u * kUnit;
    const bool all_exist = lo + kUnit <= a.V_t;
    TileRaw<kPer> raw;
    load_tmap<kPer>(a.tmap, a.V_t, lo + lane, 64, all_exist, dv);
    load_tile<kPer>(R, a.V_t, lo + lane, 64, all_exist, dv, raw);
    return unit_mass<kPer>(R, a.V_t, lo, lane, dv, raw);
  };
  if (R.exps && !kBlocks) {
    // The draft row is in LDS, and all that a turn waits for is the target's logits and the inverse map: asked for a turn ahead (two
    // are no faster), four consecutive ids a lane and load, without a branch between a load and its use.  The target's normaliser
    // is left to the sum.
    const double ratio = -(R.invSq / R.invS);
    for (; unit < n_whole; unit += kWaves) {
      f32x4_any z[kVecs];
      int4 d[kVecs];
#pragma unroll
      for (int j = 0; j < kVecs; ++j) { z[j] = z4[j]; d[j] = d4[j]; }
      fetch(unit + kWaves);
      double x = 0.0;
#pragma unroll
      for (int j = 0; j < kVecs; ++j) {
        const int dj[4] = {d[j].x, d[j].y, d[j].z, d[j].w};
        uint32_t q[4];
        load_draft_exps<4>(R.lds_at, dj, q);
        double r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = R.residual_of(z[j][e], __uint_as_float(q[e]), ratio);
        x += (r[0] + r[1]) + (r[2] + r[3]);
      }
      x = wave_sum(x) * R.invS;
      // an override of Eq. 2 among the unit's ids, or no residual mass: that of p is wanted
      if (x == 0.0 || overridden(unit * kUnit)) x = general_mass(unit);
      deliver(unit, x);
    }
    if (unit < unit1) deliver(unit, general_mass(unit));   // the ragged last one
  } else {
    for (; unit < unit1; unit += kWaves) {
      double mass = 0.0;
      int blk = 0;
      do {
        const int lo = (unit * blocks + blk) * kUnit;
        TileRaw<kPer> raw;
        load_tile<kPer>(R, a.V_t, lo + lane, 64, lo + kUnit <= a.V_t, dv, raw);
        int dv_next[kPer] = {};                          // asked for behind what this turn waits for
        const bool inside = kBlocks && blk + 1 < blocks;
        const int lo_next = inside ? lo + kUnit : (unit + kWaves) * blocks * kUnit;
        if (inside || unit + kWaves < unit1)
          load_tmap<kPer>(a.tmap, a.V_t, lo_next + lane, 64, lo_next + kUnit <= a.V_t, dv_next);
        const double m = unit_mass<kPer>(R, a.V_t, lo, lane, dv, raw);
        mass = kBlocks ? joined_mass(mass, m) : m;
        if (!inside) deliver(unit, mass);
#pragma unroll
        for (int e = 0; e < kPer; ++e) dv[e] = dv_next[e];
      } while (kBlocks && ++blk < blocks);
    }
  }
  if (!alone) stores_done();                              // of this wavefront; behind the barrier, of all of them
  __syncthreads();
  auto sum_chunks = [&](bool of_p, bool from_memory) {
    for (int c = wave; c < n_chunks; c += kWaves) {
      const int t = c * 64 + lane;
      double x = 0.0;
      if (from_memory) {
        x = observe(masses + min(t, n_units - 1));
        if (no_mass(x)) L->missing = 1;
        s_mass[t] = x;
      } else {
        x = s_mass[t];
      }
      x = wave_sum(t < n_units ? drawn_mass(x, of_p) : 0.0);
      if (lane == 0) s_sums[c] = x;
    }
  };
  sum_chunks(false, !alone);
  __syncthreads();
  if (!alone) {
    if (L->missing) return;
    for (int t = tid; t < n_units; t += kThreads) publish(masses + t, __longlong_as_double((long long)kNoMassBits));
  }

  // ---- inverse CDF over the masses (every wavefront for itself), then inside the unit that holds the draw: kPer wavefronts
  // take 64 ids each
  UnitPick P = pick_unit(s_mass, s_sums, n_units, f.u2, lane, false);
  if (P.empty) {                                          // residual of zero mass: draw from p
    R.residual = false;
    __syncthreads();
    sum_chunks(true, false);
    __syncthreads();
    P = pick_unit(s_mass, s_sums, n_units, f.u2, lane, true);
    P.empty = true;
  }
  if constexpr (kBlocks) {                                // the same among the unit's blocks, whose masses take the place of the units'
    __syncthreads();
    for (int blk = wave; blk < blocks; blk += kWaves) {
      const int lo = (uniform(P.unit) * blocks + blk) * kUnit;
      const bool all_exist = lo + kUnit <= a.V_t;
      TileRaw<kPer> raw;
      load_tmap<kPer>(a.tmap, a.V_t, lo + lane, 64, all_exist, dv);
      load_tile<kPer>(R, a.V_t, lo + lane, 64, all_exist, dv, raw);
      const double m = unit_mass<kPer>(R, a.V_t, lo, lane, dv, raw);
      if (lane == 0) s_mass[blk] = m;
    }
    __syncthreads();
    for (int c = wave; c * 64 < blocks; c += kWaves) {
      const double x = wave_sum(c * 64 + lane < blocks ? drawn_mass(s_mass[c * 64 + lane], false) : 0.0);
      if (lane == 0) s_sums[c] = x;
    }
    __syncthreads();
    const UnitPick Q = pick_unit<true>(s_mass, s_sums, blocks, 0.0, lane, false, P);
    P.unit = P.unit * blocks + Q.unit;
    P.base = Q.base;
  }
  double r = 0.0, incl = 0.0;
  const int lo = uniform(P.unit) * kUnit + wave * 64;
  if (wave < kPer) {
    const bool all_exist = lo + 64 <= a.V_t;
    int dvp;
    TileRaw<1> raw;
    load_tmap<1>(a.tmap, a.V_t, lo + lane, 0, all_exist, &dvp);
    load_tile<1>(R, a.V_t, lo + lane, 0, all_exist, &dvp, raw);
    tile_values<1>(R, a.V_t, lo + lane, 0, lo, lo + 64, &dvp, raw, &r);
    incl = wave_scan(r);
    if (lane == 63) L->w[wave] = incl;
  }
  __syncthreads();
  if (wave < kPer) {
    // lane w: what the first w + 1 wavefronts hold.  The wavefront in whose ids the running sum passes the target writes: the same
    // sums in every wavefront, so it is one of them (rounding past the end: the last with mass)
    const double own = lane < kPer ? L->w[lane] : 0.0, sums = wave_scan(own);
    const unsigned long long past = __ballot(own > 0.0 && P.base + sums > P.target), some = __ballot(own > 0.0);
    const int at = past ? (int)__builtin_ctzll(past) : some ? 63 - (int)__builtin_clzll(some) : 0;
    if (wave == at) {
      const double before = P.base + (wave > 0 ? lane_value(sums, wave - 1) : 0.0);
      const unsigned long long past1 = __ballot(r > 0.0 && before + incl > P.target), some1 = __ballot(r > 0.0);
      const int i = past1 ? (int)__builtin_ctzll(past1) : some1 ? 63 - (int)__builtin_clzll(some1) : -1;
      if (lane == 0) {
        a.out.out_tokens[f.row] = i >= 0 ? lo + i : -1;
        a.out.flags[b] = f.flags | (P.empty ? OT_FLAG_RESID_ZERO : 0);
      }
    }
  }
}

}  // namespace otv
