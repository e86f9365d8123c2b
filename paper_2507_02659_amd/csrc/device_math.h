// Small device helpers shared by the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace otv {

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// exp(x) for x <= 0 in binary64 with a relative error of about one binary32 ulp (1e-7), at a dozen instructions
// instead of a full binary64 exponential: the range reduction x*log2(e) = n + f, |f| <= 1/2, is done in binary64, the
// fraction goes through the hardware 2^f, and the result is scaled by 2^n.  Used where millions of terms are summed
// (residual masses); single decisive values (p(t_j), q') use the full-precision exp().
__device__ inline double exp_neg_fast(double x) {
  const double t = fmax(x, -1000.0) * 1.4426950408889634;
  const double n = rint(t);
  const float e = __builtin_amdgcn_exp2f((float)(t - n));
  return ldexp((double)e, (int)n);
}

// A value that every lane of the wavefront holds alike, moved to scalar registers (addresses formed from it cost no
// vector instructions).
__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
__device__ inline double uniform(double x) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)), __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// The value that lane l holds (l the same in every lane), in every lane.
__device__ inline double lane_value(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Sum over the 64 lanes in one fixed order, the result in every lane.  The partners come through data-parallel moves
// inside a row of 16 lanes and row broadcasts above it: no trip through the LDS permute network, whose latency six steps
// of __shfl_xor would pay one after the other.
template <int kCtrl, int kRowMask = 0xF>
__device__ inline double dpp_f64(double x) {
  constexpr bool kAllRows = kRowMask == 0xF;             // then lanes without a partner are zeroed by the move itself
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), kCtrl, kRowMask, 0xF, kAllRows);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), kCtrl, kRowMask, 0xF, kAllRows);
  return __hiloint2double(hi, lo);                       // rows outside the mask receive +0.0
}
__device__ inline double row16_sum(double x) {
  x += dpp_f64<0xB1>(x);             // neighbours 1 apart
  x += dpp_f64<0x4E>(x);             // 2 apart
  x += dpp_f64<0x141>(x);            // mirrored halves of eight lanes
  x += dpp_f64<0x140>(x);            // mirrored row of sixteen: every lane holds its row's sum
  return x;
}
__device__ inline double wave_sum(double x) {
  x = row16_sum(x);
  x += dpp_f64<0x142, 0xA>(x);       // lane 15 of row 0 into row 1, of row 2 into row 3
  x += dpp_f64<0x143, 0xC>(x);       // lane 31 into rows 2 and 3: lane 63 holds the total
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63), __builtin_amdgcn_readlane(__double2loint(x), 63));
}
// Inclusive running sum over the lanes in ascending order.
__device__ inline double wave_scan(double x) {
  x += dpp_f64<0x111>(x);            // from 1, 2, 4, 8 lanes below within the row of sixteen (nothing: +0.0)
  x += dpp_f64<0x112>(x);
  x += dpp_f64<0x114>(x);
  x += dpp_f64<0x118>(x);
  x += dpp_f64<0x142, 0xA>(x);
  x += dpp_f64<0x143, 0xC>(x);
  return x;
}
// Maximum / minimum over the 64 lanes, in every lane (a masked-off lane meets its own value).
template <int kCtrl, int kRowMask = 0xF>
__device__ inline int dpp_self(int x) { return __builtin_amdgcn_update_dpp(x, x, kCtrl, kRowMask, 0xF, false); }
template <int kCtrl, int kRowMask = 0xF>
__device__ inline float dpp_self(float x) { return __int_as_float(dpp_self<kCtrl, kRowMask>(__float_as_int(x))); }
__device__ inline float row16_max(float x) {
  x = fmaxf(x, dpp_self<0xB1>(x)); x = fmaxf(x, dpp_self<0x4E>(x)); x = fmaxf(x, dpp_self<0x141>(x));
  return fmaxf(x, dpp_self<0x140>(x));
}
__device__ inline int row16_min(int x) {
  x = min(x, dpp_self<0xB1>(x)); x = min(x, dpp_self<0x4E>(x)); x = min(x, dpp_self<0x141>(x));
  return min(x, dpp_self<0x140>(x));
}
__device__ inline float wave_max(float x) {
  x = row16_max(x);
  x = fmaxf(x, dpp_self<0x142, 0xA>(x)); x = fmaxf(x, dpp_self<0x143, 0xC>(x));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ inline int wave_min(int x) {
  x = row16_min(x);
  x = min(x, dpp_self<0x142, 0xA>(x)); x = min(x, dpp_self<0x143, 0xC>(x));
  return __builtin_amdgcn_readlane(x, 63);
}

// Sequence that owns `row`: rows of sequence b start at off[b] - shift*b (shift = 0 target rows, 1 draft rows).  Called by
// a whole wavefront: 64 evenly spaced sequences are looked at in one round trip, then 64 between two of those, and so on
// (two round trips up to 4096 sequences; a binary search was nine at 300).
__device__ inline int find_sequence(const int32_t* off, int B, int row, int shift, int lane) {
  int base = 0, n = B;
  for (;;) {
    const int step = (n + 63) / 64, b = base + lane * step;
    const bool before = b < base + n && off[min(b, B - 1)] - shift * b <= row;
    const int at = max(0, (int)__popcll(__ballot(before)) - 1);
    base += at * step;
    if (step == 1) return base;
    n = min(step, n - at * step);
  }
}

// Agent-scope accesses to what the workgroups of one launch hand to each other and to their arrival counters.  They run on
// different XCDs,
// each with its own L2, and exchange these few words through memory: the stores are write-through, the loads bypass
// the local L2 and the counter lives in memory, so no whole-cache write-back or invalidate is needed.
__device__ inline void publish(double* p, double v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double observe(double* p) {
  return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<unsigned long long*>(p), __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT));
}

__device__ inline void publish(int32_t* p, int32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline int32_t observe(int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Returns when this wavefront's stores have reached memory.
__device__ inline void stores_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): vector-memory stores count there as well
  asm volatile("" ::: "memory");
}
// Counts this thread's earlier stores in (they have reached memory first); true for the n-th of n, which resets the counter.
__device__ inline bool arrive(int32_t* count, int n) {
  stores_done();
  const bool last = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
  if (last) publish(count, 0);
  return last;
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies and key-mixed xors.
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                                     uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Uniform in [0, 1): the top 24 bits of a word, exactly representable in binary32 and binary64.
__device__ inline double u24(uint32_t w) { return (double)(w >> 8) * (1.0 / 16777216.0); }

}  // namespace otv
