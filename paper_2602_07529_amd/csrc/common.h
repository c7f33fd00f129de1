// Internal helpers shared by the HIP translation units of libdagattn (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dagattn.h"
#include "sizes.h"

#define DAG_HIP_CHECK(expr)                    \
  do {                                         \
    hipError_t e__ = (expr);                   \
    if (e__ != hipSuccess) return DAG_ERR_HIP; \
  } while (0)

#define DAG_LAUNCH_CHECK()                             \
  do {                                                 \
    if (hipGetLastError() != hipSuccess) return DAG_ERR_HIP; \
  } while (0)

static inline bool dag_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// fp32 -> bf16 bits, round to nearest even (NaN not expected on these paths but kept quiet).
__device__ __forceinline__ uint32_t dag_f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
// Two fp32 -> packed bf16 pair (lo in bits 0..15) with the hardware conversion (round to nearest
// even, one v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t dag_pack_bf2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float dag_f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 dag_bf16x2;
  const dag_f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, dag_bf16x2));
}
__device__ __forceinline__ float dag_bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float dag_bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

static inline int dag_compute_units() {  // of the current device; 0: it cannot be asked
  int dev = 0, n = 0;
  return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
}

// Whether a row of D bf16 (16-byte aligned) holds an Inf or NaN.
template <int D>
__device__ __forceinline__ bool dag_row_not_finite(const void* row) {
  bool bad = false;
#pragma unroll
  for (int s = 0; s < D / 8; ++s) {
    const u32x4 x = ((const u32x4*)row)[s];
#pragma unroll
    for (int e = 0; e < 4; ++e) bad |= (x[e] & 0x7f80u) == 0x7f80u || (x[e] & 0x7f800000u) == 0x7f800000u;
  }
  return bad;
}

// RoPE frequencies theta^(-2 m / D), m = 0 .. D / 2 - 1, for every kernel that rotates: a key has the same angles in dag_rope_qk and
// in dag_kv_append_rope.  exp2 of -2 m / D log2(theta) with the product in two doubles: as close as pow (largest and mean error
// over 20 thetas from 1e-45 to 3e38, D 64 to 256: 1.14 and 0.30 units in the last place, pow 1.21 and 0.31) in a third of its
// instructions (an append of one token 3.3 us, with pow 3.7).
struct RopeTheta {
  double hi, lo;  // log2(theta)
};
static inline RopeTheta dag_rope_theta(float theta) {
  if (isinf(theta)) return {1e300, 0.};  // (frequency 0 but for m = 0; an infinite logarithm would make NaN of it)
  const long double l = log2l((long double)theta);
  return {(double)l, (double)(l - (long double)(double)l)};
}
__device__ __forceinline__ double dag_rope_freq(RopeTheta t, int m, int D) {
  const double r = -2.0 * (double)m / (double)D, y = r * t.hi;
  const double e = fma(r, t.hi, -y) + r * t.lo;
  const double f = exp2(y);
  return fma(f, e * 0.69314718055994530942, f);
}

// Reductions and scans over the 64 lanes of a wave, in registers: DPP moves inside the rows of 16 lanes and the swaps of rows and
// of halves between them.  A shuffle goes through LDS and takes its latency at every one of the six steps: the sum of a
// wave 0.35 us instead of 0.03, which is what the one-workgroup table kernels were made of.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dag_dpp(uint32_t x) {  // lanes without a source, and rows outside ROWS: 0
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
// x of lane (lane ^ N), for an x that is the same in every aligned group of N lanes
template <int N>
__device__ __forceinline__ uint32_t dag_other_group(uint32_t x) {
  static_assert(N == 1 || N == 2 || N == 4 || N == 8 || N == 16 || N == 32, "");
  if constexpr (N == 1) return dag_dpp<0xb1>(x);         // quad_perm [1, 0, 3, 2]
  else if constexpr (N == 2) return dag_dpp<0x4e>(x);    // quad_perm [2, 3, 0, 1]
  else if constexpr (N == 4) return dag_dpp<0x141>(x);   // row_half_mirror
  else if constexpr (N == 8) return dag_dpp<0x140>(x);   // row_mirror
  else {
    const auto r = [&] {
      if constexpr (N == 16) return __builtin_amdgcn_permlane16_swap(x, x, false, false);
      else return __builtin_amdgcn_permlane32_swap(x, x, false, false);
    }();
    return (threadIdx.x & N) ? r[0] : r[1];
  }
}
template <int N = 32>
__device__ __forceinline__ int dag_wave_sum(int x) {  // over aligned groups of 2 N lanes
  if constexpr (N > 1) x = dag_wave_sum<N / 2>(x);
  return x + (int)dag_other_group<N>((uint32_t)x);
}
template <int N = 32>
__device__ __forceinline__ float dag_wave_sum(float x) {
  if constexpr (N > 1) x = dag_wave_sum<N / 2>(x);
  return x + __uint_as_float(dag_other_group<N>(__float_as_uint(x)));
}
template <int N = 32>
__device__ __forceinline__ float dag_wave_max(float x) {
  if constexpr (N > 1) x = dag_wave_max<N / 2>(x);
  return fmaxf(x, __uint_as_float(dag_other_group<N>(__float_as_uint(x))));
}
template <int N = 32>
__device__ __forceinline__ int64_t dag_wave_sum(int64_t x) {
  if constexpr (N > 1) x = dag_wave_sum<N / 2>(x);
  return x + (int64_t)((uint64_t)dag_other_group<N>((uint32_t)((uint64_t)x >> 32)) << 32 | dag_other_group<N>((uint32_t)x));
}
// Sum over the lanes up to this one.
__device__ __forceinline__ int dag_wave_scan(int x) {
  x += (int)dag_dpp<0x111>((uint32_t)x);       // row_shr 1, 2, 4, 8
  x += (int)dag_dpp<0x112>((uint32_t)x);
  x += (int)dag_dpp<0x114>((uint32_t)x);
  x += (int)dag_dpp<0x118>((uint32_t)x);
  x += (int)dag_dpp<0x142, 0xa>((uint32_t)x);  // the sums of rows 0 and 2 to rows 1 and 3
  x += (int)dag_dpp<0x143, 0xc>((uint32_t)x);  // that of the lower half to the upper one
  return x;
}
__device__ __forceinline__ int64_t dag_wave_scan(int64_t x) {
  auto step = [&](auto move) __attribute__((always_inline)) {
    x += (int64_t)((uint64_t)move((uint32_t)((uint64_t)x >> 32)) << 32 | move((uint32_t)x));
  };
  step([](uint32_t y) { return dag_dpp<0x111>(y); });
  step([](uint32_t y) { return dag_dpp<0x112>(y); });
  step([](uint32_t y) { return dag_dpp<0x114>(y); });
  step([](uint32_t y) { return dag_dpp<0x118>(y); });
  step([](uint32_t y) { return dag_dpp<0x142, 0xa>(y); });
  step([](uint32_t y) { return dag_dpp<0x143, 0xc>(y); });
  return x;
}
__device__ __forceinline__ int64_t dag_readlane(int64_t x, int lane) {
  return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)((uint64_t)x >> 32), lane) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)x, lane));
}

// Largest sequence index b with start[b] <= x, for a non-decreasing array start[0..n] (start[0] = 0).
template <typename T>
__device__ __forceinline__ int dag_find_segment(const T* start, int n, T x) {
  int lo = 0, hi = n;  // invariant: start[lo] <= x < start[hi] (conceptually start[n] > x)
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (start[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}
