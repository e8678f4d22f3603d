// Cross-lane sums, maxima and broadcasts of doubles within a 64-lane wave (device code
// only), through DPP and the lane-swap instructions.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

namespace ffo {

__device__ __forceinline__ double sgn(double x) { return (double)((x > 0.0) - (x < 0.0)); }

// Cross-lane moves of a double through DPP (two 32-bit halves; every source lane valid
// for the controls used here: quad_perm, the row mirrors, row_ror and row_newbcast).
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
constexpr int DPP_SWAP1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int DPP_SWAP2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141; // lane i <- 7 - i within each 8-lane half-row
constexpr int DPP_MIRROR = 0x140;      // lane i <- 15 - i within each 16-lane row
constexpr int DPP_ROR4 = 0x124;        // lane i <- (i - 4) mod 16 within each row
constexpr int DPP_ROR8 = 0x128;        // lane i <- i ^ 8 within each row
constexpr int DPP_BCAST = 0x150;       // + c: every lane of a row <- lane c of that row

// Sums over aligned groups of 4, 8 and 16 lanes; every lane of the group gets the sum.
__device__ __forceinline__ double sum4(double x) { x += dpp<DPP_SWAP1>(x); return x + dpp<DPP_SWAP2>(x); }
__device__ __forceinline__ double sum8(double x) { x = sum4(x); return x + dpp<DPP_HALF_MIRROR>(x); }
__device__ __forceinline__ double sum16(double x) { x = sum8(x); return x + dpp<DPP_MIRROR>(x); }
__device__ __forceinline__ double max8(double x) {
  x = fmax(x, dpp<DPP_SWAP1>(x));
  x = fmax(x, dpp<DPP_SWAP2>(x));
  return fmax(x, dpp<DPP_HALF_MIRROR>(x));
}
__device__ __forceinline__ double max16(double x) { x = max8(x); return fmax(x, dpp<DPP_MIRROR>(x)); }
__device__ __forceinline__ double lane_of(double x, int l) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Wave-wide sum / max (fixed order), uniform across the wave.
__device__ __forceinline__ double wave_sum(double x) {
  x = sum16(x);
  return (lane_of(x, 15) + lane_of(x, 31)) + (lane_of(x, 47) + lane_of(x, 63));
}
__device__ __forceinline__ double wave_max(double x) {
  x = max16(x);
  return fmax(fmax(lane_of(x, 15), lane_of(x, 31)), fmax(lane_of(x, 47), lane_of(x, 63)));
}

// Pair sums across half-waves and across neighbouring rows of 16 lanes.
// pair_sum32: lanes 0-31 get a(l) + a(l + 32), lanes 32-63 get b(l - 32) + b(l).
// pair_sum16: even rows get a(l) + a(l + 16), odd rows b(l - 16) + b(l).
__device__ __forceinline__ double u2d(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double pair_sum32(double a, double b) {
  const unsigned long long ua = (unsigned long long)__double_as_longlong(a), ub = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  return u2d(lo[0], hi[0]) + u2d(lo[1], hi[1]);
}
__device__ __forceinline__ double pair_sum16(double a, double b) {
  const unsigned long long ua = (unsigned long long)__double_as_longlong(a), ub = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
  return u2d(lo[0], hi[0]) + u2d(lo[1], hi[1]);
}

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>): a loop whose index
// is a compile-time constant (DPP controls are).
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// LDS-qualified element types: indexing through these compiles to ds_read/ds_write
// instead of generic (flat) memory instructions.
typedef __attribute__((address_space(3))) double ldbl;
typedef __attribute__((address_space(3))) int lint;

// Device-coherent (agent scope) accesses of exchanged words.
__device__ __forceinline__ double ldd(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void std_(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void addd(double* p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Budget-multiplier bracket shared by the solve kernels: candidates
// cen + f_q * hw, f = (-64, -16, -4, -1, 1, 4, 16, 64), clamped at 0.  The central pair
// (q = 3, 4) is the predicted bracket [lo, hi].
__device__ __forceinline__ double cand(double cen, double hw, int q) {
  const double f = (q < 4 ? -1.0 : 1.0) * (double)(1 << (2 * (q < 4 ? 3 - q : q - 4)));
  return fmax(cen + f * hw, 0.0);
}

// Relative half-width policy after a bracket decision r: kept on a hit, shrunk when
// breakpoints fell inside the central pair, grown when the root was outside.
__device__ __forceinline__ double adapt_width(int r, double w) {
  if (r == 1 || r == 2) return w;
  if (r == 0) return fmax(w * 0.7, 1e-13);
  return fmin(w * 1.6, 0.25);   // r = 3, 4: the root fell outside the central pair
}

}  // namespace ffo
