// Exchange among the workgroups of a team, shared by the row-register kernels (device code
// only): device-scope atomic adds into grouped copies of a triple-buffered slot, a two-level
// counter barrier with bounded waits, and device-scope loads of the totals, so that no L2
// fence is needed.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "internal.h"
#include "wave_ops.h"

namespace ffo {

__device__ __forceinline__ int wave_of(int tid) { return __builtin_amdgcn_readfirstlane(tid >> 6); }

// The thread index, opaque to the compiler: addresses and masks made from it stay in the
// block that uses them (hoisted out of the iteration they would take registers from the rows).
__device__ __forceinline__ int fresh(int tid) {
  asm volatile("" : "+v"(tid));
  return tid;
}

// A value that is the same in every lane, as a scalar register pair.
__device__ __forceinline__ double uni(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return u2d((unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u),
             (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32)));
}

// A pointer likewise.
template <class T>
__device__ __forceinline__ T* uni(T* q) {
  const unsigned long long u = (unsigned long long)q;
  return (T*)((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(u >> 32)) << 32 |
              (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)u));
}

template <class T>
using gptr = __attribute__((address_space(1))) T*;   // loads through it count against vmcnt only
template <class T>
__device__ __forceinline__ gptr<T> glob(T* q) { return (gptr<T>)q; }

// Exchange state of one workgroup.
struct RegX {
  gptr<double> xbuf;
  gptr<unsigned long long> bar;
  uint32_t epoch;                        // exchanges done, modulo 2^32 (some hours of them)
  int at;                                // epoch % 3: slot of the next exchange
  int nwg, wg, ng, grp, gsize, vmax;
  int zper;                              // words that this workgroup clears
  uint32_t spin_limit;
};

// Contribution to entry j of the current slot: a sum, or the maximum of non-negative values
// (whose bit patterns order like the values).
__device__ __forceinline__ gptr<double> team_slot(const RegX& X) { return X.xbuf + (size_t)(X.at * X.ng * X.vmax); }
__device__ __forceinline__ void team_add(const RegX& X, int j, double s) {
  if (s != 0.0)
    __hip_atomic_fetch_add(team_slot(X) + X.grp * X.vmax + j, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void team_max(const RegX& X, int j, double s) {
  if (s > 0.0)
    __hip_atomic_fetch_max((gptr<unsigned long long>)(team_slot(X) + X.grp * X.vmax + j),
                           (unsigned long long)__double_as_longlong(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The barrier's counters run on from exchange to exchange: their low words are compared, modulo
// 2^32 like the epoch (64 bits of it take registers from the rows: 256 instances 174 -> 197 ms).
// arrivals: of `members` after the exchange `epoch`; reached: whether `have` is `want` or past it.
__host__ __device__ __forceinline__ uint32_t arrivals(uint32_t epoch, int members) { return (epoch + 1) * (uint32_t)members; }
__host__ __device__ __forceinline__ bool reached(uint32_t have, uint32_t want) { return (int32_t)(have - want) >= 0; }

__device__ __forceinline__ uint32_t arrive(gptr<unsigned long long> counter) {
  return (uint32_t)__hip_atomic_fetch_add(counter, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
}

// Arrival and wait of the whole workgroup (ok: an LDS word); false when the bounded wait expired.
__device__ __forceinline__ bool team_barrier(const RegX& X, int tid, int* ok_lds, uint32_t spin_limit) {
  __builtin_amdgcn_s_waitcnt(0);   // this wave's atomics and clears are complete
  __syncthreads();
  if (tid == 0) {
    uint32_t target;
    gptr<unsigned long long> poll = X.bar;
    if (X.ng > 1) {
      target = X.epoch + 1;
      if (arrive(X.bar + XGSTRIDE * (1 + X.grp)) == arrivals(X.epoch, X.gsize)) {
        if (arrive(X.bar) == arrivals(X.epoch, X.ng))
          for (int g = 0; g < X.ng; ++g)
            __hip_atomic_store(X.bar + XGSTRIDE * (1 + XG_MAX + g), (unsigned long long)target, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
      }
      poll = X.bar + XGSTRIDE * (1 + XG_MAX + X.grp);
    } else {
      target = arrivals(X.epoch, X.nwg);
      arrive(X.bar);
    }
    uint32_t spins = 0;
    int ok = 1;
    while (!reached((uint32_t)__hip_atomic_load(poll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), target)) {
      if (++spins > 64) __builtin_amdgcn_s_sleep(1);
      if (spins >= spin_limit) { ok = 0; break; }
    }
    *ok_lds = ok;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*ok_lds) != 0;
}

// Total of entry j over the team (mx: its maximum).
__device__ __forceinline__ double team_total(const RegX& X, int j, bool mx) {
  gptr<double> cur = team_slot(X) + j;
  if (X.ng == 1) return __hip_atomic_load(cur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  double u[XG_MAX];   // the copies combine in a fixed order, every load issued before the first use
#pragma unroll
  for (int g = 0; g < XG_MAX; ++g)
    u[g] = g < X.ng ? __hip_atomic_load(cur + g * X.vmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
  double t = u[0];
#pragma unroll
  for (int g = 1; g < XG_MAX; ++g) t = mx ? fmax(t, u[g]) : t + u[g];
  return t;
}

// Frees the slot: clears the one used two exchanges from now (its last readers passed this
// exchange's barrier) with `nt` threads.
__device__ __forceinline__ void team_end(RegX& X, int tid, int nt) {
  gptr<double> z = X.xbuf + (size_t)((X.at == 0 ? 2 : X.at - 1) * X.ng * X.vmax);
  const int zl = X.ng * X.vmax;
  for (int j = X.wg * X.zper + tid; j < min(zl, (X.wg + 1) * X.zper); j += nt)
    __hip_atomic_store(z + j, 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  X.epoch++;
  X.at = X.at == 2 ? 0 : X.at + 1;
}

__device__ __forceinline__ RegX team_init(const DevState& s, const DevControl& ctl, int wg) {
  RegX X;
  X.xbuf = glob(s.xbuf); X.bar = glob(s.bar); X.epoch = 0; X.at = 0; X.nwg = ctl.nwg; X.wg = wg;
  X.ng = max(1, min(ctl.xgroups, min(XG_MAX, ctl.nwg)));
  X.grp = wg % X.ng;
  X.gsize = (X.nwg - X.grp + X.ng - 1) / X.ng;
  X.vmax = ctl.vmax;
  X.zper = (X.ng * X.vmax + X.nwg - 1) / X.nwg;
  X.spin_limit = ctl.spin_limit;
  return X;
}

// 1 / x and sqrt(x) by Newton's and Goldschmidt's iterations on the hardware's estimates (x normal and positive;
// within 1 ulp, without the scaling of subnormal and huge operands that the library's have).
__device__ __forceinline__ double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double root(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double e = fma(-g, h, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  e = fma(-g, h, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  return fma(fma(-g, g, x), h, g);
}

// The same pointer, opaque to the compiler: loads through it stay where they are written
// (hoisted out of the iteration, the fields that only a check needs would take registers
// from the rows).
template <class T>
__device__ __forceinline__ const T* opaque(const T* q) {
  asm volatile("" : "+s"(q));
  return q;
}

// Conjugate of the trade cost at e (conj_cost of cost_math.h for d = 3/2 and d = 2).
__device__ __forceinline__ double conj15(double e, double a, double b, double d) {
  const double r = fabs(e) - a;
  if (r <= 0.0) return 0.0;
  if (b <= 0.0) return INFINITY;
  const double t = r / (b * d);
  return d == 2.0 ? 0.5 * r * t : r * t * t / 3.0;
}

// prox of t'(a|x| + b|x|^d) at z (prox_cost of cost_math.h) for d = 3/2 and d = 2, with the step times a and b given.
// (c is capped where its square would overflow, and the result is below 1e-300 r^2 anyway)
__device__ __forceinline__ double prox15(double z, double ta, double tb, double d) {
  const double r = fmax(fabs(z) - ta, 0.0);
  double t;
  if (d == 2.0) {
    t = r / (1.0 + 2.0 * tb);
  } else {
    const double c = fmin(1.5 * tb, 1e150), u = 2.0 * r * recip(c + root(fmax(fma(c, c, 4.0 * r), 1e-280)));
    t = u * u;
  }
  return r <= 0.0 ? 0.0 : (z > 0.0 ? t : -t);
}

// Next prediction of a multiplier: centre at its trend, half-width w * mu.
__device__ __forceinline__ void predict(double mu, double mprev, double w, double& cen, double& hw) {
  if (mu <= 0.0) { cen = 0.0; hw = 0.0; return; }
  cen = uni(fmax(mu + (mu - mprev), 0.5 * mu));
  hw = uni(w * mu);
}

}  // namespace ffo
