// Risk-model construction of paper Section 3.2 on the device: from a window of daily
// factor returns Fr [days][p] and asset returns R [days][n] (with an optional observation
// mask), per-asset least-squares loadings beta_i (r_i ~ Fr beta_i over the asset's
// observed days, no intercept, only for assets with at least min_obs observations), the
// factor covariance Sigma_f (centred, 1/(days-1)) and the specific variances D_ii (the
// centred sample variance of the residuals over the observed days).
//
// Each asset has its own Gram matrix (the mask selects its days), so this is a batch of
// small normal-equation systems: per asset one pass over its returns accumulates the
// p(p+1)/2 Gram entries, the p cross products, the sum and sum of squares of its returns,
// its observation count and the p factor sums; a Cholesky factorisation solves the p x p
// system, and D follows from the sums (sum theta^2 = sum r^2 - 2 beta^T c + beta^T G beta).
//
// One launch: a workgroup takes 16 assets (a day's returns of them are one 128-byte
// segment) and all days, 16 threads an asset; their sums meet in LDS, where 16 threads
// solve the systems.  One more workgroup forms Sigma_f beside them.
//
// What bounds it: latency, of the loads (32 days a thread in eight steps, one step ahead) and of
// the solve's divisions (3.4 us).  504 days x 5000 assets, p = 6, masked: 18 us, against 49 in
// three launches with the partial sums of each 64 days in device memory; the call 71 -> 43 us.
// 512 threads a workgroup (one per compute unit) take 19 us, 128 threads 27; with the sums
// held to 128 registers they spill and it takes 39.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <cmath>
#include "internal.h"
#include "wave_ops.h"

namespace ffo {
namespace {

constexpr int RM_TILE = 16;                     // assets of a workgroup
constexpr int RM_CHUNK = 512;                   // days of factor returns in LDS at a time
constexpr int RM_U = 4;                         // days of a thread per step, and in flight
constexpr int RM_XCDS = 8;
// 512 threads a workgroup for windows of at least so many days, where one workgroup per compute unit
// holds the assets: the days in steps of 256 threads took 285 us against 206 at 32,000 days x 8 assets, p = 3,
// and 85 against 70 at 4000 x 8, p = 6; at 4000 x 20,000, where the chip is full, 254 against 294.
constexpr int RM_LONG = 2048, RM_FEW = 256;

template <int P>
struct RmDim {
  static constexpr int G = P * (P + 1) / 2;    // Gram entries (upper triangle, row-major)
  static constexpr int NV = G + P + 3 + P;     // + cross, sum r, sum r^2, count, factor sums
};

// NT: threads of a workgroup.
template <int NT>
struct RmShape {
  static constexpr int W = NT / 64, GROUPS = NT / RM_TILE;   // waves; threads per asset
  static_assert(RM_CHUNK % (RM_U * GROUPS) == 0, "a step stays in its chunk");
};

template <int P, int NT>
union RmLds {
  double fs[RM_CHUNK * P];                                       // factor returns of a chunk of days
  double red[(RmShape<NT>::W + 1) * RmDim<P>::NV * RM_TILE];     // the waves' sums, then the totals
};

// The p x p system and the residual variance of asset i from its sums in LDS, value v at
// s[v * RM_TILE] (read where they are used: copies would take the registers that the sums need).
template <int P>
__device__ __forceinline__ void solve_asset(const double* s, int min_obs, int i, double* __restrict__ beta,
                                            double* __restrict__ D, int32_t* __restrict__ valid) {
  constexpr int G = RmDim<P>::G;
  const auto at = [&](int v) { return s[v * RM_TILE]; };
  const auto tri = [](int r, int c) { return r * (r + 1) / 2 + c; };            // lower factor, row-major
  const auto gram = [](int a, int b) { return a * P - a * (a - 1) / 2 + b - a; };   // entry (a, b), a <= b
  const double cnt = at(G + P + 2);
  double b[P];
#pragma unroll
  for (int a = 0; a < P; ++a) b[a] = 0.0;
  bool ok = cnt >= (double)min_obs && cnt >= (double)(P + 1);
  if (ok) {
    // Cholesky of the Gram matrix, then two triangular solves
    double Lc[G];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      double dj = at(gram(j, j));
#pragma unroll
      for (int q = 0; q < j; ++q) dj -= Lc[tri(j, q)] * Lc[tri(j, q)];
      if (!(dj > 1e-300)) ok = false;
      const double rj = ok ? sqrt(dj) : 1.0;
      Lc[tri(j, j)] = rj;
#pragma unroll
      for (int r = j + 1; r < P; ++r) {
        double v = at(gram(j, r));
#pragma unroll
        for (int q = 0; q < j; ++q) v -= Lc[tri(r, q)] * Lc[tri(j, q)];
        Lc[tri(r, j)] = v / rj;
      }
    }
    if (ok) {
      double y[P];
#pragma unroll
      for (int a = 0; a < P; ++a) {
        double v = at(G + a);
#pragma unroll
        for (int q = 0; q < a; ++q) v -= Lc[tri(a, q)] * y[q];
        y[a] = v / Lc[tri(a, a)];
      }
#pragma unroll
      for (int a = P - 1; a >= 0; --a) {
        double v = y[a];
#pragma unroll
        for (int q = a + 1; q < P; ++q) v -= Lc[tri(q, a)] * b[q];
        b[a] = v / Lc[tri(a, a)];
      }
    }
  }
  // residual sums: theta = r - beta^T f over the observed days
  double st = at(G + P), st2 = at(G + P + 1);
  if (ok) {
    double bc = 0.0, bGb = 0.0, bf = 0.0;
#pragma unroll
    for (int a = 0; a < P; ++a) {
      bc = fma(b[a], at(G + a), bc);
      bf = fma(b[a], at(G + P + 3 + a), bf);
#pragma unroll
      for (int c = a; c < P; ++c) bGb += (a == c ? 1.0 : 2.0) * b[a] * b[c] * at(gram(a, c));
    }
    st -= bf;
    st2 = st2 - 2.0 * bc + bGb;
  }
  double d = 0.0;
  if (cnt >= 2.0) d = fmax((st2 - st * st / cnt) / (cnt - 1.0), 0.0);
#pragma unroll
  for (int a = 0; a < P; ++a) beta[(size_t)i * P + a] = b[a];
  D[i] = d;
  valid[i] = ok ? 1 : 0;
}

// Sigma_f = (Fr - mean)^T (Fr - mean) / (days - 1) by one workgroup, centred in a second pass
// over the days: in each, wave w sums the entries w, w + W, ... over the chunk in LDS.
template <int P, int NT>
__device__ __forceinline__ void factor_cov(int days, const double* __restrict__ Fr, double* __restrict__ Sf, double* fs,
                                           double* mu) {
  constexpr int W = RmShape<NT>::W, G = RmDim<P>::G, NE = ((G > P ? G : P) + W - 1) / W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int ea[NE], eb[NE];
  double s[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {   // entry (ea, eb) of the upper triangle, row-major
    int a = 0, r = min(wave + e * W, G - 1);
    while (r >= P - a) { r -= P - a; ++a; }
    ea[e] = a;
    eb[e] = a + r;
  }
  for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
    for (int e = 0; e < NE; ++e) s[e] = 0.0;
    for (int k0 = 0; k0 < days; k0 += RM_CHUNK) {
      const int nk = min(RM_CHUNK, days - k0);
      __syncthreads();
      for (int e = tid; e < nk * P; e += NT) fs[e] = Fr[(size_t)k0 * P + e];
      __syncthreads();
      for (int k = lane; k < nk; k += 64) {
        if (pass == 0) {   // (at least as many entries as means)
#pragma unroll
          for (int e = 0; e < NE; ++e) s[e] += fs[k * P + min(wave + e * W, P - 1)];
        } else {
#pragma unroll
          for (int e = 0; e < NE; ++e) s[e] = fma(fs[k * P + ea[e]] - mu[ea[e]], fs[k * P + eb[e]] - mu[eb[e]], s[e]);
        }
      }
    }
    if (pass == 0) {
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const double t = wave_sum(s[e]);
        if (lane == 0 && wave + e * W < P) mu[wave + e * W] = t / (double)days;
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const double v = wave_sum(s[e]) / (double)(days - 1);
    if (lane == 0 && wave + e * W < G) {
      Sf[ea[e] * P + eb[e]] = v;
      Sf[eb[e] * P + ea[e]] = v;
    }
  }
}

template <int P, bool MASKED, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_risk(
    int days, int n, int tiles, const double* __restrict__ R, const double* __restrict__ Fr,
    const uint8_t* __restrict__ mask, int min_obs, double* __restrict__ beta, double* __restrict__ Sf,
    double* __restrict__ D, int32_t* __restrict__ valid) {
  constexpr int NV = RmDim<P>::NV, G = RmDim<P>::G, W = RmShape<NT>::W, GROUPS = RmShape<NT>::GROUPS;
  __shared__ RmLds<P, NT> L;
  __shared__ double mu[P];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0) {   // (first, so that it is not the last one to start)
    factor_cov<P, NT>(days, Fr, Sf, L.fs, mu);
    return;
  }
  // neighbouring tiles on one XCD: a line of the mask holds eight tiles' days
  const int per = (tiles + RM_XCDS - 1) / RM_XCDS, bx = blockIdx.x - 1;
  const int tile = (bx % RM_XCDS) * per + bx / RM_XCDS;
  if (tile >= tiles) return;
  const int a = tid & (RM_TILE - 1), grp = tid / RM_TILE, i = tile * RM_TILE + a;
  const bool col = i < n;
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  const double* Rc = R + min(i, n - 1);
  const uint8_t* Mc = mask + (MASKED ? min(i, n - 1) : 0);
  // every load unconditional (the last day and asset again past the end): a compare in
  // between would wait for the load before the next one is issued
  double rv[RM_U], rn[RM_U];
  uint8_t mv[RM_U], mn[RM_U];
  const auto load = [&](double (&r)[RM_U], uint8_t (&m)[RM_U], int k) {
#pragma unroll
    for (int u = 0; u < RM_U; ++u) {
      const size_t at = (size_t)min(k + u * GROUPS, days - 1) * n;
      r[u] = Rc[at];
      m[u] = MASKED ? Mc[at] : (uint8_t)1;
    }
  };
  load(rv, mv, grp);
  for (int k0 = 0; k0 < days; k0 += RM_U * GROUPS) {
    if (k0 % RM_CHUNK == 0) {
      __syncthreads();
      for (int e = tid; e < min(RM_CHUNK, days - k0) * P; e += NT) L.fs[e] = Fr[(size_t)k0 * P + e];
      __syncthreads();
    }
    load(rn, mn, k0 + RM_U * GROUPS + grp);
#pragma unroll
    for (int u = 0; u < RM_U; ++u) {
      const int k = k0 + u * GROUPS + grp;
      const bool ob = col && k < days && mv[u] != 0;
      const double* fs = L.fs + min(k, days - 1) % RM_CHUNK * P;
      double f[P];   // zero on a day that does not count, so that its terms are zero
#pragma unroll
      for (int b = 0; b < P; ++b) f[b] = fs[b];
#pragma unroll
      for (int b = 0; b < P; ++b) f[b] = ob ? f[b] : 0.0;
      const double r = ob ? rv[u] : 0.0;
      int g = 0;
#pragma unroll
      for (int b = 0; b < P; ++b)
#pragma unroll
        for (int c = b; c < P; ++c) { acc[g] = fma(f[b], f[c], acc[g]); ++g; }
#pragma unroll
      for (int b = 0; b < P; ++b) acc[G + b] = fma(f[b], r, acc[G + b]);
      acc[G + P] += r;
      acc[G + P + 1] = fma(r, r, acc[G + P + 1]);
      acc[G + P + 2] += ob ? 1.0 : 0.0;
#pragma unroll
      for (int b = 0; b < P; ++b) acc[G + P + 3 + b] += f[b];
    }
#pragma unroll
    for (int u = 0; u < RM_U; ++u) { rv[u] = rn[u]; mv[u] = mn[u]; }
  }
  // an asset's sums: its four lanes of a wave, then the waves in order
  __syncthreads();
#pragma unroll
  for (int v = 0; v < NV; v += 4) {
    const double t0 = pair_sum32(acc[v], v + 1 < NV ? acc[v + 1] : 0.0);
    const double t1 = v + 2 < NV ? pair_sum32(acc[v + 2], v + 3 < NV ? acc[v + 3] : 0.0) : 0.0;
    const double t = pair_sum16(t0, t1);
    const int ag = lane >> 4, vv = v + 2 * (ag & 1) + (ag >> 1);
    if (vv < NV) L.red[(wave * NV + vv) * RM_TILE + a] = t;
  }
  __syncthreads();
  for (int e = tid; e < NV * RM_TILE; e += NT) {
    double t = L.red[e];
#pragma unroll
    for (int w = 1; w < W; ++w) t += L.red[w * NV * RM_TILE + e];
    L.red[W * NV * RM_TILE + e] = t;
  }
  __syncthreads();
  if (tid < RM_TILE && col) solve_asset<P>(L.red + W * NV * RM_TILE + tid, min_obs, i, beta, D, valid);
}

template <int P, int NT>
int launch_nt(int days, int n, const double* R, const double* Fr, const uint8_t* mask, int min_obs, double* beta,
              double* Sf, double* D, int32_t* valid, hipStream_t st) {
  const int tiles = (n + RM_TILE - 1) / RM_TILE, grid = 1 + (tiles + RM_XCDS - 1) / RM_XCDS * RM_XCDS;
  if (mask)
    hipLaunchKernelGGL((k_risk<P, true, NT>), dim3(grid), dim3(NT), 0, st, days, n, tiles, R, Fr, mask, min_obs, beta, Sf, D, valid);
  else
    hipLaunchKernelGGL((k_risk<P, false, NT>), dim3(grid), dim3(NT), 0, st, days, n, tiles, R, Fr, mask, min_obs, beta, Sf, D, valid);
  return (int)hipGetLastError();
}

template <int P>
int launch_rm(int days, int n, const double* R, const double* Fr, const uint8_t* mask, int min_obs, double* beta,
              double* Sf, double* D, int32_t* valid, hipStream_t st) {
  return days < RM_LONG || n > RM_FEW * RM_TILE
             ? launch_nt<P, 256>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st)
             : launch_nt<P, 512>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
}

}  // namespace

int launch_risk_model(int days, int n, int p, const double* R, const double* Fr, const uint8_t* mask, int min_obs,
                      double* beta, double* Sf, double* D, int32_t* valid, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  switch (p) {
    case 1: return launch_rm<1>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 2: return launch_rm<2>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 3: return launch_rm<3>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 4: return launch_rm<4>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 5: return launch_rm<5>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 6: return launch_rm<6>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 7: return launch_rm<7>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    case 8: return launch_rm<8>(days, n, R, Fr, mask, min_obs, beta, Sf, D, valid, st);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace ffo
