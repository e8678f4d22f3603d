// Single-period solve with the constraint rows in registers (impact exponent 3/2 or 2).
//
// Same iteration as solve_kernel.hip (restarted, reflected Halpern PDHG with the exact
// budget multiplier), laid out for one period: a team of workgroups of eight waves, two
// waves per SIMD and up to 256 registers per lane.  Wave w of a workgroup owns 4 CA
// assets; lane (ag, rg) = (lane / 16, lane % 16) holds the block of scaled rows
// rg + 16 q (q < RA) times the assets ag CA + c (c < CA), RA x CA doubles, for the whole
// solve.  Both products read that block:
//   K~^T y:  each lane sums its rows per asset, then the 16 lanes of a DPP row combine
//            (halving the number of sums per step), which leaves asset ag CA + rg % CA
//            in lane (ag, rg): the lane that owns the asset's iterates.
//   K~ x:    lane c of each row broadcasts its x to the row (one DPP move), each lane
//            sums its assets per row, and the four rows of lanes combine through lane
//            swaps; the eight waves' sums meet in LDS.
// Iterates and step constants stay in registers, restart anchors and asset data in LDS;
// rows [0, 16 RA) belong to the first 16 RA threads.  Control scalars are computed by
// every thread from the same totals, so no thread waits for a broadcast of a decision.
//
// In the FP32 form (ctl.prec) the values are the general kernel's: rows rounded to float,
// iterates float offsets from the restart anchor, FP64 everywhere else, and exact rows again
// for a check, whose block every lane reloads.  The arithmetic is the FP64 form's: half the
// width would save none of the chains that bound an iteration.  FP32 solves on the general
// kernel and here: n = 473, 95 rows 22.4 and 9.1 ms, n = 1777, 41 rows 39.6 and 17.1, n = 4935,
// 70 rows 55.7 and 28.7; four markets of 419 assets, 73 rows, 52.5 and 13.3.
//
// What bounds it: latency.  At n = 5000, 140 rows (20 workgroups of 250 assets) an iteration
// takes 6.9 us (14.7 in the general kernel): about 2 for the exchange between the
// workgroups, 0.7 of issue for the products (72 + 144 FMA per lane, two waves per SIMD),
// the rest dependent chains (sums across lanes, the decision, the two proximal maps).  Few,
// full workgroups keep the exchange short: between 8 and 16 workgroups of 1024 threads one
// measured 1.6-2.0 us, among 32 2.8 us and among 250 12 us.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include "internal.h"
#include "team_exchange.h"
#include "wave_ops.h"

namespace ffo {
namespace {

constexpr int NT = 512, NWV = NT / 64;   // threads and waves of a workgroup
constexpr int NC = 8;                    // bracket candidates
constexpr int NST = 2 + 3 * NC;          // statistics: [S(0), max |b|, (S, A0, count)(c_q)]
constexpr int MSC = 32, MS_ROUNDS = 40;  // multisection candidates per round, rounds at most
constexpr int OR = 32;                   // first row entry of an exchange (statistics before it)
constexpr int NSC = 12;                  // scalar sums of a check

template <int RA, int CA>
struct RegLds {
  static constexpr int NRP = 16 * RA;                                   // padded rows
  static constexpr int PV = OR + 2 * NRP < 96 ? 96 : OR + 2 * NRP;      // values of an exchange at most
  double y[NRP], y0r[NRP], ty[NRP], dv[NRP];   // row duals, anchor, image, check displacement
  double dr[NRP], lo[NRP], up[NRP], bF[NRP];   // row scales, exposure bounds, factor offsets
  double sd[NRP], rs[NRP];               // sigma dr, and 1 / (sigma dr) or the factor rows' shrinkage
  double part[NWV][PV], tot[PV];         // per-wave partial sums, exchanged totals
  double ab[NWV][4 * CA], ia[NWV][4 * CA];   // |b| and 1/a of each wave's assets
  double x0[NT], y0[NT], al[NT], ar[NT], w0[NT], ca[NT], cb[NT];   // per thread: anchors, asset data
  double sc[NSC][NT];                    // a check's per-thread terms
  double c1[NSC], red[NWV][4];           // a check's sums
  int ok, restarts, checks, miss, miss_in, miss_out, rounds;
  long long t_start;                     // thread 0's, many instances: the clock that the time limit counts from
};

// Sum over the waves of partial sum j (mx: the maximum for j = 1), in wave order.
template <int RA, int CA>
__device__ __forceinline__ double wave_parts(const RegLds<RA, CA>& L, int j, bool mx) {
  double u[NWV];
#pragma unroll
  for (int w = 0; w < NWV; ++w) u[w] = L.part[w][j];
  const bool m = mx && j == 1;
  double s = u[0];
#pragma unroll
  for (int w = 1; w < NWV; ++w) s = m ? fmax(s, u[w]) : s + u[w];
  return s;
}

// Publishes the workgroup's partial sums part[.][0, V) and waits for the other workgroups.
// On return total(X, L, j) is the sum over all waves and workgroups (mx: the maximum for
// j = 1); exchange_end then frees the slot.  A single workgroup only synchronises: part
// holds everything, and must not be written again before the next barrier.
template <int RA, int CA>
__device__ __forceinline__ bool exchange_begin(RegX& X, RegLds<RA, CA>& L, int tid, int V, bool mx,
                                               uint32_t spin_limit) {
  __syncthreads();   // every wave's partial sums are in part
  if (X.nwg == 1) return true;
  if (tid < V) {
    const double s = wave_parts(L, tid, mx);
    if (mx && tid == 1) team_max(X, tid, s);
    else team_add(X, tid, s);
  }
  return team_barrier(X, tid, &L.ok, spin_limit);
}

template <int RA, int CA>
__device__ __forceinline__ double total(const RegX& X, const RegLds<RA, CA>& L, int j, bool mx) {
  return X.nwg == 1 ? wave_parts(L, j, mx) : team_total(X, j, mx && j == 1);
}

__device__ __forceinline__ void exchange_end(RegX& X, int tid) {
  if (X.nwg > 1) team_end(X, tid, NT);
}

// The whole exchange, totals to LDS.
template <int RA, int CA>
__device__ __forceinline__ bool exchange(RegX& X, RegLds<RA, CA>& L, int tid, int V, bool mx, uint32_t spin_limit) {
  if (!exchange_begin(X, L, tid, V, mx, spin_limit)) return false;
  if (tid < V) L.tot[tid] = total(X, L, tid, mx);
  exchange_end(X, tid);
  __syncthreads();
  return true;
}

// K~^T y for the lane's owned asset; y in LDS [16 RA].
template <int RA, int CA>
__device__ __forceinline__ double kty(const double (&K)[RA][CA], const double* y, int tid) {
  const int rg = tid & 15;
  double v[CA];
#pragma unroll
  for (int c = 0; c < CA; ++c) v[c] = 0.0;
#pragma unroll
  for (int q = 0; q < RA; ++q) {
    const double yq = y[rg + 16 * q];
#pragma unroll
    for (int c = 0; c < CA; ++c) v[c] = fma(K[q][c], yq, v[c]);
  }
  // each step sends half of the sums to the partner lane and adds the half it keeps
  const auto halve = [&](auto ctrl, auto h, int bit) {
    constexpr int H = decltype(h)::value;
    const bool up = (rg & bit) != 0;
#pragma unroll
    for (int c = 0; c < H; ++c) {
      const double keep = up ? v[c + H] : v[c], send = up ? v[c] : v[c + H];
      v[c] = keep + dpp<decltype(ctrl)::value>(send);
    }
  };
  using std::integral_constant;
  if constexpr (CA == 16) halve(integral_constant<int, DPP_MIRROR>{}, integral_constant<int, 8>{}, 8);
  if constexpr (CA >= 8) halve(integral_constant<int, DPP_HALF_MIRROR>{}, integral_constant<int, 4>{}, 4);
  halve(integral_constant<int, DPP_SWAP2>{}, integral_constant<int, 2>{}, 2);
  halve(integral_constant<int, DPP_SWAP1>{}, integral_constant<int, 1>{}, 1);
  double r = v[0];
  if constexpr (CA == 4) r += dpp<DPP_ROR4>(r);
  if constexpr (CA <= 8) r += dpp<DPP_ROR8>(r);
  return r;
}

// K~ x1 (and K~ x2) of the wave's assets into out[r] (and out[NRP + r]), r < 16 RA; x1,
// x2: the owned asset's values (zero where the lane's asset does not exist).
template <int RA, int CA>
__device__ __forceinline__ void rows2(const double (&K)[RA][CA], double x1, double x2, double* out, int tid) {
  double a1[RA], a2[RA];
#pragma unroll
  for (int q = 0; q < RA; ++q) { a1[q] = 0.0; a2[q] = 0.0; }
  static_for<CA>([&](auto c) {
    constexpr int C = decltype(c)::value;
    const double v1 = dpp<DPP_BCAST + C>(x1), v2 = dpp<DPP_BCAST + C>(x2);
#pragma unroll
    for (int q = 0; q < RA; ++q) {
      a1[q] = fma(K[q][C], v1, a1[q]);
      a2[q] = fma(K[q][C], v2, a2[q]);
    }
  });
  const int rg = tid & 15, ag = (tid >> 4) & 3;
#pragma unroll
  for (int q = 0; q < RA; ++q) a1[q] = pair_sum32(a1[q], a2[q]);   // low half-wave: x1, high: x2
#pragma unroll
  for (int q = 0; q < RA; q += 2) {
    const double t = pair_sum16(a1[q], q + 1 < RA ? a1[q + 1] : 0.0);
    const int qq = q + (ag & 1);
    if (qq < RA) out[(ag >> 1) * 16 * RA + rg + 16 * qq] = t;
  }
}

template <int RA, int CA>
__device__ __forceinline__ void rows1(const double (&K)[RA][CA], double x1, double* out, int tid) {
  double a[RA];
#pragma unroll
  for (int q = 0; q < RA; ++q) a[q] = 0.0;
  static_for<CA>([&](auto c) {
    constexpr int C = decltype(c)::value;
    const double v1 = dpp<DPP_BCAST + C>(x1);
#pragma unroll
    for (int q = 0; q < RA; ++q) a[q] = fma(K[q][C], v1, a[q]);
  });
  const int rg = tid & 15, ag = (tid >> 4) & 3;
#pragma unroll
  for (int q = 0; q < RA; q += 4) {
    const double t0 = pair_sum32(a[q], q + 1 < RA ? a[q + 1] : 0.0);
    const double t1 = q + 2 < RA ? pair_sum32(a[q + 2], q + 3 < RA ? a[q + 3] : 0.0) : 0.0;
    const double t = pair_sum16(t0, t1);
    const int qq = q + 2 * (ag & 1) + (ag >> 1);
    if (qq < RA) out[rg + 16 * qq] = t;
  }
}

// Statistics of S(mu) = sum max(|b| - mu, 0)/a over the wave's assets at the bracket
// candidates (eight lanes per candidate), into out[0, NST).
template <int W>
__device__ __forceinline__ void stats(const double* ab, const double* ia, double cen, double hw, double* out, int tid) {
  const int lane = tid & 63, g = lane >> 3, sub = lane & 7;
  const double cq = cand(cen, hw, g);
  double S = 0.0, A0 = 0.0, N = 0.0, S0 = 0.0, mx = 0.0;
#pragma unroll
  for (int li = 0; li < W; li += 8) {
    const double a = ab[li + sub], r = ia[li + sub];
    S0 = fma(a, r, S0);
    mx = fmax(mx, a);
    if (a > cq) { S = fma(a - cq, r, S); A0 += r; N += 1.0; }
  }
  S = sum8(S); A0 = sum8(A0); N = sum8(N); S0 = sum8(S0); mx = max8(mx);
  if (sub == 0) { out[2 + 3 * g] = S; out[3 + 3 * g] = A0; out[4 + 3 * g] = N; }
  if (lane == 0) { out[0] = S0; out[1] = mx; }
}

// The bracket decision of solve_kernel.hip (bracket_decide) from statistic `lane` in each
// lane; uniform result (1 = exact from the central pair, 4 = exact from another interval
// without breakpoints, 2 = zero, 0 / 3 = multisection on [lo, hi]).
__device__ __forceinline__ int decide(double st, double cen, double hw, double& lo, double& hi, double& mu,
                                      int tid) {
  const double S0 = lane_of(st, 0), maxb = lane_of(st, 1);
  if (__builtin_amdgcn_readfirstlane(S0 <= 1.0)) {
    mu = 0.0;
    return __builtin_amdgcn_readfirstlane(cen + hw <= 0.0 ? 1 : 2);
  }
  constexpr unsigned long long sel = 0x924924ull;   // lanes 2 + 3 q
  const unsigned long long ge = __ballot(st >= 1.0) & sel;
  int qs = ge ? (61 - __clzll((long long)ge)) / 3 : -1;   // S is non-increasing: {q : S(c_q) >= 1} = [0, qs]
  double a, b;
  if (qs < 0) { a = 0.0; b = cand(cen, hw, 0); }
  else if (qs == NC - 1) { a = cand(cen, hw, NC - 1); b = maxb; }
  else { a = cand(cen, hw, qs); b = cand(cen, hw, qs + 1); }
  if (qs >= 0 && qs < NC - 1) {
    const double S = lane_of(st, 2 + 3 * qs), A0 = lane_of(st, 3 + 3 * qs);
    if (__builtin_amdgcn_readfirstlane(lane_of(st, 4 + 3 * qs) == lane_of(st, 7 + 3 * qs) && A0 > 0.0)) {
      mu = uni(fmin(fmax(fma(S - 1.0, recip(A0), a), a), b));
      return qs == 3 ? 1 : 4;
    }
  }
  if (!(b >= a)) { a = 0.0; b = maxb; qs = -1; }
  lo = uni(a);
  hi = uni(b);
  return qs == 3 ? 0 : 3;
}

// Multisection on [lo, hi] (S(lo) >= 1 >= S(hi)) over L.ab / L.ia: MSC candidates per
// round, two lanes per candidate.  Returns false when a bounded wait expired.
template <int RA, int CA>
__device__ __forceinline__ bool multisect(RegX& X, RegLds<RA, CA>& L, double lo, double hi, double& mu, int tid) {
  const int lane = tid & 63, wave = wave_of(tid), q = lane >> 1, sub = lane & 1;
  for (int round = 0; round < MS_ROUNDS; ++round) {
    if (tid == 0) ++L.rounds;
    const double cq = lo + (hi - lo) * (double)q / (double)(MSC - 1);
    double S = 0.0, A0 = 0.0, N = 0.0;
    for (int li = sub; li < 4 * CA; li += 2) {
      const double a = L.ab[wave][li], r = L.ia[wave][li];
      if (a > cq) { S = fma(a - cq, r, S); A0 += r; N += 1.0; }
    }
    S += dpp<DPP_SWAP1>(S); A0 += dpp<DPP_SWAP1>(A0); N += dpp<DPP_SWAP1>(N);
    if (sub == 0) { L.part[wave][3 * q] = S; L.part[wave][3 * q + 1] = A0; L.part[wave][3 * q + 2] = N; }
    if (!exchange(X, L, tid, 3 * MSC, false, X.spin_limit)) return false;
    const double* T0 = L.tot;
    const unsigned long long ge = __ballot(lane < MSC && T0[3 * (lane < MSC ? lane : 0)] >= 1.0);
    const int qs = ge ? 63 - __clzll((long long)ge) : 0;
    if (qs == MSC - 1) { mu = hi; return true; }   // (qs and the tests below are uniform)
    const double c0 = lo + (hi - lo) * (double)qs / (double)(MSC - 1);
    const double c1 = lo + (hi - lo) * (double)(qs + 1) / (double)(MSC - 1);
    const double Sq = T0[3 * qs], Aq = T0[3 * qs + 1];
    const bool linear = T0[3 * qs + 2] == T0[3 * qs + 5];
    const bool tiny = (c1 - c0) <= 4.0 * 2.220446049250313e-16 * fabs(c1);
    if (__builtin_amdgcn_readfirstlane(linear || tiny || round == MS_ROUNDS - 1)) {
      const double m = Aq > 0.0 ? c0 + (Sq - 1.0) / Aq : c0;
      mu = uni(fmin(fmax(m, c0), c1));
      return true;
    }
    lo = uni(c0);
    hi = uni(c1);
  }
  return true;
}

// Sum of each thread's NV values over the workgroup (fixed order), for every thread.
template <int NV, int RA, int CA>
__device__ __forceinline__ void wg_total(RegLds<RA, CA>& L, double (&v)[NV], int tid) {
  static_assert(NV <= 4, "reduction scratch");
  const int lane = tid & 63, wave = wave_of(tid);
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const double t = wave_sum(v[q]);
    if (lane == 0) L.red[wave][q] = t;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double t = L.red[0][q];
#pragma unroll
    for (int w = 1; w < NWV; ++w) t += L.red[w][q];
    v[q] = t;
  }
  __syncthreads();
}

// A thread's place: its wave and lane, the row of lanes' asset `slot` among the wave's and
// `li` among the workgroup's, whether that asset exists (val) and this lane is its owner
// (mine: the other lanes of the row replicate it), and whether the thread owns a row (rown).
struct Place {
  int tid, lane, wave, rg, slot, li;
  bool val, mine, rown;
};
template <int CA>
__device__ __forceinline__ Place place(int tid0, int nwa, int nr) {
  Place t;
  t.tid = fresh(tid0);
  t.lane = t.tid & 63;
  t.wave = wave_of(t.tid);
  t.rg = t.tid & 15;
  t.slot = ((t.tid >> 4) & 3) * CA + (t.tid & (CA - 1));
  t.li = t.wave * 4 * CA + t.slot;
  t.val = t.li < nwa;
  t.mine = t.val && t.rg < CA;
  t.rown = t.tid < nr;
  return t;
}

template <int RA, int CA, bool QUEUE>
__device__ __forceinline__ void reg_body(const DevProblem* pp, const DevState* sp, const DevControl* cp, int wg,
                                         RegLds<RA, CA>& L, uint32_t first_spins) {
  const DevProblem& p = *pp;
  const DevState& s = *sp;
  const DevControl& ctl = *cp;
  constexpr int NRP = 16 * RA, WA = 4 * CA, OS = OR + NRP;   // OS: scalar sums of a check
  static_assert(NSC <= NRP, "scalar sums fit behind the rows");
  const int tid0 = threadIdx.x;
  const int n = p.n, nr = p.nr, m = p.m, nwg = ctl.nwg;
  const int i0 = wg * ctl.nw, nwa = max(0, min(ctl.nw, n - i0));
  const double rho = ctl.rho, d = p.d, g1 = p.g1;
  const bool f32 = ctl.prec == PREC_FP32, rc32 = f32 && ctl.rc32;
  const auto rc = [rc32](double v) { return rc32 ? (double)(float)v : v; };
  const auto stored = [f32](double v, double z0) { return f32 ? z0 + (double)(float)(v - z0) : v; };   // an iterate

  RegX X = team_init(s, ctl, wg);
  if constexpr (QUEUE) {
    // (loaded per ticket these are vectors, and the first to be spilled: each reload is a trip to
    // memory between an exchange's barrier and its totals.  2048 iterations of 64 instances with 140
    // rows 52.7 and 46.2 ms; in a single solve, n = 5000, as scalars 29.3 ms against 28.7)
    X.xbuf = glob(uni(s.xbuf));
    X.bar = glob(uni(s.bar));
  }

  double K[RA][CA];
  double x, yc, tx, ty, dc;   // the owned asset: iterates, their images, column scale
  {
    const auto [tid, lane, wave, rg, slot, li, val, mine, rown] = place<CA>(tid0, nwa, nr);
    const int ag = (tid >> 4) & 3, i = i0 + li;
#pragma unroll
    for (int q = 0; q < RA; ++q) {
      const int r = rg + 16 * q;
      const double sc = r < nr ? (p.kscaled ? 1.0 : p.dr[r]) : 0.0;
#pragma unroll
      for (int c = 0; c < CA; ++c) {
        const int l = wave * WA + ag * CA + c;
        const double k = r < nr && l < nwa ? p.K[(size_t)r * p.ldk + i0 + l] : 0.0;
        K[q][c] = (f32 ? (double)(float)k : k) * sc;
      }
    }
    for (int e = tid; e < NWV * L.PV; e += NT) (&L.part[0][0])[e] = 0.0;
    // asset data; trade rows are unscaled for one period (drC = 1)
    dc = val ? p.dc[i] : 1.0;
    L.al[tid] = val ? p.alpha[i] : 0.0;
    L.ar[tid] = val ? p.arisk[i] : 1.0;
    L.w0[tid] = val ? p.w0[i] : 0.0;
    L.ca[tid] = val ? p.ca[i] : 0.0;
    L.cb[tid] = val ? p.cb[i] : 0.0;
    // starting point: w0 (paper Section 4.1) or the caller's; duals zero or the caller's
    x = val ? (s.w_init ? s.w_init[i] : L.w0[tid]) / dc : 0.0;
    yc = val && s.y_init ? s.y_init[nr + i] : 0.0;
    tx = x;
    ty = yc;
    L.x0[tid] = x;
    L.y0[tid] = yc;
    if (tid < NRP) {
      const double dr = rown ? p.dr[tid] : 1.0, yr = rown && s.y_init ? s.y_init[tid] / dr : 0.0;
      L.dr[tid] = dr;
      L.lo[tid] = rown && tid < m ? p.L[tid] : 0.0;
      L.up[tid] = rown && tid < m ? p.U[tid] : 0.0;
      L.bF[tid] = rown && tid >= m ? p.bF[tid - m] : 0.0;
      L.y[tid] = L.y0r[tid] = L.ty[tid] = yr;
      L.dv[tid] = 0.0;
    }
    if (tid == 0) L.restarts = L.checks = L.miss = L.miss_in = L.miss_out = L.rounds = 0;
    __syncthreads();
  }

  long long t_start = wall_clock64();
  long long t_check = 0;
  double omega = ctl.omega0 > 0.0 ? ctl.omega0 : 1.0, r0 = -1.0, rprev = INFINITY;
  long long it = 0;
  uint32_t kk = 0;   // since the last restart (from 2^30 on the Halpern weights no longer matter)
  int left = (int)min((long long)ctl.check_every, (long long)ctl.max_iter);   // iterations to the next check
  int status = DS_RUNNING;

  // ---- power iteration: lambda ~ ||K~ v||^2 / ||v||^2, v <- K~^T K~ v / (lambda ||v||)
  double lam = 0.0;
  {
    double v;
    {
      const Place t = place<CA>(tid0, nwa, nr);
      v = t.val ? 1.0 + 0.25 * (double)(((i0 + t.li) * 7919) % 1000) / 1000.0 : 0.0;
    }
    for (int pw = 0; pw < ctl.npow; ++pw) {
      const auto [tid, lane, wave, rg, slot, li, val, mine, rown] = place<CA>(tid0, nwa, nr);
      const double a = wave_sum(mine ? v * v : 0.0), b = wave_sum(mine ? dc * v * dc * v : 0.0);
      if (lane == 0) { L.part[wave][0] = a; L.part[wave][1] = b; }
      rows1(K, v, L.part[wave] + OR, tid);
      if (!exchange(X, L, tid, OS, false, pw == 0 ? first_spins : X.spin_limit)) goto fail;
      if constexpr (QUEUE) {
        if (pw == 0 && tid == 0) L.t_start = s.clock0 ? *s.clock0 : wall_clock64();   // the call's start, or ...
      } else {
        if (pw == 0) t_start = wall_clock64();   // ... when the team is complete
      }
      double kv = 0.0;
      for (int r = lane; r < NRP; r += 64) kv = fma(L.tot[OR + r], L.tot[OR + r], kv);
      kv = wave_sum(kv) + L.tot[1];
      const double vv = L.tot[0];
      lam = uni(vv > 0.0 ? kv / vv : 0.0);
      const double scale = (lam > 0.0 && vv > 0.0) ? 1.0 / (lam * sqrt(vv)) : 1.0;
      const double Ru = kty(K, L.tot + OR, tid);   // (every lane: the sums cross lanes)
      v = val ? (Ru + dc * dc * v) * scale : 0.0;
    }
  }
  {
    const double eta = uni(ctl.eta_safety / sqrt(fmax(lam, 1e-300)));
    const long long t_loop = wall_clock64();
    double mu = 0.0, mprev = 0.0, cen = 0.0, hw = 0.0, wid = 1e-3;           // budget multiplier and its bracket
    double dmu = 0.0, dcen = 0.0, dhw = 0.0, dwid = 1e-3;                    // the same, dual inner problem

    while (true) {
      const double sigma = uni(eta * omega), isig = uni(1.0 / sigma);
      const double idc = 1.0 / dc, itd = omega / eta * idc;          // b = x / (tau dc) - R / dc + alpha
      const double ia = 1.0 / (itd * idc + rc(L.ar[tid0])), gia = ia * idc;
      if (tid0 < nr) {
        const double dr = L.dr[tid0], sd = sigma * dr;
        L.sd[tid0] = sd;
        L.rs[tid0] = tid0 < m ? 1.0 / sd : 2.0 * g1 / (sd * dr + 2.0 * g1);
      }
      bool restart = false;
      // ---- iterations with one primal weight
      while (!restart) {
        const auto [tid, lane, wave, rg, slot, li, val, mine, rown] = place<CA>(tid0, nwa, nr);
        const bool check = --left == 0;
        if (check) left = (int)min((long long)ctl.check_every, ctl.max_iter - (it + 1));
        // Halpern weights of this iteration (here, off the chain that follows the exchange)
        // (FP32: the quotients themselves, since the first steps from an anchor fall on ties of the
        // float offsets, which the last bit of a weight decides)
        const double k1 = (double)kk;
        double a0 = uni(recip(k1 + 2.0)), a1 = uni((k1 + 1.0) * a0);
        if (f32) { a0 = uni(1.0 / (k1 + 2.0)); a1 = uni((k1 + 1.0) / (k1 + 2.0)); }
        // prox input b and the statistics at the bracket candidates
        const double Ry = kty(K, L.y, tid) + dc * yc;
        const double b = x * itd - Ry * idc + rc(L.al[tid]), ab = fabs(b);
        if (rg < CA) { L.ab[wave][slot] = val ? ab : 0.0; L.ia[wave][slot] = val ? ia : 0.0; }
        __builtin_amdgcn_wave_barrier();
        stats<WA>(L.ab[wave], L.ia[wave], cen, hw, L.part[wave], tid);
        // affine pieces at the central pair's upper end: P1 = K~ (2 xhat(c4) - x), P2 = K~ d xhat / d mu
        const double c4 = cand(cen, hw, 4);
        {
          const double g = copysign(gia, b);
          const double x1 = 2.0 * (ab > c4 ? g * (ab - c4) : 0.0) - x, x2 = ab > c4 ? -g : 0.0;
          rows2(K, val ? x1 : 0.0, val ? x2 : 0.0, L.part[wave] + OR, tid);
        }
        if (!exchange_begin(X, L, tid, OR + 2 * NRP, true, X.spin_limit)) goto fail;
        const double st = total(X, L, lane < NST ? lane : 0, true);
        double kx = 0.0, p2 = 0.0;
        if (rown) {
          kx = total(X, L, OR + tid, false);
          p2 = total(X, L, OS + tid, false);
        }
        exchange_end(X, tid);
        double lo = 0.0, hi = 0.0, mnew = 0.0;
        const int r = decide(st, cen, hw, lo, hi, mnew, tid);
        wid = uni(adapt_width(r, wid));
        mprev = mu;
        if (r == 1) {
          mu = mnew;
          kx = fma(2.0 * (mu - c4), p2, kx);
        } else {
          __syncthreads();   // a single workgroup's totals are read from part, which is written next
          if (tid == 0) { ++L.miss; L.miss_in += r == 0; L.miss_out += r == 3; }
          if (r == 2 || r == 4) mu = mnew;
          else if (!multisect(X, L, lo, hi, mu, tid)) goto fail;
          const double xh = ab > mu ? copysign(gia, b) * (ab - mu) : 0.0;
          rows1(K, val ? 2.0 * xh - x : 0.0, L.part[wave] + OR, tid);
          if (!exchange_begin(X, L, tid, OS, false, X.spin_limit)) goto fail;
          if (rown) kx = total(X, L, OR + tid, false);
          exchange_end(X, tid);
        }
        predict(mu, mprev, wid, cen, hw);

        // T(z): primal point, trade duals, row duals
        {
          const double xh = ab > mu ? copysign(gia, b) * (ab - mu) : 0.0;
          const double w0 = L.w0[tid], vs = yc + sigma * (dc * (2.0 * xh - x));
          const double pr = prox15(vs * isig - w0, isig * rc(L.ca[tid]), isig * rc(L.cb[tid]), d);
          tx = stored(xh, L.x0[tid]);
          ty = stored(vs - sigma * w0 - sigma * pr, L.y0[tid]);
        }
        if (rown) {
          const double vs = fma(sigma, kx, L.y[tid]), sd = L.sd[tid], rs = L.rs[tid];
          double tyr;
          if (tid < m) {
            const double Lr = L.lo[tid], Ur = L.up[tid];
            tyr = fma(-sd, fmin(fmax(vs * rs, Lr), Ur), vs);
            // an infinite bound side forces the dual's sign exactly
            if (isinf(Ur) && tyr > 0.0) tyr = 0.0;
            if (isinf(Lr) && tyr < 0.0) tyr = 0.0;
          } else {
            tyr = rs * fma(-sd, L.bF[tid], vs);
          }
          L.ty[tid] = tyr;
        }

        if (check) {
          const long long tc0 = wall_clock64();
          const DevProblem& p = *opaque(pp);
          const DevState& s = *opaque(sp);
          const DevControl& ctl = *opaque(cp);
          const auto [tid, lane, wave, rg, slot, li, val, mine, rown] = place<CA>(tid0, nwa, nr);
          const int i = i0 + li;
          const double al = L.al[tid], ar = L.ar[tid];
          if (f32) {   // the check is of the unrounded problem
            const int ag = (tid >> 4) & 3;
#pragma unroll
            for (int q = 0; q < RA; ++q) {
              const int r = rg + 16 * q;
#pragma unroll
              for (int c = 0; c < CA; ++c) {
                const int l = wave * WA + ag * CA + c;
                K[q][c] = r < nr && l < nwa ? p.K[(size_t)r * p.ldk + i0 + l] : 0.0;
              }
            }
          }
          // terms of the sums, one by one through LDS: fixed-point residual, |dx|^2, |dy|^2,
          // Phi's linear and quadratic part, costs, their conjugates, y_C . w0, |y|^2, time-out,
          // non-finite count, dual-domain violation^2, budget
          {
            const double dx = x - tx, dl = tx - L.x0[tid], dy = yc - ty, dly = ty - L.y0[tid];
            double f = omega * dx * dx + dy / omega * dy, g = dly * dly, h = ty * ty;
            const double ca = L.ca[tid], cb = L.cb[tid], w0 = L.w0[tid], w = dc * tx, au = fabs(w - w0);
            double ex = fmax(fabs(ty) - ca, 0.0);
            ex = cb <= 0.0 ? ex * ex : 0.0;
            if (!mine) f = g = h = ex = 0.0;
            if (wg == 0 && rown) {   // replicated row duals enter the sums once
              const double tyr = L.ty[tid], dr2 = L.y[tid] - tyr, dlr = tyr - L.y0r[tid], yu = L.dr[tid] * tyr;
              f = fma(dr2 / omega, dr2, f);
              g = fma(dlr, dlr, g);
              h = fma(yu, yu, h);
              if (tid < m && ((isinf(L.lo[tid]) && yu < 0.0) || (isinf(L.up[tid]) && yu > 0.0))) ex = fma(yu, yu, ex);
            }
            L.sc[0][tid] = f;
            L.sc[1][tid] = mine ? dl * dl : 0.0;
            L.sc[2][tid] = g;
            L.sc[3][tid] = mine ? -al * w + 0.5 * ar * w * w : 0.0;
            L.sc[4][tid] = mine ? ca * au + cb * (d == 2.0 ? au * au : au * sqrt(au)) : 0.0;
            L.sc[5][tid] = mine ? conj15(ty, ca, cb, d) : 0.0;
            L.sc[6][tid] = mine ? ty * w0 : 0.0;
            L.sc[7][tid] = h;
            L.sc[8][tid] = wg == 0 && tid == 0 &&
                           (double)(wall_clock64() - (QUEUE ? L.t_start : t_start)) / ctl.wall_hz > ctl.time_limit_s;
            L.sc[9][tid] = mine ? (isfinite(tx) ? 0.0 : 1.0) + (isfinite(ty) ? 0.0 : 1.0) : 0.0;
            L.sc[10][tid] = ex;
            L.sc[11][tid] = mine ? fabs(w) : 0.0;
          }
          if (tid < NRP) L.dv[tid] = tid < m ? L.ty[tid] - L.y[tid] : 0.0;
          __syncthreads();   // (part is free again, the row images and terms are written)
          rows1(K, val ? tx : 0.0, L.part[wave] + OR, tid);
          for (int q = wave; q < NSC; q += NWV) {   // one wave per sum; the other waves' entries stay zero
            double t = 0.0;
            for (int e = lane; e < NT; e += 64) t += L.sc[q][e];
            t = wave_sum(t);
            if (lane < NWV) L.part[lane][OS + q] = lane == wave ? t : 0.0;
          }
          // dual inner problem: b' = alpha - R' with R' = unscaled K^T Y at T(y), weights a' = arisk
          const double bd = al - (kty(K, L.ty, tid) + dc * ty) / dc, abd = fabs(bd), iad = 1.0 / ar;
          if (rg < CA) { L.ab[wave][slot] = val ? abd : 0.0; L.ia[wave][slot] = val ? iad : 0.0; }
          __builtin_amdgcn_wave_barrier();
          stats<WA>(L.ab[wave], L.ia[wave], dcen, dhw, L.part[wave], tid);
          if (!exchange(X, L, tid, OS + NSC, true, X.spin_limit)) goto fail;
          if (tid < NSC) L.c1[tid] = L.tot[OS + tid];   // (read after the barriers of wg_total)
          double dlo = 0.0, dhi = 0.0, dm = 0.0;
          const int rd = decide(L.tot[lane < NST ? lane : 0], dcen, dhw, dlo, dhi, dm, tid);
          // row terms: primal residual, clip norm, factor risk, row part of the dual objective
          double rv[4] = {0.0, 0.0, 0.0, 0.0};
          if (rown) {
            const double dr = L.dr[tid], w = L.tot[OR + tid] / dr, yu = dr * L.ty[tid];   // unscaled (A W)_j or (G^T W)_l
            if (tid < m) {
              const double Lr = L.lo[tid], Ur = L.up[tid];
              const double cl = fmin(fmax(w, Lr), Ur);
              rv[0] = (w - cl) * (w - cl);
              rv[1] = cl * cl;
              if (yu > 0.0) rv[3] = -(isinf(Ur) ? INFINITY : Ur * yu);
              else if (yu < 0.0) rv[3] = -(isinf(Lr) ? INFINITY : Lr * yu);
            } else {
              const double bF = L.bF[tid], g = w - bF;
              rv[2] = g1 * g * g;
              rv[3] = -(yu * bF + yu * yu / (4.0 * g1));
            }
          }
          wg_total<4>(L, rv, tid);
          const double dprev = dmu;
          dwid = uni(adapt_width(rd, dwid));
          if (rd == 0 || rd == 3) {
            if (!multisect(X, L, dlo, dhi, dmu, tid)) goto fail;
          } else {
            dmu = dm;
          }
          predict(dmu, dprev, dwid, dcen, dhw);
          // inner value sum (a'/2 w^2 - b' w), w = sign(b') max(|b'| - mu', 0) / a'; with
          // exposure rows also max_i |(A^T d)_i| for the infeasibility test (d = T(y_A) - y_A)
          const bool inf_test = ctl.infeas && m > 0;
          {
            const double w = abd > dmu ? sgn(bd) * (abd - dmu) * iad : 0.0;
            const double iv = wave_sum(mine ? 0.5 * w * w / iad - bd * w : 0.0);
            double am = 0.0;
            if (inf_test) {
              const double Ad = kty(K, L.dv, tid);
              am = wave_max(val ? fabs(Ad / dc) : 0.0);
            }
            if (lane == 0) { L.part[wave][0] = iv; L.part[wave][1] = am; }
          }
          if (!exchange(X, L, tid, 2, true, X.spin_limit)) goto fail;
          bool infeasible = false;
          if (inf_test) {   // a Farkas certificate for the feasible set (see solve_kernel.hip)
            double sup = 0.0, mag = 0.0;
            for (int j = lane; j < m; j += 64) {
              const double du = L.dr[j] * L.dv[j];
              double term = 0.0;
              if (du > 0.0) term = isinf(L.up[j]) ? INFINITY : L.up[j] * du;
              else if (du < 0.0) term = isinf(L.lo[j]) ? INFINITY : L.lo[j] * du;
              sup += term;
              mag += fabs(term);
            }
            sup = wave_sum(sup);
            mag = wave_sum(mag);
            const double amax = L.tot[1];
            infeasible = amax + mag > 0.0 && sup + amax < -1e-9 * (mag + amax);
          }
          const double ex = fmax(L.c1[11] - 1.0, 0.0);
          const double phi = L.c1[3] + L.c1[4] + rv[2];
          const double psi = L.tot[0] - L.c1[6] - L.c1[5] + rv[3];
          const double rel_pri = sqrt(rv[0] + ex * ex) / (1.0 + sqrt(rv[1]));
          const double rel_dual = sqrt(L.c1[10]) / (1.0 + sqrt(L.c1[7]));
          const double den = fabs(phi) + fabs(psi);
          const double rel_gap = den > 0.0 ? fabs(phi - psi) / den : 0.0;
          const double relkkt = fmax(rel_pri, fmax(rel_dual, rel_gap));
          const double fpr = sqrt(L.c1[0]);
          const bool nonfinite = L.c1[9] > 0.0 || !isfinite(phi) || !isfinite(psi) || !isfinite(rel_gap) || !isfinite(relkkt);
          if (wg == 0 && tid == 0) {
            ++L.checks;
            s.info[IX_RELKKT] = relkkt; s.info[IX_RELPRI] = rel_pri; s.info[IX_RELDUAL] = rel_dual;
            s.info[IX_RELGAP] = rel_gap; s.info[IX_FPR] = fpr; s.info[IX_POBJ] = phi; s.info[IX_DOBJ] = psi;
          }
          t_check += wall_clock64() - tc0;
          int st = DS_RUNNING;
          if (nonfinite) st = DS_NUMERIC;
          else if (infeasible) st = DS_INFEASIBLE;
          else if (relkkt <= ctl.tol) st = DS_OK;
          else if (L.c1[8] > 0.0) st = DS_TIMEOUT;
          else if (it + 1 >= ctl.max_iter) st = DS_NOT_CONVERGED;
          else {
            if (r0 < 0.0) r0 = uni(fpr);
            const bool rs = (fpr <= ctl.r_suff * r0) || (fpr <= ctl.r_nec * r0 && fpr > rprev) ||
                            ((double)kk + 1.0 >= ctl.r_art * (double)(it + 1));
            restart = __builtin_amdgcn_readfirstlane(rs);
            rprev = uni(fpr);
            kk = min(kk, 1u << 30);
            if (restart) {
              const double dxn = sqrt(L.c1[1]), dyn = sqrt(L.c1[2]);
              if (dxn > 1e-300 && dyn > 1e-300) omega = uni(sqrt(dyn / dxn) * sqrt(omega));   // half-way on a log scale
              r0 = uni(fpr);
              rprev = INFINITY;
              if (tid == 0) ++L.restarts;
              mprev = mu;   // a restart jumps the iterate: drop the multiplier trend
              predict(mu, mu, wid, cen, hw);
            }
          }
          status = __builtin_amdgcn_readfirstlane(st);
          if (status != DS_RUNNING) {
            const bool bad = status == DS_NUMERIC;
            if (mine) s.w_out[i] = dc * (bad ? L.x0[tid] : tx);
            if (s.y_out) {
              // infeasible: the exposure part holds the certificate direction d of the test
              if (wg == 0 && rown)
                s.y_out[tid] = L.dr[tid] * (bad ? L.y0r[tid] : (status == DS_INFEASIBLE && tid < m ? L.dv[tid] : L.ty[tid]));
              if (mine) s.y_out[nr + i] = bad ? L.y0[tid] : ty;
            }
            ++it;
            if (wg == 0 && tid == 0) {
              const long long t_end = wall_clock64();
              s.info[IX_ITERS] = (double)it;
              s.info[IX_RESTARTS] = (double)L.restarts;
              s.info[IX_OMEGA] = omega;
              s.info[IX_ETA] = eta;
              s.info[IX_NORMK] = ctl.eta_safety / eta;
              s.info[IX_SPEC_MISS] = (double)L.miss;
              s.info[IX_EXCHANGES] = (double)X.epoch;
              s.info[IX_CHECKS] = (double)L.checks;
              s.info[IX_T_ITER] = (double)(t_end - t_loop) / ctl.wall_hz;
              s.info[IX_T_CHECK] = (double)t_check / ctl.wall_hz;
              s.info[IX_T_POWER] = (double)(t_loop - (QUEUE ? L.t_start : t_start)) / ctl.wall_hz;
              s.info[IX_MS_ROUNDS] = (double)L.rounds;
              s.info[IX_MISS_IN] = (double)L.miss_in;
              s.info[IX_MISS_OUT] = (double)L.miss_out;
              s.status[0] = status;
            }
            return;
          }
        }
        if (check && f32) {
#pragma unroll
          for (int q = 0; q < RA; ++q)
#pragma unroll
            for (int c = 0; c < CA; ++c) K[q][c] = (double)(float)K[q][c];
        }
        // reflected Halpern step, or the restart at T(z)
        if (restart) {
          x = tx;
          yc = ty;
          L.x0[tid] = tx;
          L.y0[tid] = ty;
          if (rown) L.y[tid] = L.y0r[tid] = L.ty[tid];
          kk = 0;
        } else {
          x = stored(a1 * ((1.0 + rho) * tx - rho * x) + a0 * L.x0[tid], L.x0[tid]);
          yc = stored(a1 * ((1.0 + rho) * ty - rho * yc) + a0 * L.y0[tid], L.y0[tid]);
          if (rown) L.y[tid] = a1 * ((1.0 + rho) * L.ty[tid] - rho * L.y[tid]) + a0 * L.y0r[tid];
          ++kk;
        }
        ++it;
        __syncthreads();
        if (check && cp->snaps) {
          const auto [tid, lane, wave, rg, slot, li, val, mine, rown] = place<CA>(tid0, nwa, nr);
          const long long j = it / cp->check_every;
          double* o = opaque(sp)->snaps + (size_t)(j % cp->snaps) * (2 * n + nr + 2);
          if (mine) { o[i0 + li] = dc * x; o[n + nr + i0 + li] = yc; }
          if (wg == 0 && rown) o[n + tid] = L.dr[tid] * L.y[tid];
          if (wg == 0 && tid == 0) { o[2 * n + nr] = omega; o[2 * n + nr + 1] = (double)L.restarts; }
        }
        if (check && it == cp->stop_at) {   // hand the iterate over, unscaled, as a warm start
          const auto [tid, lane, wave, rg, slot, li, val, mine, rown] = place<CA>(tid0, nwa, nr);
          const DevState& s = *opaque(sp);
          if (mine) { s.w_out[i0 + li] = dc * x; s.y_out[nr + i0 + li] = yc; }
          if (wg == 0 && rown) s.y_out[tid] = L.dr[tid] * L.y[tid];
          if (wg == 0 && tid == 0) {
            s.info[IX_ITERS] = (double)it;
            s.info[IX_RESTARTS] = (double)L.restarts;
            s.info[IX_OMEGA] = omega;
            s.status[0] = DS_NOT_CONVERGED;
          }
          return;
        }
      }
    }
  }
fail:
  if (tid0 == 0) __hip_atomic_store(s.status, (int32_t)DS_BARRIER, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int RA, int CA>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_reg(
    const DevProblem* __restrict__ dp, const DevState* __restrict__ ds, const DevControl* __restrict__ dc) {
  __shared__ RegLds<RA, CA> L;
  reg_body<RA, CA, false>(dp, ds, dc, blockIdx.x, L, dc->spin_limit);
}

// Many instances: resident workgroups take (instance, rank) tickets in order, an instance's
// ranks one after another, so at any time the unfinished instance with the first tickets
// has all its workgroups running or about to be taken up by those that finish earlier
// ones: every team completes, whatever the sizes.  A team's first wait is for that.
template <int RA, int CA>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_reg_queue(
    const DevProblem* __restrict__ dp, const DevState* __restrict__ ds, const DevControl* __restrict__ dc,
    const int* __restrict__ inst, const int* __restrict__ rank, int tickets, int* next) {
  __shared__ RegLds<RA, CA> L;
  __shared__ int s_t;
  while (true) {
    __syncthreads();
    if (threadIdx.x == 0) s_t = __hip_atomic_fetch_add(next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(s_t);
    if (t >= tickets) return;
    const int b = inst[t];
    reg_body<RA, CA, true>(dp + b, ds + b, dc + b, rank[t], L, 0xffffffffu);
  }
}

}  // namespace

// Row groups of 16 and assets per lane group instantiated: RA x CA doubles of rows per
// lane, at most 80 (160 of the 256 registers).
static const void* reg_fn(int ra, int ca, bool queue) {
#define FFO_REG(R, C) \
  if (ra == R && ca == C) return queue ? (const void*)k_reg_queue<R, C> : (const void*)k_reg<R, C>;
  FFO_REG(1, 4) FFO_REG(1, 8) FFO_REG(1, 16)
  FFO_REG(2, 4) FFO_REG(2, 8) FFO_REG(2, 16)
  FFO_REG(3, 8) FFO_REG(3, 16)
  FFO_REG(5, 8) FFO_REG(5, 16)
  FFO_REG(7, 4) FFO_REG(7, 8)
  FFO_REG(9, 4) FFO_REG(9, 8)
  FFO_REG(10, 4) FFO_REG(10, 8)
#undef FFO_REG
  return nullptr;
}

int reg_vmax(int ra) { return std::max(96, OR + 32 * ra); }

bool reg_plan(int64_t n, int nr, int cus, RegPlan* out) {
  static const int ras[7] = {1, 2, 3, 5, 7, 9, 10};
  int ra = 0;
  for (int r : ras)
    if (16 * r >= nr) { ra = r; break; }
  if (!ra) return false;
  for (int ca : {4, 8, 16}) {
    if (!reg_fn(ra, ca, false)) continue;
    const int64_t g = (n + 32 * ca - 1) / (32 * ca);
    const bool last = !reg_fn(ra, 2 * ca, false);
    if (g > (last ? cus : 1)) continue;
    out->ra = ra;
    out->ca = ca;
    out->nwg = (int)g;
    return true;
  }
  return false;
}

int launch_reg(const RegPlan& pl, const DevProblem* dp, const DevState* ds, const DevControl* dc, void* stream) {
  void* args[] = {(void*)&dp, (void*)&ds, (void*)&dc};
  const hipError_t e = hipLaunchCooperativeKernel(reg_fn(pl.ra, pl.ca, false), dim3(pl.nwg), dim3(NT), args, 0, (hipStream_t)stream);
  return e == hipSuccess ? 0 : (int)e;
}

int launch_reg_queue(const RegPlan& pl, const DevProblem* dp, const DevState* ds, const DevControl* dc, const int* inst,
                     const int* rank, int tickets, int* next, int grid, void* stream) {
  void* args[] = {(void*)&dp, (void*)&ds, (void*)&dc, (void*)&inst, (void*)&rank, (void*)&tickets, (void*)&next};
  const hipError_t e = hipLaunchCooperativeKernel(reg_fn(pl.ra, pl.ca, true), dim3(grid), dim3(NT), args, 0, (hipStream_t)stream);
  return e == hipSuccess ? 0 : (int)e;
}

}  // namespace ffo
