// Multi-period solve with the constraint rows in registers (FP64, impact exponent 3/2 or 2).
//
// Same iteration as solve_kernel.hip, laid out for 1 to 31 decision periods: a team of
// workgroups of eight waves, 64 assets each.  Lane = asset and wave w owns periods w, w + 8,
// ..., so an element's iterates stay in one lane's registers and a period's sums stay in one
// wave.  The two products are matrix products over the periods, on the FP64 matrix cores:
//   K~^T Y:  wave (a, h) holds 16 assets' columns and takes a period tile (more than 15
//            periods) or half of the rows (fewer);
//   K~ Xbar: wave holds 16 rows and takes all of the 64 assets, or a part of them where
//            there are fewer row tiles than waves.
// Each wave keeps its operand of the rows in registers for the whole solve (up to 28 and 16
// doubles per lane); Y and Xbar come from LDS.
//
// Budget multipliers: the statistics S, A0, count at eight candidates per period go through
// one exchange.  With no breakpoint between the bracketing candidates the root is the left
// piece's; with one, S is the larger of the two pieces there (it is convex), so the root is
// the larger of their roots; with more, another round of eight points between that lower
// bound and the chord's root (the bracket is narrow, one such round does).  Another exchange
// carries the row products.
//
// What bounds it: latency.  T = 20, n = 3000, 100 rows (47 workgroups) takes 26.5 us per
// iteration (67.5 in the general kernel) with 3.1 exchanges of about 2.5 us each, 3.5 us of
// matrix-instruction issue, and dependent chains between (statistics, decisions, the row
// duals, which every workgroup updates for itself); T = 10, n = 3000, 22 rows 11.7 us (21.9).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include "internal.h"
#include "team_exchange.h"
#include "wave_ops.h"

namespace ffo {
namespace {

constexpr int NT = 512, NWV = NT / 64;
constexpr int NA = 64, LDA = NA + 1;      // assets per workgroup, row stride of per-period LDS arrays
constexpr int NST = 24;                   // statistics of a period: S(c_q), A0(c_q), count(c_q), q < 8
constexpr int NSC = 12;                   // scalar sums of a check
constexpr int ROUNDS = 40;

typedef double d4 __attribute__((ext_vector_type(4)));
// Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; register j holds D[4 j + l / 16][l % 16].
__device__ __forceinline__ d4 mfma(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// JT: periods (and trades) per wave; NRT: tiles of 16 rows.
template <int JT, int NRT>
struct Shape {
  static constexpr int MT = JT <= 2 ? 1 : 2;                       // tiles of 16 periods
  static constexpr int NRP = 16 * NRT, LDY = NRP + 1;
  static constexpr int PK = NRT <= 2 ? 4 : (NRT <= 4 ? 2 : 1);     // parts of the assets in K~ x
  static constexpr int KS = 16 / PK, QS = MT == 1 ? 2 * NRT : 4 * NRT;
  static constexpr int RP = MT == 1 ? 2 : 1;                       // parts of the rows in K~^T y
};

// Exchange entries: scalars, per-period budgets, statistics, rows.
__host__ __device__ constexpr int off_stats(int P) { return 16 + P; }
__host__ __device__ constexpr int off_rows(int P) { return 16 + P + NST * P; }

// LDS (doubles), in this order; the host sizes the launch with the same sum.
template <int JT, int NRT>
struct Lds {
  using S = Shape<JT, NRT>;
  double *y, *y0, *ty, *dv;               // [P][LDY] row duals, anchor, image, check displacement
  double *xs, *R, *sC;                    // [P][LDA] x operand; [RP][P][LDA] K~^T y; [P + 1][LDA] drC yC
  double *st;                             // staging of an exchange: off_rows + PK P nr
  double *dr, *sd, *rs, *lo, *up, *bF;    // [NRP] row scale, sigma dr, 1 / (sigma dr) or shrinkage, bounds, offset
  double *red;                            // [NWV][16]
  int *flag;                              // [NWV] wave flags, [NWV] the barrier's word, [NWV + 1 ...] counters
  __host__ __device__ static size_t doubles(int P, int nr) {
    return (size_t)4 * P * S::LDY + (size_t)P * LDA * (1 + S::RP) + (size_t)(P + 1) * LDA + off_rows(P) +
           (size_t)S::PK * P * nr + 6 * S::NRP + NWV * 16 + 16;
  }
  __device__ __forceinline__ Lds(double* p, int P, int nr) {
    auto take = [&](size_t n) { double* r = p; p += n; return r; };
    y = take((size_t)P * S::LDY); y0 = take((size_t)P * S::LDY); ty = take((size_t)P * S::LDY); dv = take((size_t)P * S::LDY);
    xs = take((size_t)P * LDA); R = take((size_t)S::RP * P * LDA); sC = take((size_t)(P + 1) * LDA);
    st = take(off_rows(P) + (size_t)S::PK * P * nr);
    dr = take(S::NRP); sd = take(S::NRP); rs = take(S::NRP); lo = take(S::NRP); up = take(S::NRP); bF = take(S::NRP);
    red = take(NWV * 16);
    flag = (int*)take(16);
  }
};
constexpr int F_OK = NWV, F_RESTARTS = NWV + 1, F_CHECKS = NWV + 2, F_MISS = NWV + 3, F_ROUNDS = NWV + 4;

extern __shared__ double mp_lds[];

// R[part][t][asset] = sum_r y[t][r] K~[r][asset] over the wave's rows (synchronise before reading R).
template <int JT, int NRT>
__device__ __forceinline__ void kty(const double (&K)[Shape<JT, NRT>::QS], const double* y, double* R, int P, int tid) {
  using S = Shape<JT, NRT>;
  const int lane = tid & 63, wave = wave_of(tid), a = wave & 3, h = wave >> 2;
  const int t0 = S::MT == 2 ? 16 * h : 0, q0 = S::MT == 2 ? 0 : h * S::QS;
  const double* yp = y + min(t0 + (lane & 15), P - 1) * S::LDY + 4 * q0 + (lane >> 4);   // (rows past P give outputs not kept)
  d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < S::QS; ++q) acc = mfma(yp[4 * q], K[q], acc);
  double* out = R + (S::MT == 2 ? 0 : h * P * LDA) + 16 * a + (lane & 15);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int t = t0 + 4 * j + (lane >> 4);
    if (t < P) out[t * LDA] = acc[j];
  }
}
template <int JT, int NRT>
__device__ __forceinline__ double kty_at(const double* R, int P, int t, int lane) {
  const double r = R[t * LDA + lane];
  return Shape<JT, NRT>::RP == 2 ? r + R[(P + t) * LDA + lane] : r;
}

// st[off_rows + part P nr + t nr + r] = sum over the part's assets of K~[r][i] xs[t][i].
template <int JT, int NRT>
__device__ __forceinline__ void kx(const double (&K)[Shape<JT, NRT>::KS], const double* xs, double* st, int P, int nr, int tid) {
  using S = Shape<JT, NRT>;
  const int lane = tid & 63, wave = wave_of(tid);
  if (wave >= NRT * S::PK) return;
  const int rt = wave % NRT, part = wave / NRT, r = 16 * rt + (lane & 15);
  double* out = st + off_rows(P) + part * P * nr + r;
#pragma unroll
  for (int mt = 0; mt < S::MT; ++mt) {
    const double* xp = xs + min(16 * mt + (lane & 15), P - 1) * LDA + 4 * part * S::KS + (lane >> 4);
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < S::KS; ++q) acc = mfma(xp[4 * q], K[q], acc);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int t = 16 * mt + 4 * j + (lane >> 4);
      if (t < P && r < nr) out[t * nr] = acc[j];
    }
  }
}

// Exchanges entries [lo, hi) of st (the rows' parts added first); of these, [m0, m1) combine
// by maximum.  Synchronises st before, and the team after.
template <int JT, int NRT>
__device__ __forceinline__ bool exchange(RegX& X, const Lds<JT, NRT>& L, int P, int nr, int lo, int hi, int m0, int m1, int tid) {
  using S = Shape<JT, NRT>;
  const int oR = off_rows(P), Pn = P * nr;
  __syncthreads();
  for (int e = lo + tid; e < hi; e += NT) {
    double s = L.st[e];
    if (S::PK > 1 && e >= oR) {
#pragma unroll
      for (int k = 1; k < S::PK; ++k) s += L.st[e + k * Pn];
    }
    if (X.nwg == 1) L.st[e] = s;
    else if (e >= m0 && e < m1) team_max(X, e, s);
    else team_add(X, e, s);
  }
  if (X.nwg == 1) { __syncthreads(); return true; }
  return team_barrier(X, tid, &L.flag[F_OK], X.spin_limit);
}
template <int JT, int NRT>
__device__ __forceinline__ double total(const RegX& X, const Lds<JT, NRT>& L, int e, bool mx = false) {
  return X.nwg == 1 ? L.st[e] : team_total(X, e, mx);
}
__device__ __forceinline__ void done_reading(RegX& X, int tid) {
  if (X.nwg > 1) team_end(X, tid, NT);
}

// Statistics of one period (the wave's lanes are its assets) at the candidates c(0..7) into
// out[0, 24): S and A0 by halving sums across the wave, the counts by ballots.
template <class C>
__device__ __forceinline__ void stats(double ab, double ia, C c, double* out, int lane) {
  double v[16];
  int cnt = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const double d = ab - c(q);
    const bool in = d > 0.0;
    v[2 * q + 1] = in ? ia : 0.0;
    v[2 * q] = in ? d * ia : 0.0;
    const int k = __popcll(__ballot(in));
    cnt = lane == q ? k : cnt;
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = pair_sum32(v[2 * q], v[2 * q + 1]);   // low half-wave: S(c_q), high: A0(c_q)
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = pair_sum16(v[2 * q], v[2 * q + 1]);   // even rows: c_2q, odd rows: c_2q+1
  const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const double keep = b3 ? v[q + 2] : v[q], send = b3 ? v[q] : v[q + 2];
    v[q] = keep + dpp<DPP_MIRROR>(send);
  }
  {
    const double keep = b2 ? v[1] : v[0], send = b2 ? v[0] : v[1];
    v[0] = sum4(keep + dpp<DPP_HALF_MIRROR>(send));
  }
  if ((lane & 3) == 0) out[(lane >> 5) * 8 + 2 * (2 * (lane >> 3 & 1) + (lane >> 2 & 1)) + (lane >> 4 & 1)] = v[0];
  if (lane < 8) out[16 + lane] = (double)cnt;
}

// Multiplier state of the wave's periods, slot j in lanes 8 j .. 8 j + 7 (JT <= 8): prediction,
// adaptive width, last two values, and the bracket of the rounds in progress (todo: 0 settled,
// 1 another round on [lo, hi], 2 S(0) and max |b| needed first).
struct Mult {
  double mu, mprev, cen, hw, wid, lo, hi;
  int todo;
};

// Candidate lane % 8 of the lane's slot.
__device__ __forceinline__ double point(const Mult& M, int round, int lane) {
  const int q = lane & 7;
  return round == 0 ? cand(M.cen, M.hw, q) : fma((M.hi - M.lo) * (1.0 / 7.0), (double)q, M.lo);
}

// Decisions of all slots from their exchanged statistics, lane = (slot, candidate).  Lane q
// works out the interval [c_q, c_q+1]; the one that brackets the root is then broadcast.
__device__ __forceinline__ void decide(Mult& M, double S, double A, double N, int round, int lane) {
  constexpr int NEXT = 0x101;   // DPP row_shl:1, lane i <- lane i + 1
  const int q = lane & 7;
  const bool act = round == 0 || M.todo != 0;
  const double c0 = point(M, round, lane), c1 = dpp<NEXT>(c0), S1 = dpp<NEXT>(S), N1 = dpp<NEXT>(N);
  const double root = A > 0.0 ? fma(S - 1.0, recip(A), c0) : 0.0, root1 = dpp<NEXT>(root);   // of the linear pieces
  const unsigned ge = (unsigned)(__ballot(S >= 1.0) >> (lane & 56)) & 0xffu;
  const int qs = 31 - __clz(ge);                    // S is non-increasing: S(c_q) >= 1 for q <= qs (-1: none)
  const double m = N - N1;                          // breakpoints inside
  const double low = fmin(fmax(m > 0.0 ? fmax(root, root1) : root, c0), c1);
  // S lies between its tangents and its chord, so the root does too
  const double high = fmin(fmax(fma(c1 - c0, (S - 1.0) * recip(S - S1), c0), low), c1);
  const bool fin = m <= 1.0 || (c1 - low) <= 4.0 * 2.220446049250313e-16 * fabs(c1) || round == ROUNDS;
  const bool here = q == qs;
  const double low8 = max8(here ? low : -1.0), high8 = max8(here ? high : -1.0), fin8 = max8(here && fin ? 1.0 : 0.0);
  const double first = max8(q == 0 ? c0 : -1.0), last = max8(c0);
  if (round == 0) M.mprev = M.mu;
  int todo = 0, r = 1;
  double mu = M.mu, lo = M.lo, hi = M.hi;
  if (qs >= 0 && qs < 7) {
    if (fin8 > 0.0) { mu = low8; r = qs == 3 ? 1 : 4; }
    else { lo = low8; hi = high8; todo = 1; r = qs == 3 ? 0 : 3; }
  } else if (round > 0) {
    mu = qs < 0 ? lo : hi;                          // the root is an end of the bracket, up to rounding
  } else if (M.cen + M.hw <= 0.0 && S <= 1.0) {
    mu = 0.0;                                       // predicted zero: every candidate is 0 and S(c_0) = S(0)
  } else {
    lo = qs < 0 ? 0.0 : last;
    hi = qs < 0 && M.cen + M.hw > 0.0 ? first : -1.0;   // -1: the upper end is max |b|
    todo = 2;
    r = 3;
  }
  if (act) {
    M.mu = mu; M.lo = lo; M.hi = hi; M.todo = todo;
    if (round == 0) M.wid = adapt_width(r, M.wid);
  }
}

__device__ __forceinline__ void predict_all(Mult& M) {
  const double c = fmax(M.mu + (M.mu - M.mprev), 0.5 * M.mu);
  M.cen = M.mu > 0.0 ? c : 0.0;
  M.hw = M.mu > 0.0 ? M.wid * M.mu : 0.0;
}

// Settles the multipliers of the wave's periods: `ab(j)` is |b| of slot j, ia 1/a.  The
// statistics of round 0 are in st already.  False when a bounded wait expired.
template <int JT, int NRT, class FA>
__device__ __forceinline__ bool settle(Mult& M, RegX& X, const Lds<JT, NRT>& L, int P, int nr, FA ab, double ia, int tid) {
  const int oD = off_stats(P), lane = tid & 63, wave = wave_of(tid);
  const int ts = wave + 8 * (lane >> 3);            // the lane's period in a decision
  const bool own = (lane >> 3) < JT && ts < P;
  if (!exchange(X, L, P, nr, oD, oD + NST * P, 0, 0, tid)) return false;
  for (int round = 0;; ++round) {
    {
      const int o = oD + NST * (own ? ts : wave) + (lane & 7);
      const double S = total(X, L, o), A = total(X, L, o + 8), N = total(X, L, o + 16);
      decide(M, S, A, N, round, lane);
      if (!own) M.todo = 0;
    }
    done_reading(X, tid);
    const int todo = (__ballot(M.todo & 1) ? 1 : 0) | (__ballot(M.todo & 2) ? 2 : 0);
    if (lane == 0) L.flag[wave] = todo;
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) all |= L.flag[w];
    all = __builtin_amdgcn_readfirstlane(all);
    if (!all) return true;
    if (tid == 0) ++L.flag[F_ROUNDS];
    if (all & 2) {   // S(0) and max |b| of the periods that need them
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const int t = wave + 8 * j;
        if (t >= P) continue;
        double s = 0.0, m = 0.0;
        if (__builtin_amdgcn_readlane(M.todo, 8 * j) & 2) { s = wave_sum(ab(j) * ia); m = wave_max(ab(j)); }
        if (lane == 0) { L.st[oD + t] = s; L.st[oD + P + t] = m; }
      }
      if (!exchange(X, L, P, nr, oD, oD + 2 * P, oD + P, oD + 2 * P, tid)) return false;
      const double s = total(X, L, oD + (own ? ts : wave)), m = total(X, L, oD + P + (own ? ts : wave), true);
      if (M.todo & 2) {
        M.todo = 1;
        if (s <= 1.0) { M.mu = 0.0; M.todo = 0; }
        if (!(M.hi >= 0.0)) M.hi = m;
        if (!(M.hi >= M.lo)) { M.lo = 0.0; M.hi = m; }
      }
      done_reading(X, tid);
      __syncthreads();
    }
    const double c = point(M, 1, lane);
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      const int t = wave + 8 * j;
      if (t >= P) continue;
      double* o = L.st + oD + NST * t;
      if (__builtin_amdgcn_readlane(M.todo, 8 * j)) stats(ab(j), ia, [&](int q) { return lane_of(c, 8 * j + q); }, o, lane);
      else if (lane < NST) o[lane] = 0.0;
    }
    if (!exchange(X, L, P, nr, oD, oD + NST * P, 0, 0, tid)) return false;
  }
}

template <int JT, int NRT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mp(
    const DevProblem* __restrict__ pp, const DevState* __restrict__ sp, const DevControl* __restrict__ cp) {
  using S = Shape<JT, NRT>;
  const DevProblem& p = *pp;
  const DevState& s = *sp;
  const DevControl& ctl = *cp;
  const int P = p.P, nr = p.nr, m = p.m, n = p.n, wg = blockIdx.x;
  const Lds<JT, NRT> L(mp_lds, P, nr);
  const int tid0 = threadIdx.x;
  const int i0 = wg * ctl.nw, nwa = max(0, min(ctl.nw, n - i0));
  const double rho = ctl.rho, d = p.d, g1 = p.g1;
  const int oD = off_stats(P), oR = off_rows(P), Pnr = P * nr;
  const unsigned rcp_nr = nr > 0 ? ((1u << 20) + nr - 1) / nr : 0;   // e / nr = e rcp_nr >> 20 for e < 2^12
  RegX X = team_init(s, ctl, wg);
  constexpr double RT2 = 0.70710678118654752440;
#define FFO_DRC(t) ((t) == 0 || (t) == P ? 1.0 : RT2)   // trade-row scale (one or two unit entries)

  // the wave's operands of the rows
  double Kt[S::QS], Kx[S::KS];
  double x[JT], x0[JT], yc[JT], yc0[JT], al[JT], ca[JT], cb[JT];   // slot j: period and trade wave + 8 j
  double dc, ar, w0, wT;
  {
    const int tid = fresh(tid0), lane = tid & 63, wave = wave_of(tid);
    {
      const int a = wave & 3, h = wave >> 2, q0 = S::MT == 2 ? 0 : h * S::QS, l = 16 * a + (lane & 15);
#pragma unroll
      for (int q = 0; q < S::QS; ++q) {
        const int r = 4 * (q0 + q) + (lane >> 4);
        Kt[q] = r < nr && l < nwa ? p.K[(size_t)r * p.ldk + i0 + l] : 0.0;
      }
      const int rt = wave % NRT, part = wave / NRT, r = 16 * rt + (lane & 15);
#pragma unroll
      for (int q = 0; q < S::KS; ++q) {
        const int l2 = 4 * (part * S::KS + q) + (lane >> 4);
        Kx[q] = wave < NRT * S::PK && r < nr && l2 < nwa ? p.K[(size_t)r * p.ldk + i0 + l2] : 0.0;
      }
    }
    const bool val = lane < nwa;
    const int i = i0 + lane;
    dc = val ? p.dc[i] : 1.0;
    ar = val ? p.arisk[i] : 1.0;
    w0 = val ? p.w0[i] : 0.0;
    wT = val ? p.wT[i] : 0.0;
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      const int t = wave + 8 * j;
      const size_t e = (size_t)t * n + i;
      const bool in = val && t < P, it = val && t <= P;
      al[j] = in ? p.alpha[e] + ar * wT : 0.0;     // (cvec = w_T)
      ca[j] = it ? p.ca[e] : 0.0;
      cb[j] = it ? p.cb[e] : 0.0;
      x[j] = in ? (s.w_init ? s.w_init[e] : w0) / dc : 0.0;
      yc[j] = it && s.y_init ? s.y_init[(size_t)Pnr + e] / FFO_DRC(t) : 0.0;
      x0[j] = x[j];
      yc0[j] = yc[j];
    }
    for (int e = tid; e < NST * P + 16 + P + S::PK * Pnr; e += NT) L.st[e] = 0.0;
    for (int e = tid; e < P * S::LDY; e += NT) {
      const int t = e / S::LDY, j = e - t * S::LDY;
      double v = 0.0;
      if (s.y_init && j < nr)
        v = (j < m ? s.y_init[(size_t)t * m + j] : s.y_init[(size_t)P * m + (size_t)t * p.k + (j - m)]) / p.dr[j];
      L.y[e] = L.y0[e] = L.ty[e] = v;
      L.dv[e] = 0.0;
    }
    for (int j = tid; j < S::NRP; j += NT) {
      L.dr[j] = j < nr ? p.dr[j] : 1.0;
      L.lo[j] = j < m ? p.L[j] : 0.0;
      L.up[j] = j < m ? p.U[j] : 0.0;
      L.bF[j] = j >= m && j < nr ? p.bF[j - m] : 0.0;
      L.sd[j] = L.rs[j] = 0.0;
    }
    for (int e = tid; e < P * LDA; e += NT) L.xs[e] = 0.0;
    if (tid < 16) L.flag[tid] = 0;
    __syncthreads();
  }
  // the asset's trade-row adjoint at slot t, drC_t yC_t staged in sC
  const auto adj = [&](int t, int lane) { return dc * (L.sC[t * LDA + lane] - L.sC[(t + 1) * LDA + lane]); };
  // trade row t of K~ applied to the staged x
  const auto trade = [&](int t, int lane) {
    const double a = t < P ? L.xs[t * LDA + lane] : 0.0, b = t > 0 ? L.xs[(t - 1) * LDA + lane] : 0.0;
    return FFO_DRC(t) * dc * (a - b);
  };

  const long long t_start = wall_clock64();
  long long t_check = 0;
  double omega = ctl.omega0 > 0.0 ? ctl.omega0 : 1.0, r0 = -1.0, rprev = INFINITY, lam = 0.0;
  long long it = 0;
  uint32_t kk = 0;   // since the last restart (from 2^30 on the Halpern weights no longer matter)
  int left = (int)min((long long)ctl.check_every, (long long)ctl.max_iter), status = DS_RUNNING;

  // ---- power iteration (see solve_kernel.hip)
  {
    double v[JT];
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      const int lane = tid0 & 63, t = wave_of(tid0) + 8 * j;
      v[j] = lane < nwa && t < P ? 1.0 + 0.25 * (double)(((i0 + lane) * 7919 + t * 104729) % 1000) / 1000.0 : 0.0;
    }
    for (int pw = 0; pw < ctl.npow; ++pw) {
      const int tid = fresh(tid0), lane = tid & 63, wave = wave_of(tid);
      double vv = 0.0, uu = 0.0;
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const int t = wave + 8 * j;
        if (t < P) L.xs[t * LDA + lane] = v[j];
        vv = fma(v[j], v[j], vv);
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const int t = wave + 8 * j;
        if (t > P) continue;
        const double u = lane < nwa ? trade(t, lane) : 0.0;
        uu = fma(u, u, uu);
        L.sC[t * LDA + lane] = FFO_DRC(t) * u;
      }
      vv = wave_sum(vv);
      uu = wave_sum(uu);
      if (lane == 0) { L.red[16 * wave] = vv; L.red[16 * wave + 1] = uu; }
      kx<JT, NRT>(Kx, L.xs, L.st, P, nr, tid);
      __syncthreads();
      if (tid < 2) {
        double a = 0.0;
        for (int w = 0; w < NWV; ++w) a += L.red[16 * w + tid];
        L.st[tid] = a;
      }
      // (entries 2 .. oR - 1 stay zero)
      if (!exchange(X, L, P, nr, 0, oR + Pnr, 0, 0, tid)) goto fail;
      const double tv = uni(total(X, L, 0)), tu = uni(total(X, L, 1));
      double kv = 0.0;
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const int t = wave + 8 * j;
        if (t >= P) continue;
        for (int r = lane; r < nr; r += 64) {
          const double z = total(X, L, oR + t * nr + r);
          L.ty[t * S::LDY + r] = z;
          kv = fma(z, z, kv);
        }
      }
      done_reading(X, tid);
      kv = wave_sum(kv);
      if (lane == 0) L.red[16 * wave + 2] = kv;
      __syncthreads();
      kty<JT, NRT>(Kt, L.ty, L.R, P, tid);
      double k2 = tu;
#pragma unroll
      for (int w = 0; w < NWV; ++w) k2 += L.red[16 * w + 2];
      lam = uni(tv > 0.0 ? k2 / tv : 0.0);
      const double scale = uni((lam > 0.0 && tv > 0.0) ? 1.0 / (lam * sqrt(tv)) : 1.0);
      __syncthreads();
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const int t = wave + 8 * j;
        if (t < P) v[j] = lane < nwa ? (kty_at<JT, NRT>(L.R, P, t, lane) + adj(t, lane)) * scale : 0.0;
      }
    }
  }
  {
    const int tid = fresh(tid0), lane = tid & 63, wave = wave_of(tid);
    for (int e = tid; e < P * S::LDY; e += NT) L.ty[e] = L.y[e];
    __syncthreads();   // (sC is read above)
#pragma unroll
    for (int j = 0; j < JT; ++j)
      if (wave + 8 * j <= P) L.sC[(wave + 8 * j) * LDA + lane] = FFO_DRC(wave + 8 * j) * yc[j];
  }
  {
    const double eta = uni(ctl.eta_safety / sqrt(fmax(lam, 1e-300)));
    const long long t_loop = wall_clock64();
    Mult M{0.0, 0.0, 0.0, 0.0, 1e-3, 0.0, 0.0, 0}, D = M;   // budget multipliers, and the dual inner problem's

    while (true) {
      const double sigma = uni(eta * omega), isig = uni(1.0 / sigma);
      const double idc = 1.0 / dc, itd = omega / eta * idc;          // b = x / (tau dc) - R / dc + alpha
      const double ia = (tid0 & 63) < nwa ? 1.0 / (itd * idc + ar) : 0.0, gia = ia * idc;
      for (int j = tid0; j < nr; j += NT) {
        const double dr = L.dr[j], sd = sigma * dr;
        L.sd[j] = sd;
        L.rs[j] = j < m ? 1.0 / sd : 2.0 * g1 / (sd * dr + 2.0 * g1);
      }
      __syncthreads();
      bool restart = false;
      while (!restart) {
        const int tid = fresh(tid0), lane = tid & 63, wave = wave_of(tid);
        const bool check = --left == 0;
        if (check) left = (int)min((long long)ctl.check_every, ctl.max_iter - (it + 1));
        const double k1 = (double)kk, a0 = uni(recip(k1 + 2.0)), a1 = uni((k1 + 1.0) * a0);
        // prox inputs and the statistics at the bracket candidates
        kty<JT, NRT>(Kt, L.y, L.R, P, tid);
        __syncthreads();
        double b[JT];
        const double cq = point(M, 0, lane);
#pragma unroll
        for (int j = 0; j < JT; ++j) {
          const int t = wave + 8 * j;
          b[j] = 0.0;
          if (t >= P) continue;
          const double Ry = kty_at<JT, NRT>(L.R, P, t, lane) + adj(t, lane);
          b[j] = lane < nwa ? x[j] * itd - Ry * idc + al[j] : 0.0;
          stats(fabs(b[j]), ia, [&](int q) { return lane_of(cq, 8 * j + q); }, L.st + oD + NST * t, lane);
        }
        if (!settle<JT, NRT>(M, X, L, P, nr, [&](int j) { return fabs(b[j]); }, ia, tid)) goto fail;
        // T(x) and K~ xbar
        double tx[JT], ty[JT];
#pragma unroll
        for (int j = 0; j < JT; ++j) {
          const int t = wave + 8 * j;
          tx[j] = 0.0;
          if (t >= P) continue;
          const double ab = fabs(b[j]), mu = lane_of(M.mu, 8 * j);
          tx[j] = ab > mu ? copysign(gia, b[j]) * (ab - mu) : 0.0;
          L.xs[t * LDA + lane] = 2.0 * tx[j] - x[j];
        }
        predict_all(M);
        __syncthreads();
        kx<JT, NRT>(Kx, L.xs, L.st, P, nr, tid);
        // trade duals while the products meet
#pragma unroll
        for (int j = 0; j < JT; ++j) {
          const int t = wave + 8 * j;
          ty[j] = 0.0;
          if (t > P) continue;
          const double drc = FFO_DRC(t), bc = t == 0 ? w0 : t == P ? -wT : 0.0, sdr = sigma * drc;
          const double vs = yc[j] + sigma * trade(t, lane), h = isig * (t == 0 || t == P ? 1.0 : 1.41421356237309504880);
          const double tp = h * (t == 0 || t == P ? 1.0 : 1.41421356237309504880);   // 1 / (sigma drC^2)
          const double pr = prox15(vs * h - bc, tp * ca[j], tp * cb[j], d);
          ty[j] = vs - sdr * bc - sdr * pr;
        }
        if (!exchange(X, L, P, nr, oR, oR + Pnr, 0, 0, tid)) goto fail;
        // row duals, entry tid + 512 u of the P nr
        constexpr int NE = (8 * JT * S::NRP + NT - 1) / NT;
        double kt[NE];
#pragma unroll
        for (int u = 0; u < NE; ++u) kt[u] = tid + NT * u < Pnr ? total(X, L, oR + tid + NT * u) : 0.0;
#pragma unroll
        for (int u = 0; u < NE; ++u) {
          if (tid + NT * u >= Pnr) break;
          const int t = (int)(((unsigned)(tid + NT * u) * rcp_nr) >> 20), r = tid + NT * u - t * nr, e = t * S::LDY + r;
          const double yo = L.y[e], vs = fma(sigma, kt[u], yo), sd = L.sd[r], rs = L.rs[r];
          double v;
          if (r < m) {
            const double Lr = L.lo[r], Ur = L.up[r];
            v = fma(-sd, fmin(fmax(vs * rs, Lr), Ur), vs);
            // an infinite bound side forces the dual's sign exactly
            if (isinf(Ur) && v > 0.0) v = 0.0;
            if (isinf(Lr) && v < 0.0) v = 0.0;
          } else {
            v = rs * fma(-sd, L.bF[r], vs);
          }
          L.ty[e] = v;
          if (!check) L.y[e] = a1 * ((1.0 + rho) * v - rho * yo) + a0 * L.y0[e];
        }
        done_reading(X, tid);

        if (check) {
          const long long tc0 = wall_clock64();
          const DevProblem& p = *opaque(pp);
          const DevState& s = *opaque(sp);
          const DevControl& ctl = *opaque(cp);
          __syncthreads();
          const bool val = lane < nwa;
          // sums: fixed-point residual, |dx|^2, |dy|^2, Phi's linear and quadratic part, costs,
          // conjugates, y_C offsets, |y|^2, time-out, non-finite count, dual-domain violation^2
          double v[NSC] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            if (t >= P) continue;
            L.xs[t * LDA + lane] = tx[j];
            const double w = dc * tx[j];
            if (val) {
              const double dx = x[j] - tx[j], dl = tx[j] - x0[j], wc = w - wT;
              v[0] = fma(omega * dx, dx, v[0]);
              v[1] = fma(dl, dl, v[1]);
              v[3] += -(al[j] - ar * wT) * w + 0.5 * ar * wc * wc;
              if (!isfinite(tx[j])) v[9] += 1.0;
            }
            const double bt = wave_sum(val ? fabs(w) : 0.0);   // the period's budget
            if (lane == 0) L.st[16 + t] = bt;
          }
          __syncthreads();
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            if (t > P) continue;
            const double drc = FFO_DRC(t), q = drc * ty[j];   // unscaled trade dual
            L.sC[t * LDA + lane] = q;
            if (!val) continue;
            const double dy = yc[j] - ty[j], dl = ty[j] - yc0[j];
            v[0] = fma(dy / omega, dy, v[0]);
            v[2] = fma(dl, dl, v[2]);
            const double xa = t < P ? L.xs[t * LDA + lane] : 0.0, xb = t > 0 ? L.xs[(t - 1) * LDA + lane] : 0.0;
            const double au = fabs(t == 0 ? dc * xa - w0 : t == P ? wT - dc * xb : dc * (xa - xb));
            v[4] += ca[j] * au + cb[j] * (d == 2.0 ? au * au : au * sqrt(au));
            v[5] += conj15(q, ca[j], cb[j], d);
            if (t == 0) v[6] += q * w0;
            if (t == P) v[6] -= q * wT;
            v[7] = fma(q, q, v[7]);
            if (cb[j] <= 0.0 && fabs(q) > ca[j]) { const double ex = fabs(q) - ca[j]; v[10] = fma(ex, ex, v[10]); }
            if (!isfinite(ty[j])) v[9] += 1.0;
          }
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            if (t >= P) continue;
            for (int r = lane; r < nr; r += 64) {
              const int e = t * S::LDY + r;
              const double tv = L.ty[e], dy = L.y[e] - tv, dl = tv - L.y0[e], yu = L.dr[r] * tv;
              L.dv[e] = r < m ? -dy : 0.0;
              if (wg != 0) continue;   // replicated row duals enter the sums once
              v[0] = fma(dy / omega, dy, v[0]);
              v[2] = fma(dl, dl, v[2]);
              v[7] = fma(yu, yu, v[7]);
              if (r < m && ((isinf(L.lo[r]) && yu < 0.0) || (isinf(L.up[r]) && yu > 0.0))) v[10] = fma(yu, yu, v[10]);
            }
          }
          if (wg == 0 && tid == 0) v[8] = (double)(wall_clock64() - t_start) / ctl.wall_hz > ctl.time_limit_s ? 1.0 : 0.0;
#pragma unroll
          for (int q = 0; q < NSC; ++q) {
            const double z = wave_sum(v[q]);
            if (lane == 0) L.red[16 * wave + q] = z;
          }
          kx<JT, NRT>(Kx, L.xs, L.st, P, nr, tid);
          kty<JT, NRT>(Kt, L.ty, L.R, P, tid);
          __syncthreads();
          if (tid < 16) {
            double z = 0.0;
            if (tid < NSC)
              for (int w = 0; w < NWV; ++w) z += L.red[16 * w + tid];
            L.st[tid] = z;
          }
          // dual inner problem: b' = alpha + arisk c - R' with R' = unscaled K^T Y at T(y), weights a' = arisk
          double bd[JT];
          const double iad = val ? 1.0 / ar : 0.0;
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            bd[j] = 0.0;
            if (t >= P) continue;
            bd[j] = val ? al[j] - (kty_at<JT, NRT>(L.R, P, t, lane) + adj(t, lane)) * idc : 0.0;
          }
          // sums and row products first; the dual multipliers follow in their own exchanges
          if (!exchange(X, L, P, nr, 0, oR + Pnr, 0, 0, tid)) goto fail;
          const double cv = total(X, L, lane < NSC ? lane : 0);
          double c1[NSC];
#pragma unroll
          for (int q = 0; q < NSC; ++q) c1[q] = uni(lane_of(cv, q));
          double rv[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            if (t >= P) continue;
            if (lane == 0) {
              const double ex = fmax(total(X, L, 16 + t) - 1.0, 0.0);
              rv[0] += ex * ex;
            }
            for (int r = lane; r < nr; r += 64) {
              const double dr = L.dr[r], w = total(X, L, oR + t * nr + r) / dr, yu = dr * L.ty[t * S::LDY + r];
              if (r < m) {
                const double Lr = L.lo[r], Ur = L.up[r], cl = fmin(fmax(w, Lr), Ur);
                rv[0] = fma(w - cl, w - cl, rv[0]);
                rv[1] = fma(cl, cl, rv[1]);
                if (yu > 0.0) rv[3] -= isinf(Ur) ? INFINITY : Ur * yu;
                else if (yu < 0.0) rv[3] -= isinf(Lr) ? INFINITY : Lr * yu;
              } else {
                const double bF = L.bF[r], g = w - bF;
                rv[2] = fma(g1 * g, g, rv[2]);
                rv[3] -= yu * bF + yu * yu / (4.0 * g1);
              }
            }
          }
          done_reading(X, tid);
          __syncthreads();
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double z = wave_sum(rv[q]);
            if (lane == 0) L.red[16 * wave + q] = z;
          }
          __syncthreads();
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            double z = 0.0;
#pragma unroll
            for (int w = 0; w < NWV; ++w) z += L.red[16 * w + q];
            rv[q] = uni(z);
          }
          {
            const double cq = point(D, 0, lane);
#pragma unroll
            for (int j = 0; j < JT; ++j) {
              const int t = wave + 8 * j;
              if (t < P) stats(fabs(bd[j]), iad, [&](int q) { return lane_of(cq, 8 * j + q); }, L.st + oD + NST * t, lane);
            }
          }
          if (!settle<JT, NRT>(D, X, L, P, nr, [&](int j) { return fabs(bd[j]); }, iad, tid)) goto fail;
          // inner value, and max_i |(A^T d)_i| per period for the infeasibility test (d = T(y_A) - y_A)
          const bool inf_test = ctl.infeas && m > 0;
          double iv = 0.0;
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            if (t >= P) continue;
            const double ab = fabs(bd[j]), mu = lane_of(D.mu, 8 * j), w = ab > mu ? copysign(iad, bd[j]) * (ab - mu) : 0.0;
            if (val) iv += 0.5 * w * w * ar - bd[j] * w;
          }
          predict_all(D);
          iv = wave_sum(iv);
          if (lane == 0) L.red[16 * wave + 4] = iv;
          if (inf_test) kty<JT, NRT>(Kt, L.dv, L.R, P, tid);
          __syncthreads();
          if (tid == 0) {
            double z = 0.0;
            for (int w = 0; w < NWV; ++w) z += L.red[16 * w + 4];
            L.st[0] = z;
          }
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            const int t = wave + 8 * j;
            if (t >= P) continue;
            const double am = inf_test ? wave_max(val ? fabs(kty_at<JT, NRT>(L.R, P, t, lane) * idc) : 0.0) : 0.0;
            if (lane == 0) L.st[1 + t] = am;
          }
          if (!exchange(X, L, P, nr, 0, 1 + P, 1, 1 + P, tid)) goto fail;
          const double inner = uni(total(X, L, 0));
          int infl = 0;
          if (inf_test) {   // a Farkas certificate for one period's feasible set (see solve_kernel.hip)
#pragma unroll
            for (int j = 0; j < JT; ++j) {
              const int t = wave + 8 * j;
              if (t >= P) continue;
              double sup = 0.0, mag = 0.0;
              for (int r = lane; r < m; r += 64) {
                const double du = L.dr[r] * L.dv[t * S::LDY + r];
                double term = 0.0;
                if (du > 0.0) term = isinf(L.up[r]) ? INFINITY : L.up[r] * du;
                else if (du < 0.0) term = isinf(L.lo[r]) ? INFINITY : L.lo[r] * du;
                sup += term;
                mag += fabs(term);
              }
              sup = wave_sum(sup);
              mag = wave_sum(mag);
              const double amax = total(X, L, 1 + t, true);
              if (amax + mag > 0.0 && sup + amax < -1e-9 * (mag + amax)) infl = 1;
            }
          }
          done_reading(X, tid);
          if (lane == 0) L.flag[wave] = infl;
          __syncthreads();
          int infeasible = 0;
#pragma unroll
          for (int w = 0; w < NWV; ++w) infeasible |= L.flag[w];
          const double phi = c1[3] + c1[4] + rv[2];
          const double psi = inner + (double)P * p.crisk[0] - c1[6] - c1[5] + rv[3];
          const double rel_pri = sqrt(rv[0]) / (1.0 + sqrt(rv[1]));
          const double rel_dual = sqrt(c1[10]) / (1.0 + sqrt(c1[7]));
          const double den = fabs(phi) + fabs(psi);
          const double rel_gap = den > 0.0 ? fabs(phi - psi) / den : 0.0;
          const double relkkt = fmax(rel_pri, fmax(rel_dual, rel_gap));
          const double fpr = sqrt(c1[0]);
          const bool nonfinite = c1[9] > 0.0 || !isfinite(phi) || !isfinite(psi) || !isfinite(rel_gap) || !isfinite(relkkt);
          if (tid == 0) ++L.flag[F_CHECKS];
          if (wg == 0 && tid == 0) {
            s.info[IX_RELKKT] = relkkt; s.info[IX_RELPRI] = rel_pri; s.info[IX_RELDUAL] = rel_dual;
            s.info[IX_RELGAP] = rel_gap; s.info[IX_FPR] = fpr; s.info[IX_POBJ] = phi; s.info[IX_DOBJ] = psi;
          }
          t_check += wall_clock64() - tc0;
          int st = DS_RUNNING;
          if (nonfinite) st = DS_NUMERIC;
          else if (infeasible) st = DS_INFEASIBLE;
          else if (relkkt <= ctl.tol) st = DS_OK;
          else if (c1[8] > 0.0) st = DS_TIMEOUT;
          else if (it + 1 >= ctl.max_iter) st = DS_NOT_CONVERGED;
          else {
            if (r0 < 0.0) r0 = uni(fpr);
            const bool rs = (fpr <= ctl.r_suff * r0) || (fpr <= ctl.r_nec * r0 && fpr > rprev) ||
                            ((double)kk + 1.0 >= ctl.r_art * (double)(it + 1));
            restart = __builtin_amdgcn_readfirstlane(rs);
            rprev = uni(fpr);
            kk = min(kk, 1u << 30);
            if (restart) {
              const double dxn = sqrt(c1[1]), dyn = sqrt(c1[2]);
              if (dxn > 1e-300 && dyn > 1e-300) omega = uni(sqrt(dyn / dxn) * sqrt(omega));   // half-way on a log scale
              r0 = uni(fpr);
              rprev = INFINITY;
              if (tid == 0) ++L.flag[F_RESTARTS];
              M.mprev = M.mu;   // a restart jumps the iterate: drop the multiplier trend
              predict_all(M);
            }
          }
          status = __builtin_amdgcn_readfirstlane(st);
          if (status != DS_RUNNING) {
            const bool bad = status == DS_NUMERIC;
#pragma unroll
            for (int j = 0; j < JT; ++j) {
              const int t = wave + 8 * j;
              const size_t e = (size_t)t * n + i0 + lane;
              if (val && t < P) s.w_out[e] = dc * (bad ? x0[j] : tx[j]);
              if (s.y_out && val && t <= P) s.y_out[(size_t)Pnr + e] = FFO_DRC(t) * (bad ? yc0[j] : ty[j]);
            }
            if (s.y_out && wg == 0)
              for (int e = tid; e < Pnr; e += NT) {
                const int t = e / nr, j = e - t * nr, f = t * S::LDY + j;
                // infeasible: the exposure part holds the certificate direction d of the test
                const double yu = L.dr[j] * (bad ? L.y0[f] : (status == DS_INFEASIBLE && j < m ? L.dv[f] : L.ty[f]));
                if (j < m) s.y_out[(size_t)t * m + j] = yu;
                else s.y_out[(size_t)P * m + (size_t)t * p.k + (j - m)] = yu;
              }
            ++it;
            if (wg == 0 && tid == 0) {
              const long long t_end = wall_clock64();
              s.info[IX_ITERS] = (double)it;
              s.info[IX_RESTARTS] = (double)L.flag[F_RESTARTS];
              s.info[IX_OMEGA] = omega;
              s.info[IX_ETA] = eta;
              s.info[IX_NORMK] = ctl.eta_safety / eta;
              s.info[IX_EXCHANGES] = (double)X.epoch;
              s.info[IX_CHECKS] = (double)L.flag[F_CHECKS];
              s.info[IX_MS_ROUNDS] = (double)L.flag[F_ROUNDS];
              s.info[IX_T_ITER] = (double)(t_end - t_loop) / ctl.wall_hz;
              s.info[IX_T_CHECK] = (double)t_check / ctl.wall_hz;
              s.info[IX_T_POWER] = (double)(t_loop - t_start) / ctl.wall_hz;
              s.status[0] = status;
            }
            return;
          }
          if (!restart)   // the row duals' Halpern step, put off above
#pragma unroll
            for (int j = 0; j < JT; ++j) {
              const int t = wave + 8 * j;
              if (t >= P) continue;
              for (int r = lane; r < nr; r += 64) {
                const int e = t * S::LDY + r;
                L.y[e] = a1 * ((1.0 + rho) * L.ty[e] - rho * L.y[e]) + a0 * L.y0[e];
              }
            }
        }
        // reflected Halpern step, or the restart at T(z)
        if (restart) {
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            x[j] = x0[j] = tx[j];
            yc[j] = yc0[j] = ty[j];
            const int t = wave + 8 * j;
            if (t >= P) continue;
            for (int r = lane; r < nr; r += 64) {
              const int e = t * S::LDY + r;
              L.y[e] = L.y0[e] = L.ty[e];
            }
          }
          kk = 0;
        } else {
#pragma unroll
          for (int j = 0; j < JT; ++j) {
            x[j] = a1 * ((1.0 + rho) * tx[j] - rho * x[j]) + a0 * x0[j];
            yc[j] = a1 * ((1.0 + rho) * ty[j] - rho * yc[j]) + a0 * yc0[j];
          }
          ++kk;
        }
#pragma unroll
        for (int j = 0; j < JT; ++j)
          if (wave + 8 * j <= P) L.sC[(wave + 8 * j) * LDA + lane] = FFO_DRC(wave + 8 * j) * yc[j];
        ++it;
        __syncthreads();
      }
    }
  }
fail:
  if (tid0 == 0) __hip_atomic_store(s.status, (int32_t)DS_BARRIER, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#undef FFO_DRC
}

}  // namespace

static const void* mp_fn(int jt, int nrt) {
#define FFO_MP(J, R) if (jt == J && nrt == R) return (const void*)k_mp<J, R>;
  FFO_MP(1, 2) FFO_MP(1, 3) FFO_MP(1, 5) FFO_MP(1, 7)
  FFO_MP(2, 2) FFO_MP(2, 3) FFO_MP(2, 5) FFO_MP(2, 7)
  FFO_MP(3, 2) FFO_MP(3, 3) FFO_MP(3, 5) FFO_MP(3, 7)
  FFO_MP(4, 2) FFO_MP(4, 3) FFO_MP(4, 5) FFO_MP(4, 7)
#undef FFO_MP
  return nullptr;
}

static size_t mp_lds_doubles(int jt, int nrt, int P, int nr) {
#define FFO_MP(J, R) if (jt == J && nrt == R) return Lds<J, R>::doubles(P, nr);
  FFO_MP(1, 2) FFO_MP(1, 3) FFO_MP(1, 5) FFO_MP(1, 7)
  FFO_MP(2, 2) FFO_MP(2, 3) FFO_MP(2, 5) FFO_MP(2, 7)
  FFO_MP(3, 2) FFO_MP(3, 3) FFO_MP(3, 5) FFO_MP(3, 7)
  FFO_MP(4, 2) FFO_MP(4, 3) FFO_MP(4, 5) FFO_MP(4, 7)
#undef FFO_MP
  return 0;
}

bool mp_plan(int64_t n, int nr, int P, int cus, size_t lds_cap, MpPlan* out) {
  if (P + 1 > 32 || nr > 112) return false;
  out->jt = (P + 1 + 7) / 8;
  out->nrt = nr <= 32 ? 2 : nr <= 48 ? 3 : nr <= 80 ? 5 : 7;
  out->nwg = (int)std::min<int64_t>((n + NA - 1) / NA, 1 << 20);
  out->vmax = off_rows(P) + P * nr;
  out->lds = mp_lds_doubles(out->jt, out->nrt, P, nr) * sizeof(double);
  return out->nwg <= cus && out->lds <= lds_cap;
}

int launch_mp(const MpPlan& pl, const DevProblem* dp, const DevState* ds, const DevControl* dc, void* stream) {
  void* args[] = {(void*)&dp, (void*)&ds, (void*)&dc};
  const hipError_t e = hipLaunchCooperativeKernel(mp_fn(pl.jt, pl.nrt), dim3(pl.nwg), dim3(NT), args, (unsigned)pl.lds,
                                                  (hipStream_t)stream);
  return e == hipSuccess ? 0 : (int)e;
}

}  // namespace ffo
