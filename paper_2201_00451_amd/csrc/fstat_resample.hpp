// Steps (iii)-(v) of Sec. 3 and the weighting of step (vi), fused.
//
// One workgroup owns kResTile consecutive points of the regular source-frame
// grid tau_k = tau0 + k dt of one template.  For each detector it
//   1. stages the ephemeris intervals the tile can touch in LDS: the cubic
//      Hermite of each interval, from its two nodes projected on the sky
//      direction (n.r, n.v), as power-series coefficients, so every later
//      delay evaluation is three FMAs on LDS data;
//   2. solves the detector epochs T_k of step (iv) for the thread's own grid
//      points (FP64): the tile's first point by a fixed-point and a Newton
//      step, every other point by one Newton step from the first point's
//      solution extrapolated along dT/dtau; T_k is monotonic in k, so the
//      tile's first and last points bound the input samples it touches;
//   3. stages those samples in LDS after the step (iii) heterodyne correction
//      z_j = x_j exp(-2 pi i f_h (t_src,j - t_j)) (FP64 delay, split
//      exactly into quarter turns and an FP32 remainder, polynomial
//      rotation): each input sample is read from HBM
//      and corrected once per tile;
//   4. interpolates z at T_k with the 2D-tap Hann-windowed sinc
//      h(s) = sinc(s) (1 + cos(pi s / D)) / 2 (the paper leaves the kernel of
//      step (v) unnamed) and accumulates w_X a'(T_k) zhat_k, w_X b'(T_k) zhat_k
//      with the whitened antenna patterns of the template.
// Finally it removes the spin-down phase Phi_s(tau_k) and the sub-bin offset
// df (FP64 phase, FP32 rotation) and writes y_a', y_b' (float2) with
// coalesced stores.  FP64 is used only for times and phases.
//
// The half-width D is a template parameter: the taps are polynomials in the
// point's fraction f with compile-time coefficients (make_tap_poly).
#pragma once

#include <utility>

#include "fstat_common.hpp"

namespace fstat {

// Window constants of half-width D for the point-by-point gradient tiles,
// built at compile time into constant memory (read with uniform indices,
// whether or not the tap loop is unrolled): with c_t = D - 1 - t,
// Ct_t = cos(pi c_t / D), St_t = sin(pi c_t / D).
struct TapConst {
  float Ct[32], St[32];
};
template <int D>
__host__ __device__ constexpr TapConst make_taps() {
  TapConst k{};
  for (int t = 0; t < 2 * D; ++t) {
    const int c = D - 1 - t;
    k.Ct[t] = float(ct_cospi(c, D));
    k.St[t] = float(ct_sinpi(c, D));
  }
  return k;
}
template <int D>
__constant__ TapConst kTaps = make_taps<D>();

// The forward interpolation's taps as polynomials.  With g = f - 1/2 in
// [-1/2, 1/2] the taps at the offsets s = f + m and s = f - 1 - m (m = 0 ..
// D - 1) are h(g + m + 1/2) and, h being even, h(-g + m + 1/2): the pair is
// E_m(g^2) +- g O_m(g^2) with E_m and O_m the even and odd parts of one
// polynomial in g.  make_tap_poly builds it at compile time in FP64: the
// Chebyshev interpolant of h on 16 nodes, cut at degree 9 (8 for the outer
// quarter of the pairs, where the window is small), which is within 2e-8 of h;
// with the FP32 Horner evaluation a tap is within 1.0e-7 at D = 8 and 1.6e-7 at
// every D (the closed form sin(pi f) w(s) / s reaches 2e-7).  A pair costs 12
// operations (11 in the outer quarter) of 2.3-2.8 cycles each where the closed form cost two reciprocals (8.2 cycles each),
// four window FMAs and two products, and nothing per point besides g^2: no
// sine of the offset, no window phase, no special case at f = 0.
constexpr int kTapCoef = 5;
struct TapPoly {
  float e[kTapCoef], o[kTapCoef];
};
template <int D>
__host__ __device__ constexpr int tap_odd_terms(int m) {
  return m >= (3 * D + 3) / 4 ? kTapCoef - 1 : kTapCoef;
}
// DERIV: the same for the derivative dh/ds (within 5e-8 of it per unit of its
// largest value, pi/2): the pair is then E_m(g^2) + g O_m(g^2) and, h' being
// odd, g O_m(g^2) - E_m(g^2).
template <int D, int M, bool DERIV = false>
__host__ __device__ constexpr TapPoly make_tap_poly() {
  constexpr int K = 16, N = 2 * kTapCoef;  // nodes; coefficients of g^0 .. g^9
  double y[K] = {}, cheb[N] = {}, t0[N] = {}, t1[N] = {}, mono[N] = {};
  for (int k = 0; k < K; ++k) {
    const double g = 0.5 * ct_cospi(2 * k + 1, 2 * K);
    const double s = g + M + 0.5;
    // sin(pi s) = (-1)^M cos(pi g)
    const double sgn = (M & 1) ? -1.0 : 1.0;
    const double sinc = sgn * ct_poly_cos(kPi * g) / (kPi * s);
    const double win = 0.5 * (1.0 + ct_poly_cos(kPi * s / D));
    y[k] = sinc * win;
    if (DERIV)  // cos(pi s) = -(-1)^M sin(pi g)
      y[k] = (-sgn * ct_poly_sin(kPi * g) - sinc) / s * win -
             sinc * 0.5 * kPi / D * ct_poly_sin(kPi * s / D);
  }
  const int deg = DERIV ? 2 * kTapCoef - 1 : kTapCoef - 1 + tap_odd_terms<D>(M);
  for (int j = 0; j <= deg; ++j) {
    for (int k = 0; k < K; ++k) cheb[j] += y[k] * ct_cospi(j * (2 * k + 1), 2 * K);
    cheb[j] *= (j == 0 ? 1.0 : 2.0) / K;
  }
  // sum of cheb[j] T_j(x), x = 2 g, in powers of g
  t0[0] = 1.0;
  t1[1] = 2.0;
  for (int i = 0; i < N; ++i) mono[i] = cheb[0] * t0[i] + cheb[1] * t1[i];
  for (int j = 2; j <= deg; ++j) {
    double t2[N] = {};
    for (int i = 0; i < N; ++i) t2[i] = (i > 0 ? 4.0 * t1[i - 1] : 0.0) - t0[i];
    for (int i = 0; i < N; ++i) {
      mono[i] += cheb[j] * t2[i];
      t0[i] = t1[i];
      t1[i] = t2[i];
    }
  }
  TapPoly p{};
  for (int i = 0; i < kTapCoef; ++i) {
    p.e[i] = float(mono[2 * i]);
    p.o[i] = float(mono[2 * i + 1]);
  }
  return p;
}

// The two taps of pair M at g (u = g^2).
template <int D, int M>
__device__ __forceinline__ void tap_pair(float g, float u, float& hp, float& hm) {
  constexpr TapPoly p = make_tap_poly<D, M>();
  constexpr int no = tap_odd_terms<D>(M);
  // the first step as a product and a sum: an FMA takes one literal, so two
  // would keep the leading coefficients of every pair in registers
  float e = __fmul_rn(u, p.e[kTapCoef - 1]), o = __fmul_rn(u, p.o[no - 1]);
  e = __fadd_rn(e, p.e[kTapCoef - 2]);
  o = __fadd_rn(o, p.o[no - 2]);
#pragma unroll
  for (int i = kTapCoef - 3; i >= 0; --i) e = fmaf(e, u, p.e[i]);
#pragma unroll
  for (int i = no - 3; i >= 0; --i) o = fmaf(o, u, p.o[i]);
  hp = fmaf(g, o, e);
  hm = fmaf(-g, o, e);
}
template <int D, int M>
__device__ __forceinline__ void interp_pair(float g, float u, const float2* zp, float& sx,
                                            float& sy) {
  float hp, hm;
  tap_pair<D, M>(g, u, hp, hm);
  const float2 zl = zp[D - 1 - M], zr = zp[D + M];
  sx = fmaf(hp, zl.x, sx);
  sy = fmaf(hp, zl.y, sy);
  sx = fmaf(hm, zr.x, sx);
  sy = fmaf(hm, zr.y, sy);
}
template <int D, int... M>
__device__ __forceinline__ void interp_pairs(std::integer_sequence<int, M...>, float g, float u,
                                             const float2* zp, float& sx, float& sy) {
  // outer pairs first
  (interp_pair<D, D - 1 - M>(g, u, zp, sx, sy), ...);
}

// Step (v): the 2D-tap interpolation of the samples zp[0 .. 2D) at the
// fraction f of the point between zp[D - 1] and zp[D].
template <int D>
__device__ __forceinline__ float2 sinc_interp(float f, const float2* zp) {
  const float g = f - 0.5f;
  float sx = 0.f, sy = 0.f;
  interp_pairs<D>(std::make_integer_sequence<int, D>{}, g, g * g, zp, sx, sy);
  return make_float2(sx, sy);
}

// The weighting of step (vi): the whitened antenna patterns of detector X
// at T = tau + q dt times the interpolated value, added to acc_a, acc_b.
__device__ __forceinline__ void weight_add(const PlanConst& P, const TmplParams& tp, int X,
                                           double tau, double q, float2 zh, float2& acc_a,
                                           float2& acc_b) {
  // x = alpha - phi(T), in cycles
  const float2 ex = cis_cycles(tp.alpha_cyc[X] - P.sid_rate_cyc * (tau + q * P.dt));
  const float cx = ex.x, sx = ex.y;
  const float c2 = cx * cx - sx * sx, s2 = 2.0f * sx * cx;
  const float a = tp.ca[X][0] + tp.ca[X][1] * cx + tp.ca[X][2] * sx + tp.ca[X][3] * c2 +
                  tp.ca[X][4] * s2;
  const float b = tp.cb[X][0] + tp.cb[X][1] * cx + tp.cb[X][2] * sx + tp.cb[X][3] * c2 +
                  tp.cb[X][4] * s2;
  acc_a.x = fmaf(a, zh.x, acc_a.x);
  acc_a.y = fmaf(a, zh.y, acc_a.y);
  acc_b.x = fmaf(b, zh.x, acc_b.x);
  acc_b.y = fmaf(b, zh.y, acc_b.y);
}

// The first tap of grid point k_s + kk in the staged window (start lo, W
// samples): u = k + off + q = j0 + f, taps j0-D+1 .. j0+D; monotonic T_k keeps
// them inside the window, the clamp only guards memory.
template <int D>
__device__ __forceinline__ int tap_base(const PlanConst& P, int X, int64_t lo, int W,
                                        int64_t k_s, int kk, double q, float& f) {
  int64_t j0;
  split_u(double(k_s + kk) + P.det[X].off + q, j0, f);
  const int base = int(j0 - lo) - (D - 1);
  return base < 0 ? 0 : (base > W - 2 * D ? W - 2 * D : base);
}
// Whether any tap from base on falls on a live sample (block flags blk).
template <int D>
__device__ __forceinline__ bool taps_live(const int32_t* blk, int base) {
  return (blk[base >> 5] | blk[(base + 2 * D - 1) >> 5]) != 0;
}

// Steps (v) and the weighting of (vi) at one grid point k_s + kk of detector
// X, whose epoch is T_k = tau_k + q dt, from the staged window zs.  A point
// whose taps all fall on zero samples adds nothing.
template <int D>
__device__ __forceinline__ void interp_point(const PlanConst& P, const TmplParams& tp, int X,
                                             const float2* zs, const int32_t* blk, int64_t lo,
                                             int W, int64_t k_s, int kk, double q, double tau_s,
                                             float2& acc_a, float2& acc_b) {
  float f;
  const int base = tap_base<D>(P, X, lo, W, k_s, kk, q, f);
  if (!taps_live<D>(blk, base)) return;
  weight_add(P, tp, X, tau_s + P.dt * double(kk), q, sinc_interp<D>(f, zs + base), acc_a, acc_b);
}

// The whitened antenna patterns of detector X over one tile as quintic
// polynomials in the sidereal angle's offset d from the tile's middle point:
// with x = alpha - phi(T), a(x) = ca0 + ca1 cos x + ca2 sin x + ca3 cos 2x
// + ca4 sin 2x has the Taylor coefficients a_n = a^(n)(x_r) / n! at x_r
// (and b likewise).  The remainder is below (2|d|)^6 / 6! of the coefficients'
// scale, 1e-7 at |d| = 0.1 rad, the bound kTaylorMaxAngle under which the
// tile takes this form.  c[0..5]: a_0..a_5, c[6..11]: b_0..b_5.
constexpr int kTaylorCoef = 12;
static_assert(kTaylorCoef + 2 <= kTileRecUnits * 4, "a tile record holds the coefficients");
__device__ inline void antenna_taylor(const float* ka, const float* kb, double x_cyc,
                                      float (&c)[kTaylorCoef]) {
  const float2 e = cis_cycles(x_cyc);
  const float c1 = e.x, s1 = e.y;
  const float c2 = c1 * c1 - s1 * s1, s2 = 2.0f * s1 * c1;
#pragma unroll
  for (int ab = 0; ab < 2; ++ab) {
    const float* k = ab ? kb : ka;
    // value p and derivative q of the first and second harmonic at x_r
    const float p1 = k[1] * c1 + k[2] * s1, q1 = k[2] * c1 - k[1] * s1;
    const float p2 = k[3] * c2 + k[4] * s2, q2 = k[4] * c2 - k[3] * s2;
    float* o = c + 6 * ab;
    o[0] = k[0] + p1 + p2;
    o[1] = q1 + 2.0f * q2;
    o[2] = -(p1 + 4.0f * p2) * (1.0f / 2.0f);
    o[3] = -(q1 + 8.0f * q2) * (1.0f / 6.0f);
    o[4] = (p1 + 16.0f * p2) * (1.0f / 24.0f);
    o[5] = (q1 + 32.0f * q2) * (1.0f / 120.0f);
  }
}

// q = (T_k - tau_k)/dt at grid offset k within its knot interval from the
// interval's two knots (value, derivative per grid step) G steps apart.
__device__ __forceinline__ double knot_hermite(const double2* kn, int G, double u) {
  double2 c[2];
  hermite_interval(kn[0], kn[1], double(G), c[0], c[1]);
  return hermite_eval(c, 0, u);
}

// A value every lane of the wave holds, moved to scalar registers.
__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
  const uint64_t u = uint64_t(v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(u));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(u >> 32));
  return int64_t((uint64_t(hi) << 32) | lo);
}

// Steps (iii)-(v) and the antenna weighting for the kResTile grid points of
// the tile starting at k_s: acc_a[i], acc_b[i] receive sum_X a'_X(T_k)
// zhat_X(u_k) (and b'), k = k_s + tid + i kResThreads, before the spin-down
// phase.  Returns false, after flagging the template's status word, when the
// template must report NaN (the return is uniform across the block).
//
// Detectors are taken kDetPass at a time, each pass in five phases separated
// by barriers: (1) the pass's ephemeris intervals, and the binary delay at
// the grid knots; (2) the detector epochs at the grid knots; (3) each
// detector's staged window from them, the loads of its input samples, and the
// heterodyne phase at the sample knots while those loads are in flight;
// (4) the corrected samples into LDS; (5) interpolation and weighting.
//
// Timing (tp.knot_log2 = log2 G > 0): the grid delays q_k = (T_k - tau_k)/dt
// are solved exactly at every G-th grid point of the tile and its end, the
// heterodyne phases f_h (t_src,j - t_j) at every G-th staged sample, each
// with its derivative, and every point in between takes the cubic Hermite of
// its interval (FP64).  G is chosen per template so that the interpolation
// error stays below 2e-7 cycles of phase and 1e-7 samples of grid position.
// knot_log2 = 0: every grid point and sample is solved.
// Zero samples (gaps, and outside the data) are staged as zeros without any
// timing; a wave whose outputs' taps all fall on zero samples skips the
// interpolation (it would add zeros).
template <int D, bool KEP>
__device__ inline bool resample_tile(const PlanConst& P, const TmplParams& tp,
                                     int32_t* status_word, int64_t k_s, float2* zsa,
                                     int32_t* blka, float2 (&acc_a)[kResPerThread],
                                     float2 (&acc_b)[kResPerThread]) {
  constexpr int kRounds = (kResWcap + kResThreads - 1) / kResThreads;
  const int tid = threadIdx.x;
  __shared__ double2 coef[kDetPass][2 * kNodeCap];
  __shared__ double2 orb[kGridKnots];  // binary delay and rate at the grid knots
  // knot path: grid knots (q, dq/dk) of each detector, then its sample knots
  // (phase, dphase/dj); exact path: q of every grid point of each detector
  __shared__ double2 kbuf[kDetPass * (kGridKnots + kSampKnots)];
  __shared__ int bad;
  static_assert(kDetPass * (kGridKnots + kSampKnots) * 2 >= kDetPass * kResTile,
                "exact-path delays must fit the knot buffer");
  double2* const gk = kbuf;                          // [kDetPass][kGridKnots]
  double2* const sk = kbuf + kDetPass * kGridKnots;  // [kDetPass][kSampKnots]
  double* const qx = reinterpret_cast<double*>(kbuf);  // [kDetPass][kResTile]

  if (tid == 0) bad = 0;
  bool oob = false;
#pragma unroll
  for (int i = 0; i < kResPerThread; ++i) {
    acc_a[i] = make_float2(0.f, 0.f);
    acc_b[i] = make_float2(0.f, 0.f);
  }
  const int kl = tp.knot_log2;
  const bool knots = kl != 0;
  const int G = 1 << kl;
  const double inv_g = 1.0 / double(G);
  const int nkg = kResTile / G + 1;
  // time span any delay evaluation of this tile can reach (sample knots run
  // up to G samples past the staged window)
  const double pad = P.max_delay + double(D + 2 + (1 << kKnotLogMax)) * P.dt;
  const double t_first = P.tau0 + P.dt * double(k_s) - pad;
  const double t_last = P.tau0 + P.dt * double(k_s + kResTile - 1) + pad;
  int64_t n_lo = int64_t(floor((t_first - P.eph_t0) * P.inv_eph_dt)) - 1;
  n_lo = n_lo < 0 ? 0 : (n_lo > P.n_eph - 2 ? P.n_eph - 2 : n_lo);
  int64_t n_hi = int64_t(floor((t_last - P.eph_t0) * P.inv_eph_dt)) + 2;
  n_hi = n_hi > P.n_eph - 1 ? P.n_eph - 1 : n_hi;
  int n_count = int(n_hi - n_lo + 1);
  n_count = n_count > kNodeCap ? kNodeCap : (n_count < 2 ? 2 : n_count);
  const double node_t0 = P.eph_t0 + double(n_lo) * P.eph_dt;
  const double tau_s = P.tau0 + P.dt * double(k_s);
  // exact path: the binary delay at the own grid points (all detectors)
  double rbk[kResPerThread];
  double rb0 = 0.0;
  if (!knots) {
    rb0 = binary_delay<KEP>(tp, tau_s);
#pragma unroll
    for (int i = 0; i < kResPerThread; ++i)
      rbk[i] = binary_delay<KEP>(tp, tau_s + P.dt * double(tid + i * kResThreads));
  }

  for (int X0 = 0; X0 < P.ndet; X0 += kDetPass) {
    const int np = P.ndet - X0 < kDetPass ? P.ndet - X0 : kDetPass;
    // 1. interval coefficients from the projected nodes i and i + 1 of each
    // detector of the pass; the binary delay and its rate at the grid knots
    {
      const int ni = n_count - 1;
      for (int e = tid; e < np * ni; e += kResThreads) {
        const int xp = e >= ni ? 1 : 0;
        const int i = e - xp * ni;
        const double* n = P.det[X0 + xp].ephem + 6 * (n_lo + i);
        const double p0 = tp.nhat[0] * n[0] + tp.nhat[1] * n[1] + tp.nhat[2] * n[2];
        const double v0 = tp.nhat[0] * n[3] + tp.nhat[1] * n[4] + tp.nhat[2] * n[5];
        const double p1 = tp.nhat[0] * n[6] + tp.nhat[1] * n[7] + tp.nhat[2] * n[8];
        const double v1 = tp.nhat[0] * n[9] + tp.nhat[1] * n[10] + tp.nhat[2] * n[11];
        cubic_interval(p0, v0, p1, v1, P.eph_dt, coef[xp][2 * i], coef[xp][2 * i + 1]);
      }
      if (knots && X0 == 0 && tid < nkg) {
        double r, rp;
        orbit_delay<KEP>(tp, tau_s + P.dt * double(tid * G), r, rp);
        orb[tid] = make_double2(r, rp);
      }
    }
    __syncthreads();
    // 2. detector epochs as q = (T - tau)/dt: at the grid knots (fixed point
    // and three Newton steps, with dq/dk = (R'(tau) - roemer'(T)) /
    // (1 + roemer'(T))), or at every own grid point (the tile's first point
    // in full, the rest by one Newton step from a prediction that carries the
    // exact binary delay and linearises the Roemer delay about the first
    // point: T ~ T_s + (t_b - t_b,s) / (1 + roemer'(T_s)))
    if (knots) {
      for (int e = tid; e < np * nkg; e += kResThreads) {
        const int xp = e >= nkg ? 1 : 0;
        const int t = e - xp * nkg;
        const CubicRoemer re{coef[xp], n_count, node_t0, P.inv_eph_dt};
        const double tau = tau_s + P.dt * double(t * G);
        const double2 o = orb[t];
        double x;
        double dl = grid_delay_rb(re, o.x, tau, oob);
        dl = grid_delay_newton(re, tau, o.x, dl, x, oob);
        dl = grid_delay_newton(re, tau, o.x, dl, x, oob);
        gk[xp * kGridKnots + t] = make_double2(dl * P.inv_dt, (o.y - x) / (1.0 + x));
      }
    } else {
      for (int xp = 0; xp < np; ++xp) {
        const CubicRoemer re{coef[xp], n_count, node_t0, P.inv_eph_dt};
        double x0;
        double d0 = grid_delay_rb(re, rb0, tau_s, oob);
        d0 = grid_delay_newton(re, tau_s, rb0, d0, x0, oob);
        d0 = grid_delay_newton(re, tau_s, rb0, d0, x0, oob);
        const double inv0 = 1.0 - x0 * (1.0 - x0 * (1.0 - x0));
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i) {
          const int kk = tid + i * kResThreads;
          const double dtau = P.dt * double(kk);
          const double guess = d0 + (dtau + rbk[i] - rb0) * inv0 - dtau;
          double x;
          qx[xp * kResTile + kk] =
              grid_delay_newton(re, tau_s + dtau, rbk[i], guess, x, oob) * P.inv_dt;
        }
      }
    }
    __syncthreads();
    // 3. each detector's staged window from its first and last epochs (T_k
    // is monotonic in k; the knot path bounds the last point by the knot
    // just past the tile), the loads of its samples, and the heterodyne
    // phase at its sample knots while they are in flight
    int64_t lo[kDetPass];
    int W[kDetPass];
    bool wbad = false;
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      lo[xp] = 0;
      W[xp] = 0;
      if (xp >= np) continue;
      const double q0 = knots ? gk[xp * kGridKnots].x : qx[xp * kResTile];
      const double q1 = knots ? gk[xp * kGridKnots + nkg - 1].x : qx[xp * kResTile + kResTile - 1];
      const int64_t k1 = knots ? k_s + kResTile : k_s + kResTile - 1;
      int64_t j_first, j_last;
      float f;
      split_u(double(k_s) + P.det[X0 + xp].off + q0, j_first, f);
      split_u(double(k1) + P.det[X0 + xp].off + q1, j_last, f);
      // every thread computes the same window from LDS: keep it in scalar
      // registers
      lo[xp] = uniform_i64(j_first - D + 1);
      const int64_t nwin = j_last + D - lo[xp] + 1;
      // delay drift beyond 1/16 per tile: flag the template (NaN output)
      if (nwin > kResWcap || nwin < 2 * D) wbad = true;
      W[xp] = __builtin_amdgcn_readfirstlane(int(nwin));
    }
    if (wbad) {
      if (tid == 0) atomicOr(status_word, kStatusWindow);
      return false;
    }
    float2 xv[kDetPass][kRounds];
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      const DetConst& d = P.det[X0 + (xp < np ? xp : 0)];
#pragma unroll
      for (int r = 0; r < kRounds; ++r) {
        const int w = r * kResThreads + tid;
        const int64_t j = lo[xp] + w;
        xv[xp][r] = (xp < np && w < W[xp] && j >= 0 && j < d.n) ? d.x[j] : make_float2(0.f, 0.f);
      }
    }
    if (knots) {
      const int nks0 = ((W[0] - 1) >> kl) + 2;
      const int nks1 = np > 1 ? ((W[1] - 1) >> kl) + 2 : 0;
      for (int e = tid; e < nks0 + nks1; e += kResThreads) {
        const int xp = e >= nks0 ? 1 : 0;
        const int t = e - xp * nks0;
        const CubicRoemer re{coef[xp], n_count, node_t0, P.inv_eph_dt};
        double ph, dph;
        const int64_t lox = xp ? lo[1] : lo[0];
        sample_phase<KEP>(re, tp, P.det[X0 + xp].t0 + P.dt * double(lox + int64_t(t) * G),
                          P.f_het, ph, dph, oob);
        sk[xp * kSampKnots + t] = make_double2(ph, dph * P.dt);
      }
    }
    __syncthreads();
    // 4. corrected input samples z_j = x_j exp(-2 pi i f_h (t_src,j - t_j));
    // a zero sample (outside the data, or in a gap) stays zero, untimed
#pragma unroll 1
    for (int xp = 0; xp < np; ++xp) {
      const CubicRoemer re{coef[xp], n_count, node_t0, P.inv_eph_dt};
      const int64_t lox = xp ? lo[1] : lo[0];
      const int Wx = xp ? W[1] : W[0];
#pragma unroll
      for (int r = 0; r < kRounds; ++r) {
        const int w = r * kResThreads + tid;
        if (r * kResThreads >= Wx) break;
        const float2 x = xp ? xv[1][r] : xv[0][r];
        const bool live = x.x != 0.f || x.y != 0.f;
        float2 z = make_float2(0.f, 0.f);
        if (live) {
          double ph;
          if (knots) {
            ph = knot_hermite(sk + xp * kSampKnots + (w >> kl), G, double(w & (G - 1)) * inv_g);
          } else {
            ph = P.f_het * sample_delay<KEP>(re, tp, P.det[X0 + xp].t0 + P.dt * double(lox + w),
                                             oob);
          }
          const float2 e = cis_cycles(ph);
          // x * exp(-2 pi i f_h dl)
          z = make_float2(x.x * e.x + x.y * e.y, x.y * e.x - x.x * e.y);
        }
        if (w < Wx) zsa[xp * kResWcap + w] = z;
        // which 32-sample blocks of the window hold a live sample
        const unsigned long long m = __ballot(live);
        if ((tid & 63) == 0) {
          const int b = w >> 5;
          blka[xp * kResBlk + b] = uint32_t(m) != 0u;
          blka[xp * kResBlk + b + 1] = uint32_t(m >> 32) != 0u;
        }
      }
    }
    __syncthreads();
    // 5. interpolation and antenna weighting (each accumulator takes the
    // detectors in order)
#pragma unroll 1
    for (int xp = 0; xp < np; ++xp) {
      const int X = X0 + xp;
      const int64_t lox = xp ? lo[1] : lo[0];
      const int Wx = xp ? W[1] : W[0];
#pragma unroll
      for (int i = 0; i < kResPerThread; ++i) {
        const int kk = tid + i * kResThreads;
        const double q = knots ? knot_hermite(gk + xp * kGridKnots + (kk >> kl), G,
                                              double(kk & (G - 1)) * inv_g)
                               : qx[xp * kResTile + kk];
        interp_point<D>(P, tp, X, zsa + xp * kResWcap, blka + xp * kResBlk, lox, Wx, k_s, kk, q,
                        tau_s, acc_a[i], acc_b[i]);
      }
    }
    if (X0 + kDetPass < P.ndet) __syncthreads();
  }
  if (oob) bad = 1;
  __syncthreads();
  if (bad) {
    // a delay evaluation left the staged ephemeris nodes: the delay exceeds
    // the plan's max_delay; flag the template (NaN output)
    if (tid == 0) atomicOr(status_word, kStatusNodes);
    return false;
  }
  return true;
}

// Reads of memory that no thread of the running kernel writes, at an address
// uniform across the wave: scalar loads (one per wave instead of one per
// lane through the vector memory path).
template <class T>
__device__ __forceinline__ T scalar_load(const T* p) {
  return *reinterpret_cast<const __attribute__((address_space(4))) T*>(
      reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ int32_t uniform_i32(int32_t v) {
  return __builtin_amdgcn_readfirstlane(v);
}

// The weighting of step (vi) with the antenna patterns from the tile's Taylor
// coefficients c (uniform across the tile) at the angle offset d (radians).
__device__ __forceinline__ void weight_taylor(float2 zh, float d, const float* c, float2& acc_a,
                                              float2& acc_b) {
  float a = c[5], b = c[11];
#pragma unroll
  for (int n = 4; n >= 0; --n) {
    a = fmaf(a, d, c[n]);
    b = fmaf(b, d, c[6 + n]);
  }
  acc_a.x = fmaf(a, zh.x, acc_a.x);
  acc_a.y = fmaf(a, zh.y, acc_a.y);
  acc_b.x = fmaf(b, zh.x, acc_b.x);
  acc_b.y = fmaf(b, zh.y, acc_b.y);
}

// The heterodyne correction of one sample at t samples into its interval:
// x exp(-2 pi i f_h (t_src - t_det)), the phase in quarter turns from the
// interval's record (k0, k1, k2, k3).
__device__ __forceinline__ float2 correct_sample(float2 x, double t, double k0, double k1,
                                                 double k2, double k3) {
  const double c4 = fma(fma(fma(k3, t, k2), t, k1), t, k0);
  const double q = rint(c4);
  const float2 e = cis_quarter(int(q), static_cast<float>(c4 - q));
  return make_float2(x.x * e.x + x.y * e.y, x.y * e.x - x.x * e.y);
}

// What a span's block keeps in LDS per detector besides its window: the records
// of the sample and grid intervals it touches, the tiles' Taylor records, and
// the window's block flags.
struct alignas(16) SpanRec {
  double2 samp[kSpanSamp][2];
  float4 grid[kSpanGrid];
  float tile[kSpanTiles][kTileRecUnits * 4];
  int32_t grid_i[kSpanGrid];
  int32_t blk[kSpanBlk];
};
__host__ __device__ inline size_t span_lds_bytes(int ndet) {
  return size_t(ndet) * (kSpanCap * sizeof(float2) + sizeof(SpanRec));
}
static_assert(kSpanCap % 2 == 0, "records behind the windows stay 16-byte aligned");
static_assert(kMaxDet * 64 <= kResThreads && kSpanGrid <= 40 && kSpanTiles * kTileRecUnits <= 24,
              "64 threads load a detector's grid and tile records");
static_assert(kDetPass * 128 <= kResThreads && 2 * kSpanSamp <= 128,
              "128 threads load a detector's sample records");

// Templates whose timing knots k_timing solved ahead (knot area kn): a block
// takes a span of n_t tiles starting at tile t0.  The span's samples of every
// detector go into LDS corrected, then each tile is interpolated and weighted
// from the interval records.  A detector's window runs from the span's first
// source position to the one of the interval just past it (T_k is monotonic in
// k); it starts at a multiple of the coarsest knot spacing, so at an interval.
// The grid points take their source positions from the FP32 interval cubics
// relative to the intervals' integers, and (plans with res_taylor) the antenna
// patterns from the tile's Taylor record, so the interpolation runs without
// FP64 arithmetic.
//
// Bound by latency before it is bound by arithmetic: every record and sample
// is a first touch (a miss of L2), so the span waits for memory twice, once for
// the window's edges (with the grid and tile records in flight beside them)
// and once for the samples and their records; everything later reads LDS.
// Measured on 32 templates of 5.2 M points and two detectors, after a tile per
// block that read its records where it used them (2245 us): records in LDS and
// loads batched 2120 us, two tiles per block 1720 us, six waves per SIMD
// instead of five 1675 us (24 bytes spilled); of the time without arithmetic
// (1180 us with taps, corrections, sample loads and stores taken out) most was
// the chain of dependent misses.
// store(k, acc_a, acc_b) receives every point.  Returns false, after flagging
// the template's status word, when the template must report NaN (the return
// is uniform across the block).
template <int D, class Store>
__device__ __forceinline__ bool resample_span(const PlanConst& P, const TmplParams& tp,
                                              const double2* __restrict__ kn, int kl,
                                              int32_t* status_word, int32_t t0, int n_t,
                                              float2* zsa, SpanRec* recs, Store&& store) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w0 = uniform_i32(tid) & ~63;
  const int G = 1 << kl;
  const float inv_gf = 1.0f / float(G);
  const int32_t k_s = t0 << kResTileLog;
  // grid records 0 .. n_t 512 / G (the last one is the edge past the span) and
  // tile records, into registers; they go to LDS after the samples' loads
  // have been issued
  const int gX = tid >> 6;
  float4 grec = make_float4(0.f, 0.f, 0.f, 0.f);
  int32_t girec = 0;
  const bool has_grid = gX < P.ndet && lane <= (n_t << kResTileLog) >> kl;
  const bool has_tile = gX < P.ndet && lane >= 40 && lane < 40 + n_t * kTileRecUnits;
  if (has_grid || has_tile) {
    const double2* ka = kn + gX * P.knot_stride;
    const float4* src = has_grid
                            ? reinterpret_cast<const float4*>(ka) + (k_s >> kl) + lane
                            : reinterpret_cast<const float4*>(ka + P.knot_toff) +
                                  int64_t(t0) * kTileRecUnits + (lane - 40);
    grec = *src;
    if (has_grid) girec = reinterpret_cast<const int32_t*>(ka + P.knot_ioff)[(k_s >> kl) + lane];
  }
  bool wbad = false;
  int32_t ja_all[kMaxDet];
#pragma unroll
  for (int X0 = 0; X0 < kMaxDet; X0 += kDetPass) {
    if (X0 >= P.ndet) break;
    const int np = P.ndet - X0 < kDetPass ? P.ndet - X0 : kDetPass;
    // floor of the source position at the tiles' first points and at the one
    // past the span (theta(0) in [0, 1], 1 after rounding): every load before
    // the first use, so that one wait covers them (a single detector loads its
    // own twice)
    float eth[kDetPass][kSpanTiles + 1];
    int32_t ei[kDetPass][kSpanTiles + 1];
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      const double2* ka = kn + (X0 + (xp < np ? xp : 0)) * P.knot_stride;
#pragma unroll
      for (int h = 0; h <= kSpanTiles; ++h) {
        const int32_t e = (k_s + (h < n_t ? h : n_t) * kResTile) >> kl;
        eth[xp][h] = scalar_load(reinterpret_cast<const float*>(ka) + 4 * e);
        ei[xp][h] = scalar_load(reinterpret_cast<const int32_t*>(ka + P.knot_ioff) + e);
      }
    }
    // samples ja + w, w < W
    int32_t ja[kDetPass], W[kDetPass];
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      int32_t j[kSpanTiles + 1];
#pragma unroll
      for (int h = 0; h <= kSpanTiles; ++h)
        j[h] = k_s + (h < n_t ? h : n_t) * kResTile + ei[xp][h] + (eth[xp][h] >= 1.0f ? 1 : 0);
      ja[xp] = (j[0] - D + 1) & ~((1 << kKnotLogMax) - 1);
#pragma unroll
      for (int h = 0; h < kSpanTiles; ++h) {
        const int32_t nwin = j[h + 1] - j[h] + 2 * D;
        // delay drift beyond 1/16 per tile: flag the template (NaN output)
        wbad |= h < n_t && (nwin > kResWcap || nwin < 2 * D);
      }
      W[xp] = j[kSpanTiles] + D - ja[xp] + 1;
      ja_all[X0 + xp] = ja[xp];
    }
    if (wbad) break;
    // the samples of both detectors and their intervals' records, all loads in
    // flight at once (rounds past the first kStageRounds: windows stretched
    // by extreme delays only)
    float2 xv[kDetPass][kStageRounds];
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      if (xp >= np) break;
      const DetConst& d = P.det[X0 + xp];
      const float2* xs = d.x + ja[xp];
      const uint32_t nx = uint32_t(d.n);
#pragma unroll
      for (int r = 0; r < kStageRounds; ++r) {
        const int w = r * kResThreads + tid;
        const bool in = w < W[xp] && uint32_t(ja[xp] + w) < nx;
        xv[xp][r] = in ? xs[w] : make_float2(0.f, 0.f);
      }
    }
    {
      const int xp = tid >> 7, p = tid & 127;
      if (xp < np && p < 2 * kSpanSamp) {
        const int32_t jx = xp ? ja[1] : ja[0];
        const int32_t e_max = int32_t(P.det[X0 + xp].n - 1) >> kl;
        int32_t e = (jx >> kl) + (p >> 1);
        e = e < 0 ? 0 : (e > e_max ? e_max : e);
        recs[X0 + xp].samp[p >> 1][p & 1] =
            kn[(X0 + xp) * P.knot_stride + P.knot_soff + 2 * e + (p & 1)];
      }
    }
    if (X0 == 0) {
      if (has_grid) {
        recs[gX].grid[lane] = grec;
        recs[gX].grid_i[lane] = girec;
      }
      if (has_tile) *reinterpret_cast<float4*>(&recs[gX].tile[0][4 * (lane - 40)]) = grec;
    }
    __syncthreads();
    // corrected samples z_j = x_j exp(-2 pi i f_h (t_src,j - t_j)); a zero
    // sample (outside the data, or in a gap) stays zero
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      if (xp >= np) break;
      SpanRec& rec = recs[X0 + xp];
      float2* zx = zsa + (X0 + xp) * kSpanCap;
      auto put = [&](int wu, float2 x) {
        const int w = wu + lane;
        const bool live = x.x != 0.f || x.y != 0.f;
        float2 z = make_float2(0.f, 0.f);
        if (live) {
          const double2 k01 = rec.samp[w >> kl][0], k23 = rec.samp[w >> kl][1];
          z = correct_sample(x, double(w & (G - 1)), k01.x, k01.y, k23.x, k23.y);
        }
        if (w < W[xp]) zx[w] = z;
        // which 32-sample blocks of the window hold a live sample
        const unsigned long long mb = __ballot(live);
        if (lane == 0) {
          rec.blk[wu >> 5] = uint32_t(mb) != 0u;
          rec.blk[(wu >> 5) + 1] = uint32_t(mb >> 32) != 0u;
        }
      };
#pragma unroll
      for (int r = 0; r < kStageRounds; ++r) {
        if (r * kResThreads + w0 >= W[xp]) break;
        put(r * kResThreads + w0, xv[xp][r]);
      }
#pragma unroll 1
      for (int wu = kStageRounds * kResThreads + w0; wu < W[xp]; wu += kResThreads) {
        const bool in = wu + lane < W[xp] && uint32_t(ja[xp] + wu + lane) < uint32_t(P.det[X0 + xp].n);
        put(wu, in ? P.det[X0 + xp].x[ja[xp] + wu + lane] : make_float2(0.f, 0.f));
      }
    }
  }
  if (wbad) {
    if (tid == 0) atomicOr(status_word, kStatusWindow);
    return false;
  }
  __syncthreads();
  // d(angle)/d(grid step) of the sidereal angle x, radians
  const float dstep = float(-2.0 * kPi * P.sid_rate_cyc * P.dt);
#pragma unroll 1
  for (int h = 0; h < n_t; ++h) {
    const int32_t k_t = k_s + h * kResTile;
    float2 acc_a[kResPerThread], acc_b[kResPerThread];
#pragma unroll
    for (int i = 0; i < kResPerThread; ++i)
      acc_a[i] = acc_b[i] = make_float2(0.f, 0.f);
#pragma unroll 1
    for (int X = 0; X < P.ndet; ++X) {
      const SpanRec& rec = recs[X];
      const float2* zx = zsa + X * kSpanCap;
      const int32_t ja = X == 0 ? ja_all[0] : X == 1 ? ja_all[1] : X == 2 ? ja_all[2] : ja_all[3];
      // the window's live blocks as a bit mask in scalar registers
      const unsigned long long mask = __ballot(lane < kSpanBlk && rec.blk[lane < kSpanBlk ? lane : 0]);
      const int32_t sb = k_t - ja - (D - 1);
      const float* tr = rec.tile[h];
      const float th_r = tr[kTaylorCoef];
      const int32_t i_r = __float_as_int(tr[kTaylorCoef + 1]);
#pragma unroll
      for (int i = 0; i < kResPerThread; ++i) {
        const int kk = tid + i * kResThreads;
        const int e = (h * kResTile + kk) >> kl;
        const float4 cq = rec.grid[e];
        const int32_t im = rec.grid_i[e];
        const float v = float(kk & (G - 1)) * inv_gf;
        const float th = fmaf(fmaf(fmaf(cq.w, v, cq.z), v, cq.y), v, cq.x);
        const float fl = floorf(th);
        float f = th - fl;
        int base = sb + im + kk + int(fl);
        if (f >= 1.0f) {
          f = 0.0f;
          base += 1;
        }
        // monotonic T_k keeps the taps in the window, the clamp guards memory
        base = base < 0 ? 0 : (base > kSpanCap - 2 * D ? kSpanCap - 2 * D : base);
        // taps that all fall on zero samples add nothing (they reach two
        // blocks at most)
        if (((mask >> (base >> 5)) & 3u) == 0u) continue;
        const float2 zh = sinc_interp<D>(f, zx + base);
        if (P.res_taylor) {
          // sidereal angle offset from the tile's middle point
          const float dx = (float(kk - kResTile / 2 + (im - i_r)) + (th - th_r)) * dstep;
          weight_taylor(zh, dx, tr, acc_a[i], acc_b[i]);
        } else {
          // q = u - k - off
          const double q = (double(im) - P.det[X].off) + double(th);
          weight_add(P, tp, X, P.tau0 + P.dt * double(k_t + kk), q, zh, acc_a[i], acc_b[i]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kResPerThread; ++i)
      store(k_t + tid + i * kResThreads, acc_a[i], acc_b[i]);
  }
  return true;
}

// Grid knot at k (a whole or fractional grid point): q = (T_k - tau_k)/dt from
// the detector epoch of tau = tau0 + k dt (fixed point and two Newton steps)
// and dq/dk = (R'(tau) - roemer'(T)) / (1 + roemer'(T)); far: the delay exceeds
// `limit`.
template <bool KEP>
__device__ __forceinline__ double2 grid_knot(const PlanConst& P, const TmplParams& tp,
                                             const CachedRoemer& re, double k, double limit,
                                             bool& far) {
  const double tau = P.tau0 + P.dt * k;
  double rb, rbd, x;
  orbit_delay<KEP>(tp, tau, rb, rbd);
  double dl = grid_delay_rb(re, rb, tau);
  dl = grid_delay_newton(re, tau, rb, dl, x);
  dl = grid_delay_newton(re, tau, rb, dl, x);
  far = !(fabs(dl) <= limit);
  return make_double2(dl * P.inv_dt, (rbd - x) / (1.0 + x));
}

// The record of a grid interval from its end knots a, b (g grid steps apart;
// last: the point past the grid, its position only): the source position
// relative to its integer part as a cubic (resample_span).
__device__ __forceinline__ void grid_record(double off, double2 a, double2 b, double g, bool last,
                                            float4& rec, int32_t& whole) {
  double2 c0 = make_double2(a.x, 0.0), c1 = make_double2(0.0, 0.0);
  if (!last) hermite_interval(a, b, g, c0, c1);
  const double x = off + c0.x;
  const double fx = floor(x);
  rec = make_float4(float(x - fx), float(c0.y), float(c1.x), float(c1.y));
  whole = int32_t(fx);
}
// The record of a sample interval from its end knots (phase in cycles, change
// per sample), g samples apart: quarter turns as a cubic in the sample offset
// (scalings by powers of two: exact), the constant modulo one turn.
__device__ __forceinline__ void sample_record(double2 a, double2 b, double g, double2& lo,
                                              double2& hi) {
  double2 c0, c1;
  hermite_interval(a, b, g, c0, c1);
  const double ig = 1.0 / g;
  lo = make_double2(fmod(4.0 * c0.x, 4.0), 4.0 * c0.y * ig);
  hi = make_double2(4.0 * c1.x * ig * ig, 4.0 * c1.y * ig * ig * ig);
}

// Resampling kernels.  GROUPED = false: blockIdx.y is a template slot; the
// spin-down phase is applied and y_a', y_b' go to the slot's arrays 0 and 1.
// GROUPED = true: blockIdx.y is a sky/orbit group of the chunk; the series is
// written without the spin-down phase to the group's buffer, which every
// template of the group reads (the reuse of the sky-dependent barycentring
// across spin-down templates that Sec. 4.1 measures).
//
// Where a resampling block writes, and whether the template (group) is
// live: a leader whose sky or orbit is invalid invalidates the whole group
// (its status word tells every member's column pass not to read the buffer).
struct ResTarget {
  const TmplParams* tp;
  int32_t* status;
  float2* ya;
  float2* yb;
  const double2* kn;  // knot area (null: none)
  bool live;
};
template <bool GROUPED>
__device__ __forceinline__ ResTarget res_target(const PlanConst& P, void* ws, const ChunkMap& map,
                                                int slots) {
  const int gi = blockIdx.y;
  const int slot = GROUPED ? map.grp_slot[gi] : gi;
  ResTarget r;
  r.tp = tmpl_params(ws, P, map, slot);
  r.status = GROUPED ? group_status(ws, P, slots, map.grp_buf[gi])
                     : &tmpl_params(ws, P, map, slot)->status;
  r.ya = GROUPED ? group_buf(ws, P, slots, map.grp_buf[gi], 0) : slot_buf(ws, P, slot, 0);
  r.yb = GROUPED ? group_buf(ws, P, slots, map.grp_buf[gi], 1) : slot_buf(ws, P, slot, 1);
  r.kn = P.knot_bytes == 0 ? nullptr
         : GROUPED         ? group_knots(ws, P, slots, map.grp_buf[gi])
                           : slot_knots(ws, P, slot);
  r.live = true;
  if (GROUPED) {
    const int32_t gflag = r.tp->status & kStatusGroupMask;
    if (gflag != 0) {
      if (threadIdx.x == 0 && blockIdx.x == 0) atomicOr(r.status, gflag);
      r.live = false;
    }
  } else if (r.tp->status != 0) {
    r.live = false;
  }
  return r;
}
// Whether a template's timing knots were solved ahead (k_timing).
__device__ __forceinline__ bool knots_ahead(const ResTarget& r) {
  return r.kn != nullptr && r.tp->knot_log2 >= kKnotLogGlobal;
}
template <bool GROUPED>
__device__ __forceinline__ void res_store(const ResTarget& r, int64_t k, float2 a, float2 b) {
  if (GROUPED) {
    r.ya[k] = a;
    r.yb[k] = b;
  } else {
    // spin-down phase and sub-bin offset: y = acc * exp(-2 pi i cyc)
    const float2 e = spindown_rotation(r.tp->sd, k);
    r.ya[k] = cmul_exact(a, e);
    r.yb[k] = cmul_exact(b, e);
  }
}

// Templates whose knots were solved ahead: `span` tiles per block (at most
// kSpanTiles), as one span where the LDS records hold it (knot spacings of 32
// and 64), else tile by tile.
template <int D, bool GROUPED>
__global__ __launch_bounds__(kResThreads, kResWavesAhead) void k_resample(PlanConst P, void* ws,
                                                                       ChunkMap map, int slots,
                                                                       int span) {
  extern __shared__ float2 zs[];
  const ResTarget r = res_target<GROUPED>(P, ws, map, slots);
  if (!r.live || !knots_ahead(r)) return;
  const int32_t tiles = int32_t(P.k_pad >> kResTileLog);
  const int32_t t_b = int32_t(blockIdx.x) * span;
  const int32_t t_e = t_b + span < tiles ? t_b + span : tiles;
  SpanRec* recs = reinterpret_cast<SpanRec*>(zs + P.ndet * kSpanCap);
  const int kl = uniform_i32(r.tp->knot_log2);
  const int step = kl > kKnotLogGlobal ? span : 1;
#pragma unroll 1
  for (int32_t t = t_b; t < t_e; t += step) {
    if (t != t_b) __syncthreads();  // the last tile has read the window
    const int n_t = t_e - t < step ? t_e - t : step;
    if (!resample_span<D>(P, *r.tp, r.kn, kl, r.status, t, n_t, zs, recs,
                          [&](int32_t k, float2 a, float2 b) { res_store<GROUPED>(r, k, a, b); }))
      return;
  }
}

// Timing knots of one template (slot) or sky/orbit group whose knot spacing
// G = 2^tp.knot_log2 is at least 2^kKnotLogGlobal, for the detector X and
// its block b: the same FP64 solves as the tiles' own knots (steps (iv) and
// (iii) of Sec. 3), one knot per thread, with the Roemer delay from the
// detector's tabulated trajectory (the interval read last kept in
// registers).  Three ranges of blocks:
//  - the first blocks solve the grid knots and turn each interval's two
//    end knots into its record (the cubic Hermite form of q between them,
//    relative to the integer part of the interval's first source position);
//  - knot_tile_blocks blocks (plans with res_taylor) solve the knot at each
//    tile's middle point again and write the tile's antenna Taylor record;
//  - the rest solve the sample knots.
// A delay beyond the plan's max_delay flags the template (as a tile whose
// delay leaves its staged nodes does).
template <bool KEP>
__device__ __forceinline__ void solve_knots(const PlanConst& P, const TmplParams& tp, int kl,
                                            double2* kn, int32_t* status_word, int X, int64_t b) {
  const DetConst& d = P.det[X];
  kn += X * P.knot_stride;
  const int G = 1 << kl;
  const CachedRoemer re{d.ephem, tp.nhat, P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt};
  // blocks launched per range: enough for the coarsest spacing; a template
  // with a finer one walks its chunks of kKnotThreads - 1 knots in steps of
  // the range's block count
  int64_t scap = 0;
  for (int Y = 0; Y < P.ndet; ++Y) scap = max(scap, ((P.det[Y].n - 1) >> kKnotLogMax) + 2);
  const int64_t gblocks = knot_grid_blocks((P.k_pad >> kKnotLogMax) + 1);
  const int64_t tblocks = knot_tile_blocks(P.k_pad);
  const int64_t sblocks = knot_samp_blocks(scap);
  __shared__ double2 nb[kKnotThreads];
  bool far = false;
  if (b < gblocks) {
    const int64_t last = P.k_pad >> kl;
    const int64_t chunks = knot_grid_blocks(last + 1);
    for (int64_t c = b; c < chunks; c += gblocks) {
      const int64_t e = c * (kKnotThreads - 1) + threadIdx.x;
      double2 kv = make_double2(0.0, 0.0);
      if (e <= last) {
        bool f;
        kv = grid_knot<KEP>(P, tp, re, double(e * G), P.max_delay, f);
        far |= f;
      }
      nb[threadIdx.x] = kv;
      __syncthreads();
      if (threadIdx.x < kKnotThreads - 1 && e <= last) {
        grid_record(d.off, kv, nb[threadIdx.x + 1], double(G), e == last,
                    reinterpret_cast<float4*>(kn)[e],
                    reinterpret_cast<int32_t*>(kn + P.knot_ioff)[e]);
      }
      __syncthreads();
    }
  } else if (b < gblocks + tblocks) {
    const int64_t t = (b - gblocks) * kKnotThreads + threadIdx.x;
    if (P.res_taylor && t < (P.k_pad >> kResTileLog)) {
      // the tile's middle point is a knot (G divides half a tile)
      const int64_t k = (t << kResTileLog) + kResTile / 2;
      bool far_t;
      const double2 kv = grid_knot<KEP>(P, tp, re, double(k), P.max_delay, far_t);
      float c[kTaylorCoef];
      antenna_taylor(tp.ca[X], tp.cb[X],
                     tp.alpha_cyc[X] - P.sid_rate_cyc * (P.tau0 + P.dt * double(k) + kv.x * P.dt),
                     c);
      const double a = d.off + kv.x;
      const double fa = floor(a);
      float* tr = reinterpret_cast<float*>(kn + P.knot_toff + t * kTileRecUnits);
#pragma unroll
      for (int n = 0; n < kTaylorCoef; ++n) tr[n] = c[n];
      tr[kTaylorCoef] = float(a - fa);
      tr[kTaylorCoef + 1] = __int_as_float(int32_t(fa));
    }
  } else {
    // sample knot m: heterodyne phase at t = t0 + m G dt and its change per
    // sample; the record of interval m from knots m and m + 1
    const int64_t last = ((d.n - 1) >> kl) + 1;
    const int64_t chunks = knot_samp_blocks(last + 1);
    for (int64_t c = b - gblocks - tblocks; c < chunks; c += sblocks) {
      const int64_t m = c * (kKnotThreads - 1) + threadIdx.x;
      double2 kv = make_double2(0.0, 0.0);
      if (m <= last) {
        double ph, dph, delay;
        sample_phase_d<KEP>(re, tp, d.t0 + P.dt * double(m * G), P.f_het, ph, dph, delay);
        kv = make_double2(ph, dph * P.dt);
        far |= !(fabs(delay) <= P.max_delay);
      }
      nb[threadIdx.x] = kv;
      __syncthreads();
      if (threadIdx.x < kKnotThreads - 1 && m < last) {
        double2* rec = kn + P.knot_soff + 2 * m;
        sample_record(kv, nb[threadIdx.x + 1], double(G), rec[0], rec[1]);
      }
      __syncthreads();
    }
  }
  if (far) atomicOr(status_word, kStatusNodes);
}

// Ahead of the resampling, per template (slot) or group: the timing knots
// (kblocks blocks per detector), or, where the knot spacing is below 16
// points, the whole resampling, the tiles solving their own timing (walked by
// the blocks past the knots'; their FP64 and LDS latency chains want four waves
// per SIMD, 128 registers).  Which of the two a template takes is known on the
// device only; one launch carries both, so a bank of either kind pays for one
// kernel (a launch of the tiles alone, whose blocks all return at once, took
// 2-5 us of a small search and 10 us of a large one).  The knots pay with the
// tiles' registers and LDS, four waves per SIMD instead of five: 240 us instead
// of 200 for 32 templates of 5.2 M points, 63 / 47 for 16 of 2.6 M.  Launching them
// apart in large searches was measured again and gains too little for a second
// kernel: parameters and timing together 247 / 256 us of 5370, 32 templates of
// 1.5 M points 1325 / 1320, small searches 2 us slower.
template <int D, bool GROUPED, bool KEP>
__global__ __launch_bounds__(kResThreads, 4) void k_timing(PlanConst P, void* ws, ChunkMap map,
                                                           int slots, int kblocks) {
  static_assert(kKnotThreads == kResThreads, "one block size for both");
  const ResTarget r = res_target<GROUPED>(P, ws, map, slots);
  if (!r.live) return;
  const int b = blockIdx.x, nk = kblocks * P.ndet;
  if (b < nk) {
    if (knots_ahead(r))
      solve_knots<KEP>(P, *r.tp, r.tp->knot_log2, const_cast<double2*>(r.kn), r.status,
                       b / kblocks, b % kblocks);
    return;
  }
  if (knots_ahead(r)) return;
  __shared__ float2 zs[kDetPass * kResWcap];
  __shared__ int32_t blk[kDetPass * kResBlk];
  const int64_t tiles = P.k_pad / kResTile;
  for (int64_t t = b - nk; t < tiles; t += int(gridDim.x) - nk) {
    const int64_t k_s = t * kResTile;
    float2 acc_a[kResPerThread], acc_b[kResPerThread];
    if (!resample_tile<D, KEP>(P, *r.tp, r.status, k_s, zs, blk, acc_a, acc_b)) return;
#pragma unroll
    for (int i = 0; i < kResPerThread; ++i)
      res_store<GROUPED>(r, k_s + threadIdx.x + i * kResThreads, acc_a[i], acc_b[i]);
    // the next tile's first phase rewrites what this one's last read
    __syncthreads();
  }
}

// exp(-2 pi i nat k / N) with the product reduced exactly in integers.
__device__ inline float2 bin_twiddle(int64_t nat, int64_t k, int64_t n_fft) {
  return cis_neg_frac((nat * k) & (n_fft - 1), __builtin_ctzll(uint64_t(n_fft)));
}

// Natural FFT index of band bin i (bins ascend in frequency from bin_lo of
// the centred spectrum).
__host__ __device__ inline int64_t band_bin_nat(const PlanConst& P, int64_t i) {
  return (P.bin_lo + i + P.n_fft / 2) & (P.n_fft - 1);
}

// Single-bin forward path: the whitened transforms Fa'(m), Fb'(m) at one bin
// m per template as a direct sum over the grid, sum_k y'_k exp(-2 pi i m k/N)
// (step (vi) restricted to one output bin), reduced per tile into the slot's
// partials (Fa'.re, Fa'.im, Fb'.re, Fb'.im in FP64).  The templates whose
// timing is solved point by point (the others: k_bin_span).
// One tile per block unless WALK: in a loop the kernel spills 28 registers
// instead of 16 and takes 1096 us where it took 993 (32 templates of 1 M
// points).
template <int D, bool KEP, bool WALK>
__global__ __launch_bounds__(kResThreads, 4) void k_resample_bin(PlanConst P, void* ws, ChunkMap map,
                                                             const int64_t* __restrict__ bins) {
  const int slot = blockIdx.y;
  TmplParams* tpp = slot_params(ws, P, slot);
  const TmplParams& tp = *tpp;
  const int tid = threadIdx.x;
  if (tp.status != 0 || tp.tile_form != kTilePoints) return;
  __shared__ float2 zs[kDetPass * kResWcap];
  __shared__ int32_t blk[kDetPass * kResBlk];
  __shared__ double red[kResThreads / 64][4];
  const int64_t nat = band_bin_nat(P, bins[map.tmpl[slot]]);
  const int64_t tiles = P.k_pad / kResTile;
  int64_t t = blockIdx.x;
  do {
    double* partial = slot_partials(ws, P, slot) + size_t(t) * 8;
    const int64_t k_s = t * kResTile;
    float2 acc_a[kResPerThread], acc_b[kResPerThread];
    if (!resample_tile<D, KEP>(P, tp, &tpp->status, k_s, zs, blk, acc_a, acc_b)) return;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < kResPerThread; ++i) {
      const int64_t k = k_s + tid + i * kResThreads;
      const float2 e = cmul(spindown_rotation(tp.sd, k),
                            bin_twiddle(nat, k, P.n_fft));
      const float2 ya = cmul(acc_a[i], e), yb = cmul(acc_b[i], e);
      s[0] += double(ya.x);
      s[1] += double(ya.y);
      s[2] += double(yb.x);
      s[3] += double(yb.y);
    }
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double v = s[q];
      for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
      if (lane == 0) red[wave][q] = v;
    }
    __syncthreads();
    if (tid < 4) {
      double v = 0.0;
      for (int w = 0; w < kResThreads / 64; ++w) v += red[w][tid];
      partial[tid] = v;
    }
    if constexpr (WALK) __syncthreads();
  } while (WALK && (t += gridDim.x) < tiles);
}

// Per-template totals of per-tile partials (8 doubles per tile, the first
// NQ used) by one workgroup: each thread sums a fixed stripe of tiles, then a
// fixed tree combines the threads, so a template's totals come out the same
// on every run.  The totals land in s of thread 0.
constexpr int kFinalThreads = 256;
template <int NQ>
__device__ inline void tile_sums(const double* __restrict__ part, int64_t ntiles, double (&s)[NQ]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < NQ; ++q) s[q] = 0.0;
  for (int64_t b = tid; b < ntiles; b += kFinalThreads)
#pragma unroll
    for (int q = 0; q < NQ; ++q) s[q] += part[b * 8 + q];
  __shared__ double red[NQ][kFinalThreads];
#pragma unroll
  for (int q = 0; q < NQ; ++q) red[q][tid] = s[q];
  __syncthreads();
  for (int off = kFinalThreads / 2; off > 0; off >>= 1) {
    if (tid < off)
#pragma unroll
      for (int q = 0; q < NQ; ++q) red[q][tid] += red[q][tid + off];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) s[q] = red[q][0];
}

// Per template: Fa'(m), Fb'(m) from the tile partials (tile order), 2F at the
// bin, and the adjoint spectrum of L = 2F(m) at that bin, H = conj(F'(m))
// (kept in the parameter block for the gradient kernel).  A bin outside the
// band flags the template.
__global__ __launch_bounds__(kFinalThreads) void k_bin_final(PlanConst P, void* ws, ChunkMap map,
                                                             int64_t ntiles,
                                                             const int64_t* __restrict__ bins,
                                                             float* __restrict__ twoF) {
  const int slot = blockIdx.x;
  double f[4];
  tile_sums<4>(slot_partials(ws, P, slot), ntiles, f);
  if (threadIdx.x != 0) return;
  TmplParams& tp = *slot_params(ws, P, slot);
  const int64_t bin = bins[map.tmpl[slot]];
  if (bin < 0 || bin >= P.n_bins) tp.status |= kStatusBin;
  if (tp.status != 0) atomicAdd(flag_counter(ws), 1ull);
  tp.bin_nat = band_bin_nat(P, bin);
  tp.hbin[0] = f[0];
  tp.hbin[1] = -f[1];
  tp.hbin[2] = f[2];
  tp.hbin[3] = -f[3];
  const double v = 2.0 * (f[0] * f[0] + f[1] * f[1] + f[2] * f[2] + f[3] * f[3]);
  if (twoF) twoF[map.tmpl[slot]] = tp.status != 0 ? __builtin_nanf("") : float(v);
}

}  // namespace fstat
