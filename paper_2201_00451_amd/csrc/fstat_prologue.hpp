// Per-data-set antenna moments and the per-template prologue.
//
// A, B, C of eq. Fstat (Sec. 2) are noise-weighted sums of products of a(t),
// b(t) over the valid samples.  a and b are trigonometric polynomials of
// degree two in x = alpha - phi(t) (phi: local sidereal angle), so
//   sum_j v_j P(x_j) Q(x_j) = 1/2 Re sum_{h,g} [p_h q_g S_{h+g} + p_h conj(q_g) S_{h-g}]
// with P = Re sum_h p_h e^{i h x}, Q = Re sum_g q_g e^{i g x}, and
//   S_n = sum_j v_j e^{i n x_j} = e^{i n alpha} conj(M_n),  M_n = sum_j v_j e^{i n phi_j}.
// The moments M_0..M_4 depend on the data set only; the prologue combines
// them with the sky position in O(1) per template.
#pragma once

#include "fstat_common.hpp"

namespace fstat {

// Partial moments: block b of detector X sums a contiguous chunk of samples.
__global__ __launch_bounds__(kMomThreads) void k_moments_partial(PlanConst P, double* partial) {
  const int X = blockIdx.y;
  const DetConst& d = P.det[X];
  const int64_t n = d.n;
  const int64_t chunk = (n + kMomBlocks - 1) / kMomBlocks;
  const int64_t j_beg = int64_t(blockIdx.x) * chunk;
  const int64_t j_end = j_beg + chunk < n ? j_beg + chunk : n;
  double acc[10];
  for (int q = 0; q < 10; ++q) acc[q] = 0.0;
  const double two_pi = 2.0 * kPi;
  for (int64_t j = j_beg + threadIdx.x; j < j_end; j += kMomThreads) {
    double v = d.valid ? double(d.valid[j]) : 1.0;
    if (v == 0.0) continue;
    double cyc = d.lst0_cyc + P.sid_rate_cyc * (d.t0 + P.dt * double(j));
    cyc -= rint(cyc);
    double s1, c1;
    sincos(two_pi * cyc, &s1, &c1);
    double cr = 1.0, ci = 0.0;
    for (int h = 0; h < 5; ++h) {
      acc[2 * h] += v * cr;
      acc[2 * h + 1] += v * ci;
      double nr = cr * c1 - ci * s1;
      ci = cr * s1 + ci * c1;
      cr = nr;
    }
  }
  __shared__ double red[kMomThreads];
  for (int q = 0; q < 10; ++q) {
    red[threadIdx.x] = acc[q];
    __syncthreads();
    for (int s = kMomThreads / 2; s > 0; s >>= 1) {
      if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) partial[(size_t(X) * kMomBlocks + blockIdx.x) * 10 + q] = red[0];
    __syncthreads();
  }
}

// Final sum of the partials in block order.
__global__ void k_moments_final(int ndet, const double* partial, double* moments) {
  int t = threadIdx.x;
  if (t >= ndet * 10) return;
  int X = t / 10, q = t % 10;
  double s = 0.0;
  for (int b = 0; b < kMomBlocks; ++b) s += partial[(size_t(X) * kMomBlocks + b) * 10 + q];
  moments[X * 10 + q] = s;
}

struct cd {
  double r, i;
};
__host__ __device__ inline cd cd_mul(cd a, cd b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
__host__ __device__ inline cd cd_conj(cd a) { return {a.r, -a.i}; }

// sum_j v_j P(x_j) Q(x_j) for degree-2 polynomials p, q (complex coefficients)
// given S_0..S_4.
__host__ __device__ inline double moment_product(const cd p[3], const cd q[3], const cd S[5]) {
  double acc = 0.0;
#pragma unroll
  for (int h = 0; h < 3; ++h)
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      cd t1 = cd_mul(cd_mul(p[h], q[g]), S[h + g]);
      int dn = h - g;
      cd sd = dn >= 0 ? S[dn] : cd_conj(S[-dn]);
      cd t2 = cd_mul(cd_mul(p[h], cd_conj(q[g])), sd);
      acc += t1.r + t2.r;
    }
  return 0.5 * acc;
}

// Coefficients of a(t), b(t) (Jaranowski, Krolak & Schutz 1998 eqs. 12-13,
// cited in Sec. 2) in the basis (1, cos x, sin x, cos 2x, sin 2x) of
// x = alpha - phi(t), for one detector at declination delta, and their delta
// derivatives (d sin 2delta = 2 cos 2delta, d cos 2delta = -2 sin 2delta).
struct Jks {
  double pa[5], pb[5], dpa[5], dpb[5];
};
__host__ __device__ inline Jks jks_coeffs(const DetConst& d, double sd, double cdl) {
  const double sl = d.sl, cl = d.cl, sg = d.s2g, cg = d.c2g;
  const double s2l = 2.0 * sl * cl, c2l = cl * cl - sl * sl;
  const double s2d = 2.0 * sd * cdl, c2d = cdl * cdl - sd * sd;
  Jks k;
  k.pa[0] = 0.75 * sg * cl * cl * cdl * cdl;
  k.pa[1] = 0.25 * sg * s2l * s2d;
  k.pa[2] = -0.5 * cg * cl * s2d;
  k.pa[3] = sg * (3.0 - c2l) * (3.0 - c2d) / 16.0;
  k.pa[4] = -0.25 * cg * sl * (3.0 - c2d);
  k.pb[0] = 0.0;
  k.pb[1] = cg * cl * cdl;
  k.pb[2] = 0.5 * sg * s2l * cdl;
  k.pb[3] = cg * sl * sd;
  k.pb[4] = 0.25 * sg * (3.0 - c2l) * sd;
  k.dpa[0] = -0.75 * sg * cl * cl * s2d;
  k.dpa[1] = 0.5 * sg * s2l * c2d;
  k.dpa[2] = -cg * cl * c2d;
  k.dpa[3] = sg * (3.0 - c2l) * s2d / 8.0;
  k.dpa[4] = -0.5 * cg * sl * s2d;
  k.dpb[0] = 0.0;
  k.dpb[1] = -cg * cl * sd;
  k.dpb[2] = -0.5 * sg * s2l * sd;
  k.dpb[3] = cg * sl * cdl;
  k.dpb[4] = 0.25 * sg * (3.0 - c2l) * cdl;
  return k;
}

constexpr double kSpanOrbit = 0.3;         // circular orbit: phase of half a tile, radians
constexpr double kSpanOrbitKepler = 0.18;  // eccentric: the same, at periapsis
constexpr double kSpanAngle = 0.05;        // sidereal angle of half a tile, radians
constexpr double kSpanCurve = 1.5e-3;      // phase over the taps of one side, radians

// The form in which the gradient and single-bin kernels take a template: spans
// of tiles where knots lie at least 16 points apart and half a tile covers at
// most 0.05 rad of the Earth's rotation and 0.3 rad of a circular orbit, 0.18 of
// an eccentric one (its angular rate at periapsis, om / (1 - ecc)^2), so that
// quintics per tile carry the timing's derivatives; else point by point.  At
// these limits the quintics of the orbit's delay and rate are within 3.3e-8 of
// their amplitudes (0.3^6 / 23040 for a circle; eccentric orbits carry
// harmonics: at 0.3 rad they were off by up to 5.4e-7, at ecc = 0.4).
//
// Within a span the sum over taps with the samples' delay derivatives d,
// sum_j h(u - j) d(j) z_j, is expanded about the point u.  The term of second
// order is (w dt)^2 / 2 of d times sum_j h (j - u)^2 z_j, and that sum is at most
// about D^2 / 20 of |z|: it is the curvature of the interpolation's response
// over frequency, so it vanishes well inside the band and is largest near the
// band's edge, where the response falls off within 1 / (2 D) cycles per
// sample.  Below w dt D = 1.5e-3 the term is under 6e-8, the rounding of the
// FP32 sums; above, it is carried (kTileCurved), and the one of third order is
// under 2e-8 up to the 0.3 rad and D = 16.
//
// tile_limits (host): the limits as angular rates, so that the kernel compares
// only; a plan with more than 0.05 rad of rotation per half tile admits no spans
// at all (span_w < 0) and launches none.
inline void tile_limits(PlanConst& P) {
  const double half = 0.5 * kResTile * P.dt;
  const double sid = 2.0 * kPi * P.sid_rate_cyc;
  const double curve = kSpanCurve / (P.dt * double(P.D));
  P.span_w = sid * half <= kSpanAngle ? float(kSpanOrbit / half) : -1.0f;
  P.curve_w = sid <= curve ? float(curve) : -1.0f;
}
inline bool spans_possible(const PlanConst& P) { return P.span_w >= 0.0f; }
__host__ __device__ inline int32_t tile_form(const PlanConst& P, double om_b, double ecc,
                                             int32_t knot_log2) {
  const double e2 = (1.0 - ecc) * (1.0 - ecc);
  const double lim = (ecc > 0.0 ? kSpanOrbitKepler / kSpanOrbit : 1.0) * double(P.span_w);
  if (knot_log2 < kKnotLogGlobal || !(om_b <= lim * e2)) return kTilePoints;
  return om_b <= double(P.curve_w) * e2 ? kTileSmooth : kTileCurved;
}

// A template's row: orbit, knot spacing, spin-down phase, sky vector and its
// derivatives, and the status bits these give.
__host__ __device__ inline void row_params(const PlanConst& P, const double* row, TmplParams& tp) {
  double alpha = row[0], delta = row[1];
  tp.df = row[2];
  tp.f1dot = row[3];
  tp.f2dot = row[4];
  tp.asini = row[5];
  double porb = row[6];
  tp.tp = row[7];
  const double ecc = P.tmpl_stride >= FSTAT_TEMPLATE_STRIDE_KEPLER ? row[8] : 0.0;
  const double argp = P.tmpl_stride >= FSTAT_TEMPLATE_STRIDE_KEPLER ? row[9] : 0.0;
  int status = 0;
  // porb and tp describe the orbit only when asini != 0: an isolated
  // source (asini = 0) ignores them, whatever they hold
  if (!__builtin_isfinite(alpha) || !__builtin_isfinite(delta) || !__builtin_isfinite(tp.asini) ||
      (tp.asini != 0.0 && (!__builtin_isfinite(porb) || !__builtin_isfinite(tp.tp))))
    status |= kStatusTiming;
  if (!__builtin_isfinite(tp.df) || !__builtin_isfinite(tp.f1dot) ||
      !__builtin_isfinite(tp.f2dot))
    status |= kStatusPhase;
  if (tp.asini < 0.0 || (tp.asini != 0.0 && !(porb > 0.0))) status |= kStatusTiming;
  // Keplerian elements (used only when asini != 0)
  if (tp.asini != 0.0 && !(ecc >= 0.0 && ecc < 1.0 && __builtin_isfinite(argp)))
    status |= kStatusTiming;
  tp.kepler = (tp.asini != 0.0 && (ecc != 0.0 || argp != 0.0)) ? 1 : 0;
  tp.ecc = tp.kepler ? ecc : 0.0;
  tp.sq_e = sqrt(1.0 - tp.ecc * tp.ecc);
  if (tp.kepler) {
    sincos(argp, &tp.sin_w, &tp.cos_w);
  } else {
    tp.sin_w = 0.0;
    tp.cos_w = 1.0;
  }
  if (tp.asini > P.max_delay) status |= kStatusCoverage;
  tp.om_b = (tp.asini != 0.0 && porb > 0.0) ? 2.0 * kPi / porb : 0.0;
  tp.nu_b = (tp.asini != 0.0 && porb > 0.0) ? 1.0 / porb : 0.0;
  // Knot spacing of the resampling's timing: the largest G = 2^l <= 64 for
  // which the cubic Hermite bound (G dt)^4 / 384 max|delay''''| stays below
  // 2e-7 cycles of the heterodyne phase f_h and 1e-7 samples of grid
  // position.  The binary delay contributes asini om^4; the Earth's motion,
  // tabulated as C1-joined cubics, contributes far less than the floor
  // taken here.  Below G = 4, every point is solved (knot_log2 = 0).
  {
    // the Keplerian delay's fourth derivative grows like (om / (1 - ecc)^2)^4
    // near periapsis (a bound, not the exact maximum)
    const double w = tp.om_b / ((1.0 - tp.ecc) * (1.0 - tp.ecc));
    const double om2 = w * w;
    const double d4 = fabs(tp.asini) * om2 * om2 + 1e-16;
    const double budget = fmin(2e-7 / fmax(fabs(P.f_het), 1.0), 1e-7 * P.dt);
    tp.knot_log2 = 0;
    for (int l = kKnotLogMax; l >= kKnotLogMin; --l) {
      const double h = double(1 << l) * P.dt, h2 = h * h;
      if (h2 * h2 / 384.0 * d4 <= budget) {
        tp.knot_log2 = l;
        break;
      }
    }
  }
  spindown_coefficients(P, tp.f1dot, tp.f2dot, tp.df, tp.sd);
  double sa, ca_, sd, cdl;
  sincos(alpha, &sa, &ca_);
  sincos(delta, &sd, &cdl);
  tp.nhat[0] = cdl * ca_;
  tp.nhat[1] = cdl * sa;
  tp.nhat[2] = sd;
  tp.porb = porb;
  // d nhat / d alpha, d nhat / d delta
  tp.dnhat[0][0] = -cdl * sa;
  tp.dnhat[0][1] = cdl * ca_;
  tp.dnhat[0][2] = 0.0;
  tp.dnhat[1][0] = -sd * ca_;
  tp.dnhat[1][1] = -sd * sa;
  tp.dnhat[1][2] = cdl;
#pragma unroll
  for (int X = 0; X < kMaxDet; ++X)
    tp.alpha_cyc[X] = X < P.ndet ? alpha / (2.0 * kPi) - P.det[X].lst0_cyc : 0.0;
  tp.status = status;
}

// One detector's share of a sum of eq. Fstat at the sky position (alpha,
// delta): term 0..2 are A, B, C, 3..5 their derivatives with respect to
// alpha, 6..8 with respect to delta.  alpha enters through S_n = e^{i n alpha}
// conj(M_n): dS_n = i n S_n; delta through the coefficients (the product is
// bilinear).
constexpr int kMatrixTerms = 9;
__host__ __device__ inline double matrix_term(const DetConst& d, const double* moments,
                                              const Jks& k, double sa, double ca, int term) {
  cd ea[5];
  ea[0] = {1.0, 0.0};
  ea[1] = {ca, sa};
#pragma unroll
  for (int n = 2; n < 5; ++n) ea[n] = cd_mul(ea[n - 1], ea[1]);
  cd S[5];
#pragma unroll
  for (int n = 0; n < 5; ++n) {
    S[n] = cd_mul(ea[n], cd_conj({moments[2 * n], moments[2 * n + 1]}));
    if (term >= 3 && term < 6) S[n] = {-double(n) * S[n].i, double(n) * S[n].r};
  }
  // term mod 3: a a (A), b b (B) or a b (C)
  const bool da = term >= 6;
  const int ab = term % 3;
  double pl[5], pr[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    pl[i] = ab == 1 ? (da ? k.dpb[i] : k.pb[i]) : (da ? k.dpa[i] : k.pa[i]);
    pr[i] = ab == 0 ? k.pa[i] : k.pb[i];
  }
  const cd p[3] = {{pl[0], 0.0}, {pl[1], -pl[2]}, {pl[3], -pl[4]}};
  const cd q[3] = {{pr[0], 0.0}, {pr[1], -pr[2]}, {pr[3], -pr[4]}};
  double v = moment_product(p, q, S);
  if (da) {
    if (ab == 2) {
      const cd p2[3] = {{k.pa[0], 0.0}, {k.pa[1], -k.pa[2]}, {k.pa[3], -k.pa[4]}};
      const cd q2[3] = {{k.dpb[0], 0.0}, {k.dpb[1], -k.dpb[2]}, {k.dpb[3], -k.dpb[4]}};
      v += moment_product(p2, q2, S);
    } else {
      v *= 2.0;
    }
  }
  return d.w * v;
}

// 2F = 2 F^T M^-1 F is unchanged by a constant invertible map of (a, b).
// Whitening by the Cholesky factor of M = [[A, C], [C, B]] in FP64 makes
// M' = I, so the FP32 epilogue sums two squares instead of cancelling terms of
// size cond(M).  m: the sums of matrix_term over the detectors.
struct Whitening {
  double l11, l21, l22, r;
  double dl11[2], dr[2], dl22[2];  // d/d alpha, d/d delta (r = C/A)
  bool valid;                      // M is positive definite
};
__host__ __device__ inline Whitening whiten(const double* m) {
  const double A = m[0], B = m[1], C = m[2];
  Whitening w;
  const double Dd = A * B - C * C;
  w.valid = A > 0.0 && Dd > 0.0 && __builtin_isfinite(Dd);
  w.l11 = sqrt(A);
  w.l21 = C / w.l11;
  w.l22 = sqrt(Dd / A);
  w.r = C / A;
  // derivatives of the whitened coefficients: a' = a / l11,
  // b' = (b - r a) / l22 with r = C/A, l11^2 = A, l22^2 = B - C^2/A
#pragma unroll
  for (int th = 0; th < 2; ++th) {
    const double dA = m[3 + 3 * th], dB = m[4 + 3 * th], dC = m[5 + 3 * th];
    w.dl11[th] = dA / (2.0 * w.l11);
    w.dr[th] = (dC * A - C * dA) / (A * A);
    w.dl22[th] = (dB - (2.0 * C * dC * A - C * C * dA) / (A * A)) / (2.0 * w.l22);
  }
  return w;
}

// Whitened, weighted coefficient q of detector X and its sky derivatives.
__host__ __device__ inline void whitened_coef(const DetConst& d, const Jks& k, const Whitening& w,
                                              int X, int q, TmplParams& tp) {
  const double bq = k.pb[q] - w.r * k.pa[q];
  tp.ca[X][q] = static_cast<float>(d.w * k.pa[q] / w.l11);
  tp.cb[X][q] = static_cast<float>(d.w * bq / w.l22);
#pragma unroll
  for (int th = 0; th < 2; ++th) {
    const double dpaq = th == 1 ? k.dpa[q] : 0.0;
    const double dpbq = th == 1 ? k.dpb[q] : 0.0;
    const double dbq = dpbq - w.dr[th] * k.pa[q] - w.r * dpaq;
    tp.dca[th][X][q] =
        static_cast<float>(d.w * (dpaq / w.l11 - k.pa[q] * w.dl11[th] / (w.l11 * w.l11)));
    tp.dcb[th][X][q] =
        static_cast<float>(d.w * (dbq / w.l22 - bq * w.dl22[th] / (w.l22 * w.l22)));
  }
}

// The first wave's share of a parameter block (block_params), in two phases with
// every lane's term[][] written between them.  matrix_lane: one matrix term per
// lane (detector x term).  coef_lane: every lane sums the terms over the
// detectors and whitens; lane 0 writes the factor and its status bit, and each
// lane one coefficient (detector x coefficient; zeros past the last detector).
constexpr int kParamLanes = 64;
static_assert(kMaxDet * kMatrixTerms <= kParamLanes && kMaxDet * 5 <= kParamLanes,
              "one wave holds the terms and the coefficients");
struct SkyAngles {
  double sa, ca, sd, cd;  // sin and cos of alpha and delta
};
__host__ __device__ inline SkyAngles sky_angles(const double* row) {
  SkyAngles s;
  sincos(row[0], &s.sa, &s.ca);
  sincos(row[1], &s.sd, &s.cd);
  return s;
}
__host__ __device__ inline void matrix_lane(const PlanConst& P, const SkyAngles& s, int lane,
                                            double (&term)[kMaxDet][kMatrixTerms]) {
  const int X = lane / kMatrixTerms, t = lane % kMatrixTerms;
  if (X < P.ndet)
    term[X][t] = matrix_term(P.det[X], P.moments + X * 10, jks_coeffs(P.det[X], s.sd, s.cd), s.sa,
                             s.ca, t);
}
__host__ __device__ inline void coef_lane(const PlanConst& P, const SkyAngles& s, int lane,
                                          const double (&term)[kMaxDet][kMatrixTerms],
                                          TmplParams& tp) {
  double m[kMatrixTerms];
#pragma unroll
  for (int t = 0; t < kMatrixTerms; ++t) {
    m[t] = 0.0;
    for (int X = 0; X < P.ndet; ++X) m[t] += term[X][t];
  }
  const Whitening w = whiten(m);
  if (lane == 0) {
    tp.status |= w.valid ? 0 : kStatusTiming;
    tp.l11 = static_cast<float>(w.l11);
    tp.l21 = static_cast<float>(w.l21);
    tp.l22 = static_cast<float>(w.l22);
  }
  const int X = lane / 5, q = lane % 5;
  if (X < P.ndet) {
    whitened_coef(P.det[X], jks_coeffs(P.det[X], s.sd, s.cd), w, X, q, tp);
  } else if (X < kMaxDet) {
    tp.ca[X][q] = tp.cb[X][q] = 0.0f;
    tp.dca[0][X][q] = tp.dcb[0][X][q] = tp.dca[1][X][q] = tp.dcb[1][X][q] = 0.0f;
  }
}

// A parameter block on the host (without the coverage check and the sky shift,
// which read the trajectory): the row's parameters, then the lanes in turn.
inline void template_params(const PlanConst& P, const double* row, TmplParams& tp) {
  row_params(P, row, tp);
  tp.tile_form = tile_form(P, tp.om_b, tp.ecc, tp.knot_log2);
  const SkyAngles s = sky_angles(row);
  double term[kMaxDet][kMatrixTerms];
  for (int lane = 0; lane < kParamLanes; ++lane) matrix_lane(P, s, lane, term);
  for (int lane = 0; lane < kParamLanes; ++lane) coef_lane(P, s, lane, term, tp);
}

// Everything the kernels need about one template, by one block of
// kParamThreads: the row's parameters, the whitened coefficients, the coverage
// check of the source-frame grid and the adjoint's sky shift.  The work is a chain of dependent FP64
// operations (about 2000 per detector in one thread), so it is bound by their
// latency and is split by what is independent: the first wave takes the
// matrix terms and then the coefficients (matrix_lane, coef_lane), the second
// solves the grid's ends, one
// lane per detector and end, and projects the sky shift.  Measured, one
// thread per template against one block: 1 template of 1 detector 11.0 to 6.5
// us, 7 of 3 detectors 26.7 to 10.4 us, 16 eccentric ones of 2 detectors 30.7
// to 10.8 us.
//
// Coverage: every sample's source time lies inside the computed grid, and
// the interpolation taps of the last sample end before the last computed
// point, so grid points beyond k_pad are exactly zero.
constexpr int kParamThreads = 128;
constexpr int kParamRowLog = 16;  // log2 of the templates in a row of k_params' blocks
static_assert(kParamThreads == 2 * kParamLanes, "two waves");
static_assert(sizeof(TmplParams) % sizeof(uint64_t) == 0, "copied in 8-byte words");
__device__ inline void block_params(const PlanConst& P, const double* __restrict__ row,
                                    TmplParams* __restrict__ out) {
  __shared__ TmplParams tp;
  __shared__ double term[kMaxDet][kMatrixTerms];
  __shared__ double shift[2];
  const int lane = threadIdx.x & 63;
  const bool first = threadIdx.x < 64;
  SkyAngles sky{};
  if (first) {
    sky = sky_angles(row);
    matrix_lane(P, sky, lane, term);
  } else {
    TmplParams rp;
    row_params(P, row, rp);
    bool bad = false;
    if (lane < 2 * P.ndet) {
      if ((rp.status & kStatusGroupMask) == 0) {
        const DetConst& d = P.det[lane >> 1];
        const double k = (lane & 1) ? double(P.k_pad - 1) : 0.0;
        const GlobalRoemer re{d.ephem, rp.nhat, P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt};
        const double u = k + d.off + grid_delay<true>(re, rp, P.tau0 + k * P.dt) * P.inv_dt;
        bad = (lane & 1) ? !(u >= double(d.n - 1 + P.D)) : !(u <= 0.0);
      }
    } else if (lane >= 62) {
      const double n[3] = {lane == 62 ? rp.dnhat[0][0] : rp.dnhat[1][0],
                           lane == 62 ? rp.dnhat[0][1] : rp.dnhat[1][1],
                           lane == 62 ? rp.dnhat[0][2] : rp.dnhat[1][2]};
      const GlobalRoemer rq{P.det[0].ephem, n, P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt};
      double dv;
      rq(P.tau0 + 0.5 * double(P.k_pad) * P.dt, shift[lane - 62], dv);
    }
    const bool uncovered = __any(bad);
    if (lane == 0) {
      tp = rp;
      tp.status |= uncovered ? kStatusCoverage : 0;
    }
  }
  __syncthreads();
  if (first) {
    if (lane < 2) tp.dshift[lane] = shift[lane];
    coef_lane(P, sky, lane, term, tp);
  } else if (lane == 0) {
    // (beside the first wave's coefficients; in row_params it delayed the grid's
    // ends, 0.4 us of 9.5 with three detectors)
    tp.tile_form = tile_form(P, tp.om_b, tp.ecc, tp.knot_log2);
  }
  __syncthreads();
  const uint64_t* src = reinterpret_cast<const uint64_t*>(&tp);
  uint64_t* dst = reinterpret_cast<uint64_t*>(out);
  for (int i = threadIdx.x; i < int(sizeof(TmplParams) / sizeof(uint64_t)); i += kParamThreads)
    dst[i] = src[i];
}

// Parameter blocks of the templates of one chunk, into their slots (one block
// each).  A call's first chunk also clears its flagged-template counter.
__global__ __launch_bounds__(kParamThreads) void k_prologue(PlanConst P,
                                                            const double* __restrict__ templates,
                                                            ChunkMap map, void* ws, int clear) {
  const int g = blockIdx.x;
  if (clear && g == 0 && threadIdx.x == 0) *flag_counter(ws) = 0ull;
  block_params(P, templates + map.tmpl[g] * P.tmpl_stride, slot_params(ws, P, g));
}

// Search path, once per run: the parameter blocks of all templates into the
// per-template array P.params, the status words of the group buffers cleared
// for the first chunk, and the flagged-template counter, the candidate count
// and the per-template maxima of the run cleared (in a kernel, so that a
// captured graph needs no memset).  One block per template (param_grid).
__global__ __launch_bounds__(kParamThreads) void k_params(PlanConst P,
                                                          const double* __restrict__ templates,
                                                          int64_t ntmpl, void* ws, int slots,
                                                          RowOutput out) {
  const int64_t t = (int64_t(blockIdx.y) << kParamRowLog) + blockIdx.x;
  if (threadIdx.x == 0) {
    if (t < slots) *group_status(ws, P, slots, int(t)) = 0;
    if (t == 0) *flag_counter(ws) = 0ull;
    if (t == 0 && out.count) *out.count = 0ull;
    if (t < ntmpl && out.best) out.best[t] = 0ull;
  }
  if (t >= ntmpl) return;
  block_params(P, templates + t * P.tmpl_stride,
               reinterpret_cast<TmplParams*>(P.params + size_t(t) * kParamBytes));
}

}  // namespace fstat
