// The single-bin transform and the gradient sums of templates whose timing is
// smooth over a tile (tile_form): the same quantities as k_resample_bin and
// k_grad, which solve the timing of every point and sample, from timing solved
// at knots inside the block.  No knot area exists on these paths (their
// workspace is a parameter block and 64 bytes per tile), so each block of
// kSpanTiles tiles solves its own knots, one per thread, and keeps their records
// in LDS as resample_span does.
//
// The gradient needs, at every grid point, the source-frame derivatives of the
// detector epoch and of the sample delays.  They are the same five functions:
// t_src(t; theta) inverts T(tau; theta), so
//   d delta / d theta_q (t = T) = -(dT / d theta_q) dt_src/dt,
// and they vary on the scales of the Earth's rotation and of the orbit, which a
// tile covers a fraction of.  Per tile and detector they are evaluated exactly
// (FP64) at six Chebyshev nodes and taken as quintics in between (FP32, after
// the constant of the block's dshift is off): within the limits of tile_form the
// truncation is below 3.3e-8 of their amplitude.  The
// antenna patterns and their sky derivatives are the quintic Taylor forms of the
// forward path, here up to 0.05 rad.
//
// The sum over taps with the samples' own delay derivatives,
// S_q = sum_t h_t d_q(j_t) z_j, follows from the expansion of d_q about the point,
//   S_q = d_q(u) sum h z + d_q'(u) sum h (j - u) z + d_q''(u) / 2 sum h (j - u)^2 z,
// the last term only for templates that need it (tile_form says which).  A tap
// then costs three or four accumulations instead of seven.  Without the last
// term the gradients of the fastest orbits were off by up to 3e-4 (D = 16, a
// bin at 0.49 of the sampling rate; 3e-6 with every sample's own derivative).
//
// Bound by VALU issue and, in the solves, by their latency.  Measured on 32
// templates of 2.6 M points and two detectors: the single-bin transform 2360 to
// 1500 us (four waves per SIMD; three 1645, five 1535), the gradient sums 8630
// to 2930 us (three waves per SIMD; two 3640, four 3290); the general adjoint's
// sums on four templates of 0.3 M points 149 to 64 us.
#pragma once

#include "fstat_adjoint.hpp"

namespace fstat {

constexpr int kNodes = 6;            // Chebyshev nodes per tile
constexpr int kNodeFns = 6;          // five delay derivatives and dt/dt_src

// Monomial coefficients in v in [-1, 1] of the interpolant through the values
// at the Chebyshev nodes x_n = cos(pi (2 n + 1) / (2 kNodes)): c_j = sum_n
// m[j][n] f(x_n).
struct NodeFit {
  double m[kNodes][kNodes];
  double x[kNodes];
};
__host__ __device__ constexpr NodeFit make_node_fit() {
  NodeFit f{};
  for (int n = 0; n < kNodes; ++n) {
    f.x[n] = ct_cospi(2 * n + 1, 2 * kNodes);
    double t0[kNodes] = {1.0}, t1[kNodes] = {0.0, 1.0};
    for (int d = 0; d < kNodes; ++d) {
      const double w = (d == 0 ? 1.0 : 2.0) / kNodes * ct_cospi(d * (2 * n + 1), 2 * kNodes);
      for (int j = 0; j < kNodes; ++j) f.m[j][n] += w * t0[j];
      double t2[kNodes] = {};
      for (int j = 0; j < kNodes; ++j) t2[j] = (j > 0 ? 2.0 * t1[j - 1] : 0.0) - t0[j];
      for (int j = 0; j < kNodes; ++j) {
        t0[j] = t1[j];
        t1[j] = t2[j];
      }
    }
  }
  return f;
}
static __device__ const NodeFit kNodeFit = make_node_fit();

// LDS of a block besides the windows and their records.
struct SpanSolve {
  double2 gk[kMaxDet][kSpanGrid];      // grid knots (q, dq/dk)
  double2 sk[kMaxDet][kSpanSamp + 1];  // sample knots (phase, change per sample)
  int bad;
};

// Lanes of a detector's wave: grid knots first, then the derivative nodes.
constexpr int kNodeLane = 40;
static_assert(kSpanGrid <= kNodeLane && kNodeLane + kSpanTiles * kNodes <= 64,
              "one wave solves a detector's knots and nodes");
static_assert(kMaxDet * 64 <= kResThreads, "one wave per detector");

// Solves the timing of n_t tiles from t0 on and stages their corrected samples
// (all detectors), as resample_span leaves them: zsa, recs, and the windows'
// first samples ja.  node(X, lane, tau, re) is called by the lanes from
// kNodeLane on with the source time of their derivative node.  False (uniform)
// after flagging the template: also where a delay exceeds the plan's max_delay
// by more than `reach` samples and one trajectory interval (the general kernels
// stage the trajectory that far: k_resample_bin D + 2 + 64 samples, k_grad D + 2).
template <int D, bool KEP, class Node>
__device__ __forceinline__ bool span_solve(const PlanConst& P, const TmplParams& tp, int kl,
                                           int reach, int32_t* status_word, int32_t t0, int n_t,
                                           float2* zsa,
                                           SpanRec* recs, SpanSolve& sv, int32_t (&ja)[kMaxDet],
                                           Node&& node) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w0 = uniform_i32(tid) & ~63;
  const int G = 1 << kl;
  const int32_t k_s = t0 << kResTileLog;
  const int ng = ((n_t << kResTileLog) >> kl) + 1;
  const double limit = P.max_delay + double(reach) * P.dt + P.eph_dt;
  if (tid == 0) sv.bad = 0;
  __syncthreads();
  const int X = w0 >> 6;
  const bool mine = X < P.ndet;
  const DetConst& d = P.det[mine ? X : 0];
  const CachedRoemer re{d.ephem, tp.nhat, P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt};
  if (mine) {
    // knots and nodes in one solve
    const int nl = lane - kNodeLane;
    const bool is_node = nl >= 0 && nl < n_t * kNodes;
    if (lane < ng || is_node) {
      const double k = is_node ? double(k_s) + kResTile * (nl / kNodes + 0.5) +
                                     0.5 * kResTile * kNodeFit.x[nl % kNodes]
                               : double(k_s + lane * G);
      bool far;
      const double2 kv = grid_knot<KEP>(P, tp, re, k, limit, far);
      if (far) sv.bad = 1;
      if (is_node) {
        node(X, nl, k, kv);
      } else {
        sv.gk[X][lane] = kv;
      }
    }
  }
  __syncthreads();
  // windows: floor of the source position at the tiles' first points and past
  // the span, as the grid records round it
  int32_t W[kMaxDet];
  bool wbad = false;
#pragma unroll
  for (int Y = 0; Y < kMaxDet; ++Y) {
    ja[Y] = W[Y] = 0;
    if (Y >= P.ndet) break;
    int32_t j[kSpanTiles + 1];
#pragma unroll
    for (int h = 0; h <= kSpanTiles; ++h) {
      const int32_t k = (h < n_t ? h : n_t) * kResTile;
      const double a = P.det[Y].off + sv.gk[Y][k >> kl].x;
      const double fa = floor(a);
      j[h] = uniform_i32(k_s + k + int32_t(fa) + (float(a - fa) >= 1.0f ? 1 : 0));
    }
    ja[Y] = (j[0] - D + 1) & ~((1 << kKnotLogMax) - 1);
#pragma unroll
    for (int h = 0; h < kSpanTiles; ++h) {
      const int32_t nwin = j[h + 1] - j[h] + 2 * D;
      // delay drift beyond 1/16 per tile: flag the template (NaN output)
      wbad |= h < n_t && (nwin > kResWcap || nwin < 2 * D);
    }
    W[Y] = j[kSpanTiles] + D - ja[Y] + 1;
  }
  if (wbad || sv.bad) {
    if (tid == 0) atomicOr(status_word, wbad ? kStatusWindow : kStatusNodes);
    return false;
  }
  if (mine && lane < ng)
    grid_record(d.off, sv.gk[X][lane], sv.gk[X][lane + 1 < ng ? lane + 1 : lane], double(G),
                lane == ng - 1, recs[X].grid[lane], recs[X].grid_i[lane]);
  const int32_t jx = X == 0 ? ja[0] : X == 1 ? ja[1] : X == 2 ? ja[2] : ja[3];
  const int32_t wx = X == 0 ? W[0] : X == 1 ? W[1] : X == 2 ? W[2] : W[3];
  const int ns = ((wx - 1) >> kl) + 2;
#pragma unroll
  for (int X0 = 0; X0 < kMaxDet; X0 += kDetPass) {
    if (X0 >= P.ndet) break;
    // the samples of two detectors, in flight while the sample knots are
    // solved
    float2 xv[kDetPass][kStageRounds];
    auto sample = [&](int xp, int w) {
      const DetConst& dx = P.det[X0 + xp];
      const int32_t js = ja[X0 + xp] + w;
      const bool in = w < W[X0 + xp] && uint32_t(js) < uint32_t(dx.n);
      return in ? dx.x[js] : make_float2(0.f, 0.f);
    };
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      if (X0 + xp >= P.ndet) break;
#pragma unroll
      for (int r = 0; r < kStageRounds; ++r) xv[xp][r] = sample(xp, r * kResThreads + tid);
    }
    if (X0 == 0) {
      if (mine && lane < ns) {
        double ph, dph, delay;
        sample_phase_d<KEP>(re, tp, d.t0 + P.dt * double(jx + lane * G), P.f_het, ph, dph, delay);
        sv.sk[X][lane] = make_double2(ph, dph * P.dt);
      }
      __syncthreads();
      if (mine && lane < ns - 1)
        sample_record(sv.sk[X][lane], sv.sk[X][lane + 1], double(G), recs[X].samp[lane][0],
                      recs[X].samp[lane][1]);
      __syncthreads();
    }
    // corrected samples z_j = x_j exp(-2 pi i f_h (t_src,j - t_j)); a zero
    // sample (outside the data, or in a gap) stays zero
#pragma unroll
    for (int xp = 0; xp < kDetPass; ++xp) {
      if (X0 + xp >= P.ndet) break;
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
        if (w < W[X0 + xp]) zx[w] = z;
        // which 32-sample blocks of the window hold a live sample
        const unsigned long long mb = __ballot(live);
        if (lane == 0) {
          rec.blk[wu >> 5] = uint32_t(mb) != 0u;
          rec.blk[(wu >> 5) + 1] = uint32_t(mb >> 32) != 0u;
        }
      };
#pragma unroll
      for (int r = 0; r < kStageRounds; ++r) {
        if (r * kResThreads + w0 >= W[X0 + xp]) break;
        put(r * kResThreads + w0, xv[xp][r]);
      }
#pragma unroll 1
      for (int wu = kStageRounds * kResThreads + w0; wu < W[X0 + xp]; wu += kResThreads)
        put(wu, sample(xp, wu + lane));
    }
  }
  return true;
}

// A grid point's first tap in its window, the fraction f of the point past
// the tap before it, and whether any tap falls on a live sample (mask: the
// window's live blocks).  theta + whole: the source position.
struct SpanPoint {
  int base;
  float f, th;
  int32_t im;
  bool live;
};
template <int D>
__device__ __forceinline__ SpanPoint span_point(const SpanRec& rec, unsigned long long mask,
                                                int kl, int32_t k_rel, int32_t sb) {
  const int G = 1 << kl;
  const float4 cq = rec.grid[k_rel >> kl];
  SpanPoint p;
  p.im = rec.grid_i[k_rel >> kl];
  const float v = float(k_rel & (G - 1)) * (1.0f / float(G));
  p.th = fmaf(fmaf(fmaf(cq.w, v, cq.z), v, cq.y), v, cq.x);
  const float fl = floorf(p.th);
  p.f = p.th - fl;
  int base = sb + p.im + int(fl);
  if (p.f >= 1.0f) {
    p.f = 0.0f;
    base += 1;
  }
  // monotonic T_k keeps the taps in the window, the clamp guards memory
  p.base = base < 0 ? 0 : (base > kSpanCap - 2 * D ? kSpanCap - 2 * D : base);
  p.live = ((mask >> (p.base >> 5)) & 3u) != 0u;
  return p;
}
__device__ __forceinline__ unsigned long long span_mask(const SpanRec& rec, int lane) {
  return __ballot(lane < kSpanBlk && rec.blk[lane < kSpanBlk ? lane : 0]);
}

// The antenna Taylor records of the tiles (the middle point's position and the
// coefficients of the patterns ka, kb) into out[0 .. kTaylorCoef + 2).
__device__ __forceinline__ void tile_antenna(const PlanConst& P, const TmplParams& tp, int X,
                                             const SpanSolve& sv, int kl, int32_t t0, int h,
                                             const float* ka, const float* kb, float* out) {
  const int32_t k = h * kResTile + kResTile / 2;
  const double q = sv.gk[X][k >> kl].x;
  float c[kTaylorCoef];
  antenna_taylor(ka, kb,
                 tp.alpha_cyc[X] -
                     P.sid_rate_cyc * (P.tau0 + P.dt * (double((t0 << kResTileLog) + k) + q)),
                 c);
#pragma unroll
  for (int n = 0; n < kTaylorCoef; ++n) out[n] = c[n];
  const double a = P.det[X].off + q;
  const double fa = floor(a);
  out[kTaylorCoef] = float(a - fa);
  out[kTaylorCoef + 1] = __int_as_float(int32_t(fa));
}

// exp(-i (spin-down phase and offset)) exp(-2 pi i nat k / N): both phases in
// quarter turns (the second's share reduced exactly in integers), one rotation.
__device__ __forceinline__ float2 bin_rotation(const double sd[4], int64_t nat, int64_t k,
                                               int64_t n_fft) {
  const double x = double(int32_t(k));
  const double c4 = fma(x, fma(x, fma(x, sd[3], sd[2]), sd[1]), sd[0]) +
                    double((nat * k) & (n_fft - 1)) * (4.0 / double(n_fft));
  const double q = rint(c4);
  const float2 e = cis_quarter(int(q), static_cast<float>(c4 - q));
  return make_float2(e.x, -e.y);
}

// Sums of NQ values over the block, in a fixed order, by the first NQ threads.
template <int NQ>
__device__ __forceinline__ double block_sum(const double (&s)[NQ]) {
  __shared__ double red[kResThreads / 64][NQ];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double v = s[q];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) red[wave][q] = v;
  }
  __syncthreads();
  double v = 0.0;
  if (threadIdx.x < NQ)
    for (int w = 0; w < kResThreads / 64; ++w) v += red[w][threadIdx.x];
  return v;
}

// k_resample_bin for the templates of tile_form: kSpanTiles tiles per block
// (one tile at a time at a knot spacing of 16); the block's sums go to its
// first tile's partials, zeros to the others'.
template <int D, bool KEP>
__global__ __launch_bounds__(kResThreads, 4) void k_bin_span(PlanConst P, void* ws, ChunkMap map,
                                                            const int64_t* __restrict__ bins) {
  extern __shared__ float2 zs[];
  __shared__ SpanSolve sv;
  const int slot = blockIdx.y;
  TmplParams* tpp = slot_params(ws, P, slot);
  const TmplParams& tp = *tpp;
  if (tp.status != 0 || tp.tile_form == kTilePoints) return;
  SpanRec* recs = reinterpret_cast<SpanRec*>(zs + P.ndet * kSpanCap);
  const int tid = threadIdx.x, lane = tid & 63;
  const int kl = uniform_i32(tp.knot_log2);
  const int32_t tiles = int32_t(P.k_pad >> kResTileLog);
  const int32_t t_b = int32_t(blockIdx.x) * kSpanTiles;
  const int32_t t_e = t_b + kSpanTiles < tiles ? t_b + kSpanTiles : tiles;
  const int step = kl > kKnotLogGlobal ? kSpanTiles : 1;
  const int64_t nat = band_bin_nat(P, bins[map.tmpl[slot]]);
  // d(angle)/d(grid step) of the sidereal angle x, radians
  const float dstep = float(-2.0 * kPi * P.sid_rate_cyc * P.dt);
  double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int32_t t0 = t_b; t0 < t_e; t0 += step) {
    const int n_t = t_e - t0 < step ? t_e - t0 : step;
    int32_t ja[kMaxDet];
    if (!span_solve<D, KEP>(P, tp, kl, D + 2 + (1 << kKnotLogMax), &tpp->status, t0, n_t, zs, recs,
                            sv, ja, [](int, int, double, double2) {}))
      return;
    {
      const int X = tid >> 6;
      if (X < P.ndet && lane < n_t)
        tile_antenna(P, tp, X, sv, kl, t0, lane, tp.ca[X], tp.cb[X], recs[X].tile[lane]);
    }
    __syncthreads();
#pragma unroll 1
    for (int h = 0; h < n_t; ++h) {
      const int32_t k_t = (t0 + h) << kResTileLog;
      float2 acc_a[kResPerThread], acc_b[kResPerThread];
#pragma unroll
      for (int i = 0; i < kResPerThread; ++i) acc_a[i] = acc_b[i] = make_float2(0.f, 0.f);
#pragma unroll 1
      for (int X = 0; X < P.ndet; ++X) {
        const SpanRec& rec = recs[X];
        const int32_t jx = X == 0 ? ja[0] : X == 1 ? ja[1] : X == 2 ? ja[2] : ja[3];
        const unsigned long long mask = span_mask(rec, lane);
        const float* tr = rec.tile[h];
        const float th_r = tr[kTaylorCoef];
        const int32_t i_r = __float_as_int(tr[kTaylorCoef + 1]);
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i) {
          const int kk = tid + i * kResThreads;
          const SpanPoint p = span_point<D>(rec, mask, kl, h * kResTile + kk,
                                            k_t + kk - jx - (D - 1));
          if (!p.live) continue;
          const float dx = (float(kk - kResTile / 2 + (p.im - i_r)) + (p.th - th_r)) * dstep;
          weight_taylor(sinc_interp<D>(p.f, zs + X * kSpanCap + p.base), dx, tr, acc_a[i],
                        acc_b[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < kResPerThread; ++i) {
        const float2 e = bin_rotation(tp.sd, nat, k_t + tid + i * kResThreads, P.n_fft);
        const float2 ya = cmul(acc_a[i], e), yb = cmul(acc_b[i], e);
        s[0] += double(ya.x);
        s[1] += double(ya.y);
        s[2] += double(yb.x);
        s[3] += double(yb.y);
      }
    }
    __syncthreads();  // the next span rewrites the windows
  }
  const double v = block_sum<4>(s);
  double* partial = slot_partials(ws, P, slot) + size_t(t_b) * 8;
  if (tid < 4) {
    partial[tid] = v;
    for (int t = t_b + 1; t < t_e; ++t) partial[(t - t_b) * 8 + tid] = 0.0;
  }
}

// The sums of the gradient over one point's taps: sum h z, sum h' z,
// sum h (j - u) z and (CURVED) sum h (j - u)^2 z.
struct TapSums {
  float2 z, dz, jz, jjz;
};
template <int D, int M, bool CURVED>
__device__ __forceinline__ void grad_pair(float g, float u, const float2* zp, TapSums& s) {
  float hp, hm;
  tap_pair<D, M>(g, u, hp, hm);
  constexpr TapPoly q = make_tap_poly<D, M, true>();
  float e = __fmul_rn(u, q.e[kTapCoef - 1]), o = __fmul_rn(u, q.o[kTapCoef - 1]);
  e = __fadd_rn(e, q.e[kTapCoef - 2]);
  o = __fadd_rn(o, q.o[kTapCoef - 2]);
#pragma unroll
  for (int i = kTapCoef - 3; i >= 0; --i) {
    e = fmaf(e, u, q.e[i]);
    o = fmaf(o, u, q.o[i]);
  }
  const float dp = fmaf(g, o, e), dm = fmaf(g, o, -e);
  constexpr float c = float(M) + 0.5f;
  const float cp = hp * c, cm = hm * c;
  const float2 zl = zp[D - 1 - M], zr = zp[D + M];
  s.z.x = fmaf(hm, zr.x, fmaf(hp, zl.x, s.z.x));
  s.z.y = fmaf(hm, zr.y, fmaf(hp, zl.y, s.z.y));
  s.dz.x = fmaf(dm, zr.x, fmaf(dp, zl.x, s.dz.x));
  s.dz.y = fmaf(dm, zr.y, fmaf(dp, zl.y, s.dz.y));
  // h (s - g) z, s = u - j: +(M + 1/2) on the left, -(M + 1/2) on the right
  s.jz.x = fmaf(-cm, zr.x, fmaf(cp, zl.x, s.jz.x));
  s.jz.y = fmaf(-cm, zr.y, fmaf(cp, zl.y, s.jz.y));
  if constexpr (CURVED) {
    const float ccp = cp * c, ccm = cm * c;
    s.jjz.x = fmaf(ccm, zr.x, fmaf(ccp, zl.x, s.jjz.x));
    s.jjz.y = fmaf(ccm, zr.y, fmaf(ccp, zl.y, s.jjz.y));
  }
}
template <int D, bool CURVED, int... M>
__device__ __forceinline__ TapSums grad_taps(std::integer_sequence<int, M...>, float f,
                                             const float2* zp) {
  const float g = f - 0.5f, u = g * g;
  TapSums s;
  s.z = s.dz = s.jz = s.jjz = make_float2(0.f, 0.f);
  (grad_pair<D, D - 1 - M, CURVED>(g, u, zp, s), ...);
  // sum h (j - u)^2 z = sum h s^2 z, s = g + (s - g)
  if constexpr (CURVED) {
    s.jjz.x = fmaf(g, fmaf(g, s.z.x, 2.0f * s.jz.x), s.jjz.x);
    s.jjz.y = fmaf(g, fmaf(g, s.z.y, 2.0f * s.jz.y), s.jjz.y);
  }
  // sum h (j - u) z = -sum h s z
  s.jz.x = -fmaf(g, s.z.x, s.jz.x);
  s.jz.y = -fmaf(g, s.z.y, s.jz.y);
  return s;
}

// Value and derivative of a quintic pair (antenna patterns a, b in the angle).
__device__ __forceinline__ void taylor_pair(const float* c, float d, float& a, float& b) {
  a = c[5];
  b = c[11];
#pragma unroll
  for (int n = 4; n >= 0; --n) {
    a = fmaf(a, d, c[n]);
    b = fmaf(b, d, c[6 + n]);
  }
}
__device__ __forceinline__ void taylor_slope(const float* c, float d, float& a, float& b) {
  a = 5.0f * c[5];
  b = 5.0f * c[11];
#pragma unroll
  for (int n = 4; n >= 1; --n) {
    a = fmaf(a, d, float(n) * c[n]);
    b = fmaf(b, d, float(n) * c[6 + n]);
  }
}

// Per-block tables of k_grad_span besides the windows and their records.
struct GradLds {
  SpanSolve sv;
  double nodes[kMaxDet][kSpanTiles * kNodes][kNodeFns];
  float dpoly[kMaxDet][kSpanTiles][kNodeFns][kNodes];
  float dant[kMaxDet][kSpanTiles][2][kTaylorCoef + 2];
};
// The spans of one block (see the head of this file), with the curvature of the
// delay derivatives over the taps or without it.
template <int D, bool ONEHOT, bool KEP, bool CURVED>
__device__ __forceinline__ void grad_span(const PlanConst& P, void* ws, float2* zs, GradLds& lds) {
  SpanSolve& sv = lds.sv;
  auto& nodes = lds.nodes;
  auto& dpoly = lds.dpoly;
  auto& dant = lds.dant;
  const int slot = blockIdx.y;
  TmplParams* tpp = slot_params(ws, P, slot);
  const TmplParams& tp = *tpp;
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t tiles = int32_t(P.k_pad >> kResTileLog);
  const int32_t t_b = int32_t(blockIdx.x) * kSpanTiles;
  const int32_t t_e = t_b + kSpanTiles < tiles ? t_b + kSpanTiles : tiles;
  double* partial = slot_partials(ws, P, slot) + size_t(t_b) * 8;
  if (tp.status != 0) {
    if (tid < 8)
      for (int t = t_b; t < t_e; ++t) partial[(t - t_b) * 8 + tid] = 0.0;
    return;
  }
  if (tp.tile_form == kTilePoints) return;
  SpanRec* recs = reinterpret_cast<SpanRec*>(zs + P.ndet * kSpanCap);
  const int kl = uniform_i32(tp.knot_log2);
  const int step = kl > kKnotLogGlobal ? kSpanTiles : 1;
  const bool binary = tp.asini != 0.0;
  const float dstep = float(-2.0 * kPi * P.sid_rate_cyc * P.dt);
  const float omega = float(2.0 * kPi * P.sid_rate_cyc);
  const float two_pi_fh = float(2.0 * kPi * P.f_het);
  const float inv_dt = float(P.inv_dt);
  const float shift0 = float(tp.dshift[0]), shift1 = float(tp.dshift[1]);
  const float2 ha = ONEHOT ? make_float2(float(tp.hbin[0]), float(tp.hbin[1]))
                           : make_float2(0.f, 0.f);
  const float2 hb = ONEHOT ? make_float2(float(tp.hbin[2]), float(tp.hbin[3]))
                           : make_float2(0.f, 0.f);
  double acc[kGradParams];
#pragma unroll
  for (int q = 0; q < kGradParams; ++q) acc[q] = 0.0;
#pragma unroll 1
  for (int32_t t0 = t_b; t0 < t_e; t0 += step) {
    const int n_t = t_e - t0 < step ? t_e - t0 : step;
    int32_t ja[kMaxDet];
    // the delay derivatives d(t_src - t)/d theta at the sample time T of the
    // node, as k_grad takes them at every sample, and dt/dt_src
    auto node = [&](int X, int n, double k, double2 kv) {
      const double tau = P.tau0 + P.dt * k, T = tau + kv.x * P.dt;
      const DetConst& d = P.det[X];
      double v, rd, ra, rl, slope;
      GlobalRoemer{d.ephem, tp.nhat, P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt}(T, v, rd);
      GlobalRoemer{d.ephem, tp.dnhat[0], P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt}(T, ra, slope);
      GlobalRoemer{d.ephem, tp.dnhat[1], P.n_eph, P.eph_t0, P.eph_dt, P.inv_eph_dt}(T, rl, slope);
      double rb = 0.0, rbp = 0.0;
      if (binary) orbit_delay<KEP>(tp, tau, rb, rbp);
      const double invb = 1.0 / (1.0 + rbp);
      double* o = nodes[X][n];
      o[0] = ra * invb - tp.dshift[0];
      o[1] = rl * invb - tp.dshift[1];
      o[2] = binary ? -rb / tp.asini * invb : 0.0;
      o[3] = binary ? rbp * (tau - tp.tp) / tp.porb * invb : 0.0;
      o[4] = rbp * invb;
      o[5] = (1.0 + rbp) / (1.0 + rd);
    };
    if (!span_solve<D, KEP>(P, tp, kl, D + 2, &tpp->status, t0, n_t, zs, recs, sv, ja, node)) {
      if (tid < 8)
        for (int t = t_b; t < t_e; ++t) partial[(t - t_b) * 8 + tid] = __builtin_nan("");
      return;
    }
    {
      const int X = tid >> 6;
      if (X < P.ndet) {
        // quintics of the node functions, then the antenna records: the
        // patterns and their derivatives with respect to alpha and delta
        for (int e = lane; e < n_t * kNodeFns * kNodes; e += 64) {
          const int j = e % kNodes, fn = e / kNodes % kNodeFns, h = e / (kNodes * kNodeFns);
          double c = 0.0;
#pragma unroll
          for (int n = 0; n < kNodes; ++n) c += kNodeFit.m[j][n] * nodes[X][h * kNodes + n][fn];
          dpoly[X][h][fn][j] = float(c);
        }
        if (lane < 3 * n_t) {
          const int h = lane / 3, set = lane % 3;
          const float* ka = set == 0 ? tp.ca[X] : tp.dca[set - 1][X];
          const float* kb = set == 0 ? tp.cb[X] : tp.dcb[set - 1][X];
          tile_antenna(P, tp, X, sv, kl, t0, h, ka, kb,
                       set == 0 ? recs[X].tile[h] : dant[X][h][set - 1]);
        }
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int h = 0; h < n_t; ++h) {
      const int32_t k_t = (t0 + h) << kResTileLog;
      // adjoint weights W_k = X_k E_k (the conjugate pass stored conj(X))
      float2 Wa[kResPerThread], Wb[kResPerThread];
#pragma unroll
      for (int i = 0; i < kResPerThread; ++i) {
        const int64_t k = k_t + tid + i * kResThreads;
        if (ONEHOT) {
          const float2 e = bin_rotation(tp.sd, tp.bin_nat, k, P.n_fft);
          Wa[i] = cmul(ha, e);
          Wb[i] = cmul(hb, e);
        } else {
          const float2 e = spindown_rotation(tp.sd, k);
          const float2 ya = slot_buf(ws, P, slot, 0)[k], yb = slot_buf(ws, P, slot, 1)[k];
          Wa[i] = cmul(make_float2(ya.x, -ya.y), e);
          Wb[i] = cmul(make_float2(yb.x, -yb.y), e);
        }
      }
#pragma unroll 1
      for (int X = 0; X < P.ndet; ++X) {
        const SpanRec& rec = recs[X];
        const int32_t jx = X == 0 ? ja[0] : X == 1 ? ja[1] : X == 2 ? ja[2] : ja[3];
        const unsigned long long mask = span_mask(rec, lane);
        const float* tr = rec.tile[h];
        const float th_r = tr[kTaylorCoef];
        const int32_t i_r = __float_as_int(tr[kTaylorCoef + 1]);
#pragma unroll
        for (int i = 0; i < kResPerThread; ++i) {
          const int kk = tid + i * kResThreads;
          const SpanPoint p = span_point<D>(rec, mask, kl, h * kResTile + kk,
                                            k_t + kk - jx - (D - 1));
          if (!p.live) continue;
          const TapSums s = grad_taps<D, CURVED>(std::make_integer_sequence<int, D>{}, p.f,
                                                  zs + X * kSpanCap + p.base);
          const float dx = (float(kk - kResTile / 2 + (p.im - i_r)) + (p.th - th_r)) * dstep;
          const float2 wa = Wa[i], wb = Wb[i];
          // W = X (a', b') and its derivatives in the angle, alpha and delta
          float a, b;
          taylor_pair(tr, dx, a, b);
          const float wr = fmaf(wa.x, a, wb.x * b), wi = fmaf(wa.y, a, wb.y * b);
          // Re(W dz), Im(W z), Im(W sum h (j - u) z)
          const float r1 = fmaf(wr, s.dz.x, -(wi * s.dz.y));
          const float i0 = fmaf(wr, s.z.y, wi * s.z.x);
          const float i1 = fmaf(wr, s.jz.y, wi * s.jz.x);
          // Re(dW z)
          const float ua = fmaf(wa.x, s.z.x, -(wa.y * s.z.y));
          const float ub = fmaf(wb.x, s.z.x, -(wb.y * s.z.y));
          taylor_slope(tr, dx, a, b);
          const float rx = fmaf(ua, a, ub * b);
          taylor_pair(dant[X][h][0], dx, a, b);
          const float ral = fmaf(ua, a, ub * b);
          taylor_pair(dant[X][h][1], dx, a, b);
          const float rde = fmaf(ua, a, ub * b);
          const double dtau0 = P.dt * double(k_t + kk);
          const double dtr = P.tau0 + dtau0 - P.t_ref;
          acc[0] += dtau0 * double(i0);
          acc[1] += 0.5 * dtr * dtr * double(i0);
          // dT_q = -(d_q + shift_q) dt/dt_src; the kernel's share of the epoch
          // is r1 / dt, the antenna's -omega rx
          const float v = float(kk - kResTile / 2) * (2.0f / float(kResTile));
          const float* ct = dpoly[X][h][5];
          float inv_tau = ct[kNodes - 1];
#pragma unroll
          for (int n = kNodes - 2; n >= 0; --n) inv_tau = fmaf(inv_tau, v, ct[n]);
          const float pt = inv_tau * fmaf(omega, rx, -(r1 * inv_dt));
          const float q0 = two_pi_fh * i0;
          // d_q' per sample: d/dv over half a tile of grid steps, dt_src/dt
          // steps per sample (1 / inv_tau, first order)
          const float vj = (2.0f / float(kResTile)) * (2.0f - inv_tau);
          const float q1 = two_pi_fh * i1 * vj;
          float q2 = 0.0f;
          if constexpr (CURVED)  // Im(W sum h (j - u)^2 z)
            q2 = two_pi_fh * fmaf(wr, s.jjz.y, wi * s.jjz.x) * (vj * vj);
#pragma unroll
          for (int q = 0; q < 5; ++q) {
            const float* c = dpoly[X][h][q];
            // value, slope and half the second derivative
            float dv = c[kNodes - 1], ds = 0.0f, dc = 0.0f;
#pragma unroll
            for (int n = kNodes - 2; n >= 0; --n) {
              if constexpr (CURVED) dc = fmaf(dc, v, ds);
              ds = fmaf(ds, v, dv);
              dv = fmaf(dv, v, c[n]);
            }
            const float full = q == 0 ? dv + shift0 : q == 1 ? dv + shift1 : dv;
            float m = fmaf(full, pt, fmaf(dv, q0, CURVED ? fmaf(ds, q1, dc * q2) : ds * q1));
            if (q == 0) m += rx + ral;
            if (q == 1) m += rde;
            acc[2 + q] += double(m);
          }
        }
      }
    }
    __syncthreads();  // the next span rewrites the windows
  }
  acc[0] *= 8.0 * kPi;
  acc[1] *= 8.0 * kPi;
#pragma unroll
  for (int q = 2; q < kGradParams; ++q) acc[q] *= 4.0;
  const double v = block_sum<kGradParams>(acc);
  if (tid < kGradParams) {
    partial[tid] = v;
    for (int t = t_b + 1; t < t_e; ++t) partial[(t - t_b) * 8 + tid] = 0.0;
  }
}

// k_grad for the templates of tile_form.  The choice between the two forms is
// taken once per block, around the whole body: taken per tile the registers of
// both were live at once (32 templates of 2.6 M points, smooth ones: 4380 us a
// call with the smooth form alone, 4400 so, 4420 per span, 4495 per tile, 4610
// with every template in the curved form).
template <int D, bool ONEHOT, bool KEP>
__global__ __launch_bounds__(kResThreads, 3) void k_grad_span(PlanConst P, void* ws) {
  extern __shared__ float2 zs[];
  __shared__ GradLds lds;
  if (uniform_i32(slot_params(ws, P, blockIdx.y)->tile_form) == kTileCurved)
    grad_span<D, ONEHOT, KEP, true>(P, ws, zs, lds);
  else
    grad_span<D, ONEHOT, KEP, false>(P, ws, zs, lds);
}

}  // namespace fstat
