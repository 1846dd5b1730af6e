// Host-only check of a parameter block's lanes (matrix_lane, coef_lane: the code
// the kernels run, one lane after the other) at every detector count: over the
// valid samples the whitened antenna patterns must be orthonormal,
//   sum_X w_X sum_t a'^2 = sum_X w_X sum_t b'^2 = 1, sum_X w_X sum_t a' b' = 0
// (the stored coefficients carry the weight w_X, so each product is divided by
// it), whatever lane computed which term or coefficient, and the
// coefficients past the last detector must be zero.  FP32 coefficients: 1e-6.
// Built and run by tests/test_host_checks.py; no GPU is touched.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>

#include "fstat_prologue.hpp"

using namespace fstat;

int main() {
  const double rate = 2.0 * kPi / 86164.0905;
  double worst = 0.0;
  for (int ndet = 1; ndet <= kMaxDet; ++ndet) {
    PlanConst P;
    std::memset(&P, 0, sizeof P);
    P.ndet = ndet;
    P.D = 8;
    P.dt = 60.0;
    P.max_delay = 600.0;
    P.sid_rate_cyc = rate / (2.0 * kPi);
    double moments[kMaxDet * 10] = {};
    const double wgt[4] = {1.0, 0.8, 1.7, 0.4};
    double phi[kMaxDet][1500];
    int n[kMaxDet];
    for (int X = 0; X < ndet; ++X) {
      DetConst& d = P.det[X];
      d.lat = 0.81 - 0.4 * X;
      d.gamma = 2.98 + 0.9 * X;
      d.sl = std::sin(d.lat);
      d.cl = std::cos(d.lat);
      d.s2g = std::sin(2.0 * d.gamma);
      d.c2g = std::cos(2.0 * d.gamma);
      d.w = wgt[X];
      d.lst0_cyc = -0.33 + 0.21 * X;
      n[X] = 0;
      for (int j = 0; j < 1500; ++j) {
        if (j > 300 + 100 * X && j < 500 + 50 * X) continue;
        const double p = 2.0 * kPi * d.lst0_cyc + rate * 60.0 * j;
        phi[X][n[X]++] = p;
        for (int k = 0; k < 5; ++k) {
          moments[X * 10 + 2 * k] += std::cos(k * p);
          moments[X * 10 + 2 * k + 1] += std::sin(k * p);
        }
      }
    }
    P.moments = moments;
    const double row[8] = {1.3, -0.4, 0.0, 0.0, 0.0, 0.0, 1.0, 0.0};
    TmplParams tp;
    std::memset(&tp, 0xff, sizeof tp);
    template_params(P, row, tp);
    if (tp.status != 0) {
      printf("FAIL status %d at %d detectors\n", tp.status, ndet);
      return 1;
    }
    double aa = 0.0, bb = 0.0, ab = 0.0;
    for (int X = 0; X < ndet; ++X)
      for (int j = 0; j < n[X]; ++j) {
        const double x = row[0] - phi[X][j];
        const double bas[5] = {1.0, std::cos(x), std::sin(x), std::cos(2 * x), std::sin(2 * x)};
        double a = 0.0, b = 0.0;
        for (int q = 0; q < 5; ++q) {
          a += tp.ca[X][q] * bas[q];
          b += tp.cb[X][q] * bas[q];
        }
        aa += a * a / wgt[X];
        bb += b * b / wgt[X];
        ab += a * b / wgt[X];
      }
    const double e = std::fmax(std::fabs(aa - 1.0), std::fmax(std::fabs(bb - 1.0), std::fabs(ab)));
    printf("%d detectors: %.2e\n", ndet, e);
    worst = std::fmax(worst, e);
    for (int X = ndet; X < kMaxDet; ++X)
      for (int q = 0; q < 5; ++q)
        for (int th = 0; th < 2; ++th)
          if (tp.ca[X][q] != 0.0f || tp.cb[X][q] != 0.0f || tp.dca[th][X][q] != 0.0f ||
              tp.dcb[th][X][q] != 0.0f) {
            printf("FAIL coefficient past the last detector\n");
            return 1;
          }
  }
  if (!(worst <= 1e-6)) {
    printf("FAIL\n");
    return 1;
  }
  printf("OK\n");
  return 0;
}
