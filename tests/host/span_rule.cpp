// Host-only check of the rule that lets the gradient kernels take a template's
// delay derivatives as quintics per tile: at the fastest orbit the rule admits,
// the interpolant through the kernels' nodes is within 3.3e-8 of the amplitude
// of the orbit's delay and rate (0.3^6 / 23040, the bound of a sine at 0.3 rad),
// for circular and eccentric orbits alike.  Built and run by
// tests/test_host_checks.py; no GPU is touched.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>

#include "fstat_prologue.hpp"
#include "fstat_refine.hpp"

using namespace fstat;

static void orbit(double M, double ecc, double argp, double f[2]) {
  double E = M + ecc * std::sin(M);
  for (int i = 0; i < 30; ++i)
    E -= (E - ecc * std::sin(E) - M) / (1.0 - ecc * std::cos(E));
  const double q = std::sqrt(1.0 - ecc * ecc), s = std::sin(argp), c = std::cos(argp);
  f[0] = s * (std::cos(E) - ecc) + c * q * std::sin(E);
  f[1] = (c * q * std::cos(E) - s * std::sin(E)) / (1.0 - ecc * std::cos(E));
}

int main() {
  PlanConst P;
  std::memset(&P, 0, sizeof P);
  P.dt = 1.0;
  P.D = 8;
  tile_limits(P);
  const NodeFit fit = make_node_fit();
  double worst = 0.0;
  for (double ecc : {0.0, 0.02, 0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.8}) {
    // the fastest orbit the rule admits
    double lo = 0.0, hi = 1.0;
    for (int i = 0; i < 60; ++i) {
      const double om = 0.5 * (lo + hi);
      (tile_form(P, om, ecc, kKnotLogMax) != kTilePoints ? lo : hi) = om;
    }
    const double half = lo * 0.5 * kResTile;
    for (double argp : {0.0, 0.7, 1.57}) {
      double mn[2] = {9, 9}, mx[2] = {-9, -9}, err[2] = {0, 0}, f[2];
      for (int i = 0; i < 4000; ++i) {
        orbit(2.0 * kPi * i / 4000, ecc, argp, f);
        for (int q = 0; q < 2; ++q) {
          mn[q] = std::fmin(mn[q], f[q]);
          mx[q] = std::fmax(mx[q], f[q]);
        }
      }
      for (int i = -600; i <= 600; ++i) {
        // tiles everywhere, dense about periapsis
        const double m0 = kPi * std::pow(std::fabs(i / 600.0), 3.0) * (i < 0 ? -1.0 : 1.0);
        double y[kNodes][2];
        for (int n = 0; n < kNodes; ++n) orbit(m0 + half * fit.x[n], ecc, argp, y[n]);
        for (int t = 0; t <= 20; ++t) {
          const double v = -1.0 + 0.1 * t;
          orbit(m0 + half * v, ecc, argp, f);
          for (int q = 0; q < 2; ++q) {
            double p = 0.0;
            for (int j = kNodes - 1; j >= 0; --j) {
              double c = 0.0;
              for (int n = 0; n < kNodes; ++n) c += fit.m[j][n] * y[n][q];
              p = p * v + c;
            }
            err[q] = std::fmax(err[q], std::fabs(p - f[q]));
          }
        }
      }
      for (int q = 0; q < 2; ++q) {
        const double e = err[q] / (0.5 * (mx[q] - mn[q]));
        if (e > worst) {
          worst = e;
          printf("ecc %.2f argp %.2f fn %d half a tile %.4f rad: %.2e\n", ecc, argp, q, half, e);
        }
      }
    }
  }
  if (!(worst <= 3.3e-8)) {
    printf("FAIL\n");
    return 1;
  }
  printf("OK\n");
  return 0;
}
