// Host-side check of the growth factors' kept trajectory (cosmo.cpp), built
// and run by tests/test_host_growth.py: every scale factor is answered, also
// those that no trajectory reaches (infinity gives NaN, as an integration over
// an infinite step does), and a factor is the same whichever came before it.
#include <cmath>
#include <cstdio>
#include <limits>

#include "cosmo.h"

int main() {
  pm_cosmo p{};
  p.omega_m = 0.3;
  p.pk_kind = PM_PK_POWERLAW;
  p.pk_amp = 1.0;
  pmk::Cosmo c;
  c.init(p);
  double g[6], h[6];
  const double inf = std::numeric_limits<double>::infinity();
  c.growth(inf, g);
  int fails = 0;
  if (!std::isnan(g[0]) || !std::isnan(g[1]) || g[4] != std::sqrt(0.7)) {
    std::printf("FAIL growth at infinity: %g %g E %g\n", g[0], g[1], g[4]);
    ++fails;
  }
  const double a[3] = {0.5, 1.0, inf};
  double k1[2], dr[2], k2[2];
  c.step_factors(PM_INT_FASTPM, a, 3, k1, dr, k2);
  if (!std::isfinite(k1[0]) || !std::isnan(dr[1])) {
    std::printf("FAIL factors up to infinity: %g %g\n", k1[0], dr[1]);
    ++fails;
  }
  for (double x = 2e-6; x < 1e6; x *= 1.3) {
    pmk::Cosmo fresh;
    fresh.init(p);
    fresh.growth(x, g);
    c.growth(x, h);
    for (int i = 0; i < 6; ++i)
      if (!std::isfinite(g[i]) || g[i] != h[i]) {
        std::printf("FAIL growth at %g: %g %g\n", x, g[i], h[i]);
        ++fails;
      }
  }
  c.growth(1.0, g);
  if (g[0] != 1.0) {
    std::printf("FAIL D1(1) = %.17g\n", g[0]);
    ++fails;
  }
  if (fails) return 1;
  std::printf("growth check ok\n");
  return 0;
}
