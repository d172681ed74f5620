"""The end of a Lanczos run by the share of the residual that lies along the basis:
beta^2 is a difference, and the rule stops before it loses its digits (norms of the
next basis vector emulated in extended precision stay 1 to 1e-13 where it goes on),
at every scale; zero, negative and NaN differences end the run."""
from tests.host_util import run_host


def test_rule(tmp_path):
    out = run_host(r"""
#include <cmath>
#include <cstdio>
#include <limits>
#include <random>
#include "kernels.hpp"
int main() {
  const double nan = std::numeric_limits<double>::quiet_NaN();
  for (double w2 : {1e4, 1.0, 1e-16, 1e-32, 1e-250}) {
    if (attn::lanczos_exhausted(w2, w2) || attn::lanczos_exhausted(w2, 0.02 * w2)) { std::printf("ends early\n"); return 0; }
    for (double r : {0.005, 1e-6, 1e-15, 0.0, -1e-16})
      if (!attn::lanczos_exhausted(w2, r * w2)) { std::printf("goes on at %g of %g\n", r, w2); return 0; }
  }
  if (!attn::lanczos_exhausted(nan, nan) || !attn::lanczos_exhausted(1.0, nan) || !attn::lanczos_exhausted(0.0, 0.0)) {
    std::printf("NaN or zero\n");
    return 0;
  }
  // residuals of every share: where the run goes on, beta has its digits
  std::mt19937_64 g(1);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  double worst = 0;
  for (int k = 0; k < 200000; k++) {
    const double scale = std::pow(10.0, -40 * u(g)), beta = std::pow(10.0, -12 * u(g)), h = 1.0;
    const double x = beta * scale, y = h * scale;
    const double w2 = x * x + y * y, d = w2 - y * y;   // as the kernel forms it, one coefficient
    if (attn::lanczos_exhausted(w2, d)) continue;
    worst = std::max(worst, (double)std::fabs((long double)x / std::sqrt((long double)(d < 0 ? 0 : d)) - 1));
  }
  std::printf(worst < 1e-13 && worst > 0 ? "ok\n" : "norm off by %g\n", worst);
}
""", tmp_path)
    assert out == "ok\n", out
