// Host check of the FP32 gridding kernel (es_kernel.h) against its definition
// in FP64, every width, taps of random offsets.  Bound on the relative L2
// error: with the root r = sqrt(1 - z^2) in [1/2, 1] where the weights are
// large, the rounding of r and of 1 - z^2 (each uniform within half of 2^-24)
// moves the exponent beta (r - 1) by at most beta 2^-24 / sqrt(12) sqrt(1 + 1/4)
// rms, and that of z, the exponent and the result less: 2.30 W x 1.72e-8 x 1.25
// = 5e-8 W.  A constant factor on all weights counts in full.  Prints "ok".
#include <cmath>
#include <cstdio>
#include <random>

#include "es_kernel.h"

using namespace pc;

template <int W>
static bool check() {
  std::mt19937_64 g(W);
  std::uniform_real_distribution<double> U(0.0, 1.0);
  double err = 0, mag = 0;
  for (int k = 0; k < 100000; ++k) {
    const float s = (float)(-0.5 * W + U(g));
    for (int t = 0; t < W; ++t) {
      const double z = ((double)s + t) * 2.0 / W;
      const double q = 1.0 - z * z;
      const double want = std::exp(2.30 * W * (std::sqrt(q > 0 ? q : 0.0) - 1.0));
      const double d = (double)es_tap<W>(s, t) - want;
      err += d * d;
      mag += want * want;
    }
  }
  const double rel = std::sqrt(err / mag), bound = 5e-8 * W;
  const bool ok = rel <= bound && es_from_q(1.0f, es_c(W)) == 1.0f;
  std::printf("W=%d relative L2 error %.3g (bound %.3g)%s\n", W, rel, bound, ok ? "" : "  FAIL");
  return ok;
}

template <int W>
static bool all() {
  if constexpr (W > kMaxWidth) {
    return true;
  } else {
    const bool here = check<W>();
    return all<W + 1>() && here;
  }
}

int main() {
  const bool ok = all<2>();
  std::printf(ok ? "ok\n" : "FAILED\n");
  return ok ? 0 : 1;
}
