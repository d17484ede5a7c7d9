// The gridding kernel in FP32, the exponential of semicircle
//   phi(z) = exp(beta (sqrt(1 - z^2) - 1)),  |z| <= 1,  beta = kEsBeta W,
// as the spread, the interpolation and the w-planes evaluate it (host and
// device: its error is checked on the host, see tests/test_host_fft.py).
#ifndef PC_ES_KERNEL_H
#define PC_ES_KERNEL_H

#include <cmath>

#include "common.h"

namespace pc {

// phi from q = 1 - z^2 as exp2(c sqrt(q) - c) with one rounded constant
// c = beta log2(e): the peak is exactly one at every width.  (Two constants,
// c0 and c1 = c0 / R for sqrt(R^2 - x^2), put a factor of up to 1 +- 1e-6 on
// all weights, and a root in [R/2, R] rounds up to twice as coarsely as one in
// [1/2, 1].)  Relative L2 error of the weights on the device: 2.9e-7, 3.5e-7 and
// 4.3e-7 at W = 6, 7 and 9, with two constants 7.3e-7, 4.4e-7 and 1.0e-6.
// max(., 0) absorbs rounding at |z| = 1.
__host__ __device__ __forceinline__ float es_from_q(float q, float c) {
  q = q > 0.0f ? q : 0.0f;
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_exp2f(__builtin_fmaf(c, __builtin_amdgcn_sqrtf(q), -c));
#else
  return __builtin_exp2f(__builtin_fmaf(c, __builtin_sqrtf(q), -c));
#endif
}

__host__ __device__ constexpr float es_c(int W) {
  return (float)(kEsBeta * W * 1.4426950408889634);
}

// Weight of tap t of a visibility whose first cell lies s cells from it, s in
// (-W/2, -W/2 + 1].  Widths up to 8 form z with one FMA, as many operations as
// sqrt(R^2 - x^2) takes; above, the rounding of t / R would show (up to 5 % of
// the error), and 1 - x^2 / R^2 is formed from the exact x for one more.
template <int W>
__host__ __device__ __forceinline__ float es_tap(float s, int t) {
  float q;
  if constexpr (W <= 8) {
    const float z = __builtin_fmaf(s, (float)(2.0 / W), (float)(t * 2.0 / W));
    q = __builtin_fmaf(-z, z, 1.0f);
  } else {
    const float x = s + (float)t;
    q = __builtin_fmaf(-(x * (float)(4.0 / (W * W))), x, 1.0f);
  }
  return es_from_q(q, es_c(W));
}

// The kernel that the device's FP32 weights are in the mean, in FP64: c as
// rounded, and the hardware square root, which is low by 7.3e-9 in the mean
// over the weights (a factor of -1.1e-7 on all of them per axis at W = 7, which
// taking the root's residual into account would cost the spread 4 %).  The
// correction tables of FP32 plans are this kernel's transform.
constexpr double kRootLow = 7.3e-9;
inline double es_device(double z, int W) {
  const double q = 1.0 - z * z;
  return std::exp2((double)es_c(W) * (std::sqrt(q > 0.0 ? q : 0.0) * (1.0 - kRootLow) - 1.0));
}

}  // namespace pc

#endif  // PC_ES_KERNEL_H
