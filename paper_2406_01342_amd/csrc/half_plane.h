// The half plane that coplanar plans grid, as pass B reads it (host and device:
// the index arithmetic is checked on the host, see tests/test_host_fft.py).
#ifndef PC_HALF_PLANE_H
#define PC_HALF_PLANE_H

#include "common.h"

namespace pc {

// Two adjacent columns of the pass-A buffer at one band row.
template <typename R>
struct alignas(4 * sizeof(R)) cpair {
  cpx<R> a, b;
};

// The half plane's Hermitian completion.  Coplanar plans hold the band rows
// v >= 0 (and the kernel's reach below), H_i(c) for cells c = v0 + rel; image
// row i is Re sum_c H_i(c) e^{2 pi i c f / M} = 1/2 sum_m z_i(m) e^{...} with
// z_i(m) = H_i(m) + conj H_i(-m) (cells mod M), whose transform is real.  Two
// image rows 2k and 2k + 1 are therefore the real and imaginary parts of ONE
// complex transform, of z_2k + i z_2k+1: half the transforms, and half the
// rows of pass A and of the pass-A buffer, of a full-plane grid.
//
// z of a pair at slot c in [0, M).  Away from the half plane's edges at most
// one of the four cells c, c + M, M - c, 2M - c lies in the band: pair_main
// names it (rel, and whether its conjugate enters), pair_rest adds the others
// (called for the few slots where pair_edge says so).  The band may start past
// M/2, where no visibility lies near v = 0: slots between its two images then
// have no cell at all.
//
// 8192^2 image: pass A 150 -> 83 us and pass B 356 -> 232 us against the full
// plane.
struct PairGeom {
  int M, v0, nv;
};
__host__ __device__ __forceinline__ int pair_main(const PairGeom& q, int c, bool& conj, bool& ok) {
  conj = 2 * c < q.M;
  const int rel = (conj ? q.M - c : c) - q.v0;
  ok = (unsigned)rel < (unsigned)q.nv;  // (rel < 0 where the band starts past M/2)
  return rel;
}
__host__ __device__ __forceinline__ bool pair_edge(const PairGeom& q, int c) {
  const int k = c - q.M / 2;
  return (k < 0 ? -k : k) <= q.M / 2 - q.v0 || c + q.M - q.v0 < q.nv || 2 * q.M - c - q.v0 < q.nv;
}
// H_a + i H_b, or conj H_a + i conj H_b
template <typename R>
__host__ __device__ __forceinline__ cpx<R> pair_z(const cpair<R>& h, bool conj) {
  return conj ? cpx<R>{h.a.x + h.b.y, h.b.x - h.a.y} : cpx<R>{h.a.x - h.b.y, h.a.y + h.b.x};
}
template <typename R, typename Load>
__host__ __device__ __forceinline__ cpx<R> pair_rest(const PairGeom& q, int c, Load load) {
  cpx<R> z{R(0), R(0)};
  auto add = [&](int rel, bool conj) {
    if ((unsigned)rel < (unsigned)q.nv) {
      const cpx<R> t = pair_z<R>(load(rel), conj);
      z = {z.x + t.x, z.y + t.y};
    }
  };
  if (2 * c < q.M)
    add(c - q.v0, false);
  else
    add(q.M - c - q.v0, true);
  add(c + q.M - q.v0, false);
  add(2 * q.M - c - q.v0, true);
  return z;
}

}  // namespace pc

#endif  // PC_HALF_PLANE_H
