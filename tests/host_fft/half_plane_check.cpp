// Host check of the half plane's index arithmetic (half_plane.h) over the bands
// that plan construction makes (plan.cpp's own layout, no GPU): for every slot c
// of pass B's transform, the pass-A rows read must lie inside the band, and
// the completed column must hold every cell x that a footprint reaches exactly
// once at the slot x mod M and, conjugated, at -x mod M.  Columns are read in
// FP64 from a table of distinct values, so a missing, doubled or wrongly
// conjugated cell shows up as a wrong sum.  Prints "ok".
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "half_plane.h"
#include "plan.cpp"

namespace pc {
void fail(pc_status s, const std::string& msg) { throw Error(s, msg); }
void prof_release(pc_plan*) {}
}  // namespace pc

using namespace pc;

static bool check(const char* what, int n, double eps, int precision,
                  const std::vector<double>& turns_v) {
  const double fov = 0.02, dl = fov / n;
  std::mt19937_64 g(n);
  std::uniform_real_distribution<double> U(-0.5, 0.5);
  std::vector<double> u, v;
  for (double t : turns_v) {
    u.push_back(U(g) / dl);
    v.push_back(t / dl);
  }
  pc_geometry geo{};
  geo.nvis = (int64_t)v.size();
  geo.u = u.data();
  geo.v = v.data();
  geo.npix = n;
  geo.fov_rad = fov;
  geo.uv_units = PC_UV_WAVELENGTHS;
  geo.nufft_eps = eps;
  geo.upsamp = 2.0;
  geo.precision = precision;
  const Layout lay = build_layout(&geo, true);
  const GridGeom& gg = lay.g;
  const int M = gg.M;
  const PairGeom q{M, gg.v0, gg.nv};
  // two columns: values where a footprint reaches the row, zero elsewhere
  std::vector<cpair<double>> h((size_t)gg.nv, cpair<double>{});
  std::vector<bool> reached((size_t)gg.nv, false);
  for (uint32_t c : lay.cell)
    for (int t = 0; t < gg.W; ++t) reached[(size_t)(cell_v(c) + t - gg.v0)] = true;
  for (int r = 0; r < gg.nv; ++r)
    if (reached[r]) h[r] = {{U(g), U(g)}, {U(g), U(g)}};
  std::vector<cpx<double>> want((size_t)M, cpx<double>{0, 0});
  for (int r = 0; r < gg.nv; ++r) {
    const int x = gg.v0 + r;
    const cpx<double> a = pair_z<double>(h[r], false), b = pair_z<double>(h[r], true);
    cpx<double>& p = want[(size_t)(x & (M - 1))];
    p = {p.x + a.x, p.y + a.y};
    cpx<double>& m = want[(size_t)(-x & (M - 1))];
    m = {m.x + b.x, m.y + b.y};
  }
  int outside = 0, wrong = 0, dropped = 0, lowest = 0;
  auto load = [&](int rel) {
    if (rel < 0 || rel >= gg.nv) {
      ++outside;
      lowest = std::min(lowest, rel);
      return cpair<double>{};
    }
    return h[(size_t)rel];
  };
  for (int c = 0; c < M; ++c) {
    bool conj, ok;
    const int rel = pair_main(q, c, conj, ok);
    cpx<double> z{0, 0}, e{0, 0};
    if (ok) z = pair_z<double>(load(rel), conj);
    if (pair_edge(q, c)) e = pair_rest<double>(q, c, load);
    // (the pruned first stage leaves a slot without a main cell at zero)
    if (!ok && (e.x != 0 || e.y != 0)) ++dropped;
    const double dx = z.x + e.x - want[c].x, dy = z.y + e.y - want[c].y;
    if (!(std::hypot(dx, dy) <= 1e-14)) ++wrong;
  }
  const bool good = !outside && !wrong && !dropped;
  if (!good)
    std::printf("%s n=%d eps=%g: band [%d, %d), %d reads outside it (down to row %d), %d slots "
                "wrong, %d dropped  FAIL\n",
                what, n, eps, gg.v0, gg.v0 + gg.nv, outside, lowest, wrong, dropped);
  return good;
}

int main() {
  std::mt19937_64 g(7);
  std::uniform_real_distribution<double> U(0.0, 1.0);
  bool ok = true;
  for (int n : {16, 32, 64, 128, 256, 2048, 4096, 8192})
    for (double eps : {1e-1, 1e-5, 1e-9, 1e-15})
      for (int prec : {PC_PREC_FP32, PC_PREC_FP64}) {
        const double cell = 1.0 / (2.0 * n);
        auto range = [&](const char* what, double lo, double hi, int count) {
          std::vector<double> v;
          for (int k = 0; k < count; ++k) v.push_back((U(g) < 0.5 ? -1 : 1) * (lo + (hi - lo) * U(g)));
          ok &= check(what, n, eps, prec, v);
        };
        ok &= check("zero", n, eps, prec, {0.0});
        ok &= check("half a turn", n, eps, prec, {0.5, -0.5, 0.5 - 1e-13, -0.5 + 1e-13});
        ok &= check("one visibility", n, eps, prec, {0.3});
        ok &= check("two visibilities", n, eps, prec, {0.25, -0.26});
        range("whole turn", 0.0, 0.5, 300);
        range("zero and near it", 0.0, 3 * cell, 20);
        range("away from zero", 0.25, 0.3, 50);
        range("at the edge", 0.45, 0.5, 50);
        for (double lo : {1.0, 30.0, 41.0, 100.0, 200.0})  // fine cells
          range("from some cells on", std::min(0.49, lo * cell), std::min(0.5, 2 * lo * cell), 40);
      }
  std::printf(ok ? "ok\n" : "FAILED\n");
  return ok ? 0 : 1;
}
