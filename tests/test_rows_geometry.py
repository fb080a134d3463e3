"""Geometry of the multi-factor passes in registers, on the CPU (no GPU needed)."""
import pytest

from native_probe import available, run_native

pytestmark = pytest.mark.skipif(not available, reason="libhfci.so or hipcc missing")

# Every geometry a residual pass can be launched with must leave its partials, one double per
# block and system, within the factor buffer that holds them: grids of one tile and of several
# that overlap in x and y, thin ones, one plane and many, unset and given z-chunks, every first
# width of a step, one system to 48.
ROOM = r"""
#include <cstdio>
#include "kernels.h"
using namespace hfci;
template <class T2> bool check(const GridDesc& g, int q) {
  if (!Launch<T2>::rows_run(g)) return true;
  const int w = rows_plan(q, sizeof(T2) == 8 ? kRowsMax32 : kRowsMax64, true)[0];
  for (int count : {1, 2, 3, 5, 12, 48}) {
    const RowsShape s = Launch<T2>::rows_shape(g, w, kFacResid, count);
    if (s.per_sys < 1 || s.per_sys != s.gx * s.gy * s.nzc || (size_t)s.per_sys > Launch<T2>::rows_partial_room(g)) {
      printf("%d x %d x %d, %d-byte values, q %d, %d systems: %d blocks\n", g.nx, g.ny, g.nz, (int)sizeof(T2), q, count,
             s.per_sys);
      return false;
    }
  }
  return true;
}
int main() {
  int bad = 0, all = 0;
  for (int nx : {1, 2, 5, 30, 64, 65, 66, 119, 128, 130, 192, 256, 1024})
    for (int ny : {1, 2, 5, 8, 49, 96, 300})
      for (int nz : {1, 2, 5, 8, 48, 96, 500})
        for (int cz : {0, 1, 2, 16, 64})
          for (int q : {3, 4, 5, 8, 10, 16}) {
            GridDesc g{};
            g.nx = nx;
            g.ny = ny;
            g.nz = nz;
            g.s_h2 = 1.0;
            g.tune32.fuse = g.tune64.fuse = 1;
            g.tune32.cz = g.tune64.cz = cz;
            ++all;
            if (!check<float2>(g, q) || !check<double2>(g, q)) ++bad;
          }
  printf("bad %d of %d\n", bad, all);
}
"""


def test_residual_partials_have_room(tmp_path):
    out = run_native(ROOM, tmp_path)
    assert "bad 0 of 19110" in out, out[-2000:]


# One step's multiplier at the eigenvalue the scalars are corrected at (the nearest to the pole),
# from the stored coefficients as the passes take them, against p~(B) / p~(z) in long double.
# The rounding of the c is taken back exactly there and the scalars carry each other's, so what is
# left is the rounding of the last pass's scalar: 2^-53 in complex128; in complex64, whose last
# pass of a step also adds that rounding (in single precision), 2^-24 of it twice.  Then the same
# for the polynomial of step one, whose last pass adds nothing in complex64.
MULTIPLIER = r"""
#include <cstdio>
#include "internal.h"
using namespace hfci;
using L = long double;
int main() {
  static_assert(sizeof(L) > sizeof(double), "the exact side needs more than double");
  for (double s_h2 : {0.4, 1.6, 5.0})
    for (double eps : {0.02, 0.1, 0.5})
      for (int q : {2, 3, 5, 7, 8, 10, 12, 16}) {
        const double b1 = -1.0, b2 = 12.0 * s_h2 - 0.05;
        std::vector<cd> z, sigma;
        contour_poles(6, 1.0, eps, 1.0, z, sigma);
        for (int j = 0; j < 6; ++j) {
          double delta, nu;
          cd z0, pz;
          optimise_delta(z[j], b1, b2, 1.0, q, delta, nu, z0, 200, 80);
          if (!(nu < 1.0)) continue;
          const cd lam(std::min(std::max(z[j].real(), b1), b2), z[j].imag() > 0.0 ? 0.0 : -1.0);
          std::vector<FactorCoef> k(q + std::max(q - 1, 1));
          complete_coefficients(factor_coefficients(z[j], z0, delta, q, pz), q, z0, s_h2, lam, k.data());
          const cld mid(0.0L, -(L)delta), B = mid * (cld(lam) - cld(z0)), beta = mid * (cld(z[j]) - cld(z0));
          const cld at = cld(lam) / (L)s_h2 - 6.0L;
          std::vector<L> fact(q + 1, 1.0L);
          for (int m = 1; m <= q; ++m) fact[m] = fact[m - 1] * m;
          cld pb(0.0L), p(0.0L), p2(0.0L);
          for (int m = q; m >= 0; --m) {
            pb = pb * B + 1.0L / fact[m];
            p = p * beta + 1.0L / fact[m];
          }
          for (int m = q - 1; m >= 0; --m) {
            cld e(0.0L);
            for (int i = q; i > m; --i) e = e * beta + 1.0L / fact[i];
            p2 = p2 * B + e;
          }
          const cld want[2] = {pb / p, p2 * cld(0.0L, (L)delta) / p};
          for (int prec : {32, 64})
            for (int part = 0; part < 2; ++part) {
              const bool step = part == 0;
              const int count = step ? q : q - 1;
              if (count < 2) continue;
              int f = step ? 0 : q;
              cld have(1.0L);
              L nearest = 1e9L;
              const std::vector<int> w = rows_plan(count, prec == 32 ? kRowsMax32 : kRowsMax64, step);
              for (size_t i = 0; i < w.size(); ++i) {
                const FactorCoef& h = k[f];
                auto r = [&](double v) { return prec == 32 ? (double)(float)v : v; };
                cld al = prec == 32 ? cld(h.al32_re, h.al32_im) : cld(h.al64_re, h.al64_im);
                if (!(step && i + 1 == w.size())) al = cld(r((double)al.real()), r((double)al.imag()));
                have *= al;
                for (int u = 0; u < w[i]; ++u, ++f) {
                  cld c(r(k[f].c_re), r(k[f].c_im));
                  if (step && f == 0) {
                    const double inv = 1.0 / s_h2, zr = std::fma(-z0.real(), inv, 6.0), zi = -z0.imag() * inv;
                    c = cld(r(zr), r(zi)) + cld(r(k[0].c_re - zr), r(k[0].c_im - zi));
                  }
                  have *= c + at;
                  nearest = std::min(nearest, std::abs(c + at));
                }
              }
              if (nearest < 1e-2L) continue;  // (next to a root the rounding is not taken back)
              printf("%d %d %.3Le s_h2 %g eps %g q %d pole %d\n", prec, part, std::abs(have / want[part] - 1.0L), s_h2, eps, q,
                     j);
            }
        }
      }
}
"""


def test_step_multipliers_carry_no_rounding_of_the_constants(tmp_path):
    bars = {("32", "0"): 2.0 ** -47, ("64", "0"): 1.01 * 2.0 ** -53, ("32", "1"): 1.01 * 2.0 ** -24,
            ("64", "1"): 1.01 * 2.0 ** -53}
    rows = [r.split(maxsplit=3) for r in run_native(MULTIPLIER, tmp_path).splitlines()]
    assert len(rows) > 1000 and {(r[0], r[1]) for r in rows} == set(bars)
    for prec, part, err, case in rows:
        assert float(err) <= bars[prec, part], (prec, part, err, case)


# Geometries of batches: every instance's tiles and chunks cover its grid, for the whole work and
# for what is left of it later, and the search for all of them stays cheap beside the launches of
# a step: 512 instances in 1.1 ms on this code's first machine, 20 ms when every part of the
# work rebuilt every geometry; the bar, best of five, lies between.
BATCH = r"""
#include <chrono>
#include <cstdio>
#include <random>
#include "kernels.h"
using namespace hfci;
template <class T2> double plan(int count, int lo, int hi, const std::vector<int>& widths) {
  std::mt19937 r(count + lo);
  std::uniform_int_distribution<int> side(lo, hi);
  std::vector<GridDesc> g(count);
  for (GridDesc& x : g) {
    x.nx = side(r), x.ny = side(r), x.nz = side(r);
    x.s_h2 = 1.3;
  }
  const std::vector<double> systems(count, 4.0), parts{1.0, 0.25, 0.0625, 0.015625};
  const auto t0 = std::chrono::steady_clock::now();
  std::vector<RowsClass> c;
  std::vector<std::vector<RowsShape>> sh;
  for (int kind : {(int)kFacResid, (int)kFacAdd, 0})
    for (int width : widths) {
      RowsClass x;
      x.width = width;
      x.kind = kind;
      const size_t k = c.size();
      c.resize(k + parts.size(), x);
      sh.resize(k + parts.size());
      if (!MultiLaunch<T2>::rows_class(g, systems, parts, &c[k], &sh[k])) return -1.0;
    }
  const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  for (size_t k = 0; k < c.size(); ++k)
    for (int i = 0; i < count; ++i) {
      const RowsShape& s = sh[k][i];
      if (s.w != c[k].w || s.small != c[k].small || s.per_sys != s.gx * s.gy * s.nzc || s.czlen * s.nzc < g[i].nz ||
          (s.gx - 1) * s.sx + 64 < g[i].nx || (s.nzc - 1) * s.czlen >= g[i].nz ||
          (size_t)s.per_sys > Launch<T2>::rows_partial_room(g[i]))
        return -2.0;
    }
  return ms;
}
int main() {
  for (int count : {1, 2, 7, 40})
    for (int lo : {1, 20, 60, 300, 900}) {
      const double a = plan<float2>(count, lo, lo + lo / 2, {2, 3, 4}), b = plan<double2>(count, lo, lo + lo / 2, {2, 3});
      if (a < 0.0 || b < 0.0) printf("bad %d %d %g %g\n", count, lo, a, b);
    }
  double best = 1e9;
  for (int k = 0; k < 5; ++k) best = std::min(best, plan<float2>(512, 12, 20, {3}));
  printf("ms %.3f\n", best);
}
"""


def test_batch_geometries_cover_the_grids_and_cost_little(tmp_path):
    out = run_native(BATCH, tmp_path)
    assert "bad" not in out, out
    assert 0.0 < float(out.split()[-1]) < 8.0, out


# Blocks per CU in the cost model are bounded by LDS too: three factors in complex128 take 43 KB
# for three waves, so three blocks fit where the registers would hold five.  With five the choice
# for a thin grid is chunks of 48 planes (1.31 ms for six steps of nine factors, 44 systems), with
# three it is 64 (1.21 ms).
OCCUPANCY = r"""
#include <cstdio>
#include "kernels.h"
using namespace hfci;
int main() {
  GridDesc g{};
  g.nx = 239, g.ny = 3, g.nz = 167;
  g.s_h2 = 1.0;
  for (int kind : {0, (int)kFacResid, (int)kFacAdd}) printf("%d ", Launch<double2>::rows_shape(g, 3, kind, 45).czlen);
}
"""


def test_cost_model_counts_the_blocks_that_fit_in_lds(tmp_path):
    assert run_native(OCCUPANCY, tmp_path).split() == ["64", "64", "64"]


# The tuner's launches take system s as pole s: its tables must have a pole, and the coefficients
# of the widest launch, for every system it times.
TUNE = r"""
#include <cmath>
#include <cstdio>
#include "internal.h"
using namespace hfci;
int main() {
  Op op;
  op.s_h2 = 1.3, op.b1 = -1.0, op.b2 = 15.0;
  for (int nsys : {1, 2, 8, 64}) {
    const TuneTables t = tune_tables(op, nsys);
    bool ok = t.poles.size() == (size_t)nsys && t.cstride >= kRowsMax32 && t.coef.size() == (size_t)nsys * t.cstride;
    for (const FactorCoef& c : t.coef) ok = ok && std::isfinite(c.c_re) && c.a_re != 0.0;
    printf("%s\n", ok ? "ok" : "bad");
  }
}
"""


def test_tuner_tables_cover_every_system(tmp_path):
    assert run_native(TUNE, tmp_path).split() == ["ok"] * 4
