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
