"""Partial slots of FP64 windows, on the CPU: whatever chunk count a side's
windows have, the tiles (a row above 16384 entries is several), chunks and
segment workgroups that store partial sums have a slot each, in the array as
it was laid out before the windows were planned. The library's preparation
and launch lists run here with windows of 1 to 90 chunks put in by hand."""

import os
import subprocess

import numpy as np
import pytest

from paper_2506_17650_amd import build, capi

CSRC = build.CSRC
DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "opdhg_host.h"
using namespace opdhg;
// longs rows of len entries, then shorts rows of k: long row i takes the
// columns from i on, short row r those from 7 r on
int main(int, char** v) {
  const int longs = atoi(v[1]), len = atoi(v[2]), shorts = atoi(v[3]), k = atoi(v[4]);
  const int n = atoi(v[5]), rows = atoi(v[6]), m = longs + shorts;
  std::vector<int64_t> rp{0};
  std::vector<int32_t> ci;
  for (int r = 0; r < m; ++r) {
    const int c = r < longs ? len : k;
    for (int q = 0; q < c; ++q) ci.push_back((r < longs ? r + q : 7 * r + q * (n / k)) % n);
    rp.push_back((int64_t)ci.size());
  }
  std::vector<double> val(ci.size(), 1.0), b(m, 0.0), c(n, 1.0), l(n, 0.0), u(n, 1.0);
  std::vector<int8_t> sense(m, 1);
  opdhg_lp lp{};
  lp.m = m, lp.n = n, lp.nnz = (int64_t)ci.size();
  lp.row_ptr = rp.data(), lp.col_idx = ci.data(), lp.val = val.data();
  lp.b = b.data(), lp.row_sense = sense.data(), lp.c = c.data(), lp.l = l.data(), lp.u = u.data();
  opdhg_params p;
  opdhg_default_params(&p);
  p.prep = OPDHG_PREP_DEVICE, p.windows = OPDHG_WINDOWS_ALWAYS, p.window_rows = rows;
  if (validate_lp(&lp) || validate_params(&p)) return 2;
  const int64_t cap = kTileCap, wgs = grid_cap(&p);
  int taken = 0;
  for (int segs = 0; segs < 2; ++segs)
    for (int nch = 1; nch <= 90; ++nch) {
      Prepared P;
      if (prepare(&lp, &p, P, false) || P.cend_a[1] != longs) return 3;
      const SlotLayout L = slot_layout(P, p.precision);
      const int64_t laid = P.part_stride_a(), before = (int64_t)P.stiles_a.size();
      Win64 w{};
      w.nch = nch, w.row0 = longs, w.groups = segs ? 3 : 0;
      const bool on = take_windows64(P, false, w, cap, 0, wgs, tables_bytes({&P}, wgs));
      std::vector<LpDev> d{slot_pointers(nullptr, L, P)};
      std::vector<WorkItem> list;
      int grid, chunk;
      side_items(d, {&P}, false, wgs, &grid, &chunk, list, true, true);
      const int64_t used = d[0].nslot_sa + P.w64_a.nch + (int64_t)P.win_a.seg_items();
      if (on != (P.w64_a.nch == nch) || (!on && (int64_t)P.stiles_a.size() != before) ||
          used > d[0].ntiles_a || d[0].ntiles_a > laid) {
        printf("segments %d chunks %d taken %d: %lld slots used of %d (%lld laid out)\n", segs, nch,
               on, (long long)used, d[0].ntiles_a, (long long)laid);
        return 1;
      }
      taken += on;
    }
  printf("%d", taken);
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    src = tmp_path_factory.mktemp("slots") / "slots.cpp"
    src.write_text(DRIVER)
    exe = src.parent / "slots"
    lib = os.path.dirname(capi.LIB_PATH)
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-arch=gfx950", "--offload-host-only"]
                   + build.COMMON + [str(src), "-x", "none", capi.LIB_PATH, "-Wl,-rpath," + lib,
                                     "-o", str(exe)], check=True)
    return str(exe)


# ten split rows; one split row beside short ones that would take all slots
# but those of its tile; medium rows and long ones that are not split; none
@pytest.mark.parametrize("longs,len_,shorts,k,n,rows",
                         [(10, 20000, 2000, 4, 20000, 64), (1, 20000, 3000, 18, 20000, 55),
                          (40, 300, 2000, 10, 5000, 64), (0, 1, 3000, 7, 5000, 192)])
def test_a_slot_for_every_partial_sum(driver, longs, len_, shorts, k, n, rows):
    out = subprocess.run([driver] + [str(v) for v in (longs, len_, shorts, k, n, rows)],
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) > 0  # and some windows are taken
