"""Work units of wide slices: a launch of few slices gives at most four row strips to
a workgroup, one that fills the chip the whole slice; the lists of such plans stay in
bounds."""
import pytest

from paper_2507_21236_amd import ATTN_DRYRUN, AttnHandle
from problems import make_problem
from tests.host_util import run_host


def test_rule(tmp_path):
    out = run_host(r"""
#include <cstdio>
#include "runtime.hpp"
int main() {
  int bad = 0;
  for (int strips = 1; strips <= 8; strips++)
    for (int64_t n : {1, 32, 56, 81, 128, 129, 512, 4096}) {
      const int w = rt::sw_wg_strips(strips, n);
      bad += w < 1 || w > strips || (strips <= 4 && w != strips);
      bad += strips > 4 && n <= 128 && w > 4;   // two workgroups a slice still fit the CUs
      bad += n > 256 && w != strips;
    }
  std::printf("%d\n", bad);
}
""", tmp_path)
    assert out == "0\n", out


@pytest.mark.parametrize("L,m", [(5, 80), (8, 96), (5, 128), (5, 113)])
def test_lists_of_wide_roots_in_bounds(L, m):
    a = AttnHandle(make_problem("wide", L, "ising", m, m, 4), flags=ATTN_DRYRUN)
    a.validate()
    a.close()


def test_work_units_of_a_matvec_by_slice_shape(tmp_path):
    # 1024 a spectator where four and more strips run on the matrix cores, 768 elsewhere
    out = run_host(r"""
#include <cstdio>
#include "runtime.hpp"
int main() {
  for (auto [ma, mb] : {std::pair{16, 16}, {48, 48}, {64, 64}, {50, 64}, {128, 128}, {129, 64}, {64, 129}, {256, 256}, {200, 1}})
    std::printf("%d ", (int)rt::mv_target(ma, mb));
}
""", tmp_path)
    assert out.split() == ["768", "768", "1024", "1024", "1024", "768", "768", "768", "768"], out
