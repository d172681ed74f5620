"""The free range of a gram is cut into at most the stated number of parts, so that
the partial sums of every effective-operator update fit their scratch: ranges that
are no multiple of 64 (m = 126, where F = 15876 was cut into nine parts of 1984
instead of eight) and a host loop over all ranges up to 2^15."""
import pytest

from paper_2507_21236_amd import ATTN_DRYRUN, AttnHandle
from problems import make_problem
from tests.host_util import run_host


@pytest.mark.parametrize("L", [6, 8])
def test_partial_grams_of_bond_dimension_126_in_bounds(L):
    a = AttnHandle(make_problem("ragged", L, "ising", 126, 126, 4), flags=ATTN_DRYRUN)
    a.validate()
    a.close()


def test_ranges_are_cut_into_at_most_the_stated_parts(tmp_path):
    out = run_host(r"""
#include <cstdio>
#include "runtime.hpp"
int main() {
  for (int parts : {8, 32})
    for (int64_t F = 1; F <= 1 << 15; F++) {
      const int64_t c = rt::gram_chunk(F, parts), n = (F + c - 1) / c;
      if (c % 64 || n > parts || n != rt::gram_parts(F, parts) || (F % 64 == 0 && F % c)) {
        std::printf("F %lld parts %d: chunk %lld, %lld parts\n", (long long)F, parts, (long long)c, (long long)n);
        return 0;
      }
    }
  std::printf("ok\n");
}
""", tmp_path)
    assert out == "ok\n", out
