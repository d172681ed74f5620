"""Work items without a second operator come before those with one, whatever order
a plan lists them in: the kernels' main loop loads through the second operator
without testing it."""
from tests.host_util import run_host


def test_items_without_second_operator_come_first(tmp_path):
    out = run_host(r"""
#include <cstdio>
#include "runtime.hpp"
int main() {
  double o;
  // items of an earlier task stay as they are; the order inside both kinds is kept
  const int has_b[9] = {1, 0, 1, 0, 0, 1, 1, 0, 1};
  std::vector<attn::SWItem> v;
  for (int i = 0; i < 9; i++) v.push_back({nullptr, has_b[i] ? &o : nullptr, (double)i});
  rt::items_without_b_first(v, 2);
  for (auto& it : v) std::printf("%d%c ", (int)it.coef, it.B ? 'b' : '-');
  rt::items_without_b_first(v, 9);   // an empty list
}
""", tmp_path)
    assert out.split() == ["0b", "1-", "3-", "4-", "7-", "2b", "5b", "6b", "8b"], out
