"""The prompt attention's workgroup order (csrc/flash_map.h), compiled for the
host: every (group, workgroup) of a call is taken by exactly one block of the
grid, whichever set of an XCD it falls into."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_16292_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <vector>
#include "flash_map.h"
using namespace qsvd;
int main() {
  const int n_wgs[] = {1, 2, 3, 4, 5, 7, 8, 11, 18, 31, 63, 64, 65, 127, 128, 129, 130, 200};
  long long sets = 0, short_sets = 0, split = 0;
  for (int groups = 1; groups <= 1300; groups += groups < 70 ? 1 : 83)
    for (int n_wg : n_wgs) {
      const int parts = fa_parts(groups, n_wg);
      const long long blocks = fa_blocks(groups, n_wg, parts);
      std::vector<int> taken((size_t)groups * n_wg, 0);
      for (long long i = 0; i < blocks; ++i) {
        const FaWork w = fa_work((int)i, groups, n_wg, parts);
        if (w.group < 0 || w.wg < 0) return printf("negative: groups %d n_wg %d block %lld\n", groups, n_wg, i), 1;
        if (w.any) ++taken[(size_t)w.group * n_wg + w.wg];
      }
      for (int c : taken)
        if (c != 1) return printf("taken %d times: groups %d n_wg %d parts %d\n", c, groups, n_wg, parts), 1;
      const int wpp = (n_wg + parts - 1) / parts, per_set = kFaSet / wpp > 1 ? kFaSet / wpp : 1;
      const int ppx = (groups * parts + 7) / 8;
      sets += ppx > per_set;
      short_sets += ppx > per_set && per_set > 1 && ppx % per_set;
      split += parts > 1;
    }
  printf("sets %lld short %lld split %lld\n", sets, short_sets, split);
  return sets && short_sets && split ? 0 : 2;
}
"""


def test_every_workgroup_once(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "map.cpp", tmp_path / "map"
    src.write_text(MAIN)
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
