"""The item split and the grid of the grouped GEMMs, enumerated on the host: a
C++ program over csrc/grouped_plan.hpp, the arithmetic the kernels and their
launch use, checks that the workgroups of a launch cover every part of every run
of every item exactly once, for expert row counts at the edges of the split."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_02989_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "grouped_plan.hpp"
using namespace amoe;

// counts: rows of each expert; the block has as many routing entries as rows
static bool covered(const std::vector<int>& counts, int eb, int nblocks) {
  const int item_rows = grouped_item_rows(eb), big_rows = grouped_big_rows(eb);
  int slots = 0, n_items = 0, n_big = 0;
  for (int c : counts) {
    slots += c;
    const ItemSplit sp = split_rows(c, eb);
    int left = c, multiplied = 0;  // M-tiles: fp32 items of more than 48 rows multiply four
    if (sp.big < 0 || sp.big > sp.items) return false;
    for (int m = 0; m < sp.items; ++m) {
      const int rows = sp.rows < left ? sp.rows : left;
      if (rows < 1 || rows > item_rows || (m >= sp.big && rows > big_rows)) return false;
      left -= rows;
      multiplied += m < sp.big && rows > 48 ? grouped_item_rows(eb) / 16 : (rows + 15) / 16;
    }
    if (left != 0 || (eb == 4 && multiplied > (c + 15) / 16)) return false;
    n_items += sp.items;
    n_big += sp.big;
  }
  const int max_items = grouped_max_items(slots, static_cast<int>(counts.size()), item_rows);
  if (n_items > max_items) return false;
  std::vector<int> seen(static_cast<size_t>(n_items) * 4 * nblocks, 0);  // quarter runs
  const long long grid = grouped_workgroups(slots, max_items, nblocks, eb);
  for (long long b = 0; b < grid; ++b) {
    const GroupedShare s = grouped_share(static_cast<int>(b), n_items, n_big, grouped_split_items(nblocks), nblocks, eb);
    if (s.item >= n_items) continue;
    if (s.item < 0 || s.run < 0 || s.run >= s.parts * nblocks || (s.item < n_big && s.parts == 1)) return false;
    if (s.parts != 1 && s.parts != 2 && !(s.parts == 4 && eb == 4)) return false;
    for (int q = 0; q < 4 / s.parts; ++q)
      ++seen[static_cast<size_t>(s.item) * 4 * nblocks + s.run * (4 / s.parts) + q];
  }
  for (int n : seen)
    if (n != 1) return false;
  return true;
}

static int check(const std::vector<int>& counts, int eb, int nblocks, const char* what, int a, int m, int b, int s) {
  if (covered(counts, eb, nblocks)) return 0;
  std::printf("%s: element bytes %d, %zu experts, %d x %d rows and %d x %d rows, %d runs per item\n", what, eb,
              counts.size(), m, a, s, b, nblocks);
  return 1;
}

int main() {
  int bad = 0;
  const int runs[] = {1, 2, 6, 16, 32, 64, 128, 129, 300};
  // m experts with `a` rows and s with `b`
  for (int eb : {2, 4}) {
    const std::vector<int> big = eb == 2 ? std::vector<int>{129, 193, 257, 384, 385, 386, 577}
                                         : std::vector<int>{32, 33, 49, 64, 65, 97, 129, 193};
    for (int a : big)
      for (int b : {1, 16})
        for (int m : {0, 1, 3, 11, 20, 21, 43, 49, 64, 96, 128, 500})
          for (int s : {0, 1, 7, 8, 12, 15, 16, 32, 33, 85, 200})
            if (m + s > 0 && m + s <= 512)
              for (int nb : runs) {
                if ((m + s) * nb > 20000) continue;
                std::vector<int> counts(m, a);
                counts.insert(counts.end(), s, b);
                bad += check(counts, eb, nb, "pair", a, m, b, s);
              }
    // a longer sweep of the counts with the fewest rows per item
    for (int a : eb == 2 ? std::vector<int>{257, 385} : std::vector<int>{33, 65, 97})
      for (int m = 1; m <= 60; ++m)
        for (int s = 0; s <= 40; ++s)
          for (int nb : {8, 16}) {
            std::vector<int> counts(m, a);
            counts.insert(counts.end(), s, 1);
            bad += check(counts, eb, nb, "sweep", a, m, 1, s);
          }
    std::mt19937 rng(7);
    for (int i = 0; i < 2000; ++i) {
      std::vector<int> counts(1 + rng() % 200);
      const int top = 1 + static_cast<int>(rng() % 400);
      for (int& c : counts) c = static_cast<int>(rng() % (top + 1));
      bad += check(counts, eb, 1 + static_cast<int>(rng() % 20), "random", top, 0, 0, i);
    }
  }
  std::printf("%d uncovered\n", bad);
  return bad != 0;
}
"""


def test_every_run_is_covered_once(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o", str(exe)], check=True,
                   timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
