"""The prompt call's schedule, walked on the CPU: with the lags and the numbers
of copies of csrc/schedule.h, no stage finds its layer's copy of a buffer
taken by another layer, and no two stages of one launch touch the same copy
of a buffer that one of them writes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_14782_amd", "csrc")

WALK = r"""
#include <cstdio>
#include <map>
#include <string>
#include <vector>
#include "schedule.h"
using namespace bacon;

struct Access { std::string buf; int copy, layer; bool write; };
static std::map<std::pair<std::string, int>, int> owner;   // layer whose values a copy holds
static int faults = 0;

// One launch: every access of its stages, side by side.
static void launch(int iter, const std::vector<Access> &acc) {
  for (const Access &x : acc)
    for (const Access &y : acc)
      if (x.buf == y.buf && x.copy == y.copy && x.layer != y.layer && x.write) {
        std::printf("launch %d: layer %d writes %s[%d] beside layer %d\n", iter, x.layer, x.buf.c_str(), x.copy, y.layer);
        ++faults;
      }
  for (const Access &x : acc)
    if (!x.write) {
      auto it = owner.find({x.buf, x.copy});
      if (it == owner.end() || it->second != x.layer) {
        std::printf("launch %d: layer %d finds %s[%d] of layer %d\n", iter, x.layer, x.buf.c_str(), x.copy,
                    it == owner.end() ? -1 : it->second);
        ++faults;
      }
    }
  for (const Access &x : acc)
    if (x.write) owner[{x.buf, x.copy}] = x.layer;
}

static void walk(bool wide, bool lse, bool adaptive, int m, int layers) {
  owner.clear();
  const Lags lag = stage_lags(wide, lse, adaptive);
  const int nb = copies_b(wide, adaptive), nh = copies_hist_b(wide, adaptive), ns = history_slots(m, adaptive);
  std::vector<Access> acc;
  auto use = [&](const char *buf, int n, int layer, bool write) { acc.push_back({buf, layer % n, layer, write}); };
  auto in = [&](int l) { return l >= 0 && l < layers; };
  auto pass1 = [&](int l) { use("partials", kCopies2, l, true); };
  auto pass2 = [&](int l) {
    if (!lse) use(wide ? "partials" : "lse", kCopies2, l, false);
    use("E", ns, l, true);
    use("B", nb, l, true);
    use("hist_B", nh, l, true);
  };
  for (int i = 0; i < layers + lag.fin; ++i) {
    if (in(i)) {
      // the budget tables, ahead of the iteration's launches (the head-wise
      // allocation's pick writes the heads' itself)
      acc.clear(); use("seq_tab", kCopiesTab, i, true); launch(i, acc);
      if (!adaptive) { acc.clear(); use("head_tab", kCopiesTab, i, true); launch(i, acc); }
      if (!wide) {
        // pass 1 and its merge alone for the first layer, later ones beside
        // the previous layer's pass 2 and select
        if (!lse && i == 0) {
          acc.clear(); pass1(i); launch(i, acc);
          acc.clear(); use("partials", kCopies2, i, false); use("lse", kCopies2, i, true); launch(i, acc);
        }
        acc.clear(); pass2(i);
        if (!lse && in(i + 1)) pass1(i + 1);
        launch(i, acc);
      }
    }
    acc.clear();
    if (wide && !lse && in(i - lag.p1)) pass1(i - lag.p1);
    if (wide && in(i - lag.p2)) pass2(i - lag.p2);
    if (!wide && !lse && in(i) && in(i + 1)) {
      use("partials", kCopies2, i + 1, false);
      use("lse", kCopies2, i + 1, true);
    }
    if (adaptive) {
      if (int l = i - lag.pool; in(l)) {
        use("seq_tab", kCopiesTab, l, false); use("B", nb, l, false);
        use("A", kCopiesA, l, true); use("hist_A", kCopiesHistA, l, true);
      }
      if (int l = i - lag.list; in(l)) {
        use("seq_tab", kCopiesTab, l, false); use("A", kCopiesA, l, false); use("hist_A", kCopiesHistA, l, false);
        use("list_A", kCopies2, l, true);
      }
      if (int l = i - lag.pick; in(l)) {
        use("seq_tab", kCopiesTab, l, false); use("A", kCopiesA, l, false); use("list_A", kCopies2, l, false);
        use("head_tab", kCopiesTab, l, true);
      }
    }
    auto budgets = [&](int l) { use("seq_tab", kCopiesTab, l, false); use("head_tab", kCopiesTab, l, false); };
    if (int l = i - lag.cal; in(l)) {
      budgets(l); use("B", nb, l, false); use("hist_B", nh, l, false);
      for (int j = 0; j <= m && j <= l; ++j) use("E", ns, l - j, false);
      if (adaptive) use("hist_A", kCopiesHistA, l, true);      // cleared
      use("V", kCopies2, l, true); use("list_B", kCopies2, l, true); use("hist_S", kCopiesS, l, true);
    }
    if (int l = i - lag.score; in(l)) {
      budgets(l); use("B", nb, l, false); use("hist_B", nh, l, false); use("V", kCopies2, l, false);
      use("list_B", kCopies2, l, false);
      use("hist_S", kCopiesS, l, true); use("S", kCopiesS, l, true);
    }
    if (int l = i - lag.cand; in(l)) {
      budgets(l); use("S", kCopiesS, l, false); use("hist_S", kCopiesS, l, false);
      use("list_S", kCopies2, l, true); use("hist_B", nh, l, true);   // cleared
    }
    if (int l = i - lag.fin; in(l)) {
      budgets(l); use("list_S", kCopies2, l, false); use("S", kCopiesS, l, false); use("hist_S", kCopiesS, l, false);
    }
    launch(i, acc);
  }
}

int main() {
  for (int m : {0, 1, 4, 16})
    for (int k = 0; k < 8; ++k) walk(k & 1, k & 2, k & 4, m, 40);
  return faults ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def walk_exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("schedule")
    src = d / "walk.cpp"
    src.write_text(WALK)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", CSRC, "-o", str(d / "walk"), str(src)], check=True)
    return str(d / "walk")


def test_no_copy_is_taken_before_its_last_reader(walk_exe):
    res = subprocess.run([walk_exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout[:2000]
