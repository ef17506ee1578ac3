"""The run search's candidate columns never overflow: a host program walks every
state a column of run_columns.hpp can reach (entries in its halves, the query's
own entry, each leaf adding what it may to either half, cut back by the rule of
the kernel) for every dimension and K, and looks at the last slot written."""

import os
import subprocess

import paper_1810_04758_amd

CSRC = os.path.join(os.path.dirname(paper_1810_04758_amd.__file__), "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "run_columns.hpp"
using namespace knn;

// limit: the largest entry count left alone before a leaf (the kernel's is the
// room; a smaller one must hold too).
int check(int dims, int K, int limit, bool self) {
  const RunColumn c = run_column(dims, K);
  const int slots = run_slots(dims, c.C), add = run_leaf_adds(dims);
  const bool halves = dims >= kRunMatrixDims;
  int last = -1;
  // state: entries of both halves, has_self of the kernel (set from the start:
  // the own entry comes with the first four leaves)
  struct S { int a, b, hs; };
  const int W = slots + 1;
  std::vector<char> seen((size_t)W * W * 2, 0);
  std::vector<S> todo;
  auto push = [&](S s) {
    if (s.a >= W || s.b >= W) return;  // already an overflow, in last
    char& f = seen[((size_t)s.a * W + s.b) * 2 + s.hs];
    if (!f) f = 1, todo.push_back(s);
  };
  push({0, 0, self ? 1 : 0});
  while (!todo.empty()) {
    S s = todo.back();
    todo.pop_back();
    if (std::max(s.a, s.b) > limit && run_cut(s.a + s.b, s.hs, K)) {
      s.a = halves ? (K + 1) / 2 : K;
      s.b = halves ? K / 2 : 0;
      s.hs = 0;
    }
    for (int x = 0; x <= add; ++x)
      for (int y = 0; y <= (halves ? add : 0); ++y) {
        // the kernel writes each candidate to the next free slot, hit or not
        last = std::max({last, s.a + std::min(x, add - 1), s.b + std::min(y, add - 1)});
        push({s.a + x, s.b + y, s.hs});
      }
  }
  if (last >= slots)
    std::printf("dims %d K %d limit %d self %d: slot %d of %d\n", dims, K, limit, (int)self, last, slots);
  return last >= slots;
}

int main() {
  int bad = 0;
  for (int dims = 2; dims <= 6; ++dims)
    for (int K = 1; K <= kRunMaxK; ++K) {
      const RunColumn c = run_column(dims, K);
      const int room = run_room(dims, c.C);
      if (!run_column_fits(dims, c) || K > c.KP) ++bad, std::printf("dims %d K %d: size\n", dims, K);
      for (int limit : {room, (room + (K + 1) / 2) / 2})
        for (bool self : {false, true}) bad += check(dims, K, limit, self);
    }
  return bad ? 1 : 0;
}
"""


def test_columns_never_overflow(tmp_path):
    src, exe = tmp_path / "columns.cpp", tmp_path / "columns"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
