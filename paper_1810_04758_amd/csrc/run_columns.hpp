// run_columns.hpp -- sizes of the run search's candidate columns (runs.hip) and
// the rule by which they are cut back.  No device code: a host program can
// include it and check the rule against every size.
#pragma once

namespace knn {

constexpr int kRunLeaf = 16;       // points per leaf (consecutive in curve order)
constexpr int kRunFan = 64;        // children per node above the leaves
constexpr int kRunMaxK = 64;       // largest K of the run search
constexpr int kRunMatrixDims = 3;  // dimensions from which the matrix cores filter the candidates

// K <= KP: the register list; C: column slots per lane; VB: keys sorted per
// network call; V: leaves the list of a run holds; wide: 32-bit entries.
struct RunColumn {
  int KP, C, VB, V;
  bool wide;
};
// Column slots: the target of the predicted radius and some four times its
// noise, and a leaf.  5-6 dimensions reach a few thousand leaves a run, more
// than a list in LDS could hold, and take 32-bit entries in shorter columns.
constexpr RunColumn run_column(int dims, int K) {
  if (dims >= 5)
    return K <= 8    ? RunColumn{8, 48, 8, 2 * kRunFan, true}
           : K <= 16 ? RunColumn{16, 64, 16, 2 * kRunFan, true}
           : K <= 32 ? RunColumn{32, 80, 16, 2 * kRunFan, true}
                     : RunColumn{64, 160, 16, 2 * kRunFan, true};
  const int V = dims == 2 ? 128 : dims == 3 ? 256 : 1024;
  return K <= 8    ? RunColumn{8, 64, 8, V, false}
         : K <= 16 ? RunColumn{16, 80, 16, V, false}
         : K <= 32 ? RunColumn{32, 112, 16, V, false}
                   : RunColumn{64, 160, 16, V, false};
}

// With the matrix filter a column is two halves, and a leaf puts up to half of
// its points in either.  Slots of a column (of a half) and what one leaf may
// add to it:
constexpr int run_slots(int dims, int C) { return dims >= kRunMatrixDims ? C / 2 : C; }
constexpr int run_leaf_adds(int dims) { return dims >= kRunMatrixDims ? kRunLeaf / 2 : kRunLeaf; }
// so it may hold this many entries before a leaf, and is cut back above them:
constexpr int run_room(int dims, int C) { return run_slots(dims, C) - run_leaf_adds(dims); }

// Whether cutting back changes a column of cnt entries (has_self: the query
// itself is, or will be, one of them): it then keeps K neighbours, evenly in
// both halves.  A column left as it is holds at most K entries, perhaps all in
// one half, and those leave room for a leaf (run_column_fits).
constexpr bool run_cut(int cnt, int has_self, int K) { return cnt - has_self >= K; }
constexpr bool run_column_fits(int dims, const RunColumn& c) {
  return run_room(dims, c.C) >= c.KP && c.C % c.VB == 0 && c.VB <= c.KP;
}

}  // namespace knn
