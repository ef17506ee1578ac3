// runs.hpp -- the run search: the KNN join over runs of consecutive points
// of a space-filling curve (runs.hip).
#pragma once

#include "kernels.hpp"
#include "run_columns.hpp"

namespace knn {

constexpr int kRunLen = 64;       // queries per wavefront
constexpr int kRunLevels = 5;     // box levels of 2^31 points
constexpr int kRunCandSlots = 64; // candidate counters (statistics), 8 uint64 apart

// Curve order: cells of side `side` from `lo`, `bits` bits per dimension.
struct RunCurve {
  int32_t dims;
  int32_t bits;
  double lo[kMaxDims];
  double hi[kMaxDims];
  double inv_side;
  double side;
};

// The boxes of a sorted point set: level 0 = leaves, level l + 1 = groups of
// kRunFan boxes of level l, up to a level of at most kRunFan boxes.
struct RunTree {
  int32_t levels = 0;
  int64_t cnt[kRunLevels] = {0};
  int64_t off[kRunLevels] = {0};  // first box of the level
  int64_t total = 0;              // boxes of all levels
};
RunTree run_tree(int64_t N);
// Points of the sorted array, padded (with NaN coordinates) to whole runs.
inline int64_t run_padded(int64_t N) { return ceil_div(N, kRunLen) * kRunLen; }

struct RunArgs {
  const double* Xs;      // sorted points, point-major, run_padded(N) of them
  const int32_t* perm;   // sorted position -> id
  const void* keys;      // sorted curve keys (uint32 or uint64)
  int32_t key64;
  int64_t N;
  const double* boxes;   // 2 * dims doubles a box: lower corner, upper corner
  RunTree tree;
  // the queries in curve order: the points themselves (Qs == Xs, nothing
  // else set), or an external set with its keys
  const double* Qs;
  const int32_t* qperm;
  const void* qkeys;
  int64_t NQ;
  int32_t self;          // 1: the queries are the points, each excludes itself
  int32_t K;
  RunCurve curve;
  double target;         // points aimed at inside the predicted radius
  double ball;           // volume of the unit ball
  int32_t max_leaves;    // leaves a run may reach (set by the launcher)
  int32_t max_cuts;      // times it may cut its columns back (set by the launcher)
  int32_t* out_ids;
  double* out_d;
  int32_t* wide;         // runs left to k_run_single (one entry a run at most)
  int32_t* wide_count;   // zero before the search
  unsigned long long* cand;  // NULL, or kRunCandSlots counters 8 apart
};

// Curve keys of SoA points X (N, or N queries): keys, vals = 0..N-1.
void launch_run_keys(const double* X, int64_t N, const RunCurve& cv, bool key64, void* keys,
                     int32_t* vals, hipStream_t s);
// Sorted points from the row-major copy and their leaf boxes (boxes NULL: an
// external query set, no boxes).
void launch_run_gather(const double* XA, const int32_t* perm, int64_t N, int dims, double* Xs,
                       double* boxes, hipStream_t s);
// Boxes of the levels above the leaves.
void launch_run_boxes(double* boxes, const RunTree& t, int dims, hipStream_t s);
void launch_run_search(const RunArgs& a, int dims, hipStream_t s);

}  // namespace knn
