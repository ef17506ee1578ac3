// runs.hip -- the run search: every query's K nearest points without grid
// levels.  The points are sorted along a Hilbert curve; a wavefront takes a
// run of 64 consecutive queries, one per lane, walks a tree of bounding boxes
// (leaves of 16 consecutive points, 64 children per node above them) and
// evaluates each leaf that some lane's search ball reaches for all 64 lanes
// at once.
//
//   * A candidate is the same point for every lane, so its coordinates come
//     through the scalar cache into scalar registers (the grid search loads
//     them per lane through the vector memory unit, which bounds it).
//   * A lane's squared radius b starts from the density along the curve: the
//     curve is measure-preserving, so the keys of the points m before and
//     after the query bound the volume that holds those 2m points.
//   * Candidates with d^2 <= b go to the lane's own column of an LDS buffer:
//     no atomics, no histogram.  A column that could overflow is cut back to
//     its K nearest, which only tightens b.  A lane left with fewer than K
//     walks again with a larger b (b = infinity in the end).
//   * The K nearest of a column come from a sorting network in registers on
//     64-bit keys (the bits of d^2, the low 8 replaced by the column slot, so
//     a comparator is one v_min_f64 and one v_max_f64); keys that agree above
//     those bits are ordered exactly, by (d^2, id), in a second pass.
//
// What bounds it: the vector ALU.  A leaf is 16 x (3 dims + 4) instructions for
// 64 queries; 2e6 exponential 2-D points at K = 8 evaluate 19 leaves a run at
// about 620 cycles each, with the selection, the box tests and the walk's
// latency as much again.  Whole joins at default options against the grid
// levels (MI355X): uniform 2-D 5e4 K=5 0.62 -> 0.14 ms, exponential 2-D 2e6
// K=8 3.8 -> 0.67 ms, clustered 2-D 5e6 K=16 2.6 ms, 2e7 with the index build
// 75 -> 9.2 ms.  From 3 dimensions the candidates go through the matrix cores
// first (evaluate_matrix), which cut the search alone (FP64 distances for every
// candidate, filtered, now) of uniform 3-D 1e6 K=16 from 0.88 to 0.69 and 0.66 ms,
// the join of exponential 4-D 2e6 K=32 from 8.4 to 4.6 and 4.3 (11.7 on the grid);
// uniform 6-D 5e6 K=32 takes 36 ms, 117 on the grid: the vector ALU is 47 % busy
// with seven wavefronts per CU (20,992 bytes of LDS, 256 registers each), and 114
// GB come from HBM, 3.1 TB/s; loads two or four groups ahead gained nothing.  In 2
// dimensions the filter cost more than it saved (clustered 5e6 3.0 -> 3.7 ms).
//
// Exactness: every comparison that drops a point uses the squared distance
// in the order and rounding of the result.  A box is skipped only if its
// squared distance, computed with the same operations in the same order from
// differences that are no larger than any of its points' (rounding is
// monotone), exceeds b; a point is dropped only if d^2 > b, or from a column
// in which K points precede it by (d^2, id).  So a lane's column holds its K
// nearest once it holds K points.
#pragma clang fp contract(off)

#include <cmath>
#include <type_traits>
#include <utility>

#include "runs.hpp"

namespace knn {

namespace {

constexpr int kBlock = 256;
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));
constexpr int kRowLeaves = 6;  // 3 dimensions: leaves that cost as much as the rows' tests
constexpr int kRunGroup = 32;  // consecutive runs an XCD takes at a time

// Candidates through the scalar cache: a chunk of two 64-byte scalar loads,
// kChunkDoubles / point_stride points.
typedef int i16 __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(4))) i16* scalar_ptr;
constexpr int kChunkDoubles = 16;
struct Chunk {
  i16 a, b;
  __device__ __forceinline__ void load(scalar_ptr p) {
    a = p[0];
    b = p[1];
  }
  // waits for the chunk here: scalar loads return out of order, so a wait
  // after the next chunk's loads were issued would wait for those too
  __device__ __forceinline__ void arrived() {
    asm volatile("" : "+s"(a));
    asm volatile("" : "+s"(b));
  }
  template <int I>
  __device__ __forceinline__ double at() const {
    constexpr int W = 2 * (I & 7);
    const int lo = I < 8 ? a[W] : b[W], hi = I < 8 ? a[W + 1] : b[W + 1];
    return __hiloint2double(hi, lo);
  }
};

__device__ __forceinline__ double vmin(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double vmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// the smaller one, or the one that is a number
__device__ __forceinline__ float fmin_raw(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

__device__ __forceinline__ float fmin3_raw(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ double read_lane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Wavefront reductions on the vector ALU: rotations by 1, 2, 4, 8 inside the
// rows of 16 lanes, then the four rows (no LDS round trips).
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = (int)(uint32_t)b, hi = (int)(uint32_t)((uint64_t)b >> 32);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
}
constexpr int kRowRor = 0x120;  // DPP row_ror:n is kRowRor + n
// the maximum of the lane's row of 16
__device__ __forceinline__ double row_max(double v) {
  v = vmax(v, row_move<kRowRor + 1>(v));
  v = vmax(v, row_move<kRowRor + 2>(v));
  v = vmax(v, row_move<kRowRor + 4>(v));
  return vmax(v, row_move<kRowRor + 8>(v));
}
__device__ __forceinline__ double wave_max(double v) {
  v = row_max(v);
  const double a = vmax(read_lane(v, 0), read_lane(v, 16));
  return vmax(a, vmax(read_lane(v, 32), read_lane(v, 48)));
}
__device__ __forceinline__ double wave_min(double v) { return -wave_max(-v); }
__device__ __forceinline__ int wave_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(v, v, kRowRor + 1, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, kRowRor + 2, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, kRowRor + 4, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, kRowRor + 8, 0xF, 0xF, false));
  return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

template <int DIM>
__device__ __forceinline__ void load_pt(const double* __restrict__ Xs, int64_t p,
                                        double (&x)[DIM]) {
  constexpr int S = point_stride(DIM);
  const double2* src = reinterpret_cast<const double2*>(Xs + p * S);
#pragma unroll
  for (int h = 0; h < S / 2; ++h) {
    const double2 t = src[h];
    x[2 * h] = t.x;
    if (2 * h + 1 < DIM) x[2 * h + 1] = t.y;
  }
}

template <int DIM>
__device__ __forceinline__ double dist2(const double (&x)[DIM], const double (&q)[DIM]) {
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < DIM; ++j) {
    const double t = __dsub_rn(x[j], q[j]);
    s = __dadd_rn(s, __dmul_rn(t, t));
  }
  return s;
}

// ---------------------------------------------------------------------------
// curve order
// ---------------------------------------------------------------------------

// Hilbert index of cell coordinates c (bits bits each), by Skilling's
// transpose method (J. Skilling, "Programming the Hilbert curve", AIP Conf.
// Proc. 707, 2004): per bit plane from the top, a set bit inverts the lower
// bits of dimension 0 and a clear one exchanges them with dimension 0's; then
// the planes are Gray-decoded across the dimensions and interleaved.
template <int DIM>
__device__ __forceinline__ uint64_t hilbert_key(uint32_t (&c)[DIM], int bits) {
  for (int b = bits - 1; b > 0; --b) {
    const uint32_t low = (1u << b) - 1u;
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      const bool set = (c[j] >> b) & 1u;
      const uint32_t x = set ? low : ((c[0] ^ c[j]) & low);
      c[0] ^= x;
      if (j > 0) c[j] ^= set ? 0u : x;
    }
  }
#pragma unroll
  for (int j = 1; j < DIM; ++j) c[j] ^= c[j - 1];
  uint32_t t = 0;
  for (int b = bits - 1; b > 0; --b)
    if ((c[DIM - 1] >> b) & 1u) t ^= (1u << b) - 1u;
#pragma unroll
  for (int j = 0; j < DIM; ++j) c[j] ^= t;
  uint64_t key = 0;
  for (int b = bits - 1; b >= 0; --b) {
#pragma unroll
    for (int j = 0; j < DIM; ++j) key = (key << 1) | ((c[j] >> b) & 1u);
  }
  return key;
}

// Bound by the integer steps of the curve (about 8 bits x dims operations a
// point); reads 8 dims and writes 8-12 bytes a point.
template <int DIM, class KeyT>
__global__ void k_run_keys(const double* __restrict__ X, int64_t N, RunCurve cv,
                           KeyT* __restrict__ keys, int32_t* __restrict__ vals) {
  const double top = (double)((1ll << cv.bits) - 1);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N;
       i += (int64_t)gridDim.x * blockDim.x) {
    uint32_t c[DIM];
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      // external queries may lie outside the box: clamped to its cells
      const double u = (X[(int64_t)j * N + i] - cv.lo[j]) * cv.inv_side;
      c[j] = (uint32_t)fmin(fmax(u, 0.0), top);
    }
    keys[i] = (KeyT)hilbert_key<DIM>(c, cv.bits);
    vals[i] = (int32_t)i;
  }
}

// Sorted points (point-major, the tail of the last run NaN: a NaN distance
// passes no test) and, for indexed points, the boxes of their leaves: the 16
// lanes of a leaf reduce its corners by lane exchanges, so the points are not
// read back.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_run_gather(const double* __restrict__ XA, const int32_t* __restrict__ perm, int64_t N,
             int64_t Np, double* __restrict__ Xs, double* __restrict__ boxes) {
  constexpr int S = point_stride(DIM);
  // Np is a multiple of 64 and so is the stride: a wavefront is in range as a whole
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < Np;
       p += (int64_t)gridDim.x * blockDim.x) {
    const bool in = p < N;
    double x[S];
#pragma unroll
    for (int j = 0; j < S; ++j) x[j] = 0.0;
    if (in) {
      const double* src = XA + (int64_t)perm[p] * DIM;
#pragma unroll
      for (int j = 0; j < DIM; ++j) x[j] = src[j];
    }
    double2* out = reinterpret_cast<double2*>(Xs + p * S);
    const double none = __longlong_as_double(0x7FF8000000000000ll);
#pragma unroll
    for (int h = 0; h < S / 2; ++h)
      out[h] = in ? make_double2(x[2 * h], x[2 * h + 1]) : make_double2(none, none);
    if (boxes) {
      double lo[DIM], hi[DIM];
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        lo[j] = in ? x[j] : INFINITY;
        hi[j] = in ? x[j] : -INFINITY;
      }
#pragma unroll
      for (int o = 1; o < kRunLeaf; o <<= 1) {
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          lo[j] = fmin(lo[j], __shfl_xor(lo[j], o, 64));
          hi[j] = fmax(hi[j], __shfl_xor(hi[j], o, 64));
        }
      }
      if (in && (p & (kRunLeaf - 1)) == 0) {
        double* b = boxes + (p / kRunLeaf) * 2 * DIM;
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          b[j] = lo[j];
          b[DIM + j] = hi[j];
        }
      }
    }
  }
}

// One wavefront per box of a level: the union of its kRunFan boxes below.
template <int DIM>
__global__ void __launch_bounds__(64)
k_run_boxes(const double* __restrict__ in, int64_t nin, double* __restrict__ out) {
  const int64_t c = (int64_t)blockIdx.x * kRunFan + threadIdx.x;
  double lo[DIM], hi[DIM];
#pragma unroll
  for (int j = 0; j < DIM; ++j) {
    lo[j] = c < nin ? in[c * 2 * DIM + j] : INFINITY;
    hi[j] = c < nin ? in[c * 2 * DIM + DIM + j] : -INFINITY;
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      lo[j] = fmin(lo[j], __shfl_xor(lo[j], o, 64));
      hi[j] = fmax(hi[j], __shfl_xor(hi[j], o, 64));
    }
  }
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      out[(int64_t)blockIdx.x * 2 * DIM + j] = lo[j];
      out[(int64_t)blockIdx.x * 2 * DIM + DIM + j] = hi[j];
    }
  }
}

// ---------------------------------------------------------------------------
// sorting networks in registers
// ---------------------------------------------------------------------------
template <int M>
struct Net {
  int n = 0;
  int a[M] = {}, b[M] = {};
};
// Batcher's odd-even merge sort of V values.
template <int V>
constexpr Net<V * 10> sort_net() {
  Net<V * 10> r;
  for (int p = 1; p < V; p *= 2)
    for (int k = p; k >= 1; k /= 2)
      for (int j = k % p; j + k < V; j += 2 * k)
        for (int i = 0; i < k && i + j + k < V; ++i)
          if ((i + j) / (2 * p) == (i + j + k) / (2 * p)) {
            r.a[r.n] = i + j;
            r.b[r.n] = i + j + k;
            ++r.n;
          }
  return r;
}
// Sorts a bitonic sequence of V values.
template <int V>
constexpr Net<V * 10> merge_net() {
  Net<V * 10> r;
  for (int st = V / 2; st >= 1; st /= 2)
    for (int i = 0; i < V; ++i)
      if (!(i & st)) {
        r.a[r.n] = i;
        r.b[r.n] = i + st;
        ++r.n;
      }
  return r;
}
template <int A, int B, int V>
__device__ __forceinline__ void order2(double (&v)[V]) {
  const double lo = vmin(v[A], v[B]), hi = vmax(v[A], v[B]);
  v[A] = lo;
  v[B] = hi;
}
template <int V, size_t... I>
__device__ __forceinline__ void net_sort_(double (&v)[V], std::index_sequence<I...>) {
  constexpr auto net = sort_net<V>();
  (order2<net.a[I], net.b[I]>(v), ...);
}
template <int V>
__device__ __forceinline__ void net_sort(double (&v)[V]) {
  net_sort_(v, std::make_index_sequence<(size_t)sort_net<V>().n>{});
}
template <int V, size_t... I>
__device__ __forceinline__ void net_merge_(double (&v)[V], std::index_sequence<I...>) {
  constexpr auto net = merge_net<V>();
  (order2<net.a[I], net.b[I]>(v), ...);
}
template <int V>
__device__ __forceinline__ void net_merge(double (&v)[V]) {
  net_merge_(v, std::make_index_sequence<(size_t)merge_net<V>().n>{});
}

// Selection keys: the bits of d^2 with the low kSlotBits replaced by the
// buffer slot; an infinite d^2 counts as the largest finite one (a payload
// in an infinity would be a NaN), and a missing entry is +infinity.
constexpr int kSlotBits = 8;
constexpr uint32_t kSlotMask = (1u << kSlotBits) - 1u;
__device__ __forceinline__ double pack_key(double d2, int slot) {
  const uint64_t b = (uint64_t)__double_as_longlong(vmin(d2, 0x1.fffffffffffffp1023));
  return __longlong_as_double((long long)((b & ~(uint64_t)kSlotMask) | (uint32_t)slot));
}
__device__ __forceinline__ uint32_t key_slot(double k) {
  return (uint32_t)__double_as_longlong(k) & kSlotMask;
}
__device__ __forceinline__ bool same_key(double a, double b) {
  return (((uint64_t)__double_as_longlong(a) ^ (uint64_t)__double_as_longlong(b)) >> kSlotBits) == 0;
}
// Where keys are the same: (d^2, id) order inside the groups of same keys, with
// the rest of d^2 (an infinity comes after the largest finite one), the id and
// the slot below a group number, at most 2^56 and so an ordinary positive
// double again.
__device__ __forceinline__ double tie_key(int group, double d2, int32_t id, int slot) {
  const uint64_t b = (uint64_t)__double_as_longlong(d2);
  const uint64_t low = d2 == INFINITY ? kSlotMask + 1 : b & kSlotMask;
  return __longlong_as_double((long long)(((((uint64_t)group << (kSlotBits + 1) | low) << 31 |
                                            (uint32_t)id)
                                           << kSlotBits) |
                                          (uint32_t)slot));
}
// An upper bound of the d^2 behind a key.
__device__ __forceinline__ double key_bound(double k) {
  const uint64_t b = (uint64_t)__double_as_longlong(k) | kSlotMask;
  return b >= 0x7FEFFFFFFFFFFFFFull ? INFINITY : __longlong_as_double((long long)b);
}

template <size_t... I, class F>
__device__ __forceinline__ void each_index(std::index_sequence<I...>, F&& f) {
  (f(std::integral_constant<int, (int)I>{}), ...);
}

// ---------------------------------------------------------------------------
// the search
// ---------------------------------------------------------------------------
template <class KeyT>
__device__ __forceinline__ double key_span(const void* keys, int64_t i0, int64_t i1) {
  const KeyT* k = static_cast<const KeyT*>(keys);
  return (double)(uint64_t)(k[i1] - k[i0]) + 1.0;
}

// First position whose key is >= k.
template <class KeyT>
__device__ __forceinline__ int64_t key_place(const void* keys, int64_t N, uint64_t k) {
  const KeyT* ks = static_cast<const KeyT*>(keys);
  int64_t lo = 0, hi = N;
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    if ((uint64_t)ks[mid] < k)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// Predicted squared radius of the ball around q that holds a.target points:
// the densest of three windows along the curve (around, before and after the
// query: a window that crosses empty space underestimates the density), the
// part of the ball outside the data's box taken off (each dimension as a slab
// of the ball's marginal variance).
template <int DIM>
__device__ __forceinline__ double predict(const RunArgs& a, int64_t ip, const double (&q)[DIM]) {
  const int64_t m = DIM < 4 ? 48 : 96;
  const int64_t last = a.N - 1;
  ip = min(ip, last);
  double inv_density = INFINITY;  // cells per point
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    const int64_t i0 = max(ip - (w == 0 ? m : w == 1 ? 2 * m : 0), (int64_t)0);
    const int64_t i1 = min(ip + (w == 0 ? m : w == 1 ? 0 : 2 * m), last);
    if (i1 - i0 >= min(m, last)) {
      const double span = a.key64 ? key_span<uint64_t>(a.keys, i0, i1)
                                  : key_span<uint32_t>(a.keys, i0, i1);
      inv_density = fmin(inv_density, span / (double)max(i1 - i0, (int64_t)1));
    }
  }
  float v = (float)(a.target * inv_density / a.ball);  // cells^n
  const float e = 2.0f / DIM;
  float r2 = exp2f(log2f(v) * e);  // squared radius in cells
  // the ball's part inside the box, and how far q lies outside it
  const float rho = sqrtf(r2 * (3.0f / (DIM + 2)));
  float part = 1.0f;
  double out2 = 0.0;
#pragma unroll
  for (int j = 0; j < DIM; ++j) {
    const double dl = (q[j] - a.curve.lo[j]) * a.curve.inv_side;
    const double dh = (a.curve.hi[j] - q[j]) * a.curve.inv_side;
    const float cut = fminf(rho, fmaxf((float)dl, 0.0f)) + fminf(rho, fmaxf((float)dh, 0.0f));
    part *= fmaxf(cut / (2.0f * rho), 0.5f);
    const double o = fmax(fmax(-dl, -dh), 0.0);
    out2 += o * o;
  }
  r2 *= exp2f(-log2f(part) * e);
  double r = sqrt((double)r2);
  if (out2 > 0.0) r += sqrt(out2);
  const double b = (r * a.curve.side) * (r * a.curve.side);
  return b >= 0.0 ? b : INFINITY;  // NaN: search everything
}

// Statistics: leaves evaluated, summed over the queries.
__device__ __forceinline__ void count_candidates(const RunArgs& a, int64_t leaves) {
  if (a.cand && threadIdx.x == 0 && leaves > 0)
    atomicAdd(&a.cand[(blockIdx.x % kRunCandSlots) * 8], (unsigned long long)leaves * kRunLeaf);
}

// KP: the register list (a power of two >= K); C: column slots per lane; VB:
// keys sorted per network call; V: leaves the list of a run holds (run_column).
//
// WIDE = false: a column entry is 16 bits, (position in the leaf list) * 16 +
// the point's place in its leaf, so that a column of C entries takes half the
// LDS (which bounds the wavefronts in flight).  WIDE: entries are 32-bit
// positions, and the leaf list is emptied as it is evaluated.  A run that
// reaches more than a.max_leaves leaves is left to k_run_single.
template <int DIM, int KP, int C, int VB, int V, bool WIDE>
__device__ __forceinline__ void search_run(const RunArgs& a, const int64_t run) {
  static_assert(run_column_fits(DIM, RunColumn{KP, C, VB, V, WIDE}) && C <= (1 << kSlotBits),
                "a column that is not cut back leaves room for a leaf");
  static_assert(V >= 2 * kRunFan && (WIDE || V * kRunLeaf <= 65536), "");
  static_assert((KP + 1) * 4 <= C * (WIDE ? 4 : 2), "the rows reuse the columns' space");
  constexpr int S = point_stride(DIM);
  constexpr bool kMat = DIM >= kRunMatrixDims;
  constexpr int kRoom = run_room(DIM, C);  // entries above which columns (halves) are cut back
  using Entry = std::conditional_t<WIDE, uint32_t, uint16_t>;
  __shared__ Entry buf[C * 64];   // the lanes' columns (column_slot)
  __shared__ uint32_t list[V];    // leaves to evaluate (and those evaluated, unless WIDE)
  const int lane = threadIdx.x;
  const uint64_t lane_lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int K = a.K;
  const double* __restrict__ Xs = a.Xs;
  const int top = a.tree.levels - 1;
  const int64_t qp = run * kRunLen + lane;
  const bool valid = qp < a.NQ;
  double q[DIM];
  load_pt<DIM>(a.Qs, valid ? qp : run * kRunLen, q);
  double b = -1.0;
  {
    int64_t ip = qp;
    if (!a.self) {
      const int64_t qi = valid ? qp : run * kRunLen;
      ip = a.key64 ? key_place<uint64_t>(a.keys, a.N, static_cast<const uint64_t*>(a.qkeys)[qi])
                   : key_place<uint32_t>(a.keys, a.N, static_cast<const uint32_t*>(a.qkeys)[qi]);
    }
    if (valid) b = predict<DIM>(a, ip, q);
  }
  double b_try = b;
  // entries of the lane's column, and whether the query itself is one of them
  // (its own leaf is evaluated like any other; the selection leaves it out)
  int cnt = 0, has_self = 0;
  const uint32_t self_pos = a.self ? (uint32_t)qp : 0xFFFFFFFFu;
  int nlist = 0, ndone = 0;  // leaves listed, and evaluated
  double best[KP], nxt;      // the final selection
  double b_end = -1.0;       // the radius of the lane's last walk
  bool was_cut = false;      // the column was cut back to K entries in this walk
  bool tightened = false;    // some radius was cut since bmax was taken
  int cuts = 0;              // times the columns were cut back
  int64_t leaves = 0;

  // Where entry s of lane L's column lies.  With the matrix filter a query's
  // candidates arrive in two lanes (half of each leaf in either), so its
  // column is two, of which the first holds c0 entries.
  auto column_slot = [](int s, int L, int c0) -> int {
    if constexpr (!kMat) return s * 64 + L;
    const int sub = (L & 32) * 2 + (L & 31);
    return s < c0 ? s * 128 + sub : (s - c0) * 128 + sub + 32;
  };
  int cnt0 = 0;               // matrix filter: entries in the column's first half
  int cnt_a = 0, cnt_b = 0;   // and those of the half columns this lane fills:
                              // query lane % 32's and query 32 + lane % 32's
  auto collect = [&] {
    if constexpr (kMat) {
      const int a0 = __shfl(cnt_a, lane & 31, 64), b0 = __shfl(cnt_b, lane & 31, 64);
      const int a1 = __shfl(cnt_a, 32 + (lane & 31), 64), b1 = __shfl(cnt_b, 32 + (lane & 31), 64);
      cnt0 = lane < 32 ? a0 : b0;
      cnt = cnt0 + (lane < 32 ? a1 : b1);
    }
  };
  auto spread = [&] {
    if constexpr (kMat) {
      const int v = cnt - cnt0;
      const int a0 = __shfl(cnt0, lane & 31, 64), a1 = __shfl(v, lane & 31, 64);
      const int b0 = __shfl(cnt0, 32 + (lane & 31), 64), b1 = __shfl(v, 32 + (lane & 31), 64);
      cnt_a = lane < 32 ? a0 : a1;
      cnt_b = lane < 32 ? b0 : b1;
    }
  };

  auto entry_pos = [&](uint32_t e) -> uint32_t {
    return WIDE ? e : list[e / kRunLeaf] * kRunLeaf + e % kRunLeaf;
  };

  // Entries of a column whose loads are on their way together.  One at a time, each
  // behind a branch, a selection waited for every one of its loads in turn.  Two
  // (MI355X, one / two / four): integer 4-D 6e5 K=64 5.1 / 4.1 / 4.4 ms, uniform 3-D
  // 6e5 K=64 1.38 / 1.20 / 1.37, exponential 4-D 2e6 K=32 4.30 / 4.22 / 4.58, 6-D 6e5
  // K=16 5.5 / 5.3 / 5.4: more take registers from the rest.  Four where the columns
  // allow one wavefront a SIMD anyway (integer 5-D 6e5 K=64 11.8 / 10.3 / 9.7).  One,
  // with branches, where already one more costs spills (uniform 6-D 5e6 K=32 36.5 /
  // 38.3 / 37.6).
  constexpr bool kSerial = DIM == 6 && KP == 32;
  constexpr int kFlight = kSerial ? 1 : DIM >= 5 && KP > 32 ? 4 : 2;
  constexpr int kApart = kSerial ? 4 : 8;  // the compiler mixes no more entries than these
  static_assert(VB % kFlight == 0, "");
  // ---- the K nearest of every lane's column, as sorted keys -----------------
  // nxt: the smallest key not in the list.  Equal keys (exact ties and d^2
  // that differ in the last kSlotBits) take a second pass by tie_key: kSet
  // finds which entries of the key `at` are among the K, kOrder orders the
  // groups of a column that is in key order.  All lanes at once: a
  // 3-D lattice of 1e6 points, K=26, takes 1.3 ms, and took 3.6 with one column
  // ranked at a time by 64 lanes.
  enum { kKeys, kSet, kOrder };
  auto select = [&](int mode, double at, double (&best)[KP], double& nxt)
      __attribute__((always_inline)) {
    const int cmax = wave_max(cnt);
#pragma unroll
    for (int i = 0; i < KP; ++i) best[i] = INFINITY;
    nxt = INFINITY;
    int group = 0;
    double before = -1.0;
    for (int s0 = 0; s0 < cmax; s0 += VB) {
      double kk[VB];
#pragma unroll
      for (int i0 = 0; i0 < VB; i0 += kFlight) {
        uint32_t p[kFlight];
        if constexpr (kSerial) {
          p[0] = s0 + i0 < cnt ? entry_pos(buf[column_slot(s0 + i0, lane, cnt0)]) : 0u;
        } else {
          // no branch (past the column's end: some slot, and then point 0)
#pragma unroll
          for (int i = 0; i < kFlight; ++i) {
            const int s = s0 + i0 + i;
            const uint32_t e = buf[s < cnt ? column_slot(s, lane, cnt0) : lane];
            p[i] = s < cnt ? e : 0u;
          }
#pragma unroll
          for (int i = 0; i < kFlight; ++i) {
            const uint32_t v = entry_pos(p[i]);
            p[i] = s0 + i0 + i < cnt ? v : 0u;
          }
        }
        double x[kFlight][DIM], d2[kFlight];
#pragma unroll
        for (int i = 0; i < kFlight; ++i) load_pt<DIM>(Xs, p[i], x[i]);
#pragma unroll
        for (int i = 0; i < kFlight; ++i) {
          const int s = s0 + i0 + i;
          d2[i] = dist2<DIM>(x[i], q);
          const double k = pack_key(d2[i], s);
          kk[i0 + i] = s < cnt && p[i] != self_pos ? k : INFINITY;
        }
        if (mode != kKeys) {
          int32_t id[kFlight];
#pragma unroll
          for (int i = 0; i < kFlight; ++i) id[i] = a.perm[p[i]];
#pragma unroll
          for (int i = 0; i < kFlight; ++i) {
            const double k = kk[i0 + i];
            const bool edge = same_key(k, at);
            group = mode == kSet ? (int)edge : group + (same_key(k, before) ? 0 : 1);
            before = k;
            const bool in = k < INFINITY && (mode == kOrder || k <= at || edge);
            const double t = tie_key(group, d2[i], id[i], s0 + i0 + i);
            kk[i0 + i] = in ? t : INFINITY;
          }
        }
        if (i0 % kApart == kApart - kFlight) __builtin_amdgcn_sched_barrier(0);
      }
      net_sort<VB>(kk);
#pragma unroll
      for (int i = 0; i < VB; ++i) {
        const double lo = vmin(best[KP - VB + i], kk[VB - 1 - i]);
        nxt = vmin(nxt, vmax(best[KP - VB + i], kk[VB - 1 - i]));
        best[KP - VB + i] = lo;
      }
      net_merge<KP>(best);
    }
  };
  // the K-th of the list and the key after it
  auto kth_of = [&](const double (&best)[KP], double nxt, double& kth, double& after)
      __attribute__((always_inline)) {
    kth = after = INFINITY;
#pragma unroll
    for (int r = 0; r < KP; ++r)
      if (r == K - 1) {
        kth = best[r];
        after = r + 1 < KP ? best[r + 1 < KP ? r + 1 : r] : nxt;
      }
  };
  // the list's entries to the slots 0..K-1 of the columns of the lanes in `which`
  auto write_back = [&](const double (&best)[KP], bool which) __attribute__((always_inline)) {
    Entry pr[KP];
#pragma unroll
    for (int r = 0; r < KP; ++r) pr[r] = buf[column_slot(key_slot(best[r]), lane, cnt0)];
    wave_sync();
    if (which) {
#pragma unroll
      for (int r = 0; r < KP; ++r)
        if (r < K) buf[column_slot(r, lane, (K + 1) / 2)] = pr[r];
      cnt = K;
      cnt0 = (K + 1) / 2;
      has_self = 0;
    }
    wave_sync();
  };

  // ---- cut every column with K neighbours or more back to its K nearest -------
  // Afterwards every column (half column) has room for a leaf (run_cut).
  auto compact = [&]() __attribute__((always_inline)) {
    collect();
    const bool cut = run_cut(cnt, has_self, K);
    double best[KP], nxt, kth = INFINITY, after;
    for (int mode = kKeys;; mode = kSet) {
      select(mode, kth, best, nxt);
      if (mode == kSet) break;
      kth_of(best, nxt, kth, after);
      if (!__ballot(cut && same_key(kth, after))) break;
    }
    write_back(best, cut);
    if (cut) {
      b = fmin(b, key_bound(kth));
      was_cut = true;
    }
    spread();
    tightened = true;
    ++cuts;
    wave_sync();
  };

  // ---- the candidates of the listed leaves [ndone, nlist), 2 dimensions ---------
  // Bound by the vector ALU: 3 dims operations, a comparison and 3 for the
  // column per candidate, for 64 queries at once.  A chunk's scalar loads are
  // issued one chunk ahead, across leaves too.
  auto evaluate_scalar = [&]() __attribute__((always_inline)) {
    constexpr int PC = kChunkDoubles / S;  // points per chunk
    constexpr int NC = kRunLeaf / PC;      // chunks per leaf
    static_assert(NC % 2 == 0, "the two chunk buffers alternate");
    constexpr uint32_t kStep = 64 * sizeof(Entry);
    auto leaf_ptr = [&](uint32_t leaf) {
      leaf = (uint32_t)__builtin_amdgcn_readfirstlane((int)leaf);
      return (scalar_ptr)(uintptr_t)(Xs + (int64_t)leaf * (kRunLeaf * S));
    };
    const int v1 = __builtin_amdgcn_readfirstlane(nlist);
    for (int v0 = __builtin_amdgcn_readfirstlane(ndone); v0 < v1; v0 += 64) {
      const int ids = (int)list[min(v0 + lane, v1 - 1)];  // 64 leaves, one per lane
      const int m = min(v1 - v0, 64);
      uint32_t leaf = (uint32_t)__builtin_amdgcn_readlane(ids, 0);
      Chunk ch[2];
      ch[0].load(leaf_ptr(leaf));
      for (int u = 0;; ++u) {
        if (__ballot(cnt > kRoom)) compact();
        if (u == m) break;
        const uint32_t next = (uint32_t)__builtin_amdgcn_readlane(ids, min(u + 1, m - 1));
        const uint32_t e0 = (WIDE ? leaf : (uint32_t)(v0 + u)) * kRunLeaf;
        uint32_t at = (uint32_t)(cnt * 64 + lane) * (uint32_t)sizeof(Entry);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          Chunk& cur = ch[c & 1];
          cur.arrived();
          ch[(c + 1) & 1].load(c + 1 < NC ? leaf_ptr(leaf) + (c + 1) * 2 : leaf_ptr(next));
          __builtin_amdgcn_sched_barrier(0);
          each_index(std::make_index_sequence<PC>{}, [&](auto pi) __attribute__((always_inline)) {
            constexpr int P = decltype(pi)::value;
            const double x[DIM] = {cur.template at<P * S>(), cur.template at<P * S + 1>()};
            *reinterpret_cast<Entry*>(reinterpret_cast<char*>(buf) + at) =
                (Entry)(e0 + c * PC + P);
            at += dist2<DIM>(x, q) <= b ? kStep : 0u;
          });
        }
        cnt = (int)(at / kStep);
        leaf = next;
      }
    }
  };

  // ---- the same with a matrix-core filter (3 dimensions and more) --------------
  // A 32x32x16 product gives an approximate d^2 - |q|^2 of 32 candidates (two
  // leaves) for 32 queries, two of them for the run, so a pair costs a
  // comparison instead of 3 dims FP64 operations.  Coordinates are taken
  // relative to the middle of the searching lanes' box, scaled so that every
  // ball lies within kReach, and rounded to f16; lanes 0-31 hold the first H
  // dimensions of a candidate and lanes 32-63 the rest, each with its part of
  // |x|^2 as two f16 terms.  With x~ and q~ the rounded points, a candidate
  // within r of q is within r + |q - q~| + |x - x~| of q~: the threshold is the
  // square of that, plus the error of the f32 sums.  So the filter passes
  // every point within the radius and a few beyond it; the selection computes
  // every passed point's d^2 in FP64, and a row is final only if its K-th
  // lies within the radius.
  constexpr int H = (DIM + 1) / 2;
  constexpr float kReach = 63.0f;
  const int half = lane >> 5;
  double mid[H] = {};      // the middle, of the lane's half of the dimensions
  double scale = 0.0;
  float q_off = 0.0f, q_sq = 0.0f;  // |q' - q~|, |q~|^2
  float thr_a = 0.0f, thr_b = 0.0f;
  bool take_all = false;   // no usable scale: every point passes
  h8 op_a = {}, op_b = {};
  auto thresholds = [&]() __attribute__((always_inline)) {
    // |x - x~|: rounding toward zero below 64 errs by at most 2^-5 a
    // coordinate; the sums: 16 terms of magnitude below 2^17 in f32
    const float x_off = 0.03125f * 1.01f * __builtin_sqrtf((float)DIM) + 2e-3f;
    const float rr = (float)(sqrt(fmax(b, 0.0)) * scale) * 1.00001f;
    const float u = rr + q_off + x_off;
    const float t = b >= 0.0 ? (take_all ? 0.0f : u * u * 1.00001f - q_sq + 0.5f) : -INFINITY;
    thr_a = __shfl(t, lane & 31, 64);
    thr_b = __shfl(t, 32 + (lane & 31), 64);
  };
  auto prepare_filter = [&](const double (&wlo)[DIM], const double (&whi)[DIM], double bmax)
      __attribute__((always_inline)) {
    double reach = 0.0, ctr[DIM];
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      const double h = (whi[j] - wlo[j]) * 0.5;
      reach = fmax(reach, h);
      ctr[j] = wlo[j] + h;
    }
    reach += sqrt(bmax);
    take_all = !(reach > 1e-150 && reach < 1e150);
    scale = take_all ? 0.0 : (double)kReach / reach;
    float qt[2 * H] = {}, off = 0.0f;
    q_sq = 0.0f;
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
      const float f = b >= 0.0 ? (float)((q[j] - ctr[j]) * scale) : 0.0f;
      qt[j] = (float)(_Float16)f;
      off += (f - qt[j]) * (f - qt[j]);
      q_sq += qt[j] * qt[j];
    }
    q_off = __builtin_sqrtf(off) * 1.001f + 1e-4f;
#pragma unroll
    for (int k = 0; k < H; ++k) {
      mid[k] = half == 0 ? ctr[k] : (H + k < DIM ? ctr[H + k < DIM ? H + k : 0] : 0.0);
      const float a0 = __shfl(qt[k], lane & 31, 64), a1 = __shfl(qt[H + k], lane & 31, 64);
      const float b0 = __shfl(qt[k], 32 + (lane & 31), 64);
      const float b1 = __shfl(qt[H + k], 32 + (lane & 31), 64);
      op_a[k] = (_Float16)(-2.0f * (half == 0 ? a0 : a1));
      op_b[k] = (_Float16)(-2.0f * (half == 0 ? b0 : b1));
    }
    op_a[H] = op_a[H + 1] = op_b[H] = op_b[H + 1] = (_Float16)1.0f;
    thresholds();
  };
  auto evaluate_matrix = [&]() __attribute__((always_inline)) {
    constexpr uint32_t kStep = 128 * sizeof(Entry);
    const int v1 = __builtin_amdgcn_readfirstlane(nlist);
    for (int v0 = __builtin_amdgcn_readfirstlane(ndone); v0 < v1; v0 += 64) {
      const int ids = (int)list[min(v0 + lane, v1 - 1)];  // 64 leaves, one per lane
      const int m = min(v1 - v0, 64);
      const int groups = (m + 1) / 2;
      // candidate lane % 32 of leaves 2g and 2g + 1 (the last one again past the end)
      auto leaf_of = [&](int g) { return list[min(v0 + 2 * g + ((lane & 31) >> 4), v1 - 1)]; };
      auto load = [&](uint32_t leaf, double (&x)[H]) __attribute__((always_inline)) {
        const double* src = Xs + ((int64_t)leaf * kRunLeaf + (lane & 15)) * S + half * H;
#pragma unroll
        for (int k = 0; k < H; ++k) x[k] = H + k < S || half == 0 ? src[k] : 0.0;
      };
      double x[H], xn[H];
      load(leaf_of(0), x);
      uint32_t ahead = leaf_of(1);
      int first = 0;  // 1: the group's first leaf is done (the columns were cut back after it)
      for (int g = 0; g < groups;) {
        if (__ballot(max(cnt_a, cnt_b) > kRoom)) {
          compact();
          thresholds();
        }
        float f[H], sq = 0.0f;
#pragma unroll
        for (int k = 0; k < H; ++k) f[k] = (float)((x[k] - mid[k]) * scale);
        load(ahead, xn);
        const uint32_t ahead2 = leaf_of(g + 2);
        h8 cand = {};
#pragma unroll
        for (int k = 0; k < H; k += 2) {
          const h2 p = __builtin_bit_cast(
              h2, __builtin_amdgcn_cvt_pkrtz(f[k], k + 1 < H ? f[k + 1 < H ? k + 1 : k] : 0.0f));
          cand[k] = p[0];
          sq += (float)p[0] * (float)p[0];
          if (k + 1 < H) {
            cand[k + 1] = p[1];
            sq += (float)p[1] * (float)p[1];
          }
        }
        const h2 s0 = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(sq, 0.0f));
        const h2 s1 = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(sq - (float)s0[0], 0.0f));
        cand[H] = s0[0];
        cand[H + 1] = s1[0];
        const f16v none = {};
        const f16v acc_a = __builtin_amdgcn_mfma_f32_32x32x16_f16(cand, op_a, none, 0, 0, 0);
        const f16v acc_b = __builtin_amdgcn_mfma_f32_32x32x16_f16(cand, op_b, none, 0, 0, 0);
        bool full = false;
        // register r of lane l: candidate 8 (r / 4) + 4 (l / 32) + r % 4, query l % 32
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          if (hh < first || 2 * g + hh >= m) continue;
          if (hh == 1 && first == 0 && __ballot(max(cnt_a, cnt_b) > kRoom)) {
            full = true;
            continue;
          }
          const uint32_t leaf = (uint32_t)__builtin_amdgcn_readlane(ids, 2 * g + hh);
          const uint32_t e0 = (WIDE ? leaf : (uint32_t)(v0 + 2 * g + hh)) * kRunLeaf + 4 * half;
          uint32_t at_a = (uint32_t)(cnt_a * 128 + lane) * (uint32_t)sizeof(Entry);
          uint32_t at_b = (uint32_t)(cnt_b * 128 + 64 + lane) * (uint32_t)sizeof(Entry);
          // every candidate is written to the next free slot, which moves on if it passed
          auto put = [&](uint32_t& at, bool hit, uint32_t e) __attribute__((always_inline)) {
            *reinterpret_cast<Entry*>(reinterpret_cast<char*>(buf) + at) = (Entry)e;
            at += hit ? kStep : 0u;
          };
          if (take_all) {
            for (int rr = 0; rr < 8; ++rr) {
              const int i = 8 * (rr / 4) + rr % 4;
              const bool in = (int64_t)leaf * kRunLeaf + 4 * half + i < a.N;
              put(at_a, in && thr_a > -INFINITY, e0 + i);
              put(at_b, in && thr_b > -INFINITY, e0 + i);
            }
          } else {
            // four registers (8 candidates) at a time, most of them without a hit
#pragma unroll
            for (int r4 = 0; r4 < 8; r4 += 4) {
              const int o = 8 * hh + r4;
              const float least_a =
                  fmin3_raw(acc_a[o], acc_a[o + 1], fmin_raw(acc_a[o + 2], acc_a[o + 3]));
              const float least_b =
                  fmin3_raw(acc_b[o], acc_b[o + 1], fmin_raw(acc_b[o + 2], acc_b[o + 3]));
              if (__ballot(least_a <= thr_a || least_b <= thr_b)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  put(at_a, acc_a[o + r] <= thr_a, e0 + 2 * r4 + r);
                  put(at_b, acc_b[o + r] <= thr_b, e0 + 2 * r4 + r);
                }
              }
            }
          }
          cnt_a = (int)(at_a / kStep);
          cnt_b = (int)(at_b / kStep);
        }
        first = full ? 1 : 0;
        if (full) continue;  // the second leaf again, after the columns are cut back
        ++g;
        ahead = ahead2;
#pragma unroll
        for (int k = 0; k < H; ++k) x[k] = xn[k];
      }
    }
  };
  auto evaluate = [&]() __attribute__((always_inline)) {
    if constexpr (kMat)
      evaluate_matrix();
    else
      evaluate_scalar();
    collect();
    leaves += nlist - ndone;
    ndone = nlist;
  };

  int attempt = 0;
  auto widen = [&] {
    if (attempt >= 3) {
      b_try = INFINITY;
    } else {
      const float f = (float)(a.target + 1.0) / (float)(cnt + 1);
      b_try *= 1.2 * (double)exp2f(log2f(fmaxf(f, 1.6f)) * (2.0f / DIM));
    }
    b = b_try;
    cnt = cnt0 = 0;
    was_cut = false;
  };

  // ---- walks ------------------------------------------------------------------
  bool again;
  do {
    for (;; ++attempt) {
      // the box of the lanes that search, and their largest radius
      double wlo[DIM], whi[DIM], bmax = wave_max(b);
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        wlo[j] = wave_min(b >= 0.0 ? q[j] : INFINITY);
        whi[j] = wave_max(b >= 0.0 ? q[j] : -INFINITY);
      }
      // the same per row of 16 lanes (consecutive on the curve)
      double rlo[DIM], rhi[DIM];
      if constexpr (kMat) {
#pragma unroll
        for (int j = 0; j < (DIM <= 4 ? DIM : 0); ++j) {
          rlo[j] = -row_max(b >= 0.0 ? -q[j] : -INFINITY);
          rhi[j] = row_max(b >= 0.0 ? q[j] : -INFINITY);
        }
        prepare_filter(wlo, whi, bmax);
      }
      // Children of the node (level, base): a box per lane against the lanes'
      // common box, then the hits one by one against every lane's ball.
      auto expand = [&](int level, int64_t base) __attribute__((always_inline)) -> uint64_t {
        const int64_t c = base + lane;
        const bool in = c < a.tree.cnt[level];
        const double* bx = a.boxes + (a.tree.off[level] + (in ? c : base)) * (2 * DIM);
        double lo[DIM], hi[DIM];
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          lo[j] = bx[j];
          hi[j] = bx[DIM + j];
        }
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          const double g = vmax(vmax(lo[j] - whi[j], wlo[j] - hi[j]), 0.0);
          s += g * g;
        }
        uint64_t m = __ballot(in && s <= bmax), hits = 0;
        if (a.self && level == 0 && (base >> 6) == run >> 4)  // the run's own leaves are done
          m &= ~(0xFull << ((run & 15) * 4));
        if (kMat && level == 0 && (DIM > 3 || __popcll(m) > kRowLeaves)) {
          // leaves: a filtered leaf costs less than its exact test; in 3-4
          // dimensions a test against the box of each row of lanes, in more the
          // common box decides (3: unless there are few, for the four rows'
          // tests cost as much as six leaves')
          if (DIM > 4) return m;
          const double rb = row_max(b);
#pragma unroll
          for (int g = 0; g < 64; g += 16) {
            double t = 0.0;
#pragma unroll
            for (int j = 0; j < DIM; ++j) {
              const double d =
                  vmax(vmax(lo[j] - read_lane(rhi[j], g), read_lane(rlo[j], g) - hi[j]), 0.0);
              t += d * d;
            }
            hits |= __ballot(t <= read_lane(rb, g));
          }
          return hits & m;
        }
        while (m) {
          const int k = __builtin_ctzll(m);
          m &= m - 1;
          double t = 0.0;
#pragma unroll
          for (int j = 0; j < DIM; ++j) {
            const double g = vmax(vmax(read_lane(lo[j], k) - q[j], q[j] - read_lane(hi[j], k)), 0.0);
            t += g * g;
          }
          if (__ballot(t <= b)) hits |= 1ull << k;
        }
        return hits;
      };

      if (WIDE) nlist = ndone = 0;
      // A self-join starts with the run's own leaves, then the other leaves of
      // their parent: where the radius is far too large (sparse regions, a
      // window across empty space) these near points tighten it before the walk
      // of the whole tree.
      int batch = kRunFan;
      bool stop = false;
      // Depth first; lane l of st_* holds the pending children of level l.
      // Leaves go to the list, which is evaluated about 64 at a time.
      int st_lo = 0, st_hi = 0, st_base = 0;
      int level = top + 1;
      int64_t base = 0;
      uint64_t mask = 1;
      bool near = false;  // still below the own parent
      if (a.self) {
        const int64_t l0 = run * (kRunLen / kRunLeaf);
        const int have = (int)min((int64_t)(kRunLen / kRunLeaf), a.tree.cnt[0] - l0);
        if (nlist + have > a.max_leaves) {
          stop = true;
        } else {
          if (lane < have) list[nlist + lane] = (uint32_t)(l0 + lane);
          nlist += have;
        }
        if (b >= 0.0) has_self = 1;
        batch = 0;
        near = true;
        level = 1;
        base = run >> 10 << 6;
        mask = 1ull << ((run >> 4) & 63);
      }
      bool walking = !stop;
      for (;;) {
        while (walking && nlist - ndone < batch) {
          if (mask == 0) {
            if (near) {
              if (level == 1) {  // the own parent is done: from the root
                near = false;
                level = top + 1;
                base = 0;
                mask = 1;
                if (nlist > ndone) break;
                continue;
              }
            } else if (level > top) {
              walking = false;
              break;
            }
            ++level;
            mask = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(st_hi, level) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane(st_lo, level);
            base = (int64_t)(uint32_t)__builtin_amdgcn_readlane(st_base, level);
            continue;
          }
          if (level == 0) {
            const int n = (int)__popcll(mask);
            // too many leaves for one wavefront (a WIDE list is emptied as it is evaluated),
            // or too many cuts
            if ((WIDE ? leaves : 0) + nlist + n > a.max_leaves || cuts > a.max_cuts) {
              stop = true;
              walking = false;
              break;
            }
            if ((mask >> lane) & 1ull)
              list[nlist + (int)__popcll(mask & lane_lt)] = (uint32_t)(base + lane);
            nlist += n;
            mask = 0;
            continue;
          }
          const int k = __builtin_ctzll(mask);
          mask &= mask - 1;
          st_lo = lane == level ? (int)(uint32_t)mask : st_lo;
          st_hi = lane == level ? (int)(uint32_t)(mask >> 32) : st_hi;
          st_base = lane == level ? (int)(uint32_t)base : st_base;
          base = (base + k) * kRunFan;
          --level;
          mask = expand(level, base);
          if (a.self && !near) {  // the own parent is done
            if (level == 1 && base >> 6 == run >> 10) mask &= ~(1ull << ((run >> 4) & 63));
            if (level == 0 && top == 0) mask = 0;
          }
        }
        if (stop || nlist == ndone) break;
        wave_sync();
        evaluate();
        if (tightened) bmax = wave_max(b);
        tightened = false;
        if (WIDE) nlist = ndone = 0;
        batch = kRunFan;
      }
      if (stop) {
        if (lane == 0) a.wide[atomicAdd(a.wide_count, 1)] = (int32_t)run;
        count_candidates(a, leaves * min((int64_t)kRunLen, a.NQ - run * kRunLen));
        return;
      }
      // lanes short of K walk again with a larger radius
      if (b >= 0.0) b_end = b;
      // (two more where candidates are filtered: some may lie beyond the radius,
      // and a lane that the check after the selection finds short walks again
      // alone; exponential 4-D 1.5e5 K=64: none more 1.72 ms, one 1.57, two 1.51,
      // four 1.51, uniform 3-D 1e6 K=16 four 0.88, two 0.83)
      const bool more =
          b >= 0.0 && cnt - has_self < (kMat && !was_cut && b_try < INFINITY ? K + 2 : K);
      if (!__ballot(more)) break;
      if (more) {
        widen();
      } else {
        b = -1.0;
      }
      spread();
    }
    select(kKeys, 0.0, best, nxt);
    again = false;
    if constexpr (kMat) {
      // filtered candidates may lie beyond the radius: the row is final if its
      // K-th does not
      double kth = INFINITY;
#pragma unroll
      for (int r = 0; r < KP; ++r)
        if (r == K - 1) kth = best[r];
      const bool more = valid && !(key_bound(kth) <= b_end);
      again = __ballot(more) != 0;
      b = -1.0;
      if (more) widen();
      spread();
      ++attempt;
    }
  } while (again);

  // ---- order and write ---------------------------------------------------------
  // equal keys: which of them are among the K, then their order
  for (int mode = kKeys; mode != kOrder;) {
    if (mode == kKeys) {
      bool edge = false, inner = false;
#pragma unroll
      for (int r = 0; r < KP; ++r) {
        const bool same = same_key(best[r], r + 1 < KP ? best[r + 1 < KP ? r + 1 : r] : nxt);
        edge = edge || (r == K - 1 && same);
        inner = inner || (r < K - 1 && same);
      }
      if (!__ballot(valid && (edge || inner))) break;
      mode = __ballot(valid && edge) ? kSet : kOrder;
    } else {
      mode = kKeys;
    }
    double kth, after;
    kth_of(best, nxt, kth, after);
    if (mode != kSet) write_back(best, valid);
    select(mode, kth, best, nxt);
  }
  uint32_t* rows = reinterpret_cast<uint32_t*>(buf);  // positions of row g: rows[g * (K | 1) + r]
  {
    uint32_t pr[KP];
#pragma unroll
    for (int r = 0; r < KP; ++r) {
      const uint32_t e = buf[column_slot((int)key_slot(best[r]), lane, cnt0)];
      pr[r] = valid && r < K ? e : 0u;
    }
#pragma unroll
    for (int r = 0; r < KP; ++r) pr[r] = entry_pos(pr[r]);
    wave_sync();
    const int pitch = K | 1;
#pragma unroll
    for (int r = 0; r < KP; ++r)
      if (r < K) rows[lane * pitch + r] = pr[r];
    wave_sync();
  }
  // rows in order, K consecutive lanes a row: coalesced stores
  const uint32_t inv_k = ((1u << 19) + (uint32_t)K - 1u) / (uint32_t)K;  // e / K for e < 64 K
#pragma unroll 4
  for (int e = lane; e < 64 * K; e += 64) {
    const int g = (int)(((uint32_t)e * inv_k) >> 19);
    const int r = e - g * K;
    const int64_t qi = run * kRunLen + g;
    if (qi < a.NQ) {
      const uint32_t p = rows[g * (K | 1) + r];
      double x[DIM], y[DIM];
      load_pt<DIM>(Xs, p, x);
      load_pt<DIM>(a.Qs, qi, y);
      const int64_t row = a.qperm[qi];
      a.out_ids[row * K + r] = a.perm[p];
      a.out_d[row * K + r] = sqrt(dist2<DIM>(x, y));
    }
  }
  count_candidates(a, leaves * min((int64_t)kRunLen, a.NQ - run * kRunLen));
}

template <int DIM, int KP, int C, int VB, int V, bool WIDE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_run_search(const RunArgs a) {
  // Workgroups go round-robin over the XCDs: each XCD takes every eighth
  // group of kRunGroup consecutive runs, so that its L2 holds few regions of
  // the points at a time and dense and sparse regions are spread over all XCDs
  // at any time.  The end of the curve first: data with a dense corner at
  // its origin has its sparse, expensive runs there, which would otherwise
  // start last.
  const int64_t nruns = (a.NQ + kRunLen - 1) / kRunLen;
  const int64_t j = (gridDim.x - 1 - blockIdx.x) / kXcds;
  const int64_t run = (j / kRunGroup * kXcds + blockIdx.x % kXcds) * kRunGroup + j % kRunGroup;
  if (run < nruns) search_run<DIM, KP, C, VB, V, WIDE>(a, run);
}

// The queries of the runs that reached more leaves than a wavefront takes
// (sparse regions: 64 queries far apart, whose leaves are large), one query
// per wavefront: a lane tests one box, or evaluates one candidate of four
// leaves.  b and the candidate list belong to the wavefront.  Bound by the
// latency of one step after the other, so eight wavefronts share a SIMD, the
// query's own four leaves come first and the rest of their parent next (a
// tight radius for the walk), and the list is cut back by bisection, which
// takes some 300 instructions where ranking the entries takes thousands
// (clustered 2-D, 5e6 points, K=16, at 256 leaves a run: the join 3.4 -> 2.9
// ms, of which this kernel was 0.53).  Many points at exactly the K-th's
// distance: the id decides before they enter the list (2e4 duplicates among 1e5
// points, K=10: 31 -> 2.4 ms).
constexpr int kSingleSlots = 256;
template <int DIM>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8)))
k_run_single(const RunArgs a) {
  constexpr int E = kSingleSlots / 64;
  __shared__ double buf_d[kSingleSlots];
  __shared__ uint32_t buf_p[kSingleSlots];
  const int lane = threadIdx.x;
  const uint64_t lane_lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int K = a.K;
  const int top = a.tree.levels - 1;
  const int64_t n = (int64_t)*a.wide_count * kRunLen;
  for (int64_t w = blockIdx.x; w < n; w += gridDim.x) {
    const int64_t qp = (int64_t)a.wide[w / kRunLen] * kRunLen + w % kRunLen;
    if (qp >= a.NQ) continue;
    double q[DIM];
    load_pt<DIM>(a.Qs, qp, q);
    const uint32_t self_pos = a.self ? (uint32_t)qp : 0xFFFFFFFFu;
    int64_t ip = qp;
    if (!a.self)
      ip = a.key64 ? key_place<uint64_t>(a.keys, a.N, static_cast<const uint64_t*>(a.qkeys)[qp])
                   : key_place<uint32_t>(a.keys, a.N, static_cast<const uint32_t*>(a.qkeys)[qp]);
    ip = min(ip, a.N - 1);
    const int64_t parent = __builtin_amdgcn_readfirstlane((int)(ip / (kRunLeaf * kRunFan)));
    uint64_t own = 0xFull << (__builtin_amdgcn_readfirstlane((int)(ip / kRunLen) & 15) * 4);
    if (a.tree.cnt[0] - parent * kRunFan < kRunFan)
      own &= (1ull << (a.tree.cnt[0] - parent * kRunFan)) - 1;
    double b = read_lane(predict<DIM>(a, ip, q), 0);
    double b_try = b;
    int32_t b_id = 0x7FFFFFFF;  // at distance b exactly, only smaller ids count
    int cnt = 0;
    int32_t leaves = 0;

    // Ranks of the entries by (d^2, id); the first K go out in order, or stay
    // in the list.
    auto rank = [&](auto&& take) __attribute__((always_inline)) {
      wave_sync();
      double de[E];
      int32_t ie[E];
      uint32_t pe[E];
      int rk[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int s = e * 64 + lane;
        pe[e] = s < cnt ? buf_p[s] : 0u;
        de[e] = s < cnt ? buf_d[s] : INFINITY;
        ie[e] = s < cnt ? a.perm[pe[e]] : 0x7FFFFFFF;
        rk[e] = 0;
      }
#pragma unroll
      for (int f = 0; f < E; ++f) {
        const int cf = min(cnt - f * 64, 64);
        for (int u = 0; u < cf; ++u) {
          const double du = read_lane(de[f], u);
          const int32_t iu = __builtin_amdgcn_readlane(ie[f], u);
#pragma unroll
          for (int e = 0; e < E; ++e)
            if (e * 64 < cnt) rk[e] += (du < de[e] || (du == de[e] && iu < ie[e])) ? 1 : 0;
        }
      }
      wave_sync();
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * 64 + lane < cnt && rk[e] < K) take(rk[e], de[e], ie[e], pe[e]);
    };
    // Drops entries beyond the K-th (a few more than K stay): the smallest
    // upper half of a d^2, found by bisection, that at least K do not exceed.
    auto cut = [&]() __attribute__((always_inline)) {
      if (cnt <= K) return;
      wave_sync();
      int hw[E];
#pragma unroll
      for (int e = 0; e < E; ++e)
        hw[e] = e * 64 + lane < cnt ? __double2hiint(buf_d[e * 64 + lane]) : 0x7FFFFFFF;
      auto within = [&](int t) __attribute__((always_inline)) {
        int c = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) c += (int)__popcll(__ballot(hw[e] <= t));
        return c;
      };
      int lo = -1, hi = __builtin_amdgcn_readfirstlane(__double2hiint(b)), c = cnt;
      // most often the K-th lies within a factor of 16 of the radius
      int mid = max(hi - (4 << 20), 0);
      while (lo + 1 < hi && c > K + 16) {
        const int t = within(mid);
        if (t >= K) {
          hi = mid;
          c = t;
        } else {
          lo = mid;
        }
        mid = lo + (hi - lo) / 2;
      }
      double de[E];
      uint32_t pe[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        de[e] = buf_d[e * 64 + lane];
        pe[e] = buf_p[e * 64 + lane];
      }
      wave_sync();
      int at = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const uint64_t m = __ballot(hw[e] <= hi);
        if (hw[e] <= hi) {
          buf_d[at + (int)__popcll(m & lane_lt)] = de[e];
          buf_p[at + (int)__popcll(m & lane_lt)] = pe[e];
        }
        at += (int)__popcll(m);
      }
      cnt = at;
      if (hi < 0x7FF00000 && __hiloint2double(hi, -1) < b) {
        b = __hiloint2double(hi, -1);
        b_id = 0x7FFFFFFF;
      }
      if (cnt > kSingleSlots - 64) {  // equal distances: by (d^2, id)
        rank([&](int r, double d, int32_t, uint32_t p) __attribute__((always_inline)) {
          buf_d[r] = d;
          buf_p[r] = p;
        });
        cnt = K;
        wave_sync();
        b = buf_d[K - 1];
        b_id = __builtin_amdgcn_readfirstlane(a.perm[buf_p[K - 1]]);
      }
      wave_sync();
    };
    // the children of the node (level, base) within the radius
    auto reach = [&](int level, int64_t base) __attribute__((always_inline)) -> uint64_t {
      const int64_t c = base + lane;
      const bool in = c < a.tree.cnt[level];
      const double* bx = a.boxes + (a.tree.off[level] + (in ? c : base)) * (2 * DIM);
      double t = 0.0;
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        const double g = vmax(vmax(bx[j] - q[j], q[j] - bx[DIM + j]), 0.0);
        t += g * g;
      }
      return __ballot(in && t <= b);
    };
    for (int attempt = 0;; ++attempt) {
      int st_lo = 0, st_hi = 0, st_base = 0;
      int near = 2;  // 2: the own leaves, 1: their parent's others, 0: the tree
      int level = 0;
      int64_t base = parent * kRunFan;
      uint64_t mask = own;
      for (;;) {
        if (mask == 0) {
          if (near == 2) {
            cut();
            near = 1;
            mask = reach(0, base) & ~own;
            continue;
          }
          if (near == 1) {
            cut();
            near = 0;
            level = top + 1;
            base = 0;
            mask = 1;
            continue;
          }
          if (level > top) break;
          ++level;
          mask = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(st_hi, level) << 32) |
                 (uint32_t)__builtin_amdgcn_readlane(st_lo, level);
          base = (int64_t)(uint32_t)__builtin_amdgcn_readlane(st_base, level);
          continue;
        }
        if (level == 0) {  // four leaves
          if (cnt > kSingleSlots - 64) cut();
          int mine = -1;
          leaves += min((int)__popcll(mask), 4);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            if (mask) {
              const int k = __builtin_ctzll(mask);
              mask &= mask - 1;
              if (lane / kRunLeaf == g) mine = k;
            }
          }
          const uint32_t p = (uint32_t)((base + max(mine, 0)) * kRunLeaf + lane % kRunLeaf);
          double x[DIM];
          load_pt<DIM>(a.Xs, p, x);
          const double d2 = dist2<DIM>(x, q);
          bool hit = mine >= 0 && d2 <= b && p != self_pos;
          if (b_id != 0x7FFFFFFF && __ballot(hit && d2 == b))
            hit = hit && (d2 < b || a.perm[p] < b_id);
          const uint64_t hm = __ballot(hit);
          if (hit) {
            const int s = cnt + (int)__popcll(hm & lane_lt);
            buf_d[s] = d2;
            buf_p[s] = p;
          }
          cnt += (int)__popcll(hm);
          continue;
        }
        const int k = __builtin_ctzll(mask);
        mask &= mask - 1;
        st_lo = lane == level ? (int)(uint32_t)mask : st_lo;
        st_hi = lane == level ? (int)(uint32_t)(mask >> 32) : st_hi;
        st_base = lane == level ? (int)(uint32_t)base : st_base;
        base = (base + k) * kRunFan;
        --level;
        mask = reach(level, base);
        // the own parent is done
        if (level == 1 && base >> 6 == parent >> 6) mask &= ~(1ull << (parent & 63));
        if (level == 0 && top == 0) mask = 0;
      }
      if (cnt >= K) break;
      if (attempt >= 3) {
        b_try = INFINITY;
      } else {
        const float f = (float)(a.target + 1.0) / (float)(cnt + 1);
        b_try *= 1.2 * (double)exp2f(log2f(fmaxf(f, 1.6f)) * (2.0f / DIM));
      }
      b = b_try;
      b_id = 0x7FFFFFFF;
      cnt = 0;
    }
    cut();
    const int64_t row = a.qperm[qp];
    rank([&](int r, double d, int32_t id, uint32_t) __attribute__((always_inline)) {
      a.out_ids[row * K + r] = id;
      a.out_d[row * K + r] = sqrt(d);
    });
    count_candidates(a, leaves);
    wave_sync();
  }
}

int blocks_for(int64_t n, int cap = 8192) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, kBlock), cap));
}

template <int DIM, int KP, int C, int VB, int V, bool WIDE>
void search_k(RunArgs a, hipStream_t s) {
  const int64_t nruns = ceil_div(a.NQ, kRunLen);
  // Leaves a run may reach before it is left to k_run_single.  Where the runs
  // do not fill the GPU (4096 in flight) a long one is better spread over 64
  // wavefronts than finished alone: then fewer.  2 dimensions: a run of
  // twice its usual 20 to 40 leaves reaches across sparse ground (clustered,
  // 1e6 points, K=50: 2.65 ms at 256, 2.3 at 96, 2.4 at 64); 3: the same from
  // 256 on; 4: exponential 2e6 K=32 4.2 ms at 1024 and 768, 4.5 at 512; 5-6:
  // normal 6-D 1e5 K=16 2.06 ms at 4096, 2.4 at 6144, exponential 3e5 2.96 ms at
  // 4096, 3.4 at 8192; 6-D K > 16, where the search query by query falls further
  // behind, 3072 more: normal 2e5 K=32 8.4 ms at 4096, 6.5 at 6144 and 8192 (grid
  // levels 7.3), 3e5 K=64 28.9, 22.5, 19.8 (17.5), exponential 1.5e5 K=32 2.7, 3.0, 3.2.
  // Sets of few runs take none at all: one wavefront on every second SIMD leaves
  // the GPU idle, and one per query fills it (1e4 points, K=64, the join:
  // exponential 3-D 0.59 -> 0.19 ms, 4-D 0.75 -> 0.21, 6-D 0.57 -> 0.29; 1e5 points
  // would lose: 3-D K=16 0.35 -> 0.50).
  constexpr int64_t kFewRuns = DIM == 2 ? 192 : 512;
  // Queries that are few beside the points lie far apart along the curve, and a
  // run of them reaches many leaves in 5-6 dimensions: query by query up to 6.5e4
  // queries, 1.3e5 at K > 32 (5e4 among 5e5, run by run / query by query / on the
  // grid levels: uniform 6-D K=4 1.76 / 1.37 / 1.52 ms, normal 6-D K=64 8.2 / 4.8 /
  // 6.0; the other side of the line: uniform 5-D 6.7e4 among 4e5 K=4 0.84 / 1.00 /
  // 1.14, 1.6e5 among 5e6 K=16 3.3 / 4.1 / 3.0, K=64 8.3 / 5.5 / 4.5).
  const int64_t few = DIM >= 5 && !a.self && a.N >= 4 * a.NQ ? (KP <= 32 ? 1024 : 2048) : kFewRuns;
  // Nor may a run cut its columns back more often than this: a cut costs as much
  // as 10 to 50 leaves, a run of ordinary queries makes a few, and one with a few
  // far queries, to which everything is about equally near, makes one every leaf
  // or two.  Uniform points and three far ones, K=32: 4-D 2e5 4.3 ms without a
  // limit, 0.9 with 5, 1.25 with 16; 5-D 2e5 15.0, 2.4 with 5, 1.7 with 16; 6-D 6e5
  // K=16 18.1, 5.1, 4.1.  Other limits lose elsewhere: normal 4-D 6e5 K=64 5.6 at 5,
  // 6.2 at 3, axes of unequal scale 4-D 2e5 K=32 0.75 at 5, 0.98 at 8; normal 6-D 2e5
  // K=32 6.4 at 16, 11.6 at 8, tight 5-D clusters 5e4 K=32 0.70 at 16, 1.06 at 32.
  a.max_cuts = DIM <= 4 ? 5 : 16;
  if (nruns <= few) {
    a.max_leaves = 0;
  } else if constexpr (WIDE) {
    const int64_t more = DIM == 6 && KP > 16 ? 3072 : 0;
    a.max_leaves = (int32_t)std::min<int64_t>(std::max<int64_t>(nruns + more, 4096), 16384);
  } else {
    const int64_t most = DIM == 2 ? 96 : V, least = kRunFan << (DIM - 2);
    a.max_leaves = (int32_t)std::max(least, most * std::min<int64_t>(nruns, 4096) / 4096);
  }
  const unsigned blocks = (unsigned)(ceil_div(nruns, kXcds * kRunGroup) * kXcds * kRunGroup);
  k_run_search<DIM, KP, C, VB, V, WIDE><<<blocks, 64, 0, s>>>(a);
  KNN_LAUNCHED();
  k_run_single<DIM><<<(unsigned)std::min<int64_t>(nruns * kRunLen, 8192), 64, 0, s>>>(a);
  KNN_LAUNCHED();
}

template <int DIM, int K>
void search_col(const RunArgs& a, hipStream_t s) {
  constexpr RunColumn c = run_column(DIM, K);
  search_k<DIM, c.KP, c.C, c.VB, c.V, c.wide>(a, s);
}

template <int DIM>
void search_dim(const RunArgs& a, hipStream_t s) {
  if (a.K <= 8)
    search_col<DIM, 8>(a, s);
  else if (a.K <= 16)
    search_col<DIM, 16>(a, s);
  else if (a.K <= 32)
    search_col<DIM, 32>(a, s);
  else
    search_col<DIM, 64>(a, s);
}

template <int DIM>
void keys_dim(const double* X, int64_t N, const RunCurve& cv, bool key64, void* keys,
              int32_t* vals, hipStream_t s) {
  if (key64)
    k_run_keys<DIM, uint64_t><<<blocks_for(N), kBlock, 0, s>>>(X, N, cv,
                                                              static_cast<uint64_t*>(keys), vals);
  else
    k_run_keys<DIM, uint32_t><<<blocks_for(N), kBlock, 0, s>>>(X, N, cv,
                                                              static_cast<uint32_t*>(keys), vals);
  KNN_LAUNCHED();
}

#define KNN_RUN_DIMS(dims, call)                                      \
  switch (dims) {                                                     \
    case 2: call(2); break;                                           \
    case 3: call(3); break;                                           \
    case 4: call(4); break;                                           \
    case 5: call(5); break;                                           \
    case 6: call(6); break;                                           \
    default: throw Error(KNN_EINTERNAL, "run search: dims out of range"); \
  }

}  // namespace

RunTree run_tree(int64_t N) {
  RunTree t;
  int64_t c = ceil_div(N, kRunLeaf);
  for (;;) {
    KNN_CHECK(t.levels < kRunLevels, KNN_EINTERNAL, "run search: too many box levels");
    t.cnt[t.levels] = c;
    t.off[t.levels] = t.total;
    t.total += c;
    ++t.levels;
    if (c <= kRunFan) return t;
    c = ceil_div(c, kRunFan);
  }
}

void launch_run_keys(const double* X, int64_t N, const RunCurve& cv, bool key64, void* keys,
                     int32_t* vals, hipStream_t s) {
  KNN_CHECK(cv.bits >= 1 && cv.bits <= 31 && cv.dims * cv.bits <= (key64 ? 62 : 32), KNN_EINTERNAL,
            "run search: key bits out of range");
#define KNN_CALL(D) keys_dim<D>(X, N, cv, key64, keys, vals, s)
  KNN_RUN_DIMS(cv.dims, KNN_CALL)
#undef KNN_CALL
}

void launch_run_gather(const double* XA, const int32_t* perm, int64_t N, int dims, double* Xs,
                       double* boxes, hipStream_t s) {
  const int64_t Np = run_padded(N);
#define KNN_CALL(D) k_run_gather<D><<<blocks_for(Np), kBlock, 0, s>>>(XA, perm, N, Np, Xs, boxes)
  KNN_RUN_DIMS(dims, KNN_CALL)
#undef KNN_CALL
  KNN_LAUNCHED();
}

void launch_run_boxes(double* boxes, const RunTree& t, int dims, hipStream_t s) {
  for (int l = 0; l + 1 < t.levels; ++l) {
    const double* in = boxes + t.off[l] * 2 * dims;
    double* out = boxes + t.off[l + 1] * 2 * dims;
    const unsigned nb = (unsigned)t.cnt[l + 1];
#define KNN_CALL(D) k_run_boxes<D><<<nb, 64, 0, s>>>(in, t.cnt[l], out)
    KNN_RUN_DIMS(dims, KNN_CALL)
#undef KNN_CALL
    KNN_LAUNCHED();
  }
}

void launch_run_search(const RunArgs& a, int dims, hipStream_t s) {
  KNN_CHECK(a.K >= 1 && a.K <= kRunMaxK && a.NQ >= 1 && a.N >= 1, KNN_EINTERNAL,
            "run search: sizes out of range");
#define KNN_CALL(D) search_dim<D>(a, s)
  KNN_RUN_DIMS(dims, KNN_CALL)
#undef KNN_CALL
}

}  // namespace knn
