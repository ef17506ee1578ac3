// eps.hip -- the two sampling kernels of the search-distance selection
// (Sec. 4.4): the mean distance between the points of a small sample
// (eps_mean), and the histogram of distances from sample points to every
// point of D, binned up to eps_mean.
#pragma clang fp contract(off)

#include <cmath>

#include "kernels.hpp"

namespace knn {

namespace {

constexpr int kBlock = 256;

// SX[j * ns + i] = X[j * N + sample[i]]: the sample's coordinates, compact
// (the pair loop then reads a few hundred KB instead of gathering from D).
__global__ void k_gather_sample(const double* __restrict__ X, int64_t N, int n,
                                const int64_t* __restrict__ sample, int64_t ns,
                                double* __restrict__ SX) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ns;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t id = sample[i];
    for (int j = 0; j < n; ++j) SX[(int64_t)j * ns + i] = X[(int64_t)j * N + id];
  }
}

// Block `a` sums the distances of sample point a to the sample points after
// it.  Bound by the FP64 square root (the sums' order fixes eps_mean).
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_pair_sums(const double* __restrict__ SX, int64_t ns, double* __restrict__ part) {
  __shared__ double red[kBlock];
  for (int64_t a = blockIdx.x; a < ns; a += gridDim.x) {
    double qa[DIM];
#pragma unroll
    for (int j = 0; j < DIM; ++j) qa[j] = SX[(int64_t)j * ns + a];
    double s = 0.0;
#pragma unroll 4
    for (int64_t b = a + 1 + threadIdx.x; b < ns; b += kBlock) {
      double d2 = 0.0;
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        const double t = __dsub_rn(SX[(int64_t)j * ns + b], qa[j]);
        d2 = __dadd_rn(d2, __dmul_rn(t, t));
      }
      s += sqrt(d2);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[a] = red[0];
    __syncthreads();
  }
}

constexpr int kSampleChunk = 256;
// points per thread in the distance histogram (1 on small sets)
constexpr int kPtsAll = 4;
constexpr int kMaxBins = 4096;

// Bin of a distance, floor(sqrt(d2) * inv_bw) with the correctly rounded
// square root.  A single-precision estimate (relative error below 2^-21:
// the conversion of d2, the hardware square root and two products) decides
// the bin unless it lies within 2^-18 (relative) of an integer; only then is
// the double-precision value taken.  That error bound holds only while every
// float involved is a normal number, so the estimate is used only for d2 in
// [2^-100, 2^100] and when inv_bw lies in [2^-60, 2^60] (use_f, checked once
// on the host): sqrt(d2) is then within [2^-50, 2^50] and the estimate within
// [2^-110, 2^110], far inside float's normal range.  Other values take the
// double-precision path.
__device__ __forceinline__ int dist_bin(double d2, double inv_bw, float inv_bw_f, bool use_f) {
  if (use_f && d2 >= 0x1p-100 && d2 <= 0x1p100) {
    const float t = __builtin_amdgcn_sqrtf((float)d2) * inv_bw_f;
    const float r = rintf(t);
    if (fabsf(t - r) > t * 0x1p-18f) return (int)floorf(t);
  }
  return (int)floor(sqrt(d2) * inv_bw);
}

struct Centre {
  double mid[kMaxDims];
};

// Each thread takes points p = i * pstride (every point when pstride = 1);
// the sample points of a chunk sit in LDS.  Only bins below count_bins are
// counted (pairs certainly beyond them skip the bin arithmetic).  The
// per-block histogram is accumulated in LDS (uint32) and added to the global
// uint64 counts at the end.
// skip_f: a single-precision squared distance above it proves the pair's
// double-precision d^2 above skip_d2 (see launch_dist_histogram), so most far
// pairs are rejected at single-precision rate; +inf disables the test.
// err: the absolute error, in bins, of the single-precision distance of the
// coordinates relative to mid (see launch_dist_histogram): away from a bin's
// edge by more than that it decides the bin.  Bound by the vector ALU: 1e6 3-D
// points x 500, all bins: 763 us with every bin from the double-precision
// d^2, 372 us with that only for the few near an edge (a wavefront in ten).
// kFloatBin = false: no such bound (err unused), every bin from the
// double-precision d^2, without the single-precision bin's instructions.
template <int DIM, int kPts, bool kFloatBin>
__global__ void k_dist_histogram(const double* __restrict__ X, int64_t N, int64_t pstride,
                                 const int64_t* __restrict__ sample, int64_t ns, double inv_bw,
                                 int count_bins, double skip_d2, float skip_f, Centre at,
                                 float err, uint64_t* __restrict__ counts,
                                 const uint32_t* __restrict__ named, uint32_t most) {
  if (named && *named <= most) return;  // counted by cell
  const int n_bins = count_bins;
  __shared__ uint32_t h[kMaxBins];
  const float inv_bw_f = (float)inv_bw;
  const bool use_f = inv_bw >= 0x1p-60 && inv_bw <= 0x1p60;
  __shared__ double sx[DIM][kSampleChunk];
  __shared__ float sxf[DIM][kSampleChunk];
  __shared__ int64_t sid[kSampleChunk];
  for (int b = threadIdx.x; b < n_bins; b += blockDim.x) h[b] = 0;
  // blockIdx.y: the sample's share of this block (few points: more blocks)
  const int64_t per = (ns + gridDim.y - 1) / gridDim.y;
  const int64_t s_end = (blockIdx.y + 1) * per < ns ? (blockIdx.y + 1) * per : ns;
  for (int64_t c0 = blockIdx.y * per; c0 < s_end; c0 += kSampleChunk) {
    const int cn = (int)((s_end - c0) < kSampleChunk ? (s_end - c0) : kSampleChunk);
    __syncthreads();
    for (int i = threadIdx.x; i < cn; i += blockDim.x) {
      int64_t id = sample[c0 + i];
      sid[i] = id;
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        sx[j][i] = X[(int64_t)j * N + id];
        sxf[j][i] = (float)(sx[j][i] - at.mid[j]);
      }
    }
    __syncthreads();
    // each thread takes kPts points (the LDS read of a sample point serves
    // all of them): point index t0 + u * blockDim (u < kPts), point p =
    // index * pstride
    const int64_t nP = (N + pstride - 1) / pstride;
    for (int64_t t0 = blockIdx.x * (int64_t)blockDim.x * kPts + threadIdx.x; t0 < nP;
         t0 += (int64_t)gridDim.x * blockDim.x * kPts) {
      double x[kPts][DIM];
      float xf[kPts][DIM];
      int64_t pp[kPts];
#pragma unroll
      for (int u = 0; u < kPts; ++u) {
        const int64_t t = t0 + (int64_t)u * blockDim.x;
        pp[u] = t < nP ? t * pstride : -1;
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          x[u][j] = pp[u] >= 0 ? X[(int64_t)j * N + pp[u]] : 0.0;
          // no point: NaN, which fails both tests below
          xf[u][j] = pp[u] >= 0 ? (float)(x[u][j] - at.mid[j]) : NAN;
        }
      }
      for (int i = 0; i < cn; ++i) {
        float sq[DIM];
#pragma unroll
        for (int j = 0; j < DIM; ++j) sq[j] = sxf[j][i];
#pragma unroll
        for (int u = 0; u < kPts; ++u) {
          // each square added with one rounding (a fused multiply-add)
          float sf = 0.0f;
#pragma unroll
          for (int j = 0; j < DIM; ++j) {
            const float t = __fsub_rn(xf[u][j], sq[j]);
            sf = __builtin_fmaf(t, t, sf);
          }
          if (sf > skip_f) continue;  // provably beyond skip_d2
          int b = 0;
          bool edge = true;
          if constexpr (kFloatBin) {
            const float bf = __builtin_amdgcn_sqrtf(sf) * inv_bw_f;
            b = (int)floorf(bf);
            edge = !(fabsf(bf - rintf(bf)) > __builtin_fmaf(bf, 0x1p-20f, err));
          }
          if (edge) {
            if (pp[u] < 0) continue;
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < DIM; ++j) {
              const double t = __dsub_rn(x[u][j], sx[j][i]);
              s = __dadd_rn(s, __dmul_rn(t, t));
            }
            if (s > skip_d2 || pp[u] == sid[i]) continue;  // beyond the last bin, or self
            b = dist_bin(s, inv_bw, inv_bw_f, use_f);
          }
          if (b < n_bins) atomicAdd(&h[b], 1u);
        }
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < n_bins; b += blockDim.x)
    if (h[b]) atomicAdd((unsigned long long*)&counts[b], (unsigned long long)h[b]);
}

// The histogram of near distances on a large set: a coarse grid over the
// points' box, one 512-bit mask a cell (the sample points within the counted
// distance of it), so that a point looks at the sample points its cell names
// instead of all of them.  With the counted distance a small part of the box
// that is almost none: the pass is then bound by reading the points
// (clustered 2-D, 2e7 points x 500: 1910 us by the pairs; see the launcher).
constexpr int kCellSamples = 512;
constexpr int kCellWords = kCellSamples / 64;
constexpr int64_t kMaxCells = 65536;
struct SampleCells {
  int32_t g;  // cells per dimension
  double lo[kMaxDims], inv_w[kMaxDims], w[kMaxDims];
  double slack;  // added to a cell's faces: the rounding of a point's cell
};

// One thread per (cell, mask word): the box distance to 64 sample points.
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_sample_cells(const double* __restrict__ X, int64_t N, const int64_t* __restrict__ sample,
               int ns, SampleCells sc, int64_t cells, double lim_d2,
               unsigned long long* __restrict__ mask, uint8_t* __restrict__ used) {
  __shared__ double sx[DIM][kCellSamples];
  for (int i = threadIdx.x; i < ns; i += kBlock)
#pragma unroll
    for (int j = 0; j < DIM; ++j) sx[j][i] = X[(int64_t)j * N + sample[i]];
  __syncthreads();
  for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < cells * kCellWords;
       e += (int64_t)gridDim.x * kBlock) {
    int64_t c = e / kCellWords;
    const int word = (int)(e % kCellWords);
    double lo[DIM], hi[DIM];
#pragma unroll
    for (int j = DIM - 1; j >= 0; --j) {
      const int cj = (int)(c % sc.g);
      c /= sc.g;
      lo[j] = sc.lo[j] + cj * sc.w[j] - sc.slack;
      hi[j] = sc.lo[j] + (cj + 1) * sc.w[j] + sc.slack;
    }
    unsigned long long m = 0;
    for (int i = 0; i < 64 && word * 64 + i < ns; ++i) {
      double d2 = 0.0;
#pragma unroll
      for (int j = 0; j < DIM; ++j) {
        const double x = sx[j][word * 64 + i];
        const double g = fmax(fmax(lo[j] - x, x - hi[j]), 0.0);
        d2 += g * g;
      }
      if (d2 <= lim_d2) m |= 1ull << i;
    }
    mask[e] = m;
    // the cell's words that hold a bit, gathered from its kCellWords lanes
    // (every lane of a group of eight is here: cells * kCellWords is a
    // multiple of eight and so is the stride)
    const unsigned long long any = __ballot(m != 0);
    if (word == 0) used[e / kCellWords] = (uint8_t)(any >> (threadIdx.x & 63));
  }
}

// The cell of point p, whose coordinates go to x.
template <int DIM>
__device__ __forceinline__ int64_t sample_cell(const double* __restrict__ X, int64_t N, int64_t p,
                                               const SampleCells& sc, double (&x)[DIM]) {
  int64_t c = 0;
#pragma unroll
  for (int j = 0; j < DIM; ++j) {
    x[j] = X[(int64_t)j * N + p];
    const int u = (int)((x[j] - sc.lo[j]) * sc.inv_w[j]);
    c = c * sc.g + (u < sc.g ? u : sc.g - 1);
  }
  return c;
}

// How many sample points the cells of every stride-th point name, kNamePoints
// points in all: what the lookup by cell would save (one point a thread).
constexpr int kNamePoints = 8192;
template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_named_samples(const double* __restrict__ X, int64_t N, int64_t stride, SampleCells sc,
                const unsigned long long* __restrict__ mask, uint32_t* __restrict__ named) {
  const int64_t p = (blockIdx.x * (int64_t)kBlock + threadIdx.x) * stride;
  uint32_t m = 0;
  if (p < N) {
    double x[DIM];
    const unsigned long long* mp = mask + sample_cell<DIM>(X, N, p, sc, x) * kCellWords;
    for (int w = 0; w < kCellWords; ++w) m += (uint32_t)__popcll(mp[w]);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) m += __shfl_xor(m, o, 64);
  if ((threadIdx.x & 63) == 0) atomicAdd(named, m);
}

template <int DIM>
__global__ void __launch_bounds__(kBlock)
k_dist_histogram_cells(const double* __restrict__ X, int64_t N,
                       const int64_t* __restrict__ sample, int ns, SampleCells sc, double inv_bw,
                       int count_bins, double skip_d2,
                       const unsigned long long* __restrict__ mask,
                       const uint8_t* __restrict__ used, uint64_t* __restrict__ counts,
                       const uint32_t* __restrict__ named, uint32_t most) {
  if (*named > most) return;  // counted pair by pair
  __shared__ uint32_t h[kMaxBins];
  __shared__ double sx[DIM][kCellSamples];
  __shared__ int64_t sid[kCellSamples];
  const float inv_bw_f = (float)inv_bw;
  const bool use_f = inv_bw >= 0x1p-60 && inv_bw <= 0x1p60;
  for (int b = threadIdx.x; b < count_bins; b += kBlock) h[b] = 0;
  for (int i = threadIdx.x; i < ns; i += kBlock) {
    sid[i] = sample[i];
#pragma unroll
    for (int j = 0; j < DIM; ++j) sx[j][i] = X[(int64_t)j * N + sid[i]];
  }
  __syncthreads();
  for (int64_t p = blockIdx.x * (int64_t)kBlock + threadIdx.x; p < N;
       p += (int64_t)gridDim.x * kBlock) {
    double x[DIM];
    const int64_t c = sample_cell<DIM>(X, N, p, sc, x);
    const unsigned long long* mp = mask + c * kCellWords;
    uint32_t words = used[c];
    while (words) {
      const int w = __builtin_ctz(words);
      words &= words - 1;
      unsigned long long m = mp[w];
      while (m) {
        const int i = w * 64 + __builtin_ctzll(m);
        m &= m - 1;
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
          const double t = __dsub_rn(x[j], sx[j][i]);
          s = __dadd_rn(s, __dmul_rn(t, t));
        }
        if (s > skip_d2 || p == sid[i]) continue;
        const int b = dist_bin(s, inv_bw, inv_bw_f, use_f);
        if (b < count_bins) atomicAdd(&h[b], 1u);
      }
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < count_bins; b += kBlock)
    if (h[b]) atomicAdd((unsigned long long*)&counts[b], (unsigned long long)h[b]);
}

}  // namespace

int launch_sample_pair_sums(const double* X, int64_t N, int n, const int64_t* sample,
                            int64_t ns, double* SX, double* part, hipStream_t s) {
  if (ns < 2) return 0;
  k_gather_sample<<<(int)std::min<int64_t>(ceil_div(ns, kBlock), 1024), kBlock, 0, s>>>(
      X, N, n, sample, ns, SX);
  KNN_LAUNCHED();
  int nb = (int)(ns < 65535 ? ns : 65535);
  switch (n) {
    case 1: k_pair_sums<1><<<nb, kBlock, 0, s>>>(SX, ns, part); break;
    case 2: k_pair_sums<2><<<nb, kBlock, 0, s>>>(SX, ns, part); break;
    case 3: k_pair_sums<3><<<nb, kBlock, 0, s>>>(SX, ns, part); break;
    case 4: k_pair_sums<4><<<nb, kBlock, 0, s>>>(SX, ns, part); break;
    case 5: k_pair_sums<5><<<nb, kBlock, 0, s>>>(SX, ns, part); break;
    case 6: k_pair_sums<6><<<nb, kBlock, 0, s>>>(SX, ns, part); break;
    default: throw Error(KNN_EINVAL, "dims out of range");
  }
  KNN_LAUNCHED();
  return (int)ns;
}

void launch_dist_histogram(const double* X, int64_t N, int n, const int64_t* sample,
                           int64_t ns, double inv_bw, int n_bins, uint64_t* counts,
                           hipStream_t s, int count_bins, int64_t pstride, double max_abs,
                           const double* lo, const double* hi, DevBuf<uint64_t>* cell_masks) {
  KNN_CHECK(n_bins >= 1 && n_bins <= kMaxBins, KNN_EINVAL, "n_bins must be in [1, 4096]");
  if (count_bins <= 0 || count_bins > n_bins) count_bins = n_bins;
  KNN_CHECK(pstride >= 1, KNN_EINTERNAL, "histogram point stride must be >= 1");
  launch_zero(counts, n_bins * sizeof(uint64_t), s);
  if (ns <= 0 || N <= 0) return;
  // distances whose bin is certainly >= count_bins skip the square root
  double lim = (double)count_bins / inv_bw;
  double skip_d2 = lim * lim * 1.0001 + 1e-300;
  // The masks by cell pay when they leave few pairs: the counted balls within
  // an eighth of the box or less, on sets whose pass over every pair takes
  // longer than building them (2e6 points on; about 25 us), in 2-4 dimensions
  // (in 5-6 a skewed set's dense cells name most of the sample: exponential
  // 6-D 2.2e6 built in 1.7 ms instead of 1.4).  Clustered 2-D, 2e7 points x 500
  // sample points: 1910 us by the pairs, 255 us and 61 us for the masks.
  // But where a few points far out make the box wide, most points share a cell
  // and its mask names most of the sample (three far points at 100 times the
  // others' extent, 8e6: 2-D 0.98 ms by cell and 1.32 by the pairs, 3-D 2.89 and
  // 1.51).  So: no masks if a cell is wider than the mean distance, and else a
  // count over 8192 points decides on the device which of the two passes runs
  // (the other's blocks end at once; 10 us): by cell if the cells name at most a
  // third of the sample (of the pairs 1/8 and 1/16 lose the 2-D case above).
  uint32_t* named = nullptr;
  uint32_t named_most = 0;
  constexpr int64_t kNamedShare = 3;
  if (n <= 4 && lo && cell_masks && pstride == 1 && count_bins < n_bins && ns <= kCellSamples &&
      N >= ((int64_t)1 << 21) && max_abs < 1e150 && skip_d2 < 1e300) {
    SampleCells sc{};
    int g = 1;
    for (;;) {
      int64_t c = 1;
      for (int j = 0; j < n; ++j) c *= g + 1;
      if (c > kMaxCells) break;
      ++g;
    }
    sc.g = g;
    double part = 1.0, w_max = 0.0;
    const double rad = std::sqrt(skip_d2);
    int64_t cells = 1;
    for (int j = 0; j < n; ++j) {
      const double ext = hi[j] - lo[j];
      sc.lo[j] = lo[j];
      sc.w[j] = ext / g;
      sc.inv_w[j] = ext > 0 && std::isfinite(g / ext) ? g / ext : 0.0;
      w_max = std::max(w_max, sc.w[j]);
      if (sc.inv_w[j] > 0) part *= std::min(1.0, (2.0 * rad + sc.w[j]) / ext);
      else sc.w[j] = ext;  // one cell
      cells *= g;
    }
    sc.slack = 1e-6 * w_max + 1e-12 * max_abs;
    if (part <= 0.125 && w_max * inv_bw <= n_bins) {
      static_assert(kCellWords == 8, "a byte of used words a cell");
      cell_masks->reserve((size_t)(cells * kCellWords + cells / 8 + 2));
      auto* mask = reinterpret_cast<unsigned long long*>(cell_masks->p);
      auto* used = reinterpret_cast<uint8_t*>(mask + cells * kCellWords);
      named = reinterpret_cast<uint32_t*>(mask + cells * kCellWords + cells / 8 + 1);
      named_most = (uint32_t)(kNamePoints * ns / kNamedShare);
      launch_zero(named, sizeof(uint64_t), s);
      const int nbc = (int)std::min<int64_t>(ceil_div(cells * kCellWords, kBlock), 2048);
      const int nbp = (int)std::min<int64_t>(ceil_div(N, kBlock), 4096);
#define KNN_CELLS(D)                                                                            \
  k_sample_cells<D><<<nbc, kBlock, 0, s>>>(X, N, sample, (int)ns, sc, cells,                    \
                                           skip_d2 * (1.0 + 1e-9), mask, used);                 \
  KNN_LAUNCHED();                                                                               \
  k_named_samples<D><<<kNamePoints / kBlock, kBlock, 0, s>>>(X, N, N / kNamePoints, sc, mask,   \
                                                             named);                            \
  KNN_LAUNCHED();                                                                               \
  k_dist_histogram_cells<D><<<nbp, kBlock, 0, s>>>(X, N, sample, (int)ns, sc, inv_bw, count_bins, \
                                                   skip_d2, mask, used, counts, named, named_most)
      switch (n) {
        case 2: KNN_CELLS(2); break;
        case 3: KNN_CELLS(3); break;
        case 4: KNN_CELLS(4); break;
        default: throw Error(KNN_EINVAL, "dims out of range");
      }
#undef KNN_CELLS
      KNN_LAUNCHED();
    }
  }
  // The single-precision test.  With A = max_abs (every |coordinate|), each
  // coordinate's conversion to float errs by at most A 2^-24 (plus 2^-149
  // below float's normal range), so a float difference df_j of the converted
  // values satisfies |df_j| <= (|x_j - q_j| + e)(1 + 2^-24), e = 2 A 2^-24 +
  // 2^-148; the float sum sf of the n squares, each added by a fused
  // multiply-add (one rounding of 2^-24 per step), is at most
  // sum df_j^2 (1 + 2^-24)^n <= sum df_j^2 (1 + 2^-20).  Hence
  // d = ||x - q|| >= sqrt(sf / (1 + 2^-20)) /
  // (1 + 2^-24) - sqrt(n) e, and sf > (L + sqrt(n) e)^2 (1 + 2^-18) gives
  // d > L = sqrt(skip_d2 (1 + 2^-49)), so the double-precision d^2 (n + 1
  // roundings of 2^-53 each) exceeds skip_d2: such a pair is never counted.
  // The relative bounds need the float values in the normal range: the test
  // is used only for thresholds in [2^-100, 1e38] (below, the 2^-149
  // absolute rounding of subnormal squares is no longer negligible).
  float skip_f = INFINITY;
  if (max_abs >= 0 && max_abs < 1e30 && std::isfinite(skip_d2)) {
    const double e = 2.0 * max_abs * 0x1p-24 + 0x1p-148;
    const double L = std::sqrt(skip_d2 * (1.0 + 0x1p-49));
    const double lim_f = L + std::sqrt((double)n) * e;
    const double T = lim_f * lim_f * (1.0 + 0x1p-18);
    if (T < 1e38 && T >= 0x1p-100) {
      float tf = (float)T;
      if ((double)tf < T) tf = std::nextafter(tf, INFINITY);
      skip_f = tf;
    }
  }
  // The single-precision bin.  With y = x - mid, |y_j| <= A (half the box), and
  // its conversion, a float difference is (y_j - q_j + e_j)(1 + 2^-24),
  // |e_j| <= A 2^-23, and the root of the float sum, times inv_bw, is
  // ||y - q + e|| inv_bw (1 + r) with |r| < 2^-21 (n + 2 half roundings of
  // 2^-24, the hardware root's 2^-23, the two roundings of the product).  So it
  // differs from the exact value by at most sqrt(n) A inv_bw 2^-23 + 2^-21 of
  // itself.  The kernel allows 2^-20 of itself and a quarter more of the first
  // term, which also covers the rounding of y and, for A >= 2^-38, squares
  // below float's normal range.  A pair of the point with itself has 0, an edge,
  // and is left to the double-precision path.  With a larger bound most
  // wavefronts hold a pair near an edge and go through both: 2-3 dimensions take
  // it up to 0.004 (6e5 2-D points in a box 100 times as wide as most of them,
  // 0.02: index built in 0.75 ms, in 0.69 by double precision alone), 4-6, whose
  // d^2 costs more, up to 0.025 (the same 2.2e6 in 6-D, 0.02: 1.06 and 1.18 ms;
  // lognormal 5-D 6e5, 0.05: 0.94 and 0.87).
  Centre at{};
  float err = INFINITY;
  if (lo && hi) {
    double A = 0.0;
    for (int j = 0; j < n; ++j) {
      at.mid[j] = lo[j] + (hi[j] - lo[j]) * 0.5;
      A = std::max(A, std::max(hi[j] - at.mid[j], at.mid[j] - lo[j]));
    }
    const double e = 1.25 * std::sqrt((double)n) * A * inv_bw * 0x1p-23;
    if (A >= 0x1p-38 && A <= 0x1p60 && inv_bw >= 0x1p-60 && inv_bw <= 0x1p60 &&
        e <= (n <= 3 ? 0.004 : 0.025))
      err = (float)(e * (1.0 + 0x1p-20));
    if (!(err < INFINITY)) at = Centre{};
  }
  // four points per thread (one LDS read of a sample point serves them all)
  // on 2^18 points and more, and the sample split over the blocks until there
  // are 1024 (1e4 points took 10 blocks of the whole sample: the index was
  // built in 709 us, now 149)
  const int64_t nP = ceil_div(N, pstride);
  const int pts = nP < ((int64_t)1 << 18) ? 1 : kPtsAll;
  const int64_t want = ceil_div(nP, (int64_t)kBlock * pts);
  const int nx = (int)(want < 2048 ? want : 2048);
  const int ny = (int)std::max<int64_t>(1, std::min<int64_t>(1024 / nx, ns / 16));
  const dim3 nb(nx, ny);
  // without the bound (points so far out that the single precision of the others'
  // coordinates is coarse beside a bin; points given without their box): 6e5 2-D
  // points, three of them far out, index built in 0.85 ms with the single-precision
  // bin's instructions, 0.68 without
#define KNN_HIST(D, P, F)                                                                       \
  k_dist_histogram<D, P, F><<<nb, kBlock, 0, s>>>(X, N, pstride, sample, ns, inv_bw, count_bins, \
                                                  skip_d2, skip_f, at, err, counts, named, named_most)
#define KNN_HIST_BINS(D, P)  \
  if (err < INFINITY)        \
    KNN_HIST(D, P, true);    \
  else                       \
    KNN_HIST(D, P, false);   \
  break
  switch (n * 8 + pts) {
    case 2 * 8 + 1: KNN_HIST_BINS(2, 1);
    case 3 * 8 + 1: KNN_HIST_BINS(3, 1);
    case 4 * 8 + 1: KNN_HIST_BINS(4, 1);
    case 5 * 8 + 1: KNN_HIST_BINS(5, 1);
    case 6 * 8 + 1: KNN_HIST_BINS(6, 1);
    case 2 * 8 + kPtsAll: KNN_HIST_BINS(2, kPtsAll);
    case 3 * 8 + kPtsAll: KNN_HIST_BINS(3, kPtsAll);
    case 4 * 8 + kPtsAll: KNN_HIST_BINS(4, kPtsAll);
    case 5 * 8 + kPtsAll: KNN_HIST_BINS(5, kPtsAll);
    case 6 * 8 + kPtsAll: KNN_HIST_BINS(6, kPtsAll);
    default: throw Error(KNN_EINVAL, "dims out of range");
  }
#undef KNN_HIST_BINS
#undef KNN_HIST
  KNN_LAUNCHED();
}

}  // namespace knn
