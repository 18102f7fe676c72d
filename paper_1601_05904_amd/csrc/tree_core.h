// Hierarchical summation of Eq. 1: the shared definitions of tree.hip and its callers.
//
// The sums num = sum_i w_i z_i and den = sum_i w_i, w_i = |q - p_i|^-alpha, run over all n data
// points.  Points near the query are evaluated pair by pair; a distant square of points is
// evaluated through its moments about the square's centre c (side h):
//   with r = (p - c) / h and v = h (q - c) / |q - c|^2 (complex numbers),
//   |q - p|^-alpha = |q - c|^-alpha  sum_{j,k} b_j b_k (r conj(v))^j conj(r conj(v))^k,
//   b_j = (alpha/2)(alpha/2 + 1) ... (alpha/2 + j - 1) / j!,
// the product of the two binomial series of (1 - u)^(-alpha/2) and its conjugate, u = r conj(v).
// The moments sum_i {z_i, 1} r_i^j conj(r_i)^k do not contain alpha, so one set serves every query
// whatever its alpha.  Collected by l = j - k >= 0 and m = k (order j + k = l + 2m <= kOrder):
//   M[l][m] = (2 if l > 0) sum_i {z_i, 1} r_i^l |r_i|^(2m).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "aidw_internal.h"
#include "knn_core.h"

namespace aidw {
namespace tree {

constexpr int kOrder = 16;               // highest order of the moments
constexpr int kTiers = kOrder / 2;       // orders 2, 4, ..., kOrder are the evaluation's choices
constexpr int kNear = 1;                 // squares within kNear of the query's are opened
constexpr float kCoarse = 1.0f;           // largest e of Plan::widen in leaves, 1/8 of it below them
constexpr int kLeafPoints = 32;          // wanted mean points per leaf
constexpr int kTopSide = 8;              // squares per side at which no further level is built
constexpr int kLevels = 14;
constexpr int kMaxSide = 1 << 14;         // squares per side (a stack entry holds 14 bits of each)
// Leaves of more than kRefine points have four squares below them, and these likewise, kFine times.
constexpr int kFine = 2;
constexpr int kRefine = 128;
constexpr int kFineNear = 1500;          // near points from which a group looks for smaller squares
// Opened squares of one wavefront: at most 64 from the list, and 48 more per level below it.
constexpr int kStack = 64 + 48 * (kLevels + kFine);
static_assert(kLevels + kFine <= 16, "a stack entry holds 4 bits of the level");
constexpr int kCoefs = 81;               // (l, m) pairs
constexpr int kRec = 320;                // floats per square: 4 + sum of 2 (order + 1), padded to 64 B
// Integers in the record's padding: the first of the four squares below (0: none), and in the first of
// four the coordinates of the square above.
constexpr int kChild = 316, kParentX = 317, kParentY = 318;
constexpr int kGroup = 64;               // queries per group (one per lane)
constexpr int kClasses = 9;              // alpha classes 0 (general), 1 .. 8
constexpr int kSplitPoints = 6000;       // near points from which a group is worth splitting
constexpr int kFarCost = 3000;           // a group's far squares in pair evaluations
constexpr int kDenseLeaf = 1 << 14;      // most points that any job's leaf may hold

// A square's record: count, sum |z|, centre x, centre y, then for each (l, m) the real numbers
// (num, den) for l = 0, (num re, num im, den re, den im) for l > 0.  The first line (64 bytes) ends
// with the orders l + 2m <= 2; the further ones follow by l, m ascending, the order in which they
// are consumed: the scalar loads of one l are contiguous.
__host__ __device__ constexpr int coef_first(int l) {  // m of the first coefficient past the first line
  return l == 0 ? 2 : l <= 2 ? 1 : 0;
}
__host__ __device__ constexpr int coef_count(int l) { return (kOrder - l) / 2 + 1 - coef_first(l); }
__host__ __device__ constexpr int coef_offset(int l, int m) {
  if (m < coef_first(l)) return l == 0 ? (m == 0 ? 4 : 6) : l == 1 ? 8 : 12;
  int at = 16;
  for (int i = 1; i < l; ++i) at += 4 * coef_count(i);
  if (l == 0) {
    for (int i = 1; i <= kOrder; ++i) at += 4 * coef_count(i);
    return at + 2 * (m - 2);
  }
  return at + 4 * (m - coef_first(l));
}

// Place of mu_{jk} = sum r^j conj(r)^k, j >= k, in the coefficient order: orders ascending, l = j - k
// ascending within an order.
__host__ __device__ constexpr int coef_place(int j, int k) {
  const int o = j + k;
  const int before = (o / 2) * ((o + 1) / 2) + o - o / 2;  // coefficients of the orders below o
  return before + (j - k - (o & 1)) / 2;
}

// log2 of the largest Q rho^o for which the order P = 2 tier + 2 is taken, o = P + 1: the terms of order o of one
// square sum to at most w0 C_o(alpha) rho^o times its count (or sum |z|), C_o = Gamma(o + alpha) /
// (Gamma(alpha) o!) the Gegenbauer bound and rho = (half diagonal) / distance, and these may reach
// 2^-22 of the query's sums.  The terms of the further orders are not counted: at most some three times these
// together at alpha = 8, less below.
inline float order_bound(double alpha, int tier) {
  const int o = 2 * tier + 3;
  return (float)(-22.0 - (lgamma(o + alpha) - lgamma(alpha) - lgamma(o + 1.0)) / M_LN2);
}

// Geometry of a job's squares, made on the device from the grid scalars: level 0 squares (leaves)
// are 2^bs x 2^bs grid cells, a level l + 1 square is 2 x 2 squares of level l.  Below the leaves with
// many points levels -1 .. -fine go on; their squares are in the pools, four under one square together.
struct Plan {
  int32_t bad;       // the sums are formed directly (geometry or data out of the moments' range)
  int32_t bs, levels;
  int32_t ncol, nrow;
  float minx, miny, inv;
  int32_t nx[kLevels], ny[kLevels], off[kLevels];  // squares per row / column, first record
  double h[kLevels];                               // side
  // A centre is a float32 number, so it is off by up to half of float32's spacing at the coordinates,
  // and a point may lie past its square's side by the slack of its cell: a point's offset is up to
  // (1 + e) h / sqrt 2, e = (spacing + 2 slack) / h.  widen = log2(1 + e) of the leaves, widen_fine of the
  // smallest squares; rim = log2(1 + rho) at the largest rho of a square that is not near, with e of the
  // smallest squares (1 + e) sqrt(1/2) / (1.5 - e).
  float widen, widen_fine, rim;
  int32_t fine, pool[kFine];                       // levels below the leaves, each one's first record
  uint32_t refined[kFine];                         // squares above with four in the pool
  uint32_t next;                                   // where it is off: the pair kernel's next item
};

// Squares of more than kRefine points that n points can make at one level.
__host__ __device__ inline int refine_capacity(int64_t n) { return (int)(n / kRefine) + 1; }

// |z| from here on (or NaN) takes the direct sums: the moments' sums stay far from overflow.
constexpr float kZLimit = 1.2676506002282294e30f;  // 2^100

__device__ inline bool off(const Plan* p) { return p->bad != 0; }

// One job's share of the arrays that the jobs of a launch have in common.
struct Job {
  const GridScalars* gs;
  Plan* plan;
  const int32_t* cell_start;  // the job's cells; their entries index the common point arrays
  float* nodes;               // node_cap records
  int32_t n, node_cap, level_cap;
  int32_t dense;              // points in one leaf above which the direct sums are used
  int32_t q0, m;              // its queries: positions [q0, q0 + m) of the query order
  int32_t group0;             // its first group of kGroup queries
  uint32_t fast_mask;         // integer alpha classes that have their own weights
  int64_t out0;               // double2 output: query q at out0 + q
  float thr0[kTiers];         // log2 bounds of the orders for a group of general alpha
};

// Whether leaf i of a job holds too many points; i from the number of leaves on: false.  (Leaves of many rows, as very
// fine grids have them, are left to the kernel that forms the moments.)
__device__ inline bool dense_leaf_at(const Job& job, int i) {
  const Plan* p = job.plan;
  const int nx = p->nx[0], bs = p->bs;
  if (i >= nx * p->ny[0] || bs > 5) return false;
  const int iy = i / nx, ix = i - iy * nx;
  const int c0 = ix << bs, c1 = min(p->ncol, (ix + 1) << bs), r1 = min(p->nrow, (iy + 1) << bs);
  int count = 0;
  for (int r = iy << bs; r < r1; ++r)
    count += job.cell_start[(int64_t)r * p->ncol + c1] - job.cell_start[(int64_t)r * p->ncol + c0];
  return count > job.dense;
}

// Centre of a square, the same float32 values wherever they are needed.
__device__ inline void centre(const Plan* p, int lvl, int ix, int iy, float& cx, float& cy) {
  const double h = lvl >= 0 ? p->h[lvl] : p->h[0] / (double)(1 << -lvl);
  cx = (float)((double)p->minx + ((double)ix + 0.5) * h);
  cy = (float)((double)p->miny + ((double)iy + 0.5) * h);
}

// Index of (x, y) along the Hilbert curve over 2^bits x 2^bits tiles.
__host__ __device__ inline uint32_t hilbert(int bits, uint32_t x, uint32_t y) {
  uint32_t d = 0;
  for (int i = bits - 1; i >= 0; --i) {
    const uint32_t rx = (x >> i) & 1u, ry = (y >> i) & 1u;
    d = (d << 2) | ((3u * rx) ^ ry);
    const uint32_t mask = (1u << i) - 1u;
    x &= mask;
    y &= mask;
    if (ry == 0) {
      if (rx) {
        x = mask - x;
        y = mask - y;
      }
      const uint32_t t = x;
      x = y;
      y = t;
    }
  }
  return d;
}

// log2 of the bounds of the orders for the integer classes: v[c][t] bounds Q rho^(P + 1), P = 2 t + 2.
struct Thresholds {
  float v[kClasses][kTiers];
};

// Hilbert index of a query's tile, both axes in the same scale, the longer side spanning the curve.
__device__ inline uint32_t tile(const Plan* p, int hbits, float x, float y) {
  const float scale = (float)(1 << hbits) / (float)max(p->ncol, p->nrow);
  return hilbert(hbits, (uint32_t)knn::clamp_cell((x - p->minx) * p->inv * scale, 1 << hbits),
                 (uint32_t)knn::clamp_cell((y - p->miny) * p->inv * scale, 1 << hbits));
}

}  // namespace tree
}  // namespace aidw
