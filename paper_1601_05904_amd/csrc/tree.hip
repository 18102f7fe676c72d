// Hierarchical summation of the weighted mean (Eq. 1) for large jobs; see tree_core.h for the
// expansion.  The squares are blocks of the even grid's cells, so their points are runs of the
// cell-ordered arrays and need no further sort.
//
// Steps: k_tree_plan (geometry), k_tree_gather (z in cell order, and whether the sums pay), k_tree_p2m (moments of the
// leaves and of the level above, from the points), k_tree_up (each further level from the one below,
// and the squares inside dense leaves), the queries ordered along the Hilbert curve, k_tree_eval (the sums).
#include <float.h>
#include <math.h>

#include "aidw_internal.h"
#include "knn_core.h"
#include "pair_core.h"
#include "tree_core.h"

namespace aidw {

namespace {

using namespace tree;

// (l, m) of each coefficient, orders ascending and l ascending within an order, and its place.
struct CoefTable {
  uint8_t l[kCoefs], m[kCoefs];
  uint16_t off[kCoefs];
};
constexpr CoefTable make_coefs() {
  CoefTable t{};
  int c = 0;
  for (int o = 0; o <= kOrder; ++o)
    for (int l = o & 1; l <= o; l += 2) {
      t.l[c] = (uint8_t)l;
      t.m[c] = (uint8_t)((o - l) / 2);
      t.off[c] = (uint16_t)coef_offset(l, (o - l) / 2);
      ++c;
    }
  return t;
}
__device__ constexpr CoefTable kCoef = make_coefs();
static_assert(coef_offset(0, kOrder / 2) + 2 <= kChild, "a record holds every order and its links");

// Entries (J, k), J + k <= kOrder, of the shift's first stage.
constexpr int kTri = (kOrder + 1) * (kOrder + 2) / 2;
struct TriTable {
  uint8_t J[kTri], k[kTri];
  float c[kTri];  // C(J, j) / 2^j at J (J + 1) / 2 + j
};
constexpr TriTable make_tri() {
  TriTable t{};
  int c = 0;
  for (int J = 0; J <= kOrder; ++J)
    for (int k = 0; k + J <= kOrder; ++k) {
      t.J[c] = (uint8_t)J;
      t.k[c] = (uint8_t)k;
      ++c;
    }
  for (int J = 0; J <= kOrder; ++J) {
    double b = 1.0;
    for (int j = 0; j <= J; ++j) {
      t.c[J * (J + 1) / 2 + j] = (float)b;
      b = b * (J - j) / (j + 1) / 2;
    }
  }
  return t;
}
__device__ constexpr TriTable kTriT = make_tri();
__device__ inline int tri_row(int J) { return J * (kOrder + 1) - J * (J - 1) / 2; }  // first entry of row J

// The jobs of a launch: one, passed by value, or an array.
struct OneJob {
  Job j;
  __device__ const Job& operator[](int) const { return j; }
};
struct ManyJobs {
  const Job* j;
  __device__ const Job& operator[](int i) const { return j[i]; }
};

// Geometry from the grid scalars (one workgroup per job).  Leaves of about kLeafPoints points: 2^bs cells a side, bs the
// nearest to log2 sqrt(kLeafPoints cells / points), then as much larger as the node budget needs.
template <typename Jobs>
__global__ void k_tree_plan(Jobs jobs, uint32_t* __restrict__ zero_word) {
  if (threadIdx.x != 0) return;
  const Job& job = jobs[blockIdx.x];
  if (zero_word && blockIdx.x == 0) *zero_word = 0u;
  const GridScalars g = *job.gs;
  const int n = job.n, node_cap = job.node_cap, level_cap = job.level_cap;
  Plan p{};
  p.ncol = g.ncol;
  p.nrow = g.nrow;
  p.minx = g.minx;
  p.miny = g.miny;
  p.inv = g.inv_cw;
  // the side must square into float32's range with room for the scaled distances
  if (g.status != AIDW_OK || !(g.cwd > 1e-12) || !(g.cwd < 1e12)) p.bad = 1;
  const double per_cell = (double)n / (double)g.ncells;
  int bs = 0;
  while (bs < 20 && per_cell * (double)(1ll << (2 * bs)) * 2.0 < (double)kLeafPoints) ++bs;
  for (;; ++bs) {
    int64_t total = 0;
    int nx = (int)(((int64_t)g.ncol + (1ll << bs) - 1) >> bs), ny = (int)(((int64_t)g.nrow + (1ll << bs) - 1) >> bs);
    int l = 0;
    bool fits = true;
    for (;; ++l) {
      if (total + (int64_t)nx * ny > node_cap || nx > kMaxSide || ny > kMaxSide) {
        fits = false;
        break;
      }
      p.nx[l] = nx;
      p.ny[l] = ny;
      p.off[l] = (int)total;
      p.h[l] = g.cwd * (double)(1ll << bs) * (double)(1ll << l);
      total += (int64_t)nx * ny;
      if ((nx <= kTopSide && ny <= kTopSide) || l + 1 == level_cap) break;
      nx = (nx + 1) >> 1;
      ny = (ny + 1) >> 1;
    }
    if (fits) {
      p.levels = l + 1;
      break;
    }
    if (bs >= 30) {
      p.bad = 1;
      p.levels = 1;
      p.nx[0] = p.ny[0] = 1;
      break;
    }
  }
  p.bs = bs;
  // an opened square's coordinates have 14 bits on the stack
  p.fine = p.nx[0] <= kMaxSide / 2 && p.ny[0] <= kMaxSide / 2 ? min(bs, kFine) : 0;
  // how far points lie from the centres (Plan::widen)
  const float far = fmaxf(fmaxf(fabsf(g.minx), fabsf(g.maxx)), fmaxf(fabsf(g.miny), fabsf(g.maxy))) +
                    2.0f * (float)p.h[0];
  const float spacing = __builtin_amdgcn_ldexpf(1.0f, __builtin_amdgcn_frexp_expf(far) - 24);
  const float cells = __builtin_amdgcn_ldexpf(1.0f, bs);  // of a leaf's side
  const float off0 = (spacing * g.inv_cw + 2.0f * (float)slack_cells(g.ncol, g.nrow)) / cells;
  if (!(off0 <= kCoarse)) p.bad = 1;
  auto finest = [&]() { return __builtin_amdgcn_ldexpf(off0, p.fine); };
  while (p.fine > 0 && !(finest() <= 0.125f * kCoarse)) --p.fine;
  p.widen = __builtin_amdgcn_logf(1.0f + off0);
  p.widen_fine = __builtin_amdgcn_logf(1.0f + finest());
  p.rim = __builtin_amdgcn_logf(1.0f + (1.0f + finest()) * (float)M_SQRT1_2 / (1.5f - finest()));
  for (int d = 0; d < kFine; ++d) p.pool[d] = node_cap + d * 4 * refine_capacity(n);
  *job.plan = p;
}

// The cell-ordered points with room for a chunk's over-read.  A z beyond the limit (a NaN's bits are
// above every number's) turns the plan off, as does a leaf of too many points, before any is summed.
__global__ __launch_bounds__(256) void k_tree_gather(Job job, const float* __restrict__ sx, const float* __restrict__ sy,
                                                     const int32_t* __restrict__ sidx, const float* __restrict__ z,
                                                     int npad, float* __restrict__ tx, float* __restrict__ ty,
                                                     float* __restrict__ tz) {
  const int n = job.n;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t b = 0u;
  bool dense = false;
  if (i < npad) {
    const bool in = i < n;
    const float v = in ? z[sidx[i]] : 0.0f;
    dense = dense_leaf_at(job, i);
    tx[i] = in ? sx[i] : 0.0f;
    ty[i] = in ? sy[i] : 0.0f;
    tz[i] = v;
    b = __float_as_uint(v) & 0x7fffffffu;
  }
  // only values in reach of the limit are reported
  if (__any(dense || b >= __float_as_uint(kZLimit)) && (threadIdx.x & 63) == 0) job.plan->bad = 1;
}

// ---------------------------------------------------------------- moments

// Orders a wavefront's LDS accesses before and after (its lanes run in step).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

constexpr int kTabStride = 37;                 // r^l (34 floats), |r|^2, z, padded to an odd stride
constexpr int kChunkPoints = 32;               // points per table
constexpr int kWaveLds = 64 * 20;              // floats: a point table, or half of the lanes' 40 sums
constexpr int kFoldPoints = 512;               // points per float32 sum

// One wavefront's points (tx, ty, tz at first[row] ..., the rows' points numbered through) about
// the centre (cx, cy), added to acc[kCoefs][4] (num re, num im, den re, den im; float64, LDS), up to
// order O.  kChunkPoints points at a time leave their powers r^l, |r|^2 and z in tab.  A lane takes the pair
// l = p, O - p (O / 2 + 2 coefficients whatever p) for every G-th point, so a point's powers are read
// O / 2 + 1 times and the multiplications by |r|^2 run over m in registers; the G lanes' sums meet
// in LDS.  Returns the lane's part of sum |z|.
template <int O>
__device__ double add_points(const float* __restrict__ tx, const float* __restrict__ ty, const float* __restrict__ tz,
                             int lo, int incl, int len, int nrows, int total, float cx, float cy, float ih,
                             float* __restrict__ tab, double* __restrict__ acc) {
  constexpr int kPairs = O / 2 + 1, kSlots = O / 2 + 2, G = 64 / kPairs;
  static_assert(kSlots == 10 && kChunkPoints * kTabStride <= kWaveLds, "the table and the exchange fit");
  const int lane = threadIdx.x & 63;
  const int p = lane % kPairs, g = lane / kPairs;
  const int la = p, lb = O - p, na = (O - la) / 2 + 1;  // slots 0 .. na - 1 are (la, m), the rest (lb, m)
  double sabs = 0.0;
  for (int f0 = 0; f0 < total; f0 += kFoldPoints) {
    float a[kSlots][4];
#pragma unroll
    for (int i = 0; i < kSlots; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) a[i][j] = 0.0f;
    const int f1 = min(total, f0 + kFoldPoints);
    for (int b = f0; b < f1; b += kChunkPoints) {
      const int e = b + lane;
      const int cnt = min(kChunkPoints, f1 - b);
      int pos = 0;  // the point's place in the cell order: its row's first plus its number there
      for (int k = 0; k < nrows; ++k) {
        const int end = __builtin_amdgcn_readlane(incl, k), beg = end - __builtin_amdgcn_readlane(len, k);
        if (e >= beg && e < end) pos = __builtin_amdgcn_readlane(lo, k) + (e - beg);
      }
      wave_sync();
      if (lane < cnt) {
        const float x = (tx[pos] - cx) * ih, y = (ty[pos] - cy) * ih, z = tz[pos];
        float* t = tab + lane * kTabStride;
        float re = 1.0f, im = 0.0f;
#pragma unroll
        for (int l = 0; l <= O; ++l) {
          t[2 * l] = re;
          t[2 * l + 1] = im;
          const float nr = __builtin_fmaf(re, x, -(im * y));
          im = __builtin_fmaf(re, y, im * x);
          re = nr;
        }
        t[34] = __builtin_fmaf(x, x, y * y);
        t[35] = z;
        sabs += (double)fabsf(z);
      }
      wave_sync();
      if (g < G) {
        for (int j = g; j < cnt; j += G) {
          const float* t = tab + j * kTabStride;
          float re = t[2 * la], im = t[2 * la + 1];
          const float re_b = t[2 * lb], im_b = t[2 * lb + 1];
          const float s = t[34], z = t[35];
#pragma unroll
          for (int i = 0; i < kSlots; ++i) {
            if (i > 0) {
              re = i == na ? re_b : re * s;
              im = i == na ? im_b : im * s;
            }
            a[i][0] = __builtin_fmaf(z, re, a[i][0]);
            a[i][1] = __builtin_fmaf(z, im, a[i][1]);
            a[i][2] += re;
            a[i][3] += im;
          }
        }
      }
      wave_sync();
    }
    // the G lanes of a pair, half of the slots at a time: slot i of lane (g, p) at
    // tab[(4 (i mod 5) + j) * 64 + lane]
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) tab[(4 * i + j) * 64 + lane] = a[5 * half + i][j];
      wave_sync();
      for (int q = lane; q < 4 * kCoefs; q += 64) {
        const int c = q >> 2, j = q & 3, l = kCoef.l[c], m = kCoef.m[c];
        const bool first = l <= O / 2;
        const int pp = first ? l : O - l, slot = (first ? m : (O - pp) / 2 + 1 + m) - 5 * half;
        if (slot < 0 || slot >= 5) continue;
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < G; ++k) v += (double)tab[(4 * slot + j) * 64 + k * kPairs + pp];
        acc[q] += v;
      }
      wave_sync();
    }
  }
  return sabs;
}

// Writes a record from the float64 moments (unscaled: the factor 2 of l > 0 is applied here).
__device__ inline void store_moments(float* __restrict__ rec, int q, double v) {
  const int c = q >> 2, j = q & 3, l = kCoef.l[c], o = kCoef.off[c];
  if (l == 0) {
    if (j == 0) rec[o] = (float)v;
    if (j == 2) rec[o + 1] = (float)v;
  } else {
    rec[o + j] = (float)(2.0 * v);
  }
}

// The points of columns [c0, c1), rows [r0, r1) of the grid about (cx, cy) (add_points); returns their count.
// More than `limit`, which turn the plan off, are not summed: a wavefront sums 16 in a microsecond, and one
// far outlier can put all points into a leaf (2^18 and 16,384 queries: 34.2 -> 2.3 ms, every pair 1.1).
__device__ __forceinline__ int add_cells(const float* __restrict__ tx, const float* __restrict__ ty,
                                         const float* __restrict__ tz, const int32_t* __restrict__ cell_start, int ncol,
                                         int c0, int c1, int r0, int r1, float cx, float cy, float ih,
                                         float* __restrict__ tab, double* __restrict__ acc, double& sabs, int limit) {
  const int lane = threadIdx.x & 63;
  int count = 0;
  for (int rb = r0; rb < r1; rb += 64) {
    const int row = rb + lane;
    int lo = 0, len = 0;
    if (row < r1) {
      lo = cell_start[(int64_t)row * ncol + c0];
      len = cell_start[(int64_t)row * ncol + c1] - lo;
    }
    int incl = len;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (lane >= o) incl += t;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63), nrows = min(64, r1 - rb);
    count += total;
    if (count > limit) return count;
    sabs += add_points<kOrder>(tx, ty, tz, lo, incl, len, nrows, total, cx, cy, ih, tab, acc);
  }
  return count;
}

// One lane: four squares for a square of many points, -1 - depth levels below the leaves' parents.
__device__ inline void refine(Plan* __restrict__ plan, float* __restrict__ nodes, int idx, int count, int depth, int ix,
                              int iy) {
  int base = 0;
  if (count > kRefine && depth < plan->fine) {
    base = plan->pool[depth] + 4 * (int)atomicAdd(&plan->refined[depth], 1u);
    int* first = reinterpret_cast<int*>(nodes + (size_t)base * kRec);
    first[kParentX] = ix;
    first[kParentY] = iy;
  }
  reinterpret_cast<int*>(nodes + (size_t)idx * kRec)[kChild] = base;
}

// A wavefront's work space for the moments of points.
struct PointSums {
  float tab[kWaveLds];
  double acc[4 * kCoefs];
};

// Levels 0 and 1 from the points: one workgroup per level-1 square, one wavefront per leaf of it.
// Each wavefront adds its points about the leaf's centre and about the square's; the four shares of
// the square are then added.
template <typename Jobs>
__global__ __launch_bounds__(256, 5) void k_tree_p2m(Jobs jobs, const float* __restrict__ tx,
                                                     const float* __restrict__ ty, const float* __restrict__ tz) {
  __shared__ PointSums s_sum[4];
  __shared__ double s_abs[4];
  __shared__ int s_cnt[4];
  __shared__ int s_off;
  const Job& job = jobs[blockIdx.y];
  Plan* const plan = job.plan;
  const int32_t* __restrict__ cell_start = job.cell_start;
  float* __restrict__ nodes = job.nodes;
  // other workgroups of this launch may turn the plan off: one thread asks for all
  if (threadIdx.x == 0) s_off = *(volatile const int32_t*)&plan->bad;
  __syncthreads();
  if (s_off) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const bool two = plan->levels > 1;
  const int nx1 = two ? plan->nx[1] : (plan->nx[0] + 1) >> 1, ny1 = two ? plan->ny[1] : (plan->ny[0] + 1) >> 1;
  const int ncol = plan->ncol, bs = plan->bs;
  for (int id = blockIdx.x; id < nx1 * ny1; id += gridDim.x) {
    const int py = id / nx1, px = id - py * nx1;
    const int ix = 2 * px + (w & 1), iy = 2 * py + (w >> 1);
    const bool live = ix < plan->nx[0] && iy < plan->ny[0];
    const int c0 = ix << bs, c1 = min(ncol, (ix + 1) << bs);
    const int r0 = iy << bs, r1 = live ? min(plan->nrow, (iy + 1) << bs) : r0;
    float cx0, cy0, cx1, cy1;
    centre(plan, 0, ix, iy, cx0, cy0);
    centre(plan, 1, px, py, cx1, cy1);
    const float ih0 = (float)(1.0 / plan->h[0]);
    double sabs = 0.0, unused = 0.0;
    int count = 0;
    double* const acc = s_sum[w].acc;
    for (int pass = 0; pass < (two ? 2 : 1); ++pass) {
      for (int q = lane; q < 4 * kCoefs; q += 64) acc[q] = 0.0;
      wave_sync();
      if (pass == 0)
        count = add_cells(tx, ty, tz, cell_start, ncol, c0, c1, r0, r1, cx0, cy0, ih0, s_sum[w].tab, acc, sabs,
                          job.dense);
      else
        add_cells(tx, ty, tz, cell_start, ncol, c0, c1, r0, r1, cx1, cy1, 0.5f * ih0, s_sum[w].tab, acc, unused,
                  job.dense);
      if (pass == 0) {
        for (int o = 32; o > 0; o >>= 1) sabs += __shfl_xor(sabs, o, 64);
        if (live) {
          const int idx = plan->off[0] + iy * plan->nx[0] + ix;
          float* rec = nodes + (size_t)idx * kRec;
          for (int q = lane; q < 4 * kCoefs; q += 64) store_moments(rec, q, acc[q]);
          if (lane == 0) {
            rec[0] = (float)count;
            rec[1] = (float)sabs;
            rec[2] = cx0;
            rec[3] = cy0;
            refine(plan, nodes, idx, count, 0, ix, iy);
          }
        }
        if (lane == 0) {
          s_abs[w] = sabs;
          s_cnt[w] = count;
          if (count > job.dense) plan->bad = 1;
        }
      }
    }
    if (two) {
      __syncthreads();
      float* rec = nodes + (size_t)(plan->off[1] + id) * kRec;
      for (int q = threadIdx.x; q < 4 * kCoefs; q += 256)
        store_moments(rec, q, (s_sum[0].acc[q] + s_sum[1].acc[q]) + (s_sum[2].acc[q] + s_sum[3].acc[q]));
      if (threadIdx.x == 0) {
        rec[0] = (float)(s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3]);
        rec[1] = (float)((s_abs[0] + s_abs[1]) + (s_abs[2] + s_abs[3]));
        rec[2] = cx1;
        rec[3] = cy1;
      }
      __syncthreads();
    }
  }
}

// Moments of a level from the four squares below, in float64: with lambda = h_child / h_parent = 1/2
// and d = (c_child - c_parent) / h_parent, r' = lambda r + d, hence
//   mu'_{JK} = sum_{j,k} C(J,j) lambda^j d^(J-j)  C(K,k) lambda^k conj(d)^(K-k)  mu_{jk},
// first over j, then over k.  One wavefront per child, one workgroup per parent.
struct ShiftSums {
  double2 pow[4][kOrder + 1];  // d^i
  float c[kTri];               // C(J,j) / 2^j at J (J + 1) / 2 + j
  double t[4][kTri][4];        // the first stage
  double m[4][kCoefs][4];      // child's mu, then its share of the parent's
  float head[4][2];
};
__device__ __forceinline__ void shift_up(const Plan* __restrict__ plan, float* __restrict__ nodes, int lvl, int block, int blocks,
                         ShiftSums& sh) {
  auto& s_pow = sh.pow;
  auto& s_c = sh.c;
  auto& s_t = sh.t;
  auto& s_m = sh.m;
  auto& s_head = sh.head;
  const int nx = plan->nx[lvl];
  const int all = nx * plan->ny[lvl];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int t = threadIdx.x; t < kTri; t += 256) s_c[t] = kTriT.c[t];
  for (int id = block; id < all; id += blocks) {
    const int py = id / nx, px = id - py * nx;
    const int chx = 2 * px + (w & 1), chy = 2 * py + (w >> 1);
    const bool live = chx < plan->nx[lvl - 1] && chy < plan->ny[lvl - 1];
    const float* child = nodes + (size_t)(plan->off[lvl - 1] + (live ? chy * plan->nx[lvl - 1] + chx : 0)) * kRec;
    float pcx, pcy, ccx, ccy;
    centre(plan, lvl, px, py, pcx, pcy);
    centre(plan, lvl - 1, chx, chy, ccx, ccy);
    if (lane <= kOrder) {
      const double ih = 1.0 / plan->h[lvl];
      double bx = ((double)ccx - (double)pcx) * ih, by = ((double)ccy - (double)pcy) * ih;
      double re = 1.0, im = 0.0;
#pragma unroll
      for (int bit = 1; bit <= kOrder; bit <<= 1) {
        if (lane & bit) {
          const double a = re * bx - im * by;
          im = re * by + im * bx;
          re = a;
        }
        const double a = bx * bx - by * by;
        by = 2.0 * bx * by;
        bx = a;
      }
      s_pow[w][lane] = make_double2(re, im);
    }
    for (int q = lane; q < kCoefs; q += 64) {
      const int l = kCoef.l[q], o = kCoef.off[q];
      double v[4] = {0, 0, 0, 0};
      if (live) {
        if (l == 0) {
          v[0] = child[o];
          v[2] = child[o + 1];
        } else {
          for (int i = 0; i < 4; ++i) v[i] = 0.5 * (double)child[o + i];
        }
      }
      for (int i = 0; i < 4; ++i) s_m[w][q][i] = v[i];
    }
    if (lane == 0) {
      s_head[w][0] = live ? child[0] : 0.0f;
      s_head[w][1] = live ? child[1] : 0.0f;
    }
    __syncthreads();
    for (int t = lane; t < kTri; t += 64) {
      const int J = kTriT.J[t], k = kTriT.k[t];
      double a[4] = {0, 0, 0, 0};
      for (int j = 0; j <= J; ++j) {
        const double c = (double)s_c[J * (J + 1) / 2 + j];
        const double2 d = s_pow[w][J - j];
        const double ex = c * d.x, ey = c * d.y;
        const bool up = j >= k;
        const double* mu = s_m[w][up ? coef_place(j, k) : coef_place(k, j)];
        const double i0 = up ? mu[1] : -mu[1], i1 = up ? mu[3] : -mu[3];
        a[0] += ex * mu[0] - ey * i0;
        a[1] += ex * i0 + ey * mu[0];
        a[2] += ex * mu[2] - ey * i1;
        a[3] += ex * i1 + ey * mu[2];
      }
      for (int i = 0; i < 4; ++i) s_t[w][t][i] = a[i];
    }
    __syncthreads();
    for (int q = lane; q < kCoefs; q += 64) {
      const int K = kCoef.m[q], J = kCoef.l[q] + K;
      double a[4] = {0, 0, 0, 0};
      for (int k = 0; k <= K; ++k) {
        const double c = (double)s_c[K * (K + 1) / 2 + k];
        const double2 d = s_pow[w][K - k];
        const double ex = c * d.x, ey = c * d.y;
        const double* tt = s_t[w][tri_row(J) + k];
        a[0] += ex * tt[0] + ey * tt[1];
        a[1] += ex * tt[1] - ey * tt[0];
        a[2] += ex * tt[2] + ey * tt[3];
        a[3] += ex * tt[3] - ey * tt[2];
      }
      for (int i = 0; i < 4; ++i) s_m[w][q][i] = a[i];
    }
    __syncthreads();
    float* rec = nodes + (size_t)(plan->off[lvl] + id) * kRec;
    for (int q = threadIdx.x; q < 4 * kCoefs; q += 256) {
      const int c = q >> 2, i = q & 3;
      store_moments(rec, q, (s_m[0][c][i] + s_m[1][c][i]) + (s_m[2][c][i] + s_m[3][c][i]));
    }
    if (threadIdx.x == 0) {
      rec[0] = (s_head[0][0] + s_head[1][0]) + (s_head[2][0] + s_head[3][0]);
      rec[1] = (s_head[0][1] + s_head[1][1]) + (s_head[2][1] + s_head[3][1]);
      rec[2] = pcx;
      rec[3] = pcy;
    }
    __syncthreads();
  }
}

// Moments of the squares below refined ones, depth levels below the leaves: one workgroup per
// refined square, one wavefront per square below.
__device__ __forceinline__ void fine_squares(Plan* __restrict__ plan, const int32_t* __restrict__ cell_start, float* __restrict__ nodes,
                             const float* __restrict__ tx, const float* __restrict__ ty, const float* __restrict__ tz,
                             int depth, int block, int blocks, PointSums& sum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int count = (int)plan->refined[depth - 1], pool = plan->pool[depth - 1], sh = plan->bs - depth;
  const float ih = (float)((double)(1 << depth) / plan->h[0]);
  for (int id = block; id < count; id += blocks) {
    const int* first = reinterpret_cast<const int*>(nodes + (size_t)(pool + 4 * id) * kRec);
    const int ix = 2 * first[kParentX] + (w & 1), iy = 2 * first[kParentY] + (w >> 1);
    const int c0 = min(plan->ncol, ix << sh), c1 = min(plan->ncol, (ix + 1) << sh);
    const int r0 = min(plan->nrow, iy << sh), r1 = min(plan->nrow, (iy + 1) << sh);
    float cx, cy;
    centre(plan, -depth, ix, iy, cx, cy);
    for (int q = lane; q < 4 * kCoefs; q += 64) sum.acc[q] = 0.0;
    wave_sync();
    double sabs = 0.0;
    const int n = add_cells(tx, ty, tz, cell_start, plan->ncol, c0, c1, r0, r1, cx, cy, ih, sum.tab, sum.acc, sabs,
                            kDenseLeaf);
    for (int o = 32; o > 0; o >>= 1) sabs += __shfl_xor(sabs, o, 64);
    const int idx = pool + 4 * id + w;
    float* rec = nodes + (size_t)idx * kRec;
    for (int q = lane; q < 4 * kCoefs; q += 64) store_moments(rec, q, sum.acc[q]);
    if (lane == 0) {
      rec[0] = (float)n;
      rec[1] = (float)sabs;
      rec[2] = cx;
      rec[3] = cy;
      refine(plan, nodes, idx, n, depth, ix, iy);
    }
    wave_sync();
  }
}

// Level lvl from the squares below it, and, by the first fine_blocks workgroups of a job, the squares
// depth levels below the leaves (depth 0: none); neither needs the other, and one launch fills the
// chip better than two (2^18 mixture: 960 us of summation against 1010).
template <typename Jobs>
__global__ __launch_bounds__(256, 5) void k_tree_up(Jobs jobs, int lvl, int depth, int fine_blocks,
                                                    const float* __restrict__ tx, const float* __restrict__ ty,
                                                    const float* __restrict__ tz) {
  __shared__ __align__(16) unsigned char s_mem[sizeof(ShiftSums) > 4 * sizeof(PointSums) ? sizeof(ShiftSums)
                                                                                         : 4 * sizeof(PointSums)];
  const Job& job = jobs[blockIdx.y];
  if (job.plan->bad) return;
  const int block = (int)blockIdx.x;
  if (block < fine_blocks)
    fine_squares(job.plan, job.cell_start, job.nodes, tx, ty, tz, depth, block, fine_blocks,
                 reinterpret_cast<PointSums*>(s_mem)[threadIdx.x >> 6]);
  else if (lvl < job.plan->levels)
    shift_up(job.plan, job.nodes, lvl, block - fine_blocks, (int)gridDim.x - fine_blocks,
             *reinterpret_cast<ShiftSums*>(s_mem));
}

// The query order: the Hilbert index of the query's tile.  (Ordering by alpha class inside stretches
// of the curve gives more groups of one class, whose weights are cheaper, but wider ones: 2^20 uniform
// 2.10 ms in plain order, 2.33 ms with stretches of 1024 queries.)
// Where the plan is off the pair kernel takes over, with the keys as they are (the alpha classes) and the
// points in their own order.
__global__ __launch_bounds__(256) void k_tree_keys(const Plan* __restrict__ plan, const float* __restrict__ qx,
                                                   const float* __restrict__ qy, int m, int hbits,
                                                   uint32_t* __restrict__ keys, const float* __restrict__ x,
                                                   const float* __restrict__ y, const float* __restrict__ z, int n,
                                                   int npad, float* __restrict__ tx, float* __restrict__ ty,
                                                   float* __restrict__ tz) {
  const int stride = gridDim.x * blockDim.x;
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (!off(plan)) {
    if (i < m) keys[i] = tile(plan, hbits, qx[i], qy[i]);
    return;
  }
  for (; i < npad; i += stride) {
    const bool in = i < n;
    tx[i] = in ? x[i] : 0.0f;
    ty[i] = in ? y[i] : 0.0f;
    tz[i] = in ? z[i] : 0.0f;
  }
}

// ---------------------------------------------------------------- evaluation

// w = t^(-alpha/2) with the class chosen at run time (pw = 0: general,
// nh = -alpha/2), r = rsq(t).  The general form splits t = m 2^e: the hardware log2 of a large t has
// an absolute error of several 1e-7 (its last bit), which alpha/2 multiplies, while log2 m is good to
// 6e-8; nh e is kept with its rounding error.
__device__ __forceinline__ float weight(float t, float r, int pw, float nh) {
  if (pw == 0) {
    const float lm = __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(t));
    const float e = (float)__builtin_amdgcn_frexp_expf(t);
    const float p = nh * e;
    return __builtin_amdgcn_exp2f(p) * __builtin_amdgcn_exp2f(__builtin_fmaf(nh, lm, __builtin_fmaf(nh, e, -p)));
  }
  const float r2 = r * r, r4 = r2 * r2;
  float w = (pw & 1) ? r : 1.0f;
  if (pw & 2) w *= r2;
  if (pw & 4) w *= r4;
  if (pw & 8) w *= r4 * r4;
  return w;
}

// A lane's query (the scaled form of pair_core.h: sc a power of two, distances times sc) and sums.
// Terms are added in float32 four at a time and those sums in float64: the error of a result is
// then that of the weights, not of the summation.
struct Query {
  float qxs, qys, ns, nh;
  float num_t, den_t;  // float32 sums since the last fold
  double num, den;
  float sabs;          // sum of w |z|, a lower bound of it
  float least;         // the smallest weight in a distant square in units of its centre's
};

// POW = -1: the class pw chosen at run time.
template <int POW>
__device__ __forceinline__ void pair(Query& L, float x, float y, float z, int pw) {
  const float dx = __builtin_fmaf(x, L.ns, L.qxs);
  const float dy = __builtin_fmaf(y, L.ns, L.qys);
  const float t = __builtin_fmaf(dx, dx, dy * dy);
  float w;
  if constexpr (POW == -1)
    w = weight(t, __builtin_amdgcn_rsqf(t), pw, L.nh);
  else if constexpr (POW == 0)
    w = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(t) * L.nh);
  else
    w = pair::ipow<POW>(__builtin_amdgcn_rsqf(t));
  L.num_t = __builtin_fmaf(w, z, L.num_t);
  L.sabs = __builtin_fmaf(w, fabsf(z), L.sabs);
  L.den_t += w;
}

__device__ __forceinline__ void fold(Query& L) {
  L.num += (double)L.num_t;
  L.den += (double)L.den_t;
  L.num_t = L.den_t = 0.0f;
}

// The points [lo, hi) of the cell order, eight per wave-uniform fetch, the next fetch issued while
// one is evaluated (it may read up to 15 points past hi: the arrays are padded).
template <int POW>
__device__ __forceinline__ void run_pairs(Query& L, const float* __restrict__ tx, const float* __restrict__ ty,
                                          const float* __restrict__ tz, int lo, int hi, int pw) {
  constexpr int C = 8;
  float cx[C], cy[C], cz[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    cx[i] = tx[lo + i];
    cy[i] = ty[lo + i];
    cz[i] = tz[lo + i];
  }
  int p = lo;
  for (; p + C <= hi; p += C) {
    float nx[C], ny[C], nz[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      nx[i] = tx[p + C + i];
      ny[i] = ty[p + C + i];
      nz[i] = tz[p + C + i];
    }
#pragma unroll
    for (int i = 0; i < C; ++i) {
      pair<POW>(L, cx[i], cy[i], cz[i], pw);
      if (i % 4 == 3) fold(L);
    }
#pragma unroll
    for (int i = 0; i < C; ++i) {
      cx[i] = nx[i];
      cy[i] = ny[i];
      cz[i] = nz[i];
    }
  }
#pragma unroll
  for (int i = 0; i < C - 1; ++i)
    if (p + i < hi) {
      pair<POW>(L, cx[i], cy[i], cz[i], pw);
      if (i == 3) fold(L);
    }
  fold(L);
}

struct Points {
  const int32_t* __restrict__ cs;
  const float* __restrict__ tx;
  const float* __restrict__ ty;
  const float* __restrict__ tz;
  int ncol;
};

// The points of the cells [cx0, cx1] of the rows r0, r0 + step, ... <= r1: 64 rows' bounds are
// loaded at a time, one per lane.
template <int POW>
__device__ __forceinline__ void near_rows(Query& L, const Points& P, int cx0, int cx1, int r0, int r1, int step,
                                          int pw = 0) {
  const int lane = threadIdx.x & 63;
  for (; r0 <= r1; r0 += 64 * step) {
    const int r = r0 + lane * step;
    int lo = 0, hi = 0;
    if (r <= r1) {
      lo = P.cs[(int64_t)r * P.ncol + cx0];
      hi = P.cs[(int64_t)r * P.ncol + cx1 + 1];
    }
    uint64_t live = __ballot(lo < hi);
    while (live) {
      const int i = __builtin_ctzll(live);
      live &= live - 1;
      run_pairs<POW>(L, P.tx, P.ty, P.tz, __builtin_amdgcn_readlane(lo, i), __builtin_amdgcn_readlane(hi, i),
                     pw);
    }
  }
}

// Points of the cells [cx0, cx1] of the rows r0 .. r1.
__device__ __forceinline__ int count_points(const Points& P, int cx0, int cx1, int r0, int r1) {
  int c = 0;
  for (int r = r0 + (int)(threadIdx.x & 63); r <= r1; r += 64)
    c += P.cs[(int64_t)r * P.ncol + cx1 + 1] - P.cs[(int64_t)r * P.ncol + cx0];
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  return __builtin_amdgcn_readfirstlane(c);
}

// The square's expansion to order P at v (|v|^2 = s): Horner in s for each l, then in v over l.
// quad(o): the four numbers at offset o of the record (a multiple of four).
template <int P, typename Quad>
__device__ __forceinline__ void expand(Quad quad, float vx, float vy, float s, const float* f, float& pn, float& pd) {
  float sf[P / 2 + 1];
#pragma unroll
  for (int m = 1; m <= P / 2; ++m) sf[m] = s * f[m];
  float tr = 0.0f, ti = 0.0f, ur = 0.0f, ui = 0.0f;  // num and den, Horner over l
#pragma unroll
  for (int l = P; l >= 1; --l) {
    const int K = (P - l) / 2;
    float4 y = quad(coef_offset(l, K));
#pragma unroll
    for (int m = K; m >= 1; --m) {
      const float g = sf[m] * f[l + m];
      const float4 c = quad(coef_offset(l, m - 1));
      y.x = __builtin_fmaf(y.x, g, c.x);
      y.y = __builtin_fmaf(y.y, g, c.y);
      y.z = __builtin_fmaf(y.z, g, c.z);
      y.w = __builtin_fmaf(y.w, g, c.w);
    }
    if (l < P) {
      const float wx = f[l + 1] * vx, wy = f[l + 1] * vy;
      y.x = __builtin_fmaf(tr, wx, __builtin_fmaf(ti, wy, y.x));
      y.y = __builtin_fmaf(ti, wx, __builtin_fmaf(-tr, wy, y.y));
      y.z = __builtin_fmaf(ur, wx, __builtin_fmaf(ui, wy, y.z));
      y.w = __builtin_fmaf(ui, wx, __builtin_fmaf(-ur, wy, y.w));
    }
    tr = y.x;
    ti = y.y;
    ur = y.z;
    ui = y.w;
    // the reads of the next l wait for this one's sums: all reads at once would not fit the registers
    if (P >= 8) asm volatile("" : : "v"(tr), "v"(ti), "v"(ur), "v"(ui) : "memory");
  }
  // l = 0: the pairs (num, den) of m = 0, 1 are one quad, those of 2, 3 the next ...
  auto pair0 = [&](int m, float& x, float& y) {
    const float4 c = quad(m < 2 ? 4 : coef_offset(0, m & ~1));
    x = (m & 1) ? c.z : c.x;
    y = (m & 1) ? c.w : c.y;
  };
  constexpr int K = P / 2;
  float a, c;
  pair0(K, a, c);
#pragma unroll
  for (int m = K; m >= 2; --m) {
    const float g = sf[m] * f[m];
    float x, y;
    pair0(m - 1, x, y);
    a = __builtin_fmaf(a, g, x);
    c = __builtin_fmaf(c, g, y);
  }
  const float g = sf[1] * f[1], wx = f[1] * vx, wy = f[1] * vy;
  a = __builtin_fmaf(a, g, __builtin_fmaf(tr, wx, ti * wy));
  c = __builtin_fmaf(c, g, __builtin_fmaf(ur, wx, ui * wy));
  float x, y;
  pair0(0, x, y);
  pn = x + a;
  pd = y + c;
}

// One distant square to order P; head = (count, sum |z|, centre x, centre y).
template <int P, typename Quad>
__device__ __forceinline__ void add_square(Query& L, Quad quad, float hs, int pw, const float* f) {
  const float4 head = quad(0);
  const float dx = __builtin_fmaf(head.z, L.ns, L.qxs), dy = __builtin_fmaf(head.w, L.ns, L.qys);
  const float t = __builtin_fmaf(dx, dx, dy * dy);
  const float r = __builtin_amdgcn_rsqf(t);
  const float w0 = weight(t, r, pw, L.nh);
  const float g = hs * r, vs = g * r;
  float pn, pd;
  expand<P>(quad, dx * vs, dy * vs, g * g, f, pn, pd);
  L.num += (double)(w0 * pn);
  L.den += (double)(w0 * pd);
  L.sabs = __builtin_fmaf(L.least * w0, head.y, L.sabs);
}

// The first line of a record: head and the orders up to 2.
struct Line {
  float4 v[4];
};
__device__ __forceinline__ Line load_line(const float* __restrict__ rec) {
  Line h;
#pragma unroll
  for (int i = 0; i < 4; ++i) h.v[i] = make_float4(rec[4 * i], rec[4 * i + 1], rec[4 * i + 2], rec[4 * i + 3]);
  return h;
}

// The squares listed by the lanes of `mask` (record number idx, side h), all to the low order P: the
// coefficients are scalar operands, and the next square's first line is fetched while one is evaluated.
template <int P>
__device__ __forceinline__ void add_squares(Query& L, uint64_t mask, int idx, float h, float sc,
                                            const float* __restrict__ nodes, int pw, const float* f) {
  int i = __builtin_ctzll(mask);
  const float* rec = nodes + (size_t)__builtin_amdgcn_readlane(idx, i) * kRec;
  Line line = load_line(rec);
  do {
    mask &= mask - 1;
    const int j = mask ? __builtin_ctzll(mask) : i;
    const float* next = nodes + (size_t)__builtin_amdgcn_readlane(idx, j) * kRec;
    const Line ahead = load_line(next);
    const float hs = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h), i)) * sc;
    add_square<P>(
        L, [&](int o) { return o < 16 ? line.v[o / 4] : make_float4(rec[o], rec[o + 1], rec[o + 2], rec[o + 3]); }, hs, pw,
        f);
    line = ahead;
    rec = next;
    i = j;
  } while (mask);
}

// The same for a high order, whose coefficients do not fit the scalar registers: a wavefront's lanes
// copy the record to LDS (the next one's loads are in flight meanwhile) and read it by broadcasts.
template <int P>
__device__ __forceinline__ void add_squares_lds(Query& L, uint64_t mask, int idx, float h, float sc,
                                                const float* __restrict__ nodes, int pw, const float* f,
                                                float* __restrict__ buf) {
  static_assert(kRec == 320, "80 quads: one per lane and 16 more");
  const int lane = threadIdx.x & 63;
  const float4* nodes4 = reinterpret_cast<const float4*>(nodes);
  float4* buf4 = reinterpret_cast<float4*>(buf);
  int i = __builtin_ctzll(mask);
  const float4* rec = nodes4 + (size_t)__builtin_amdgcn_readlane(idx, i) * (kRec / 4);
  float4 r0 = rec[lane], r1 = rec[64 + (lane & 15)];
  do {
    mask &= mask - 1;
    const int j = mask ? __builtin_ctzll(mask) : i;
    wave_sync();
    buf4[lane] = r0;
    if (lane < 16) buf4[64 + lane] = r1;
    wave_sync();
    rec = nodes4 + (size_t)__builtin_amdgcn_readlane(idx, j) * (kRec / 4);
    r0 = rec[lane];
    r1 = rec[64 + (lane & 15)];
    const float hs = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(h), i)) * sc;
    add_square<P>(L, [&](int o) { return buf4[o / 4]; }, hs, pw, f);
    i = j;
  } while (mask);
}

__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_min(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// One workgroup of S wavefronts per group of 64 queries that follow each other on the Hilbert
// curve.  First the points of the cells near the group's box, rows dealt to the wavefronts; their
// sums of w and w |z| set how accurately a distant square has to be evaluated.  Then, level by
// level from the leaves, the squares whose parents are near and which are not themselves: a lane
// takes a square, finds the order that serves every query of the group, and the squares of one
// order are then evaluated one after the other, each by all lanes.
// A group whose box holds many points (queries on both sides of a gap) is taken in parts; in a dense
// place it starts below the leaves instead: the near points of a leaf of 700 cost 60,000
// instructions a query, the squares of 176 inside it and their near points 34,000.
// What bounds it: the vector instructions of the pairs and expansions (about 40,000 per query at
// 2^20 uniform, against 11 million for all pairs) and the latency of the scalar and header loads,
// which four wavefronts a SIMD do not hide altogether (three, five and six were slower: 1.47 ms of
// summation with four, 1.60 with three, 1.51 with five and six, whose registers spill).
// Measured, whole summation: 2^20 uniform 209 -> 1.6 ms, 2^18 mixture 13.3 -> 0.9 ms, 2^20 mixture 210 ->
// 2.7 (3.9 from the leaves on).
// Output: qz, or with PARTIAL the float64 (num, den).
template <typename Jobs, bool PARTIAL>
__global__ __launch_bounds__(512, 4) void k_tree_eval(Jobs jobs, int njobs, const float* __restrict__ tx,
                                                      const float* __restrict__ ty, const float* __restrict__ tz,
                                                      const float* __restrict__ qx, const float* __restrict__ qy,
                                                      const float* __restrict__ alpha_f,
                                                      const float* __restrict__ d1sq,
                                                      const uint32_t* __restrict__ perm, Thresholds thr,
                                                      float* __restrict__ qz, double2* __restrict__ partial) {
  // per wavefront: a record, the stack of opened squares, and with S > 1 the sums of its queries
  extern __shared__ __align__(16) unsigned char s_mem[];
  const int lane = threadIdx.x & 63;
  const int wave = uniform((int)threadIdx.x >> 6);
  const int S = uniform((int)blockDim.x >> 6);
  float* const buf = reinterpret_cast<float*>(s_mem) + wave * kRec;
  uint32_t* const stack = reinterpret_cast<uint32_t*>(s_mem) + S * kRec + wave * kStack;
  double2 (*s_sum)[kGroup] = reinterpret_cast<double2 (*)[kGroup]>(s_mem + (size_t)S * 4 * (kRec + kStack));
  float (*s_abs)[kGroup] = reinterpret_cast<float (*)[kGroup]>(s_sum + S);
  // consecutive groups are neighbours: chunks of them go to one XCD, whose L2 then holds their squares
  constexpr int kChunkGroups = 16;
  int grp = (int)blockIdx.x;
  {
    const int span = 8 * kChunkGroups;
    const int base = grp / span * span, r = grp - base;
    if (base + span <= (int)gridDim.x) grp = base + (r & 7) * kChunkGroups + (r >> 3);
  }
  int at = 0;  // the group's job: the last one whose first group is not past it
  for (int hi = njobs - 1; at < hi;) {
    const int mid = (at + hi + 1) >> 1;
    if (jobs[mid].group0 <= grp)
      at = mid;
    else
      hi = mid - 1;
  }
  const Job& job = jobs[at];
  const Plan* __restrict__ plan = job.plan;
  if (off(plan)) return;
  const int32_t* __restrict__ cell_start = job.cell_start;
  const float* __restrict__ nodes = job.nodes;
  const uint32_t fast_mask = job.fast_mask;
  const int p0 = job.q0 + (grp - job.group0) * kGroup;
  const int nq = min(kGroup, job.q0 + job.m - p0);
  const uint32_t q = perm[p0 + min(lane, nq - 1)];
  const float fx = qx[q], fy = qy[q], alpha = alpha_f[q], d1 = d1sq[q];
  // the group's class: the integer power that all its queries have, 0 if none has one; a mixed group
  // takes the general weights in their more accurate form, as its integer classes had better ones
  const bool whole = alpha >= 1.0f && alpha <= 8.0f && alpha == floorf(alpha) && ((fast_mask >> (int)alpha) & 1u);
  const float a0 = __uint_as_float(uniform((int)__float_as_uint(alpha)));
  const bool mixed = __any(whole) && __any(alpha != a0);
  const int pw = uniform(whole && !mixed ? (int)alpha : 0);
  const float sc = pair::pow2_scale(d1);
  // (read beside the group's first loads: read where they are used, 10^5 uniform points take 12 % longer)
  const float rim = plan->rim, widen = plan->widen, widen_fine = plan->widen_fine;
  Query L{fx * sc, fy * sc, -sc, -0.5f * alpha, 0.0f, 0.0f, 0.0, 0.0, 0.0f, exp2f(-rim * alpha)};
  const int bs = plan->bs, ncol = plan->ncol, nrow = plan->nrow, levels = plan->levels, fine = plan->fine;
  // squares per side at a level, from the cells: a load of each would be waited for level by level
  auto squares = [&](int cells, int l) { return (int)(((int64_t)cells + (1ll << (bs + l)) - 1) >> (bs + l)); };
  const int colq = knn::clamp_cell((fx - plan->minx) * plan->inv, ncol);
  const int rowq = knn::clamp_cell((fy - plan->miny) * plan->inv, nrow);
  const Points P{cell_start, tx, ty, tz, ncol};
  float f[kOrder + 1];
  const float ch = 0.5f * alpha - 1.0f;
#pragma unroll
  for (int i = 1; i <= kOrder; ++i) f[i] = __builtin_fmaf(ch, 1.0f / (float)i, 1.0f);

  for (int qa = 0, qb; qa < nq; qa = qb) {
    // the part [qa, qb) of the group: halved while that saves more than the far squares of another part
    int x0, x1, y0, y1;
    int dep = 0;  // the part's smallest squares are dep levels below the leaves
    auto box = [&](int a, int b) {
      const bool in = lane >= a && lane < b;
      const int lx = colq >> (bs - dep), ly = rowq >> (bs - dep);
      x0 = in ? lx : 0x7fffffff;
      x1 = in ? lx : 0;
      y0 = in ? ly : 0x7fffffff;
      y1 = in ? ly : 0;
      for (int o = 32; o > 0; o >>= 1) {
        x0 = min(x0, __shfl_xor(x0, o, 64));
        x1 = max(x1, __shfl_xor(x1, o, 64));
        y0 = min(y0, __shfl_xor(y0, o, 64));
        y1 = max(y1, __shfl_xor(y1, o, 64));
      }
      x0 = uniform(x0);
      x1 = uniform(x1);
      y0 = uniform(y0);
      y1 = uniform(y1);
    };
    auto near_points = [&](int a, int b) {
      box(a, b);
      const int b2 = bs - dep;
      return count_points(P, max(0, x0 - kNear) << b2, min(ncol, (x1 + kNear + 1) << b2) - 1,
                          max(0, y0 - kNear) << b2, min(nrow, (y1 + kNear + 1) << b2) - 1);
    };
    qb = nq;
    int c = near_points(qa, qb);
    // in dense places smaller squares leave fewer points near; a box across a gap stays as wide
    while (dep < fine && c > kFineNear && c > kRefine / 2 * (x1 - x0 + 1 + 2 * kNear) * (y1 - y0 + 1 + 2 * kNear)) {
      ++dep;
      const int c1 = near_points(qa, qb);
      if (c1 > c - (c >> 2)) {
        --dep;
        break;
      }
      c = c1;
    }
    while (c > kSplitPoints && qb - qa > 1) {
      // at the largest step between two consecutive queries
      const int lx = colq >> (bs - dep), ly = rowq >> (bs - dep);
      const int step = max(abs(__shfl_down(lx, 1, 64) - lx), abs(__shfl_down(ly, 1, 64) - ly));
      int best = lane >= qa && lane < qb - 1 ? step * 64 + (63 - lane) : -1;
      for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
      const int mid = uniform(64 - (best & 63));
      const int c1 = near_points(qa, mid), c2 = near_points(mid, qb);
      if (c1 + c2 + kFarCost > c - (c >> 3)) break;
      qb = mid;
      c = c1;
    }
    box(qa, qb);
    const bool in = lane >= qa && lane < qb;
    L.num = L.den = 0.0;
    L.sabs = 0.0f;
    {
      const int b2 = bs - dep;
      const int cx0 = max(0, x0 - kNear) << b2, cx1 = min(ncol, (x1 + kNear + 1) << b2) - 1;
      const int ry0 = max(0, y0 - kNear) << b2, ry1 = min(nrow, (y1 + kNear + 1) << b2) - 1;
      switch (pw) {
#define AIDW_CASE(p) \
  case p: near_rows<p>(L, P, cx0, cx1, ry0 + wave, ry1, S); break;
        AIDW_CASE(1)
        AIDW_CASE(2)
        AIDW_CASE(3)
        AIDW_CASE(4)
        AIDW_CASE(5)
        AIDW_CASE(6)
        AIDW_CASE(7)
        AIDW_CASE(8)
#undef AIDW_CASE
        default:
          if (mixed)
            near_rows<-1>(L, P, cx0, cx1, ry0 + wave, ry1, S, 0);
          else
            near_rows<0>(L, P, cx0, cx1, ry0 + wave, ry1, S);
      }
    }
    double base_den = 0.0;
    float base_abs = 0.0f;
    if (S > 1) {
      s_sum[wave][lane] = make_double2(L.num, L.den);
      s_abs[wave][lane] = L.sabs;
      __syncthreads();
      for (int w = 0; w < S; ++w)
        if (w != wave) {
          base_den += s_sum[w][lane].y;
          base_abs += s_abs[w][lane];
        }
      __syncthreads();
    }
    // (a coincident query has infinite sums, which the fix-up replaces: it asks for no accuracy; one whose
    // d1sq is 0 without a data point at its place keeps its sums)
    const float qx0 = wave_min(in ? fx : INFINITY), qx1 = wave_max(in ? fx : -INFINITY);
    const float qy0 = wave_min(in ? fy : INFINITY), qy1 = wave_max(in ? fy : -INFINITY);
    const float amin = wave_min(in ? alpha : INFINITY), amax = wave_max(in ? alpha : 0.0f);
    // a square's share of a query's sums is at most (1 + rho)^alpha
    const float lcap = amax * rim;
    for (int l0 = -dep; l0 < levels; ++l0) {
      const float h0 = (float)plan->h[max(l0, 0)] * __uint_as_float((uint32_t)(127 + min(l0, 0)) << 23);
      // log2 of the largest weight per unit of a query's sums, for a square at distance h0
      const float ld = log2f(h0);
      const float lw = alpha * (ld + log2f(sc));
      const float rden = in ? __builtin_amdgcn_rcpf((float)(base_den + L.den)) : 0.0f;
      const float rabs = in ? __builtin_amdgcn_rcpf(base_abs + L.sabs) : 0.0f;
      const float kden = wave_max(in ? __builtin_amdgcn_logf(rden) - lw : -INFINITY);
      const float kabs = wave_max(in ? __builtin_amdgcn_logf(rabs) - lw : -INFINITY);
      const int nx = squares(ncol, l0), ny = squares(nrow, l0), up = l0 + dep;
      const int ax0 = max(0, (x0 >> up) - kNear), ax1 = min(nx - 1, (x1 >> up) + kNear);
      const int ay0 = max(0, (y0 >> up) - kNear), ay1 = min(ny - 1, (y1 >> up) + kNear);
      int bx0 = 0, bx1 = nx - 1, by0 = 0, by1 = ny - 1;
      if (l0 + 1 < levels) {
        bx0 = 2 * max(0, (x0 >> (up + 1)) - kNear);
        bx1 = min(nx - 1, 2 * ((x1 >> (up + 1)) + kNear) + 1);
        by0 = 2 * max(0, (y0 >> (up + 1)) - kNear);
        by1 = min(ny - 1, 2 * ((y1 >> (up + 1)) + kNear) + 1);
      }
      const int W = bx1 - bx0 + 1, total = W * (by1 - by0 + 1);
      int sp = 0;  // squares on the stack
      for (int b = wave; b < total || sp > 0;) {
        // 64 squares, one per lane: the four of up to 16 opened ones, else the next of the list
        int lvl, ix, iy;
        bool live;
        if (sp > 0) {
          const int cnt = min(16, sp);
          sp -= cnt;
          live = (lane >> 2) < cnt;
          const uint32_t e = live ? stack[sp + (lane >> 2)] : 0u;
          lvl = max(-fine, (int)(e >> 28) - kFine - 1);
          ix = 2 * (int)(e & 0x3fffu) + (lane & 1);
          iy = 2 * (int)((e >> 14) & 0x3fffu) + ((lane >> 1) & 1);
          live = live && ix < squares(ncol, lvl) && iy < squares(nrow, lvl);
        } else {
          const int k = b + lane * S;
          b += 64 * S;
          const int ky = k / W;
          lvl = l0;
          ix = bx0 + (k - ky * W);
          iy = by0 + ky;
          live = k < total && !(ix >= ax0 && ix <= ax1 && iy >= ay0 && iy <= ay1);
        }
        int idx = live && lvl >= 0 ? plan->off[lvl] + iy * plan->nx[lvl] + ix : 0;
        int few = -1;  // below the leaves: the points of a square that has no record
        if (__any(lvl < 0)) {
          if (live && lvl < 0) {
            idx = plan->off[0] + (iy >> -lvl) * plan->nx[0] + (ix >> -lvl);
            for (int j = -lvl - 1; j >= 0 && few < 0; --j) {
              const int base = reinterpret_cast<const int*>(nodes + (size_t)idx * kRec)[kChild];
              if (base == 0)
                few = 0;
              else
                idx = base + 2 * ((iy >> j) & 1) + ((ix >> j) & 1);
            }
            if (few == 0) {
              const int sh = bs + lvl, r1 = min(nrow, (iy + 1) << sh), c1 = min(ncol, (ix + 1) << sh);
              for (int row = iy << sh; row < r1; ++row)
                few += cell_start[(int64_t)row * ncol + c1] - cell_start[(int64_t)row * ncol + (ix << sh)];
            }
          }
        }
        const float h = __uint_as_float(__float_as_uint(h0) - ((uint32_t)(l0 - lvl) << 23));  // h0 2^(lvl - l0)
        const float4 hd = *reinterpret_cast<const float4*>(nodes + (size_t)idx * kRec);
        const float cnt = !live ? 0.0f : few >= 0 ? (float)few : hd.x;
        const float ex = fmaxf(fmaxf(qx0 - hd.z, hd.z - qx1), 0.0f), ey = fmaxf(fmaxf(qy0 - hd.w, hd.w - qy1), 0.0f);
        const float lr = 0.5f * __builtin_amdgcn_logf(__builtin_fmaf(ex, ex, ey * ey));  // log2 of the distance
        float lq = fmaxf(__builtin_amdgcn_logf(cnt) + kden, __builtin_amdgcn_logf(hd.y) + kabs) - amin * (lr - ld);
        lq = fminf(lq, lcap);
        // rho = (1 + e) (h / sqrt 2) / distance
        const float lrho = ld - 0.5f + (lvl < 0 ? widen_fine : widen) - lr - (float)(l0 - lvl);
        int tier = kTiers;
#pragma unroll
        for (int i = kTiers - 1; i >= 0; --i)
          if (!(lq + (float)(2 * i + 3) * lrho > (pw ? thr.v[pw][i] : job.thr0[i]))) tier = i;
        // the float32 roundings of the moments grow by (1 - rho)^-alpha: a square close by that holds
        // much of the sums is opened, its parts are relatively farther
        if (lrho > -2.0f && lq - amax * __builtin_amdgcn_logf(1.0f - __builtin_amdgcn_exp2f(lrho)) > 0.0f)
          tier = kTiers;
        const int order = 2 * tier + 2;
        bool end = few >= 0;
        if (tier == kTiers && lvl < 1 && !end) end = reinterpret_cast<const int*>(nodes + (size_t)idx * kRec)[kChild] == 0;
        const bool points = end ||
                            cnt * 12.0f + (float)(16 << (bs + lvl)) <= (float)(60 + 2 * (order + 1) * (order + 2));
        const int kind = cnt > 0.0f ? (points ? kTiers + 1 : tier) : -1;
        uint64_t mask = __ballot(kind == kTiers);
        if (mask) {
          if (kind == kTiers)
            stack[sp + __popcll(mask & ((1ull << lane) - 1ull))] =
                ((uint32_t)(lvl + kFine) << 28) | ((uint32_t)iy << 14) | (uint32_t)ix;
          sp += (int)__popcll(mask);
          wave_sync();
        }
        if ((mask = __ballot(kind == 0))) add_squares<2>(L, mask, idx, h, sc, nodes, pw, f);
        if ((mask = __ballot(kind == 1))) add_squares<4>(L, mask, idx, h, sc, nodes, pw, f);
        if ((mask = __ballot(kind == 2))) add_squares<6>(L, mask, idx, h, sc, nodes, pw, f);
        if ((mask = __ballot(kind == 3))) add_squares_lds<8>(L, mask, idx, h, sc, nodes, pw, f, buf);
        if ((mask = __ballot(kind == 4))) add_squares_lds<10>(L, mask, idx, h, sc, nodes, pw, f, buf);
        if ((mask = __ballot(kind == 5))) add_squares_lds<12>(L, mask, idx, h, sc, nodes, pw, f, buf);
        if ((mask = __ballot(kind == 6))) add_squares_lds<14>(L, mask, idx, h, sc, nodes, pw, f, buf);
        if ((mask = __ballot(kind == 7))) add_squares_lds<16>(L, mask, idx, h, sc, nodes, pw, f, buf);
        mask = __ballot(kind == kTiers + 1);
        while (mask) {
          const int i = __builtin_ctzll(mask);
          mask &= mask - 1;
          const int sx = __builtin_amdgcn_readlane(ix, i), sy = __builtin_amdgcn_readlane(iy, i);
          const int sh = bs + __builtin_amdgcn_readlane(lvl, i);
          near_rows<-1>(L, P, sx << sh, min(ncol, (sx + 1) << sh) - 1, sy << sh, min(nrow, (sy + 1) << sh) - 1, 1, pw);
        }
      }
    }
    double num = L.num, den = L.den;
    if (S > 1) {
      s_sum[wave][lane] = make_double2(num, den);
      __syncthreads();
      num = den = 0.0;
      for (int w = 0; w < S; ++w) {
        num += s_sum[w][lane].x;
        den += s_sum[w][lane].y;
      }
      __syncthreads();
    }
    if (in && wave == 0) {
      if constexpr (PARTIAL)
        partial[job.out0 + q] = make_double2(num, den);
      else
        qz[q] = (float)(num / den);
    }
  }
}

inline int div_up(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

}  // namespace

namespace tree {

int node_capacity(int64_t n) { return (int)(n / 12 + 512); }

int hilbert_bits(int64_t n) {
  int b = 1;
  while (b < 10 && (int64_t)(kLeafPoints / 2) << (2 * b) < n) ++b;
  return b;
}

int padded_points(int64_t n) { return (int)((n + 7) / 8 * 8 + 16); }

size_t plan_bytes() { return sizeof(Plan); }

size_t node_bytes(int64_t n) {
  return sizeof(float) * (size_t)kRec * ((size_t)node_capacity(n) + 4 * kFine * (size_t)refine_capacity(n));
}

}  // namespace tree

static Thresholds class_bounds() {
  Thresholds t{};
  for (int c = 1; c < kClasses; ++c)
    for (int i = 0; i < kTiers; ++i) t.v[c][i] = order_bound((double)c, i);
  return t;
}

// The largest leaf that hierarchical sums are kept for, by times in us: the pairs (5.2e12 a second, and the 8 %
// and the launches that a plan which turns out off adds) against the sums, for even data 110 + 4e-4 m + 3e-4 n
// and for each point of the largest leaf 0.2 + 6e-7 n: one wavefront forms a leaf's moments, and a group of
// queries pays for every point near it.  Half as many points again are let pass, for the sums are more exact.
// Whole runs, every pair / hierarchical, mixtures of 16 | 8 | 3 | 1 components, whose largest leaves hold some
// 1000 | 2000 | 3700 | 11,000 points; behind || they are off:
//   45,000 x 45,000:    624/547  | 634/700   || 700/1067  | 846/2276
//   100,000 x 100,000:  2269/752 | 2312/928  | 2348/1266  | 2611/2664
//   200,000 x 20,000:   1084/783 | 1078/1000 || 1155/1480 | 1253/3625
//   262,144 x 30,000:   1882/912 | 1951/1249 | 1998/1685  || 2094/4070
//   2^20 x 9000:       2423/2071 | 2446/2632 || 2487/4109 | 2649/10421
//   2^20 x 20,000:     4657/2025 | 4653/2349 | 4735/3977  || 4915/8826
// Jobs that share their launches hide each other's chains: pairs are then those of all of them, and a job's own
// are set against 0.0115 a point of the largest leaf (a replay of 40 jobs of 16,384 x 16,384, every pair /
// hierarchical: 2637/1379 even, 2975/2086 with 8 components, 3861/4349 with 1).
static int dense_leaf(int64_t n, int64_t m, double pairs) {
  const double room = 1.08 * pairs / 5.2e6 - 50.0 - 4e-4 * (double)m - 3e-4 * (double)n;
  const double own = fmax(0.9 * (double)n * (double)m / 5.2e6 - 14.0, 29.0);
  const double most = fmin(1.5 * room / (0.2 + 6e-7 * (double)n), own / 0.0115);
  return (int)fmin(fmax(most, (double)kRefine), (double)kDenseLeaf);
}

void tree::fill_job(Job* j, int64_t n, int64_t m, double pairs, const double* levels) {
  j->n = (int32_t)n;
  j->m = (int32_t)m;
  j->dense = dense_leaf(n, m, pairs);
  j->node_cap = node_capacity(n);
  // levels of a square box's tree, and two more for other shapes; a longer strip's top level simply
  // has more squares
  j->level_cap = 3;
  while (j->level_cap < kLevels && ((int64_t)(kLeafPoints / 2 * kTopSide * kTopSide) << (2 * (j->level_cap - 3))) < n)
    ++j->level_cap;
  double top = 0.0;
  j->fast_mask = 0;
  for (int i = 0; i < 5; ++i) {
    top = fmax(top, levels[i]);
    if (levels[i] >= 1.0 && levels[i] <= 8.0 && levels[i] == floor(levels[i])) j->fast_mask |= 1u << (int)levels[i];
  }
  for (int i = 0; i < kTiers; ++i) j->thr0[i] = order_bound(top, i);
}

namespace {

template <typename Jobs>
void launch_plan(const Jobs& jobs, int njobs, uint32_t* zero_word, hipStream_t s) {
  hipLaunchKernelGGL(k_tree_plan<Jobs>, dim3(njobs), dim3(64), 0, s, jobs, zero_word);
}

// n, level_cap: of the largest job
template <typename Jobs>
void launch_moments(const Jobs& jobs, int njobs, int64_t n, int level_cap, const float* tx, const float* ty,
                    const float* tz, hipStream_t s) {
  // squares of level 1 of a square box; a workgroup loops where a ragged shape has more
  int64_t blocks = n / (4 * kLeafPoints) + 64;
  hipLaunchKernelGGL(k_tree_p2m<Jobs>, dim3((unsigned)blocks, njobs), dim3(256), 0, s, jobs, tx, ty, tz);
  for (int l = 2; l < level_cap || l < 2 + kFine; ++l) {
    blocks = l < level_cap ? blocks / 4 + 16 : 0;
    const int depth = l < 2 + kFine ? l - 1 : 0;
    const int fine = depth ? (int)(n / (4 * kRefine) + 16 < 2048 ? n / (4 * kRefine) + 16 : 2048) : 0;
    hipLaunchKernelGGL(k_tree_up<Jobs>, dim3((unsigned)blocks + fine, njobs), dim3(256), 0, s, jobs, l, depth, fine, tx,
                       ty, tz);
  }
}

template <typename Jobs, bool PARTIAL>
void launch_eval(const Jobs& jobs, int njobs, int groups, const float* tx, const float* ty, const float* tz,
                 const float* qx, const float* qy, const float* alpha_f, const float* d1sq, const uint32_t* perm,
                 float* qz, double2* partial, hipStream_t s) {
  int S = 1;
  while (S < 8 && groups * S < 16384) S *= 2;  // wavefronts to fill the chip four times over
  const size_t lds = (size_t)S * (4 * (kRec + kStack) + (S > 1 ? kGroup * (sizeof(double2) + sizeof(float)) : 0));
  hipLaunchKernelGGL((k_tree_eval<Jobs, PARTIAL>), dim3(groups), dim3(64 * S), lds, s, jobs, njobs, tx, ty, tz, qx, qy,
                     alpha_f, d1sq, perm, class_bounds(), qz, partial);
}

}  // namespace

hipError_t launch_tree_build(const tree::Job& job, const float* sx, const float* sy, const int32_t* sidx,
                             const float* z, float* tx, float* ty, float* tz, uint32_t* zero_word, hipStream_t s) {
  launch_plan(OneJob{job}, 1, zero_word, s);
  const int npad = tree::padded_points(job.n);
  hipLaunchKernelGGL(k_tree_gather, dim3(div_up(npad, 256)), dim3(256), 0, s, job, sx, sy, sidx, z, npad, tx, ty, tz);
  launch_moments(OneJob{job}, 1, job.n, job.level_cap, tx, ty, tz, s);
  return hipGetLastError();
}

hipError_t launch_tree_eval(const tree::Job& job, const float* tx, const float* ty, const float* tz, const float* qx,
                            const float* qy, const float* alpha_f, const float* d1sq, const uint32_t* perm, float* qz,
                            hipStream_t s) {
  launch_eval<OneJob, false>(OneJob{job}, 1, div_up(job.m, kGroup), tx, ty, tz, qx, qy, alpha_f, d1sq, perm, qz,
                             nullptr, s);
  return hipGetLastError();
}

hipError_t launch_tree_plans(const tree::Job* jobs, int njobs, hipStream_t s) {
  launch_plan(ManyJobs{jobs}, njobs, nullptr, s);
  return hipGetLastError();
}

hipError_t launch_tree_moments(const tree::Job* jobs, int njobs, int64_t max_n, int max_levels, const float* tx,
                               const float* ty, const float* tz, hipStream_t s) {
  launch_moments(ManyJobs{jobs}, njobs, max_n, max_levels, tx, ty, tz, s);
  return hipGetLastError();
}

hipError_t launch_tree_evals(const tree::Job* jobs, int njobs, int groups, const float* tx, const float* ty,
                             const float* tz, const float* qx, const float* qy, const float* alpha_f, const float* d1sq,
                             const uint32_t* perm, double2* partial, hipStream_t s) {
  launch_eval<ManyJobs, true>(ManyJobs{jobs}, njobs, groups, tx, ty, tz, qx, qy, alpha_f, d1sq, perm, nullptr, partial,
                              s);
  return hipGetLastError();
}

hipError_t launch_tree_keys(const tree::Plan* plan, const float* qx, const float* qy, int m, int hbits, uint32_t* keys,
                            const float* x, const float* y, const float* z, int n, float* tx, float* ty, float* tz,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_tree_keys, dim3(div_up(m, 256)), dim3(256), 0, s, plan, qx, qy, m, hbits, keys, x, y, z, n,
                     tree::padded_points(n), tx, ty, tz);
  return hipGetLastError();
}

}  // namespace aidw
