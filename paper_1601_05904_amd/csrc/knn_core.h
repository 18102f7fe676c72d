// Device code shared by the kNN kernels of the single-job path (knn.hip) and the
// batched path (batch.hip): the exact grid search of Section 3.2.4 / 4.1.4 over
// one job's grid, and the coincident-query mean.  The search rule, the stop rule
// and the (squared distance, index) ordering are described in knn.hip.
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aidw {
namespace knn {

// Cell coordinate of a float32 offset t = (x - min) * inv_cw: truncated, clamped
// into [0, nc); negative or NaN -> 0.
__device__ inline int clamp_cell(float t, int nc) {
  if (!(t >= 0.0f)) return 0;
  if (t >= 2147483520.0f) return nc - 1;
  const int c = (int)t;
  return c > nc - 1 ? nc - 1 : c;
}

// One job's grid scalars.  The CSR arrays travel beside it: cell_start indexed
// from the job's first cell, sx, sy, sidx in cell order.
struct View {
  float minx, miny, inv;
  int ncol, nrow;
  double cwd;
};

// v_min_f64 / v_max_f64 of numbers (fmin and fmax quiet their operands first, one more instruction each).
__device__ __forceinline__ double min_f64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double max_f64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// The lists of candidates.  Slots [0, KMAX - k) hold a -1 sentinel that no candidate can pass, the k
// live slots [KMAX - k, KMAX) ascending squared distances; with indices, in (d2, index) order.
template <int KMAX, int S = 0>
__device__ __forceinline__ void clear(int k, double (&bk)[KMAX]) {
  if constexpr (S < KMAX) {
    bk[S] = S < KMAX - k ? -1.0 : INFINITY;
    clear<KMAX, S + 1>(k, bk);
  }
}
template <int KMAX>
__device__ __forceinline__ void clear(int k, double (&bk)[KMAX], int32_t (&bi)[KMAX]) {
  clear<KMAX>(k, bk);
#pragma unroll
  for (int s = 0; s < KMAX; ++s) bi[s] = s < KMAX - k ? -1 : INT32_MAX;
}

// Distances only: every slot's new value depends on two old ones, a minimum and a maximum and no
// comparison, 2 KMAX - 1 instructions at a depth of two; with indices it is 11 a slot, in a chain.
template <int KMAX, int S = KMAX - 1>
__device__ __forceinline__ void insert(double (&bk)[KMAX], double d2) {
  if constexpr (S > 0) {
    bk[S] = min_f64(bk[S], max_f64(bk[S - 1], d2));
    insert<KMAX, S - 1>(bk, d2);
  } else {
    bk[0] = min_f64(bk[0], d2);
  }
}
template <int KMAX>
__device__ __forceinline__ void insert(double (&bk)[KMAX], int32_t (&bi)[KMAX], double d2, int32_t id) {
  // the comparisons of the (d2, index) order are combined with bitwise operators: each is then one
  // vector compare, where short-circuit forms compile to branches on the exec mask
  const bool take = (d2 < bk[KMAX - 1]) | ((d2 == bk[KMAX - 1]) & (id < bi[KMAX - 1]));
  if (!take) return;
  bk[KMAX - 1] = d2;
  bi[KMAX - 1] = id;
#pragma unroll
  for (int s = KMAX - 1; s > 0; --s) {
    const bool sw = (bk[s] < bk[s - 1]) | ((bk[s] == bk[s - 1]) & (bi[s] < bi[s - 1]));
    const double lo = bk[s], hi = bk[s - 1];
    const int32_t ilo = bi[s], ihi = bi[s - 1];
    bk[s - 1] = sw ? lo : hi;
    bk[s] = sw ? hi : lo;
    bi[s - 1] = sw ? ilo : ihi;
    bi[s] = sw ? ihi : ilo;
  }
}

// Distance from the query to the nearest open side (one beyond which cells remain) of the cells in
// columns [ca, cz] and rows [ra, rz].
__device__ __forceinline__ double side_distance(const View& g, double px, double py, int ca, int cz, int ra, int rz) {
  const double minxd = g.minx, minyd = g.miny, cwd = g.cwd;
  double dout = INFINITY;
  if (ca > 0) dout = fmin(dout, px - (minxd + (double)ca * cwd));
  if (cz < g.ncol - 1) dout = fmin(dout, (minxd + (double)(cz + 1) * cwd) - px);
  if (ra > 0) dout = fmin(dout, py - (minyd + (double)ra * cwd));
  if (rz < g.nrow - 1) dout = fmin(dout, (minyd + (double)(rz + 1) * cwd) - py);
  return dout;
}
// The same for the block of cells within L of the cell (c0, r0), less the slack.
__device__ __forceinline__ double reach(const View& g, double px, double py, int c0, int r0, int L, double slack) {
  return side_distance(g, px, py, c0 - L, c0 + L, r0 - L, r0 + L) - slack;
}

// The largest over the LANES lanes of a query (an aligned group of LANES consecutive lanes)
// of each lane's ceil(k / LANES)-th best d2 (+inf where a lane holds fewer):
// the group holds at least k candidates at or below it, so the k-th nearest is no larger.
template <int KMAX, int LANES>
__device__ __forceinline__ double group_kth(const double (&bk)[KMAX], int k) {
  const int kq = (k + LANES - 1) / LANES;  // the lane's kq-th best: slot KMAX - k + kq - 1
  double v = bk[KMAX - 1];
#pragma unroll
  for (int s = 0; s < KMAX; ++s)
    if (s == KMAX - k + kq - 1) v = bk[s];
#pragma unroll
  for (int o = 1; o < LANES; o <<= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Whether the k-th smallest distance over the LANES lanes of a query is below limit.
template <int KMAX, int S = 0>
__device__ __forceinline__ int below(const double (&bk)[KMAX], double limit) {
  if constexpr (S < KMAX)
    return (bk[S] < limit ? 1 : 0) + below<KMAX, S + 1>(bk, limit);
  else
    return 0;
}
template <int KMAX, int LANES>
__device__ __forceinline__ bool k_below(const double (&bk)[KMAX], int k, double limit) {
  if constexpr (LANES == 1) return bk[KMAX - 1] < limit;
  int c = below<KMAX>(bk, limit) - (KMAX - k);  // less the sentinels
#pragma unroll
  for (int o = 1; o < LANES; o <<= 1) c += __shfl_xor(c, o, 64);
  return c >= k;
}

// The k nearest data points of (fx, fy), by blocks of cells.
//
// The first block is the 5 x 5 cells around the query's (at the usual two points a cell it holds
// the ten nearest of nearly every query), or 3 x 3 where those 25 cells hold so many points that 9
// should do (with one lane and a short list, before these the cells that a still denser place
// should need); its rows are contiguous runs of points whose bounds are read together, and a lane walks
// them as one sequence, so the lanes of a wavefront differ by their blocks' totals and not row by
// row.  A block that fails the stop test grows to the level that the k-th distance asks for (twice
// the level while it holds fewer than k points), by rows and the runs beside it.
//
// LANES > 1: LANES consecutive lanes (sub = 0 .. LANES - 1) search for the same query together;
// each takes every LANES-th candidate and keeps the k best of its own, so the union of their lists
// holds the k nearest.  They stop together, when k candidates of all lanes are near enough, and
// merge_lanes reads the k nearest out in ascending order.
//
// Without indices the list is distances alone; collect then finds the indices by a second walk.
struct Block {
  int o0, o1, o2, o3, o4, e0, e1, e2, e3, e4;  // row r: candidates e(r - 1) .. e(r) - 1 of the walk, each at its number + o(r)
};

constexpr int kDenseBlock = 11;  // points per neighbour in the 25 cells from which the block is 3 x 3

// Up to five rows of cells, first .. last (from 0 on), columns [ca, cz].
__device__ __forceinline__ Block block_rows(const View& g, const int32_t* __restrict__ cell_start, int first, int last,
                                            int ca, int cz) {
  auto run = [&](int r, int& from) __attribute__((always_inline)) {
    const bool in = first + r >= 0 && first + r <= last;
    const int32_t* __restrict__ cs = cell_start + (in ? first + r : last) * g.ncol;
    from = cs[ca];
    return cs[in ? cz + 1 : ca] - from;
  };
  Block b;
  b.e0 = run(0, b.o0);
  b.e1 = b.e0 + run(1, b.o1);
  b.e2 = b.e1 + run(2, b.o2);
  b.e3 = b.e2 + run(3, b.o3);
  b.e4 = b.e3 + run(4, b.o4);
  b.o1 -= b.e0;
  b.o2 -= b.e1;
  b.o3 -= b.e2;
  b.o4 -= b.e3;
  return b;
}

// Candidate t of a block's walk.  By value: a choice between members of a struct becomes a load from a
// chosen address, which would put the struct in memory.
__device__ __forceinline__ int position(int t, int e0, int e1, int e2, int e3, int o0, int o1, int o2, int o3, int o4) {
  int o = t >= e0 ? o1 : o0;
  o = t >= e1 ? o2 : o;
  o = t >= e2 ? o3 : o;
  o = t >= e3 ? o4 : o;
  return t + o;
}

template <class F>
__device__ __forceinline__ void walk_block(const Block b, int sub, int lanes, F&& two) {
  const int total = b.e4;
  for (int t = sub; t < total; t += 2 * lanes) {
    const bool pair = t + lanes < total;
    const int p = position(t, b.e0, b.e1, b.e2, b.e3, b.o0, b.o1, b.o2, b.o3, b.o4);
    const int u = t + lanes;
    two(p, pair ? position(u, b.e0, b.e1, b.e2, b.e3, b.o0, b.o1, b.o2, b.o3, b.o4) : p, pair);
  }
}

// The cells within L1 of (c0, r0) but not within L0.
template <class F>
__device__ __forceinline__ void walk_growth(const View& g, const int32_t* __restrict__ cell_start, int c0, int r0, int L0,
                                            int L1, int sub, int lanes, F&& two) {
  const int ra = max(r0 - L1, 0), rz = min(r0 + L1, g.nrow - 1);
  const int ca = max(c0 - L1, 0), cz = min(c0 + L1, g.ncol - 1);
  for (int row = ra; row <= rz; ++row) {
    const int32_t* __restrict__ cs = cell_start + row * g.ncol;
    const bool inner = row >= r0 - L0 && row <= r0 + L0;
    const bool left = !inner || c0 - L0 > 0, right = inner && c0 + L0 < g.ncol - 1;
    // both runs' bounds are read before either is walked
    int p0 = 0, p1 = 0, p2 = 0, p3 = 0;
    if (left) {
      p0 = cs[ca];
      p1 = cs[inner ? c0 - L0 : cz + 1];
    }
    if (right) {
      p2 = cs[c0 + L0 + 1];
      p3 = cs[cz + 1];
    }
    const int first = p1 - p0, total = first + p3 - p2;
    for (int t = sub; t < total; t += 2 * lanes) {
      const bool pair = t + lanes < total;
      const int u = pair ? t + lanes : t;
      two(t < first ? p0 + t : p2 + t - first, u < first ? p0 + u : p2 + u - first, pair);
    }
  }
}

template <int KMAX, int LANES, bool IDX>
__device__ __forceinline__ void nearest(const View& g, const int32_t* __restrict__ cell_start,
                                        const float* __restrict__ sx, const float* __restrict__ sy,
                                        const int32_t* __restrict__ sidx, float fx, float fy, int k, double slack_cells,
                                        double (&bk)[KMAX], int32_t (&bi)[KMAX], int sub = 0) {
  // a coordinate that is no number is at no distance: the list keeps its +inf, and its indices (an
  // insertion by comparison rejects a NaN, one by minimum and maximum would take it)
  const double px = IDX || fx == fx ? (double)fx : (double)INFINITY;
  const double py = IDX || fy == fy ? (double)fy : (double)INFINITY;
  const int ncol = g.ncol, nrow = g.nrow;
  const int c0 = clamp_cell((fx - g.minx) * g.inv, ncol);
  const int r0 = clamp_cell((fy - g.miny) * g.inv, nrow);
  const double slack = slack_cells * g.cwd;
  clear<KMAX>(k, bk);
  if constexpr (IDX) clear<KMAX>(k, bk, bi);
  auto two = [&](int p, int p2, bool pair, bool late = false) __attribute__((always_inline)) {
    const float x = sx[p], y = sy[p], x2 = sx[p2], y2 = sy[p2];
    const double dx = (double)x - px, dy = (double)y - py;
    const double ex = (double)x2 - px, ey = (double)y2 - py;
    const double d2 = dx * dx + dy * dy;
    const double e2 = pair ? ex * ex + ey * ey : (double)INFINITY;
    if constexpr (IDX) {
      const int32_t id = sidx[p], id2 = sidx[p2];
      insert<KMAX>(bk, bi, d2, id);
      if (pair) insert<KMAX>(bk, bi, e2, id2);
    } else {
      // far out few candidates enter: a wavefront in which none does goes on
      if (!late || min_f64(d2, e2) < bk[KMAX - 1]) {
        insert<KMAX>(bk, d2);
        insert<KMAX>(bk, e2);
      }
    }
  };
  auto around = [&](int l) __attribute__((always_inline)) {
    return block_rows(g, cell_start, max(r0 - l, 0), min(r0 + l, nrow - 1), max(c0 - l, 0), min(c0 + l, ncol - 1));
  };
  int L = 2;
  Block b = around(2);
  if (b.e4 >= kDenseBlock * k) {
    L = 1;
    b = around(1);
    if constexpr (LANES == 1 && KMAX <= 16) {
      // first the cells within 1.5 times the k-th distance that the density of the 3 x 3 lets expect
      const float r = sqrtf(6.45f * (float)k / (float)b.e4);  // 1.5 sqrt(9 k / (pi points)) cells
      const float u = (fx - g.minx) * g.inv, v = (fy - g.miny) * g.inv;
      const int ca = min(max((int)floorf(u - r), max(c0 - 1, 0)), c0);
      const int cz = max(min((int)floorf(u + r), min(c0 + 1, ncol - 1)), c0);
      const int ra = min(max((int)floorf(v - r), max(r0 - 1, 0)), r0);
      const int rz = max(min((int)floorf(v + r), min(r0 + 1, nrow - 1)), r0);
      walk_block(block_rows(g, cell_start, ra, rz, ca, cz), 0, 1, two);
      const double dout = side_distance(g, px, py, ca, cz, ra, rz) - slack;
      if (dout > 0.0 && bk[KMAX - 1] < dout * dout) return;
      clear<KMAX>(k, bk);
    }
  }
  int count = b.e4;
  walk_block(b, sub, LANES, two);
  const int span = max(ncol, nrow);
  for (;;) {
    if (c0 - L <= 0 && c0 + L >= ncol - 1 && r0 - L <= 0 && r0 + L >= nrow - 1) break;  // the block covers the grid
    const double dout = reach(g, px, py, c0, r0, L, slack);
    // the level that 1.15 times the k-th distance at the block's density reaches, at most twice this one
    int next = count > 0 ? (int)fminf(0.65f * (float)(2 * L + 1) * sqrtf((float)k / (float)count), (float)span) + 1 : span;
    next = min(next, 2 * L);
    if (count >= k) {
      if (dout > 0.0 && k_below<KMAX, LANES>(bk, k, dout * dout)) break;
      // no farther than the level whose sides lie beyond the k-th distance so far (over several
      // lanes, a bound of it)
      const double kth = LANES > 1 ? group_kth<KMAX, LANES>(bk, k) : bk[KMAX - 1];
      if (kth < INFINITY)
        next = min(next, L + 1 + (int)fmin((double)span, fmax(0.0, (sqrt(kth) - dout) * (double)g.inv)));
    }
    next = min(max(next, L + 1), span);
    // LANES > 1: the lanes of a query agree on L, next and count
    int seen = 0;
    walk_growth(g, cell_start, c0, r0, L, next, sub, LANES, [&](int p, int p2, bool pair) __attribute__((always_inline)) {
      seen += pair ? 2 : 1;
      two(p, p2, pair, true);
    });
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) seen += __shfl_xor(seen, o, 64);
    count += seen;
    L = next;
  }
}

// The indices of the k nearest into row, from their squared distances bk.  A second walk, over the
// cells that the k-th distance reaches, lists the candidates no farther (list: KMAX entries, STRIDE
// apart); where these are k and no two are as far, a candidate's place is the number of nearer ones.
// Otherwise a third walk orders equal distances by index.
template <int KMAX, int STRIDE>
__device__ __forceinline__ void collect(const View& g, const int32_t* __restrict__ cell_start,
                                        const float* __restrict__ sx, const float* __restrict__ sy,
                                        const int32_t* __restrict__ sidx, float fx, float fy, int k,
                                        double slack_cells, const double (&bk)[KMAX], int32_t* list,
                                        int32_t* __restrict__ row) {
  const double px = fx, py = fy;
  const double kth = bk[KMAX - 1];
  const int sh = KMAX - k;
  bool tie = false;
#pragma unroll
  for (int s = 1; s < KMAX; ++s) tie |= s > sh && bk[s] == bk[s - 1];
  // the cells of coordinates within the k-th distance; a query that is no number takes all
  const double r = sqrt(kth) * (1.0 + 0x1p-40), inv = 1.0 / g.cwd;
  auto first_cell = [&](double p, float lo, int nc) {
    return (int)fmin(fmax((p - r - (double)lo) * inv - slack_cells, 0.0), (double)(nc - 1));
  };
  auto last_cell = [&](double p, float lo, int nc) {
    return (int)fmax(fmin((p + r - (double)lo) * inv + slack_cells, (double)(nc - 1)), 0.0);
  };
  const int ca = first_cell(px, g.minx, g.ncol), cz = last_cell(px, g.minx, g.ncol);
  const int ra = first_cell(py, g.miny, g.nrow), rz = last_cell(py, g.miny, g.nrow);
  auto dist = [&](int p) __attribute__((always_inline)) {
    const double dx = (double)sx[p] - px, dy = (double)sy[p] - py;
    return dx * dx + dy * dy;
  };
  auto walk = [&](auto&& two) __attribute__((always_inline)) {
    for (int r0 = ra; r0 <= rz; r0 += 5) walk_block(block_rows(g, cell_start, r0, rz, ca, cz), 0, 1, two);
  };
  int cnt = 0;
  walk([&](int p, int p2, bool pair) __attribute__((always_inline)) {
    const double d2 = dist(p), e2 = dist(p2);
    if (d2 <= kth) {
      if (cnt < KMAX) list[cnt * STRIDE] = p;
      ++cnt;
    }
    if (pair && e2 <= kth) {
      if (cnt < KMAX) list[cnt * STRIDE] = p2;
      ++cnt;
    }
  });
  if (!tie && cnt == k) {
#pragma unroll 2
    for (int i = 0; i < k; ++i) {
      const int p = list[i * STRIDE];
      const int32_t id = sidx[p];
      const double d2 = dist(p);
      int at = -sh;
#pragma unroll
      for (int s = 0; s < KMAX; ++s) at += bk[s] < d2 ? 1 : 0;
      row[at] = id;
    }
    return;
  }
  int32_t bi[KMAX];
#pragma unroll
  for (int s = 0; s < KMAX; ++s) bi[s] = INT32_MAX;
  auto place = [&](int p) __attribute__((always_inline)) {
    const double d2 = dist(p);
    if (!(d2 <= kth)) return;
    int32_t id = sidx[p];
#pragma unroll
    for (int s = 0; s < KMAX; ++s) {
      const bool in = (d2 == bk[s]) & (id < bi[s]);
      const int32_t out = bi[s];
      bi[s] = in ? id : out;
      id = in ? out : id;
    }
  };
  walk([&](int p, int p2, bool pair) __attribute__((always_inline)) {
    place(p);
    if (pair) place(p2);
  });
#pragma unroll
  for (int s = 0; s < KMAX; ++s)
    if (s >= sh) row[s - sh] = bi[s];
}

// A copy of part of the grid in LDS: rows [r0, r1], columns [c0, c1] (rows empty when r1 < r0).
// Each of its rows is one contiguous run of the cell-ordered arrays; row r's points sit at
// x[p + off[r - r0]] (and y, idx) for the global position p.  The pointers are generic, so a
// lane reads a segment from LDS or from global memory with the same loads; the pointers stay
// at the arrays' starts and the shift goes into the index, which is in range.
struct Window {
  int r0, r1, c0, c1;
  const int* off;
  const float* x;
  const float* y;
  const int32_t* idx;
};

// The k nearest data points of (fx, fy) by rings of cells: on return slots [KMAX - k, KMAX) of
// (bk, bi) hold their squared distances and indices in ascending (d2, index) order.  WIN: segments
// inside the window are read from LDS.
//
// PAPER = true: the paper's stop rule instead (Section 3.2.4 and its Remark):
// grow the level until the block holds >= k points, search one more level, stop.
// Not exact in general; kept to measure that rule.
template <int KMAX, bool PAPER, bool WIN>
__device__ __forceinline__ void search(const View& g, const int32_t* __restrict__ cell_start,
                                       const float* __restrict__ sx, const float* __restrict__ sy,
                                       const int32_t* __restrict__ sidx, float fx, float fy, int k,
                                       double slack_cells, double (&bk)[KMAX], int32_t (&bi)[KMAX],
                                       const Window* win = nullptr) {
  const double px = fx, py = fy;
  const int ncol = g.ncol, nrow = g.nrow;
  const int c0 = clamp_cell((fx - g.minx) * g.inv, ncol);
  const int r0 = clamp_cell((fy - g.miny) * g.inv, nrow);
  const double slack = slack_cells * g.cwd;
  clear<KMAX>(k, bk, bi);
  int count = 0;
  int final_level = -1;  // PAPER: the level after the one where the block first held >= k points

  for (int L = 0;; ++L) {
    const int cl = c0 - L, cr = c0 + L, rb = r0 - L, rt = r0 + L;
    const int ca = cl > 0 ? cl : 0;
    const int cb = cr < ncol - 1 ? cr : ncol - 1;
    const int ra = rb + 1 > 0 ? rb + 1 : 0;
    const int re = rt - 1 < nrow - 1 ? rt - 1 : nrow - 1;
    const int nside = re >= ra ? re - ra + 1 : 0;
    // ring L as segments: [0] bottom row, [1] top row (each one contiguous run of
    // points in cell order), then the left / right cell of every row in between.
    const int nseg = L == 0 ? 1 : 2 + 2 * nside;
    for (int sg = 0; sg < nseg; ++sg) {
      int row, a, b;
      bool ok;
      if (L == 0) {
        row = r0;
        a = b = c0;
        ok = true;
      } else if (sg < 2) {
        row = sg == 0 ? rb : rt;
        a = ca;
        b = cb;
        ok = sg == 0 ? rb >= 0 : rt < nrow;
      } else {
        const bool right = (sg - 2) & 1;
        row = ra + ((sg - 2) >> 1);
        a = b = right ? cr : cl;
        ok = right ? cr < ncol : cl >= 0;
      }
      if (!ok) continue;
      const int base = row * ncol;
      const int p0 = cell_start[base + a];
      const int p1 = cell_start[base + b + 1];
      count += p1 - p0;
      const float* X = sx;
      const float* Y = sy;
      const int32_t* I = sidx;
      int shift = 0;
      if constexpr (WIN) {
        if (row >= win->r0 && row <= win->r1 && a >= win->c0 && b <= win->c1) {
          shift = win->off[row - win->r0];
          X = win->x;
          Y = win->y;
          I = win->idx;
        }
      }
      for (int p = p0; p < p1; ++p) {
        const double dx = (double)X[p + shift] - px;
        const double dy = (double)Y[p + shift] - py;
        const double d2 = dx * dx + dy * dy;
        const int32_t id = I[p + shift];
        insert<KMAX>(bk, bi, d2, id);
      }
    }
    const bool open_l = cl > 0, open_r = cr < ncol - 1, open_b = rb > 0, open_t = rt < nrow - 1;
    if (!(open_l || open_r || open_b || open_t)) break;  // the block covers the grid
    if constexpr (PAPER) {
      if (final_level < 0 && count >= k) final_level = L + 1;
      if (L == final_level) break;
      continue;
    }
    if (count >= k) {
      const double dout = reach(g, px, py, c0, r0, L, slack);
      if (dout > 0.0 && bk[KMAX - 1] < dout * dout) break;
    }
  }
}

// The k nearest over a group of LANES lanes that searched together (nearest with
// LANES > 1): popped in ascending (d2, index) order, the same order summarise
// uses, so r_obs and d1 are bitwise those of a one-lane search.  Every lane of the
// group returns r_obs and d1; with IDX, idx receives the indices from lane sub 0.
template <int KMAX, int LANES, bool IDX>
__device__ __forceinline__ void merge_lanes(double (&bk)[KMAX], int32_t (&bi)[KMAX], int k, int sub, float& r_obs,
                                            float& d1, int32_t* __restrict__ idx) {
  // move the k live slots to the front: left shift by KMAX - k, one power of two at a time
  const int sh = KMAX - k;
#pragma unroll
  for (int b = 1; b < KMAX; b <<= 1) {
    if (sh & b) {
#pragma unroll
      for (int s = 0; s < KMAX; ++s) {
        bk[s] = s + b < KMAX ? bk[s + b] : INFINITY;
        if constexpr (IDX) bi[s] = s + b < KMAX ? bi[s + b] : INT32_MAX;
      }
    }
  }
  double sum = 0.0;
  d1 = 0.0f;
  for (int it = 0; it < k; ++it) {
    double mv = bk[0];
    int32_t mi = IDX ? bi[0] : sub;  // without indices the first lane of equal heads gives its own
    const int32_t mine = mi;
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) {
      const double ov = __shfl_xor(mv, o, 64);
      const int32_t oi = __shfl_xor(mi, o, 64);
      if (ov < mv || (ov == mv && oi < mi)) {
        mv = ov;
        mi = oi;
      }
    }
    if (bk[0] == mv && mine == mi) {  // this lane's head was the smallest: pop it
#pragma unroll
      for (int s = 0; s < KMAX; ++s) {
        bk[s] = s + 1 < KMAX ? bk[s + 1] : INFINITY;
        if constexpr (IDX) bi[s] = s + 1 < KMAX ? bi[s + 1] : INT32_MAX;
      }
    }
    sum += sqrt(mv);
    if (it == 0) d1 = mv == 0.0 ? 0.0f : fmaxf((float)mv, FLT_MIN);
    if (IDX && sub == 0) idx[it] = mi;
  }
  r_obs = (float)(sum / (double)k);
}

// Eq. 3 from the search result: r_obs = (1/k) sum of the k distances, added in
// ascending order in float64; d1 = the nearest squared distance (0 for a
// coincident query, else at least FLT_MIN so that 1/d1 stays finite).
template <int KMAX, int S = 0>
__device__ __forceinline__ void add_distances(const double (&bk)[KMAX], int k, double& sum) {
  if constexpr (S < KMAX) {
    if (S >= KMAX - k) sum += sqrt(bk[S]);
    add_distances<KMAX, S + 1>(bk, k, sum);
  }
}
template <int KMAX, int S = 0>
__device__ __forceinline__ double slot(const double (&bk)[KMAX], int at) {
  if constexpr (S < KMAX - 1)
    return at == S ? bk[S] : slot<KMAX, S + 1>(bk, at);
  else
    return bk[S];
}
template <int KMAX>
__device__ __forceinline__ void summarise(const double (&bk)[KMAX], int k, float& r_obs, float& d1) {
  double sum = 0.0;
  add_distances<KMAX>(bk, k, sum);
  const double v = slot<KMAX>(bk, KMAX - k);
  d1 = v == 0.0 ? 0.0f : fmaxf((float)v, FLT_MIN);
  r_obs = (float)(sum / (double)k);
}

// A coincident query's value: the mean z of the data points at its exact
// position (the limit of Eq. 1).  Those points share the query's cell, which is
// ordered by index, so the float64 sum runs in index order.  Returns false if
// no data point is at (fx, fy).
__device__ inline bool coincident_mean(const View& g, const int32_t* __restrict__ cell_start,
                                       const float* __restrict__ sx, const float* __restrict__ sy,
                                       const int32_t* __restrict__ sidx, const float* __restrict__ z, float fx,
                                       float fy, float& out) {
  const int col = clamp_cell((fx - g.minx) * g.inv, g.ncol);
  const int row = clamp_cell((fy - g.miny) * g.inv, g.nrow);
  const int c = row * g.ncol + col;
  double s = 0.0;
  int hits = 0;
  for (int p = cell_start[c]; p < cell_start[c + 1]; ++p) {
    if (sx[p] == fx && sy[p] == fy) {
      s += (double)z[sidx[p]];
      ++hits;
    }
  }
  if (hits > 0) out = (float)(s / hits);
  return hits > 0;
}

}  // namespace knn
}  // namespace aidw
