// Collision side of the time step (Algorithm 1's MaxStepSize and Algorithm 3,
// UpdateActiveSet): which surface primitive pairs collide along the straight
// path x -> x_hat, and when.
//
// Broad phase: a linear BVH (Karras 2012) over the swept boxes of the
// surface triangles (point-triangle queries, one thread per surface vertex)
// and of the surface edges (edge-edge queries, one thread per edge, pairs
// (i, j) with i < j).  Boxes are FP32, rounded outward from the FP64
// positions, so the tree test is conservative; every pair it reports is
// tested again exactly in FP64 (swept boxes within delta on every axis) and
// pairs sharing a vertex are skipped.
//
// The queries of both kinds run in one launch and append the pairs that pass
// the exact test to a candidate list; a second launch runs the narrow phase
// with one thread per candidate.  Run by the querying thread itself, the
// narrow phase made a few threads walk through all their candidates one after
// the other while the rest of the chip was idle (a 2,300-edge scene took 515 +
// 212 us per call in the two queries, one of 66,000 edges 645 + 343 us; the
// split form takes 61 + 10 and 78 + 28 us).  A list is bounded (activeset.hip);
// a kind with more candidates than that goes the old way.
//
// Narrow phase: additive CCD (Li, Kaufman and Jiang 2021) in FP64: remove the pair's common translation, bound the rate at which
// the distance can shrink by l_p (largest displacement of a vertex of each
// primitive, summed), and advance by steps that cannot close the gap --
// (1 - s) d0 / l_p first, then 0.9 d / l_p -- until a step lands below s d0
// (collision at the time before that step) or passes t = 1.  After 10^4 steps
// a pair counts as colliding at the time reached; a pair at distance 0 at
// t = 0 collides at 0.  Colliding pairs are appended with their time.
//
// The active-set update then keeps, of the colliding pairs not already
// constrained, those whose time is the earliest of one of their vertices
// (per-vertex atomicMin over the FP64 bit patterns, which order like the
// values for t >= 0; "earliest" up to 1e-9 relative, the times' rounding),
// sorts them into a canonical order, and rebuilds the
// constraint arrays: surviving current PT constraints (gamma >= 0.01, in
// their order), new PT pairs, surviving current EE constraints, new EE pairs.
#include <hipcub/hipcub.hpp>

#include "common.h"

namespace bfal {

namespace {

constexpr int kCcdBlock = 256;
constexpr int kAccdMaxSteps = 10000;
constexpr int kStackDepth = 64;
constexpr int kTraverseBlock = 64; // one wavefront per workgroup
constexpr int kNarrowBlock = 64;   // one wavefront: it ends with its own longest pair

struct d3 {
  double x, y, z;
};
__device__ inline d3 ld3(const double* p, int v) { return {p[3LL * v], p[3LL * v + 1], p[3LL * v + 2]}; }
__device__ inline d3 sub(d3 a, d3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline d3 add(d3 a, d3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ inline d3 mul(d3 a, double s) { return {a.x * s, a.y * s, a.z * s}; }
__device__ inline double dot(d3 a, d3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline double norm2(d3 a) { return dot(a, a); }
__device__ inline double norm(d3 a) { return sqrt(dot(a, a)); }
__device__ inline double clamp01(double t) { return t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t); }
__device__ inline double seg_param(d3 p, d3 u, d3 v) {
  const d3 e = sub(v, u);
  return clamp01(dot(sub(p, u), e) / dot(e, e));
}

// Distance from p to the closed triangle (t0, t1, t2): the interior
// projection when it lies inside, else the nearest of the three edge points.
__device__ inline double pt_dist(d3 p, d3 t0, d3 t1, d3 t2) {
  const d3 e1 = sub(t1, t0), e2 = sub(t2, t0), r = sub(p, t0);
  const double a11 = dot(e1, e1), a12 = dot(e1, e2), a22 = dot(e2, e2);
  const double r1 = dot(e1, r), r2 = dot(e2, r);
  const double det = a11 * a22 - a12 * a12;
  const double u = (a22 * r1 - a12 * r2) / det, v = (a11 * r2 - a12 * r1) / det;
  double best = INFINITY;   // squared: the root of the smallest square is the smallest root
  if (u >= 0.0 && v >= 0.0 && u + v <= 1.0) best = norm2(sub(p, add(t0, add(mul(e1, u), mul(e2, v)))));
  const d3 T[3] = {t0, t1, t2};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const d3 a = T[k], b = T[(k + 1) % 3];
    const double s = seg_param(p, a, b);
    best = fmin(best, norm2(sub(p, add(a, mul(sub(b, a), s)))));
  }
  return sqrt(best);
}

// Distance between segments a0 a1 and b0 b1: the interior stationary point
// when it lies in the unit square, else the best of the four clamped ones.
__device__ inline double ee_dist(d3 a0, d3 a1, d3 b0, d3 b1) {
  const d3 ea = sub(a1, a0), eb = sub(b1, b0), r = sub(a0, b0);
  const double aa = dot(ea, ea), bb = dot(eb, eb), ab = dot(ea, eb);
  const double ar = dot(ea, r), br = dot(eb, r);
  const double det = aa * bb - ab * ab;
  double best = INFINITY;
  if (det > 0.0) {
    const double s = (-ar * bb + ab * br) / det, t = (aa * br - ab * ar) / det;
    if (s >= 0.0 && s <= 1.0 && t >= 0.0 && t <= 1.0) best = norm2(sub(add(a0, mul(ea, s)), add(b0, mul(eb, t))));
  }
  const double cs[4] = {0.0, 1.0, seg_param(b0, a0, a1), seg_param(b1, a0, a1)};
  const double ct[4] = {seg_param(a0, b0, b1), seg_param(a1, b0, b1), 0.0, 1.0};
#pragma unroll
  for (int k = 0; k < 4; ++k) best = fmin(best, norm2(sub(add(a0, mul(ea, cs[k])), add(b0, mul(eb, ct[k])))));
  return sqrt(best);
}

template <bool kEE>
__device__ inline double pair_dist(const d3 X[4]) {
  return kEE ? ee_dist(X[0], X[1], X[2], X[3]) : pt_dist(X[0], X[1], X[2], X[3]);
}

// Additive CCD of one pair along X0 -> X1; returns the collision time, or a
// negative value when the pair does not collide in [0, 1].
template <bool kEE>
__device__ double accd(const d3 X0[4], const d3 X1[4], double s) {
  d3 P[4], X[4];
  d3 m = {0.0, 0.0, 0.0};
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    P[a] = sub(X1[a], X0[a]);
    m = add(m, P[a]);
  }
  m = mul(m, 0.25);
  double la = 0.0, lb = 0.0;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    P[a] = sub(P[a], m);
    X[a] = X0[a];
    const double n = norm(P[a]);
    if (a < (kEE ? 2 : 1)) la = fmax(la, n);
    else lb = fmax(lb, n);
  }
  const double lp = la + lb;
  const double d0 = pair_dist<kEE>(X);
  if (d0 == 0.0) return 0.0;
  if (!(lp > 0.0)) return -1.0;
  const double gap = s * d0;
  double t = 0.0, tl = (1.0 - s) * d0 / lp;
  for (int it = 0; it < kAccdMaxSteps; ++it) {
#pragma unroll
    for (int a = 0; a < 4; ++a) X[a] = add(X[a], mul(P[a], tl));
    const double d = pair_dist<kEE>(X);
    if (it > 0 && d < gap) return t;
    t += tl;
    if (t > 1.0) return -1.0;
    tl = 0.9 * d / lp;
  }
  return t;   // step cap: collision at the time reached
}

// ---------------------------------------------------------------- boxes

struct Box {
  float lo[3], hi[3];
};

__device__ inline void box_of(const double* x, const double* xh, const int* v, int k, double lo[3], double hi[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lo[c] = INFINITY;
    hi[c] = -INFINITY;
  }
  for (int a = 0; a < k; ++a) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double p = x[3LL * v[a] + c], q = xh[3LL * v[a] + c];
      lo[c] = fmin(lo[c], fmin(p, q));
      hi[c] = fmax(hi[c], fmax(p, q));
    }
  }
}

// The trees of a query (triangles and edges) are built side by side: a launch's
// first workgroups take the one, the others the other.  A build is a chain of
// launches of a few microseconds each whatever the tree's size, so two chains
// in one cost what one does (2k leaves: 125 us a chain with the gaps).
struct Trees {
  TreeSide side[2];
  int groups0;   // workgroups of side 0
};
__device__ __forceinline__ const TreeSide& tree_of(const Trees& t, int& block) {
  const bool first = (int)blockIdx.x < t.groups0;
  block = first ? blockIdx.x : blockIdx.x - t.groups0;
  return t.side[first ? 0 : 1];
}

// FP32 swept boxes of the primitives (k vertices each, ids AoS [n][k]), rounded
// outward, and per workgroup the bounds of its boxes.
__global__ void __launch_bounds__(kCcdBlock)
k_prim_boxes(Trees trees, const double* __restrict__ x, const double* __restrict__ xh) {
  int block;
  const TreeSide& T = tree_of(trees, block);
  Box* __restrict__ box = static_cast<Box*>(T.box);
  __shared__ float red[6][kCcdBlock / kWave];
  float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int i = block * kCcdBlock + threadIdx.x; i < T.n; i += T.nparts * kCcdBlock) {
    int v[3];
    for (int a = 0; a < T.k; ++a) v[a] = T.ids[(long long)T.k * i + a];
    double lo[3], hi[3];
    box_of(x, xh, v, T.k, lo, hi);
    Box o;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      o.lo[c] = __double2float_rd(lo[c]);
      o.hi[c] = __double2float_ru(hi[c]);
      b[c] = fminf(b[c], o.lo[c]);
      b[3 + c] = fmaxf(b[3 + c], o.hi[c]);
    }
    box[i] = o;
  }
#pragma unroll
  for (int c = 0; c < 6; ++c) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      const float o = __shfl_xor(b[c], off, kWave);
      b[c] = c < 3 ? fminf(b[c], o) : fmaxf(b[c], o);
    }
    if (threadIdx.x % kWave == 0) red[c][threadIdx.x / kWave] = b[c];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    Box o;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      o.lo[c] = red[c][0];
      o.hi[c] = red[3 + c][0];
#pragma unroll
      for (int w = 1; w < kCcdBlock / kWave; ++w) {
        o.lo[c] = fminf(o.lo[c], red[c][w]);
        o.hi[c] = fmaxf(o.hi[c], red[3 + c][w]);
      }
    }
    static_cast<Box*>(T.part)[block] = o;
  }
}

__device__ inline unsigned int spread10(unsigned int v) {
  v &= 1023u;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// 64-bit sort keys: the 30-bit Morton code of the box centre (in the scene
// bounds) above the primitive index, so equal codes order by index.
__global__ void __launch_bounds__(kCcdBlock) k_morton(Trees trees) {
  int block;
  const TreeSide& T = tree_of(trees, block);
  const int n = T.n, nparts = T.nparts;
  const Box* __restrict__ box = static_cast<const Box*>(T.box);
  const Box* __restrict__ part = static_cast<const Box*>(T.part);
  unsigned long long* __restrict__ key = T.key;
  // the scene's bounds from the partial boxes
  __shared__ float red[6][kCcdBlock / kWave];
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int p = threadIdx.x; p < nparts; p += kCcdBlock)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      lo[c] = fminf(lo[c], part[p].lo[c]);
      hi[c] = fmaxf(hi[c], part[p].hi[c]);
    }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
      lo[c] = fminf(lo[c], __shfl_xor(lo[c], off, kWave));
      hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], off, kWave));
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
      red[c][threadIdx.x / kWave] = lo[c];
      red[3 + c][threadIdx.x / kWave] = hi[c];
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int w = 0; w < kCcdBlock / kWave; ++w) {
      lo[c] = fminf(lo[c], red[c][w]);
      hi[c] = fmaxf(hi[c], red[3 + c][w]);
    }
  const int i = block * kCcdBlock + threadIdx.x;
  if (i >= n) return;
  unsigned int code = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float ext = hi[c] - lo[c];
    const float u = ext > 0.f ? (0.5f * (box[i].lo[c] + box[i].hi[c]) - lo[c]) / ext : 0.f;
    const unsigned int q = (unsigned int)fminf(fmaxf(u * 1024.f, 0.f), 1023.f);
    code |= spread10(q) << (2 - c);
  }
  key[i] = ((unsigned long long)code << 32) | (unsigned int)i;
}

// ------------------------------------------------------------ tree build

__device__ inline int common_prefix(const unsigned long long* key, int n, int i, int j) {
  if (j < 0 || j >= n) return -1;
  return __clzll(key[i] ^ key[j]);   // keys are unique (index in the low bits)
}

// Karras' construction: internal node i (0 <= i < n - 1) covers the key range
// found by a binary search on the common-prefix length; children are internal
// nodes or leaves (leaf k is node n - 1 + k).
// The same launch writes level 0 of the table of node boxes: the primitive
// boxes in key order.
__global__ void __launch_bounds__(kCcdBlock) k_karras(Trees trees) {
  int block;
  const TreeSide& T = tree_of(trees, block);
  const int n = T.n;
  const unsigned long long* __restrict__ key = T.sorted;
  int2* __restrict__ child = T.child;
  int2* __restrict__ range = T.range;
  const int i = block * kCcdBlock + threadIdx.x;
  if (i < n) static_cast<Box*>(T.table)[i] = static_cast<const Box*>(T.box)[(int)(key[i] & 0xffffffffu)];
  if (i >= n - 1) return;
  const int d = common_prefix(key, n, i, i + 1) - common_prefix(key, n, i, i - 1) >= 0 ? 1 : -1;
  const int dmin = common_prefix(key, n, i, i - d);
  int lmax = 2;
  while (common_prefix(key, n, i, i + lmax * d) > dmin) lmax *= 2;
  int l = 0;
  for (int t = lmax / 2; t >= 1; t /= 2)
    if (common_prefix(key, n, i, i + (l + t) * d) > dmin) l += t;
  const int j = i + l * d;
  const int dnode = common_prefix(key, n, i, j);
  int s = 0;
  for (int t = (l + 1) / 2;; t = (t + 1) / 2) {
    if (common_prefix(key, n, i, i + (s + t) * d) > dnode) s += t;
    if (t == 1) break;
  }
  const int g = i + s * d + (d < 0 ? -1 : 0);
  const int left = (min(i, j) == g) ? (n - 1 + g) : g;
  const int right = (max(i, j) == g + 1) ? (n - 1 + g + 1) : g + 1;
  child[i] = make_int2(left, right);
  range[i] = make_int2(min(i, j), max(i, j));
}

// Node boxes without atomics: an internal node covers the contiguous range
// [a, b] of sorted leaves, so its box is the union of two overlapping runs of
// 2^m leaves (2^m <= b - a + 1 < 2^(m+1)), read from a sparse table whose
// level k holds the union of the 2^k leaves starting at each position.
__device__ inline Box box_union(const Box& a, const Box& b) {
  Box u;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    u.lo[q] = fminf(a.lo[q], b.lo[q]);
    u.hi[q] = fmaxf(a.hi[q], b.hi[q]);
  }
  return u;
}

// Levels k to k + kTableStep - 1 (those there are) from level k - 1, whose
// entries span h = 2^(k-1) leaves: entry i of level k + j spans 2^(j+1) of them
// and is there if i + 2^(j+1) h <= n.  A level alone is a few microseconds of
// launch for a few hundred nanoseconds of work: four in one launch read twice
// the boxes, out of the cache, and wait once (the levels of a tree of 2k
// leaves 23 -> 11 us, of 44k to 66k 37 -> 17, gaps between launches not counted).
constexpr int kTableStep = 4;
__global__ void __launch_bounds__(kCcdBlock)
k_sparse_levels(Trees trees, int k) {
  int block;
  const TreeSide& T = tree_of(trees, block);
  const int n = T.n, h = 1 << (k - 1), levels = T.levels - k;
  const Box* __restrict__ prev = static_cast<const Box*>(T.table) + (long long)(k - 1) * n;
  Box* __restrict__ next = static_cast<Box*>(T.table) + (long long)k * n;
  const int i = block * kCcdBlock + threadIdx.x;
  if (i + 2LL * h > n) return;
  Box b[1 << kTableStep];
#pragma unroll
  for (int j = 0; j < 1 << kTableStep; ++j) b[j] = prev[min((long long)i + (long long)j * h, (long long)n - h)];
#pragma unroll
  for (int l = 0; l < kTableStep; ++l) {
#pragma unroll
    for (int j = 0; j < 1 << (kTableStep - 1 - l); ++j) b[j] = box_union(b[2 * j], b[2 * j + 1]);
    if (l < levels && i + ((2LL << l) * h) <= n) next[(long long)l * n + i] = b[0];
  }
}

// An internal node as a query reads it: its children with their boxes, so that
// one load decides about both and a subtree that is missed is never visited.
struct alignas(64) Node {   // read as four float4
  Box left, right;
  int2 child;
  int pad[2];
};
static_assert(sizeof(Box) == 24 && sizeof(Node) == 64, "two boxes, then the children at byte 48");

__device__ inline Box box_of_node(int v, int n, const int2* __restrict__ range, const Box* __restrict__ table) {
  if (v >= n - 1) return table[v - (n - 1)];
  const int2 r = range[v];
  const int m = 31 - __clz(r.y - r.x + 1);
  const Box* lv = table + (long long)m * n;
  return box_union(lv[r.x], lv[r.y - (1 << m) + 1]);
}

__global__ void __launch_bounds__(kCcdBlock) k_nodes(Trees trees) {
  int block;
  const TreeSide& T = tree_of(trees, block);
  const int n = T.n;
  const int2* __restrict__ child = T.child;
  const int2* __restrict__ range = T.range;
  const Box* __restrict__ table = static_cast<const Box*>(T.table);
  Node* __restrict__ node = static_cast<Node*>(T.node);
  const int i = block * kCcdBlock + threadIdx.x;
  if (i >= n - 1) return;
  Node o;
  o.child = child[i];
  o.left = box_of_node(o.child.x, n, range, table);
  o.right = box_of_node(o.child.y, n, range, table);
  o.pad[0] = o.pad[1] = 0;
  node[i] = o;
}

// ------------------------------------------------------------ queries

// (all six comparisons: a short-circuit would wait for one load after another)
__device__ inline bool overlap(float lx, float ly, float lz, float hx, float hy, float hz, const float lo[3],
                               const float hi[3]) {
  return (lx <= hi[0]) & (lo[0] <= hx) & (ly <= hi[1]) & (lo[1] <= hy) & (lz <= hi[2]) & (lo[2] <= hz);
}

// The oracle's exact test: FP64 swept boxes within delta on every axis.
__device__ inline bool near_exact(const double alo[3], const double ahi[3], const double blo[3], const double bhi[3],
                                  double delta) {
  bool ok = true;
#pragma unroll
  for (int c = 0; c < 3; ++c) ok = ok && (alo[c] - delta <= bhi[c]) && (blo[c] - delta <= ahi[c]);
  return ok;
}

// One thread per query primitive (a surface vertex for PT, an edge for EE), one
// wavefront per workgroup, in lockstep: every thread walks the tree of the
// other kind and leaves the leaves it meets in an LDS list (the stack is in
// LDS too: indexed private arrays live in memory); when the list fills, and at
// the end, the wavefront takes it through the exact test, kLeafUnroll times 64
// pairs at a time, and appends those that pass with one atomic.  Testing
// leaves where they are met would make all lanes wait for each one's loads (20
// to 30 leaves per query, most of them neighbours that share a vertex), and an
// atomic per 64 pairs is a round trip each: 154 and 80 us at 2,300 edges,
// against 61 us.
constexpr int kLeafCap = 2048;
constexpr int kLeafUnroll = 4;
static_assert(kTraverseBlock == kWave, "the wavefront works in lockstep");

struct TraverseLds {
  int stack[kStackDepth * kTraverseBlock];
  int leaf[kLeafCap];               // leaf in key order; after the test the tree primitive
  unsigned char lane[kLeafCap];     // whose query met it
  double lo[3][kTraverseBlock], hi[3][kTraverseBlock];   // the queries' swept boxes
  int ids[2][kTraverseBlock];       // and vertices
};

// The narrow phase of one candidate.
template <bool kEE>
__device__ __forceinline__ void narrow(const QuerySide& q, int2 pr, const double* __restrict__ x,
                                       const double* __restrict__ xh, double s, int* __restrict__ count) {
  int ids[4];
  if (kEE) {
    ids[0] = q.qids[2LL * pr.x];
    ids[1] = q.qids[2LL * pr.x + 1];
    ids[2] = q.tids[2LL * pr.y];
    ids[3] = q.tids[2LL * pr.y + 1];
  } else {
    ids[0] = q.qids[pr.x];
    ids[1] = q.tids[3LL * pr.y];
    ids[2] = q.tids[3LL * pr.y + 1];
    ids[3] = q.tids[3LL * pr.y + 2];
  }
  d3 X0[4], X1[4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    X0[a] = ld3(x, ids[a]);
    X1[a] = ld3(xh, ids[a]);
  }
  const double t = accd<kEE>(X0, X1, s);
  if (t >= 0.0) {
    const int slot = atomicAdd(count, 1);
    if (slot < q.cap) {
      q.pairs[slot] = pr;
      q.toc[slot] = t;
    }
  }
}

template <bool kEE, bool kDirect>
__device__ __forceinline__ void test_leaves(int n, int i0, const QuerySide& q, const double* __restrict__ x,
                                            const double* __restrict__ xh, double delta, double s,
                                            int* __restrict__ count, TraverseLds& L) {
  constexpr int kq = kEE ? 2 : 1;
  constexpr int kt = kEE ? 2 : 3;
  const int lane = threadIdx.x;
  const unsigned long long below = (1ull << lane) - 1ull;
  int kept = 0;
  __syncthreads();
  for (int k0 = 0; k0 < n; k0 += kLeafUnroll * kWave) {
    int j[kLeafUnroll], tv[kLeafUnroll][kt], ql[kLeafUnroll];
    bool ok[kLeafUnroll];
    double tlo[kLeafUnroll][3], thi[kLeafUnroll][3];
#pragma unroll
    for (int u = 0; u < kLeafUnroll; ++u) {
      const int k = min(k0 + u * kWave + lane, n - 1);
      ql[u] = L.lane[k];
      j[u] = (int)(q.key[L.leaf[k]] & 0xffffffffu);
    }
#pragma unroll
    for (int u = 0; u < kLeafUnroll; ++u)
#pragma unroll
      for (int a = 0; a < kt; ++a) tv[u][a] = q.tids[(long long)kt * j[u] + a];
#pragma unroll
    for (int u = 0; u < kLeafUnroll; ++u) box_of(x, xh, tv[u], kt, tlo[u], thi[u]);
#pragma unroll
    for (int u = 0; u < kLeafUnroll; ++u) {
      double qlo[3], qhi[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        qlo[c] = L.lo[c][ql[u]];
        qhi[c] = L.hi[c][ql[u]];
      }
      ok[u] = k0 + u * kWave + lane < n && !(kEE && j[u] <= i0 + ql[u]) &&
              near_exact(qlo, qhi, tlo[u], thi[u], delta);
#pragma unroll
      for (int a = 0; a < kq; ++a)
#pragma unroll
        for (int b = 0; b < kt; ++b) ok[u] = ok[u] && L.ids[a][ql[u]] != tv[u][b];
    }
    // keep the survivors at the front of the list (every entry of this round has been read)
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kLeafUnroll; ++u) {
      const unsigned long long mask = __ballot(ok[u]);
      if (ok[u]) {
        const int p = kept + __popcll(mask & below);
        L.leaf[p] = j[u];
        L.lane[p] = (unsigned char)ql[u];
      }
      kept += __popcll(mask);
    }
    __syncthreads();
  }
  if (kept == 0) return;
  unsigned long long base = 0;
  if (lane == 0)
    base = atomicAdd(reinterpret_cast<unsigned long long*>(count + 2), (unsigned long long)kept);
  base = __shfl(base, 0, kWave);
  if (kDirect && !q.cand) {
    for (int k = lane; k < kept; k += kWave) narrow<kEE>(q, make_int2(i0 + L.lane[k], L.leaf[k]), x, xh, s, count);
  } else {
    for (int k = lane; k < kept; k += kWave)
      if (base + k < (unsigned long long)q.cand_cap) q.cand[base + k] = make_int2(i0 + L.lane[k], L.leaf[k]);
  }
  __syncthreads();
}

template <bool kEE, bool kDirect>
__device__ __forceinline__ void traverse(int i0, const QuerySide& q, const double* __restrict__ x,
                                         const double* __restrict__ xh, double delta, double s,
                                         int* __restrict__ count, TraverseLds& L) {
  constexpr int kq = kEE ? 2 : 1;
  if (q.nt <= 0) return;
  const Node* __restrict__ node = static_cast<const Node*>(q.node);
  const int lane = threadIdx.x, i = i0 + lane;
  const unsigned long long below = (1ull << lane) - 1ull;
  const bool mine = i < q.nq;
  int qv[kq];
#pragma unroll
  for (int a = 0; a < kq; ++a) {
    qv[a] = q.qids[(long long)kq * min(i, q.nq - 1) + a];
    L.ids[a][lane] = qv[a];
  }
  double qlo[3], qhi[3];
  box_of(x, xh, qv, kq, qlo, qhi);
  float flo[3], fhi[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    L.lo[c][lane] = qlo[c];
    L.hi[c][lane] = qhi[c];
    flo[c] = __double2float_rd(qlo[c] - delta);
    fhi[c] = __double2float_ru(qhi[c] + delta);
  }
  int* stack = L.stack + lane;
  int sp = 0, n = 0;
  bool overflow = false;
  auto meet = [&](bool is, int k) {   // leaf k in key order
    const unsigned long long mask = __ballot(is);
    if (is) {
      const int p = n + __popcll(mask & below);
      L.leaf[p] = k;
      L.lane[p] = (unsigned char)lane;
    }
    n += __popcll(mask);
  };
  int v = mine ? 0 : -1;
  if (q.nt == 1) {
    meet(mine, 0);
    v = -1;
  }
  while (__any(v >= 0)) {
    const float4* nd = reinterpret_cast<const float4*>(node + max(v, 0));
    const float4 n0 = nd[0], n1 = nd[1], n2 = nd[2], n3 = nd[3];
    const int cl = __float_as_int(n3.x), cr = __float_as_int(n3.y);
    const bool hl = (v >= 0) & overlap(n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, flo, fhi);
    const bool hr = (v >= 0) & overlap(n1.z, n1.w, n2.x, n2.y, n2.z, n2.w, flo, fhi);
    const bool ll = hl & (cl >= q.nt - 1), lr = hr & (cr >= q.nt - 1);
    if (n > kLeafCap - 2 * kWave) {
      test_leaves<kEE, kDirect>(n, i0, q, x, xh, delta, s, count, L);
      n = 0;
    }
    meet(ll, cl - (q.nt - 1));
    meet(lr, cr - (q.nt - 1));
    const int a = hl & !ll ? cl : -1, b = hr & !lr ? cr : -1;
    if ((a >= 0) & (b >= 0)) {
      if (sp < kStackDepth) stack[kTraverseBlock * sp++] = b;
      else overflow = true;   // cannot happen for trees of depth < 63; reported, never dropped silently
    }
    v = a >= 0 ? a : b >= 0 ? b : sp > 0 && v >= 0 ? stack[kTraverseBlock * --sp] : -1;
  }
  if (overflow) count[1] = 1;
  if (n) test_leaves<kEE, kDirect>(n, i0, q, x, xh, delta, s, count, L);
}

// kDirect: a kind may come without a list; its candidates then go through the
// narrow phase here, a wavefront's 64 at a time (activeset.hip: when, and what
// it costs).  A kernel of its own, as the others need not hold its registers.
template <bool kDirect>
__global__ void __launch_bounds__(kTraverseBlock)
k_traverse(QuerySide pt, QuerySide ee, int pt_groups, const double* __restrict__ x, const double* __restrict__ xh,
           double delta, double s, int* __restrict__ count) {
  __shared__ TraverseLds L;
  const int b = blockIdx.x;
  if (b < pt_groups)
    traverse<false, kDirect>(b * kTraverseBlock, pt, x, xh, delta, s, count, L);
  else
    traverse<true, kDirect>((b - pt_groups) * kTraverseBlock, ee, x, xh, delta, s, count + 8, L);
}

// The narrow phase, one thread per candidate of either kind (grid-stride over
// the lists, whose lengths only the device knows; a kind without one has none).
template <bool kEE>
__device__ __forceinline__ void narrow_all(const QuerySide& q, int block, int blocks, const double* __restrict__ x,
                                           const double* __restrict__ xh, double s, int* __restrict__ count) {
  const long long total = *reinterpret_cast<const unsigned long long*>(count + 2);
  const long long n = total < q.cand_cap ? total : q.cand_cap;
  for (long long k = (long long)block * kNarrowBlock + threadIdx.x; k < n; k += (long long)blocks * kNarrowBlock)
    narrow<kEE>(q, q.cand[k], x, xh, s, count);
}

__global__ void __launch_bounds__(kNarrowBlock)
k_narrow(QuerySide pt, QuerySide ee, int pt_groups, const double* __restrict__ x, const double* __restrict__ xh,
         double s, int* __restrict__ count) {
  const int b = blockIdx.x;
  if (b < pt_groups)
    narrow_all<false>(pt, b, pt_groups, x, xh, s, count);
  else
    narrow_all<true>(ee, b - pt_groups, gridDim.x - pt_groups, x, xh, s, count + 8);
}

// Canonical 64-bit order of a colliding pair: query index above tree index
// (PT: surface-vertex position, which follows the vertex id, then triangle;
// EE: edge i < edge j).
__global__ void k_pair_keys(int n, const int2* __restrict__ pairs, unsigned long long* __restrict__ key,
                            int* __restrict__ idx) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i >= n) return;
  key[i] = ((unsigned long long)(unsigned int)pairs[i].x << 32) | (unsigned int)pairs[i].y;
  idx[i] = i;
}

// ------------------------------------------------------------ active set

__device__ inline void sort3(int& a, int& b, int& c) {
  if (a > b) { const int t = a; a = b; b = t; }
  if (b > c) { const int t = b; b = c; c = t; }
  if (a > b) { const int t = a; a = b; b = t; }
}

// Canonical 4-int key of a constraint: PT (p, sorted triangle); EE (sorted
// edges, the smaller edge first).
__device__ inline int4 canon(int4 t, bool ee) {
  if (!ee) {
    sort3(t.y, t.z, t.w);
    return t;
  }
  int a0 = min(t.x, t.y), a1 = max(t.x, t.y), b0 = min(t.z, t.w), b1 = max(t.z, t.w);
  if (a0 > b0 || (a0 == b0 && a1 > b1)) {
    const int u0 = a0, u1 = a1;
    a0 = b0; a1 = b1; b0 = u0; b1 = u1;
  }
  return make_int4(a0, a1, b0, b1);
}

__device__ inline unsigned long long hash4(int4 k, bool ee) {
  unsigned long long h = ee ? 0x9E3779B97F4A7C15ull : 0xC2B2AE3D27D4EB4Full;
  const int v[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    h ^= (unsigned long long)(unsigned int)v[a] + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
    h *= 0xFF51AFD7ED558CCDull;
  }
  return h ^ (h >> 33);
}

// Open-addressing set of the current constraints (slot value = constraint index).
__global__ void k_hash_insert(int n_c, int n_pt, const int4* __restrict__ ids, int* __restrict__ table,
                              unsigned int mask) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i >= n_c) return;
  const bool ee = i >= n_pt;
  unsigned int h = (unsigned int)hash4(canon(ids[i], ee), ee) & mask;
  while (atomicCAS(&table[h], -1, i) != -1) h = (h + 1) & mask;
}

__device__ inline bool hash_find(int4 key, bool ee, int n_pt, const int4* __restrict__ ids,
                                 const int* __restrict__ table, unsigned int mask) {
  unsigned int h = (unsigned int)hash4(key, ee) & mask;
  while (true) {
    const int c = table[h];
    if (c < 0) return false;
    if ((c >= n_pt) == ee) {
      const int4 k = canon(ids[c], ee);
      if (k.x == key.x && k.y == key.y && k.z == key.z && k.w == key.w) return true;
    }
    h = (h + 1) & mask;
  }
}

__device__ inline int4 pair_ids(bool ee, int2 pr, const int* __restrict__ qids, const int* __restrict__ tids) {
  if (ee) return make_int4(qids[2LL * pr.x], qids[2LL * pr.x + 1], tids[2LL * pr.y], tids[2LL * pr.y + 1]);
  return make_int4(qids[pr.x], tids[3LL * pr.y], tids[3LL * pr.y + 1], tids[3LL * pr.y + 2]);
}

// New colliding pairs (sorted order): not in the current set; their times
// lower the per-vertex earliest time.
// An edge pair (near-)parallel at x: its distance gradient is not unique and
// the linearization rejects it, so it cannot enter the active set.
__device__ inline bool ee_parallel(const double* __restrict__ x, int4 id) {
  const d3 ea = sub(ld3(x, id.y), ld3(x, id.x)), eb = sub(ld3(x, id.w), ld3(x, id.z));
  const d3 cr = {ea.y * eb.z - ea.z * eb.y, ea.z * eb.x - ea.x * eb.z, ea.x * eb.y - ea.y * eb.x};
  return dot(cr, cr) < 1e-8 * dot(ea, ea) * dot(eb, eb);
}

__global__ void k_new_and_tv(int n, bool ee, const int* __restrict__ order, const int2* __restrict__ pairs,
                             const double* __restrict__ toc, const int* __restrict__ qids,
                             const int* __restrict__ tids, int n_pt, const int4* __restrict__ cids,
                             const int* __restrict__ table, unsigned int mask, const double* __restrict__ x,
                             int* __restrict__ is_new, unsigned long long* __restrict__ tv) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i >= n) return;
  const int o = order[i];
  const int4 id = pair_ids(ee, pairs[o], qids, tids);
  const bool found = (ee && ee_parallel(x, id)) ||
                     (table != nullptr && hash_find(canon(id, ee), ee, n_pt, cids, table, mask));
  is_new[i] = found ? 0 : 1;
  if (!found) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(toc[o]);
    atomicMin(&tv[id.x], b);
    atomicMin(&tv[id.y], b);
    atomicMin(&tv[id.z], b);
    atomicMin(&tv[id.w], b);
  }
}

__global__ void k_keep_new(int n, bool ee, const int* __restrict__ order, const int2* __restrict__ pairs,
                           const double* __restrict__ toc, const int* __restrict__ qids, const int* __restrict__ tids,
                           const unsigned long long* __restrict__ tv, int* __restrict__ keep) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i >= n) return;
  if (!keep[i]) return;   // holds is_new on entry
  const int o = order[i];
  const int4 id = pair_ids(ee, pairs[o], qids, tids);
  // the earliest time of a vertex, up to the times' own rounding
  const double t = toc[o];
  auto earliest = [&](int v) { return t <= __longlong_as_double((long long)tv[v]) * (1.0 + 1e-9); };
  keep[i] = (earliest(id.x) || earliest(id.y) || earliest(id.z) || earliest(id.w)) ? 1 : 0;
}

__global__ void k_keep_current(int lo, int hi, const double* __restrict__ gam, double gmin, int* __restrict__ keep) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (lo + i < hi) keep[i] = gam[lo + i] >= gmin ? 1 : 0;
}

// Scatter the surviving current constraints of [lo, hi) to out + pos.
__global__ void k_scatter_current(int lo, int hi, const int* __restrict__ keep, const int* __restrict__ pos,
                                  int base, const int4* __restrict__ ids, const double* __restrict__ lam,
                                  const double* __restrict__ gam, int4* __restrict__ oids, double* __restrict__ olam,
                                  double* __restrict__ ogam) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (lo + i >= hi || !keep[i]) return;
  const int o = base + pos[i];
  oids[o] = ids[lo + i];
  olam[o] = lam[lo + i];
  ogam[o] = gam[lo + i];
}

__global__ void k_scatter_new(int n, bool ee, const int* __restrict__ keep, const int* __restrict__ pos, int base,
                              const int* __restrict__ order, const int2* __restrict__ pairs,
                              const int* __restrict__ qids, const int* __restrict__ tids, int4* __restrict__ oids,
                              double* __restrict__ olam, double* __restrict__ ogam) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i >= n || !keep[i]) return;
  const int o = base + pos[i];
  oids[o] = pair_ids(ee, pairs[order[i]], qids, tids);
  olam[o] = 0.0;
  ogam[o] = 1.0;
}

__global__ void k_pair_rows(int n, bool ee, const int2* __restrict__ pairs, const int* __restrict__ qids,
                            const int* __restrict__ tids, int4* __restrict__ rows) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i < n) rows[i] = pair_ids(ee, pairs[i], qids, tids);
}

__global__ void k_fill_u64(unsigned long long* a, unsigned long long v, int n) {
  const int i = blockIdx.x * kCcdBlock + threadIdx.x;
  if (i < n) a[i] = v;
}

// ------------------------------------------------------------ step size

// Per workgroup the smallest collision time of a pair list.
__global__ void k_min_toc(int n, const double* __restrict__ toc, double* __restrict__ part) {
  __shared__ double red[kCcdBlock];
  double m = 1.0;
  for (int i = blockIdx.x * kCcdBlock + threadIdx.x; i < n; i += gridDim.x * kCcdBlock) m = fmin(m, toc[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int off = kCcdBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__device__ inline double det3(d3 a, d3 b, d3 c) {   // det of the matrix with columns a, b, c
  return a.x * (b.y * c.z - b.z * c.y) - b.x * (a.y * c.z - a.z * c.y) + c.x * (a.y * b.z - a.z * b.y);
}

// Per tet the first t in (0, 1] where det D_s(t) / det D_s(0) falls to s (1 if
// none), for either orientation of the tet: the cubic's coefficients by
// interpolation at t = 0, 1/3, 2/3, 1, taken times the sign of det D_s(0); its
// derivative's roots split [0, 1] into monotone pieces, the first piece whose
// end falls to the level s |det D_s(0)| is bisected (60 halvings, the lower end
// kept).
__global__ void k_inversion_bound(int T, const int4* __restrict__ tets, const double* __restrict__ x,
                                  const double* __restrict__ xh, double s, double* __restrict__ part) {
  __shared__ double red[kCcdBlock];
  const int e = blockIdx.x * kCcdBlock + threadIdx.x;
  double out = 1.0;
  if (e < T) {
    const int4 t = tets[e];
    const d3 p0 = ld3(x, t.x), p1 = ld3(x, t.y), p2 = ld3(x, t.z), p3 = ld3(x, t.w);
    const d3 q0 = ld3(xh, t.x), q1 = ld3(xh, t.y), q2 = ld3(xh, t.z), q3 = ld3(xh, t.w);
    const d3 a0 = sub(p1, p0), b0 = sub(p2, p0), c0 = sub(p3, p0);
    const d3 da = sub(sub(q1, q0), a0), db = sub(sub(q2, q0), b0), dc = sub(sub(q3, q0), c0);
    auto J = [&](double tt) { return det3(add(a0, mul(da, tt)), add(b0, mul(db, tt)), add(c0, mul(dc, tt))); };
    const double f0 = J(0.0), f1 = J(1.0 / 3.0), f2 = J(2.0 / 3.0), f3 = J(1.0);
    // Newton form at 0, 1/3, 2/3, 1 (h = 1/3), expanded to the monomial coefficients
    const double h = 1.0 / 3.0;
    const double d1a = (f1 - f0) / h, d1b = (f2 - f1) / h, d1c = (f3 - f2) / h;
    const double d2a = (d1b - d1a) / (2 * h), d2b = (d1c - d1b) / (2 * h);
    const double d3v = (d2b - d2a) / (3 * h);
    // p(t) = f0 + d1a t + d2a t (t - h) + d3v t (t - h)(t - 2h)
    const double sg = f0 < 0.0 ? -1.0 : 1.0;
    const double c3 = sg * d3v;
    const double c2 = sg * (d2a - 3 * h * d3v);
    const double c1 = sg * (d1a - h * d2a + 2 * h * h * d3v);
    const double c0v = sg * f0;
    const double level = s * c0v;
    auto F = [&](double tt) { return ((c3 * tt + c2) * tt + c1) * tt + c0v - level; };
    double knots[4];
    int nk = 0;
    knots[nk++] = 0.0;
    const double A = 3 * c3, B = 2 * c2, C = c1;
    double r[2];
    int nr = 0;
    if (A != 0.0) {
      const double disc = B * B - 4 * A * C;
      if (disc >= 0.0) {
        const double sq = sqrt(disc);
        r[0] = (-B - sq) / (2 * A);
        r[1] = (-B + sq) / (2 * A);
        if (r[0] > r[1]) { const double u = r[0]; r[0] = r[1]; r[1] = u; }
        nr = 2;
      }
    } else if (B != 0.0) {
      r[0] = -C / B;
      nr = 1;
    }
    for (int k = 0; k < nr; ++k)
      if (r[k] > 0.0 && r[k] < 1.0) knots[nk++] = r[k];
    knots[nk++] = 1.0;
    for (int k = 0; k + 1 < nk; ++k) {
      double lo = knots[k], hi = knots[k + 1];
      if (F(hi) <= 0.0) {
        for (int it = 0; it < 60; ++it) {
          const double mid = 0.5 * (lo + hi);
          if (F(mid) > 0.0) lo = mid;
          else hi = mid;
        }
        out = lo;
        break;
      }
    }
  }
  red[threadIdx.x] = out;
  __syncthreads();
  for (int off = kCcdBlock / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

}  // namespace

// ---------------------------------------------------------------- launchers

size_t ccd_sort_tmp_bytes(int n) {
  size_t bytes = 0;
  (void)hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, (unsigned long long*)nullptr, (unsigned long long*)nullptr,
                                     (int*)nullptr, (int*)nullptr, n, 0, 64, (hipStream_t)0);
  return bytes;
}

hipError_t ccd_sort_pairs(void* tmp, size_t tmp_bytes, const unsigned long long* kin, unsigned long long* kout,
                          const int* vin, int* vout, int n, hipStream_t s) {
  return hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, kin, kout, vin, vout, n, 0, 64, s);
}

// The keys' order is that of their 30-bit codes: equal codes keep the order they
// come in, which is that of the indices below them (the sort is stable).
constexpr int kKeyBit0 = 32, kKeyBit1 = 62;

size_t ccd_sort_keys_tmp_bytes(int n) {
  size_t bytes = 0;
  (void)hipcub::DeviceRadixSort::SortKeys(nullptr, bytes, (unsigned long long*)nullptr, (unsigned long long*)nullptr, n,
                                          kKeyBit0, kKeyBit1, (hipStream_t)0);
  return bytes;
}

hipError_t ccd_sort_keys(void* tmp, size_t tmp_bytes, const unsigned long long* kin, unsigned long long* kout, int n,
                         hipStream_t s) {
  return hipcub::DeviceRadixSort::SortKeys(tmp, tmp_bytes, kin, kout, n, kKeyBit0, kKeyBit1, s);
}

// (four workgroups per compute unit, and no more partial boxes than k_morton reads at once in a few loads)
int ccd_bounds_parts(int n) { return std::min(div_up(n, kCcdBlock), 1024); }

int ccd_table_levels(int n) {
  int L = 1;
  while ((2LL << (L - 1)) <= n) ++L;   // levels 0 .. L-1 with 2^(L-1) <= n
  return L;
}

namespace {
// Workgroups of both sides for as many threads each.
unsigned split(Trees& t, long long n0, long long n1) {
  t.groups0 = div_up(std::max(n0, 0LL), kCcdBlock);
  return (unsigned)(t.groups0 + div_up(std::max(n1, 0LL), kCcdBlock));
}
}  // namespace

void launch_tree_keys(const TreeSide& a, const TreeSide& b, const double* x, const double* xh, hipStream_t s) {
  Trees t{{a, b}, a.n > 0 ? a.nparts : 0};
  const unsigned g = t.groups0 + (b.n > 0 ? b.nparts : 0);
  if (!g) return;
  hipLaunchKernelGGL(k_prim_boxes, dim3(g), dim3(kCcdBlock), 0, s, t, x, xh);
  const unsigned gm = split(t, a.n, b.n);
  hipLaunchKernelGGL(k_morton, dim3(gm), dim3(kCcdBlock), 0, s, t);
}

void launch_build_trees(const TreeSide& a, const TreeSide& b, hipStream_t s) {
  Trees t{{a, b}, 0};
  unsigned g = split(t, a.n, b.n);
  if (!g) return;
  hipLaunchKernelGGL(k_karras, dim3(g), dim3(kCcdBlock), 0, s, t);
  for (int k = 1; k < std::max(a.levels, b.levels); k += kTableStep) {
    const long long h2 = 2LL << (k - 1);
    g = split(t, a.n - h2 + 1, b.n - h2 + 1);
    if (g) hipLaunchKernelGGL(k_sparse_levels, dim3(g), dim3(kCcdBlock), 0, s, t, k);
  }
  g = split(t, a.n - 1, b.n - 1);
  if (g) hipLaunchKernelGGL(k_nodes, dim3(g), dim3(kCcdBlock), 0, s, t);
}

size_t ccd_node_bytes(int n) { return sizeof(Node) * std::max(n - 1, 1); }

void launch_queries(const QuerySide& pt, const QuerySide& ee, bool do_pt, bool do_ee, const double* x, const double* xh,
                    double delta, double sep, int* count, hipStream_t s) {
  const int gp = do_pt ? div_up(pt.nq, kTraverseBlock) : 0, ge = do_ee ? div_up(ee.nq, kTraverseBlock) : 0;
  const bool direct = (do_pt && !pt.cand) || (do_ee && !ee.cand);
  if (gp + ge)
    hipLaunchKernelGGL(direct ? k_traverse<true> : k_traverse<false>, dim3(gp + ge), dim3(kTraverseBlock), 0, s, pt, ee,
                       gp, x, xh, delta, sep, count);
  // 16 wavefronts per compute unit and list: the lists are walked with a stride
  const int np = gp ? 256 * 16 : 0, ne = ge ? 256 * 16 : 0;
  if (np + ne) hipLaunchKernelGGL(k_narrow, dim3(np + ne), dim3(kNarrowBlock), 0, s, pt, ee, np, x, xh, sep, count);
}

void launch_pair_keys(int n, const int2* pairs, unsigned long long* key, int* idx, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_pair_keys, dim3(div_up(n, kCcdBlock)), dim3(kCcdBlock), 0, s, n, pairs, key, idx);
}

void launch_hash_insert(int n_c, int n_pt, const int4* ids, int* table, unsigned int mask, hipStream_t s) {
  if (n_c > 0)
    hipLaunchKernelGGL(k_hash_insert, dim3(div_up(n_c, kCcdBlock)), dim3(kCcdBlock), 0, s, n_c, n_pt, ids, table,
                       mask);
}

void launch_pair_rows(int n, bool ee, const int2* pairs, const int* qids, const int* tids, int4* rows, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_pair_rows, dim3(div_up(n, kCcdBlock)), dim3(kCcdBlock), 0, s, n, ee, pairs, qids, tids, rows);
}

void launch_fill_u64(unsigned long long* a, unsigned long long v, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill_u64, dim3(div_up(n, kCcdBlock)), dim3(kCcdBlock), 0, s, a, v, n);
}

void launch_new_and_tv(int n, bool ee, const int* order, const int2* pairs, const double* toc, const int* qids,
                       const int* tids, int n_pt, const int4* cids, const int* table, unsigned int mask,
                       const double* x, int* is_new, unsigned long long* tv, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_new_and_tv, dim3(div_up(n, kCcdBlock)), dim3(kCcdBlock), 0, s, n, ee, order, pairs, toc,
                       qids, tids, n_pt, cids, table, mask, x, is_new, tv);
}

void launch_keep_new(int n, bool ee, const int* order, const int2* pairs, const double* toc, const int* qids,
                     const int* tids, const unsigned long long* tv, int* keep, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_keep_new, dim3(div_up(n, kCcdBlock)), dim3(kCcdBlock), 0, s, n, ee, order, pairs, toc, qids,
                       tids, tv, keep);
}

void launch_keep_current(int lo, int hi, const double* gam, double gmin, int* keep, hipStream_t s) {
  if (hi > lo)
    hipLaunchKernelGGL(k_keep_current, dim3(div_up(hi - lo, kCcdBlock)), dim3(kCcdBlock), 0, s, lo, hi, gam, gmin,
                       keep);
}

void launch_scatter_current(int lo, int hi, const int* keep, const int* pos, int base, const int4* ids,
                            const double* lam, const double* gam, int4* oids, double* olam, double* ogam,
                            hipStream_t s) {
  if (hi > lo)
    hipLaunchKernelGGL(k_scatter_current, dim3(div_up(hi - lo, kCcdBlock)), dim3(kCcdBlock), 0, s, lo, hi, keep, pos,
                       base, ids, lam, gam, oids, olam, ogam);
}

void launch_scatter_new(int n, bool ee, const int* keep, const int* pos, int base, const int* order,
                        const int2* pairs, const int* qids, const int* tids, int4* oids, double* olam, double* ogam,
                        hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_scatter_new, dim3(div_up(n, kCcdBlock)), dim3(kCcdBlock), 0, s, n, ee, keep, pos, base,
                       order, pairs, qids, tids, oids, olam, ogam);
}

int ccd_min_parts(int n) { return std::max(1, std::min(div_up(n, kCcdBlock), 256)); }

void launch_min_toc(int n, const double* toc, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_min_toc, dim3(ccd_min_parts(n)), dim3(kCcdBlock), 0, s, n, toc, part);
}

int inversion_parts(int T) { return std::max(1, div_up(T, kCcdBlock)); }

void launch_inversion_bound(int T, const int4* tets, const double* x, const double* xh, double sep, double* part,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_inversion_bound, dim3(inversion_parts(T)), dim3(kCcdBlock), 0, s, T, tets, x, xh, sep, part);
}

}  // namespace bfal
