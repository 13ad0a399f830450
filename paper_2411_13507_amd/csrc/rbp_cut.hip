// Cutting graph edges against convex obstacles (Sec. III-B, Alg. 2, eq. Cut-QP;
// Assumption 1): axis-aligned boxes lo <= x <= hi and convex polytopes
// {x : A x <= b}.
//
// A pair is an edge (control points P_0..P_p of its Bezier curve) and an
// obstacle O.  By the convex-hull property (Property 1) the curve is free of
// O when conv(P) and O are disjoint.  Alg. 2 decides this in three steps:
//   1. a control point inside O                  -> 0 (may collide);
//   2. the supporting plane of O with normal n = centroid - (point of O
//      nearest the centroid) has every control point strictly beyond it
//                                                -> 1 (free);
//   3. otherwise the Cut-QP: |delta*|^2 > 0       -> 1, else 0.
// The Cut-QP's optimum is min over conv(P) of |(A x - b)_+|^2: for a box
// (unit rows) the squared distance between conv(P) and the box.  Step 3
// decides by the distance between conv(P) and O, computed with the
// Gilbert-Johnson-Keerthi iteration on the Minkowski difference (support
// points in closed form for a box, over the vertex table for a polytope),
// in FP64; the distance is zero exactly when the Cut-QP optimum is.  For a
// polytope the optimum itself is then computed, when asked for, by a second
// pass with one wavefront per pair (Newton steps over the pieces of the
// objective, each piece minimised exactly; see cut_value_kernel).
//
// Work split, three kernels (a fourth for the Cut-QP values of polytopes):
//   cut_edge_kernel    per edge: centroid c of the control points and the reach
//                      that decides far pairs (below);
//   cut_prefilter_kernel  every pair: most edges are far from most obstacles, and
//                      then steps 1 and 2 need no look at the control points:
//                      with R = max |P_k - c| and n = c - (point of O nearest c),
//                      n . P_k - max_O n . x >= |n| (|n| - R), so dist(c, O) > R
//                      means no control point in O (step 1) and every one beyond
//                      the supporting plane (step 2).  The distance to O's box
//                      bounds dist(c, O) from below (exact for a box).  Such
//                      pairs get their code here; the others go to a list;
//   cut_qp_kernel    the listed pairs, one thread each: steps 1, 2 and 3.
// For a box the nearest point is a clamp and the supporting plane's offset a
// corner; for a polytope both come from its vertices (a GJK projection of the
// centroid, a maximum over the vertices).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rbp_internal.hpp"
#include "rbp_wave.hpp"

namespace rbp {
namespace {

constexpr int kCutBlock = 256;
constexpr int kWave = 64;
constexpr int kObsChunk = 8;    // obstacles per block of the filter
constexpr int kEdges = 4;       // edges per thread of the filter
constexpr int kTile = kCutBlock * kEdges;   // edges per block of the filter
// list entries are (obstacle << 32 | edge); this bit marks the polytope pairs
// whose Cut-QP value is still to be computed
constexpr int64_t kWantsValue = int64_t(1) << 62;

// The pairs a filter block can list have a region of the list of their own,
// as many entries as the block has pairs; region r belongs to edge tile r % n_tile
// and obstacle chunk r / n_tile.
__device__ __forceinline__ int64_t region_base(const CutArgs& A, int r) {
  const int oc = r / A.n_tile, x = r - oc * A.n_tile, o0 = oc * kObsChunk;
  const int rows = A.n_obst - o0 < kObsChunk ? A.n_obst - o0 : kObsChunk;
  return (int64_t)o0 * A.n_edges + (int64_t)x * kTile * rows;
}

struct V3 {
  double x, y, z;
};
__device__ __forceinline__ V3 sub(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ double dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 axpy(double t, V3 a, V3 b) { return {b.x + t * a.x, b.y + t * a.y, b.z + t * a.z}; }

// Per edge: centroid of the control points and (R + margin)^2 for the far
// test, 0 obstacles counted; the counters of the run start at 0.  The margin
// covers the rounding of the far test and of the plane test it stands for
// (about 1e-15 of the coordinates) and, for polytopes, the 1e-9 to which
// vertices and rows agree.
template <int P>
__global__ __launch_bounds__(kCutBlock) void cut_edge_kernel(CutArgs A) {
  constexpr int NP = P + 1;
  const int e = blockIdx.x * kCutBlock + threadIdx.x;
  if (e == 0) *A.most = 0;
  if (e >= A.n_edges) return;
  A.n_collide[e] = 0;
  double p[3 * NP];
#pragma unroll
  for (int i = 0; i < 3 * NP; ++i) p[i] = A.P[(int64_t)e * (3 * NP) + i];
  double c[3] = {0.0, 0.0, 0.0}, scale = 1.0, r2 = 0.0;
#pragma unroll
  for (int i = 0; i < 3 * NP; ++i) { c[i % 3] += p[i]; scale = fmax(scale, fabs(p[i])); }
#pragma unroll
  for (int i = 0; i < 3; ++i) c[i] /= NP;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const double x = p[3 * k] - c[0], y = p[3 * k + 1] - c[1], z = p[3 * k + 2] - c[2];
    const double d = x * x + y * y + z * z;
    r2 = d > r2 || !(d == d) ? d : r2;       // a NaN stays: no pair is far then
  }
  const double reach = sqrt(r2) * (1.0 + 1e-6) + 1e-6 * scale;
  A.ctr[e] = {c[0], c[1], c[2], reach * reach};
}

// Far pairs, kEdges edges per thread and kObsChunk obstacles per block: a pair
// costs the distance of a point to a box (about 12 operations) and its output
// bytes.  kVec: the thread's edges are consecutive, so that a row's codes go
// out as one 4-byte word (and the NaNs as two 16-byte ones) where every row of
// the outputs starts aligned; otherwise they lie a wavefront apart, so that a
// store still covers consecutive bytes.  Pairs that are not far go to the block's
// own region of the list, their number to n_near: with one atomic on a common
// counter per block, let alone per wavefront, the counter itself bounds the kernel.
// 50,000 edges x 200 boxes: 70.4 us with steps 1 and 2 on every pair, 26.5 us with
// the far test and one counter, 19 us with regions; 20,000 edges x (200 boxes + 100
// polytopes), with steps and values: 315, 23 and 18 us.
template <bool kVec>
__global__ __launch_bounds__(kCutBlock) void cut_prefilter_kernel(CutArgs A) {
  __shared__ int n_near;
  const int tid = threadIdx.x;
  if (tid == 0) n_near = 0;
  __syncthreads();
  const int e0 = blockIdx.x * (kCutBlock * kEdges) + (kVec ? tid * kEdges : (tid & ~(kWave - 1)) * kEdges + (tid & (kWave - 1)));
  constexpr int kStep = kVec ? 1 : kWave;
  CutCtr c[kEdges];
#pragma unroll
  for (int u = 0; u < kEdges; ++u) {
    const int e = e0 + u * kStep;
    c[u] = A.ctr[e < A.n_edges ? e : A.n_edges - 1];
  }
  const int region = (A.obst_base / kObsChunk + blockIdx.y) * A.n_tile + blockIdx.x;
  int64_t* const near = A.list + region_base(A, region);
  const int o0 = A.obst_base + blockIdx.y * kObsChunk, o1 = o0 + kObsChunk < A.n_obst ? o0 + kObsChunk : A.n_obst;
  // the boxes of the chunk's obstacles (their own corners, or those of their
  // vertices), a corner coordinate per lane: one wait for all of them
  double corner = 0.0;
  {
    const int l = tid & (kWave - 1), i = l / 6, k = l - 6 * i;
    const int64_t o = o0 + i;
    if (o < o1 && i < kObsChunk)
      corner = o >= A.n_box ? A.pbox[6 * (o - A.n_box) + k] : k < 3 ? A.box_lo[3 * o + k] : A.box_hi[3 * o + k - 3];
  }
  for (int o = o0; o < o1; ++o) {
    const int l = 6 * (o - o0);
    const double lx = wave::bcast(corner, l), ly = wave::bcast(corner, l + 1), lz = wave::bcast(corner, l + 2),
                 hx = wave::bcast(corner, l + 3), hy = wave::bcast(corner, l + 4), hz = wave::bcast(corner, l + 5);
    // a box that is not finite, or inverted, has no far pairs
    const bool proper = hx - lx >= 0.0 && hy - ly >= 0.0 && hz - lz >= 0.0 && hx - lx <= 1e300 && hy - ly <= 1e300 &&
                        hz - lz <= 1e300;
    uint32_t codes = 0u, steps = 0u;
#pragma unroll
    for (int u = 0; u < kEdges; ++u) {
      const double nx = c[u].x - fmin(fmax(c[u].x, lx), hx), ny = c[u].y - fmin(fmax(c[u].y, ly), hy),
                   nz = c[u].z - fmin(fmax(c[u].z, lz), hz);
      const bool far = proper && nx * nx + ny * ny + nz * nz > c[u].reach2;
      codes |= (far ? 1u : 0u) << (8 * u);
      steps |= (far ? 2u : 3u) << (8 * u);
    }
    const int64_t row = (int64_t)o * A.n_edges;
    if constexpr (kVec) {
      if (e0 < A.n_edges) {
        *reinterpret_cast<uint32_t*>(A.code + row + e0) = codes;
        if (A.step) *reinterpret_cast<uint32_t*>(A.step + row + e0) = steps;
        if (A.qp_dist2) {
          const double nan = __builtin_nan("");
          double2* q = reinterpret_cast<double2*>(A.qp_dist2 + row + e0);
          q[0] = make_double2(nan, nan);
          q[1] = make_double2(nan, nan);
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < kEdges; ++u) {
        const int e = e0 + u * kStep;
        if (e < A.n_edges) {
          A.code[row + e] = (uint8_t)(codes >> (8 * u));
          if (A.step) A.step[row + e] = (uint8_t)(steps >> (8 * u));
          if (A.qp_dist2) A.qp_dist2[row + e] = __builtin_nan("");
        }
      }
    }
    if (codes != 0x01010101u) {
#pragma unroll
      for (int u = 0; u < kEdges; ++u) {
        const int e = e0 + u * kStep;
        if (((codes >> (8 * u)) & 1u) == 0u && e < A.n_edges) {
          near[atomicAdd(&n_near, 1)] = ((int64_t)o << 32) | (int64_t)e;
        }
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    A.n_near[region] = n_near;
    if (n_near > kWave) atomicMax(A.most, n_near);   // readers take 64 for less
  }
}

// 1 / x to an ulp or two: the hardware's estimate, corrected twice.
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

// Closest point to the origin of conv(w[0..k)), k <= 4, where w[0] is the
// point added last: the nearest accepted projection over the faces that hold
// w[0].  The closest point of conv(w[1..k)) is known and w[0] lies beyond the
// plane through it, so no other face can hold the new one: 7 faces instead of
// 15, all with the same base point, whose differences and Gram matrix are
// formed once.  On return w[0..k) holds the face found.
__device__ __forceinline__ void closest_face(V3 (&w)[4], int& k, V3& v) {
  const V3 w0 = w[0];
  V3 d[3];
  double G[3][3], r[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) { d[a] = sub(w[a + 1], w0); r[a] = -dot(d[a], w0); }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b) { G[a][b] = dot(d[a], d[b]); G[b][a] = G[a][b]; }
  double best = dot(w0, w0);
  int bm = 0;               // bit a: d[a] spans the face
  v = w0;
  auto offer = [&](bool ok, int mask, V3 x) {
    const double xx = dot(x, x);
    const bool take = ok & (xx < best);
    best = take ? xx : best;
    bm = take ? mask : bm;
    v.x = take ? x.x : v.x;
    v.y = take ? x.y : v.y;
    v.z = take ? x.z : v.z;
  };
  // weights of the other points positive (to rounding), those of w0 too, and
  // the face not degenerate; without branches, so that the faces' chains of
  // dependent operations overlap
  auto edge = [&](int a, bool on) {
    const double g = G[a][a], t = r[a] * rcp_nr(g);
    offer(on & (g > 1e-30 * fmax(g, 1e-300)) & (t > -1e-14) & (1.0 - t > -1e-14), 1 << a, axpy(t, d[a], w0));
  };
  auto tri = [&](int a, int b, bool on) {
    const double gaa = G[a][a], gab = G[a][b], gbb = G[b][b];
    const double scale = fmax(gaa, gbb), det = gaa * gbb - gab * gab, inv = rcp_nr(det);
    const double ta = (r[a] * gbb - gab * r[b]) * inv, tb = (gaa * r[b] - r[a] * gab) * inv;
    offer(on & (fabs(det) > 1e-24 * scale * scale) & (ta > -1e-14) & (tb > -1e-14) & (1.0 - ta - tb > -1e-14),
          (1 << a) | (1 << b), axpy(tb, d[b], axpy(ta, d[a], w0)));
  };
  edge(0, true);
  if (k > 2) {
    const bool four = k > 3;
    edge(1, true);
    edge(2, four);
    tri(0, 1, true);
    tri(0, 2, four);
    tri(1, 2, four);
    const double c00 = G[1][1] * G[2][2] - G[1][2] * G[1][2], c01 = G[0][2] * G[1][2] - G[0][1] * G[2][2],
                 c02 = G[0][1] * G[1][2] - G[0][2] * G[1][1], c11 = G[0][0] * G[2][2] - G[0][2] * G[0][2],
                 c12 = G[0][1] * G[0][2] - G[0][0] * G[1][2], c22 = G[0][0] * G[1][1] - G[0][1] * G[0][1];
    const double det = G[0][0] * c00 + G[0][1] * c01 + G[0][2] * c02, inv = rcp_nr(det);
    const double scale = fmax(G[0][0], fmax(G[1][1], G[2][2]));
    const double t0 = (c00 * r[0] + c01 * r[1] + c02 * r[2]) * inv, t1 = (c01 * r[0] + c11 * r[1] + c12 * r[2]) * inv,
                 t2 = (c02 * r[0] + c12 * r[1] + c22 * r[2]) * inv;
    offer(four & (fabs(det) > 1e-24 * scale * scale * scale) & (t0 > -1e-14) & (t1 > -1e-14) & (t2 > -1e-14) &
              (1.0 - t0 - t1 - t2 > -1e-14),
          7, axpy(t2, d[2], axpy(t1, d[1], axpy(t0, d[0], w0))));
  }
  // keep the face's points, in order
  const V3 w1 = w[1], w2 = w[2], w3 = w[3];
  w[1] = (bm & 1) ? w1 : (bm & 2) ? w2 : w3;
  w[2] = (bm & 3) == 3 ? w2 : w3;
  k = 1 + __builtin_popcount(bm);
}

// The first of the points v0..v1-1 of pv that maximises u . p, and the maximum;
// four points in flight (a lane's loads hit L2, one after the other they are
// most of a support call).
__device__ __forceinline__ V3 farthest(const double* pv, int v0, int v1, V3 u, double& best) {
  V3 bv{0.0, 0.0, 0.0};
  best = 0.0;
  for (int q = v0; q < v1; q += 4) {
    V3 p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t qi = 3 * (int64_t)(q + i < v1 ? q + i : v1 - 1);
      p[i] = {pv[qi], pv[qi + 1], pv[qi + 2]};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double d = dot(u, p[i]);
      if ((q == v0 && i == 0) || d > best) { best = d; bv = p[i]; }
    }
  }
  return bv;
}

// Squared distance from the origin to a convex set given by its support
// mapping (support(u) minimises u . w over the set), starting from the point
// w0 of the set: the Gilbert-Johnson-Keerthi iteration, stopping when
// |v|^2 - v . w <= 1e-13 |v|^2 (the gap bound), when no progress is made or
// when the origin lies in a tetrahedron of set points.  Results at or below
// zero2 count as 0.  v returns the closest point found.
template <class Support>
__device__ double gjk_dist2(Support support, V3 w0, double zero2, V3& v) {
  V3 w[4] = {w0, w0, w0, w0};
  int k = 1;
  v = w0;
  double vv = dot(v, v);
  for (int it = 0; it < 64 && vv > zero2; ++it) {
    const V3 wn = support(v);
    if (vv - dot(v, wn) <= 1e-13 * vv) break;
    bool dup = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) dup |= (i < k) & (w[i].x == wn.x) & (w[i].y == wn.y) & (w[i].z == wn.z);
    if (dup) break;
    w[3] = w[2];
    w[2] = w[1];
    w[1] = w[0];
    w[0] = wn;
    ++k;
    V3 nv;
    closest_face(w, k, nv);
    const double nvv = dot(nv, nv);
    if (!(nvv < vv)) break;   // no progress: v is optimal to rounding
    v = nv;
    vv = nvv;
    if (k == 4) { vv = 0.0; v = V3{0.0, 0.0, 0.0}; break; }   // the origin lies in a tetrahedron
  }
  return vv > zero2 ? vv : 0.0;
}

// ---- Cut-QP value of a polytope pair (one wavefront per pair)
//
// With the slacks eliminated (for fixed weights the best slack of a row is
// its violation) the Cut-QP optimum is  f* = min over x in conv(P) of
// f(x) = |(A x - b)_+|^2, a convex piecewise quadratic; on the rows S
// violated at x it equals q_S(x) = |A_S x - b_S|^2.  Each outer step
//   1. evaluates f and the Lagrange-dual bound h(mu) = min_j mu . (A P_j - b)
//      - |mu|^2 / 4 <= f* at mu = 2 (A x - b)_+, and stops when f - h is at
//      most 1e-11 f or f no longer decreases;
//   2. minimises q_S over conv(P) exactly (Wolfe's minimum-norm-point method:
//      q_S(P^T lam) is the squared norm of sum_j lam_j w_j with
//      w_j = A_S P_j - b_S, whose Gram matrix follows from the moments
//      H = A_S^T A_S, g = A_S^T b_S, c = |b_S|^2);
//   3. moves to the minimiser of f on the segment towards that point (f is a
//      convex piecewise quadratic along it: safeguarded Newton on its slope,
//      exact once the segment's violated rows are found).
// Once S is the violated set of the optimum, step 2 lands on it.  The rows
// are spread one per lane (at most 32); x and the moments are uniform.

// 3 x 3 symmetric matrix as (xx, xy, xz, yy, yz, zz)
__device__ __forceinline__ V3 sym_mul(const double (&H)[6], V3 v) {
  return {H[0] * v.x + H[1] * v.y + H[2] * v.z, H[1] * v.x + H[3] * v.y + H[4] * v.z,
          H[2] * v.x + H[4] * v.y + H[5] * v.z};
}

// Wolfe's minimum-norm-point method for min over the simplex of
// q(x) = x^T H x - 2 g^T x + c, x = sum_j lam_j P_j, H positive
// semidefinite.  q is the squared norm of sum_j lam_j w_j for points w_j of
// an affine space of dimension at most 3, so the corral (the affinely
// independent points carrying the current weights) holds at most four; its
// points, weights and indices stay in registers.  Returns the minimiser x.
template <int NP>
__device__ V3 min_norm_point(const V3 (&pts)[NP], const double (&H)[6], V3 g, double c) {
  V3 cp[4];
  int cid[4];
  double al[4];
  // start at the vertex with the smallest q
  double qbest = __builtin_huge_val(), dmax = 0.0;
  cp[0] = pts[0];
  cid[0] = 0;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const double qk = dot(pts[k], sym_mul(H, pts[k])) - 2.0 * dot(g, pts[k]) + c;
    dmax = fmax(dmax, fabs(qk));
    if (qk < qbest) { qbest = qk; cp[0] = pts[k]; cid[0] = k; }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) al[i] = i == 0 ? 1.0 : 0.0;
#pragma unroll
  for (int i = 1; i < 4; ++i) { cp[i] = cp[0]; cid[i] = -1; }
  int nc = 1;
  auto point = [&]() {
    V3 x{0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 4; ++i) x = axpy(i < nc ? al[i] : 0.0, cp[i], x);
    return x;
  };
  bool done = false;
  for (int major = 0; major < 16 && !done; ++major) {
    const V3 x = point();
    const V3 v = sub(sym_mul(H, x), g);   // x_w . w_j = v . P_j - g . x + c
    const double gx = dot(g, x);
    const double xx = dot(v, x) - gx + c;
    double best = __builtin_huge_val();
    int jb = -1;
    V3 pb = pts[0];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const double vk = dot(v, pts[k]);
      if (vk < best) { best = vk; jb = k; pb = pts[k]; }
    }
    if (best - gx + c >= xx - 1e-14 * dmax) break;     // x is optimal
    bool dup = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) dup |= (i < nc) & (cid[i] == jb);
    if (dup || nc == 4) break;                         // no independent point left (rounding)
#pragma unroll
    for (int i = 1; i < 4; ++i)
      if (i == nc) { cp[i] = pb; cid[i] = jb; al[i] = 0.0; }
    ++nc;
    // minor cycles: the affine minimiser of the corral, clipped back into
    // its hull while it has a weight <= 0
    for (int minor = 0; minor < 4; ++minor) {
      // y minimises q(cp0 + sum_i y_i (cp_i - cp0)): [D^T H D] y = -D^T (H cp0 - g)
      const int n = nc - 1;
      V3 D[3];
      double M[3][3], y[3];
      const V3 r0 = sub(sym_mul(H, cp[0]), g);
#pragma unroll
      for (int i = 0; i < 3; ++i) D[i] = sub(cp[i + 1], cp[0]);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const V3 HDi = sym_mul(H, D[i]);
#pragma unroll
        for (int j = 0; j < 3; ++j) M[i][j] = (i < n && j < n) ? dot(D[j], HDi) : (i == j ? 1.0 : 0.0);
        y[i] = i < n ? -dot(D[i], r0) : 0.0;
      }
      // symmetric elimination (no pivoting: M is positive definite when the
      // corral is affinely independent); a pivot that vanishes against its
      // diagonal entry means it is not
      double d0[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) d0[i] = M[i][i];
      bool sing = false;
      double ip[3];             // 1 / pivot
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        sing |= !(M[k][k] > 1e-12 * d0[k]) | !(d0[k] > 0.0);
        ip[k] = rcp_nr(M[k][k] > 0.0 ? M[k][k] : 1.0);
#pragma unroll
        for (int i = k + 1; i < 3; ++i) {
          const double l = M[i][k] * ip[k];
#pragma unroll
          for (int j = k + 1; j < 3; ++j) M[i][j] -= l * M[k][j];
          y[i] -= l * y[k];
        }
      }
#pragma unroll
      for (int k = 2; k >= 0; --k) {
        double acc = y[k];
#pragma unroll
        for (int j = k + 1; j < 3; ++j) acc -= M[k][j] * y[j];
        y[k] = acc * ip[k];
      }
      if (sing) {          // stop: al are convex weights of the corral as it stands
        done = true;
        break;
      }
      double be[4];
      be[0] = 1.0;
#pragma unroll
      for (int i = 1; i < 4; ++i) { be[i] = i < nc ? y[i - 1] : 0.0; be[0] -= be[i]; }
      bool inside = true;
#pragma unroll
      for (int i = 0; i < 4; ++i) inside &= (i >= nc) | (be[i] > 0.0);
      if (inside) {
#pragma unroll
        for (int i = 0; i < 4; ++i) al[i] = be[i];
        break;
      }
      // largest step from al towards be that keeps every weight >= 0, and the point
      // whose weight it takes to 0 (some be is <= 0; where both weights are 0 the
      // step is 0)
      double th = 2.0;
      int kd = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i < nc && be[i] <= 0.0) {
          const double ti = al[i] > 0.0 ? fmin(al[i] * rcp_nr(al[i] - be[i]), 1.0) : 0.0;
          if (ti < th) { th = ti; kd = i; }
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) al[i] = (1.0 - th) * al[i] + th * be[i];
      // remove corral point kd (its weight is now 0)
#pragma unroll
      for (int i = 0; i < 3; ++i)
        if (i >= kd) { cp[i] = cp[i + 1]; cid[i] = cid[i + 1]; al[i] = al[i + 1]; }
      --nc;
      double sa = 0.0;
#pragma unroll
      for (int i = 0; i < 4; ++i) { al[i] = i < nc ? fmax(al[i], 0.0) : 0.0; sa += al[i]; }
      const double is = rcp_nr(sa);
#pragma unroll
      for (int i = 0; i < 4; ++i) al[i] *= is;
      if (nc == 1) break;
    }
  }
  return point();
}

template <int NP>
__global__ __launch_bounds__(kCutBlock) void cut_value_kernel(CutArgs A) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kCutBlock / kWave) + threadIdx.x / kWave));
  const int64_t nw = (int64_t)gridDim.x * (kCutBlock / kWave);
  const int64_t R = A.n_region, n = R * (*A.most > kWave ? *A.most : kWave);
  // a wavefront looks at 64 entries at once, nw apart in the order first entry
  // of every region, second entry, .. (a region's entries are alike, so the
  // marked ones spread over the wavefronts)
  for (int64_t t0 = wv; t0 < n; t0 += nw * kWave) {
    const int64_t tl = t0 + nw * lane, slot = tl / R;
    const int r = (int)(tl - slot * R);
    const int64_t el = tl < n && slot < A.n_near[r] ? A.list[region_base(A, r) + slot] : 0;
    for (unsigned long long todo = __ballot((el & kWantsValue) != 0); todo; todo &= todo - 1) {
      const int src = __builtin_ctzll(todo);
      const int o = __builtin_amdgcn_readlane((int)((el & ~kWantsValue) >> 32), src);
      const int e = __builtin_amdgcn_readlane((int)(el & 0xffffffffll), src);
      const int64_t qi = (int64_t)o * A.n_edges + e;
      const int jp = o - A.n_box;
      const int r0 = A.pob_off[jp], m = A.pob_off[jp + 1] - r0;
      // row of this lane (idle lanes: 0 . x - 1 < 0, never violated)
      const bool rl = lane < m;
      const V3 a = rl ? V3{A.pob_A[3 * (r0 + lane)], A.pob_A[3 * (r0 + lane) + 1], A.pob_A[3 * (r0 + lane) + 2]}
                      : V3{0.0, 0.0, 0.0};
      // in coordinates about the first control point: the moments are sums of
      // squares of coordinates, and far from the origin their differences cancel
      // (at 1e6 and sizes of 1, one value in thirty was off by 1e-9 to 70 %)
      V3 pts[NP];
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int64_t b = (int64_t)e * (3 * NP) + 3 * k;
        pts[k] = {A.P[b], A.P[b + 1], A.P[b + 2]};
      }
      const V3 at = pts[0];
      const double bk = rl ? A.pob_b[r0 + lane] - dot(a, at) : 1.0;
      V3 x{0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        pts[k] = sub(pts[k], at);
        x = axpy(1.0 / NP, pts[k], x);
      }
      double fbest = __builtin_huge_val(), fprev = __builtin_huge_val();
      for (int it = 0; it < 32; ++it) {
        const double r = dot(a, x) - bk;
        const double rp = fmax(r, 0.0);
        double s4[4] = {rp * rp, rp * a.x, rp * a.y, rp * a.z};
        wave::sum4(s4);
        const double f = s4[0];
        const double beta = wave::sum(rp * bk);
        fbest = fmin(fbest, f);
        if (!(f > 0.0) || !(f < fprev)) break;
        fprev = f;
        const V3 u{s4[1], s4[2], s4[3]};
        double mn = __builtin_huge_val();
#pragma unroll
        for (int k = 0; k < NP; ++k) mn = fmin(mn, dot(u, pts[k]));
        const double h = 2.0 * (mn - beta) - f;
        if (f - h <= 1e-11 * f) break;
        // moments of the violated rows
        const double sw = r > 0.0 ? 1.0 : 0.0;
        double m1[4] = {sw * a.x * a.x, sw * a.x * a.y, sw * a.x * a.z, sw * a.y * a.y};
        double m2[4] = {sw * a.y * a.z, sw * a.z * a.z, sw * bk * a.x, sw * bk * a.y};
        double m3[4] = {sw * bk * a.z, sw * bk * bk, 0.0, 0.0};
        wave::sum4(m1);
        wave::sum4(m2);
        wave::sum4(m3);
        const double H[6] = {m1[0], m1[1], m1[2], m1[3], m2[0], m2[1]};
        const V3 xs = min_norm_point<NP>(pts, H, V3{m2[2], m2[3], m3[0]}, m3[1]);
        // half the slope of f at x along xs - x is u . (xs - x): stop unless it
        // descends
        if (!(dot(u, sub(xs, x)) < 0.0)) break;
        // line search on f along x + t (xs - x), t in [0, 1]: half its slope
        // is sum_k (r_k + t d_k)_+ d_k, nondecreasing in t
        const double dk = dot(a, sub(xs, x));
        auto slope = [&](double t, double& s2) {
          const double rt = r + t * dk;
          double v2[2] = {rt > 0.0 ? rt * dk : 0.0, rt > 0.0 ? dk * dk : 0.0};
          // two sums, interleaved through the same stages
          double v4[4] = {v2[0], v2[1], 0.0, 0.0};
          wave::sum4(v4);
          s2 = v4[1];
          return v4[0];
        };
        double s2;
        double t = 1.0;
        const double g1 = slope(1.0, s2);
        if (g1 > 0.0) {
          double lo = 0.0, hi = 1.0;
          // the piece at t = 1 is linear: its root is the Newton point
          double tn = s2 > 0.0 ? 1.0 - g1 / s2 : 0.5;
          for (int ls = 0; ls < 40; ++ls) {
            t = (tn > lo && tn < hi) ? tn : 0.5 * (lo + hi);
            double q2;
            const double gt = slope(t, q2);
            if (gt == 0.0) break;
            if (gt > 0.0) hi = t; else lo = t;
            if (!(hi - lo > 1e-15)) break;
            tn = q2 > 0.0 ? t - gt / q2 : 0.5 * (lo + hi);
            if (tn == t) break;
          }
        }
        if (!(t > 0.0)) break;
        x = axpy(t, sub(xs, x), x);
      }
      if (lane == 0) A.qp_dist2[qi] = fbest;
    }
  }
}

// Steps 1 to 3 of Alg. 2 for the listed pairs, one thread per pair: bound by
// the latency of the chain of one pair (the GJK iterations), so a pair's steps
// run one after the other in the same thread instead of in launches of their
// own.  Blocks of one wavefront spread a short list over the compute units.
// 50,000 edges x 200 boxes (8,500 pairs listed, 3,800 of them to step 3): 38 us with
// every face of the simplex tried and divisions, 23 us now; 20,000 edges x (200
// boxes + 100 polytopes): 100 -> 50 us.  With longer edges more pairs are near; the
// list still pays then, since the branches of step 3 no longer hold up the lanes
// that steps 1 and 2 decide.  50,000 x 200 with steps 1 and 2 on every pair / now,
// whole runs, for edges of 0.5, 2, 6 and 10 m in a 10 m cube (0.1, 2, 19 and 45 % of
// the pairs to step 3): 158 / 59, 1,332 / 146, 2,314 / 777 and 2,845 / 1,179 us.
template <int P>
__global__ __launch_bounds__(kWave) void cut_qp_kernel(CutArgs A) {
  constexpr int NP = P + 1;
  // A wavefront takes 64 entries of a group of consecutive regions (see
  // cut_plan), the first 64 of every group before the next.
  const int lane = threadIdx.x, G = A.group, n_group = (A.n_region + G - 1) / G;
  const int64_t n_chunk = ((int64_t)(*A.most > kWave ? *A.most : kWave) * G + kWave - 1) / kWave;
  const int64_t step_c = gridDim.x / n_group;
  const int step_g = gridDim.x % n_group;
  unsigned n3 = 0;                                            // pairs that reached step 3
  int gi = blockIdx.x % n_group;
  for (int64_t ch = blockIdx.x / n_group; ch < n_chunk;) {
    const int first = gi * G;
    const int64_t t = ch * kWave + lane;
    gi += step_g;
    ch += step_c + (gi >= n_group ? 1 : 0);
    if (gi >= n_group) gi -= n_group;
    const int cn = lane < G && first + lane < A.n_region ? A.n_near[first + lane] : 0;
    int upto = cn, reg = 0;
    if (G > 1) {
      for (int d = 1; d < kWave; d <<= 1) {
        const int up = __shfl_up(upto, d, kWave);
        if (lane >= d) upto += up;
      }
      // the regions that end at or before entry t
      for (int d = kWave / 2; d; d >>= 1)
        if (__shfl(upto, reg + d - 1, kWave) <= t) reg += d;
    }
    const int total = __builtin_amdgcn_readlane(upto, G > 1 ? kWave - 1 : 0);
    const int before = __shfl(upto - cn, reg, kWave);
    const bool live = t < total;
    const int64_t pos = live ? region_base(A, first + reg) + t - before : 0;
    if (__ballot(live) == 0ull) continue;
    const int64_t ent = live ? A.list[pos] : 0;
    const int o = (int)(ent >> 32), e = (int)(ent & 0xffffffffll);
    V3 pts[NP];
    V3 c{0.0, 0.0, 0.0};
    double scale = 1.0;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int64_t b = (int64_t)e * (3 * NP) + 3 * k;
      pts[k] = {A.P[b], A.P[b + 1], A.P[b + 2]};
      c = {c.x + pts[k].x, c.y + pts[k].y, c.z + pts[k].z};
      scale = fmax(scale, fmax(fabs(pts[k].x), fmax(fabs(pts[k].y), fabs(pts[k].z))));
    }
    c = {c.x / NP, c.y / NP, c.z / NP};
    bool inside = false, beyond = false;
    if (live && o < A.n_box) {
      const double lx = A.box_lo[3 * o], ly = A.box_lo[3 * o + 1], lz = A.box_lo[3 * o + 2];
      const double hx = A.box_hi[3 * o], hy = A.box_hi[3 * o + 1], hz = A.box_hi[3 * o + 2];
      // step 1: a control point inside the (closed) box
#pragma unroll
      for (int k = 0; k < NP; ++k)
        inside |= (pts[k].x >= lx) & (pts[k].x <= hx) & (pts[k].y >= ly) & (pts[k].y <= hy) & (pts[k].z >= lz) &
                  (pts[k].z <= hz);
      // step 2: supporting plane of the box with normal centroid - clamp(centroid)
      const V3 m{c.x - fmin(fmax(c.x, lx), hx), c.y - fmin(fmax(c.y, ly), hy), c.z - fmin(fmax(c.z, lz), hz)};
      const double l = (m.x > 0.0 ? m.x * hx : m.x * lx) + (m.y > 0.0 ? m.y * hy : m.y * ly) + (m.z > 0.0 ? m.z * hz : m.z * lz);
      beyond = (m.x != 0.0) | (m.y != 0.0) | (m.z != 0.0);
#pragma unroll
      for (int k = 0; k < NP; ++k) beyond &= dot(m, pts[k]) > l;
    } else if (live) {
      const int j = o - A.n_box;
      // step 1: a control point that satisfies every row (bit k set: point k
      // violates some row)
      const int r0 = A.pob_off[j], r1 = A.pob_off[j + 1];
      unsigned outside = 0u;
      for (int r = r0; r < r1; r += 4) {
        V3 a[4];
        double bb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {          // the last row again past the end
          const int ri = r + i < r1 ? r + i : r1 - 1;
          a[i] = {A.pob_A[3 * ri], A.pob_A[3 * ri + 1], A.pob_A[3 * ri + 2]};
          bb[i] = A.pob_b[ri];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < NP; ++k) outside |= (dot(a[i], pts[k]) > bb[i] ? 1u : 0u) << k;
      }
      inside = outside != (1u << NP) - 1u;
      if (!inside) {
        // step 2: the point of O nearest the centroid c (GJK over the set
        // c - O, whose support is c minus the vertex maximising u . v); the
        // normal m = c - that point; offset = max over the vertices of m . v
        const int v0 = A.pv_off[j], v1 = A.pv_off[j + 1];
        auto vmax = [&](V3 u, double& best) -> V3 {
          return farthest(A.pv, v0, v1, u, best);
        };
        auto support = [&](V3 u) -> V3 { double bd; return sub(c, vmax(u, bd)); };
        V3 m;
        const V3 w0 = sub(c, V3{A.pv[3 * v0], A.pv[3 * v0 + 1], A.pv[3 * v0 + 2]});
        (void)gjk_dist2(support, w0, 1e-24 * scale * scale, m);
        double l;
        (void)vmax(m, l);
        beyond = (m.x != 0.0) | (m.y != 0.0) | (m.z != 0.0);
#pragma unroll
        for (int k = 0; k < NP; ++k) beyond &= dot(m, pts[k]) > l;
      }
    }
    // pairs that reach step 3, counted for rbp_cut_qp_count
    n3 += (unsigned)__popcll(__ballot(live && !inside && !beyond));
    if (!live) continue;
    const int64_t q = (int64_t)o * A.n_edges + e;
    if (inside || beyond) {
      A.code[q] = inside ? 0 : 1;
      if (A.step) A.step[q] = inside ? 1 : 2;
      if (inside) atomicAdd(&A.n_collide[e], 1);
      continue;
    }
    // step 3: squared distance between conv(P) and the obstacle
    const double zero2 = 1e-24 * scale * scale;
    double d2, value;
    if (o < A.n_box) {
      const V3 lo{A.box_lo[3 * o], A.box_lo[3 * o + 1], A.box_lo[3 * o + 2]};
      const V3 hi{A.box_hi[3 * o], A.box_hi[3 * o + 1], A.box_hi[3 * o + 2]};
      // support point of conv(P) - box minimising u . w (kept by selection)
      auto support = [&](V3 u) -> V3 {
        V3 bp = pts[0];
        double bd = dot(u, pts[0]);
#pragma unroll
        for (int k = 1; k < NP; ++k) {
          const double d = dot(u, pts[k]);
          if (d < bd) { bd = d; bp = pts[k]; }
        }
        const V3 bx{u.x > 0.0 ? hi.x : lo.x, u.y > 0.0 ? hi.y : lo.y, u.z > 0.0 ? hi.z : lo.z};
        return sub(bp, bx);
      };
      const V3 c0{fmin(fmax(pts[0].x, lo.x), hi.x), fmin(fmax(pts[0].y, lo.y), hi.y), fmin(fmax(pts[0].z, lo.z), hi.z)};
      V3 v;
      d2 = gjk_dist2(support, sub(pts[0], c0), zero2, v);
      value = d2;   // unit rows: the Cut-QP optimum is the squared distance
    } else {
      const int jp = o - A.n_box;
      const int v0 = A.pv_off[jp], v1 = A.pv_off[jp + 1];
      // support point of conv(P) - conv(vertices) minimising u . w
      auto support = [&](V3 u) -> V3 {
        V3 bp = pts[0];
        double bd = dot(u, pts[0]);
#pragma unroll
        for (int k = 1; k < NP; ++k) {
          const double d = dot(u, pts[k]);
          if (d < bd) { bd = d; bp = pts[k]; }
        }
        double best;
        return sub(bp, farthest(A.pv, v0, v1, u, best));
      };
      V3 v;
      d2 = gjk_dist2(support, sub(pts[0], V3{A.pv[3 * v0], A.pv[3 * v0 + 1], A.pv[3 * v0 + 2]}), zero2, v);
      // 0 when conv(P) meets O; otherwise the value pass overwrites it with
      // the Cut-QP optimum
      value = d2;
    }
    const int code = d2 > 0.0 ? 1 : 0;
    A.code[q] = (uint8_t)code;
    if (A.qp_dist2) {
      A.qp_dist2[q] = value;
      if (code && o >= A.n_box) A.list[pos] = ent | kWantsValue;
    }
    if (!code) atomicAdd(&A.n_collide[e], 1);
  }
  if (lane == 0) A.n_third[blockIdx.x] = n3;
}

template <int P>
hipError_t launch_cut_p(const CutArgs& a, hipStream_t s, int n_cu) {
  hipLaunchKernelGGL((cut_edge_kernel<P>), dim3((a.n_edges + kCutBlock - 1) / kCutBlock), dim3(kCutBlock), 0, s, a);
  if (a.n_obst <= 0) return hipGetLastError();
  // grid.y is limited to 65,535 blocks: more obstacles go in further launches
  constexpr int kMost = 65535 * kObsChunk;
  const int n_poly = a.n_obst - a.n_box;
  const int gx = a.n_tile;
  // words of four edges: every row o * n_edges of the outputs starts on one
  const bool vec = a.n_edges % kEdges == 0 && (reinterpret_cast<uintptr_t>(a.code) & 3) == 0 &&
                   (reinterpret_cast<uintptr_t>(a.step) & 3) == 0 && (reinterpret_cast<uintptr_t>(a.qp_dist2) & 15) == 0;
  for (int o = 0; o < a.n_obst; o += kMost) {   // kMost is a multiple of kObsChunk
    CutArgs b = a;
    b.obst_base = o;
    const int n = a.n_obst - o < kMost ? a.n_obst - o : kMost;
    const dim3 grid(gx, (n + kObsChunk - 1) / kObsChunk);
    if (vec) hipLaunchKernelGGL(cut_prefilter_kernel<true>, grid, dim3(kCutBlock), 0, s, b);
    else hipLaunchKernelGGL(cut_prefilter_kernel<false>, grid, dim3(kCutBlock), 0, s, b);
  }
  hipLaunchKernelGGL((cut_qp_kernel<P>), dim3(a.n_blocks), dim3(kWave), 0, s, a);
  if (a.qp_dist2 && n_poly > 0)
    hipLaunchKernelGGL((cut_value_kernel<P + 1>), dim3(4 * n_cu), dim3(kCutBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// The list's regions of n_edges x n_obst pairs, the blocks of the step kernel and
// how many regions one of its wavefronts looks at together.
void cut_plan(CutArgs& a, int n_cu) {
  a.n_tile = (a.n_edges + kTile - 1) / kTile;
  a.n_region = a.n_tile * ((a.n_obst + kObsChunk - 1) / kObsChunk);
  a.n_blocks = 16 * n_cu;
  // two wavefronts per CU where few pairs are listed: the chain of the slowest
  // pair sets the time, and more wavefronts only share the instruction cache
  // (50,000 x 200: 26.7 us with one region each, 1,225 wavefronts; 23.3 with three).
  // Whole runs with one / two / four / eight per CU: 50,000 x 200 boxes 50 / 50 / 52 /
  // 55 us, x 300 55 / 57 / 61 / 60, 100,000 x 300 72 / 75 / 74 / 75, 20,000 x (200 + 100
  // polytopes) 76 / 71 / 71 / 71, with values 132 / 127 / 126 / 127
  const int g = a.n_region / (2 * n_cu) + 1;
  a.group = g < kWave ? g : kWave;
}

hipError_t launch_cut(const CutArgs& a, hipStream_t s, int n_cu) {
  if (a.n_edges <= 0) return hipSuccess;
  switch (a.degree) {
    case 1: return launch_cut_p<1>(a, s, n_cu);
    case 2: return launch_cut_p<2>(a, s, n_cu);
    case 3: return launch_cut_p<3>(a, s, n_cu);
    case 4: return launch_cut_p<4>(a, s, n_cu);
    case 5: return launch_cut_p<5>(a, s, n_cu);
    case 6: return launch_cut_p<6>(a, s, n_cu);
    case 7: return launch_cut_p<7>(a, s, n_cu);
    case 8: return launch_cut_p<8>(a, s, n_cu);
    case 9: return launch_cut_p<9>(a, s, n_cu);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rbp
