// Building the graph of Bezier curves (Sec. III-A, Thm. 2) and the adjacent
// hyperplanes of its nodes (Alg. 2, Sec. III-D).
//
// Edge i -> j when F [v_i; v_j] <= G, i.e. max_k (A_ik + B_jk) <= 0 with the
// per-node row values A = F1 v (start columns) and B = F2 v - G (end
// columns): an all-pairs (max, +) product of two N x m matrices followed by a
// sign test, in FP64.  Two kernels: graph_rows_kernel forms A and B with the
// minima of every 64-node tile, graph_pairs_kernel the adjacency, one word of
// 32 end nodes for 64 start nodes (one per lane) at a time.  Exact bounds cut
// the work: a tile of start nodes and a tile of end nodes are skipped if
// min_i A_ik + min_j B_jk > 0 for some row k, and a single end node j if
// min_i A_ik + B_jk > 0.  With nodes numbered along a space-filling curve most
// far pairs go this way, so the work follows the number of near pairs rather
// than N^2; the result does not depend on it where every row value is a number.
// (The bounds pass over NaN: a NaN row value violates nothing in a pair that is
// looked at, but its tile may be skipped for the other nodes' sake, and is
// where none of them has a number in that row.)
// Output: the adjacency as a row-major bitmask (bit j % 32 of word j / 32 of
// row i) and out-degrees.
//
// Adjacent hyperplanes: per node, the nearest axis-aligned box (Euclidean
// distance, lowest index on ties), the closest point on it (a clamp) and the
// plane through that point with unit normal toward the node.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>

#include "rbp_internal.hpp"
#include "rbp_wave.hpp"

namespace rbp {

// Workspace of the allocation-free graph run (rows A and B, tile minima):
// a fixed array in device memory, one copy per GPU, held until the process
// ends.  Host code never uses the name itself as an address: the device
// address of each GPU's copy comes from hipGetSymbolAddress.
// The flags after the row values and minima (one byte per 64 nodes and 16 rows,
// fewer than 65,536 wherever those fit) have room of their own.
static __device__ __align__(256) double scratch[kGraphScratchDoubles + kGraphFlagDoubles];

namespace {

constexpr int kTile = 64;       // nodes per tile side
constexpr int kWords = 4;       // words (of 32 end nodes) per block
constexpr int kEnds = 16;       // end nodes per wavefront
constexpr int kPairWaves = kWords * 32 / kEnds;
constexpr int kRowsPerBlock = 16;   // rows k per block of graph_rows_kernel
constexpr int kPlaneWaves = 16; // most wavefronts per block of hyperplane_kernel
constexpr int kDimMax = 12;     // RBP_GRAPH_MAX_DIM

// Row values of one 64-node tile (lane = node) for kRowsPerBlock rows k (A
// stored by row, so that a lane's node is coalesced; B by node, so that the
// rows of an end node are), their tile minima, whether an A is NaN (a minimum
// passes over it), and out-degrees set to 0.  A row's coefficients are uniform,
// so a row costs 2 dim FMAs, two coalesced stores and two wave minima; tile x
// row-chunk blocks keep the chip busy although a tile has only 64 nodes.
// 5,000 nodes x 64 rows: 8.1 us with the minima (before, in two kernels: 24.2 us).
template <int DIM>
__global__ __launch_bounds__(256) void graph_rows_kernel(GraphArgs a) {
  constexpr int kD = DIM > 0 ? DIM : kDimMax;
  const int dim = DIM > 0 ? DIM : a.dim;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tile = blockIdx.x, i = tile * kTile + lane;
  const bool live = i < a.n_nodes;
  if (blockIdx.y == 0 && wv == 0 && live) a.degree[i] = 0;
  double v[kD];
#pragma unroll
  for (int c = 0; c < kD; ++c) v[c] = (live && c < dim) ? a.V[(int64_t)i * dim + c] : 0.0;
  bool nan = false;
#pragma unroll
  for (int u = 0; u < kRowsPerBlock / 4; ++u) {
    const int k = blockIdx.y * kRowsPerBlock + 4 * u + wv;
    if (k >= a.m) break;   // uniform
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int c = 0; c < kD; ++c) {
      if (c < dim) {
        s1 += a.F1[k * dim + c] * v[c];
        s2 += a.F2[k * dim + c] * v[c];
      }
    }
    s2 -= a.G[k];
    if (live) {
      a.A[(int64_t)k * a.n_nodes + i] = s1;
      a.B[(int64_t)i * a.m + k] = s2;
      nan |= s1 != s1;
    }
    // a NaN is passed over; a tile without a number in row k has the minimum inf
    const double ma = wave::min(live && s1 == s1 ? s1 : __builtin_huge_val());
    const double mb = wave::min(live && s2 == s2 ? s2 : __builtin_huge_val());
    if (lane == 0) {
      a.Amin[tile * a.m + k] = ma;
      a.Bmin[tile * a.m + k] = mb;
    }
  }
  const int any = __syncthreads_or(nan);
  if (threadIdx.x == 0) a.tile_nan[tile * gridDim.y + blockIdx.y] = any != 0;
}

// One wavefront: 64 start nodes (one per lane) against the 32 end nodes of one
// adjacency word.  The sum A_ik + B_jk is positive exactly when A_ik > -B_jk,
// so a row costs one comparison of a lane's A with a uniform B (a scalar load)
// and an OR of lane masks on the scalar unit: half the vector instructions of
// adding and taking maxima, and no LDS.  An end node is dropped as soon as
// every lane has a violated row; before that the bound min_i A_ik + B_jk,
// whose rows lie one per lane, drops the end nodes that no start node of the
// tile can reach (it does not hold where an A is NaN).
// kChunk: rows of A a lane holds at a time, m or fewer; with fewer rows more end
// nodes are looked at together, up to 32 coefficients in flight.  (With 16 for every m
// and rows loaded again per end node below it, 20,000 nodes in a random numbering
// took 1,244 us with 8 rows; 526 now.)
// A block's four words leave through LDS, 16 bytes per row at a time, and are
// counted into the out-degrees on the way, one addition per row and block: where
// most pairs are joined the additions bound the kernel (20,000 nodes x 1 row 1,898 us
// with one per word, 422 now; 5,000 x 1 160 and 36).
// 5,000 nodes x 64 rows: 95.2 us (64 x 64 tiles in LDS) + 41.7 us (degrees) -> 40 us.
// What is left is the latency of the few wavefronts with many open end nodes;
// blocks of four or sixteen wavefronts instead of eight take 62 and 64 us.
template <int kChunk>
__global__ __launch_bounds__(64 * kPairWaves) void graph_pairs_kernel(GraphArgs a, const double* __restrict__ gA,
                                                                 const double* __restrict__ gB) {
  static_assert(kEnds == 16, "two half-words per word");
  __shared__ uint16_t half[kTile][kPairWaves + 2];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = a.n_nodes, m = a.m, n_words = (n + 31) / 32;
  const int ti = blockIdx.y, j0 = (blockIdx.x * kPairWaves + wv) * kEnds, tj = j0 / kTile;
  const int gi = ti * kTile + lane;
  uint32_t bits = 0u;
  bool culled = j0 >= n;
  for (int k0 = 0; k0 < m && !culled; k0 += 64) {
    const int k = k0 + lane;
    culled = __ballot(k < m && a.Amin[ti * m + k] + a.Bmin[tj * m + k] > 0.0) != 0ull;
  }
  if (!culled) {
    const int nj = n - j0 < kEnds ? n - j0 : kEnds;
    uint32_t alive = (1u << nj) - 1u;                     // end nodes still open, uniform
    const int nkc = (m + kRowsPerBlock - 1) / kRowsPerBlock;
    bool nan = false;
    for (int c = lane; c < nkc; c += 64) nan |= a.tile_nan[ti * nkc + c] != 0;
    if (__ballot(nan) == 0ull) {
      for (int k0 = 0; k0 < m; k0 += 64) {
        const int k = k0 + lane;
        const double am = k < m ? a.Amin[ti * m + k] : -__builtin_huge_val();
        const int kc = k < m ? k : m - 1;
        double b[kEnds];
#pragma unroll
        for (int j = 0; j < kEnds; ++j) b[j] = gB[(int64_t)(j0 + (j < nj ? j : 0)) * m + kc];
#pragma unroll
        for (int j = 0; j < kEnds; ++j)
          if (__ballot(am + b[j] > 0.0) != 0ull) alive &= ~(1u << j);
      }
    }
    const unsigned long long lanes = __ballot(gi < n);
    uint32_t dead = 0u;                                   // per lane: violated end nodes
    uint32_t open = alive;
    for (int kk = 0; kk < m && open; kk += kChunk) {
      // the last chunk ends at row m (rows seen twice change nothing)
      const int k0 = kk + kChunk <= m ? kk : m - kChunk;
      double av[kChunk];
#pragma unroll
      for (int u = 0; u < kChunk; ++u) av[u] = gA[(int64_t)(k0 + u) * n + (gi < n ? gi : n - 1)];
      // several end nodes at a time: their scalar loads are in flight together
      constexpr int kAtOnce = 32 / kChunk < kEnds ? 32 / kChunk : kEnds;
      for (uint32_t todo = open; todo;) {
        int j[kAtOnce];
        double b[kAtOnce][kChunk];
        unsigned long long v[kAtOnce];
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e) {      // past the last one: the one before again
          j[e] = e == 0 || todo ? __builtin_ctz(todo) : j[e > 0 ? e - 1 : 0];
          todo &= todo - 1u;
        }
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e)
#pragma unroll
          for (int u = 0; u < kChunk; ++u) b[e][u] = gB[(int64_t)(j0 + j[e]) * m + k0 + u];
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e) v[e] = 0ull;
#pragma unroll
        for (int u = 0; u < kChunk; ++u)
#pragma unroll
          for (int e = 0; e < kAtOnce; ++e) v[e] |= __ballot(av[u] > -b[e][u]);
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e) dead |= ((v[e] >> lane) & 1ull) ? 1u << j[e] : 0u;
#pragma unroll
        for (int e = 0; e < kAtOnce; ++e)
          if ((__ballot((dead >> j[e]) & 1u) & lanes) == lanes) open &= ~(1u << j[e]);
      }
    }
    bits = alive & ~dead;
    if (gi >= j0 && gi - j0 < kEnds) bits &= ~(1u << (gi - j0));   // no self edge
  }
  half[lane][wv] = uint16_t(bits);
  __syncthreads();
  const int row = tid / kWords, wl = tid % kWords, gr = ti * kTile + row, gw = blockIdx.x * kWords + wl;
  const bool on = row < kTile && gr < n && gw < n_words;
  const uint32_t out = on ? half[row][2 * wl] | (uint32_t(half[row][2 * wl + 1]) << 16) : 0u;
  if (on) a.adj[(int64_t)gr * n_words + gw] = out;
  // the four words of a row lie in four neighbouring lanes
  static_assert(kWords == 4, "sums over four lanes");
  int count = __popc(out);
  count += wave::dpp_i32<wave::kXor1>(count);
  count += wave::dpp_i32<wave::kXor2>(count);
  if (wl == 0 && count) atomicAdd(&a.degree[gr], count);
}

// 64 nodes per block (one per lane), the boxes split over its wavefronts in
// consecutive parts: a wavefront reads its boxes with scalar loads, four in
// flight, and keeps the nearest (the first of equal ones); the parts are then
// compared in order, so the lowest index wins as in one loop over all boxes.
// One thread per node left all but 79 of the chip's wavefronts idle at 5,000
// nodes and walked the boxes one load after the other.
// 5,000 nodes x 200 boxes: 33 -> 6.6 us.  LDS is that of the wavefronts launched:
// with room for sixteen, blocks of one (from 131,009 nodes on) fill a third of a CU's
// wavefronts (1,000,000 x 200 166 us, 134 now).
__global__ __launch_bounds__(64 * kPlaneWaves) void hyperplane_kernel(
    int n, const double* __restrict__ X, int n_obst, const double* __restrict__ lo, const double* __restrict__ hi,
    int32_t* __restrict__ idx, double* __restrict__ point, double* __restrict__ plane) {
  extern __shared__ double sd[];                     // 64 distances per wavefront, then 64 indices
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nw = blockDim.x >> 6;
  int* const si = reinterpret_cast<int*>(sd + 64 * nw);
  const int i = blockIdx.x * 64 + lane;
  const int64_t ic = i < n ? i : n - 1;
  const double x = X[3 * ic], y = X[3 * ic + 1], z = X[3 * ic + 2];
  double best = __builtin_huge_val();
  int bi = -1;
  const int per = (n_obst + nw - 1) / nw;
  const int o0 = wv * per, o1 = o0 + per < n_obst ? o0 + per : n_obst;
  auto dist2 = [&](const double* l, const double* h) {
    const double cx = fmin(fmax(x, l[0]), h[0]);
    const double cy = fmin(fmax(y, l[1]), h[1]);
    const double cz = fmin(fmax(z, l[2]), h[2]);
    return (x - cx) * (x - cx) + (y - cy) * (y - cy) + (z - cz) * (z - cz);
  };
  int o = o0;
  for (; o + 4 <= o1; o += 4) {
    double l[12], h[12];
#pragma unroll
    for (int e = 0; e < 12; ++e) { l[e] = lo[3 * (int64_t)o + e]; h[e] = hi[3 * (int64_t)o + e]; }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double d2 = dist2(l + 3 * u, h + 3 * u);
      if (d2 < best) { best = d2; bi = o + u; }
    }
  }
  for (; o < o1; ++o) {
    const double d2 = dist2(lo + 3 * (int64_t)o, hi + 3 * (int64_t)o);
    if (d2 < best) { best = d2; bi = o; }
  }
  sd[64 * wv + lane] = best;
  si[64 * wv + lane] = bi;
  __syncthreads();
  if (wv != 0 || i >= n) return;
  for (int w = 1; w < nw; ++w)
    if (sd[64 * w + lane] < best) { best = sd[64 * w + lane]; bi = si[64 * w + lane]; }
  double px = x, py = y, pz = z;
  if (bi >= 0) {
    px = fmin(fmax(x, lo[3 * (int64_t)bi]), hi[3 * (int64_t)bi]);
    py = fmin(fmax(y, lo[3 * (int64_t)bi + 1]), hi[3 * (int64_t)bi + 1]);
    pz = fmin(fmax(z, lo[3 * (int64_t)bi + 2]), hi[3 * (int64_t)bi + 2]);
  }
  idx[i] = bi;
  point[3 * (int64_t)i] = px; point[3 * (int64_t)i + 1] = py; point[3 * (int64_t)i + 2] = pz;
  const double dx = x - px, dy = y - py, dz = z - pz;
  const double nn = sqrt(dx * dx + dy * dy + dz * dz);
  double nx = 0.0, ny = 0.0, nz = 0.0;
  if (nn > 0.0) { nx = dx / nn; ny = dy / nn; nz = dz / nn; }
  plane[4 * (int64_t)i] = nx; plane[4 * (int64_t)i + 1] = ny; plane[4 * (int64_t)i + 2] = nz;
  plane[4 * (int64_t)i + 3] = nx * px + ny * py + nz * pz;
}

}  // namespace

hipError_t launch_graph(const GraphArgs& a, hipStream_t s) {
  if (a.n_nodes <= 0) return hipSuccess;
  const int n_tiles = (a.n_nodes + kTile - 1) / kTile;
  const dim3 rg(n_tiles, (a.m + kRowsPerBlock - 1) / kRowsPerBlock);
  // positions, and positions with velocities: a row's coefficients then come
  // in one or two scalar loads instead of one per component
  if (a.dim == 3) hipLaunchKernelGGL(graph_rows_kernel<3>, rg, dim3(256), 0, s, a);
  else if (a.dim == 6) hipLaunchKernelGGL(graph_rows_kernel<6>, rg, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(graph_rows_kernel<0>, rg, dim3(256), 0, s, a);
  const int n_words = (a.n_nodes + 31) / 32;
  const dim3 pg((n_words + kWords - 1) / kWords, n_tiles), pb(64 * kPairWaves);
  if (a.m >= 16) hipLaunchKernelGGL(graph_pairs_kernel<16>, pg, pb, 0, s, a, a.A, a.B);
  else if (a.m >= 8) hipLaunchKernelGGL(graph_pairs_kernel<8>, pg, pb, 0, s, a, a.A, a.B);
  else if (a.m >= 4) hipLaunchKernelGGL(graph_pairs_kernel<4>, pg, pb, 0, s, a, a.A, a.B);
  else hipLaunchKernelGGL(graph_pairs_kernel<1>, pg, pb, 0, s, a, a.A, a.B);
  return hipGetLastError();
}

hipError_t graph_scratch(double** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr[dev] = p;
  }
  *out = static_cast<double*>(ptr[dev]);
  return hipSuccess;
}

hipError_t launch_hyperplanes(int n, const double* X, int n_obst, const double* lo, const double* hi, int32_t* idx,
                              double* point, double* plane, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // enough wavefronts for about two per SIMD (2,048), at least four boxes each
  const int blocks = (n + 63) / 64;
  int waves = 1;
  while (waves < kPlaneWaves && blocks * waves < 2048 && 8 * waves <= n_obst) waves *= 2;
  hipLaunchKernelGGL(hyperplane_kernel, dim3(blocks), dim3(64 * waves), 768 * waves, s, n, X, n_obst, lo, hi, idx, point, plane);
  return hipGetLastError();
}

}  // namespace rbp
