// Batched MPC refinement QP (eq. MPC, Sec. III-D): one workgroup of four
// wavefronts per instance (one for short horizons in large batches), primal-dual
// interior point (Mehrotra predictor-corrector), FP64.
//
// Stage variables z_k = (x_k, u_k), k = 0..N-1, with x = (position, velocity)
// and u = acceleration; x_{k+1} = A x_k + B u_k is the exact discretisation of
// the double integrator over dt.  x_0 = x0 and x_N = r_N are fixed.  Stage
// cost 1/2 z'H z + h'z with h_k = (-2 Q r_k, 0) (no tracking at k = 0), so
// the cost of the problem is the sum plus the constants r_k'Q r_k.  Rows of
// stage k, each scaled to unit norm, c_i'z_k <= d_i: the m reachable rows
// F1 x_k + F2 x_{k+1} <= G (Thm. 2) with x_{k+1} substituted, then four
// keep-out rows n_k . P_j >= l_k on the control points of the cubic that
// joins the two states (Lemma 1), P_j = p + a_j v + b_j u.
//
// Every Newton system is an equality-constrained LQ problem:
//   min sum_k 1/2 dz_k' Ht_k dz_k + g_k' dz_k,  dynamics, dx_0 = 0, dx_N = 0,
// with Ht_k = H_k + sum_i (lam_i / s_i) c_i c_i'.  It is solved by a Riccati
// recursion in Cholesky form (Quu = L L', Y = L^-1 Qux, P = Qxx - Y'Y) with
// the cost-to-go symmetrised at every stage: the plain update
// P = Qxx - Qxu Quu^-1 Qux drifts away from symmetry and loses all accuracy
// once some barrier weights are large.  The terminal state is fixed by
// eliminating the last two stages exactly: [u_{N-2}; u_{N-1}] =
// [AB B]^-1 (-A^2 x_{N-2}), so z_{N-2} = T2 x_{N-2} and z_{N-1} = T1 x_{N-2}.
//
// The dual residual is not carried along: every iteration fits the costates
// (x-stationarity fixes pi_k from pi_{k+1}; pi_N is chosen by least squares)
// and feeds the remaining u-stationarity residual into the Newton system, so
// errors of earlier directions do not accumulate.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rbp_internal.hpp"
#include "rbp_wave.hpp"

namespace rbp {
namespace {

constexpr int kW = 64;
constexpr int kWaves = 4;              // most wavefronts per instance
constexpr int kOneSlots = 4;           // register slots per lane where one wavefront holds every row
constexpr int kRing = 6;               // stages of barrier Hessians per batch of the factorisation
constexpr int kSolved = 0, kInfeasible = 1, kMaxIter = 2, kNumerical = 4, kInvalid = 5;

// LDS carve, in doubles.  The per-row state (slack, multiplier, primal
// residual, Newton weight) lives in registers of the lane that owns the row;
// LDS holds one value per row, X, for the reads that cross lanes: the
// multipliers (dual residual), the barrier weights lam/s (factorisation), the
// Newton weights (gradient build), and meanwhile each row's c'dz for its own
// lane.  The gradient of the LQ solve shares its storage with the direction
// it produces.
struct MpcSm {
  double *prm, *z, *g, *dz, *ref, *pl, *X, *Lc, *Y, *yv, *rho, *P, *tmp;
  // scratch of the factorisation, inside the gradient buffer (free while it runs)
  double *Ht, *Qh, *HtT;
  double *ring;   // 2 x kRing x 45: barrier Hessians of the stages ahead (upper triangles)
  double *part;   // 64: running sums handed from wavefront to wavefront
  double *red;    // 4 per reduction in flight: one value per wavefront
};

// the gradient / direction buffer also holds the factorisation's scratch
// (Ht 81, Qh 81, Ht T 54)
__host__ __device__ inline int mpc_g_doubles(int N) { return 9 * N > 288 ? 9 * N : 288; }

__host__ __device__ inline int mpc_lds_doubles(int N, int m) {
  const MpcLayout L = mpc_param_layout(m);
  const int RT = N * (m + 4);
  return L.total + 9 * N /*z*/ + mpc_g_doubles(N) /*g = dz*/ + 6 * (N + 1) /*ref*/ + 4 * N /*pl*/ +
         RT /*X*/ + 6 * N /*Lc*/ + 18 * N /*Y*/ + 3 * N /*yv*/ + 3 * N /*rho*/ + 36 /*P*/ + 12 /*tmp*/ +
         2 * kRing * 45 /*ring*/ + kW /*part*/ + 2 * kWaves /*red*/;
}

__device__ inline MpcSm carve_mpc(double* base, int N, int m) {
  const MpcLayout L = mpc_param_layout(m);
  const int RT = N * (m + 4);
  MpcSm S;
  double* p = base;
  S.prm = p; p += L.total;
  S.z = p; p += 9 * N;
  S.g = p; S.dz = p;
  S.Ht = p; S.Qh = p + 81; S.HtT = p + 162;
  p += mpc_g_doubles(N);
  S.ref = p; p += 6 * (N + 1);
  S.pl = p; p += 4 * N;
  S.X = p; p += RT;
  S.Lc = p; p += 6 * N;
  S.Y = p; p += 18 * N;
  S.yv = p; p += 3 * N;
  S.rho = p; p += 3 * N;
  S.P = p; p += 36;
  S.tmp = p; p += 12;
  S.ring = p; p += 2 * kRing * 45;
  S.part = p; p += kW;
  S.red = p;
  return S;
}

// tmp layout: [0, 6) start state, [8] factorisation flag
constexpr int kTmpFlag = 8;

// The value of x, opaque to the optimiser: what is derived from it (addresses,
// indices) is formed where it is used, instead of being hoisted out of the
// iteration loop and held in registers throughout.
__device__ __forceinline__ int opq(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Column b of [A B] (6 x 9) has at most two non-zeros: row q0 with weight w0
// and row q1 with weight w1 (q1 < 0: none).
__device__ inline void ab_col(int b, double dt, int& q0, double& w0, int& q1, double& w1) {
  if (b < 3) { q0 = b; w0 = 1.0; q1 = -1; w1 = 0.0; }
  else if (b < 6) { q0 = b; w0 = 1.0; q1 = b - 3; w1 = dt; }
  else { q0 = b - 3; w0 = dt; q1 = b - 6; w1 = 0.5 * dt * dt; }
}

// 1/sqrt(x) and a / b from the hardware approximations (v_rsq_f64, v_rcp_f64)
// refined by Newton steps to full double precision: the chains of a
// factorisation stage and the per-row weights stay short.  x, b > 0 here
// (a non-positive pivot is caught by the caller).
__device__ inline double rsqrt_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  r = r * fma(-hx * r, r, 1.5);
  r = r * fma(-hx * r, r, 1.5);
  return r;
}
__device__ inline double div_nr(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  r = fma(fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ double uni(double x) { return wave::bcast(x, 0); }

// W: wavefronts per instance (1 or kWaves)
template <int W>
struct MpcCtx {
  static constexpr int kT = kW * W;
  const MpcArgs& A;
  MpcSm S;
  MpcLayout Ly;
  int N, m, mr, RT, lane, wv, tid;
  double dt;
  int ua, ub;          // upper-triangle entry (ua <= ub) of a 9 x 9 matrix owned by lanes < 45
  int spw;             // passes of reachable rows per wavefront
  double h2, a11, a12, a22, det;   // dt^2 / 2; normal equations of the terminal costate (the same every time)
  int pa, pb;          // upper-triangle entry (pa <= pb) of the 6 x 6 cost-to-go owned by lanes < 21
  int pidx[4];         // entries of the cost-to-go in entry (ua, ub) of [A B]' P [A B], and their weights
  double pw[4];

  __device__ __forceinline__ void init_lane() {
    h2 = uni(0.5 * dt * dt);
    double s11 = 0.0, s12 = 0.0;
    for (int k = 0; k < N; ++k) {
      const double al = dt * dt * (N - k - 0.5);
      s11 += al * al;
      s12 += dt * al;
    }
    a11 = uni(s11);
    a12 = uni(s12);
    a22 = uni(N * dt * dt);
    det = uni(a11 * a22 - a12 * a12);
    ua = 0;
    int t = lane < 45 ? lane : 0;
    while (t >= 9 - ua) { t -= 9 - ua; ++ua; }
    ub = ua + t;
    pa = 0;
    t = lane < 21 ? lane : 0;
    while (t >= 6 - pa) { t -= 6 - pa; ++pa; }
    pb = pa + t;
    int qa[2], qb[2];
    double wa[2], wb[2];
    ab_col(ua, dt, qa[0], wa[0], qa[1], wa[1]);
    ab_col(ub, dt, qb[0], wb[0], qb[1], wb[1]);
    if (qa[1] < 0) qa[1] = qa[0];
    if (qb[1] < 0) qb[1] = qb[0];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int lo = qa[i] < qb[j] ? qa[i] : qb[j], hi = qa[i] < qb[j] ? qb[j] : qa[i];
        pidx[2 * i + j] = 6 * lo + hi;
        pw[2 * i + j] = wa[i] * wb[j];
      }
  }

  // orders LDS accesses between the lanes of this wavefront only (its LDS
  // operations execute in program order)
  __device__ __forceinline__ void wsync() const {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  // largest / smallest value over the instance's wavefronts
  __device__ __forceinline__ double bmax(double v) const {
    v = wave::max(v);
    if constexpr (W > 1) {
      if (lane == 0) S.red[wv] = v;
      __syncthreads();
      v = fmax(fmax(S.red[0], S.red[1]), fmax(S.red[2], S.red[3]));
    }
    __syncthreads();
    return uni(v);
  }
  __device__ __forceinline__ double bmin(double v) const { return -bmax(-v); }
  __device__ __forceinline__ void bmax2(double& a, double& b) const {
    a = wave::max(a);
    b = wave::max(b);
    if constexpr (W > 1) {
      if (lane == 0) { S.red[wv] = a; S.red[kWaves + wv] = b; }
      __syncthreads();
      a = fmax(fmax(S.red[0], S.red[1]), fmax(S.red[2], S.red[3]));
      b = fmax(fmax(S.red[4], S.red[5]), fmax(S.red[6], S.red[7]));
    }
    __syncthreads();
  }
  // Sum over the rows: add(acc) continues a lane's running sum over the rows
  // its wavefront holds, in order; the wavefronts take turns, so that the
  // order is that of one wavefront walking every slot (how far an unsolvable
  // horizon gets depends on the last bits of these sums).  The sums are written as
  // fma: of two products added in registers the compiler may round either.
  template <typename F>
  __device__ __forceinline__ double chain_sum(F&& add) const {
    double v;
    if constexpr (W > 1) {
      for (int w = 0; w < W; ++w) {
        if (wv == w) S.part[lane] = add(w == 0 ? 0.0 : S.part[lane]);
        __syncthreads();
      }
      v = wave::sum(S.part[lane]);
    } else {
      v = wave::sum(add(0.0));
    }
    __syncthreads();
    return uni(v);
  }

  // component a of C_k' w for per-row weights w (rows of stage k at w[0..mr))
  __device__ __forceinline__ double ct_times(int k, int a, const double* w) const {
    const double* c = S.prm + Ly.Cr + a * Ly.cs;
    double t = 0.0, t1 = 0.0;
    int i = 0;
    const int m8 = m & ~7;
    for (; i < m8; i += 4) {             // loads of four rows issued together
      double x[4], y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { x[q] = c[i + q]; y[q] = w[i + q]; }
#pragma unroll
      for (int q = 0; q < 4; q += 2) {
        t += x[q] * y[q];
        t1 += x[q + 1] * y[q + 1];
      }
    }
    for (; i < m; ++i) t += c[i] * w[i];
    t += t1;
    const double* f = S.prm + Ly.pf + a / 3;
    const double tp = f[0] * w[m] + f[3] * w[m + 1] + f[6] * w[m + 2] + f[9] * w[m + 3];
    return t - S.pl[4 * k + a % 3] * tp;
  }
  __device__ __forceinline__ const double* Hk(int k) const { return S.prm + (k == 0 ? Ly.H0 : Ly.H1); }
  // x-part of h_k: -2 Q r_k (k >= 1)
  __device__ __forceinline__ double hk(int k, int a) const {
    if (k == 0 || a >= 6) return 0.0;
    double v = 0.0;
    for (int b = 0; b < 6; ++b) v += S.prm[Ly.Qm + 6 * a + b] * S.ref[6 * k + b];
    return -2.0 * v;
  }

  // upper entry (ua, ub) of Ht_k = H_k + sum_i sigma_i c_i c_i', with the
  // barrier weights sigma of stage k's rows in S.X
  __device__ __forceinline__ double ht_entry(int k) const {
    const int ua = opq(this->ua), ub = opq(this->ub);
    const double* sg = S.X + k * mr;
    const double* ca = S.prm + Ly.Cr + ua * Ly.cs;
    const double* cb = S.prm + Ly.Cr + ub * Ly.cs;
    double v = Hk(k)[9 * ua + ub], v1 = 0.0;
    int i = 0;
    const int m8 = m & ~7;
    for (; i < m8; i += 4) {             // loads of four rows issued together
      double w[4], x[4], y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) { w[q] = sg[i + q]; x[q] = ca[i + q]; y[q] = cb[i + q]; }
#pragma unroll
      for (int q = 0; q < 4; q += 2) {
        v += w[q] * x[q] * y[q];
        v1 += w[q + 1] * x[q + 1] * y[q + 1];
      }
    }
    for (; i < m; ++i) v += sg[i] * ca[i] * cb[i];
    v += v1;
    asm volatile("" : "+v"(v) : : "memory");   // the plane rows' operands are not held across the rows
    const double* fa = S.prm + Ly.pf + ua / 3;
    const double* fb = S.prm + Ly.pf + ub / 3;
    const double s0 = sg[m], s1 = sg[m + 1], s2 = sg[m + 2], s3 = sg[m + 3];
    const double fa0 = fa[0], fa3 = fa[3], fa6 = fa[6], fa9 = fa[9];
    const double fb0 = fb[0], fb3 = fb[3], fb6 = fb[6], fb9 = fb[9];
    const double pla = S.pl[4 * k + ua % 3], plb = S.pl[4 * k + ub % 3];
    const double tp = s0 * fa0 * fb0 + s1 * fa3 * fb3 + s2 * fa6 * fb6 + s3 * fa9 * fb9;
    return v + pla * plb * tp;
  }

  // Riccati factorisation of the Newton LQ with the barrier weights in S.X
  // (zero weights: H_k alone).  Returns false (uniformly) when a pivot of
  // some Quu is not positive.
  __device__ __forceinline__ bool factor() {
    // The barrier Hessians do not depend on the recursion: they are formed
    // kRing stages at a time, the first batch by every wavefront, each next one
    // by wavefronts 1..3 while wavefront 0 runs the recursion over the batch
    // before it (one wavefront alone takes them in turn).
    auto batch = [&](int b, int first) {       // stages N-1 - kRing b, going down
      for (int u = wv - first; u < kRing; u += W - first) {
        const int k = N - 1 - (kRing * b + u);
        if (u >= 0 && k >= 0 && lane < 45) S.ring[((b & 1) * kRing + u) * 45 + lane] = ht_entry(k);
      }
    };
    if (tid == 0) S.tmp[kTmpFlag] = 0.0;
    batch(0, 0);
    __syncthreads();
    const int nb = (N + kRing - 1) / kRing;
    for (int b = 0; b < nb; ++b) {
      if (wv == 0) {
        const double* ring = S.ring + (b & 1) * kRing * 45;
        if (b == 0) terminal(ring);
        for (int u = b == 0 ? 2 : 0; u < kRing; ++u) {
          const int k = N - 1 - (kRing * b + u);
          if (k < 0) break;
          stage(k, ring + u * 45);
        }
      }
      if ((W == 1 || wv > 0) && b + 1 < nb) batch(b + 1, W > 1 ? 1 : 0);
      __syncthreads();
    }
    return S.tmp[kTmpFlag] == 0.0;
  }

  // terminal block (wavefront 0): P = T2' Ht_{N-2} T2 + T1' Ht_{N-1} T1
  __device__ __forceinline__ void terminal(const double* ring) {
    const int lane = opq(this->lane), ua = opq(this->ua), ub = opq(this->ub);
    for (int e = lane; e < 36; e += kW) S.P[e] = 0.0;
    for (int t = 0; t < 2; ++t) {
      const double* T = S.prm + (t == 0 ? Ly.T2 : Ly.T1);
      if (lane < 45) {
        const double v = ring[(1 - t) * 45 + lane];
        S.Ht[9 * ua + ub] = v;
        S.Ht[9 * ub + ua] = v;
      }
      wsync();
      // Ht T (9 x 6)
      for (int e = lane; e < 54; e += kW) {
        const int a = e / 6, c = e - 6 * (e / 6);
        double v = 0.0;
        for (int b = 0; b < 9; ++b) v += S.Ht[9 * a + b] * T[6 * b + c];
        S.HtT[e] = v;
      }
      wsync();
      for (int e = lane; e < 36; e += kW) {
        const int c = e / 6, d = e - 6 * (e / 6);
        double v = 0.0;
        for (int a = 0; a < 9; ++a) v += T[6 * a + c] * S.HtT[6 * a + d];
        S.P[e] += v;
      }
      wsync();
    }
    for (int e = lane; e < 36; e += kW) {
      const int a = e / 6, b = e - 6 * (e / 6);
      if (a < b) {
        const double v = 0.5 * (S.P[e] + S.P[6 * b + a]);
        S.P[e] = v; S.P[6 * b + a] = v;
      }
    }
    wsync();
  }

  // one stage of the recursion (wavefront 0), with the stage's barrier Hessian
  __device__ __forceinline__ void stage(int k, const double* ht) {
    const int lane = opq(this->lane), pa = opq(this->pa), pb = opq(this->pb), ua = opq(this->ua), ub = opq(this->ub);
    // Qh = Ht + [A B]' P [A B] (symmetric: lanes own the upper triangle; the
    // four entries of P and their weights are the lane's own, see pidx, pw;
    // absent terms have weight 0 and load a valid entry)
    double vq = 0.0;
    if (lane < 45) {
      const double p00 = S.P[pidx[0]], p01 = S.P[pidx[1]], p10 = S.P[pidx[2]], p11 = S.P[pidx[3]];
      const double h = ht[lane];
      double v = pw[0] * p00;
      v += pw[1] * p01;
      v += pw[2] * p10;
      v += pw[3] * p11;
      v += h;
      vq = v;
      S.Qh[ub >= 6 ? 9 * ub + ua : 9 * ua + ub] = v;   // where it is read below
    }
    // the entries of Quu come straight from their lanes (39..44), so that the
    // pivots do not wait for the other entries' way through LDS
    const double q60 = wave::bcast(vq, 39), q69 = wave::bcast(vq, 40), q78 = wave::bcast(vq, 41),
                 q70 = wave::bcast(vq, 42), q79 = wave::bcast(vq, 43), q80 = wave::bcast(vq, 44);
    wsync();
    // Quu = L L' and the columns of Y = L^-1 Qux that entry (a, b) of the
    // next cost-to-go P = Qxx - Y'Y needs, all in the lane of that entry
    // (lanes < 21); lanes 0..5 (entries (0, c)) store column c of Y, lane 0
    // stores L as (1/l00, l10, 1/l11, l20, l21, 1/l22).
    if (lane < 21) {
      const int a = pa, b = pb;
      // every entry this lane reads, loaded before the pivot chain starts
      const double qa0 = S.Qh[54 + a], qa1 = S.Qh[63 + a], qa2 = S.Qh[72 + a];
      const double qb0 = S.Qh[54 + b], qb1 = S.Qh[63 + b], qb2 = S.Qh[72 + b];
      const double qab = S.Qh[9 * a + b];
      const double d0 = q60;
      const double i00 = rsqrt_nr(d0);
      const double l10 = q69 * i00, l20 = q78 * i00;
      const double d1 = q70 - l10 * l10;
      const double i11 = rsqrt_nr(d1);
      const double l21 = (q79 - l20 * l10) * i11;
      const double d2 = q80 - l20 * l20 - l21 * l21;
      const double i22 = rsqrt_nr(d2);
      const double ya0 = qa0 * i00;
      const double ya1 = (qa1 - l10 * ya0) * i11;
      const double ya2 = (qa2 - l20 * ya0 - l21 * ya1) * i22;
      const double yb0 = qb0 * i00;
      const double yb1 = (qb1 - l10 * yb0) * i11;
      const double yb2 = (qb2 - l20 * yb0 - l21 * yb1) * i22;
      if (lane < 6) {
        double* Y = S.Y + 18 * k;
        Y[b] = yb0; Y[6 + b] = yb1; Y[12 + b] = yb2;
      }
      if (lane == 0) {
        double* L = S.Lc + 6 * k;
        L[0] = i00; L[1] = l10; L[2] = i11; L[3] = l20; L[4] = l21; L[5] = i22;
        if (!(d0 > 0.0 && d1 > 0.0 && d2 > 0.0) || !isfinite(i00 * i11 * i22)) S.tmp[kTmpFlag] = 1.0;
      }
      if (k > 0) {
        S.P[6 * a + b] = qab - (ya0 * yb0 + ya1 * yb1 + ya2 * yb2);   // a <= b: the upper triangle is read
      }
    }
    wsync();
  }

  // Solve the factorised LQ for the gradients in S.g; the direction replaces
  // them (S.dz aliases S.g: the backward sweep reads every g_k before the
  // forward sweep writes dz_k).  Sequential over stages in wavefront 0, each
  // stage's operands loaded while the stage before it is worked on.
  __device__ __forceinline__ void lq_solve() {
    if (wv == 0) {
      const int lane = opq(this->lane);
      const double* T2 = S.prm + Ly.T2;
      const double* T1 = S.prm + Ly.T1;
      // backward sweep, one costate component per lane: lane c < 6 holds p_c;
      // the u-part of [A B]'p needs p_{c+3} and the x-part p_{c-3}, both a DPP
      // row shift by three lanes away, and y = L^-1 qu takes qu from lanes 0..2
      {
        const int c = lane < 6 ? lane : 5;
        const int cu = lane < 3 ? lane : 2;
        double pc = 0.0;
        for (int a = 0; a < 9; ++a) pc += T2[6 * a + c] * S.g[9 * (N - 2) + a] + T1[6 * a + c] * S.g[9 * (N - 1) + a];
        struct Ops { double gx, gu, Y[3], L[6]; };
        auto fetch = [&](int k, Ops& b) {
          const int kc = k >= 0 ? k : 0;
          b.gx = S.g[9 * kc + c]; b.gu = S.g[9 * kc + 6 + cu];
#pragma unroll
          for (int e = 0; e < 3; ++e) b.Y[e] = S.Y[18 * kc + 6 * e + c];
#pragma unroll
          for (int e = 0; e < 6; ++e) b.L[e] = S.Lc[6 * kc + e];
        };
        auto step = [&](int k, const Ops& b) {
          const double p_up = wave::dpp_f64<0x103>(pc);     // p_{c+3}
          const double p_dn = wave::dpp_f64<0x113>(pc);     // p_{c-3}
          // qh = g + [A B]' p
          const double qx = lane < 3 ? b.gx + pc : b.gx + dt * p_dn + pc;
          const double qu = b.gu + h2 * pc + dt * p_up;
          const double qu0 = wave::bcast(qu, 0), qu1 = wave::bcast(qu, 1), qu2 = wave::bcast(qu, 2);
          const double y0 = qu0 * b.L[0];
          const double y1 = (qu1 - b.L[1] * y0) * b.L[2];
          const double y2 = (qu2 - b.L[3] * y0 - b.L[4] * y1) * b.L[5];
          if (lane < 3) S.yv[3 * k + lane] = lane == 0 ? y0 : (lane == 1 ? y1 : y2);
          pc = qx - (b.Y[0] * y0 + b.Y[1] * y1 + b.Y[2] * y2);
        };
        Ops b0, b1;
        fetch(N - 3, b0);
        for (int k = N - 3; k >= 0; k -= 2) {
          fetch(k - 1, b1);
          step(k, b0);
          if (k == 0) break;
          fetch(k - 2, b0);
          step(k - 1, b1);
        }
      }
      wsync();
      // forward from dx_0 = 0: du = -L^-T (Y dx + y).  Lane i < 3 forms entry i
      // of Y dx + y; the rest of a stage is the same in every lane, lane 0
      // writes it.
      {
        const int i = lane < 3 ? lane : 2;
        double dx[6] = {0, 0, 0, 0, 0, 0};
        struct Ops { double Y[6], y; };
        auto fetch = [&](int k, Ops& b) {
          const int kc = k <= N - 3 ? k : 0;
#pragma unroll
          for (int e = 0; e < 6; ++e) b.Y[e] = S.Y[18 * kc + 6 * i + e];
          b.y = S.yv[3 * kc + i];
        };
        auto step = [&](int k, const Ops& b) {
          double v = b.y, Lk[6];
#pragma unroll
          for (int e = 0; e < 6; ++e) Lk[e] = S.Lc[6 * k + e];   // arrives during the products
#pragma unroll
          for (int c = 0; c < 6; ++c) v += b.Y[c] * dx[c];
          const double r[3] = {wave::bcast(v, 0), wave::bcast(v, 1), wave::bcast(v, 2)};
          const double u2 = -r[2] * Lk[5];
          const double u1 = -(r[1] + Lk[4] * u2) * Lk[2];
          const double u0 = -(r[0] + Lk[1] * u1 + Lk[3] * u2) * Lk[0];
          if (lane == 0) {
            double* d = S.dz + 9 * k;
#pragma unroll
            for (int c = 0; c < 6; ++c) d[c] = dx[c];
            d[6] = u0; d[7] = u1; d[8] = u2;
          }
          const double uu[3] = {u0, u1, u2};
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const double pn = dx[c] + dt * dx[3 + c] + h2 * uu[c];
            dx[3 + c] = dx[3 + c] + dt * uu[c];
            dx[c] = pn;
          }
        };
        if (N >= 3) {
          Ops b0, b1;
          fetch(0, b0);
          for (int k = 0; k <= N - 3; k += 2) {
            fetch(k + 1, b1);
            step(k, b0);
            if (k + 1 > N - 3) break;
            fetch(k + 2, b0);
            step(k + 1, b1);
          }
        }
        if (lane < 9) {
          double v2 = 0.0, v1 = 0.0;
#pragma unroll
          for (int c = 0; c < 6; ++c) { v2 += T2[6 * lane + c] * dx[c]; v1 += T1[6 * lane + c] * dx[c]; }
          S.dz[9 * (N - 2) + lane] = v2;
          S.dz[9 * (N - 1) + lane] = v1;
        }
      }
    }
    __syncthreads();
  }

  // visit the rows of this wavefront: f(slot, r, c'z_k, c'dz_k, d, e) with
  // right-hand side d e (a product that the caller's FMAs take unrounded).
  // Wavefronts 0..2 share the reachable rows (coefficient table): with row t in
  // lane t % 64 of pass t / 64, each takes spw consecutive passes; wavefront 3
  // holds the plane rows.  (One wavefront alone takes the plane rows after its
  // spw passes.)  The loops are unrolled, so slot is a constant
  // wherever f indexes a register array with it.  c'z and c'dz are formed only
  // when CZ / CD ask for them.
  template <int NS, bool CZ, bool CD, typename F>
  __device__ __forceinline__ void for_rows(F&& f) const {
    // the lane index is made opaque here, so the per-slot row indices and
    // addresses are recomputed in every pass instead of being hoisted out of
    // the iteration loop (where they would hold registers throughout)
    const int ln = opq(lane);
    const int mm = m > 0 ? m : 1, rq = kW / mm, rr = kW - rq * mm, t0 = ln + kW * (wv * spw);
    int kr = t0 / mm, ir = t0 - mm * kr;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      bool on;
      int r = 0;
      double cz = 0.0, cd = 0.0, d = 0.0, de = 1.0;
      if (W > 1 ? wv < W - 1 : j < spw) {
        on = j < spw && t0 + kW * j < N * m;
        if (on) {
          const double* c = S.prm + Ly.Cr + ir;
          const double* zk = S.z + 9 * kr;
          const double* dk = S.dz + 9 * kr;
#pragma unroll
          for (int a = 0; a < 9; ++a) {
            const double ca = c[a * Ly.cs];
            if (CZ) cz += ca * zk[a];
            if (CD) cd += ca * dk[a];
          }
          r = kr * mr + ir;
          d = S.prm[Ly.dr + ir];
        }
        kr += rq;
        ir += rr;
        if (ir >= mm) { ir -= mm; ++kr; }
      } else {
        const int t = ln + kW * (W > 1 ? j : j - spw);
        on = (W == 1 || j < 4) && t < 4 * N;
        if (on) {
          const int k = t >> 2, jj = t & 3;
          const double* f3 = S.prm + Ly.pf + 3 * jj;
          const double* n = S.pl + 4 * k;
          const double* zk = S.z + 9 * k;
          const double* dk = S.dz + 9 * k;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if (CZ) cz += n[c] * (f3[0] * zk[c] + f3[1] * zk[3 + c] + f3[2] * zk[6 + c]);
            if (CD) cd += n[c] * (f3[0] * dk[c] + f3[1] * dk[3 + c] + f3[2] * dk[6 + c]);
          }
          cz = -cz;
          cd = -cd;
          r = k * mr + m + jj;
          d = -n[3];
          de = f3[0];
        }
      }
      if (on) f(j, r, cz, cd, d, de);
    }
  }

  // the same slots without the rows' values
  template <int NS, typename F>
  __device__ __forceinline__ void for_slots(F&& f) const {
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const bool on = (W > 1 ? wv < W - 1 : j < spw)
                          ? (j < spw && lane + kW * (wv * spw + j) < N * m)
                          : ((W == 1 || j < 4) && lane + kW * (W > 1 ? j : j - spw) < 4 * N);
      if (on) f(j);
    }
  }

  // g_k = [0; rho_k] + C_k' w, with the per-row weights in S.X
  __device__ __forceinline__ void build_g() {
    const int tid = opq(this->tid);
    for (int e = tid; e < 9 * N; e += kT) {
      const int k = e / 9, a = e - 9 * (e / 9);
      const double v = a >= 6 ? S.rho[3 * k + a - 6] : 0.0;
      S.g[e] = v + ct_times(k, a, S.X + k * mr);
    }
    __syncthreads();
  }

  // least-squares costates and the u-stationarity residual rho_k (into
  // S.rho), with the multipliers in S.X; returns max |rho| and the scale of
  // the gradient terms.  kCost = false leaves the cost out: rho is then the
  // gradient in the inputs of sum_i w_i c_i'z + pi'x_N along trajectories of
  // the dynamics from x0, with the terminal costate pi (returned in pi6 when
  // given) chosen by least squares.
  template <bool kCost = true>
  __device__ __forceinline__ void dual_residual(double& rmax, double& gscale, double* pi6 = nullptr) {
    const int lane = opq(this->lane), tid = opq(this->tid);
    double gs = 0.0;
    for (int e = tid; e < 9 * N; e += kT) {
      const int k = e / 9, a = e - 9 * (e / 9);
      double hz = 0.0;
      if constexpr (kCost) {
        const double* H = Hk(k);
        hz = hk(k, a);
        for (int b = 0; b < 9; ++b) hz += H[9 * a + b] * S.z[9 * k + b];
        asm volatile("" : "+v"(hz) : : "memory");   // its operands are not held across the rows
      }
      const double ct = ct_times(k, a, S.X + k * mr);
      S.g[e] = hz + ct;
      gs = fmax(gs, fmax(fabs(hz), fabs(ct)));
    }
    gscale = bmax(gs);
    // backward: f_k = e_k + B' sig_{k+1};  sig_k = c_k + A' sig_{k+1} (k >= 1).
    // The axes do not mix: lane c < 3 carries (sig_p,c, sig_v,c), with each
    // stage's three gradient entries loaded two stages ahead
    if (tid < 3) {
      const int c = lane;
      double sp_ = 0.0, sv_ = 0.0;
      auto fetch = [&](int k, double& gp, double& gv, double& gu) {
        const int kc = k < 0 ? 0 : k;
        gp = S.g[9 * kc + c]; gv = S.g[9 * kc + 3 + c]; gu = S.g[9 * kc + 6 + c];
      };
      auto stage = [&](int k, double gp, double gv, double gu) {
        S.rho[3 * k + c] = gu + h2 * sp_ + dt * sv_;
        if (k >= 1) {
          const double sp = gp + sp_;
          sv_ = gv + dt * sp_ + sv_;
          sp_ = sp;
        }
      };
      double pA, vA, uA, pB, vB, uB;
      fetch(N - 1, pA, vA, uA);
      fetch(N - 2, pB, vB, uB);
      int k = N - 1;
      for (; k - 1 >= 0; k -= 2) {
        double pC, vC, uC, pD, vD, uD;
        fetch(k - 2, pC, vC, uC);
        fetch(k - 3, pD, vD, uD);
        stage(k, pA, vA, uA);
        stage(k - 1, pB, vB, uB);
        pA = pC; vA = vC; uA = uC; pB = pD; vB = vD; uB = uD;
      }
      if (k >= 0) stage(k, pA, vA, uA);
    }
    __syncthreads();
    // rho_k,c = f_k,c + al_k pi_p,c + dt pi_v,c, al_k = dt^2 (N - k - 1/2);
    // pi_N minimises sum_k |rho_k|^2 (per coordinate, 2 x 2 normal equations)
    double s_af = 0.0, s_f = 0.0;
    const int c = lane % 3;
    for (int k = lane / 3; k < N && lane < 63; k += 21) {
      const double al = dt * dt * (N - k - 0.5);
      s_af += al * S.rho[3 * k + c];
      s_f += S.rho[3 * k + c];
    }
    // per-coordinate sums: lanes with the same lane % 3
    double t_af[3], t_f[3];
    for (int cc = 0; cc < 3; ++cc) {
      t_af[cc] = wave::sum((c == cc && lane < 63) ? s_af : 0.0);
      t_f[cc] = wave::sum((c == cc && lane < 63) ? s_f : 0.0);
    }
    double pp[3], pv[3];
    for (int cc = 0; cc < 3; ++cc) {
      const double b1 = -t_af[cc], b2 = -dt * t_f[cc];
      pp[cc] = (a22 * b1 - a12 * b2) / det;
      pv[cc] = (a11 * b2 - a12 * b1) / det;
    }
    if (pi6) {
      for (int cc = 0; cc < 3; ++cc) { pi6[cc] = pp[cc]; pi6[3 + cc] = pv[cc]; }
    }
    __syncthreads();
    double rm = 0.0;
    for (int e = tid; e < 3 * N; e += kT) {
      const int k = e / 3, cc = e - 3 * (e / 3);
      const double al = dt * dt * (N - k - 0.5);
      const double ppc = cc == 0 ? pp[0] : (cc == 1 ? pp[1] : pp[2]);
      const double pvc = cc == 0 ? pv[0] : (cc == 1 ? pv[1] : pv[2]);
      const double v = S.rho[e] + al * ppc + dt * pvc;
      S.rho[e] = v;
      rm = fmax(rm, fabs(v));
    }
    rmax = bmax(rm);
  }
};

// Four wavefronts per instance.  The recursions over the stages are a serial
// chain and stay in wavefront 0, at the latency of a few LDS round trips per
// stage; everything beside them is spread over the others: the barrier
// Hessians of the stages ahead, the rows (each wavefront holds its own in
// registers), the gradients.  One wavefront doing all of it in turn left a
// SIMD's vector unit 71 % idle and could not hide its own waits: LDS (40 KB
// per instance) allows four instances per CU, so one wavefront each is one per
// SIMD.  Arithmetic and summation order are those of one wavefront, bit for bit.
// 16 horizons of 50 steps, 16 reachable rows: 2.07 -> 1.19 ms; 4,096: 11.1 -> 8.1 ms.
// Registers for three wavefronts per SIMD (149; at 128, for four, it spills and
// takes 8.4 ms); the kernel for more rows per lane needs 186.
// NS: register slots per lane (reachable passes per wavefront, at least the
// four of the plane rows; with W = 1 passes of reachable and of plane rows)
template <int NS, int W>
__global__ __launch_bounds__(kW * W) __attribute__((amdgpu_waves_per_eu(NS <= 5 ? 3 : 2))) void mpc_kernel(MpcArgs A) {
  constexpr int kT = kW * W;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int inst = blockIdx.x;
  if (inst >= A.n) return;
  const int N = A.N, m = A.m, mr = m + 4, RT = N * mr, tid = threadIdx.x, lane = tid & (kW - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  MpcCtx<W> C{A, carve_mpc(reinterpret_cast<double*>(smem_raw), N, m), mpc_param_layout(m), N, m, mr, RT, lane, wv, tid,
           A.dt};
  C.spw = W > 1 ? ((N * m + kW - 1) / kW + W - 2) / (W - 1) : (N * m + kW - 1) / kW;
  C.init_lane();
  MpcSm& S = C.S;
  const MpcLayout& Ly = C.Ly;
  const double dt = A.dt;

  // ---- load
  for (int e = tid; e < Ly.total; e += kT) S.prm[e] = A.params[e];
  bool bad = false;
  for (int e = tid; e < 6 * (N + 1); e += kT) {
    const double v = A.ref[(int64_t)inst * 6 * (N + 1) + e];
    S.ref[e] = v;
    bad |= !isfinite(v);
  }
  for (int k = tid; k < N; k += kT) {
    const double* q = A.planes + ((int64_t)inst * N + k) * 4;
    const double nn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
    bad |= !(nn > 0.0) || !isfinite(nn) || !isfinite(q[3]);
    const double in = nn > 0.0 ? 1.0 / nn : 0.0;
    S.pl[4 * k] = q[0] * in; S.pl[4 * k + 1] = q[1] * in; S.pl[4 * k + 2] = q[2] * in; S.pl[4 * k + 3] = q[3] * in;
  }
  double* x0 = S.tmp;          // start state, read with lane-dependent indices
  if (tid < 6) S.tmp[lane] = A.x0[6 * (int64_t)inst + lane];
  __syncthreads();
  for (int c = 0; c < 6; ++c) bad |= !isfinite(x0[c]);
  auto finish_nan = [&](int status, int its) {
    for (int e = tid; e < 6 * (N + 1); e += kT) A.X[(int64_t)inst * 6 * (N + 1) + e] = __builtin_nan("");
    for (int e = tid; e < 3 * N; e += kT) A.U[(int64_t)inst * 3 * N + e] = __builtin_nan("");
    if (tid == 0) {
      A.cost[inst] = __builtin_nan("");
      A.status[inst] = status;
      A.kkt[inst] = __builtin_nan("");
      if (A.iters) A.iters[inst] = its;
    }
  };
  if (__syncthreads_or(bad)) { finish_nan(kInvalid, 0); return; }

  // ---- start point: zero input up to x_{N-2}, then the two inputs that
  // reach r_N; then the Newton step of the LQ without rows (its optimum)
  for (int e = tid; e < 9 * (N - 2); e += kT) {
    const int k = e / 9, a = e - 9 * (e / 9);
    double v;
    if (a < 3) v = x0[a] + k * dt * x0[3 + a];
    else if (a < 6) v = x0[a];
    else v = 0.0;
    S.z[e] = v;
  }
  if (tid == 0) {
    double xa[6];
    for (int c = 0; c < 3; ++c) { xa[c] = x0[c] + (N - 2) * dt * x0[3 + c]; xa[3 + c] = x0[3 + c]; }
    // rhs = r_N - A^2 x_{N-2}
    double rr[6];
    for (int c = 0; c < 3; ++c) {
      rr[c] = S.ref[6 * N + c] - (xa[c] + 2.0 * dt * xa[3 + c]);
      rr[3 + c] = S.ref[6 * N + 3 + c] - xa[3 + c];
    }
    double uu[6];
    for (int i = 0; i < 6; ++i) {
      double v = 0.0;
      for (int c = 0; c < 6; ++c) v += S.prm[Ly.Mi + 6 * i + c] * rr[c];
      uu[i] = v;
    }
    double* z2 = S.z + 9 * (N - 2);
    double* z1 = S.z + 9 * (N - 1);
    for (int c = 0; c < 6; ++c) z2[c] = xa[c];
    for (int c = 0; c < 3; ++c) {
      z2[6 + c] = uu[c];
      z1[c] = xa[c] + dt * xa[3 + c] + 0.5 * dt * dt * uu[c];
      z1[3 + c] = xa[3 + c] + dt * uu[c];
      z1[6 + c] = uu[3 + c];
    }
  }
  for (int e = tid; e < RT; e += kT) S.X[e] = 0.0;     // no rows yet
  __syncthreads();
  C.factor();
  // g = H z + h
  for (int e = tid; e < 9 * N; e += kT) {
    const int k = e / 9, a = e - 9 * (e / 9);
    const double* H = C.Hk(k);
    double v = C.hk(k, a);
    for (int b = 0; b < 9; ++b) v += H[9 * a + b] * S.z[9 * k + b];
    S.g[e] = v;
  }
  __syncthreads();
  C.lq_solve();
  for (int e = tid; e < 9 * N; e += kT) S.z[e] += S.dz[e];
  __syncthreads();
  // slacks and multipliers; per row, in registers of the owning lane: slack
  // s, multiplier l and primal residual rp = c'z + s - d
  double rs[NS], rl[NS], rp[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) { rs[j] = 1.0; rl[j] = 1.0; rp[j] = 0.0; }
  C.template for_rows<NS, true, false>([&](int j, int r, double cz, double, double d, double de) {
    rs[j] = fmax(fma(d, de, -cz), 1.0);
    S.X[r] = 1.0;
  });
  __syncthreads();

  // ---- interior-point iterations
  int it = 0;
  bool converged = false;
  double mu = 0.0, rpmax = 0.0, rdmax = 0.0, gscale = 0.0;
  for (;; ++it) {
    C.dual_residual(rdmax, gscale);             // multipliers in S.X
    double rpm = 0.0;
    C.template for_rows<NS, true, false>([&](int j, int r, double cz, double, double d, double de) {
      const double v = fma(-d, de, cz + rs[j]);
      rp[j] = v;
      rpm = fmax(rpm, fabs(v));
      S.X[r] = div_nr(rl[j], rs[j]);            // barrier weight for the factorisation
    });
    __syncthreads();
    mu = C.chain_sum([&](double acc) {
      C.template for_slots<NS>([&](int j) { acc = fma(rs[j], rl[j], acc); });
      return acc;
    }) / RT;
    rpmax = C.bmax(rpm);
    if (mu <= A.tol && rpmax <= 1e-10 && rdmax <= 1e-8 * (1.0 + gscale)) { converged = true; break; }
    if (it >= A.max_iters || !isfinite(mu)) break;
    if (!C.factor()) break;                     // a Quu lost definiteness: keep the current iterate
    // predictor: w = (l / s) rp - l
    C.template for_rows<NS, false, false>([&](int j, int r, double, double, double, double) {
      S.X[r] = div_nr(rl[j], rs[j]) * rp[j] - rl[j];
    });
    __syncthreads();
    C.build_g();
    C.lq_solve();
    // affine step: ds = -rp - c'dz, dl = -l - (l / s) ds; c'dz kept in S.X
    double amax_l = 1.0;
    C.template for_rows<NS, false, true>([&](int j, int r, double, double cd, double, double) {
      const double ds = -rp[j] - cd;
      const double dl = -rl[j] - div_nr(rl[j], rs[j]) * ds;
      if (ds < 0.0) amax_l = fmin(amax_l, div_nr(rs[j], -ds));
      if (dl < 0.0) amax_l = fmin(amax_l, div_nr(rl[j], -dl));
      S.X[r] = cd;
    });
    const double aa = C.bmin(amax_l);
    double ma[NS], mb[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) ma[j] = mb[j] = 0.0;
    C.template for_rows<NS, false, false>([&](int j, int r, double, double, double, double) {
      const double ds = -rp[j] - S.X[r];
      const double dl = -rl[j] - div_nr(rl[j], rs[j]) * ds;
      ma[j] = rs[j] + aa * ds;
      mb[j] = rl[j] + aa * dl;
      S.X[r] = ds * dl;                         // affine product for the corrector
    });
    const double mua = C.chain_sum([&](double acc) {
      C.template for_slots<NS>([&](int j) { acc = fma(ma[j], mb[j], acc); });
      return acc;
    }) / RT;
    const double sc = (mua / mu) * (mua / mu) * (mua / mu);
    const double smu_t = sc * mu;
    // corrector: rc = s l + ds_aff dl_aff - sc mu, w = (l rp - rc) / s
    C.template for_rows<NS, false, false>([&](int j, int r, double, double, double, double) {
      const double rc = rs[j] * rl[j] + S.X[r] - smu_t;
      S.X[r] = div_nr(rl[j] * rp[j] - rc, rs[j]);
    });
    __syncthreads();
    C.build_g();
    C.lq_solve();
    // step: ds = -rp - c'dz, dl = (-rc - l ds) / s with rc = l rp - s w (w in S.X)
    double am = 1.0;
    C.template for_rows<NS, false, true>([&](int j, int r, double, double cd, double, double) {
      const double ds = -rp[j] - cd;
      const double rc = rl[j] * rp[j] - rs[j] * S.X[r];
      const double dl = div_nr(-rc - rl[j] * ds, rs[j]);
      if (ds < 0.0) am = fmin(am, div_nr(rs[j], -ds));
      if (dl < 0.0) am = fmin(am, div_nr(rl[j], -dl));
    });
    const double alpha = fmin(1.0, 0.995 * C.bmin(am));
    bool nonfinite = !(alpha > 0.0) || !isfinite(alpha);
    for (int e = tid; e < 9 * N; e += kT) nonfinite |= !isfinite(S.dz[e]);
    if (__syncthreads_or(nonfinite)) break;     // a broken direction: keep the current iterate
    C.template for_rows<NS, false, true>([&](int j, int r, double, double cd, double, double) {
      const double ds = -rp[j] - cd;
      const double rc = rl[j] * rp[j] - rs[j] * S.X[r];
      const double dl = div_nr(-rc - rl[j] * ds, rs[j]);
      rs[j] += alpha * ds;
      rl[j] += alpha * dl;
      S.X[r] = rl[j];
    });
    __syncthreads();
    for (int e = tid; e < 9 * N; e += kT) S.z[e] += alpha * S.dz[e];
    __syncthreads();
  }

  // ---- outputs: states (x_N from the dynamics), inputs, cost, residuals
  double cst = 0.0;
  for (int e = lane; e < 9 * N; e += kW) {
    const int k = e / 9, a = e - 9 * (e / 9);
    const double* H = C.Hk(k);
    double hz = 0.0;
    for (int b = 0; b < 9; ++b) hz += H[9 * a + b] * S.z[9 * k + b];
    cst += 0.5 * S.z[e] * hz + C.hk(k, a) * S.z[e];
    if (a < 6 && k >= 1) {
      double qr = 0.0;
      for (int b = 0; b < 6; ++b) qr += S.prm[Ly.Qm + 6 * a + b] * S.ref[6 * k + b];
      cst += S.ref[6 * k + a] * qr;
    }
  }
  const double cost = wave::sum(cst);
  double pres = 0.0, pscale = 0.0, cres = 0.0, lmax = 0.0;
  C.template for_rows<NS, true, false>([&](int j, int, double v, double, double d, double de) {
    pres = fmax(pres, fma(-d, de, v));
    pscale = fmax(pscale, fmax(fabs(v), fabs(d * de)));
    cres = fmax(cres, rl[j] * fabs(fma(d, de, -v)));
    lmax = fmax(lmax, rl[j]);
  });
  C.bmax2(pres, pscale);
  C.bmax2(cres, lmax);
  const double kkt = fmax(fmax(fmax(pres, 0.0) / (1.0 + pscale), rdmax / (1.0 + gscale)), cres / (1.0 + lmax));
  const int64_t xo = (int64_t)inst * 6 * (N + 1);
  for (int e = tid; e < 6 * N; e += kT) {
    const int k = e / 6, a = e - 6 * (e / 6);
    A.X[xo + e] = (k == 0) ? x0[a] : S.z[9 * k + a];
  }
  if (tid < 6) {
    const double* zl = S.z + 9 * (N - 1);
    const int c = lane % 3;
    const double v = lane < 3 ? zl[c] + dt * zl[3 + c] + 0.5 * dt * dt * zl[6 + c] : zl[3 + c] + dt * zl[6 + c];
    A.X[xo + 6 * N + lane] = v;
  }
  for (int e = tid; e < 3 * N; e += kT) A.U[(int64_t)inst * 3 * N + e] = S.z[9 * (e / 3) + 6 + e % 3];
  const bool solved = kkt <= 1e-6 && isfinite(cost);
  if (tid == 0) {
    A.cost[inst] = cost;
    A.kkt[inst] = kkt;
    A.status[inst] = solved ? kSolved : (converged ? kNumerical : kMaxIter);
    if (A.iters) A.iters[inst] = it;
  }
  if (solved || converged || !A.ubox_ok) return;

  // ---- infeasibility certificate for a horizon the iterations did not solve.
  // With w >= 0 on the rows (the last multipliers, scaled to max 1) and the
  // terminal costate pi, Phi(u) = sum_i w_i (c_i'z(u) - d_i) + pi'(x_N(u) - r_N)
  // is affine in the inputs u along trajectories of the dynamics from x0,
  // Phi(u) = Phi(0) + rho'u, and Phi(u) <= 0 for every feasible u.  Every
  // feasible u_k also lies in the input box of the rows that act on u alone.
  // So Phi(0) + min over the box of rho'u > 0 proves that no feasible
  // trajectory exists (FP64, with a margin for rounding).
  {
    double lm = 0.0;
    C.template for_rows<NS, false, false>([&](int j, int, double, double, double, double) { lm = fmax(lm, rl[j]); });
    lm = C.bmax(lm);
    const double isc = (lm > 0.0 && isfinite(lm)) ? 1.0 / lm : 0.0;
    C.template for_rows<NS, false, false>([&](int j, int r, double, double, double, double) { S.X[r] = rl[j] * isc; });
    __syncthreads();
    double rdm = 0.0, gsc = 0.0, pi6[6];
    C.template dual_residual<false>(rdm, gsc, pi6);
    // free response: zero inputs from x0
    for (int e = tid; e < 9 * N; e += kT) {
      const int k = e / 9, a = e - 9 * (e / 9);
      S.z[e] = a < 3 ? x0[a] + k * dt * x0[3 + a] : (a < 6 ? x0[a] : 0.0);
    }
    __syncthreads();
    const double phi = C.chain_sum([&](double acc) {
      C.template for_rows<NS, true, false>([&](int, int r, double cz, double, double d, double de) { acc = fma(S.X[r], fma(-d, de, cz), acc); });
      return acc;
    });
    const double pab = C.chain_sum([&](double acc) {
      C.template for_rows<NS, true, false>(
          [&](int, int r, double cz, double, double d, double de) { acc = fma(S.X[r], fabs(cz) + fabs(d * de), acc); });
      return acc;
    });
    double tn = 0.0, tnab = 0.0;
    for (int c = 0; c < 3; ++c) {
      const double ep = x0[c] + N * dt * x0[3 + c] - S.ref[6 * N + c], ev = x0[3 + c] - S.ref[6 * N + 3 + c];
      tn += pi6[c] * ep + pi6[3 + c] * ev;
      tnab += fabs(pi6[c] * ep) + fabs(pi6[3 + c] * ev);
    }
    double mb = 0.0, mbab = 0.0, umax = 0.0;
    for (int e = lane; e < 3 * N; e += kW) {
      const int c = e - 3 * (e / 3);
      const double lo = c == 0 ? A.ulo[0] : (c == 1 ? A.ulo[1] : A.ulo[2]);
      const double hi = c == 0 ? A.uhi[0] : (c == 1 ? A.uhi[1] : A.uhi[2]);
      const double r = S.rho[e];
      mb += r > 0.0 ? r * lo : r * hi;
      mbab += fabs(r) * fmax(fabs(lo), fabs(hi));
      umax = fmax(umax, fmax(fabs(lo), fabs(hi)));
    }
    mb = wave::sum(mb);
    mbab = wave::sum(mbab);
    umax = wave::max(umax);
    // rounding: relative 1e-9 of every magnitude that entered, including the
    // costate recursion behind rho (N stages, growth N dt)
    const double margin = 1e-9 * (pab + tnab + mbab + 3.0 * N * umax * gsc * N * (1.0 + N * dt)) + 1e-300;
    if (phi + tn + mb > margin && isfinite(phi + tn + mb)) {
      for (int e = tid; e < 6 * (N + 1); e += kT) A.X[xo + e] = __builtin_nan("");
      for (int e = tid; e < 3 * N; e += kT) A.U[(int64_t)inst * 3 * N + e] = __builtin_nan("");
      if (tid == 0) {
        A.cost[inst] = __builtin_huge_val();
        A.kkt[inst] = __builtin_nan("");
        A.status[inst] = kInfeasible;
      }
    }
  }
}

}  // namespace

size_t mpc_lds_bytes(int N, int m) { return sizeof(double) * size_t(mpc_lds_doubles(N, m)); }

// One wavefront per instance where its few rows fit kOneSlots slots of a lane and the
// batch holds more instances than CUs fit with four wavefronts each (three, by
// registers; up to twelve with one): the other three are mostly idle there, and a
// CU takes its instances in rounds.  Four / one, the same results bit for bit: 768
// horizons of 4 steps 190 / 176 us, of 8 343 / 399, of 16 519 / 679 (12 rows); 1,024 of
// 4, 8 (16 rows) and 16 893 / 710, 592 / 421 and 821 / 705; 4,096 of 2, 4, 8, 12 and
// 16 2,965 / 948, 1,000 / 434, 1,375 / 768, 1,858 / 1,176 and 2,417 / 1,656 (12 rows), of 2 and 6
// with 32 rows 3,962 / 1,568 and 3,343 / 2,190.  Past four slots the lead goes: 1,536 of 12
// steps, 20 rows 1,757 / 1,935.
static bool mpc_one_wave(const MpcArgs& a) {
  return a.n > 3 * a.n_cu && (a.N * a.m + kW - 1) / kW + (4 * a.N + kW - 1) / kW <= kOneSlots;
}

hipError_t launch_mpc(const MpcArgs& a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  const size_t lds = mpc_lds_bytes(a.N, a.m);
  // register slots: passes of 64 reachable rows over three wavefronts (at most
  // 11); the plane rows (4 N <= 256) take four in the last
  const int rows = a.N * a.m;
  if (a.N < 2 || a.N > 64 || a.m < 0 || rows > 32 * kW) return hipErrorInvalidValue;
  const int slots = ((rows + kW - 1) / kW + kWaves - 2) / (kWaves - 1);
  if (mpc_one_wave(a))
    hipLaunchKernelGGL((mpc_kernel<kOneSlots, 1>), dim3(a.n), dim3(kW), lds, s, a);
  else if (slots <= 5)
    hipLaunchKernelGGL((mpc_kernel<5, kWaves>), dim3(a.n), dim3(kW * kWaves), lds, s, a);
  else
    hipLaunchKernelGGL((mpc_kernel<11, kWaves>), dim3(a.n), dim3(kW * kWaves), lds, s, a);
  return hipGetLastError();
}

}  // namespace rbp
