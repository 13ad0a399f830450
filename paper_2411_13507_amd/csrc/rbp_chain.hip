// Multi-segment paths: S degree-p segments joined with continuous position,
// velocity and acceleration, one 64-lane wavefront per path, or four.
//
// Each segment keeps its control points in its own free-space polytope
// (Property 1 of the paper), respects the velocity and acceleration bounds
// and its reachable Bezier polytope (Theorem 2) from its own start state
// (the path's start state for the first segment, the join state
// (P^s_0, p/T (P^s_1 - P^s_0)) for the others); start and goal are pinned.
//
// Elimination of the joins.  With equal durations, C0/C1/C2 fix the first
// three control points of segment s >= 1 from the last three of segment s-1:
//   P^s_0 = w2,  P^s_1 = 2 w2 - w1,  P^s_2 = 4 w2 - 4 w1 + w0,  P^s_k = w_k (k >= 3)
// for the window w = (P^{s-1}_{p-2}, P^{s-1}_{p-1}, P^{s-1}_p, P^s_3 .. P^s_p).
// The free variables are the "global points" g_1 .. g_{NG-2} (g_0 = start,
// g_{NG-1} = goal); segment s reads the p+1 consecutive global points from
// ws(s) = (p-2) s.  The cost is sum_c g_c^T G1 g_c with G1 banded (bandwidth
// p), so the Hessian is G1 (x) I3.
//
// Forward pass: FP32 ADMM warm start with the banded K = P + rho A^T D^2 A
// factored in LDS; FP64 dual active-set polish (Goldfarb-Idnani in the
// Hessian's metric) using products with L^-1 and L^-T, G1 = L L^T (one lane per
// global point), and the inverse of the Cholesky factor of the small Schur
// complement N^T G^-1 N of the working set; Farkas vectors verified in FP64.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>
#include <vector>

#include "rbp_internal.hpp"
#include "rbp_wave.hpp"

namespace rbp {

__constant__ DegConst c_chain_deg[kMaxDeg + 1];

// The Hessian of a path on its free global points depends on the number of
// segments S alone (times T^-3), G = L L^T.  Per S the inverse of L, NF x NF
// (NF = 5 S + 1 free points), laid out so that lane i reads entry i of a
// contiguous row: by columns, and by rows for its transpose.  Formed on the host
// in extended precision when a device's first batch is built.  G^-1 itself is of
// no use: a row's normal is a difference of neighbouring points, and products
// of G^-1 with it lose about five digits more than L^-1 and L^-T in turn.
constexpr int kChainDeg = 7, kChainMaxSeg = 12;
constexpr int chain_free(int S) { return (kChainDeg - 1) + (S - 1) * (kChainDeg - 2); }
constexpr int chain_tab(int S) {   // offset of S segments' tables
  int o = 0;
  for (int t = 1; t < S; ++t) o += chain_free(t) * chain_free(t);
  return o;
}
constexpr int kChainTab = chain_tab(kChainMaxSeg + 1);
static __device__ double t_Lc[kChainTab], t_Lr[kChainTab];

namespace {

constexpr int kWave = 64;
constexpr int kSolved = 0, kInfeasible = 1, kPolishFailed = 3, kNumerical = 4, kInvalid = 5;
// internal: the working set outgrew a reduced-cap pass; the full-cap pass
// that follows continues the path from the working set it stored and
// overwrites every output
constexpr int kRetry = 6;
constexpr float kBigF = 1e30f;
// wavefronts per path of the team kernel, and what the first asks of the others
constexpr int kTeamWaves = 4;
constexpr int kJobExit = 0, kJobScan = 1, kJobLower = 2, kJobUpper = 3;
typedef float floatx16 __attribute__((ext_vector_type(16)));

// 1 / sqrt(x), x > 0, from the hardware approximation refined to full precision
__device__ __forceinline__ double rsqrt_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  r = r * fma(-hx * r, r, 1.5);
  return r * fma(-hx * r, r, 1.5);
}
__device__ __forceinline__ double sel3(int c, double a, double b, double d) {
  return c == 0 ? a : (c == 1 ? b : d);
}

template <int P>
struct CLds {
  static constexpr int NP = P + 1, NC = 3 * (P + 1), BW = 3 * (P + 1) - 1;
  static constexpr int NB = NC | 1;   // row stride of the cached normals (read one row per lane)
  int *nf, *nr, *f0, *rowoff;
  int64_t *r0, *hb;
  double *Af, *bfs, *rb, *Pseg, *gfull, *G1b, *qv, *xu, *x, *scal;
  float *fan, *rn;
  int* cand;
  unsigned* actbits;
  // ADMM region
  float *Kb, *zr, *yr, *accp, *xt, *Cs;
  double* Wm;
  // polish region
  double *W, *beta, *acte, *u, *w, *zv, *np;
  int *actid, *actside, *actseg;
};

template <int P>
__device__ CLds<P> ccarve(char* s, const ChainDims& D) {
  CLds<P> L;
  L.nf = (int*)(s + D.o_segi);
  L.nr = L.nf + D.s_cap;
  L.f0 = L.nr + D.s_cap;
  L.rowoff = L.f0 + D.s_cap;             // s_cap + 1 entries
  L.r0 = (int64_t*)(s + D.o_seg64);
  L.hb = L.r0 + D.s_cap;
  L.Af = (double*)(s + D.o_Af);
  L.bfs = (double*)(s + D.o_bfs);
  L.fan = (float*)(s + D.o_fan);
  L.rb = (double*)(s + D.o_rb);
  L.rn = (float*)(s + D.o_rn);
  L.Pseg = (double*)(s + D.o_Pseg);
  L.gfull = (double*)(s + D.o_gfull);
  L.G1b = (double*)(s + D.o_G1b);
  L.qv = (double*)(s + D.o_qv);
  L.xu = L.qv + 3 * D.nf_pts_cap;
  L.x = (double*)(s + D.o_x);
  L.scal = (double*)(s + D.o_scal);
  L.cand = (int*)(s + D.o_cand);
  L.actbits = (unsigned*)(s + D.o_bits);
  L.Kb = (float*)(s + D.o_Kb);
  L.zr = (float*)(s + D.o_zr);
  L.yr = (float*)(s + D.o_yr);
  L.accp = (float*)(s + D.o_accp);
  L.xt = (float*)(s + D.o_xt);
  L.Cs = (float*)(s + D.o_Cs);
  L.Wm = (double*)(s + D.o_Wm);
  L.W = (double*)(s + D.o_W);
  L.beta = (double*)(s + D.o_beta);
  L.acte = (double*)(s + D.o_acte);
  L.u = (double*)(s + D.o_u);
  L.w = L.u + D.n_cap;
  L.zv = L.w + D.n_cap;
  L.np = L.zv + D.n_cap;
  L.actid = (int*)(s + D.o_actid);
  L.actside = L.actid + D.q_cap;
  L.actseg = L.actside + D.q_cap;
  return L;
}

// window map of segment s >= 1: control point k as a combination of window
// points (coefficients for w0, w1, w2; identity for k >= 3)
__device__ __forceinline__ double mcoef(int s, int k, int j) {
  if (s == 0 || k >= 3) return (k == j) ? 1.0 : 0.0;
  if (k == 0) return j == 2 ? 1.0 : 0.0;
  if (k == 1) return j == 2 ? 2.0 : (j == 1 ? -1.0 : 0.0);
  return j == 2 ? 4.0 : (j == 1 ? -4.0 : (j == 0 ? 1.0 : 0.0));   // k == 2
}

// kTeam = false: one wavefront per path.  kTeam = true: a workgroup of four; the
// first runs the method, the others take their share of the two jobs that are
// wide, the violation scan and the products with L^-1, and wait in between.
template <int P, bool kTeam>
__device__ __forceinline__ void chain_instance(const ChainArgs& A, const int ch, char* smem) {
  using L_t = CLds<P>;
  constexpr int NP = L_t::NP, NC = L_t::NC, BW = L_t::BW, NB = L_t::NB;
  static_assert(P == kChainDeg, "the tables of L^-1 are for this degree");
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = kTeam ? __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)) : 0;
  // orders LDS accesses between the lanes of this wavefront
  auto sync = [&]() {
    if constexpr (kTeam) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    } else {
      __syncthreads();
    }
  };
  const DegConst& K = c_chain_deg[P];
  const ChainDims& D = A.dims;
  L_t L = ccarve<P>(smem, D);

  const int64_t s0 = A.seg_off[ch];
  const int S = int(A.seg_off[ch + 1] - s0);
  const int NF = (P - 1) + (S - 1) * (P - 2);   // free global points
  const int NG = NF + 2;
  const int n = 3 * NF;
  const double T = A.T, T15 = T * sqrt(T), iT3 = 1.0 / (T * T * T);
  const double sv = double(P) / T, sa = double(P) * (P - 1) / (T * T);
  double x0[6], dg[3];
  bool bad = false;
  for (int e = 0; e < 6; ++e) { x0[e] = A.x0[6 * (int64_t)ch + e]; bad |= !isfinite(x0[e]); }
  for (int c = 0; c < 3; ++c) { dg[c] = A.goal[3 * (int64_t)ch + c] - x0[c]; bad |= !isfinite(dg[c]); }
  const int64_t pbase = (int64_t)NC * s0;   // output offset (doubles)

  auto finish = [&](int status) {
    for (int e = lane; e < S * NC; e += kWave) A.P_out[pbase + e] = __builtin_nan("");
    if (lane == 0) {
      A.cost_out[ch] = status == kInfeasible ? __builtin_huge_val() : __builtin_nan("");
      A.status_out[ch] = status;
      A.kkt_out[ch] = __builtin_nan("");
    }
  };

  // ---- the two wide jobs, in parts (part of parts; one wavefront each)
  const int NFC = D.nf_cap, RC = D.r_cap;
  const int toff = ((S - 1) * (36 + 6 * 5 * (S - 2)) + 25 * ((S - 2) * (S - 1) * (2 * S - 3) / 6));
  const int li = lane < NF ? lane : NF - 1;
  constexpr int kU = 16;                      // rows of a table in flight
  // Products with L^-1 and L^-T (x) I3 from the tables, one lane per free
  // point, three coordinates per lane: y_i = T^1.5 times the sum over j <= i
  // (lower, L^-1) or j >= i of tab[j NF + i] b_j, whose other entries are 0 in
  // the table: every lane loads every row, without a branch.  b must be 0 in
  // lanes past the last free point.  The banded substitution these
  // replace walks the points one after the other, four sweeps of up to 61 points
  // per polish step; a product reads 30 KB from L2 at most but nothing in it
  // waits for anything else.  L^-1 is applied on its own, as the substitution
  // was, so that |L^-1 d|^2 stays a sum of squares.
  auto tri_part = [&](int part, int parts, bool lower, double b0, double b1, double b2, double& y0, double& y1,
                      double& y2) {
    const double* tab = (lower ? t_Lc : t_Lr) + toff;
    y0 = 0.0; y1 = 0.0; y2 = 0.0;
    double t[kU];
    auto fetch = [&](int j0) {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int j = j0 + u;
        t[u] = tab[(j < NF ? j : NF - 1) * NF + li];
      }
    };
    fetch(part * kU);
    for (int j0 = part * kU; j0 < NF; j0 += parts * kU) {
      double c[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) c[u] = t[u];
      fetch(j0 + parts * kU);
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int j = j0 + u;                   // < 64; b is 0 past NF
        y0 += c[u] * wave::bcast(b0, j);
        y1 += c[u] * wave::bcast(b1, j);
        y2 += c[u] * wave::bcast(b2, j);
      }
    }
    const double f = lane < NF ? T15 : 0.0;
    y0 *= f; y1 *= f; y2 *= f;
  };
  // The most violated row outside the working set at the points in Pseg: its
  // score, key and violation, the same in every lane.  Rows' scaling is 1 /
  // |alpha|.
  auto scan_part = [&](int part, int parts, double& best, int& key, double& viol) {
    best = -1.0;
    key = 0x7fffffff;
    viol = 0.0;
    // row ``id`` with value v, bounds lo and hi, scaling d: a candidate if it
    // is not in the working set (looked up only for a row that would win)
    auto consider = [&](int id, double v, double lo, double hi, double d) {
      const double vu = v - hi, vl = lo - v;
      const bool up = vu > A.feas_tol * (1.0 + fabs(hi)) && vu * d > best;
      const bool dn = lo > -1e300 && vl > A.feas_tol * (1.0 + fabs(lo)) && vl * d > (up ? vu * d : best);
      if (!up && !dn) return;
      if ((L.actbits[id >> 5] >> (id & 31)) & 1u) return;
      best = dn ? vl * d : vu * d;
      viol = dn ? vl : vu;
      key = 2 * id + (dn ? 0 : 1);
    };
    const double minf = -__builtin_huge_val();
    // faces: one lane per face, its normal in registers while the eight points
    // pass; two segments at a time, one per half of the wavefront, where no
    // polytope has more than 32 faces
    {
      const int halves = NFC <= 32 ? 2 : 1, lanes = kWave / halves;
      const int h = halves == 2 ? lane >> 5 : 0, j = lane & (lanes - 1);
      for (int s1 = part * halves; s1 < S; s1 += parts * halves) {
        const int s = s1 + h;
        if (s < S && j < L.nf[s]) {
          const int nfs = L.nf[s];
          const double* a = L.Af + (s * NFC + j) * 3;
          const double a0 = a[0], a1 = a[1], a2 = a[2], hi = L.bfs[s * NFC + j], d = L.fan[s * NFC + j];
          const double* Pp = L.Pseg + s * NC;
          const int id0 = L.rowoff[s] + j;
#pragma unroll
          for (int k = 0; k < NP; ++k)
            consider(id0 + k * nfs, a0 * Pp[3 * k] + a1 * Pp[3 * k + 1] + a2 * Pp[3 * k + 2], minf, hi, d);
        }
      }
    }
    // velocity and acceleration rows: one lane per row of a segment
    if (lane < 6 * P - 3) {
      const bool vel = lane < 3 * P;
      const int e = vel ? lane : lane - 3 * P;              // 3 k + c
      const double b = vel ? A.vmax : A.amax;
      const double d = vel ? 1.0 / (sv * 1.4142135623730951) : 1.0 / (sa * 2.449489742783178);
      for (int s = part; s < S; s += parts) {
        const double* Pp = L.Pseg + s * NC + e;
        const double p0 = Pp[0], p1 = Pp[3], p2 = Pp[vel ? 3 : 6];
        const double v = vel ? sv * (p1 - p0) : sa * (p2 - 2.0 * p1 + p0);
        consider(L.rowoff[s] + NP * L.nf[s] + lane, v, -b, b, d);
      }
    }
    // reachable rows, whose coefficients come from global memory: two segments
    // per pass (<= 64 rows together where each has at most 32), the next pass's
    // rows loaded while this one's are worked on
    {
      struct Row { double h[NC], g[6]; };
      auto rows_of = [&](int s, int& n0, int& n1) {
        n0 = s < S ? L.rowoff[s + 1] - L.rowoff[s] - (NP * L.nf[s] + 6 * P - 3) : 0;
        n1 = s + 1 < S ? L.rowoff[s + 2] - L.rowoff[s + 1] - (NP * L.nf[s + 1] + 6 * P - 3) : 0;
      };
      auto fetch = [&](int s, int u, Row& w) {
        int n0, n1;
        rows_of(s, n0, n1);
        const bool on = u < n0 + n1;
        const int sp = !on ? 0 : (u < n0 ? s : s + 1), l = !on ? 0 : (u < n0 ? u : u - n0);
        const double* H = A.H + L.hb[sp] + (int64_t)l * NC;
        const double* G = A.G + 6 * (L.r0[sp] + l);
#pragma unroll
        for (int e = 0; e < NC; ++e) w.h[e] = on ? H[e] : 0.0;
#pragma unroll
        for (int e = 0; e < 6; ++e) w.g[e] = (on && sp > 0) ? G[e] : 0.0;
      };
      auto use = [&](int s, int u, const Row& w) {
        int n0, n1;
        rows_of(s, n0, n1);
        if (u >= n0 + n1) return;
        const int sp = u < n0 ? s : s + 1, l = u < n0 ? u : u - n0;
        const double* Pp = L.Pseg + sp * NC;
        double v = 0.0;
#pragma unroll
        for (int e = 0; e < NC; ++e) v += w.h[e] * Pp[e];
        if (sp > 0) {
#pragma unroll
          for (int c = 0; c < 3; ++c) v += (-w.g[c] + sv * w.g[3 + c]) * Pp[c] - sv * w.g[3 + c] * Pp[3 + c];
        }
        consider(L.rowoff[sp] + NP * L.nf[sp] + 6 * P - 3 + l, v, minf, L.rb[sp * RC + l], L.rn[sp * RC + l]);
      };
      Row ra, rb_;
      const int st = 2 * parts;
      fetch(2 * part, lane, ra);
      for (int s = 2 * part; s < S; s += 2 * st) {
        fetch(s + st, lane, rb_);
        use(s, lane, ra);
        fetch(s + 2 * st, lane, ra);
        use(s + st, lane, rb_);
      }
      // segments with more than 32 rows: what a pass of 64 lanes left
      if (RC > 32) {
        for (int s = 2 * part; s < S; s += st) {
          int n0, n1;
          rows_of(s, n0, n1);
          for (int u = lane + kWave; u < n0 + n1; u += kWave) {
            fetch(s, u, ra);
            use(s, u, ra);
          }
        }
      }
    }
    // the largest score; among equal ones the lowest row
    {
      double bm = best;
      int km = key;
      wave::argmax(bm, km);
      const unsigned long long own = __ballot(best == bm && key == km);
      best = bm;
      key = km;
      viol = wave::bcast(viol, own ? __builtin_ctzll(own) : 0);
    }
  };
  // workgroup's mailbox: job, its results, the right-hand side and partial
  // products
  double* const team = reinterpret_cast<double*>(smem + D.o_team);
  int* const job = reinterpret_cast<int*>(team);
  double* const found = team + 2;                       // 3 per wavefront
  double* const rhs_t = team + 2 + 3 * kTeamWaves;      // 3 x 64
  double* const part_t = rhs_t + 3 * kWave;             // 3 x 64 per helper
  if constexpr (kTeam) {
    if (wv > 0) {
      for (;;) {
        __syncthreads();                                // a job is posted
        const int what = *job;
        if (what == kJobExit) return;
        if (what == kJobScan) {
          double b, vi;
          int k;
          scan_part(wv, kTeamWaves, b, k, vi);
          if (lane == 0) { found[3 * wv] = b; found[3 * wv + 1] = double(k); found[3 * wv + 2] = vi; }
        } else {
          double y0, y1, y2;
          tri_part(wv, kTeamWaves, what == kJobLower, rhs_t[lane], rhs_t[kWave + lane], rhs_t[2 * kWave + lane], y0, y1, y2);
          double* o = part_t + 3 * kWave * (wv - 1);
          o[lane] = y0; o[kWave + lane] = y1; o[2 * kWave + lane] = y2;
        }
        __syncthreads();                                // done
      }
    }
  }
  auto tri = [&](bool lower, double b0, double b1, double b2, double& y0, double& y1, double& y2) {
    if constexpr (kTeam) {
      rhs_t[lane] = b0; rhs_t[kWave + lane] = b1; rhs_t[2 * kWave + lane] = b2;
      if (lane == 0) *job = lower ? kJobLower : kJobUpper;
      __syncthreads();
      tri_part(0, kTeamWaves, lower, b0, b1, b2, y0, y1, y2);
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kTeamWaves - 1; ++w) {
        const double* o = part_t + 3 * kWave * w;
        y0 += o[lane]; y1 += o[kWave + lane]; y2 += o[2 * kWave + lane];
      }
    } else {
      tri_part(0, 1, lower, b0, b1, b2, y0, y1, y2);
    }
  };
  auto scan = [&](double& best, int& key, double& viol) {
    if constexpr (kTeam) {
      if (lane == 0) *job = kJobScan;
      __syncthreads();
      scan_part(0, kTeamWaves, best, key, viol);
      __syncthreads();
#pragma unroll
      for (int w = 1; w < kTeamWaves; ++w) {
        const double b = found[3 * w], vi = found[3 * w + 2];
        const int k = int(found[3 * w + 1]);
        if (b > best || (b == best && k < key)) { best = b; key = k; viol = vi; }
      }
    } else {
      scan_part(0, 1, best, key, viol);
    }
  };

  // ---- segment tables
  if (lane < S) {
    const int64_t sg = s0 + lane;
    const int poly = A.poly_idx[sg];
    L.f0[lane] = A.poly_off[poly];
    L.nf[lane] = A.poly_off[poly + 1] - A.poly_off[poly];
    L.r0[lane] = A.reach_off[sg];
    L.nr[lane] = int(A.reach_off[sg + 1] - A.reach_off[sg]);
    L.hb[lane] = A.H_off[sg];
  }
  sync();
  if (lane == 0) {
    int acc = 0;
    for (int s = 0; s < S; ++s) { L.rowoff[s] = acc; acc += NP * L.nf[s] + 6 * P - 3 + L.nr[s]; }
    L.rowoff[S] = acc;
  }
  sync();
  const int m = L.rowoff[S];
  // faces (shifted bound) and reachable rows (shifted bound, 1/|alpha|)
  for (int s = 0; s < S; ++s) {
    const int nf = L.nf[s], nr = L.nr[s];
    for (int j = lane; j < nf; j += kWave) {
      const int64_t f = L.f0[s] + j;
      double a[3], an = 0.0;
      for (int c = 0; c < 3; ++c) { a[c] = A.A_face[3 * f + c]; L.Af[(s * NFC + j) * 3 + c] = a[c]; an += a[c] * a[c]; }
      const double b = A.b_face[f];
      L.bfs[s * NFC + j] = b - (a[0] * x0[0] + a[1] * x0[1] + a[2] * x0[2]);
      L.fan[s * NFC + j] = float(1.0 / sqrt(an));
      bad |= !(an > 0.0) || !isfinite(b);
    }
    for (int l = lane; l < nr; l += kWave) {
      const int64_t rr = L.r0[s] + l;
      const double* H = A.H + L.hb[s] + (int64_t)l * NC;
      const double* G = A.G + 6 * rr;
      double hs[3] = {0, 0, 0};
      double alpha2 = 0.0;
      for (int k = 0; k < NP; ++k)
        for (int c = 0; c < 3; ++c) hs[c] += H[3 * k + c];
      double b = A.h0[rr] - (hs[0] * x0[0] + hs[1] * x0[1] + hs[2] * x0[2]);
      if (s == 0) { for (int e = 0; e < 6; ++e) b += G[e] * x0[e]; }
      else { for (int c = 0; c < 3; ++c) b += G[c] * x0[c]; }
      for (int k = 0; k < NP; ++k)
        for (int c = 0; c < 3; ++c) {
          double a = H[3 * k + c];
          if (s > 0 && k == 0) a += -G[c] + sv * G[3 + c];
          if (s > 0 && k == 1) a += -sv * G[3 + c];
          alpha2 += a * a;
        }
      L.rb[s * RC + l] = b;
      L.rn[s * RC + l] = float(alpha2 > 0.0 ? 1.0 / sqrt(alpha2) : 0.0);
      bad |= !isfinite(b);
    }
  }
  if (__ballot(bad) != 0ull) { finish(kInvalid); return; }
  // the velocity rows chained along the joined polygon (S p edges) bound
  // every coordinate of goal - start by S vmax T: beyond that no path exists
  if (__ballot(lane < 3 && fabs(sel3(lane, dg[0], dg[1], dg[2])) > S * A.vmax * T * (1.0 + 1e-12)) != 0ull) {
    if (lane == 0 && A.iters_out) { A.iters_out[2 * ch] = 0; A.iters_out[2 * ch + 1] = 0; }
    finish(kInfeasible);
    return;
  }

  // ---- row helpers (local row numbering within segment s)
  // value of row (s, loc) on the control points of segment s (array Pp, stride 1)
  auto row_value = [&](int s, int loc, const double* Pp) -> double {
    const int nf = L.nf[s];
    const int F = NP * nf;
    if (loc < F) {
      const int k = loc / nf, j = loc - k * nf;
      const double* a = L.Af + (s * NFC + j) * 3;
      return a[0] * Pp[3 * k] + a[1] * Pp[3 * k + 1] + a[2] * Pp[3 * k + 2];
    }
    if (loc < F + 3 * P) {
      const int l = loc - F, k = l / 3, c = l - 3 * (l / 3);
      return sv * (Pp[3 * (k + 1) + c] - Pp[3 * k + c]);
    }
    if (loc < F + 6 * P - 3) {
      const int l = loc - F - 3 * P, k = l / 3, c = l - 3 * (l / 3);
      return sa * (Pp[3 * (k + 2) + c] - 2.0 * Pp[3 * (k + 1) + c] + Pp[3 * k + c]);
    }
    const int l = loc - F - 6 * P + 3;
    const double* H = A.H + L.hb[s] + (int64_t)l * NC;
    double v = 0.0;
    for (int e = 0; e < NC; ++e) v += H[e] * Pp[e];
    if (s > 0) {
      const double* G = A.G + 6 * (L.r0[s] + l);
      for (int c = 0; c < 3; ++c) v += (-G[c] + sv * G[3 + c]) * Pp[c] - sv * G[3 + c] * Pp[3 + c];
    }
    return v;
  };
  // bounds of row (s, loc): lo, hi (lo = -inf for one-sided rows)
  auto row_bounds = [&](int s, int loc, double& lo, double& hi) {
    const int nf = L.nf[s];
    const int F = NP * nf;
    if (loc < F) { lo = -__builtin_huge_val(); hi = L.bfs[s * NFC + (loc - (loc / nf) * nf)]; }
    else if (loc < F + 3 * P) { lo = -A.vmax; hi = A.vmax; }
    else if (loc < F + 6 * P - 3) { lo = -A.amax; hi = A.amax; }
    else { lo = -__builtin_huge_val(); hi = L.rb[s * RC + (loc - F - 6 * P + 3)]; }
  };
  // 1/|alpha| of a row (ADMM scaling, normalisation of violations)
  auto row_scale = [&](int s, int loc) -> double {
    const int nf = L.nf[s];
    const int F = NP * nf;
    if (loc < F) return L.fan[s * NFC + (loc - (loc / nf) * nf)];
    if (loc < F + 3 * P) return 1.0 / (sv * 1.4142135623730951);
    if (loc < F + 6 * P - 3) return 1.0 / (sa * 2.449489742783178);
    return L.rn[s * RC + (loc - F - 6 * P + 3)];
  };
  // control-point coefficient alpha_e (e = 3k + c) of row (s, loc)
  auto alpha_at = [&](int s, int loc, int e) -> double {
    const int nf = L.nf[s];
    const int F = NP * nf;
    const int ke = e / 3, ce = e - 3 * (e / 3);
    if (loc < F) {
      const int k = loc / nf, j = loc - k * nf;
      return ke == k ? L.Af[(s * NFC + j) * 3 + ce] : 0.0;
    }
    if (loc < F + 3 * P) {
      const int l = loc - F, k = l / 3, c = l - 3 * (l / 3);
      if (ce != c) return 0.0;
      return ke == k + 1 ? sv : (ke == k ? -sv : 0.0);
    }
    if (loc < F + 6 * P - 3) {
      const int l = loc - F - 3 * P, k = l / 3, c = l - 3 * (l / 3);
      if (ce != c) return 0.0;
      return ke == k + 2 ? sa : (ke == k + 1 ? -2.0 * sa : (ke == k ? sa : 0.0));
    }
    const int l = loc - F - 6 * P + 3;
    double a = A.H[L.hb[s] + (int64_t)l * NC + e];
    if (s > 0 && ke <= 1) {
      const double* G = A.G + 6 * (L.r0[s] + l);
      a += (ke == 0) ? (-G[ce] + sv * G[3 + ce]) : (-sv * G[3 + ce]);
    }
    return a;
  };
  // segment of a chain row id
  auto seg_of = [&](int id) -> int {
    int s = 0;
    while (s + 1 < S && L.rowoff[s + 1] <= id) ++s;
    return s;
  };
  // global full point vector from the free points x (n, interleaved xyz),
  // then the control points of every segment (shifted frame)
  auto build_points = [&](const double* xv) {
    for (int e = lane; e < 3 * NG; e += kWave) {
      const int g = e / 3, c = e - 3 * (e / 3);
      double v;
      if (g == 0) v = 0.0;
      else if (g == NG - 1) v = sel3(c, dg[0], dg[1], dg[2]);
      else v = xv[3 * (g - 1) + c];
      L.gfull[e] = v;
    }
    sync();
    for (int e = lane; e < S * NC; e += kWave) {
      const int s = e / NC, r = e - NC * (e / NC), k = r / 3, c = r - 3 * (r / 3);
      const int ws = (P - 2) * s;
      double v = 0.0;
      for (int j = 0; j < 3; ++j) v += mcoef(s, k, j) * L.gfull[3 * (ws + j) + c];
      if (k >= 3) v = L.gfull[3 * (ws + k) + c];
      L.Pseg[e] = v;
    }
    sync();
  };

  // ---- Hessian G1 (banded, bandwidth P) and its Cholesky factor on the free points
  // window Hessians: Wm[0] = 2 Q1 / T^3 (segment 0), Wm[1] = M^T Wm[0] M
  for (int e = lane; e < NP * NP; e += kWave) {
    const int a = e / NP, b = e - NP * (e / NP);
    L.Wm[e] = 2.0 * iT3 * K.Q1[a][b];
    double v = 0.0;
    for (int k = 0; k < NP; ++k)
      for (int k2 = 0; k2 < NP; ++k2) v += mcoef(1, k, a) * 2.0 * iT3 * K.Q1[k][k2] * mcoef(1, k2, b);
    L.Wm[NP * NP + e] = v;
  }
  sync();
  for (int e = lane; e < NG * (P + 1); e += kWave) {
    const int g = e / (P + 1), d = e - (P + 1) * (e / (P + 1));
    const int h = g - d;
    double v = 0.0;
    if (h >= 0) {
      for (int s = 0; s < S; ++s) {
        const int ws = (P - 2) * s;
        if (g >= ws && g <= ws + P && h >= ws) v += L.Wm[(s > 0 ? NP * NP : 0) + (g - ws) * NP + (h - ws)];
      }
    }
    L.G1b[e] = v;
  }
  sync();
  // Products with L^-1 and L^-T (x) I3: tri (above), one lane per free point
  auto gfwd = [&](const double* rhs, double& y0, double& y1, double& y2) {
    const bool on = lane < NF;
    tri(true, on ? rhs[3 * li] : 0.0, on ? rhs[3 * li + 1] : 0.0, on ? rhs[3 * li + 2] : 0.0, y0, y1, y2);
  };
  auto gbwd = [&](double y0, double y1, double y2, double* out) {
    double z0, z1, z2;
    tri(false, y0, y1, y2, z0, z1, z2);
    if (lane < NF) { out[3 * lane] = z0; out[3 * lane + 1] = z1; out[3 * lane + 2] = z2; }
    sync();
  };
  auto gsolve = [&](const double* rhs, double* out) {
    double y0, y1, y2;
    gfwd(rhs, y0, y1, y2);
    gbwd(y0, y1, y2, out);
  };
  // linear term from the pinned goal: q = G1[free, goal] * dg; unconstrained minimiser
  for (int e = lane; e < n; e += kWave) {
    const int i = e / 3, c = e - 3 * (e / 3);
    const int g = i + 1, d = (NG - 1) - g;
    L.qv[e] = (d <= P) ? L.G1b[(NG - 1) * (P + 1) + d] * sel3(c, dg[0], dg[1], dg[2]) : 0.0;
  }
  sync();
  gsolve(L.qv, L.xu);
  for (int e = lane; e < n; e += kWave) L.xu[e] = -L.xu[e];
  sync();

  // ======================================================================
  // FP32 ADMM warm start (banded K in LDS)
  // ======================================================================
  const int K_admm = A.admm_iters;
  int ncand = 0;
  if (K_admm > 0 && !A.retry_only) {
    const float rho = A.rho, alpha = A.alpha, irho = 1.0f / A.rho;
    // K = G (x) I3 + rho * sum_s embed(M_s^T C_s M_s); band storage Kb[i][d] = K[i][i-d]
    for (int e = lane; e < n * (BW + 1); e += kWave) {
      const int i = e / (BW + 1), d = e - (BW + 1) * (e / (BW + 1));
      const int j = i - d;
      float v = 0.0f;
      if (j >= 0 && (i % 3) == (j % 3)) {
        const int gi = i / 3, gj = j / 3;
        if (gi - gj <= P) v = float(L.G1b[(gi + 1) * (P + 1) + (gi - gj)]);
      }
      L.Kb[e] = v;
    }
    sync();
    for (int s = 0; s < S; ++s) {
      // C_s in control-point space: faces, difference rows, reachable rows (matrix cores)
      const int nf = L.nf[s], nr = L.nr[s];
      double gf[6];
      {
        double a0 = 0, a1 = 0, a2 = 0, w = 0;
        if (lane < nf) {
          a0 = L.Af[(s * NFC + lane) * 3]; a1 = L.Af[(s * NFC + lane) * 3 + 1]; a2 = L.Af[(s * NFC + lane) * 3 + 2];
          w = 1.0 / (a0 * a0 + a1 * a1 + a2 * a2);
        }
        gf[0] = wave::sum(w * a0 * a0); gf[1] = wave::sum(w * a0 * a1); gf[2] = wave::sum(w * a0 * a2);
        gf[3] = wave::sum(w * a1 * a1); gf[4] = wave::sum(w * a1 * a2); gf[5] = wave::sum(w * a2 * a2);
      }
      floatx16 acc;
#pragma unroll
      for (int g = 0; g < 16; ++g) acc[g] = 0.0f;
      const int col = lane & 31, half = lane >> 5;
      for (int t = 0; 2 * t < nr; ++t) {
        const int l = 2 * t + half;
        float a = 0.0f;
        if (l < nr && col < NC) {
          const double* H = A.H + L.hb[s] + (int64_t)l * NC;
          double v = H[col];
          if (s > 0) {
            const double* G = A.G + 6 * (L.r0[s] + l);
            if (col < 3) v += -G[col] + sv * G[3 + col];
            else if (col < 6) v -= sv * G[col];
          }
          a = float(v * L.rn[s * RC + l]);
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, a, acc, 0, 0, 0);
      }
      for (int e = lane; e < NC * NC; e += kWave) L.Cs[e] = 0.0f;
      sync();
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        const int i = 8 * (g >> 2) + 4 * half + (g & 3);
        if (i < NC && col < NC) L.Cs[i * NC + col] = acc[g];
      }
      sync();
      for (int e = lane; e < NC * NC; e += kWave) {
        const int i = e / NC, j = e - NC * (e / NC);
        const int ki = i / 3, ci = i - 3 * ki, kj = j / 3, cj = j - 3 * kj;
        float v = L.Cs[e];
        if (ki == kj) {
          const int a = ci < cj ? ci : cj, b = ci < cj ? cj : ci;
          const int ix = a == 0 ? b : (a == 1 ? 2 + b : 5);
          const double g = ix == 0 ? gf[0] : ix == 1 ? gf[1] : ix == 2 ? gf[2] : ix == 3 ? gf[3] : ix == 4 ? gf[4] : gf[5];
          v += float(g);
        }
        if (ci == cj) {
          // velocity rows k: (P_{k+1} - P_k)^2 / 2 ; acceleration rows: (D2)^2 / 6
          double dv = 0.0;
          for (int k = 0; k < P; ++k) {
            const double ai = double(ki == k + 1) - double(ki == k), aj = double(kj == k + 1) - double(kj == k);
            dv += 0.5 * ai * aj;
          }
          for (int k = 0; k < P - 1; ++k) {
            const double ai = double(ki == k + 2) - 2.0 * double(ki == k + 1) + double(ki == k);
            const double aj = double(kj == k + 2) - 2.0 * double(kj == k + 1) + double(kj == k);
            dv += ai * aj / 6.0;
          }
          v += float(dv);
        }
        L.Cs[e] = v;
      }
      sync();
      // window transform M^T C M and accumulation into the band (free points only)
      constexpr int EPL = (NC * NC + kWave - 1) / kWave;
      float tv[EPL];
#pragma unroll
      for (int ti = 0; ti < EPL; ++ti) {
        const int e = lane + kWave * ti;
        tv[ti] = 0.0f;
        if (e >= NC * NC) continue;
        const int i = e / NC, j = e - NC * (e / NC);
        const int wi = i / 3, ci = i - 3 * wi, wj = j / 3, cj = j - 3 * wj;
        double v = 0.0;
        for (int k = 0; k < NP; ++k) {
          const double mi = mcoef(s, k, wi);
          if (mi == 0.0) continue;
          for (int k2 = 0; k2 < NP; ++k2) {
            const double mj = mcoef(s, k2, wj);
            if (mj == 0.0) continue;
            v += mi * double(L.Cs[(3 * k + ci) * NC + 3 * k2 + cj]) * mj;
          }
        }
        tv[ti] = float(v) * rho;
      }
      sync();
      const int ws = (P - 2) * s;
#pragma unroll
      for (int ti = 0; ti < EPL; ++ti) {
        const int e = lane + kWave * ti;
        if (e >= NC * NC) continue;
        const int i = e / NC, j = e - NC * (e / NC);
        const int gi = ws + i / 3, gj = ws + j / 3;
        if (gi >= 1 && gi <= NG - 2 && gj >= 1 && gj <= NG - 2) {
          const int vi = 3 * (gi - 1) + (i - 3 * (i / 3)), vj = 3 * (gj - 1) + (j - 3 * (j / 3));
          if (vj <= vi) L.Kb[vi * (BW + 1) + (vi - vj)] += tv[ti];
        }
      }
      sync();
    }
    // band Cholesky of K (FP32), right-looking
    for (int i = 0; i < n; ++i) {
      const float dd = sqrtf(fmaxf(L.Kb[i * (BW + 1)], 1e-30f));
      sync();
      if (lane == 0) L.Kb[i * (BW + 1)] = dd;
      if (lane >= 1 && lane <= BW && i + lane < n) L.Kb[(i + lane) * (BW + 1) + lane] /= dd;
      sync();
      for (int t = lane; t < BW * (BW + 1) / 2; t += kWave) {
        int a = 0, rem = t;
        while (rem > a) { rem -= a + 1; ++a; }
        const int kk = i + 1 + a, jj = i + 1 + rem;
        if (kk < n) L.Kb[kk * (BW + 1) + (kk - jj)] -= L.Kb[kk * (BW + 1) + (kk - i)] * L.Kb[jj * (BW + 1) + (jj - i)];
      }
      sync();
    }
    for (int e = lane; e < m; e += kWave) { L.zr[e] = 0.0f; L.yr[e] = 0.0f; }
    sync();
    for (int it = 0; it < K_admm; ++it) {
      // control-point accumulations sum_rows alpha * d (rho (z - d c) - y)
      for (int e = lane; e < S * NC; e += kWave) {
        const int s = e / NC, r = e - NC * (e / NC), k = r / 3, c = r - 3 * (r / 3);
        const int nf = L.nf[s], nr = L.nr[s], ro = L.rowoff[s], F = NP * nf;
        // rows of the last segment carry the pinned goal as a constant part
        auto vrow = [&](int loc, float d) -> float {
          float cst = 0.0f;
          if (s == S - 1)
            cst = float(alpha_at(s, loc, 3 * P) * dg[0] + alpha_at(s, loc, 3 * P + 1) * dg[1] +
                        alpha_at(s, loc, 3 * P + 2) * dg[2]);
          return d * (rho * (L.zr[ro + loc] - d * cst) - L.yr[ro + loc]);
        };
        float t = 0.0f;
        for (int j = 0; j < nf; ++j) t += float(L.Af[(s * NFC + j) * 3 + c]) * vrow(k * nf + j, L.fan[s * NFC + j]);
        const float dv = float(1.0 / (sv * 1.4142135623730951)), da = float(1.0 / (sa * 2.449489742783178));
        if (k >= 1) t += float(sv) * vrow(F + 3 * (k - 1) + c, dv);
        if (k <= P - 1) t -= float(sv) * vrow(F + 3 * k + c, dv);
        if (k >= 2) t += float(sa) * vrow(F + 3 * P + 3 * (k - 2) + c, da);
        if (k >= 1 && k - 1 <= P - 2) t -= float(2.0 * sa) * vrow(F + 3 * P + 3 * (k - 1) + c, da);
        if (k <= P - 2) t += float(sa) * vrow(F + 3 * P + 3 * k + c, da);
        for (int l = 0; l < nr; ++l) {
          const double* H = A.H + L.hb[s] + (int64_t)l * NC;
          double a = H[3 * k + c];
          if (s > 0 && k <= 1) {
            const double* G = A.G + 6 * (L.r0[s] + l);
            a += (k == 0) ? (-G[c] + sv * G[3 + c]) : (-sv * G[3 + c]);
          }
          t += float(a) * vrow(F + 6 * P - 3 + l, L.rn[s * RC + l]);
        }
        L.accp[e] = t;
      }
      sync();
      // right-hand side on the free global points (both windows touching a point)
      for (int e = lane; e < n; e += kWave) {
        const int g = e / 3 + 1, c = e - 3 * (e / 3);
        float t = -float(L.qv[e]);
        for (int s = 0; s < S; ++s) {
          const int ws = (P - 2) * s;
          const int j = g - ws;
          if (j < 0 || j > P) continue;
          for (int k = 0; k < NP; ++k) {
            const double mk = mcoef(s, k, j);
            if (mk != 0.0) t += float(mk) * L.accp[s * NC + 3 * k + c];
          }
        }
        L.xt[e] = t;
      }
      sync();
      // x~ = K^-1 rhs with the band factor (lane i%64 holds entries i, i+64, i+128, ...)
      {
        constexpr int MAXV = 4;                 // n <= 256
        float b[MAXV];
#pragma unroll
        for (int v = 0; v < MAXV; ++v) { const int i = lane + kWave * v; b[v] = i < n ? L.xt[i] : 0.0f; }
        for (int i = 0; i < n; ++i) {
          const int sl = i >> 6;
          float bi = 0.0f;
#pragma unroll
          for (int v = 0; v < MAXV; ++v) if (v == sl) bi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b[v]), i & 63));
          const float yi = bi / L.Kb[i * (BW + 1)];
#pragma unroll
          for (int v = 0; v < MAXV; ++v) {
            const int k = lane + kWave * v;
            if (k == i) b[v] = yi;
            else if (k > i && k <= i + BW && k < n) b[v] -= L.Kb[k * (BW + 1) + (k - i)] * yi;
          }
        }
        for (int i = n - 1; i >= 0; --i) {
          const int sl = i >> 6;
          float bi = 0.0f;
#pragma unroll
          for (int v = 0; v < MAXV; ++v) if (v == sl) bi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b[v]), i & 63));
          const float yi = bi / L.Kb[i * (BW + 1)];
#pragma unroll
          for (int v = 0; v < MAXV; ++v) {
            const int k = lane + kWave * v;
            if (k == i) b[v] = yi;
            else if (k < i && k >= i - BW) b[v] -= L.Kb[i * (BW + 1) + (i - k)] * yi;
          }
        }
#pragma unroll
        for (int v = 0; v < MAXV; ++v) { const int i = lane + kWave * v; if (i < n) L.xt[i] = b[v]; }
      }
      sync();
      // control points of x~ (FP32) and row update
      for (int e = lane; e < 3 * NG; e += kWave) {
        const int g = e / 3, c = e - 3 * (e / 3);
        double v = g == 0 ? 0.0 : (g == NG - 1 ? sel3(c, dg[0], dg[1], dg[2]) : double(L.xt[3 * (g - 1) + c]));
        L.gfull[e] = v;
      }
      sync();
      for (int e = lane; e < S * NC; e += kWave) {
        const int s = e / NC, r = e - NC * (e / NC), k = r / 3, c = r - 3 * (r / 3);
        const int ws = (P - 2) * s;
        double v = 0.0;
        for (int j = 0; j < 3; ++j) v += mcoef(s, k, j) * L.gfull[3 * (ws + j) + c];
        if (k >= 3) v = L.gfull[3 * (ws + k) + c];
        L.Pseg[e] = v;
      }
      sync();
      for (int s = 0; s < S; ++s) {
        const int ms = L.rowoff[s + 1] - L.rowoff[s], ro = L.rowoff[s];
        for (int loc = lane; loc < ms; loc += kWave) {
          const float d = float(row_scale(s, loc));
          double lo, hi;
          row_bounds(s, loc, lo, hi);
          const float zh = d * float(row_value(s, loc, L.Pseg + s * NC));
          const float flo = isfinite(lo) ? d * float(lo) : -kBigF, fhi = isfinite(hi) ? d * float(hi) : kBigF;
          float z = L.zr[ro + loc], y = L.yr[ro + loc];
          const float zrl = alpha * zh + (1.0f - alpha) * z;
          float zn = zrl + y * irho;
          zn = zn < flo ? flo : (zn > fhi ? fhi : zn);
          y += rho * (zrl - zn);
          L.zr[ro + loc] = zn;
          L.yr[ro + loc] = y;
        }
      }
      sync();
    }
    // proposals: most active first (|y|), at most q_cap of them
    for (int t = 0; t < D.q_cap; ++t) {
      double best = -1.0;
      int key = 0x7fffffff;
      for (int s = 0; s < S; ++s) {
        const int ms = L.rowoff[s + 1] - L.rowoff[s], ro = L.rowoff[s];
        for (int loc = lane; loc < ms; loc += kWave) {
          const float y = L.yr[ro + loc], z = L.zr[ro + loc];
          if (y == 0.0f) continue;
          const float d = float(row_scale(s, loc));
          double lo, hi;
          row_bounds(s, loc, lo, hi);
          const float flo = isfinite(lo) ? d * float(lo) : -kBigF, fhi = isfinite(hi) ? d * float(hi) : kBigF;
          int side = 0;
          if (fhi - z < y) side = 1;
          else if (z - flo < -y) side = -1;
          if (side != 0 && double(fabsf(y)) > best) { best = fabsf(y); key = 2 * (ro + loc) + (side > 0 ? 1 : 0); }
        }
      }
      wave::argmax(best, key);
      if (!(best > 0.0) || key < 0 || (key >> 1) >= m) break;
      if (lane == 0) { L.cand[t] = key; L.yr[key >> 1] = 0.0f; }
      ++ncand;
      sync();
    }
  }
  sync();

  // ======================================================================
  // FP64 dual active-set polish
  // ======================================================================
  const int QC = D.q_cap;
  for (int e = lane; e < (m + 31) / 32; e += kWave) L.actbits[e] = 0u;
  // box of every feasible point (velocity rows chained along the joined
  // polygon from both pinned ends): free coordinate e belongs to global point
  // g = e/3 + 1 at polygon position pos(g)
  auto box_of = [&](int e, double& lo, double& hi) {
    const int g = e / 3 + 1, c = e - 3 * (e / 3);
    int pos;
    if (g <= P) pos = g;
    else { const int s2 = (g - P - 1) / (P - 2) + 1; pos = s2 * P + 3 + (g - P - 1) % (P - 2); }
    const double vv = A.vmax * T / P, dgc = sel3(c, dg[0], dg[1], dg[2]);
    lo = fmax(-pos * vv, dgc - (S * P - pos) * vv);
    hi = fmin(pos * vv, dgc + (S * P - pos) * vv);
  };
  // (G1 (x) I3) v at free coordinate e (band storage of the Hessian), with
  // |G1| entries when ``absval``
  auto gmul_at = [&](const double* v, int e, bool absval) -> double {
    const int i = e / 3, c = e - 3 * (e / 3);
    double acc = 0.0;
    for (int d = -P; d <= P; ++d) {
      const int j = i + d;
      if (j < 0 || j >= NF) continue;
      const int hi_ = i > j ? i : j, lo_ = i > j ? j : i;
      const double gv = L.G1b[(hi_ + 1) * (P + 1) + (hi_ - lo_)];
      acc += (absval ? fabs(gv) : gv) * v[3 * j + c];
    }
    return acc;
  };
  // Ub bounds 1/2 (x - x_u)' G (x - x_u) (the path's cost, whose unconstrained
  // minimum is 0: the straight line at constant speed) over the feasible
  // points, by the smaller of: over the box, with centre x_c and half-widths
  // w, |x - x_u|_G <= |x_c - x_u|_G + |x - x_c|_G and d' G d <= sum_ij |G_ij|
  // |d_i| |d_j|; and S 3 amax^2 T, since the acceleration rows bound every
  // coordinate of every control point of each segment's b'' by amax.  A dual
  // value (relative to the unconstrained minimum) above Ub proves that no
  // feasible path exists.
  double Ub = 0.0;
  {
    for (int e = lane; e < n; e += kWave) {
      double lo, hi;
      box_of(e, lo, hi);
      L.zv[e] = 0.5 * (lo + hi) - L.xu[e];
      L.w[e] = fmax(0.5 * (hi - lo), 0.0);
    }
    sync();
    double cc = 0.0, ww = 0.0;
    for (int e = lane; e < n; e += kWave) {
      cc += L.zv[e] * gmul_at(L.zv, e, false);
      ww += L.w[e] * gmul_at(L.w, e, true);
    }
    cc = wave::sum(cc);
    ww = wave::sum(ww);
    const double rt = sqrt(fmax(cc, 0.0)) + sqrt(fmax(ww, 0.0));
    Ub = fmin(0.5 * rt * rt, 3.0 * S * A.amax * A.amax * T * (1.0 + 1e-12));
    sync();
  }
  for (int e = lane; e < n; e += kWave) L.x[e] = L.xu[e];
  sync();
  int q = 0, steps = 0, status = kPolishFailed;
  // Working set of up to QC - 1 <= 127 rows: lane l holds entries l and l + 64
  // of every working-set vector (multipliers, right-hand sides of the Schur
  // solves).  Of the factor L_S of N^T G^-1 N the inverse W is kept, packed by
  // rows, row k in k + 1 slots.
  double lam0 = 0.0, lam1 = 0.0;   // multipliers of entries lane and lane + 64
  const int e0 = lane, e1 = lane + kWave;
  auto row_at = [](int k) -> int { return (k * (k + 1)) >> 1; };
  auto pick = [&](double v0, double v1, int k) -> double {
    return wave::bcast(k < kWave ? v0 : v1, k & (kWave - 1));
  };
  const double ftol = A.feas_tol;
  const int max_steps = A.max_steps > 0 ? A.max_steps : 8 * n + 64;

  // entering normal of (id, side): beta cache slot ``slot``; also writes the
  // global normal into L.np
  // (entries on the pinned points are 0)
  auto load_normal = [&](int id, int side, int slot) {
    const int s = seg_of(id);
    const int loc = id - L.rowoff[s];
    const int ws = (P - 2) * s;
    const int j = lane / 3, c = lane - 3 * (lane / 3);
    double al = 0.0;
    if (lane < NC) {
      al = alpha_at(s, loc, lane);
      if (lane < 9) L.scal[lane] = al;
    }
    if (lane == 0) L.actseg[slot] = s;
    sync();
    if (lane < NC) {
      // window coefficients beta = M_s^T alpha (per coordinate; M_s is the
      // identity but for the first three points of a segment past the first)
      double v = 0.0;
      if (s > 0 && j < 3) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double mk = mcoef(s, k, j);
          if (mk != 0.0) v += mk * L.scal[3 * k + c];
        }
      } else {
        v = al;
      }
      const int g = ws + j;
      L.beta[slot * NB + lane] = (g >= 1 && g <= NG - 2) ? double(side) * v : 0.0;
    }
    sync();
    for (int e = lane; e < n; e += kWave) {
      const int w = e - 3 * (ws - 1);
      L.np[e] = (w >= 0 && w < NC) ? L.beta[slot * NB + w] : 0.0;
    }
    sync();
  };
  // dot of the window normal in slot k with a global vector (whose entries at
  // the pinned points do not exist: any entry stands in, times 0)
  auto ndot = [&](int k, const double* v) -> double {
    const int sgk = L.actseg[k], o = 3 * ((P - 2) * sgk - 1);
    const double* b = L.beta + k * NB;
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < NC; ++e) {
      const int i = e < 3 ? (sgk > 0 ? o + e : 0) : (e >= NC - 3 ? (sgk < S - 1 ? o + e : 0) : o + e);
      acc += b[e] * v[i];
    }
    return acc;
  };
  // u = G^-1 n for the window normal n in slot k (segment sgk): L^-1 n takes
  // eight rows of the table
  auto gsolve_window = [&](int k, int sgk, double* out) {
    const int i0 = (P - 2) * sgk - 1;          // free index of the window's first point
    double t[NP], y0 = 0.0, y1 = 0.0, y2 = 0.0;
#pragma unroll
    for (int w = 0; w < NP; ++w) {
      const int j = i0 + w;                    // beta is 0 where j is no free point
      t[w] = lane < NF ? t_Lc[toff + (j < 0 ? 0 : (j < NF ? j : NF - 1)) * NF + li] : 0.0;
    }
#pragma unroll
    for (int w = 0; w < NP; ++w) {
      y0 += t[w] * L.beta[k * NB + 3 * w];
      y1 += t[w] * L.beta[k * NB + 3 * w + 1];
      y2 += t[w] * L.beta[k * NB + 3 * w + 2];
    }
    gbwd(T15 * y0, T15 * y1, T15 * y2, out);
  };
  // c = N^T u for the working set, u in L.u
  auto nt_u = [&](double& c0, double& c1) {
    c0 = e0 < q ? ndot(e0, L.u) : 0.0;
    c1 = e1 < q ? ndot(e1, L.u) : 0.0;
  };
  // L_S^-1 v (kFwd) or L_S^-T v on the first qq entries: products with W or its
  // transpose, four rows in flight, where substitution with L_S waits for each
  // entry before the next (1,024 paths: 4.70 -> 4.46 ms; eight rows in flight: 4.50,
  // and slower on short working sets).  Entries from qq on
  // come out 0.  Up to 64 rows each lane has one entry and the second slot's
  // work is left out.
  auto w_times = [&](auto fwd, auto two, double& v0, double& v1, int qq) {
    constexpr bool kFwd = decltype(fwd)::value, kTwo = decltype(two)::value;
    constexpr int kV = 4;
    const int o0 = row_at(e0 < qq ? e0 : 0), o1 = row_at(e1 < qq ? e1 : 0);
    double y0 = 0.0, y1 = 0.0;
    for (int k0 = 0; k0 < qq; k0 += kV) {
      double x0[kV], x1[kV];
#pragma unroll
      for (int u = 0; u < kV; ++u) {
        const int k = k0 + u, kr = k < qq ? row_at(k) : 0;
        const bool on0 = kFwd ? k <= e0 && e0 < qq : e0 <= k && k < qq;
        const bool on1 = kFwd ? k <= e1 && e1 < qq : e1 <= k && k < qq;
        x0[u] = L.W[on0 ? (kFwd ? o0 + k : kr + e0) : 0];
        x0[u] = on0 ? x0[u] : 0.0;
        if (kTwo) {
          x1[u] = L.W[on1 ? (kFwd ? o1 + k : kr + e1) : 0];
          x1[u] = on1 ? x1[u] : 0.0;
        }
      }
#pragma unroll
      for (int u = 0; u < kV; ++u) {
        const int k = k0 + u;
        const double vk = k >= qq ? 0.0 : kTwo ? pick(v0, v1, k) : wave::bcast(v0, k & (kWave - 1));
        y0 += x0[u] * vk;
        if (kTwo) y1 += x1[u] * vk;
      }
    }
    v0 = y0;
    v1 = y1;
  };
  auto ls_forward = [&](double& v0, double& v1, int qq) {
    if (qq <= 0) return;
    if (qq <= kWave) w_times(std::true_type{}, std::false_type{}, v0, v1, qq);
    else w_times(std::true_type{}, std::true_type{}, v0, v1, qq);
  };
  auto ls_backward = [&](double& v0, double& v1, int qq) {
    if (qq <= 0) return;
    if (qq <= kWave) w_times(std::false_type{}, std::false_type{}, v0, v1, qq);
    else w_times(std::false_type{}, std::true_type{}, v0, v1, qq);
  };
  // w = N r (global), r given by entries (r0, r1): each lane sums its own
  // entries of w over the rows whose window holds them
  auto n_times = [&](double r0, double r1, double* out) {
    const int g0 = e0 < q ? L.actseg[e0] : 0, g1 = e1 < q ? L.actseg[e1] : 0;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < q; k0 += 4) {
      double b[4][3], rk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u < q ? k0 + u : q - 1;
        const int sgk = __builtin_amdgcn_readlane(k < kWave ? g0 : g1, k & (kWave - 1));
        rk[u] = k0 + u < q ? pick(r0, r1, k) : 0.0;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const int w = lane + kWave * t - 3 * ((P - 2) * sgk - 1);
          b[u][t] = (w >= 0 && w < NC) ? L.beta[k * NB + w] : 0.0;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < 3; ++t) acc[t] += rk[u] * b[u][t];
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (lane + kWave * t < n) out[lane + kWave * t] = acc[t];
    sync();
  };
  auto set_bit = [&](int id, bool on) {
    if (lane == 0) {
      if (on) L.actbits[id >> 5] |= (1u << (id & 31));
      else L.actbits[id >> 5] &= ~(1u << (id & 31));
    }
  };
  // row constant at x = 0 (only rows of the last segment touching the goal)
  auto row_const = [&](int id) -> double {
    const int s = seg_of(id);
    if (s != S - 1) return 0.0;
    const int loc = id - L.rowoff[s];
    return alpha_at(s, loc, 3 * P) * dg[0] + alpha_at(s, loc, 3 * P + 1) * dg[1] +
           alpha_at(s, loc, 3 * P + 2) * dg[2];
  };
  // full-row bound with side: side * bound
  auto row_e = [&](int id, int side) -> double {
    const int s = seg_of(id);
    double lo, hi;
    row_bounds(s, id - L.rowoff[s], lo, hi);
    return side > 0 ? hi : -lo;
  };
  // constraint (id, side) with free right-hand side e_free becomes entry q of the
  // working set, its normal in beta slot q
  auto enter = [&](int id, int side, double e_free) {
    if (lane == 0) { L.actid[q] = id; L.actside[q] = side; L.acte[q] = e_free; }
    set_bit(id, true);
  };
  // the factor's row of entry q: r = S^-1 N^T G^-1 n in (r0, r1) and zz = d^T G^-1 d,
  // d = n - N r, for its normal n
  auto append_factor = [&](double r0, double r1, double zz) {
    const int ro = row_at(q);
    const double id_q = 1.0 / sqrt(zz);
    if (e0 < q) L.W[ro + e0] = -r0 * id_q;
    if (e1 < q) L.W[ro + e1] = -r1 * id_q;
    if (lane == 0) L.W[ro + q] = id_q;
    ++q;
    sync();
  };
  // Remove working-set row kd.  W S W^T = 1, so an orthogonal combination of
  // the rows of W that leaves column kd to one row alone, which goes, is the new
  // factor once column kd is dropped: rotations of (what is carried, row j + 1)
  // for j = kd, kd + 1, ..  keep it triangular.  A lane rotates its own columns
  // and writes row j where row j was read before, so nothing waits for another
  // lane's store.
  // What a column loses with the row that goes cancels in it: its rounding errors
  // stay and grow, against what is left, by the ratio of the two, which is one over
  // the angle for a row nearly parallel to the dropped one.  Where it passes
  // kMaxGrowth for some column, the rows from kd on are marked to be appended again
  // (entries q .. pending-1), which the loops around do before anything else.  With
  // pairs of rows 3e-5 apart in a warm start, the largest excess of a returned point
  // over a bound: 3e-10 without this, 6e-13 with it (7e-13 where L_S is kept); 256,
  // 1,024 and 8,192 paths take 3.59, 4.40 and 13.6 ms either way.
  constexpr double kMaxGrowth = 32.0;
  int pending = 0;
  auto drop = [&](int kd) {
    set_bit(L.actid[kd], false);
    // ids, sides, right-hand sides: entries e0 and e1 take their successors'
    const int s0i = e0 >= kd && e0 < q - 1 ? e0 + 1 : -1, s1i = e1 >= kd && e1 < q - 1 ? e1 + 1 : -1;
    int id0 = 0, sd0 = 0, sg0 = 0, id1 = 0, sd1 = 0, sg1 = 0;
    double ev0 = 0.0, ev1 = 0.0;
    sync();
    if (s0i >= 0) { id0 = L.actid[s0i]; sd0 = L.actside[s0i]; sg0 = L.actseg[s0i]; ev0 = L.acte[s0i]; }
    if (s1i >= 0) { id1 = L.actid[s1i]; sd1 = L.actside[s1i]; sg1 = L.actseg[s1i]; ev1 = L.acte[s1i]; }
    sync();
    if (s0i >= 0) { L.actid[e0] = id0; L.actside[e0] = sd0; L.actseg[e0] = sg0; L.acte[e0] = ev0; }
    if (s1i >= 0) { L.actid[e1] = id1; L.actside[e1] = sd1; L.actseg[e1] = sg1; L.acte[e1] = ev1; }
    // the cached normals, four rows in flight
    for (int k0 = kd; k0 < q - 1; k0 += 4) {
      double bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) bv[u] = (k0 + u < q - 1 && lane < NC) ? L.beta[(k0 + u + 1) * NB + lane] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k0 + u < q - 1 && lane < NC) L.beta[(k0 + u) * NB + lane] = bv[u];
    }
    {
      // entry j takes entry j + 1 (entry 64 comes from lane 0's second slot)
      const double up0 = __shfl(lam0, (lane + 1) & (kWave - 1), kWave);
      const double up1 = __shfl(lam1, (lane + 1) & (kWave - 1), kWave);
      const double first1 = wave::bcast(lam1, 0);
      const double n0 = (lane == kWave - 1) ? first1 : up0;
      if (e0 >= kd && e0 < q - 1) lam0 = n0;
      if (e1 >= kd && e1 < q - 1) lam1 = up1;
    }
    sync();
    auto at0 = [&](int j) { return (e0 <= j && j < q) ? L.W[row_at(j) + e0] : 0.0; };
    auto at1 = [&](int j) { return (e1 <= j && j < q) ? L.W[row_at(j) + e1] : 0.0; };
    double c0 = at0(kd), c1 = at1(kd), x0n = at0(kd + 1), x1n = at1(kd + 1);
    double a = pick(c0, c1, kd);
    const int w0 = e0 > kd ? e0 - 1 : e0, w1 = e1 > kd ? e1 - 1 : e1;
    // squared lengths of what is left of this lane's columns (at least: of the rows
    // before kd their diagonal entries alone)
    const double d0 = e0 < kd ? L.W[row_at(e0) + e0] : 0.0, d1 = e1 < kd ? L.W[row_at(e1) + e1] : 0.0;
    double left0 = d0 * d0, left1 = d1 * d1;
    for (int j = kd; j < q - 1; ++j) {
      const double x0c = x0n, x1c = x1n;
      x0n = at0(j + 2);
      x1n = at1(j + 2);
      const double b = pick(x0c, x1c, kd);
      const double r2 = a * a + b * b, ir = rsqrt_nr(r2);
      const double cg = a * ir, sg = b * ir;
      const double v0 = cg * x0c - sg * c0, v1 = cg * x1c - sg * c1;   // 0 above the diagonal
      left0 = fma(v0, v0, left0);
      left1 = fma(v1, v1, left1);
      if (e0 != kd && e0 <= j + 1) L.W[row_at(j) + w0] = v0;
      if (e1 != kd && e1 <= j + 1) L.W[row_at(j) + w1] = v1;
      c0 = cg * c0 + sg * x0c;
      c1 = cg * c1 + sg * x1c;
      a = r2 * ir;
    }
    constexpr double kG2 = kMaxGrowth * kMaxGrowth;
    const bool redo = __ballot(kd < q - 1 && ((e0 < q && e0 != kd && !(c0 * c0 <= kG2 * left0)) ||
                                              (e1 < q && e1 != kd && !(c1 * c1 <= kG2 * left1)))) != 0ull;
    --q;
    if (e0 >= q) lam0 = 0.0;
    if (e1 >= q) lam1 = 0.0;
    pending = redo ? q : 0;
    if (redo) q = kd;
    sync();
  };
  // smallest of the entries < q, lowest index on ties
  auto min_entry = [&](double v0, double v1, double& mn, int& kd) {
    mn = e0 < q ? v0 : 1.0;
    kd = e0;
    if (e1 < q && v1 < mn) { mn = v1; kd = e1; }
    wave::argmin(mn, kd);
  };
  auto nplus_dot = [&](int slot, const double* v) -> double { return ndot(slot, v); };

  // the full pass continues from the working set the reduced-cap pass held
  // when it overflowed (the same rows in the same order: appending them and
  // solving for their multipliers restores its iterate)
  if (A.retry_only) {
    ncand = A.ws_meta[2 * ch];
    steps = A.ws_meta[2 * ch + 1];
    for (int t = lane; t < ncand; t += kWave) L.cand[t] = A.ws_keys[(int64_t)ch * A.ws_stride + t];
    sync();
  }
  // ---- warm start from the ADMM proposals (or the stored working set)
  do {
    for (int t = 0; t < ncand && q < QC - 1; ++t) {
      const int key = L.cand[t];
      const int id = key >> 1, side = (key & 1) ? 1 : -1;
      if ((L.actbits[id >> 5] >> (id & 31)) & 1u) continue;
      load_normal(id, side, q);
      gsolve_window(q, L.actseg[q], L.u);
      double c0, c1;
      nt_u(c0, c1);
      const double nu = nplus_dot(q, L.u);
      double l0 = c0, l1 = c1;
      ls_forward(l0, l1, q);
      const double ll = wave::sum((e0 < q ? l0 * l0 : 0.0) + (e1 < q ? l1 * l1 : 0.0));
      const double zz = nu - ll;
      if (zz > 1e-10 * nu) {
        ls_backward(l0, l1, q);
        enter(id, side, row_e(id, side) - double(side) * row_const(id));
        append_factor(l0, l1, zz);
      }
    }
    // dual feasibility of the working set: S lam = N^T x_u - e
    for (int guard = 0; guard <= QC; ++guard) {
      if (q == 0) break;
      double r0 = e0 < q ? ndot(e0, L.xu) - L.acte[e0] : 0.0;
      double r1 = e1 < q ? ndot(e1, L.xu) - L.acte[e1] : 0.0;
      ls_forward(r0, r1, q);
      ls_backward(r0, r1, q);
      lam0 = e0 < q ? r0 : 0.0;
      lam1 = e1 < q ? r1 : 0.0;
      double mn;
      int kd;
      min_entry(lam0, lam1, mn, kd);
      if (mn >= 0.0) break;
      drop(kd);
      if (q < pending) break;
    }
    // rows that a drop left to be appended again: once more through the proposals
    ncand = pending - q;
    for (int t = lane; t < ncand; t += kWave) {
      const int id = L.actid[q + t];
      L.cand[t] = 2 * id + (L.actside[q + t] > 0 ? 1 : 0);
    }
    sync();
    for (int t = 0; t < ncand; ++t) set_bit(L.cand[t] >> 1, false);
    pending = 0;
    sync();
  } while (ncand > 0);
  // dual value relative to the unconstrained minimum, 1/2 |N lam|^2 in the
  // metric G^-1 at the warm start; each step adds t (s+ - t zz / 2)
  double dual = 0.0;
  if (q > 0) {
    n_times(lam0, lam1, L.w);
    {
      double f0, f1, f2;
      gfwd(L.w, f0, f1, f2);
      dual = 0.5 * wave::sum(lane < NF ? f0 * f0 + f1 * f1 + f2 * f2 : 0.0);
    }
    gsolve(L.w, L.zv);
    for (int e = lane; e < n; e += kWave) L.x[e] = L.xu[e] - L.zv[e];
    sync();
  }
  // FP64 check of the dual bound for multipliers lp >= 0 on the entering
  // row (normal in np) and max(lam, 0) on the working set: every feasible
  // x has f(x) >= min_x f(x) + rho'x - mu'e = f(x_u) + rho'x_u -
  // 1/2 rho' G^-1 rho - mu'e  (rho = sum mu_k n_k); certified when that
  // exceeds f(x_u) + Ub.  Uses L.w and L.zv as scratch.
  auto dual_bound_certified = [&](double e_free, double lp) -> bool {
    const double m0 = e0 < q ? fmax(lam0, 0.0) : 0.0, m1 = e1 < q ? fmax(lam1, 0.0) : 0.0;
    n_times(m0, m1, L.w);
    double mb = lp * e_free, mbabs = fabs(mb);
    for (int k = 0; k < q; ++k) {
      const double t = pick(m0, m1, k) * L.acte[k];
      mb += t;
      mbabs += fabs(t);
    }
    for (int e = lane; e < n; e += kWave) L.zv[e] = lp * L.np[e] + L.w[e];
    sync();
    double f0, f1, f2;
    gfwd(L.zv, f0, f1, f2);
    const double rgr = wave::sum(lane < NF ? f0 * f0 + f1 * f1 + f2 * f2 : 0.0);
    double rxu = 0.0;
    for (int e = lane; e < n; e += kWave) rxu += L.zv[e] * L.xu[e];
    rxu = wave::sum(rxu);
    const double D = rxu - 0.5 * rgr - mb;
    sync();
    return D > Ub + 1e-9 * (fabs(rxu) + 0.5 * rgr + mbabs + Ub) + 1e-12;
  };
  int bound_tries = 0;

  // ---- main loop
  bool infeasible = false;
  while (true) {
    build_points(L.x);
    double best, viol;
    int key;
    scan(best, key, viol);
    if (!(best > 0.0)) { status = kSolved; break; }
    if (q >= QC - 1 && QC < A.q_full) {
      for (int k = lane; k < q; k += kWave)
        A.ws_keys[(int64_t)ch * A.ws_stride + k] = 2 * L.actid[k] + (L.actside[k] > 0 ? 1 : 0);
      if (lane == 0) { A.ws_meta[2 * ch] = q; A.ws_meta[2 * ch + 1] = steps; }
      status = kRetry;
      break;
    }
    if (steps >= max_steps || key < 0 || (key >> 1) >= m || q >= QC - 1) { status = kPolishFailed; break; }
    const int id = key >> 1, side = (key & 1) ? 1 : -1;
    const double e_full = row_e(id, side);
    double splus = viol;                    // side * value - e_full, from the lane that owns the row
    const double e_free = e_full - double(side) * row_const(id);
    load_normal(id, side, q);       // slot q holds the entering normal
    // slot q after the set has changed: a row to be appended again, or the entering one
    auto reload = [&]() {
      const bool again = q < pending;
      load_normal(again ? __builtin_amdgcn_readfirstlane(L.actid[q]) : id,
                  again ? __builtin_amdgcn_readfirstlane(L.actside[q]) : side, q);
    };
    double lamp = 0.0;
    bool added = false;
    while (!added) {
      const bool again = q < pending;       // first the rows that a drop left to be appended again
      gsolve_window(q, L.actseg[q], L.u);     // u = G^-1 n+
      double c0, c1;
      nt_u(c0, c1);                           // c = N^T u
      double r0 = c0, r1 = c1;                // r = S^-1 c
      ls_forward(r0, r1, q);
      ls_backward(r0, r1, q);
      if (e0 >= q) r0 = 0.0;
      if (e1 >= q) r1 = 0.0;
      n_times(r0, r1, L.w);                   // w = N r
      // d = n+ - N r; z = G^-1 d and zz = d^T G^-1 d = |L^-1 d|^2, a sum of
      // squares that is small exactly when n+ lies in the span of N
      for (int e = lane; e < n; e += kWave) L.zv[e] = L.np[e] - L.w[e];
      sync();
      double f0, f1, f2;
      gfwd(L.zv, f0, f1, f2);
      const double zz = wave::sum(lane < NF ? f0 * f0 + f1 * f1 + f2 * f2 : 0.0);
      if (again) {
        append_factor(r0, r1, zz);
        reload();
        continue;
      }
      ++steps;
      gbwd(f0, f1, f2, L.zv);
      const double nu = nplus_dot(q, L.u);
      const double rmax = wave::max(fmax(fabs(r0), fabs(r1)));
      double t1 = __builtin_huge_val();
      int kd = e0;
      if (e0 < q && r0 > 1e-13 * rmax) t1 = lam0 / r0;
      if (e1 < q && r1 > 1e-13 * rmax && lam1 / r1 < t1) { t1 = lam1 / r1; kd = e1; }
      wave::argmin(t1, kd);
      // below this ratio the entering normal counts as dependent: the Schur
      // solve for r carries a relative error of about cond(S) * 1e-16
      const bool zfull = zz > 1e-14 * fmax(nu, 1e-300) && zz > 0.0;
      const double t2 = zfull ? splus / zz : __builtin_huge_val();
      if (!(t1 < 1e300) && !(t2 < 1e300)) {
        // Farkas vector: 1 on the entering constraint, -r_k >= 0 on the working set
        const double wk0 = e0 < q ? fmax(-r0, 0.0) : 0.0, wk1 = e1 < q ? fmax(-r1, 0.0) : 0.0;
        n_times(wk0, wk1, L.w);
        double beta_v = e_free;
        double wabs = fabs(e_free);
        for (int k = 0; k < q; ++k) {
          const double wkk = pick(wk0, wk1, k);
          beta_v += wkk * L.acte[k];
          wabs += fabs(wkk * L.acte[k]);
        }
        // rho = n+ + N w on the free variables; minimum of rho.x over the box
        double mb = 0.0;
        bool empty = false;
        for (int e = lane; e < n; e += kWave) {
          const double rr = L.np[e] + L.w[e];
          double lo, hi;
          box_of(e, lo, hi);
          empty |= lo > hi;
          mb += rr > 0.0 ? rr * lo : rr * hi;
        }
        mb = wave::sum(mb);
        const bool ok = (__ballot(empty) != 0ull) || (beta_v < mb - 1e-12 * (1.0 + wabs));
        status = ok ? kInfeasible : kPolishFailed;
        infeasible = true;
        break;
      }
      const double t = fmin(t1, t2);
      dual += t * (splus - 0.5 * t * (zfull ? zz : 0.0));
      if (zfull) {
        for (int e = lane; e < n; e += kWave) L.x[e] -= t * L.zv[e];
      }
      if (e0 < q) lam0 -= t * r0;
      if (e1 < q) lam1 -= t * r1;
      lamp += t;
      if (zfull) splus -= t * zz;
      sync();
      // the dual value passed the box bound: try the FP64 certificate
      if (bound_tries < 4 && dual > Ub * (1.0 + 1e-9) + 1e-12) {
        ++bound_tries;
        if (dual_bound_certified(e_free, lamp)) {
          status = kInfeasible;
          infeasible = true;
          break;
        }
      }
      if (t2 <= t1) {
        enter(id, side, e_free);
        append_factor(r0, r1, zz);
        if (e0 == q - 1) lam0 = lamp;
        if (e1 == q - 1) lam1 = lamp;
        added = true;
      } else {
        drop(kd);
        reload();
        if (steps >= max_steps) break;
      }
    }
    if (infeasible || !added) { if (!infeasible) status = kPolishFailed; break; }
  }

  if (lane == 0 && A.iters_out) { A.iters_out[2 * ch] = K_admm; A.iters_out[2 * ch + 1] = steps; }
  if (status != kSolved) { finish(status); return; }

  // ---- KKT residuals, cost, write-back
  build_points(L.x);
  double pres = 0.0, pscale = 0.0;
  for (int s = 0; s < S; ++s) {
    const int ms = L.rowoff[s + 1] - L.rowoff[s];
    for (int loc = lane; loc < ms; loc += kWave) {
      double lo, hi;
      row_bounds(s, loc, lo, hi);
      const double v = row_value(s, loc, L.Pseg + s * NC);
      pres = fmax(pres, v - hi);
      pscale = fmax(pscale, fmax(fabs(v), fabs(hi)));
      if (isfinite(lo)) pres = fmax(pres, lo - v);
    }
  }
  pres = wave::max(pres);
  pscale = wave::max(pscale);
  // stationarity on the free variables: G x + q + N lam
  n_times(fmax(lam0, 0.0), fmax(lam1, 0.0), L.w);
  double st = 0.0, sg = 0.0, sn = 0.0;
  for (int e = lane; e < n; e += kWave) {
    const int i = e / 3, c = e - 3 * (e / 3);
    double gx = 0.0;
    for (int d = -P; d <= P; ++d) {
      const int j = i + d;
      if (j < 0 || j >= NF) continue;
      const int hi_ = i > j ? i : j, lo_ = i > j ? j : i;
      gx += L.G1b[(hi_ + 1) * (P + 1) + (hi_ - lo_)] * L.x[3 * j + c];
    }
    gx += L.qv[e];
    st = fmax(st, fabs(gx + L.w[e]));
    sg = fmax(sg, fabs(gx));
    sn = fmax(sn, fabs(L.w[e]));
  }
  const double dres = wave::max(st) / (1.0 + fmax(wave::max(sg), wave::max(sn)));
  double cres = 0.0, lmax = 0.0;
  for (int k = 0; k < q; ++k) {
    const double lk = fmax(pick(lam0, lam1, k), 0.0);
    const int id = L.actid[k];
    const int s = seg_of(id);
    const double v = row_value(s, id - L.rowoff[s], L.Pseg + s * NC);
    const double slack = row_e(id, L.actside[k]) - double(L.actside[k]) * v;
    cres = fmax(cres, lk * fabs(slack));
    lmax = fmax(lmax, lk);
  }
  cres /= (1.0 + lmax);
  const double kkt = fmax(fmax(fmax(pres, 0.0) / (1.0 + pscale), dres), cres);
  // cost = sum_s sum_c P~^T Q1 P~ / T^3
  double cst = 0.0;
  for (int e = lane; e < S * NC; e += kWave) {
    const int s = e / NC, r = e - NC * (e / NC), a = r / 3, c = r - 3 * (r / 3);
    double v = 0.0;
    for (int b = 0; b < NP; ++b) v += K.Q1[a][b] * L.Pseg[s * NC + 3 * b + c];
    cst += v * L.Pseg[e];
  }
  const double cost = wave::sum(cst) * iT3;
  for (int e = lane; e < S * NC; e += kWave) A.P_out[pbase + e] = L.Pseg[e] + sel3(e % 3, x0[0], x0[1], x0[2]);
  if (lane == 0) {
    const bool ok = kkt <= A.kkt_tol && isfinite(kkt) && isfinite(cost);
    A.cost_out[ch] = cost;
    A.status_out[ch] = ok ? kSolved : kNumerical;
    A.kkt_out[ch] = kkt;
  }
}

template <int P>
__global__ __launch_bounds__(64) void chain_kernel(ChainArgs A) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x + A.inst_base;
  if (b >= A.N) return;
  const int ch = A.order ? A.order[b] : b;
  if (A.retry_only && A.status_out[ch] != kRetry) return;
  chain_instance<P, false>(A, ch, smem);
}

// The full-cap pass, and small batches whole: LDS (66-138 KB) and registers
// allow one path per CU or two, so with one wavefront per path the CU's SIMDs
// idle, and a launch ends with its slowest path.  1,024 paths of 4-12 segments,
// polish only: 8.57 ms with one wavefront per path in the full-cap pass, 6.83 ms
// with four.
template <int P>
__global__ __launch_bounds__(64 * kTeamWaves) void chain_team_kernel(ChainArgs A) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int b = blockIdx.x + A.inst_base;
  if (b >= A.N) return;
  const int ch = A.order ? A.order[b] : b;
  const bool mine = !A.retry_only || A.status_out[ch] == kRetry;
  __syncthreads();   // every wavefront has read the status before the first overwrites it
  if (!mine) return;
  chain_instance<P, true>(A, ch, smem);
  // helpers leave chain_instance at this job; the first wavefront posts it
  // wherever it left the method
  if (threadIdx.x < kWave) {
    if (threadIdx.x == 0) *reinterpret_cast<int*>(smem + A.dims.o_team) = kJobExit;
    __syncthreads();
  }
}

}  // namespace

ChainDims make_chain_dims(int p, int s_cap, int nf_cap, int r_cap, int q_cap, bool admm, bool team) {
  ChainDims d{};
  d.team = team ? 1 : 0;
  d.s_cap = s_cap < 1 ? 1 : s_cap;
  d.nf_cap = nf_cap < 1 ? 1 : nf_cap;
  d.r_cap = r_cap < 1 ? 1 : r_cap;
  d.q_cap = q_cap;
  d.nf_pts_cap = (p - 1) + (d.s_cap - 1) * (p - 2);
  d.ng_cap = d.nf_pts_cap + 2;
  d.n_cap = 3 * d.nf_pts_cap;
  d.m_cap = d.s_cap * ((p + 1) * d.nf_cap + 6 * p - 3 + d.r_cap);
  const int NP = p + 1, NC = 3 * NP, BW = NC - 1;
  int o = 0;
  auto take = [&](int bytes) { const int at = o; o += (bytes + 15) & ~15; return at; };
  d.o_segi = take((4 * d.s_cap + 1) * 4);
  d.o_seg64 = take(2 * d.s_cap * 8);
  d.o_Af = take(d.s_cap * d.nf_cap * 3 * 8);
  d.o_bfs = take(d.s_cap * d.nf_cap * 8);
  d.o_fan = take(d.s_cap * d.nf_cap * 4);
  d.o_rb = take(d.s_cap * d.r_cap * 8);
  d.o_rn = take(d.s_cap * d.r_cap * 4);
  d.o_Pseg = take(d.s_cap * NC * 8);
  d.o_gfull = take(3 * d.ng_cap * 8);
  d.o_G1b = take(d.ng_cap * NP * 8);
  d.o_qv = take(2 * 3 * d.nf_pts_cap * 8);
  d.o_x = take(d.n_cap * 8);
  d.o_scal = take(16 * 8);
  d.o_cand = take(d.q_cap * 4);
  d.o_bits = take(((d.m_cap + 31) / 32) * 4);
  const int region = o;
  int a = region;
  auto take_a = [&](int bytes) { const int at = a; a += (bytes + 15) & ~15; return at; };
  // the window Hessians are built during set-up whether or not ADMM runs
  d.o_Wm = take_a(2 * NP * NP * 8);
  const int setup_end = a;
  d.o_Kb = take_a(d.n_cap * (BW + 1) * 4);
  d.o_zr = take_a(d.m_cap * 4);
  d.o_yr = take_a(d.m_cap * 4);
  d.o_accp = take_a(d.s_cap * NC * 4);
  d.o_xt = take_a(d.n_cap * 4);
  d.o_Cs = take_a(NC * NC * 4);
  int b = region;
  auto take_b = [&](int bytes) { const int at = b; b += (bytes + 15) & ~15; return at; };
  d.o_W = take_b(((d.q_cap * (d.q_cap + 1)) >> 1) * 8);   // packed rows, k + 1 slots each
  d.o_beta = take_b(d.q_cap * (NC | 1) * 8);
  d.o_acte = take_b(d.q_cap * 8);
  d.o_u = take_b(4 * d.n_cap * 8);
  d.o_actid = take_b(3 * d.q_cap * 4);
  // polish only: nothing of the ADMM part but the window Hessians is used
  if (!admm) a = setup_end;
  d.bytes = a > b ? a : b;
  d.o_team = d.bytes;
  if (team) d.bytes += (2 + 3 * kTeamWaves + 3 * kWave * kTeamWaves) * 8;
  return d;
}

// L^-1 of every segment count (T = 1), in extended precision from the
// degree's Hessian: G sums the window Hessians 2 Q1 (first segment) and
// 2 M^T Q1 M, M the window map (mcoef).
static bool build_chain_tables(const DegConst& K, std::vector<double>& Lc, std::vector<double>& Lr) {
  typedef long double R;
  constexpr int P = kChainDeg, NP = P + 1;
  Lc.assign(kChainTab, 0.0);
  Lr.assign(kChainTab, 0.0);
  R M[NP][NP] = {}, W[2][NP][NP] = {};
  for (int k = 0; k < NP; ++k) M[k][k] = 1;
  M[0][0] = 0; M[0][2] = 1;
  M[1][1] = -1; M[1][2] = 2;
  M[2][0] = 1; M[2][1] = -4; M[2][2] = 4;
  for (int a = 0; a < NP; ++a)
    for (int b = 0; b < NP; ++b) {
      W[0][a][b] = R(2) * R(K.Q1[a][b]);
      for (int k = 0; k < NP; ++k)
        for (int l = 0; l < NP; ++l) W[1][a][b] += M[k][a] * R(2) * R(K.Q1[k][l]) * M[l][b];
    }
  for (int S = 1; S <= kChainMaxSeg; ++S) {
    const int NF = chain_free(S), o = chain_tab(S);
    std::vector<R> G(size_t(NF) * NF, R(0)), Li(size_t(NF) * NF, R(0));
    for (int s = 0; s < S; ++s)
      for (int a = 0; a < NP; ++a)
        for (int b = 0; b < NP; ++b) {
          const int i = (P - 2) * s + a - 1, j = (P - 2) * s + b - 1;
          if (i >= 0 && j >= 0 && i < NF && j < NF) G[size_t(i) * NF + j] += W[s > 0 ? 1 : 0][a][b];
        }
    for (int j = 0; j < NF; ++j) {              // Cholesky, lower triangle
      for (int k = 0; k < j; ++k)
        for (int i = j; i < NF; ++i) G[size_t(i) * NF + j] -= G[size_t(i) * NF + k] * G[size_t(j) * NF + k];
      const R d = G[size_t(j) * NF + j];
      if (!(d > 0)) return false;
      const R r = std::sqrt(d);
      for (int i = j; i < NF; ++i) G[size_t(i) * NF + j] /= r;
    }
    for (int c = 0; c < NF; ++c)                // its inverse, column by column
      for (int i = c; i < NF; ++i) {
        R v = i == c ? R(1) : R(0);
        for (int k = c; k < i; ++k) v -= G[size_t(i) * NF + k] * Li[size_t(k) * NF + c];
        Li[size_t(i) * NF + c] = v / G[size_t(i) * NF + i];
      }
    for (int i = 0; i < NF; ++i)
      for (int j = 0; j < NF; ++j) {
        Lc[size_t(o) + size_t(j) * NF + i] = double(Li[size_t(i) * NF + j]);
        Lr[size_t(o) + size_t(i) * NF + j] = double(Li[size_t(i) * NF + j]);
      }
  }
  return true;
}

hipError_t upload_chain_constants(int device) {
  (void)device;
  DegConst host[kMaxDeg + 1];
  std::memset(host, 0, sizeof(host));
  for (int p = kMinDeg; p <= kMaxDeg; ++p)
    if (!build_degree(p, host[p])) return hipErrorInvalidValue;
  std::vector<double> Lc, Lr;
  if (!build_chain_tables(host[kChainDeg], Lc, Lr)) return hipErrorInvalidValue;
  hipError_t e;
  if ((e = hipMemcpyToSymbol(HIP_SYMBOL(t_Lc), Lc.data(), kChainTab * sizeof(double), 0, hipMemcpyHostToDevice)) ||
      (e = hipMemcpyToSymbol(HIP_SYMBOL(t_Lr), Lr.data(), kChainTab * sizeof(double), 0, hipMemcpyHostToDevice)))
    return e;
  return hipMemcpyToSymbol(HIP_SYMBOL(c_chain_deg), host, sizeof(host), 0, hipMemcpyHostToDevice);
}

hipError_t launch_chains(const ChainArgs& a, hipStream_t s) {
  if (a.N - a.inst_base <= 0) return hipSuccess;
  if (a.P != 7) return hipErrorInvalidValue;
  if (a.dims.team)
    hipLaunchKernelGGL((chain_team_kernel<7>), dim3(a.N - a.inst_base), dim3(kWave * kTeamWaves), a.dims.bytes, s, a);
  else
    hipLaunchKernelGGL((chain_kernel<7>), dim3(a.N - a.inst_base), dim3(kWave), a.dims.bytes, s, a);
  return hipGetLastError();
}

}  // namespace rbp
