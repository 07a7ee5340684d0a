// Float64 polish and certification on the GPU (gfx950).
//
// At the optimum of the build's Eq. 1 instance every eligible coordinate
// either sits at a bound or at a kink of its piecewise-linear trade cost
// ("fixed") or inside one linear piece ("free", known slope).  Given that
// pattern and which bands / cap bind, the optimum solves one equality-
// constrained QP in float64:
//
//   gamma Sigma_FF w_F + C_F^T eta = mu_F - slope_F - gamma Sigma_FX w_X
//   C_F w_F = h      (budget, binding bands, binding cap)
//
// H = gamma Sigma_FF = gamma (B_F diag(f) B_F^T + D_F) is inverted through
// the factor space: H^-1 = (D^-1 - D^-1 B_F Kf^-1 B_F^T D^-1)/gamma with
// Kf = diag(f)^-1 + B_F^T D_F^-1 B_F (k x k, Cholesky in LDS), and the
// multipliers eta come from the Schur complement S = C H^-1 C^T.  When the
// free set does not pin every multiplier (S singular) the ADMM estimates are
// corrected by the minimum-norm step, as the fixed coordinates then decide.
//
// The certification kernel recomputes the external diagnostics of Sec.
// "External Diagnostics" in float64 (budget, box, exposure and turnover
// residuals; nonsmooth stationarity against the subdifferential of the
// trade cost and the normal cone of the box; complementarity of bands and
// cap).  A pattern that fails is refined primal-dual active-set style:
// free coordinates that left their piece are fixed at the crossed point,
// fixed coordinates whose stationarity is violated move into the adjacent
// piece, and bands / cap are switched on when violated or off when their
// multiplier has the wrong sign.
#include <climits>

#include "fqp_common.h"
#include "fqp_dense.h"
#include "fqp_kernels.h"
#include "../../include/fqp.h"

namespace fqp {

enum PState {
  PS_CAP = 0, PS_NF, PS_NX, PS_NC, PS_DONE, PS_ROUNDS,
  PS_BACT0, PS_BACT1, PS_BUP0, PS_BUP1, PS_STALL, PS_ND, PS_SIG,
  PS_BLOCK,            // the fixed row a null-direction step releases (row * 16 + code), or -1
  PS_TICK,             // row blocks of a null-direction pass that have finished (0 between passes)
  kNPState
};
static_assert(kNPState <= kPStateStride, "polish bookkeeping does not fit");

constexpr double kSnap = 1e-10;
constexpr int kSmallF = 64;               // free sets solved in row space
// the per-account kernels: one workgroup of 16 waves per account (their
// serial parts are latency bound); the row passes run on row blocks below
constexpr int kPTC = 1024;                // polish_pre
constexpr int kPW = kPT / 64;             // most waves of either

// The points, kinks and slopes of one asset's line, as scalar fields: a
// run-time index goes through the select chains below, never through an
// array, so that the structure stays in registers (an indexed array would
// live in scratch memory, one memory round trip per access).
struct Geom {
  int np;            // points on the asset's line: bounds and inner kinks
  int nk;            // kinks of the trade cost (w0 last when present)
  double p0, p1, p2, p3, p4, p5;       // the points (ascending)
  float f0, f1, f2, f3, f4, f5;        // the same points as the float32 prox evaluates them
  double k0, k1, k2, k3;               // kinks (ascending)
  double s0, s1, s2, s3, s4;           // slope of the trade cost on each side of the kinks
  double w0;
  __device__ __forceinline__ double pt(int i) const {
    return i <= 0 ? p0 : i == 1 ? p1 : i == 2 ? p2 : i == 3 ? p3 : i == 4 ? p4 : p5;
  }
  __device__ __forceinline__ double kink(int i) const {
    return i <= 0 ? k0 : i == 1 ? k1 : i == 2 ? k2 : k3;
  }
  __device__ __forceinline__ double ks(int i) const {
    return i <= 0 ? s0 : i == 1 ? s1 : i == 2 ? s2 : i == 3 ? s3 : s4;
  }
};

// eligibility, w0 and lot data of (account, row): the bitmask words, then
// one dependent load of the packed record for a held row
struct RowData {
  bool el;
  bool taxed;
  float w0;
  float lb, ub;      // box of the asset ([0, 0] when excluded)
  float b1, b2, b3, s0, s1, s2, s3;
};

// lbf / ubf: the account's scalar bounds (used without per-asset bounds)
__device__ __forceinline__ RowData row_data(const PolishArgs& A, int a, int i, float lbf,
                                            float ubf) {
  RowData r;
  const int wd = i >> 5, b = i & 31;
  const size_t wi = (size_t)a * A.W + wd;
  r.el = A.elig == nullptr || ((A.elig[wi] >> b) & 1u);
  asset_box(A, (size_t)a * A.n + i, r.el, lbf, ubf, r.lb, r.ub);
  const uint32_t hw = A.hold[wi];
  r.w0 = 0.f;
  r.taxed = false;
  r.b1 = r.b2 = r.b3 = r.s0 = r.s1 = r.s2 = r.s3 = 0.f;
  if ((hw >> b) & 1u) {
    const int idx = A.hold_ptr[a] + A.hold_pre[wi] + popc_below(hw, b);
    const float4 r0 = A.hold_rec[2 * idx], r1 = A.hold_rec[2 * idx + 1];
    r.w0 = r0.x;
    r.taxed = r0.y > 0.f;
    r.b1 = r0.y; r.b2 = r0.z; r.b3 = r0.w;
    r.s0 = r1.x; r.s1 = r1.y; r.s2 = r1.z; r.s3 = r1.w;
  }
  return r;
}

// row_data of U rows (indices clamped into the account, so every load is
// in bounds): the first-level loads of all U rows (the eligibility and
// holding words, the word's held prefix, per-asset bounds) are issued before
// the held records they index, so a thread waits for two memory round trips
// per U rows instead of two per row
template <int U>
__device__ __forceinline__ void row_data_n(const PolishArgs& A, int a, const int (&ii)[U],
                                           float lbf, float ubf, RowData (&r)[U]) {
  uint32_t ew[U], hw[U];
  int pre[U];
  float lb[U], ub[U];
  const int hp = A.hold_ptr[a];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = min(ii[u], A.n - 1);
    const size_t wi = (size_t)a * A.W + (i >> 5);
    ew[u] = A.elig ? A.elig[wi] : ~0u;
    hw[u] = A.hold[wi];
    pre[u] = A.hold_pre[wi];
    lb[u] = A.lbv ? A.lbv[(size_t)a * A.n + i] : lbf;
    ub[u] = A.ubv ? A.ubv[(size_t)a * A.n + i] : ubf;
  }
  float4 r0[U], r1[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int b = min(ii[u], A.n - 1) & 31;
    r0[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    r1[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if ((hw[u] >> b) & 1u) {
      const int idx = hp + pre[u] + popc_below(hw[u], b);
      r0[u] = A.hold_rec[2 * idx];
      r1[u] = A.hold_rec[2 * idx + 1];
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int b = min(ii[u], A.n - 1) & 31;
    RowData& q = r[u];
    q.el = (ew[u] >> b) & 1u;
    q.lb = q.el ? lb[u] : 0.f;
    q.ub = q.el ? ub[u] : 0.f;
    q.w0 = r0[u].x;
    q.taxed = r0[u].y > 0.f;
    q.b1 = r0[u].y; q.b2 = r0[u].z; q.b3 = r0[u].w;
    q.s0 = r1[u].x; q.s1 = r1[u].y; q.s2 = r1[u].z; q.s3 = r1[u].w;
  }
}

__device__ __forceinline__ void make_geom(Geom& g, float kap, bool phi, const RowData& r) {
  const float w0f = r.w0;
  const double lb = r.lb, ub = r.ub;
  g.w0 = w0f;
  // every field is written on every path (selects, not branches)
  const bool tx = phi && r.taxed, pl = phi && !r.taxed;
  const double kd = kap;
  g.nk = tx ? 4 : (pl ? 1 : 0);
  const float kf0 = tx ? w0f - r.b3 : w0f, kf1 = tx ? w0f - r.b2 : 0.f;
  const float kf2 = tx ? w0f - r.b1 : 0.f, kf3 = tx ? w0f : 0.f;
  g.k0 = tx ? (double)w0f - r.b3 : (double)w0f;
  g.k1 = tx ? (double)w0f - r.b2 : 0.0;
  g.k2 = tx ? (double)w0f - r.b1 : 0.0;
  g.k3 = tx ? (double)w0f : 0.0;
  g.s0 = tx ? -(kd + r.s3) : (pl ? -kd : 0.0);
  g.s1 = tx ? -(kd + r.s2) : (pl ? kd : 0.0);
  g.s2 = tx ? -(kd + r.s1) : 0.0;
  g.s3 = tx ? -(kd + r.s0) : 0.0;
  g.s4 = tx ? kd : 0.0;
  // points: lb, the kinks strictly inside (lb, ub), ub.  The kinks ascend, so
  // those inside are cnt of them after the first s: the list shifted by s
  // (two selects a slot), ub behind its cnt entries.  (Placing one kink after
  // another through the slots took three times the instructions, and the row
  // passes are bound by their issue.)
  const bool e0 = g.nk > 0, e1 = g.nk > 1, e2 = g.nk > 2, e3 = g.nk > 3;
  const bool a0 = g.k0 > lb, a1 = g.k1 > lb, a2 = g.k2 > lb, a3 = g.k3 > lb;
  const int s = (e0 && !a0 ? 1 : 0) + (e1 && !a1 ? 1 : 0) + (e2 && !a2 ? 1 : 0) +
                (e3 && !a3 ? 1 : 0);
  const int cnt = (e0 && a0 && g.k0 < ub ? 1 : 0) + (e1 && a1 && g.k1 < ub ? 1 : 0) +
                  (e2 && a2 && g.k2 < ub ? 1 : 0) + (e3 && a3 && g.k3 < ub ? 1 : 0);
  const bool s1 = s & 1, s2 = s & 2;
  const double t0 = s1 ? g.k1 : g.k0, t1 = s1 ? g.k2 : g.k1, t2 = s1 ? g.k3 : g.k2;
  const float h0 = s1 ? kf1 : kf0, h1 = s1 ? kf2 : kf1, h2 = s1 ? kf3 : kf2;
  g.p0 = lb; g.f0 = r.lb;
  g.p1 = cnt > 0 ? (s2 ? t2 : t0) : ub;   g.f1 = cnt > 0 ? (s2 ? h2 : h0) : r.ub;
  g.p2 = cnt > 1 ? (s2 ? g.k3 : t1) : ub; g.f2 = cnt > 1 ? (s2 ? kf3 : h1) : r.ub;
  g.p3 = cnt > 2 ? t2 : ub;               g.f3 = cnt > 2 ? h2 : r.ub;
  g.p4 = cnt > 3 ? g.k3 : ub;             g.f4 = cnt > 3 ? kf3 : r.ub;
  g.p5 = ub;                              g.f5 = r.ub;
  g.np = 1 + cnt + (ub > lb ? 1 : 0);
}

// number of kinks below x (the kinks ascend)
__device__ __forceinline__ int kinks_below(const Geom& g, double x) {
  return (g.nk > 0 && g.k0 < x ? 1 : 0) + (g.nk > 1 && g.k1 < x ? 1 : 0) +
         (g.nk > 2 && g.k2 < x ? 1 : 0) + (g.nk > 3 && g.k3 < x ? 1 : 0);
}

// slope of the trade cost (without cap) on the piece between points q, q+1
__device__ __forceinline__ void piece_slope(const Geom& g, int q, double& slope, double& sgn) {
  const double mid = 0.5 * (g.pt(q) + g.pt(q + 1));
  slope = g.ks(kinks_below(g, mid));
  sgn = (mid > g.w0) ? 1.0 : -1.0;
}

// subdifferential interval of phi + lam |. - w0| + N_box at x (with snap)
__device__ __forceinline__ void subdiff(const Geom& g, double x, double lam, double lb,
                                        double ub, double& lo, double& hi, double& snap) {
  // the first kink within kSnap of x, or -1
  const int at = (g.nk > 0 && fabs(x - g.k0) <= kSnap) ? 0
               : (g.nk > 1 && fabs(x - g.k1) <= kSnap) ? 1
               : (g.nk > 2 && fabs(x - g.k2) <= kSnap) ? 2
               : (g.nk > 3 && fabs(x - g.k3) <= kSnap) ? 3 : -1;
  // the piece below x, the piece above it
  const int il = at >= 0 ? at : kinks_below(g, x), ih = at >= 0 ? at + 1 : il;
  lo = g.ks(il) + ((il < g.nk) ? -lam : lam);
  hi = g.ks(ih) + ((ih < g.nk) ? -lam : lam);
  snap = at >= 0 ? fabs(x - g.kink(at)) : 0.0;
  if (g.nk == 0) lo = hi = 0.0;
  if (x <= lb + kSnap) { lo = -INFINITY; snap = fmax(snap, fmax(x - lb, 0.0)); }
  if (x >= ub - kSnap) { hi = INFINITY; snap = fmax(snap, fmax(ub - x, 0.0)); }
}

// sale-side tax of selling s >= 0 from lots with breakpoints b1 < b2 < b3
// and slopes t0..t3 (the last slope continues past b3)
__device__ __forceinline__ double lot_tax(double s, const RowData& r) {
  const double b1 = r.b1, b2 = r.b2, b3 = r.b3;
  double tc = r.s0 * fmin(s, b1);
  tc += (s > b1) ? r.s1 * (fmin(s, b2) - b1) : 0.0;
  tc += (s > b2) ? r.s2 * (fmin(s, b3) - b2) : 0.0;
  tc += (s > b3) ? r.s3 * (s - b3) : 0.0;
  return tc;
}


size_t polish_wk_stride(int k, int G) {
  const size_t ncol = (size_t)G + 3;
  // Waug, Y (k x ncol), CV (ncol^2), S (ncol^2), yX, Fy, sol (k), h, eta, eta0
  // (ncol), misc 16
  return 2 * (size_t)k * ncol + 2 * ncol * ncol + 3 * (size_t)k + 3 * ncol +
         (size_t)kMaxNull * ncol + (size_t)k + (size_t)G + 1 + 16;
}

struct Wk {
  double *Waug, *Y, *CV, *S, *yX, *Fy, *sol, *h, *eta, *eta0, *nul, *yF, *gsum, *misc;
};
__device__ __forceinline__ Wk wk_of(const PolishArgs& A, int a) {
  Wk w;
  const int k = A.k;
  const size_t ncol = (size_t)A.G + 3;
  double* p = A.wk + (size_t)a * A.wk_stride;
  w.Waug = p; p += (size_t)k * ncol;
  w.Y = p; p += (size_t)k * ncol;
  w.CV = p; p += ncol * ncol;
  w.S = p; p += ncol * ncol;
  w.yX = p; p += k;
  w.Fy = p; p += k;
  w.sol = p; p += k;
  w.h = p; p += ncol;
  w.eta = p; p += ncol;
  w.eta0 = p; p += ncol;
  w.nul = p; p += (size_t)kMaxNull * ncol;   // [kMaxNull][ncol] null directions
  w.yF = p; p += k;                            // F B^T w of the polished w
  w.gsum = p; p += (size_t)A.G + 1;            // group sums of the polished w
  w.misc = p;
  return w;
}

__device__ __forceinline__ bool band_active(const int* ps, int g) {
  return g < 32 ? ((ps[PS_BACT0] >> g) & 1) : ((ps[PS_BACT1] >> (g - 32)) & 1);
}
__device__ __forceinline__ bool band_upper(const int* ps, int g) {
  return g < 32 ? ((ps[PS_BUP0] >> g) & 1) : ((ps[PS_BUP1] >> (g - 32)) & 1);
}
// Four quantities reduced at once: each exchange hands on half of what a lane
// still carries, so four cost little more than one.  Lane l returns quantity
// l & 3 over its row of 16.
template <class F>
__device__ __forceinline__ double row_red4(const double (&v)[4], F f) {
  const int l = threadIdx.x;
  const bool b0 = l & 1, b1 = l & 2;
  const double x = f(b0 ? v[1] : v[0], dpp_d<0xB1>(b0 ? v[0] : v[1]));
  const double y = f(b0 ? v[3] : v[2], dpp_d<0xB1>(b0 ? v[2] : v[3]));
  double z = f(b1 ? y : x, dpp_d<0x4E>(b1 ? x : y));
  z = f(z, dpp_d<0x128>(z));                // rotated by 8, by 4: the same quantity
  return f(z, dpp_d<0x124>(z));
}
// ... over the workgroup, for its first wave (the others get nothing): sh
// takes 64 doubles a wave and 4 quantities; the caller has a barrier between
// the two halves and before sh is used again
template <class F>
__device__ __forceinline__ void put_red4(const double (&v)[4], double* sh, F f) {
  const double z = row_red4(v, f);
  if ((threadIdx.x & 12) == 0) sh[4 * (threadIdx.x >> 4) + (threadIdx.x & 3)] = z;
}
template <class F>
__device__ __forceinline__ void get_red4(double (&v)[4], const double* sh, F f) {
  // kPT / 16 = 64 partials of each quantity, one a lane
  const double4* s4 = reinterpret_cast<const double4*>(sh) + (threadIdx.x & 63);
  v[0] = s4->x; v[1] = s4->y; v[2] = s4->z; v[3] = s4->w;
  const double z = row_red4(v, f);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    v[q] = f(f(lane_d(z, q), lane_d(z, 16 + q)), f(lane_d(z, 32 + q), lane_d(z, 48 + q)));
}

// NS block sums and NM block maxima at once: one pair of barriers for all
// (sh: (NS + NM) x nwaves doubles); every thread gets the results.  Whole
// waves only.
template <int NS, int NM>
__device__ __forceinline__ void bred(double (&sv)[NS], double (&mv)[NM], double* sh) {
  const int nw = (int)(blockDim.x >> 6), wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NS; ++q) sv[q] = wave_red(sv[q], SumOp());
#pragma unroll
  for (int q = 0; q < NM; ++q) mv[q] = wave_red(mv[q], MaxOp());
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int q = 0; q < NS; ++q) sh[q * nw + wv] = sv[q];
#pragma unroll
    for (int q = 0; q < NM; ++q) sh[(NS + q) * nw + wv] = mv[q];
  }
  __syncthreads();
  // the waves' partials, one a lane of each row of 16
  const int l = min((int)threadIdx.x & 15, nw - 1);
#pragma unroll
  for (int q = 0; q < NS; ++q)
    sv[q] = lane_d(row_red(((int)threadIdx.x & 15) < nw ? sh[q * nw + l] : 0.0, SumOp()), 0);
#pragma unroll
  for (int q = 0; q < NM; ++q) mv[q] = lane_d(row_red(sh[(NS + q) * nw + l], MaxOp()), 0);
}
__device__ __forceinline__ double bsum(double v, double* sh) {
  double sv[1] = {v}, mv[1] = {0.0};
  bred<1, 1>(sv, mv, sh);
  return sv[0];
}

// row_coef with the row's label already loaded (grp, unused without band rows),
// and the sum of all constraint rows' coefficients at row i times x
__device__ __forceinline__ double row_coef_g(const PolishArgs& A, int i, int grp, int g) {
  return g < A.Gl ? (grp == g ? 1.0 : 0.0) : (double)A.half[(size_t)(g - A.Gl) * A.n + i];
}
__device__ __forceinline__ double rows_dot_g(const PolishArgs& A, int i, int grp,
                                            const double* x) {
  double s = A.Gl ? x[grp] : 0.0;
  // the halfspace rows four at a time (loads in flight together)
  for (int g0 = A.Gl; g0 < A.G; g0 += 4) {
    float b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = A.half[(size_t)(min(g0 + u, A.G - 1) - A.Gl) * A.n + i];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (g0 + u < A.G) s += (double)b[u] * x[g0 + u];
  }
  return s;
}

// Sums over a list of rows:
//   ys[j] = sum_t B~[i_t][j] w[i_t]       (thread j < k)
//   gs[g] = sum_t B~[i_t][k + g] w[i_t]   (thread g < G: the one-hot band
//           columns and the halfspace columns of B~)
// Entries are list[t] (rev = 0) or list[n - 1 - t] (rev = 1), t < cnt.
// Each wave takes kLU entries at a time, every row loaded before the first
// is used and the next entries' indices fetched meanwhile; its lanes are the
// columns (lane, lane + 64, lane + 128).  The waves' partials meet in red
// (nwaves x (k + G) doubles of LDS), summed in wave order.
constexpr int kLU = 8;
__device__ void list_sums(const PolishArgs& A, int tid, const int32_t* list, int n, int cnt,
                          int rev, const double* w, double* red, double& ys, double& gs) {
  const int k = A.k, G = A.G, kg = k + G;
  const int lane = tid & 63, wv = tid >> 6, nw = (int)(blockDim.x >> 6);
  const bool on0 = lane < kg, on1 = lane + 64 < kg, on2 = lane + 128 < kg;
  double s0 = 0.0, s1 = 0.0, s2 = 0.0;
  auto index = [&](int t) {
    t = min(t, cnt - 1);
    return rev ? list[n - 1 - t] : list[t];
  };
  int ix[kLU];
  if (kLU * wv < cnt) {
#pragma unroll
    for (int u = 0; u < kLU; ++u) ix[u] = index(kLU * wv + u);
  }
  for (int t0 = kLU * wv; t0 < cnt; t0 += kLU * nw) {
    double wt[kLU];
    float b0[kLU], b1[kLU], b2[kLU];
#pragma unroll
    for (int u = 0; u < kLU; ++u) {
      const float* row = A.Bt + (size_t)ix[u] * A.kp;
      wt[u] = w[ix[u]];
      b0[u] = on0 ? row[lane] : 0.f;
      b1[u] = on1 ? row[lane + 64] : 0.f;
      b2[u] = on2 ? row[lane + 128] : 0.f;
    }
    const int t1 = t0 + kLU * nw;
    if (t1 < cnt) {
#pragma unroll
      for (int u = 0; u < kLU; ++u) ix[u] = index(t1 + u);
    }
#pragma unroll
    for (int u = 0; u < kLU; ++u) {
      const double wu = (t0 + u < cnt) ? wt[u] : 0.0;   // the tail repeats the last entry
      s0 += (double)b0[u] * wu;
      s1 += (double)b1[u] * wu;
      s2 += (double)b2[u] * wu;
    }
  }
  __syncthreads();                       // red may alias the caller's staging
  if (on0) red[wv * kg + lane] = s0;
  if (on1) red[wv * kg + lane + 64] = s1;
  if (on2) red[wv * kg + lane + 128] = s2;
  __syncthreads();
  if (tid < k)
    for (int q = 0; q < nw; ++q) ys += red[q * kg + tid];
  if (tid < G)
    for (int q = 0; q < nw; ++q) gs += red[q * kg + k + tid];
  __syncthreads();
}

// ---------------------------------------------------------------------------
// polish_solve: classify (first round), lists, reduced KKT solve, w
// ---------------------------------------------------------------------------
// Row-space solve of a small free set (nF <= kSmallF): with the free rows'
// constraint coefficients V_r = [1, band coefficients, sgn_r | rhs_r] and
// H = gamma Sigma_FF = gamma (B_F diag(f) B_F^T + diag(d_F)), it forms H,
// factors it, solves X = H^-1 V and writes the Schur block
// S = V_C^T X = C H^-1 [C^T | rhs] the factor-space path forms by Woodbury
// (over H, which is done with by then).  It also adds sum_F sgn_r w0_r to the
// cap's right-hand side.  LDS: H [nF][kHld], V and X [nF][ncol], f and F yX
// [k], b_r . F yX [nF], 1 / L_jj [nF] (doubles), the free rows of B~'s first
// k + G columns (floats).
constexpr int kHld = kSmallF + 1;         // odd: a column of H spreads over the banks
struct SmallLds {
  double *Hs, *Vs, *Xs, *fs, *fys, *crs, *inv;
  float* Bs;
};
__device__ __forceinline__ SmallLds small_lds(double* sm, int k, int ncol) {
  SmallLds L;
  L.Hs = sm;
  L.Vs = L.Hs + kSmallF * kHld;
  L.Xs = L.Vs + kSmallF * ncol;
  L.fs = L.Xs + kSmallF * ncol;
  L.fys = L.fs + k;
  L.crs = L.fys + k;
  L.inv = L.crs + kSmallF;
  L.Bs = reinterpret_cast<float*>(L.inv + kSmallF);
  return L;
}

__device__ __forceinline__ void small_free_solve(const PolishArgs& A, int a, int tid, int nF, const int32_t* flist,
                                 const int8_t* code, const int* ps, int nc, int ncol, int cap_on,
                                 double gam, float lbf, float ubf, float kap, bool phi,
                                 const double* fy, const SmallLds& L, double* shd, double* hd,
                                 double* Sd, int& i_mine, float& w0_mine) {
  const int k = A.k, G = A.G, kg = k + G, n = A.n;
  double *Hs = L.Hs, *Vs = L.Vs, *Xs = L.Xs;
  // stage the free rows' B~, f and F yX; the thread's own free row (nF <=
  // kPT) starts its loads meanwhile
  RowData rd;
  int cd = 0;
  double mu_r = 0.0;
  if (tid < nF) {
    i_mine = flist[tid];
    cd = code[i_mine];
    mu_r = mu_at(A, (size_t)a * n + i_mine);
    rd = row_data(A, a, i_mine, lbf, ubf);
    w0_mine = rd.w0;
  }
  for (int e = tid; e < nF * kg; e += kPT) {
    const int r = e / kg, j = e % kg;
    L.Bs[e] = A.Bt[(size_t)flist[r] * A.kp + j];
  }
  for (int j = tid; j < k; j += kPT) {
    L.fs[j] = (double)A.f[j];
    L.fys[j] = fy[j];
  }
  __syncthreads();
  // b_r . F yX: one wave per free row, its lanes over the factors
  {
    const int lane = tid & 63, wv = tid >> 6;
    for (int r = wv; r < nF; r += kPW) {
      double c = 0.0;
      for (int j = lane; j < k; j += 64) c += (double)L.Bs[r * kg + j] * L.fys[j];
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
      if (lane == 0) L.crs[r] = c;
    }
  }
  __syncthreads();
  // the constraint / rhs row of the thread's free row
  double sgn_w0 = 0.0;
  if (tid < nF) {
    const int r = tid;
    Geom g;
    make_geom(g, kap, phi, rd);
    double slope, sgn;
    piece_slope(g, cd >> 1, slope, sgn);
    double* v = Vs + r * ncol;
    v[0] = 1.0;
    int col = 1;
    for (int gg = 0; gg < G; ++gg) {
      if (!band_active(ps, gg)) continue;
      v[col++] = (double)L.Bs[r * kg + k + gg];
    }
    if (cap_on) v[col++] = sgn;
    v[col] = mu_r - slope - gam * L.crs[r];
    sgn_w0 = sgn * (double)rd.w0;
  }
  sgn_w0 = bsum(sgn_w0, shd);            // (synchronises the staging)
  if (tid == 0 && cap_on) hd[nc - 1] += sgn_w0;
  // H, lower triangle
  for (int e = tid; e < nF * nF; e += kPT) {
    const int r = e / nF, c = e % nF;
    if (c > r) continue;
    const float* br = L.Bs + r * kg;
    const float* bc = L.Bs + c * kg;
    double h = 0.0;
    for (int j = 0; j < k; ++j) h += (double)br[j] * L.fs[j] * (double)bc[j];
    if (r == c) h += (double)A.d[flist[r]];
    Hs[r * kHld + c] = gam * h;
  }
  for (int e = tid; e < nF * ncol; e += kPT) Xs[e] = Vs[e];
  __syncthreads();
  chol_factor(Hs, nF, kHld, L.inv);
  chol_solve_cols(Hs, nF, kHld, L.inv, Xs, ncol);        // X = H^-1 V (ends synchronised)
  // S = V_C^T X
  for (int e = tid; e < nc * ncol; e += kPT) {
    const int q0 = e / ncol, q = e % ncol;
    double s = 0.0;
    for (int r = 0; r < nF; ++r) s += Vs[r * ncol + q0] * Xs[r * ncol + q];
    Sd[q0 * ncol + q] = s;
  }
}

// ---------------------------------------------------------------------------
// Row-block passes: an account's rows are split into blocks of kRB rows, one
// workgroup each, so that a pass over an account's rows spreads over many
// compute units (with few accounts left refining, a pass confined to one
// workgroup is bound by that unit's instruction issue).  Per-block results
// go to [m][n_sb][...] partials that a per-account kernel gathers in block
// order (deterministic).
// ---------------------------------------------------------------------------
constexpr int kRT = 256;                  // threads of a row-block workgroup
constexpr int kRR = 2;                    // rows per thread
constexpr int kRB = kRT * kRR;            // rows per block
constexpr int kRW = kRT / 64;             // waves
constexpr int kPU = 2;                    // rows per thread and step of the one-workgroup sweeps
constexpr int kSplitDir = 32;             // row blocks from which several null directions are
                                          // swept by row blocks, a launch each

// polish_rows partials per (account, block): the column sums of B~ over the
// block's nonzero fixed rows (k + G), then budget sum, turnover sum, free
// count, nonzero-fixed count, pattern signature
__host__ __device__ __forceinline__ int rpart_stride(int k, int G) { return k + G + 5; }

// rows of block b: [b kRB, b kRB + rows_in_block)
__device__ __forceinline__ int rows_in_block(int n, int b) { return min(kRB, n - b * kRB); }

// Rows of block b, by kRT threads (tid; the whole workgroup calls it, with the
// block's number or -1): (first round) the pattern of the iterate, else the
// proposals of the last failed check adopted as the pattern; the fixed
// rows' values; the block's free rows (front of its fseg segment, ascending)
// and nonzero fixed rows (back of the segment, ascending from the end); the
// partials above
struct RowsLds {
  double red[kRW * (kMaxK + kMaxG)];
  double sh[2 * kRW];
  double nw[kRB];              // the nonzero fixed rows' weights
  int wc[kRR][kRW][2];
  int nz[kRB];
  unsigned sg[kRW];
};
__device__ __forceinline__ void rows_block(const PolishArgs& A, int a, int b, int tid, int first,
                                           RowsLds& L) {
  const int k = A.k, G = A.G, n = A.n;
  const bool live = b >= 0;
  b = live ? b : 0;
  const float* par = A.par + (size_t)a * kNPar;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  int8_t* code = A.code + (size_t)a * n;
  const int8_t* prop = A.code_next + (size_t)a * n;
  double* w = A.wout + (size_t)a * n;
  const int nrow = live ? rows_in_block(n, b) : 0;
  int32_t* seg = A.fseg + (size_t)a * n + (size_t)b * kRB;
  const int lane = tid & 63, wv = tid >> 6;
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int ii[kRR], cc[kRR];
  float zz[kRR];
#pragma unroll
  for (int u = 0; u < kRR; ++u) {
    ii[u] = b * kRB + u * kRT + tid;
    const int ic = min(ii[u], n - 1);
    zz[u] = first ? A.z[(size_t)a * n + ic] : 0.f;
    cc[u] = first ? 0 : (int)prop[ic];
  }
  RowData rd[kRR];
  row_data_n<kRR>(A, a, ii, lbf, ubf, rd);
  unsigned sig = 0u;                          // signature of the pattern
  double sx = 0.0, sturn = 0.0;
  unsigned long long mf[kRR], mn[kRR];
  double vv[kRR] = {};
#pragma unroll
  for (int u = 0; u < kRR; ++u) {
    const int i = ii[u];
    int isfree = 0, isnz = 0;
    if (live && i < n) {
      Geom g;
      make_geom(g, kap, phi, rd[u]);
      int c = cc[u];
      if (first) {
        const float z = zz[u];
        // at point j (the float32 value the prox lands on), else inside the
        // piece above the inner points below z (the points ascend)
        c = (z == g.f0) ? 0 : (g.np > 1 && z == g.f1) ? 2 : (g.np > 2 && z == g.f2) ? 4
          : (g.np > 3 && z == g.f3) ? 6 : (g.np > 4 && z == g.f4) ? 8
          : (g.np > 5 && z == g.f5) ? 10 : -1;
        if (c < 0) {
          const double zd = z;
          const int q = (g.np > 2 && zd > g.p1 ? 1 : 0) + (g.np > 3 && zd > g.p2 ? 1 : 0) +
                        (g.np > 4 && zd > g.p3 ? 1 : 0) + (g.np > 5 && zd > g.p4 ? 1 : 0);
          c = (g.np == 1) ? 0 : 2 * q + 1;
          if (g.np > 1 && zd <= g.p0) c = 0;
          if (g.np > 1 && zd >= g.pt(g.np - 1)) c = 2 * (g.np - 1);
        }
        sig += (unsigned)(c + 1) * ((unsigned)i * 2654435761u + 1u);
      }
      code[i] = (int8_t)c;
      if (c & 1) {
        isfree = 1;
        w[i] = 0.0;
      } else {
        const double v = g.pt(c >> 1);
        w[i] = v;
        vv[u] = v;
        isnz = (v != 0.0);
        sx += v;
        sturn += fabs(v - (double)rd[u].w0);
      }
    }
    mf[u] = __ballot(isfree);
    mn[u] = __ballot(isnz);
  }
  if (lane == 0) {
#pragma unroll
    for (int u = 0; u < kRR; ++u) {
      L.wc[u][wv][0] = __popcll(mf[u]);
      L.wc[u][wv][1] = __popcll(mn[u]);
    }
  }
  __syncthreads();
  int pf = 0, pn = 0;
#pragma unroll
  for (int u = 0; u < kRR; ++u) {
    int bf = 0, bn = 0, tf = 0, tn = 0;
#pragma unroll
    for (int q = 0; q < kRW; ++q) {
      const int xf = L.wc[u][q][0], xn = L.wc[u][q][1];
      bf += (q < wv) ? xf : 0;
      bn += (q < wv) ? xn : 0;
      tf += xf;
      tn += xn;
    }
    if ((mf[u] >> lane) & 1ull) seg[pf + bf + __popcll(mf[u] & below)] = ii[u];
    if ((mn[u] >> lane) & 1ull) {
      const int t = pn + bn + __popcll(mn[u] & below);
      seg[nrow - 1 - t] = ii[u];
      L.nz[t] = ii[u];
      L.nw[t] = vv[u];
    }
    pf += tf;
    pn += tn;
  }
  __syncthreads();
  // column sums over the nonzero fixed rows: one wave per row, four rows a
  // step and two steps' loads in flight, the lanes over the columns (lane,
  // lane + 64, lane + 128; past the last column its repeats, dropped)
  const int kg = k + G;
  const bool on0 = lane < kg, on1 = lane + 64 < kg, on2 = lane + 128 < kg;
  const int j0 = min(lane, kg - 1), j1 = min(lane + 64, kg - 1), j2 = min(lane + 128, kg - 1);
  const bool wide1 = kg > 64, wide2 = kg > 128;            // uniform
  double c0 = 0.0, c1 = 0.0, c2 = 0.0;
  for (int t0 = 4 * wv; t0 < pn; t0 += 8 * kRW) {
    double wt[8];
    float b0[8], b1[8], b2[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + (u & 3) + (u >> 2) * 4 * kRW, tc = min(t, pn - 1);
      const float* row = A.Bt + (size_t)L.nz[tc] * A.kp;
      wt[u] = t < pn ? L.nw[tc] : 0.0;
      b0[u] = row[j0];
      if (wide1) b1[u] = row[j1];
      if (wide2) b2[u] = row[j2];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      c0 += (double)b0[u] * wt[u];
      if (wide1) c1 += (double)b1[u] * wt[u];
      if (wide2) c2 += (double)b2[u] * wt[u];
    }
  }
  if (on0) L.red[wv * kg + lane] = c0;
  if (on1) L.red[wv * kg + lane + 64] = c1;
  if (on2) L.red[wv * kg + lane + 128] = c2;
  // budget, turnover and signature partials
  sx = wave_red(sx, SumOp());
  sturn = wave_red(sturn, SumOp());
  if (lane == 0) { L.sh[wv] = sx; L.sh[kRW + wv] = sturn; }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) sig += __shfl_xor(sig, o, 64);
  if (lane == 0) L.sg[wv] = sig;
  __syncthreads();
  if (!live) return;
  double* rp = A.rpart + ((size_t)a * A.n_sb + b) * rpart_stride(k, G);
  for (int j = tid; j < kg; j += kRT) {
    double v = 0.0;
    for (int q = 0; q < kRW; ++q) v += L.red[q * kg + j];
    rp[j] = v;
  }
  if (tid == 0) {
    unsigned sg = 0u;
    for (int q = 0; q < kRW; ++q) sg += L.sg[q];
    rp[kg] = (L.sh[0] + L.sh[1]) + (L.sh[2] + L.sh[3]);
    rp[kg + 1] = (L.sh[kRW] + L.sh[kRW + 1]) + (L.sh[kRW + 2] + L.sh[kRW + 3]);
    rp[kg + 2] = pf;
    rp[kg + 3] = pn;
    rp[kg + 4] = (double)sg;
  }
}

__global__ __launch_bounds__(kRT) void polish_rows_kernel(PolishArgs A) {
  __shared__ RowsLds L;
  const int slot = blockIdx.y;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  const int* ps = A.pstate + (size_t)a * kPStateStride;
  if (!A.first_round && (ps[PS_DONE] || ps[PS_STALL])) return;
  rows_block(A, a, blockIdx.x, threadIdx.x, A.first_round, L);
}

// S eta = C H^-1 rhs - h for the multipliers of the active constraint
// columns, with S = C H^-1 C^T positive semidefinite (nc x ncol, the rhs
// column last).  A pivoted Cholesky finds the rank r; the pivot components
// are solved for, the others keep their value in eta0, and the null
// directions of S (the multipliers the free rows do not pin) go to nul
// (rows of nul_stride).  One thread; Sm (nc x nc), perm, x and v are its
// scratch.  Returns the number of null directions kept.
__device__ __forceinline__ int schur_solve(int nc, int ncol, const double* Sv, const double* hv,
                                           const double* e0, double* Sm, double* rr, int* perm,
                                           double* x, double* v, double* nul, int nul_stride) {
  double dmax = 0.0;
  for (int p = 0; p < nc; ++p) {
    perm[p] = p;
    dmax = fmax(dmax, Sv[p * ncol + p]);
    for (int q = 0; q < nc; ++q) Sm[p * nc + q] = Sv[p * ncol + q];
  }
  const double ptol = 1e-12 * dmax;
  int rank = 0;
  for (int j = 0; j < nc; ++j) {
    int best = j;
    for (int p = j + 1; p < nc; ++p)
      if (Sm[p * nc + p] > Sm[best * nc + best]) best = p;
    if (!(Sm[best * nc + best] > ptol)) break;
    if (best != j) {
      for (int q = 0; q < nc; ++q) { double t = Sm[j * nc + q]; Sm[j * nc + q] = Sm[best * nc + q]; Sm[best * nc + q] = t; }
      for (int q = 0; q < nc; ++q) { double t = Sm[q * nc + j]; Sm[q * nc + j] = Sm[q * nc + best]; Sm[q * nc + best] = t; }
      int t = perm[j]; perm[j] = perm[best]; perm[best] = t;
    }
    const double djj = sqrt(Sm[j * nc + j]);
    Sm[j * nc + j] = djj;
    for (int i = j + 1; i < nc; ++i) Sm[i * nc + j] /= djj;
    for (int i = j + 1; i < nc; ++i)
      for (int l = j + 1; l <= i; ++l) {
        Sm[i * nc + l] -= Sm[i * nc + j] * Sm[l * nc + j];
        Sm[l * nc + i] = Sm[i * nc + l];
      }
    ++rank;
  }
  // right-hand side on the pivot rows, null components from eta0
  for (int j = 0; j < nc; ++j) x[j] = (j >= rank) ? e0[perm[j]] : 0.0;
  for (int j = 0; j < rank; ++j) {
    const int pj = perm[j];
    double t = Sv[pj * ncol + nc] - hv[pj];
    for (int q = rank; q < nc; ++q) t -= Sv[pj * ncol + perm[q]] * x[q];
    x[j] = t;
  }
  for (int i = 0; i < rank; ++i) {
    double t = x[i];
    for (int l = 0; l < i; ++l) t -= Sm[i * nc + l] * x[l];
    x[i] = t / Sm[i * nc + i];
  }
  for (int i = rank - 1; i >= 0; --i) {
    double t = x[i];
    for (int l = i + 1; l < rank; ++l) t -= Sm[l * nc + i] * x[l];
    x[i] = t / Sm[i * nc + i];
  }
  for (int j = 0; j < nc; ++j) rr[perm[j]] = x[j];
  // null directions: v_piv = -L11^-T L21^T e_t, v_t = 1
  const int nd = min(nc - rank, kMaxNull);
  for (int t = 0; t < nd; ++t) {
    for (int j = 0; j < nc; ++j) v[j] = 0.0;
    v[rank + t] = 1.0;
    for (int i = rank - 1; i >= 0; --i) {
      double u = -Sm[(rank + t) * nc + i];
      for (int l = i + 1; l < rank; ++l) u -= Sm[l * nc + i] * v[l];
      v[i] = u / Sm[i * nc + i];
    }
    for (int j = 0; j < nc; ++j) nul[t * nul_stride + perm[j]] = v[j];
  }
  return nd;
}

// doubles of LDS the solve's matrices take
__host__ __device__ __forceinline__ int solve_doubles(int k, int G) {
  // factor-space path: Kf and the staged rows (then the list sums' per-wave
  // partials over Kf: 16 (k + G))
  int d = k * kf_ld(k) + stage_rows(k, G) * stage_stride(k, G + 3);
  const int lists = (kPT / 64) * (k + G);
  d = lists > d ? lists : d;
  // row-space path: H, V, X, f, F yX, b.F yX, 1 / L_jj, the free rows of B~
  // (floats)
  const int rows = kSmallF * kHld + 2 * kSmallF * (G + 3) + 2 * k + 2 * kSmallF +
                   (kSmallF / 2) * (k + G);
  return rows > d ? rows : d;
}
constexpr int kSolveVecs = 3 * kSchurW + kSmallF + kMaxK;   // the vectors behind them

// row blocks up to which the columns of their partials are summed in shares
// (the offsets of longer accounts' lists need the space)
constexpr int kGatherParts = 16384;

// what the per-account phases of a refinement round hand on in LDS
struct AcctLds {
  double mult[2 + kMaxG];      // in: of the previous pattern, out: of this one
  double fy[kMaxK];            // F B_X^T w_X (fixed rows)
  double gsum[kMaxG];          // constraint-row sums: of the fixed rows, then of the polished w
  double yF[kMaxK + 16];       // F B^T w of the polished w
  double sh[2 * kPW];
};

// the fixed rows' side of a pattern (yx, f: column tid < k)
struct PatternSums {
  int nF, nX;                  // free rows, nonzero fixed rows
  double sx, sturn;            // budget and turnover of the fixed rows
  double yx, f;
  unsigned sig;
};

// first round of a pass: the active rows, the cap and the multipliers of
// the iterate (by the first wave; the caller synchronises)
__device__ __forceinline__ void begin_pass(const PolishArgs& A, int a, const float* par, int* ps,
                                           double* mult) {
  const int tid = threadIdx.x, G = A.G;
  if (tid >= 64) return;
  // active rows, one lane each (G <= 64: one wave)
  bool act = false, up = false;
  if (tid < G) {
    const float zb = A.zb[(size_t)a * G + tid];
    const float lo = A.blo[(size_t)a * G + tid], hi = A.bhi[(size_t)a * G + tid];
    up = zb >= hi;
    act = up || zb <= lo;
    mult[2 + tid] = (double)par[P_RHOB] * (double)A.vb[(size_t)a * G + tid];
  }
  const unsigned long long ma = __ballot(act), mu = __ballot(up);
  if (tid == 0) {
    ps[PS_CAP] = isfinite(par[P_TAU]) && par[P_LAM] > 0.f;
    ps[PS_DONE] = 0;
    ps[PS_ROUNDS] = 0;
    ps[PS_STALL] = 0;
    ps[PS_BACT0] = (int)(unsigned)ma;
    ps[PS_BACT1] = (int)(unsigned)(ma >> 32);
    ps[PS_BUP0] = (int)(unsigned)mu;
    ps[PS_BUP1] = (int)(unsigned)(mu >> 32);
    mult[0] = par[P_NU];
    mult[1] = fmax((double)par[P_LAM], 0.0);
  }
}

// Whether this round leaves the account to the next block of iterations: a
// pattern with many free coordinates belongs to an iterate that is far from
// the optimum's vertex structure (the solve is costly), and a larger free set
// is solved only when the iterate shows the same pattern at two consecutive
// checks.  Uniform (s_same: one int of LDS; ends synchronised).
__device__ __forceinline__ bool gated(const PolishArgs& A, int first, int* ps,
                                      const PatternSums& X, int* s_same) {
  if (first) {
    if (threadIdx.x == 0) {
      const unsigned sig = X.sig + (unsigned)ps[PS_CAP] * 97u + (unsigned)ps[PS_BACT0] * 31u +
                           (unsigned)ps[PS_BACT1] * 7u + (unsigned)ps[PS_BUP0] * 5u +
                           (unsigned)ps[PS_BUP1] * 3u;
      *s_same = (unsigned)ps[PS_SIG] == sig;
      ps[PS_SIG] = (int)sig;
    }
    __syncthreads();
  }
  if ((A.nf_gate > 0 && X.nF > A.nf_gate) ||
      (first && A.nf_small > 0 && X.nF > A.nf_small && !*s_same)) {
    if (threadIdx.x == 0) { ps[PS_STALL] = 1; ps[PS_NF] = X.nF; atomicAdd(A.pcount + 1, 1); }
    return true;
  }
  if (threadIdx.x == 0) atomicAdd(A.pcount, 1);
  return false;
}

// the row blocks of polish_rows gathered: the free list at the front of
// flist and the nonzero fixed list at its back (both in ascending row
// order), the budget and turnover sums of the fixed rows, the pattern's
// signature, yX = B_X^T w_X and the fixed rows' constraint-row sums (ends
// synchronised)
__device__ __forceinline__ PatternSums gather_pattern(const PolishArgs& A, int a, int tid, int first,
                                                      double* smem_d, AcctLds& W) {
  const int k = A.k, G = A.G, n = A.n;
  int32_t* flist = A.flist + (size_t)a * n;         // free rows from the front
  PatternSums X;
  const int S = A.n_sb, kg = k + G, rps = rpart_stride(k, G);
  const double* rp = A.rpart + (size_t)a * S * rps;
  const int32_t* fseg = A.fseg + (size_t)a * n;
  double* s_part = smem_d;                      // [parts][kg + 2] column sums of a share of the blocks
  const bool shares = S <= kGatherParts;
  // [S + 1] free-list offsets (Kf not built yet)
  int* s_of = reinterpret_cast<int*>(smem_d + (shares ? kPT : 0));
  int* s_ox = s_of + (S + 1);                   // [S + 1] nonzero-list offsets
  __shared__ double s_sx[2];
  __shared__ unsigned s_sig;
  if (tid == 0) s_sig = 0u;
  for (int bb = tid; bb < S; bb += kPT) {
    s_of[bb + 1] = (int)rp[(size_t)bb * rps + kg + 2];
    s_ox[bb + 1] = (int)rp[(size_t)bb * rps + kg + 3];
  }
  __syncthreads();
  if (first) {                          // the pattern's signature: any order
    unsigned su = 0u;
    for (int bb = tid; bb < S; bb += kPT) su += (unsigned)rp[(size_t)bb * rps + kg + 4];
    if (su) atomicAdd(&s_sig, su);
  }
  // columns of the partials: a share of the blocks per part, sixteen blocks'
  // loads in flight a thread (past the share's end its last block's, dropped)
  const int cols = kg + 2;
  const int parts = shares ? max(1, min(kPT / cols, (S + 15) / 16)) : 1;
  const int share = (S + parts - 1) / parts;
  double col_sum = 0.0;
  if (tid < parts * cols) {
    const int j = tid % cols, b0 = (tid / cols) * share, b1 = min(S, b0 + share);
    double v = 0.0;
    for (int bb = b0; bb < b1; bb += 16) {
      double x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = rp[(size_t)min(bb + u, b1 - 1) * rps + j];
#pragma unroll
      for (int u = 0; u < 16; ++u) v += bb + u < b1 ? x[u] : 0.0;
    }
    col_sum = v;
    if (shares) s_part[tid] = v;
  }
  // block offsets of the two lists: prefix sums (a wave scan when the
  // account has at most 64 row blocks)
  if (S <= 64) {
    if (tid < 64) {
      int vf = tid < S ? s_of[tid + 1] : 0, vx = tid < S ? s_ox[tid + 1] : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int uf = __shfl_up(vf, o, 64), ux = __shfl_up(vx, o, 64);
        if (tid >= o) { vf += uf; vx += ux; }
      }
      if (tid < S) { s_of[tid + 1] = vf; s_ox[tid + 1] = vx; }
      if (tid == 0) { s_of[0] = 0; s_ox[0] = 0; }
    }
  } else if (tid < 64) {
    // 64 blocks at a time, the running totals carried by every lane
    int cf = 0, cx = 0;
    if (tid == 0) { s_of[0] = 0; s_ox[0] = 0; }
    for (int b0 = 0; b0 < S; b0 += 64) {
      const int bb = b0 + tid;
      int vf = bb < S ? s_of[bb + 1] : 0, vx = bb < S ? s_ox[bb + 1] : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int uf = __shfl_up(vf, o, 64), ux = __shfl_up(vx, o, 64);
        if (tid >= o) { vf += uf; vx += ux; }
      }
      if (bb < S) { s_of[bb + 1] = cf + vf; s_ox[bb + 1] = cx + vx; }
      cf += __shfl(vf, 63, 64);
      cx += __shfl(vx, 63, 64);
    }
  }
  __syncthreads();
  X.yx = 0.0;
  X.f = 0.0;
  if (tid < cols) {
    double v = col_sum;                     // (this thread's share is the column's first)
    for (int q = 1; q < parts; ++q) v += s_part[q * cols + tid];
    if (tid < k) {
      const double fj = (double)A.f[tid];
      W.fy[tid] = v * fj;
      X.yx = v;
      X.f = fj;
    }
    else if (tid < kg) W.gsum[tid - k] = v;
    else s_sx[tid - kg] = v;
  }
  const int nF = s_of[S], nX = s_ox[S];
  X.nF = nF;
  X.nX = nX;
  // entry e of a list lies in the last block whose offset is <= e
  auto block_of = [&](const int* off, int e) {
    int lo = 0, hi = S;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (off[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
  };
  for (int e = tid; e < nF; e += kPT) {
    const int bb = block_of(s_of, e);
    flist[e] = fseg[(size_t)bb * kRB + (e - s_of[bb])];
  }
  for (int e = tid; e < nX; e += kPT) {
    const int bb = block_of(s_ox, e);
    flist[n - 1 - e] = fseg[(size_t)bb * kRB + rows_in_block(n, bb) - 1 - (e - s_ox[bb])];
  }
  __syncthreads();
  X.sx = s_sx[0];
  X.sturn = s_sx[1];
  X.sig = s_sig;
  return X;
}

// the solve of one account's pattern by a workgroup of kPT threads; smem_d:
// dynamic LDS of polish_smem bytes; ps: its bookkeeping (global or LDS).
// vec: kSolveVecs doubles of LDS (behind the matrices in polish_solve, where
// a very long account's list offsets take all of it before).
// Leaves the free rows' weights in wout, W.mult, W.yF, W.gsum (not
// synchronised) and returns the turnover of the polished weights.
__device__ __forceinline__ double solve_pattern(const PolishArgs& A, int a, int tid, const float* par,
                                                int* ps, const PatternSums& X, double* smem_d,
                                                double* vec, AcctLds& W) {
  const int k = A.k, G = A.G, n = A.n;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const double gam = par[P_GAMMA];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  const Wk wk = wk_of(A, a);
  const int8_t* code = A.code + (size_t)a * n;
  const int32_t* flist = A.flist + (size_t)a * n;
  double* w = A.wout + (size_t)a * n;
  double* Kf = smem_d;                      // [k][kf_ld]
  double* const shd = W.sh;
  // the constraint system's vectors when it is solved in LDS, a small free
  // set's weights, 1 / L_jj of its factor or Kf's
  double* const s_h = vec;
  double *const s_e0 = s_h + kSchurW, *const s_eta = s_e0 + kSchurW, *const s_wf = s_eta + kSchurW;
  double* const s_inv = s_wf + kSmallF;
  const int cap_on = ps[PS_CAP], nF = X.nF, kg = k + G;

  // active constraint columns: 0 budget, bands (active order), cap
  const unsigned act0 = (unsigned)ps[PS_BACT0], act1 = (unsigned)ps[PS_BACT1];
  const int nb = __popc(act0) + __popc(act1);
  const int nc = 1 + nb + (cap_on ? 1 : 0);
  const int ncol = nc + 1;                      // + rhs column
  // the column of active row g
  auto col_of = [&](int g) {
    return g < 32 ? 1 + __popc(act0 & ((1u << g) - 1u))
                  : 1 + __popc(act0) + __popc(act1 & ((1u << (g - 32)) - 1u));
  };
  // a constraint system of at most kSchurW columns lives in LDS and is
  // solved by one wave
  const bool sl = nc <= kSchurW;
  double* hd = sl ? s_h : wk.h;
  double* Sd = sl ? smem_d : wk.S;              // where H or Kf was, once they are done with
  if (tid < G && band_active(ps, tid)) {
    const double bnd = band_upper(ps, tid) ? A.bhi[(size_t)a * G + tid] : A.blo[(size_t)a * G + tid];
    hd[col_of(tid)] = bnd - W.gsum[tid];
  }
  if (tid == 0) {
    hd[0] = 1.0 - X.sx;
    if (cap_on) hd[nc - 1] = (double)tauf - X.sturn;     // + sum_F sgn w0 added below
    ps[PS_NF] = nF;
    ps[PS_NX] = X.nX;
    ps[PS_NC] = nc;
  }
  __syncthreads();                          // the lists are complete, smem_d is free

  // A free set of at most kSmallF rows is solved in row space (its
  // gamma Sigma_FF is at most 64 x 64); a larger one through the factor space
  // below.
  const bool small = nF <= kSmallF;
  const SmallLds L = small_lds(smem_d, k, ncol);
  int i_mine = 0;                         // small path: the thread's free row, its w0
  float w0_mine = 0.f;
  if (small) {
    small_free_solve(A, a, tid, nF, flist, code, ps, nc, ncol, cap_on, gam, lbf, ubf, kap, phi, W.fy, L,
                     shd, hd, Sd, i_mine, w0_mine);
  } else {
  // ---- one pass over the free rows, SR staged at a time: Kf = diag(1/f) +
  // sum_F b b^T / d (lower triangle), Waug = sum_F b V^T / d and CV = sum_F
  // V V^T / d with V_i = [1, constraint rows (active order), sgn_i (cap),
  // rhs_i], rhs_i = mu_i - slope_i - gamma b_i . F yX.  A 4 x 4 register tile a
  // thread: the first ntile threads on Kf, the next on X^T D^-1 V, X = [b | V].
  const int ld = kf_ld(k), SR = stage_rows(k, G), SS = stage_stride(k, ncol);
  double* stg = Kf + k * ld;                // [SR][SS], 1 / d_i at index SS - 4
  const int kx = k + ncol, xt = (kx + 3) >> 2, vt = (ncol + 3) >> 2;
  double sgn_w0 = 0.0;
  {
    const int kt = (k + 3) >> 2;
    const int ntile = kt * (kt + 1) / 2;
    const bool own_k = tid < ntile;
    // Waug / CV tiles: from the other end of the workgroup
    const int t2 = kPT - 1 - tid;
    const bool own_v = !own_k && t2 < xt * vt;
    int tj = 0, tl = 0;
    if (own_k) {
      int j = (int)((sqrt(8.0 * tid + 1.0) - 1.0) * 0.5);
      while ((j + 1) * (j + 2) / 2 <= tid) ++j;
      while (j * (j + 1) / 2 > tid) --j;
      tj = j;
      tl = tid - j * (j + 1) / 2;
    } else if (own_v) {
      tj = t2 / vt;
      tl = t2 % vt;
    }
    // (both sets fit one workgroup up to ntile + xt vt <= kPT; wider systems
    // take their Waug / CV tiles in further rounds below)
    const bool fits = ntile + xt * vt <= kPT;
    const int rounds = fits ? 1 : 1 + (xt * vt + kPT - 1) / kPT;
    for (int rd = 0; rd < rounds; ++rd) {
      const bool do_k = rd == 0 && own_k;
      bool do_v = fits && own_v;
      if (rd > 0) {
        const int t3 = (rd - 1) * kPT + tid;
        do_v = t3 < xt * vt;
        tj = do_v ? t3 / vt : 0;
        tl = do_v ? t3 % vt : 0;
      }
      double acc[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) acc[c] = 0.0;
      for (int f0 = 0; f0 < nF; f0 += SR) {
        const int rows = min(SR, nF - f0);
        __syncthreads();
        // the row's own data, while its loadings are staged
        RowData r;
        int i = 0, cd = 0;
        double mu_r = 0.0, d_r = 1.0;
        int grp = 0;
        if (tid < rows) {
          i = flist[f0 + tid];
          cd = code[i];
          mu_r = mu_at(A, (size_t)a * n + i);
          d_r = (double)A.d[i];
          if (A.Gl) grp = A.group[i];
          r = row_data(A, a, i, lbf, ubf);
        }
        for (int e = tid; e < rows * k; e += kPT) {
          const int rr = e / k, j = e % k;
          stg[rr * SS + j] = (double)A.Bt[(size_t)flist[f0 + rr] * A.kp + j];
        }
        __syncthreads();
        if (tid < rows) {
          Geom g;
          make_geom(g, kap, phi, r);
          double slope, sgn;
          piece_slope(g, cd >> 1, slope, sgn);
          double* x = stg + tid * SS;
          double cross = 0.0;
          for (int j = 0; j < k; ++j) cross += x[j] * W.fy[j];
          double* v = x + k;
          v[0] = 1.0;
          int col = 1;
          for (int gg = 0; gg < G; ++gg) {
            if (!band_active(ps, gg)) continue;
            v[col++] = row_coef_g(A, i, grp, gg);
          }
          if (cap_on) v[col++] = sgn;
          v[col] = mu_r - slope - gam * cross;
          for (int q = kx; q < 4 * xt; ++q) x[q] = 0.0;
          x[SS - 4] = 1.0 / d_r;
          if (rd == 0) sgn_w0 += sgn * (double)r.w0;
        }
        __syncthreads();
        if (do_k || do_v) {
          const double* bj = stg + 4 * tj;
          const double* bl = stg + (do_k ? 4 * tl : k + 4 * tl);
          const int lim = do_k ? 4 : ncol - 4 * tl;           // columns past it are not stored
          for (int rr = 0; rr < rows; ++rr) {
            const double id = stg[rr * SS + SS - 4];
            double xj[4], xl[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              xj[q] = bj[rr * SS + q] * id;
              xl[q] = q < lim ? bl[rr * SS + q] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int s = 0; s < 4; ++s) acc[q * 4 + s] += xj[q] * xl[s];
          }
        }
      }
      if (do_k) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int j = 4 * tj + q, l = 4 * tl + s;
            if (j < k && l <= j) {
              double v = acc[q * 4 + s];
              if (j == l) v += factor_weight(A.f[j]);
              Kf[j * ld + l] = v;
            }
          }
      }
      if (do_v) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int j = 4 * tj + q, l = 4 * tl + s;
            if (j >= kx || l >= ncol) continue;
            if (j < k) {
              wk.Waug[j * ncol + l] = acc[q * 4 + s];
              wk.Y[j * ncol + l] = acc[q * 4 + s];
            } else {
              wk.CV[(j - k) * ncol + l] = acc[q * 4 + s];
            }
          }
      }
    }
  }
  sgn_w0 = bsum(sgn_w0, shd);
  if (tid == 0 && cap_on) hd[nc - 1] += sgn_w0;
  __syncthreads();
  // ---- Y = Kf^-1 Waug
  chol_factor(Kf, k, ld, s_inv);
  chol_solve_cols(Kf, k, ld, s_inv, wk.Y, ncol);
  // ---- Schur system on the constraint columns ------------------------------
  // gamma * C H^-1 V = CV[C, V] - Waug[:, C]^T Y[:, V]
  for (int e = tid; e < nc * ncol; e += kPT) {
    const int p = e / ncol, q = e % ncol;
    double s = wk.CV[p * ncol + q];
#pragma unroll 8
    for (int j = 0; j < k; ++j) s -= wk.Waug[j * ncol + p] * wk.Y[j * ncol + q];
    Sd[p * ncol + q] = s / gam;
  }
  }                                       // factor-space path
  // eta0: multipliers of the previous pattern (first pattern: ADMM's):
  // -nu, band duals, lam_cap
  if (sl) {
    if (tid < G && band_active(ps, tid)) s_e0[col_of(tid)] = W.mult[2 + tid];
    if (tid == 0) {
      s_e0[0] = -W.mult[0];
      if (cap_on) s_e0[nc - 1] = fmax(W.mult[1], 0.0);
    }
  }
  __syncthreads();
  if (sl) {
    if (tid < 64) {
      const int nd = schur_solve_wave(nc, ncol, smem_d, s_h, s_e0, smem_d + nc * ncol, s_eta,
                                      wk.nul, G + 3);
      if (tid == 0) ps[PS_ND] = nd;
    }
    __syncthreads();
    // multipliers in the build's convention
    if (tid < G) W.mult[2 + tid] = band_active(ps, tid) ? s_eta[col_of(tid)] : 0.0;
    if (tid == 0) {
      W.mult[0] = -s_eta[0];
      W.mult[1] = cap_on ? s_eta[nc - 1] : 0.0;
    }
  } else if (tid == 0) {
    double e0[kMaxG + 3];
    e0[0] = -W.mult[0];
    int col = 1;
    for (int g = 0; g < G; ++g)
      if (band_active(ps, g)) e0[col++] = W.mult[2 + g];
    if (cap_on) e0[col++] = fmax(W.mult[1], 0.0);
    int perm[kMaxG + 3];
    double x[kMaxG + 3], v[kMaxG + 3];
    ps[PS_ND] = schur_solve(nc, ncol, wk.S, wk.h, e0, wk.CV, wk.eta, perm, x, v, wk.nul, G + 3);
    W.mult[0] = -wk.eta[0];
    col = 1;
    for (int g = 0; g < G; ++g) W.mult[2 + g] = band_active(ps, g) ? wk.eta[col++] : 0.0;
    W.mult[1] = cap_on ? wk.eta[col] : 0.0;
  }
  __syncthreads();
  const double* etav = sl ? s_eta : wk.eta;
  double turn_f = 0.0;                    // turnover of the free rows
  if (small) {
    // w_F = H^-1 (rhs - C^T eta) = X[:, rhs] - X[:, C] eta
    if (tid < nF) {
      const int t = tid;
      double v = L.Xs[t * ncol + nc];
      for (int p = 0; p < nc; ++p) v -= L.Xs[t * ncol + p] * etav[p];
      const int i = i_mine;
      w[i] = v;
      s_wf[t] = v;
      turn_f += fabs(v - (double)w0_mine);
    }
  } else {
  // sol = Y[:, rhs] - Y[:, C] eta
  for (int j = tid; j < k; j += kPT) {
    double s = wk.Y[j * ncol + nc];
    for (int p = 0; p < nc; ++p) s -= wk.Y[j * ncol + p] * etav[p];
    wk.sol[j] = s;
  }
  __syncthreads();
  // ---- free rows: w_i = (rhs_i - C_i^T eta - b_i . sol) / (gamma d_i), 16
  // threads a row for the products
  for (int t0 = 0; t0 < nF; t0 += kPT / 16) {
    const int t = min(t0 + (tid >> 4), nF - 1), q = tid & 15;
    const int i = flist[t];
    double cross = 0.0, bs = 0.0;
    for (int j = q; j < k; j += 16) {
      const double b = (double)A.Bt[(size_t)i * A.kp + j];
      cross += b * W.fy[j];
      bs += b * wk.sol[j];
    }
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) {
      cross += __shfl_xor(cross, o, 16);
      bs += __shfl_xor(bs, o, 16);
    }
    if (q == 0 && t0 + (tid >> 4) < nF) {
      RowData r = row_data(A, a, i, lbf, ubf);
      Geom g;
      make_geom(g, kap, phi, r);
      double slope, sgn;
      piece_slope(g, code[i] >> 1, slope, sgn);
      const double rhs = mu_at(A, (size_t)a * n + i) - slope - gam * cross;
      double ct = etav[0];
      int col = 1;
      const int grp = A.Gl ? A.group[i] : 0;
      for (int gg = 0; gg < G; ++gg) {
        if (!band_active(ps, gg)) continue;
        ct += row_coef_g(A, i, grp, gg) * etav[col];
        ++col;
      }
      if (cap_on) ct += sgn * etav[col];
      const double wi = (rhs - ct - bs) / (gam * (double)A.d[i]);
      w[i] = wi;
      turn_f += fabs(wi - (double)r.w0);
    }
  }
  }                                       // factor-space path
  // turnover of the polished w: the fixed rows' (from the row blocks) plus
  // the free rows'
  turn_f = bsum(turn_f, shd);
  // ---- y = F B^T w and the row sums of the polished w (nonzero rows), for
  // the gradient base and the certification: the fixed rows' parts from
  // above plus the free rows' --------------------------------------------
  __syncthreads();
  if (small) {
    if (tid < kg) {
      double s = 0.0;
      for (int r = 0; r < nF; ++r) s += (double)L.Bs[r * kg + tid] * s_wf[r];
      if (tid < k) W.yF[tid] = (X.yx + s) * X.f;
      else W.gsum[tid - k] += s;
    }
  } else {
    double ys = 0.0, gs = 0.0;
    list_sums(A, tid, flist, n, nF, 0, w, Kf, ys, gs);     // the solve is done with Kf
    if (tid < k) W.yF[tid] = (X.yx + ys) * X.f;
    if (tid < G) W.gsum[tid] += gs;
  }
  return X.sturn + turn_f;
}

__global__ __launch_bounds__(kPT) void polish_solve_kernel(PolishArgs A) {
  extern __shared__ double smem_d[];
  __shared__ AcctLds W;
  __shared__ int s_same;
  const int slot = blockIdx.x;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot], tid = threadIdx.x, k = A.k, G = A.G;
  int* ps = A.pstate + (size_t)a * kPStateStride;
  if (!A.first_round && (ps[PS_DONE] || ps[PS_STALL])) return;
  const float* par = A.par + (size_t)a * kNPar;
  double* mult = A.mult + (size_t)a * (2 + G);
  if (A.first_round) begin_pass(A, a, par, ps, W.mult);
  else
    for (int e = tid; e < 2 + G; e += kPT) W.mult[e] = mult[e];
  const PatternSums X = gather_pattern(A, a, tid, A.first_round, smem_d, W);
  if (gated(A, A.first_round, ps, X, &s_same)) return;
  const double turn = solve_pattern(A, a, tid, par, ps, X, smem_d, smem_d + solve_doubles(k, G),
                                    W);
  // for the passes after it (a thread's own entries of yF and gsum)
  const Wk wk = wk_of(A, a);
  if (tid < k) wk.yF[tid] = W.yF[tid];
  __syncthreads();
  if (tid < G) wk.gsum[tid] = W.gsum[tid];
  if (tid < 2 + G) mult[tid] = W.mult[tid];
  if (tid == 0) wk.misc[3] = turn;
}

// ---------------------------------------------------------------------------
// polish_gbase: gb_i = gamma (Sigma w)_i - mu_i for every row, spread over
// (row block, account) workgroups; per block: max |gamma Sigma w|, max |mu|
// and a non-finite flag (slot 2 unused: the turnover comes from the solve)
// ---------------------------------------------------------------------------
constexpr int kGbRows = 256;              // rows per gbase workgroup (one per thread)
constexpr int kGbAcc = 16;                // accounts per gbase workgroup

// g_i = gamma (d_i w_i + b_i . y) - mu_i for kGbRows rows x kGbAcc accounts:
// each thread streams its row of B once (four columns at a time, from the copy
// that keeps them consecutive over rows: a wave's load of 64 rows of B~ was
// 64 lines, which did not survive in the L1 until their next four columns: 92 us a round
// at 8 x 384,800, 33 now)
// against the accounts' y vectors (LDS broadcasts), so the universe block is
// read once per 16 accounts; per-(account, row block) maxima / sums go to gpart
__global__ __launch_bounds__(256) void polish_gbase_kernel(PolishArgs A, int final_pass) {
  __shared__ double s_y[kGbAcc][kMaxK + 4];
  __shared__ int s_a[kGbAcc];
  __shared__ double s_gam[kGbAcc];
  __shared__ double s_red[4][kGbAcc][4];
  const int k = A.k, n = A.n, tid = threadIdx.x;
  const int m_act = *A.m_act;
  // the active accounts spread over every account group of the grid (at
  // most kGbAcc each): with few accounts left, more workgroups take part
  const int gs = min(kGbAcc, (m_act + (int)gridDim.y - 1) / (int)gridDim.y);
  const int g0 = blockIdx.y * gs;
  if (g0 >= m_act) return;
  if (tid < kGbAcc) {
    int a = -1;
    if (tid < gs && g0 + tid < m_act) {
      const int aa = A.act[g0 + tid];
      const int* ps = A.pstate + (size_t)aa * kPStateStride;
      if (!(ps[PS_DONE] || (ps[PS_STALL] && !final_pass))) a = aa;
    }
    s_a[tid] = a;
    s_gam[tid] = a >= 0 ? (double)A.par[(size_t)a * kNPar + P_GAMMA] : 0.0;
  }
  __syncthreads();
  const int k4 = (k + 3) & ~3;                 // <= kp: whole float4 of each row
  {
    // kGbAcc k4 <= 2048 entries: eight per thread, all loads issued first
    double yv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = tid + 256 * u;
      const int q = min(e / k4, kGbAcc - 1), j = e % k4;
      const int a = s_a[q];
      yv[u] = (e < kGbAcc * k4 && a >= 0 && j < k) ? wk_of(A, a).yF[j] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = tid + 256 * u;
      if (e < kGbAcc * k4) s_y[e / k4][e % k4] = yv[u];
    }
  }
  __syncthreads();
  // the accounts present (uniform): the products skip the others
  unsigned amask = 0u;
#pragma unroll
  for (int q = 0; q < kGbAcc; ++q) amask |= (s_a[q] >= 0 ? 1u : 0u) << q;
  amask = __builtin_amdgcn_readfirstlane(amask);
  const int i = blockIdx.x * kGbRows + tid;
  const bool row_ok = i < n;
  double sig[kGbAcc];
#pragma unroll
  for (int q = 0; q < kGbAcc; ++q) sig[q] = 0.0;
  if (row_ok) {
#pragma unroll 4
    for (int j4 = 0; j4 < k4 / 4; ++j4) {
      const float4 b = A.Bq[(size_t)j4 * n + i];
      const double b0 = b.x, b1 = b.y, b2 = b.z, b3 = b.w;
#pragma unroll
      for (int q = 0; q < kGbAcc; ++q) {
        if (!((amask >> q) & 1u)) continue;
        const double* y = &s_y[q][4 * j4];
        sig[q] += b0 * y[0] + b1 * y[1] + b2 * y[2] + b3 * y[3];
      }
    }
  }
  const double di = row_ok ? (double)A.d[i] : 0.0;
  const int wv = tid >> 6;
  // the accounts four at a time: their w and mu loads in flight together
#pragma unroll
  for (int q0 = 0; q0 < kGbAcc; q0 += 4) {
    double wq[4], mq[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int a = s_a[q0 + u];
      wq[u] = 0.0;
      mq[u] = 0.0;
      if (a >= 0 && row_ok) {
        wq[u] = A.wout[(size_t)a * n + i];
        mq[u] = mu_at(A, (size_t)a * n + i);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u;
      const int a = s_a[q];
      if (a < 0) continue;                     // uniform
      double gmax = 0.0, mumax = 0.0, bad = 0.0;
      if (row_ok) {
        const double wi = wq[u];
        const double sg = sig[q] + di * wi;
        const double mui = mq[u];
        const double v = s_gam[q] * sg - mui;
        A.gbase[(size_t)a * n + i] = v;
        gmax = fabs(s_gam[q] * sg);
        mumax = fabs(mui);
        if (!isfinite(v) || !isfinite(wi)) bad = 1.0;
      }
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        gmax = fmax(gmax, __shfl_xor(gmax, o, 64));
        mumax = fmax(mumax, __shfl_xor(mumax, o, 64));
        bad = fmax(bad, __shfl_xor(bad, o, 64));
      }
      if ((tid & 63) == 0) {
        s_red[wv][q][0] = gmax; s_red[wv][q][1] = mumax;
        s_red[wv][q][2] = 0.0; s_red[wv][q][3] = bad;
      }
    }
  }
  __syncthreads();
  if (tid < 4 * kGbAcc) {
    const int q = tid >> 2, c = tid & 3;
    const int a = s_a[q];
    if (a >= 0) {
      double v = s_red[0][q][c];
      for (int w = 1; w < 4; ++w) v = (c == 2) ? v + s_red[w][q][c] : fmax(v, s_red[w][q][c]);
      A.gpart[((size_t)a * A.n_rb + blockIdx.x) * 4 + c] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// polish_check: external diagnostics in float64 and refinement, after the
// gradient base: the null-direction sweep rows (row blocks; the common case
// of one open direction), polish_pre (per account: the gradient scale and the
// sweep decisions), for accounts of many row blocks polish_dir (a launch for each
// of several open directions), the diagnostic rows (row blocks: residual
// partials and refinement proposals) and polish_decide (per account: the
// certificate and the refinement decisions)
// ---------------------------------------------------------------------------

// Along a stored null direction v of the free-row equations the free rows
// stay stationary, and every fixed row's stationarity interval becomes a
// pair of linear inequalities in the step s.  The step aims at zeroing the
// multiplier of an active constraint that is not tight (its row was
// dependent, so the solve could not enforce it); otherwise it stays nearest
// to 0.  When a fixed row blocks that target, the row is the one to release
// (dual active-set step).
struct SweepDir {
  const double* nv;     // the direction, in the column order of eta
  double n0, ncap, lamc;
};

__device__ __forceinline__ SweepDir sweep_dir(const int* ps, const double* nv,
                                              const double* mult) {
  SweepDir D;
  D.nv = nv;
  // column of each multiplier inside eta = (-nu, bands..., lam_cap)
  D.n0 = nv[0];
  D.ncap = ps[PS_CAP] ? nv[ps[PS_NC] - 1] : 0.0;
  D.lamc = mult[1];
  return D;
}

// the direction's entry of every constraint row (0: inactive), into LDS: the
// column of an active row is 1 + the active rows before it
__device__ __forceinline__ void dir_rows(const int* ps, int G, const double* nv, double* s_nv) {
  const unsigned a0 = (unsigned)ps[PS_BACT0], a1 = (unsigned)ps[PS_BACT1];
  for (int g = threadIdx.x; g < G; g += blockDim.x) {
    const unsigned below = g < 32 ? a0 & ((1u << g) - 1u) : a1 & ((1u << (g - 32)) - 1u);
    const int col = 1 + __popc(below) + (g < 32 ? 0 : __popc(a0));
    s_nv[g] = band_active(ps, g) ? nv[col] : 0.0;
  }
}

// one row's bounds on the step: Lo <= s <= Up keeps it stationary; the keys
// name the row and the piece it would move into (row * 16 + code)
__device__ __forceinline__ void sweep_row(const PolishArgs& A, const SweepDir& D,
                                          const double* s_nv, const double* mult, int i, int c, double gbi,
                                          double wi, int grp, const RowData& r, float kap,
                                          bool phi, double& Lo, double& Up, int& loKey,
                                          int& upKey) {
  if ((c & 1) || !r.el) return;
  const int G = A.G;
  Geom g;
  make_geom(g, kap, phi, r);
  const double lb = r.lb, ub = r.ub;
  double nb = 0.0, lg = 0.0;
  if (G) {
    lg = rows_dot_g(A, i, grp, mult + 2);
    nb = rows_dot_g(A, i, grp, s_nv);      // (one-hot rows: the row's own label only)
  }
  const double T = -(gbi - mult[0] + lg);
  const double al = D.n0 + nb;
  const int j = c >> 1;
  // leaving the interval at its lower end: the row wants to go down
  const int keyL = (j > 0) ? i * 16 + 2 * (j - 1) + 1 : INT_MAX;
  const int keyU = (j + 1 < g.np) ? i * 16 + 2 * j + 1 : INT_MAX;
  double lo0, hi0, lo1, hi1, sn;
  subdiff(g, wi, 0.0, lb, ub, lo0, hi0, sn);
  subdiff(g, wi, 1.0, lb, ub, lo1, hi1, sn);
  // a coefficient that cancels to rounding level (a fixed row whose
  // interval moves with the free rows along v: the degenerate case of free
  // rows that all trade one way) puts no bound on the step; taken at face
  // value it would allow a step of 1/rounding
  if (isfinite(lo0)) {           // lo0 + s_lo (lamc + s ncap) <= T - al s
    const double slo = lo1 - lo0;
    const double aa = al + slo * D.ncap, bb = T - lo0 - slo * D.lamc;
    const double tz = 1e-12 * (fabs(al) + fabs(slo * D.ncap));
    if (aa > tz) { const double x = bb / aa; if (x < Up) { Up = x; upKey = keyL; } }
    else if (aa < -tz) { const double x = bb / aa; if (x > Lo) { Lo = x; loKey = keyL; } }
  }
  if (isfinite(hi0)) {           // T - al s <= hi0 + s_hi (lamc + s ncap)
    const double shi = hi1 - hi0;
    const double aa = -(al + shi * D.ncap), bb = hi0 + shi * D.lamc - T;
    const double tz = 1e-12 * (fabs(al) + fabs(shi * D.ncap));
    if (aa > tz) { const double x = bb / aa; if (x < Up) { Up = x; upKey = keyU; } }
    else if (aa < -tz) { const double x = bb / aa; if (x > Lo) { Lo = x; loKey = keyU; } }
  }
}

// what a step reads per constraint row, staged in LDS (one thread walks it:
// from global memory each row was a chain of round trips)
struct StepRows {
  double nv[kMaxG];            // the direction's entry (0: inactive)
  double gs[kMaxG];            // the row's value at the polished w
  float lo[kMaxG], hi[kMaxG];  // its bounds
};
__device__ __forceinline__ void step_bounds(const PolishArgs& A, int a, const double* gsum,
                                            StepRows& R) {
  for (int g = threadIdx.x; g < A.G; g += blockDim.x) {
    R.gs[g] = gsum[g];
    R.lo[g] = A.blo[(size_t)a * A.G + g];
    R.hi[g] = A.bhi[(size_t)a * A.G + g];
  }
}

// the step along D given the rows' bounds [Lo, Up] (keys kLo, kUp): updates
// mult; *block takes the row to release when one blocks the target.  One
// wave, a constraint row a lane (G <= 64).
__device__ __forceinline__ void sweep_step(const PolishArgs& A, const int* ps, const SweepDir& D,
                                           const StepRows& R, double Lo, double Up, int kLo,
                                           int kUp, double thr, double turn0, float tauf,
                                           double* mult, int* block) {
  const int lane = threadIdx.x & 63, g = min(lane, max(A.G - 1, 0));
  const double ncap = D.ncap, lamc = D.lamc;
  const bool cap_on = ps[PS_CAP];
  const bool act = lane < A.G && band_active(ps, g), up = band_upper(ps, g);
  // targets along this direction, by priority: (1) an active constraint the
  // solve could not enforce (dependent row) and that is violated: push its
  // multiplier outward until a fixed row blocks, and release that row; (2)
  // an active constraint that is slack: zero its multiplier
  // (complementarity)
  double tgt = 0.0, best = 0.0, worst = 0.0;
  bool has_tgt = false;
  const double vtol = 0.1 * A.eps_prim;
  if (cap_on) {                  // lam_cap + s ncap >= 0
    if (ncap > 1e-12) { const double u = -lamc / ncap; if (u > Lo) { Lo = u; kLo = INT_MAX; } }
    else if (ncap < -1e-12) { const double u = -lamc / ncap; if (u < Up) { Up = u; kUp = INT_MAX; } }
    const double sl = (double)tauf - turn0;
    if (fabs(ncap) > 1e-12) {
      if (sl < -vtol) {
        worst = -sl; tgt = (ncap > 0.0) ? INFINITY : -INFINITY; has_tgt = true;
      } else {
        const double v = fabs(lamc) * fmax(sl, 0.0);
        if (v > thr) { best = v; tgt = -lamc / ncap; has_tgt = true; }
      }
    }
  }
  if (A.G) {
    const double nbv = act ? R.nv[g] : 0.0;
    const double cur = mult[2 + g];
    // upper band: lam >= 0 ; lower band: lam <= 0
    const double sgn_req = up ? 1.0 : -1.0;
    const double aa = sgn_req * nbv, bb = sgn_req * cur;   // bb + s aa >= 0
    const double ul = aa > 1e-12 ? -bb / aa : -INFINITY, uu = aa < -1e-12 ? -bb / aa : INFINITY;
    const double ml = wave_red(ul, MaxOp()), mu = -wave_red(-uu, MaxOp());
    if (ml > Lo) { Lo = ml; kLo = INT_MAX; }
    if (mu < Up) { Up = mu; kUp = INT_MAX; }
    // the worst violation (the first row among equals), else the largest
    // slack product
    const bool in = act && fabs(nbv) > 1e-12;
    const double sl = up ? (double)R.hi[g] - R.gs[g] : R.gs[g] - (double)R.lo[g];
    const double viol = in && sl < -vtol ? -sl : 0.0;
    const double wv = wave_red(viol, MaxOp());
    if (wv > worst) {
      const int l = __ffsll((unsigned long long)__ballot(viol == wv)) - 1;
      tgt = (lane_d(aa, l) > 0.0) ? INFINITY : -INFINITY;
      has_tgt = true;
    } else if (worst == 0.0) {
      const double v0 = in ? fabs(cur) * fmax(sl, 0.0) : 0.0, v = v0 > thr ? v0 : 0.0;
      const double wb = wave_red(v, MaxOp());
      if (wb > best) {
        const int l = __ffsll((unsigned long long)__ballot(v == wb)) - 1;
        tgt = lane_d(-cur / nbv, l);
        has_tgt = true;
      }
    }
  }
  double st;
  int blk = -1;
  if (Lo <= Up) {
    st = fmin(fmax(tgt, Lo), Up);
    if (has_tgt) {
      const int key = (tgt < Lo) ? kLo : (tgt > Up) ? kUp : INT_MAX;
      if (key != INT_MAX) blk = key;
    } else if (isfinite(Lo) && isfinite(Up)) {
      st += 1e-3 * (0.5 * (Lo + Up) - st);
    }
  } else {
    st = 0.5 * (Lo + Up);
  }
  if (!isfinite(st)) st = 0.0;
  // eta += st * v  ->  nu -= st v0, bands += st v_b, lam_cap += st v_cap
  if (act) mult[2 + g] += st * R.nv[g];
  if (lane == 0) {
    if (blk >= 0 && *block < 0) *block = blk;
    mult[0] -= st * D.n0;
    if (cap_on) mult[1] += st * ncap;
  }
}

// the check passes' per-row inputs of U rows (all loads issued together)
template <int U>
struct CheckIn {
  int ii[U], cc[U], grp[U];
  double gb[U], w[U], mu[U];
  RowData rd[U];
};
template <int U>
__device__ __forceinline__ void check_in(const PolishArgs& A, int a, int tid, int base, int stride,
                                         bool want_mu, float lbf, float ubf, CheckIn<U>& I) {
  const int n = A.n;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    I.ii[u] = base + u * stride + tid;
    const int ic = min(I.ii[u], n - 1);
    const size_t off = (size_t)a * n + ic;
    I.cc[u] = A.code[off];
    I.gb[u] = A.gbase[off];
    I.w[u] = A.wout[off];
    I.mu[u] = want_mu ? mu_at(A, off) : 0.0;
    I.grp[u] = A.Gl ? A.group[ic] : 0;
  }
  row_data_n<U>(A, a, I.ii, lbf, ubf, I.rd);
}

// a value that another workgroup of the same launch reads or wrote: past the
// caches that are not shared by the device
__device__ __forceinline__ void put_dev(double* p, double x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_dev(const double* p) {
  return __hip_atomic_load(const_cast<double*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the row blocks' bounds of one direction: the extremes over the blocks and
// the smallest keys of the blocks attaining them (every thread gets them;
// s_sh: 3 doubles a wave, s_key: two ints)
__device__ __forceinline__ void gather_bounds(const PolishArgs& A, int a, double* s_sh, int* s_key,
                                              double& Lo, double& Up, int& kLo, int& kUp) {
  const double* sp = A.spart + (size_t)a * A.n_sb * 4;
  double l = -INFINITY, u = INFINITY;
  for (int bb = threadIdx.x; bb < A.n_sb; bb += blockDim.x) {
    l = fmax(l, get_dev(sp + 4 * bb));
    u = fmin(u, get_dev(sp + 4 * bb + 1));
  }
  double sv[1] = {0.0}, mv[2] = {l, -u};
  bred<1, 2>(sv, mv, s_sh);
  Lo = mv[0];
  Up = -mv[1];
  if (threadIdx.x == 0) { s_key[0] = INT_MAX; s_key[1] = INT_MAX; }
  __syncthreads();
  for (int bb = threadIdx.x; bb < A.n_sb; bb += blockDim.x) {
    if (isfinite(Lo) && get_dev(sp + 4 * bb) == Lo)
      atomicMin(&s_key[0], (int)get_dev(sp + 4 * bb + 2));
    if (isfinite(Up) && get_dev(sp + 4 * bb + 1) == Up)
      atomicMin(&s_key[1], (int)get_dev(sp + 4 * bb + 3));
  }
  __syncthreads();
  kLo = s_key[0];
  kUp = s_key[1];
}

// per-block bounds of the one-direction sweep: [m][n_sb][4] = Lo, Up and
// the smallest keys of the rows attaining them
__global__ __launch_bounds__(kRT) void polish_sweep_kernel(PolishArgs A, int final_pass) {
  __shared__ double mult[2 + kMaxG], s_nv[kMaxG];
  __shared__ double s_sh[3 * kRW];
  __shared__ int s_key[2];
  const int G = A.G, tid = threadIdx.x;
  const int b = blockIdx.x, slot = blockIdx.y;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  const int* ps = A.pstate + (size_t)a * kPStateStride;
  if (ps[PS_DONE] || (ps[PS_STALL] && !final_pass) || ps[PS_ND] != 1) return;
  const float* par = A.par + (size_t)a * kNPar;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  const double* gmult = A.mult + (size_t)a * (2 + G);
  for (int q = tid; q < 2 + G; q += kRT) mult[q] = gmult[q];
  const double* nul = wk_of(A, a).nul;
  dir_rows(ps, G, nul, s_nv);
  if (tid == 0) { s_key[0] = INT_MAX; s_key[1] = INT_MAX; }
  CheckIn<kRR> I;
  check_in(A, a, tid, b * kRB, kRT, false, lbf, ubf, I);
  __syncthreads();
  const SweepDir D = sweep_dir(ps, nul, mult);
  double Lo = -INFINITY, Up = INFINITY;
  int loKey = INT_MAX, upKey = INT_MAX;
#pragma unroll
  for (int u = 0; u < kRR; ++u)
    if (I.ii[u] < A.n)
      sweep_row(A, D, s_nv, mult, I.ii[u], I.cc[u], I.gb[u], I.w[u], I.grp[u], I.rd[u], kap, phi,
                Lo, Up, loKey, upKey);
  double sv[1] = {0.0}, mv[2] = {Lo, -Up};
  bred<1, 2>(sv, mv, s_sh);
  const double Lb = mv[0], Ub = -mv[1];
  if (Lo == Lb && isfinite(Lb)) atomicMin(&s_key[0], loKey);
  if (Up == Ub && isfinite(Ub)) atomicMin(&s_key[1], upKey);
  __syncthreads();
  if (tid == 0) {
    double* sp = A.spart + ((size_t)a * A.n_sb + b) * 4;
    sp[0] = Lb;
    sp[1] = Ub;
    sp[2] = s_key[0];
    sp[3] = s_key[1];
  }
}

// One null direction swept by the whole workgroup (every row's bounds, then
// the step): one sweep over the directions a round (a second one, for
// directions that interact, cost a full pass per direction and certified no
// more accounts: the next refinement round revisits them anyway).  Ends
// synchronised.
__device__ __forceinline__ void sweep_one(const PolishArgs& A, int a, int tid, const int* ps,
                                          const double* nul, float lbf, float ubf, float kap,
                                          bool phi, double thr, double turn0, float tauf,
                                          double* mult, StepRows& R, double* sh, int* key,
                                          int* block) {
  const int n = A.n, nt = (int)blockDim.x;
  const SweepDir D = sweep_dir(ps, nul, mult);
  dir_rows(ps, A.G, nul, R.nv);
  if (threadIdx.x == 0) { key[0] = INT_MAX; key[1] = INT_MAX; }
  __syncthreads();
  double Lo = -INFINITY, Up = INFINITY;
  int loKey = INT_MAX, upKey = INT_MAX;
  for (int base = 0; base < n; base += kPU * nt) {
    CheckIn<kPU> I;
    check_in(A, a, tid, base, nt, false, lbf, ubf, I);
#pragma unroll
    for (int u = 0; u < kPU; ++u)
      if (I.ii[u] < n)
        sweep_row(A, D, R.nv, mult, I.ii[u], I.cc[u], I.gb[u], I.w[u], I.grp[u], I.rd[u], kap, phi,
                  Lo, Up, loKey, upKey);
  }
  double sv[1] = {0.0}, mv[2] = {Lo, -Up};
  bred<1, 2>(sv, mv, sh);
  const double Lb = mv[0], Ub = -mv[1];
  if (Lo == Lb && isfinite(Lb)) atomicMin(&key[0], loKey);
  if (Up == Ub && isfinite(Ub)) atomicMin(&key[1], upKey);
  __syncthreads();
  if (threadIdx.x < 64)
    sweep_step(A, ps, D, R, Lb, Ub, key[0], key[1], thr, turn0, tauf, mult, block);
  __syncthreads();
}

// per account: the gradient scale (from polish_gbase's blocks), then the
// multipliers the free rows leave open (one direction: from the sweep
// blocks; more: swept here one after another, from kSplitDir row blocks on by
// polish_dir instead); stores the multipliers, the row to release and the scale
// for the passes after it
__global__ __launch_bounds__(kPTC) void polish_pre_kernel(PolishArgs A, int final_pass) {
  __shared__ double s_red6[6 * kPW];
  __shared__ StepRows R;
  __shared__ double mult[2 + kMaxG];
  __shared__ int s_block, s_key[2], s_bad;
  double* const s_nv = R.nv;
  const int G = A.G, n = A.n;
  const int slot = blockIdx.x;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  const int tid = threadIdx.x;
  int* ps = A.pstate + (size_t)a * kPStateStride;
  if (ps[PS_DONE] || (ps[PS_STALL] && !final_pass)) return;
  const float* par = A.par + (size_t)a * kNPar;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  double* gmult = A.mult + (size_t)a * (2 + G);
  for (int q = tid; q < 2 + G; q += kPTC) mult[q] = gmult[q];
  if (tid == 0) { s_bad = 0; s_block = -1; }
  __syncthreads();                        // flags above are initialised
  const Wk wkc = wk_of(A, a);
  step_bounds(A, a, wkc.gsum, R);
  double gmax = 0.0, mumax = 0.0;
  int bad = 0;
  for (int rb = tid; rb < A.n_rb; rb += kPTC) {
    const double* gp = A.gpart + ((size_t)a * A.n_rb + rb) * 4;
    gmax = fmax(gmax, gp[0]);
    mumax = fmax(mumax, gp[1]);
    if (gp[3] != 0.0) bad = 1;
  }
  if (bad) atomicOr(&s_bad, 1);
  {
    double sv[1] = {0.0}, mv[2] = {gmax, mumax};
    bred<1, 2>(sv, mv, s_red6);           // (also publishes R)
    gmax = mv[0]; mumax = mv[1];
  }
  const double turn0 = wkc.misc[3];       // turnover of w (polish_solve)
  const double scale = fmax(fmax(gmax, mumax), 1e-12);
  const int nd = ps[PS_ND];
  const int ncol = G + 3;
  const double thr = 0.01 * A.eps_comp * scale;
  if (nd == 1) {
    double Lo, Up;
    int kLo, kUp;
    dir_rows(ps, G, wkc.nul, s_nv);
    gather_bounds(A, a, s_red6, s_key, Lo, Up, kLo, kUp);
    if (tid < 64) {
      const SweepDir D = sweep_dir(ps, wkc.nul, mult);
      sweep_step(A, ps, D, R, Lo, Up, kLo, kUp, thr, turn0, tauf, mult, &s_block);
    }
    __syncthreads();
  } else if (nd > 1 && A.n_sb < kSplitDir) {
    for (int q = 0; q < nd; ++q)
      sweep_one(A, a, tid, ps, wkc.nul + q * ncol, lbf, ubf, kap, phi, thr, turn0, tauf, mult, R,
                s_red6, s_key, &s_block);
  }
  for (int q = tid; q < 2 + G; q += kPTC) gmult[q] = mult[q];
  if (tid == 0) {
    ps[PS_BLOCK] = s_block;
    double* misc = wkc.misc;
    misc[0] = scale;
    misc[1] = turn0;
    misc[2] = s_bad ? 1.0 : 0.0;
  }
}

// One of several null directions, for accounts of many row blocks: the
// blocks' bounds as in polish_sweep, and the block that finishes last takes
// the step (the directions interact: the next one, the next launch, starts
// from the stepped multipliers).  One workgroup sweeping all rows was 7.2 ms
// a round at n = 384,800 (8 rows a thread and direction at n = 16,384 break
// even with the eight launches); spread over 752 blocks it is bound by the
// launches.
__global__ __launch_bounds__(kRT) void polish_dir_kernel(PolishArgs A, int final_pass, int q) {
  __shared__ double mult[2 + kMaxG];
  __shared__ StepRows R;
  __shared__ double s_sh[3 * kRW];
  __shared__ int s_key[2], s_last, s_block;
  double* const s_nv = R.nv;
  const int G = A.G, tid = threadIdx.x;
  const int b = blockIdx.x, slot = blockIdx.y;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  int* ps = A.pstate + (size_t)a * kPStateStride;
  const int nd = ps[PS_ND];
  if (ps[PS_DONE] || (ps[PS_STALL] && !final_pass) || nd <= 1 || q >= nd) return;
  const float* par = A.par + (size_t)a * kNPar;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  double* gmult = A.mult + (size_t)a * (2 + G);
  const Wk wk = wk_of(A, a);
  for (int e = tid; e < 2 + G; e += kRT) mult[e] = gmult[e];
  dir_rows(ps, G, wk.nul + q * (G + 3), s_nv);
  if (tid == 0) { s_key[0] = INT_MAX; s_key[1] = INT_MAX; }
  CheckIn<kRR> I;
  check_in(A, a, tid, b * kRB, kRT, false, lbf, ubf, I);
  __syncthreads();
  const SweepDir D = sweep_dir(ps, wk.nul + q * (G + 3), mult);
  double Lo = -INFINITY, Up = INFINITY;
  int loKey = INT_MAX, upKey = INT_MAX;
#pragma unroll
  for (int u = 0; u < kRR; ++u)
    if (I.ii[u] < A.n)
      sweep_row(A, D, s_nv, mult, I.ii[u], I.cc[u], I.gb[u], I.w[u], I.grp[u], I.rd[u], kap, phi,
                Lo, Up, loKey, upKey);
  double sv[1] = {0.0}, mv[2] = {Lo, -Up};
  bred<1, 2>(sv, mv, s_sh);
  const double Lb = mv[0], Ub = -mv[1];
  if (Lo == Lb && isfinite(Lb)) atomicMin(&s_key[0], loKey);
  if (Up == Ub && isfinite(Ub)) atomicMin(&s_key[1], upKey);
  __syncthreads();
  if (tid == 0) {
    // device-wide stores, complete before the count: a fence here would write
    // the whole L2 back, once per block (188 us a launch of 6,016 blocks; 60 now)
    double* sp = A.spart + ((size_t)a * A.n_sb + b) * 4;
    put_dev(sp, Lb);
    put_dev(sp + 1, Ub);
    put_dev(sp + 2, (double)s_key[0]);
    put_dev(sp + 3, (double)s_key[1]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    s_last = atomicAdd(&ps[PS_TICK], 1) == A.n_sb - 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  if (!s_last) return;
  step_bounds(A, a, wk.gsum, R);
  double Lg, Ug;
  int kLo, kUp;
  gather_bounds(A, a, s_sh, s_key, Lg, Ug, kLo, kUp);
  if (tid < 64) {
    const double thr = 0.01 * A.eps_comp * wk.misc[0];
    if (tid == 0) s_block = ps[PS_BLOCK];
    sweep_step(A, ps, D, R, Lg, Ug, kLo, kUp, thr, wk.misc[1], tauf, mult, &s_block);
    if (tid == 0) {
      ps[PS_BLOCK] = s_block;
      ps[PS_TICK] = 0;
    }
  }
  __syncthreads();
  for (int e = tid; e < 2 + G; e += kRT) gmult[e] = mult[e];
}

// one row's diagnostics and its refinement proposal
struct CheckSums {
  double sw = 0.0, turn = 0.0, dmax = 0.0, box = 0.0, snapm = 0.0, obj = 0.0, bad = 0.0;
  int changed = 0;
};
__device__ __forceinline__ int check_row(const PolishArgs& A, int i, int c, double gbi, double wi,
                                         double mui, int grp, const RowData& r, const double* mult,
                                         float kap, bool phi, double gam, CheckSums& S) {
  const double nu = mult[0], lam = mult[1];
  Geom g;
  make_geom(g, kap, phi, r);
  const double lb = r.lb, ub = r.ub;
  const double sig = (gbi + mui) / gam;
  double gi = gbi - nu;
  if (A.G) gi += rows_dot_g(A, i, grp, mult + 2);
  double lo, hi, snap;
  subdiff(g, wi, lam, lb, ub, lo, hi, snap);
  const double t = -gi;
  const double dist = fmax(fmax(lo - t, t - hi), 0.0);
  S.sw += wi;
  S.turn += fabs(wi - g.w0);
  S.dmax = fmax(S.dmax, dist);
  if (!isfinite(dist)) S.bad = 1.0;
  S.box = fmax(S.box, fmax(lb - wi, wi - ub));
  S.snapm = fmax(S.snapm, snap);
  // objective: (gamma/2) w.Sigma w - mu w + trade cost
  double tc = (double)kap * fabs(wi - g.w0);
  if (r.taxed && wi < g.w0) tc += lot_tax(g.w0 - wi, r);
  S.obj += 0.5 * gam * wi * sig - mui * wi + tc;
  // refinement proposal (applied only if the pattern fails)
  int cn = c;
  if (g.np > 1) {
    const double tolm = A.eps_dual * 0.1;
    if (c & 1) {
      const int q = c >> 1;
      if (wi > g.pt(q + 1)) cn = 2 * (q + 1);
      else if (wi < g.pt(q)) cn = 2 * q;
    } else {
      // move off a point when -g lies outside its subdifferential (a fixed
      // row's weight is its point: the interval above)
      const int j = c >> 1;
      const double sc = fmax(fabs(mui), 1e-12);
      if (t > hi + tolm * sc && j + 1 < g.np) cn = 2 * j + 1;
      else if (t < lo - tolm * sc && j > 0) cn = 2 * (j - 1) + 1;
    }
  }
  S.changed += (cn != c) ? 1 : 0;
  return cn;
}

// per-block diagnostics of the pattern's w and the refinement proposals
// (written to code_next for every row): [m][n_sb][8] = budget, turnover and
// objective sums, largest stationarity distance, box violation and kink
// snap, proposal count, non-finite flag
__global__ __launch_bounds__(kRT) void polish_check_rows_kernel(PolishArgs A, int final_pass) {
  __shared__ double mult[2 + kMaxG];
  __shared__ double s_sh[7 * kRW];
  __shared__ int s_ch;
  const int G = A.G, n = A.n, tid = threadIdx.x;
  const int b = blockIdx.x, slot = blockIdx.y;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  const int* ps = A.pstate + (size_t)a * kPStateStride;
  if (ps[PS_DONE] || (ps[PS_STALL] && !final_pass)) return;
  const float* par = A.par + (size_t)a * kNPar;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const double gam = par[P_GAMMA];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  int8_t* code = A.code_next + (size_t)a * n;    // proposals
  const double* gmult = A.mult + (size_t)a * (2 + G);
  for (int q = tid; q < 2 + G; q += kRT) mult[q] = gmult[q];
  if (tid == 0) s_ch = 0;
  CheckIn<kRR> I;
  check_in(A, a, tid, b * kRB, kRT, true, lbf, ubf, I);
  __syncthreads();
  CheckSums S;
#pragma unroll
  for (int u = 0; u < kRR; ++u) {
    const int i = I.ii[u];
    if (i >= n) continue;
    code[i] = (int8_t)check_row(A, i, I.cc[u], I.gb[u], I.w[u], I.mu[u], I.grp[u], I.rd[u], mult,
                                kap, phi, gam, S);
  }
  if (S.changed) atomicAdd(&s_ch, S.changed);
  double sv[3] = {S.sw, S.turn, S.obj}, mv[4] = {S.dmax, S.box, S.snapm, S.bad};
  bred<3, 4>(sv, mv, s_sh);                 // (its barriers also publish s_ch)
  if (tid == 0) {
    double* cp = A.cpart + ((size_t)a * A.n_sb + b) * 8;
    cp[0] = sv[0]; cp[1] = sv[1]; cp[2] = sv[2];
    cp[3] = mv[0]; cp[4] = mv[1]; cp[5] = mv[2];
    cp[6] = s_ch;
    cp[7] = mv[3];
  }
}

// the diagnostics of a pattern over its rows
struct Diag {
  double sw, turn, obj, dmax, box, snapm, chg;   // chg: refinement proposals
  bool bad;                                      // something was not finite
};
// The certificate, and on failure the refinement of bands / cap and the row a
// null-direction step releases (the next round's pattern adopts the
// proposals): one wave, a constraint row a lane.  blk: the row to release or
// -1.  Returns whether the account is certified.
__device__ __forceinline__ bool decide_account(const PolishArgs& A, const fqp_result& R, int a,
                                               int* ps, float tauf, const double* mult,
                                               const double* gsum, const Diag& X, double scale,
                                               int blk, int final_pass) {
  const int G = A.G, lane = threadIdx.x & 63, g = min(lane, max(G - 1, 0));
  const bool on = lane < G;
  const double lo = on ? (double)A.blo[(size_t)a * G + g] : -INFINITY;
  const double hi = on ? (double)A.bhi[(size_t)a * G + g] : INFINITY;
  const double gs = on ? gsum[g] : 0.0, lg = on ? mult[2 + g] : 0.0;
  const double nu = mult[0], lam = mult[1];
  // comp: the largest |multiplier| x slack; gap: their sum, the duality
  // gap the multipliers leave (with stationarity and feasibility exact,
  // f(w) - f* <= gap)
  const double rexp = wave_red(on ? fmax(fmax(lo - gs, gs - hi), 0.0) : 0.0, MaxOp());
  // (a one-sided row's other slack is infinite)
  const double pr = lg != 0.0 ? fabs(lg) * fabs(lg > 0.0 ? hi - gs : gs - lo) : 0.0;
  double comp = fmax(wave_red(pr, MaxOp()), 0.0), gap = wave_red(pr, SumOp());
  const double tau = tauf;
  double rturn = 0.0;
  if (isfinite(tauf)) {
    rturn = fmax(X.turn - tau, 0.0);
    comp = fmax(comp, fmax(lam, 0.0) * fabs(tau - X.turn));
    gap += fmax(lam, 0.0) * fabs(tau - X.turn);
  } else {
    comp = fmax(comp, fabs(lam));
  }
  const double obj_full = X.obj + (A.obj_const ? A.obj_const[a] : 0.0);
  const double r_prim = fmax(fmax(fabs(X.sw - 1.0), fmax(X.box, 0.0)), fmax(rexp, rturn)) + X.snapm;
  const double r_dual = fmax(X.dmax, fmax(-lam, 0.0)) / scale;
  const double r_comp = comp / scale;
  const bool finite = !X.bad && isfinite(X.sw) && isfinite(X.obj) && isfinite(nu) &&
                      isfinite(lam) && isfinite(r_prim) && isfinite(r_dual) &&
                      isfinite(r_comp);
  // the certificate also bounds the relative objective error: the gap
  // against |f| (when |f| is below the gradient scale, as a benchmark term
  // can make it, r_comp <= eps alone does not)
  const bool ok = finite && r_prim <= A.eps_prim && r_dual <= A.eps_dual &&
                  r_comp <= A.eps_comp && gap <= A.eps_comp * fmax(fabs(obj_full), 1e-12);
  // bands to drop or to take up
  const bool act = on && band_active(ps, g), up = on && band_upper(ps, g);
  const unsigned long long drop = __ballot(act && ((up && lg < 0.0) || (!up && lg > 0.0)));
  const bool above = on && !act && gs > hi + 0.1 * A.eps_prim;
  const unsigned long long add_hi = __ballot(above);
  const unsigned long long add_lo = __ballot(on && !act && !above && gs < lo - 0.1 * A.eps_prim);
  if (lane == 0) {
    ps[PS_ROUNDS] += 1;
    // keep the diagnostics of the latest pattern in the result arrays
    if (ok || final_pass) {
      if (R.r_prim) R.r_prim[a] = r_prim;
      if (R.r_dual) R.r_dual[a] = r_dual;
      if (R.r_comp) R.r_comp[a] = r_comp;
      // (the benchmark's constant (gamma/2) w_b^T Sigma w_b completes Eq. 1)
      if (R.obj) R.obj[a] = obj_full;
      if (R.nu) R.nu[a] = nu;
      if (R.lam_cap) R.lam_cap[a] = lam;
    }
    if (ok) {
      ps[PS_DONE] = 1;
      R.status[a] = FQP_SOLVED;
    } else if (final_pass) {
      // the paper's quality gates (Sec. "Quality Gates and Failure
      // Vocabulary"): budget <= 1e-4 and bound violation <= 1e-6
      const bool gates =
          fabs(X.sw - 1.0) <= 1e-4 && X.box <= 1e-6 && rexp <= 1e-6 && rturn <= 1e-6;
      R.status[a] = gates ? FQP_FEASIBLE_UNCERTIFIED : FQP_MAX_ITER;
    } else {
      // bands / cap refinement
      int nchg = (int)X.chg;
      if (blk >= 0) {                    // release the row that blocks
        A.code_next[(size_t)a * A.n + (blk >> 4)] = (int8_t)(blk & 15);
        ++nchg;
      }
      nchg += __popcll(drop) + __popcll(add_hi) + __popcll(add_lo);
      const unsigned long long added = add_hi | add_lo;
      ps[PS_BACT0] = (ps[PS_BACT0] & ~(int)(unsigned)drop) | (int)(unsigned)added;
      ps[PS_BACT1] = (ps[PS_BACT1] & ~(int)(drop >> 32)) | (int)(added >> 32);
      ps[PS_BUP0] = (ps[PS_BUP0] & ~(int)(unsigned)(drop | add_lo)) | (int)(unsigned)add_hi;
      ps[PS_BUP1] = (ps[PS_BUP1] & ~(int)((drop | add_lo) >> 32)) | (int)(add_hi >> 32);
      if (isfinite(tauf)) {
        if (ps[PS_CAP] && lam < 0.0) { ps[PS_CAP] = 0; ++nchg; }
        else if (!ps[PS_CAP] && X.turn > tau + 0.1 * A.eps_prim) { ps[PS_CAP] = 1; ++nchg; }
      }
      // no proposal: further rounds on this iterate cannot help; many
      // proposals: the iterate is still far from its final pattern, and the
      // next block of iterations is a cheaper way to get closer
      if (nchg == 0 || nchg > A.max_prop) ps[PS_STALL] = 1;
    }
  }
  if ((final_pass || ok) && R.lam_band && on) R.lam_band[(size_t)a * G + g] = lg;
  return ok;
}

// per account: the diagnostics gathered in block order, the certificate and
// the refinement
__global__ __launch_bounds__(64) void polish_decide_kernel(PolishArgs A, fqp_result R,
                                                           int final_pass) {
  const int G = A.G, tid = threadIdx.x;
  const int slot = blockIdx.x;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  int* ps = A.pstate + (size_t)a * kPStateStride;
  if (ps[PS_DONE] || (ps[PS_STALL] && !final_pass)) return;
  // lane l takes blocks l, l + 64, ... in order, then the wave's reduction
  double sw = 0.0, turn = 0.0, obj = 0.0, dmax = 0.0, box = 0.0, snapm = 0.0, chg = 0.0,
         bad = 0.0;
  for (int bb = tid; bb < A.n_sb; bb += 64) {
    const double* cp = A.cpart + ((size_t)a * A.n_sb + bb) * 8;
    sw += cp[0]; turn += cp[1]; obj += cp[2];
    dmax = fmax(dmax, cp[3]); box = fmax(box, cp[4]); snapm = fmax(snapm, cp[5]);
    chg += cp[6]; bad = fmax(bad, cp[7]);
  }
  const Wk wkc = wk_of(A, a);
  Diag X;
  X.sw = wave_red(sw, SumOp());
  X.turn = wave_red(turn, SumOp());
  X.obj = wave_red(obj, SumOp());
  X.dmax = wave_red(dmax, MaxOp());
  X.box = wave_red(box, MaxOp());
  X.snapm = wave_red(snapm, MaxOp());
  X.chg = wave_red(chg, SumOp());
  X.bad = wkc.misc[2] != 0.0 || wave_red(bad, MaxOp()) != 0.0;
  decide_account(A, R, a, ps, A.par[(size_t)a * kNPar + P_TAU], A.mult + (size_t)a * (2 + G),
                 wkc.gsum, X, wkc.misc[0], ps[PS_BLOCK], final_pass);
}

// ---------------------------------------------------------------------------
// A whole certification pass of one account in one workgroup: the rounds of
// the passes above, back to back, with the account's bookkeeping in LDS.
// A round of separate launches is bound by what lies between the phases: on a
// book of 64 x 2,000 with every rule its eight kernels take 101 us, of which the
// solve is 33, the gaps between them come on top, every round waits for the
// slowest account, and the host reads a count back between rounds.  Here a
// round is 55 us: 27 the solve (serial steps of one wave), the rest the
// instructions of 16 waves over 2,000 rows.
// Same arithmetic in the same order as the row-block passes (their sums over
// rows differ in rounding only).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kPT) void polish_pass_kernel(PolishArgs A, fqp_result R, int rounds) {
  extern __shared__ double smem_d[];
  __shared__ AcctLds W;
  __shared__ StepRows SR;
  __shared__ double s_red[3 * kPW], s_vec[kSolveVecs];
  // (the gradient scale has partials of its own: wave 0 may still read them
  // when the first wave is through its rows and stores its diagnostics)
  __shared__ double4 s_sum4[kPT / 16], s_max4[kPT / 16], s_grad4[kPT / 16];
  double *const s_sum = &s_sum4[0].x, *const s_max = &s_max4[0].x, *const s_grad = &s_grad4[0].x;
  __shared__ int s_ps[kPStateStride], s_same, s_block, s_key[2], s_flag;
  const int n = A.n, k = A.k, G = A.G;
  const int slot = blockIdx.x;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  int* ps = A.pstate + (size_t)a * kPStateStride;
  const float* par = A.par + (size_t)a * kNPar;
  const float lbf = par[P_LB], ubf = par[P_UB], kap = par[P_KAPPA], tauf = par[P_TAU];
  const double gam = par[P_GAMMA];
  const bool phi = (kap > 0.f) || isfinite(tauf) || (par[P_HASTAX] != 0.f);
  const Wk wk = wk_of(A, a);
  const size_t off = (size_t)a * n;
  const int k4 = (k + 3) >> 2;
  if (threadIdx.x < kPStateStride) s_ps[threadIdx.x] = ps[threadIdx.x];
  __syncthreads();
  for (int r = 0;; ++r) {
    const int first = r == 0;
    // what depends on the thread is formed anew each round (kept across the
    // rounds it would not fit the registers)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    if (first) begin_pass(A, a, par, s_ps, W.mult);
    // ---- the pattern, kPT / kRT row blocks at a time
    RowsLds* L = reinterpret_cast<RowsLds*>(smem_d) + tid / kRT;
    for (int b0 = 0; b0 < A.n_sb; b0 += kPT / kRT) {
      const int b = b0 + tid / kRT;
      rows_block(A, a, b < A.n_sb ? b : -1, tid % kRT, first, *L);
      __syncthreads();
    }
    const PatternSums X = gather_pattern(A, a, tid, first, smem_d, W);
    if (gated(A, first, s_ps, X, &s_same)) break;             // uniform
    const double turn0 = solve_pattern(A, a, tid, par, s_ps, X, smem_d, s_vec, W);
    if (tid < 4 * k4 - k) W.yF[k + tid] = 0.0;
    __syncthreads();
    // ---- gradient base: a row a thread, B~ by columns of four (coalesced)
    double gmax = 0.0, mumax = 0.0, bad = 0.0;
    for (int i = tid; i < n; i += kPT) {
      const double wi = A.wout[off + i], mui = mu_at(A, off + i), di = (double)A.d[i];
      double sig = 0.0;
#pragma unroll 4
      for (int j = 0; j < k4; ++j) {
        const float4 b = A.Bq[(size_t)j * n + i];
        const double* y = W.yF + 4 * j;
        sig += (double)b.x * y[0] + (double)b.y * y[1] + (double)b.z * y[2] + (double)b.w * y[3];
      }
      const double sg = sig + di * wi;
      const double v = gam * sg - mui;
      A.gbase[off + i] = v;
      gmax = fmax(gmax, fabs(gam * sg));
      mumax = fmax(mumax, fabs(mui));
      if (!isfinite(v) || !isfinite(wi)) bad = 1.0;
    }
    // ---- the gradient scale, the multipliers the free rows leave open
    step_bounds(A, a, W.gsum, SR);
    if (tid == 0) s_block = -1;
    double gv[4] = {gmax, mumax, bad, 0.0};   // (of use to the first wave only)
    put_red4(gv, s_grad, MaxOp());
    __syncthreads();                          // (also publishes SR)
    if (tid < 64) get_red4(gv, s_grad, MaxOp());
    const double scale = fmax(fmax(gv[0], gv[1]), 1e-12);
    const int nd = s_ps[PS_ND];
    const double thr = 0.01 * A.eps_comp * scale;
    for (int q = 0; q < nd; ++q)
      sweep_one(A, a, tid, s_ps, wk.nul + q * (G + 3), lbf, ubf, kap, phi, thr, turn0, tauf, W.mult, SR,
                s_red, s_key, &s_block);
    // ---- diagnostics and proposals
    CheckSums S;
    for (int base = 0; base < n; base += kPU * kPT) {
      CheckIn<kPU> I;
      check_in(A, a, tid, base, kPT, true, lbf, ubf, I);
#pragma unroll
      for (int u = 0; u < kPU; ++u) {
        if (I.ii[u] >= n) continue;
        A.code_next[off + I.ii[u]] = (int8_t)check_row(A, I.ii[u], I.cc[u], I.gb[u], I.w[u], I.mu[u],
                                                       I.grp[u], I.rd[u], W.mult, kap, phi, gam, S);
      }
    }
    double sv[4] = {S.sw, S.turn, S.obj, (double)S.changed}, mv[4] = {S.dmax, S.box, S.snapm, S.bad};
    put_red4(sv, s_sum, SumOp());
    put_red4(mv, s_max, MaxOp());
    __syncthreads();
    if (tid < 64) {
      get_red4(sv, s_sum, SumOp());
      get_red4(mv, s_max, MaxOp());
      Diag D;
      D.sw = sv[0]; D.turn = sv[1]; D.obj = sv[2]; D.chg = sv[3];
      D.dmax = mv[0]; D.box = mv[1]; D.snapm = mv[2];
      D.bad = gv[2] != 0.0 || mv[3] != 0.0;
      decide_account(A, R, a, s_ps, tauf, W.mult, W.gsum, D, scale, s_block, 0);
      if (tid == 0) s_flag = s_ps[PS_DONE] || s_ps[PS_STALL];
    }
    __syncthreads();
    if (s_flag || r + 1 == rounds) break;                     // uniform
  }
  // for the adjoint and the next pass (a gated account leaves the rounds right
  // behind the stores of its flags)
  __syncthreads();
  if (threadIdx.x < kPStateStride) ps[threadIdx.x] = s_ps[threadIdx.x];
}

static size_t polish_smem(int k, int G, int n_sb) {
  const size_t solve = sizeof(double) * ((size_t)solve_doubles(k, G) + kSolveVecs);
  // the gather: a double a thread (long accounts: none), the list offsets
  const size_t gather = (n_sb > kGatherParts ? 0 : sizeof(double) * kPT) +
                        sizeof(int) * 2 * ((size_t)n_sb + 1);
  return solve > gather ? solve : gather;
}

// dynamic LDS: of the solve at k = 128 and the most constraint rows; of a pass,
// whose own variables take 14 KB
constexpr size_t kSolveLds = 156 * 1024, kPassLds = 144 * 1024;

static size_t pass_smem(int k, int G, int n_sb) {
  const size_t rows = sizeof(RowsLds) * (kPT / kRT);
  const size_t solve = polish_smem(k, G, n_sb);
  return solve > rows ? solve : rows;
}

// One workgroup walks an account's rows where the launches between phases
// cost more than the rows: polish times of two books each, row-block passes
// against this one: 64 x 2,000 9.4 ms : 5.8, 1,000 x 2,000 21.9 : 15.1,
// 3,000 x 500 32.8 : 22.2, 64 x 5,000 17.8 : 17.0, 128 x 5,000 8.8 : 8.6; beyond,
// 300 x 6,000 4.5 : 4.9, 16 x 8,000 8.8 : 10.3, 500 x 10,000 8.3 : 13.9.  The
// number of accounts does not move the line.
constexpr int kPassRows = 10 * kRB;
bool polish_pass_fits(int n, int k, int G) {
  if (pass_smem(k, G, polish_pass_blocks(n)) > kPassLds) return false;
  return n <= kPassRows;
}

hipError_t launch_polish_pass(const PolishArgs& A, const fqp_result& R, int rounds,
                              hipStream_t st) {
  const size_t smem = pass_smem(A.k, A.G, A.n_sb);
  hipError_t e = hipFuncSetAttribute((const void*)polish_pass_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kPassLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(polish_pass_kernel, dim3(A.m_total), dim3(kPT), smem, st, A, R, rounds);
  return hipGetLastError();
}

hipError_t launch_polish_solve(const PolishArgs& A, hipStream_t st) {
  hipLaunchKernelGGL(polish_rows_kernel, dim3(A.n_sb, A.m_total), dim3(kRT), 0, st, A);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t smem = polish_smem(A.k, A.G, A.n_sb);
  // (the attribute belongs to the process: at least what any book of the
  // library's limits takes, so that calls of several threads agree)
  e = hipFuncSetAttribute((const void*)polish_solve_kernel,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)(smem > kSolveLds ? smem : kSolveLds));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(polish_solve_kernel, dim3(A.m_total), dim3(kPT), smem, st, A);
  return hipGetLastError();
}

hipError_t launch_polish_check_r(const PolishArgs& A, const fqp_result& R, int final_pass,
                                 hipStream_t st) {
  hipLaunchKernelGGL(polish_gbase_kernel, dim3(A.n_rb, (A.m_total + kGbAcc - 1) / kGbAcc),
                     dim3(256), 0, st, A, final_pass);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(polish_sweep_kernel, dim3(A.n_sb, A.m_total), dim3(kRT), 0, st, A,
                     final_pass);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(polish_pre_kernel, dim3(A.m_total), dim3(kPTC), 0, st, A, final_pass);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (A.n_sb >= kSplitDir)
    for (int q = 0; q < kMaxNull; ++q) {
      hipLaunchKernelGGL(polish_dir_kernel, dim3(A.n_sb, A.m_total), dim3(kRT), 0, st, A,
                         final_pass, q);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  hipLaunchKernelGGL(polish_check_rows_kernel, dim3(A.n_sb, A.m_total), dim3(kRT), 0, st, A,
                     final_pass);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(polish_decide_kernel, dim3(A.m_total), dim3(64), 0, st, A, R, final_pass);
  return hipGetLastError();
}

int polish_row_blocks(int n) { return (n + kGbRows - 1) / kGbRows; }
int polish_pass_blocks(int n) { return (n + kRB - 1) / kRB; }
int polish_rpart_stride(int k, int G) { return rpart_stride(k, G); }

// The accounts of the active list still refining their pattern (neither
// certified nor stalled in this pass), in list order: the later rounds of a
// pass run on this list, so that their grids (the gradient base above all,
// which works on groups of accounts) cover only those accounts.
__global__ __launch_bounds__(1024) void polish_list_kernel(const int* m_act, const int* act,
                                                           const int32_t* pstate, int* pact,
                                                           int* pm_act, int* host_count) {
  __shared__ int s_wc[16];
  __shared__ int s_base;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int m = *m_act;
  if (tid == 0) s_base = 0;
  __syncthreads();
  for (int b0 = 0; b0 < m; b0 += 1024) {
    const int slot = b0 + tid;
    int keep = 0, a = -1;
    if (slot < m) {
      a = act[slot];
      const int32_t* ps = pstate + (size_t)a * kPStateStride;
      keep = !(ps[PS_DONE] || ps[PS_STALL]);
    }
    const unsigned long long mk = __ballot(keep);
    if (lane == 0) s_wc[wv] = __popcll(mk);
    __syncthreads();
    int off = s_base + __popcll(mk & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
    for (int q = 0; q < wv; ++q) off += s_wc[q];
    if (keep) pact[off] = a;
    __syncthreads();
    if (tid == 0) {
      int t = 0;
      for (int q = 0; q < 16; ++q) t += s_wc[q];
      s_base += t;
    }
    __syncthreads();
  }
  if (tid == 0) {
    *pm_act = s_base;
    if (host_count) *host_count = s_base;
  }
}

hipError_t launch_polish_list(const int* m_act, const int* act, const int32_t* pstate, int* pact,
                              int* pm_act, int* host_count, hipStream_t st) {
  hipLaunchKernelGGL(polish_list_kernel, dim3(1), dim3(1024), 0, st, m_act, act, pstate, pact,
                     pm_act, host_count);
  return hipGetLastError();
}

}  // namespace fqp
