// Dense float64 pieces shared by the polish and the adjoint (gfx950): wave
// reductions, the constraint system of a pattern, the layout of the staged rows.
#pragma once
#include "fqp_common.h"

namespace fqp {

// the per-account kernels: one workgroup of 16 waves per account (their
// serial parts are latency bound)
constexpr int kPT = 1024;
constexpr int kMaxNull = 8;                // null directions kept

// a double from another lane of the row of 16 (a DPP pattern)
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
// reduction over the 16 lanes of a row (all of them get it), and over a wave
// (uniform): quad swaps and row mirrors instead of LDS permutes, 6 round
// trips of which cost more than what is reduced here
template <class F>
__device__ __forceinline__ double row_red(double x, F f) {
  x = f(x, dpp_d<0xB1>(x));                 // lanes 1 0 3 2
  x = f(x, dpp_d<0x4E>(x));                 // lanes 2 3 0 1
  x = f(x, dpp_d<0x141>(x));                // mirrored in eight
  x = f(x, dpp_d<0x140>(x));                // mirrored in sixteen
  return x;
}
template <class F>
__device__ __forceinline__ double wave_red(double x, F f) {
  x = row_red(x, f);
  return f(f(lane_d(x, 0), lane_d(x, 16)), f(lane_d(x, 32), lane_d(x, 48)));
}
// x of lane l to lane `to` (a permutation of the lanes)
__device__ __forceinline__ double push_d(double x, int to) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_ds_permute(4 * to, (int)b);
  const int hi = __builtin_amdgcn_ds_permute(4 * to, (int)(b >> 32));
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
struct SumOp { __device__ double operator()(double a, double b) const { return a + b; } };
struct MaxOp { __device__ double operator()(double a, double b) const { return fmax(a, b); } };

// 1 / f_j on the diagonal of K_F.  A factor of no variance (f_j = 0) drops out of
// the solves by its diagonal's weight; an infinite one would meet its own
// reciprocal 0 in div_by (inf * 0).  The reciprocal of every other float32 is
// below the bound.
__device__ __forceinline__ double factor_weight(float f) { return fmin(1.0 / (double)f, 1e300); }

// S eta = C H^-1 rhs - h, S positive semidefinite (nc x ncol, the rhs column
// last), by one wave (nc <= kSchurW), lane i its row i: a pivoted Cholesky
// finds the rank, the components it does not reach keep their value in e0, and
// the null directions of S go to nul (rows of nul_stride; at most kMaxNull;
// their number is returned).  The pivot by
// a maximum and a ballot, the pivot's column of the remaining matrix from S
// and the factor's columns before it (Lt, a row of kSchurW doubles per step,
// in LDS), one unknown a lane in the triangular solves.  One thread walking
// the system through global memory was 78 us at 10 columns, 265 at 15
// (8 x 384,800), more than the rest of the solve.
constexpr int kSchurW = 44;               // S and Lt fit where H was
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ int schur_solve_wave(int nc, int ncol, const double* S, const double* hv,
                                                const double* e0, double* Lt, double* rr,
                                                double* nul, int nul_stride) {
  const int lane = threadIdx.x & 63, row = min(lane, nc - 1);
  const bool on = lane < nc;
  const double* Sr = S + row * ncol;
  double dg = on ? Sr[row] : -INFINITY;               // the remaining matrix's diagonal
  const double ptol = 1e-12 * fmax(wave_red(dg, MaxOp()), 0.0);
  // pos: the row's place in the pivoted order; ord: lane l holds the row in
  // place l; pos1: the place after the first exchange (an entry is read from
  // the side of S that is its lower triangle then, as S is symmetric only up to
  // rounding and the serial form below mirrors that side)
  int pos = lane, ord = lane, pos1 = lane;
  double ld = 1.0, id = 1.0;                          // L_pp of a pivot row, 1 / L_pp
  int rank = 0;
  for (int j = 0; j < nc; ++j) {
    double mx = on && pos >= j ? dg : -INFINITY;
    if (nc <= 16) mx = lane_d(row_red(mx, MaxOp()), 0);   // uniform: one row holds them all
    else mx = wave_red(mx, MaxOp());
    if (!(mx > ptol)) break;                          // uniform
    // the largest remaining pivot, the first in place among equals
    unsigned long long tie = __ballot(on && pos >= j && dg == mx);
    int p = __ffsll(tie) - 1, pb = __builtin_amdgcn_readlane(pos, p);
    for (tie &= tie - 1; tie; tie &= tie - 1) {
      const int q = __ffsll(tie) - 1, qb = __builtin_amdgcn_readlane(pos, q);
      if (qb < pb) { p = q; pb = qb; }
    }
    const int oj = __builtin_amdgcn_readlane(ord, j);  // the row in place j moves to place pb
    pos = lane == p ? j : (lane == oj ? pb : pos);
    ord = lane == j ? p : (lane == pb ? oj : ord);
    // (with the pivot in place j already both lines change nothing)
    if (j == 0) pos1 = pos;
    double c = pos1 >= __builtin_amdgcn_readlane(pos1, p) ? Sr[p] : S[p * ncol + row];
    for (int l0 = 0; l0 < j; l0 += 4) {                // four columns' loads together
      double x4[4], y4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int l = min(l0 + u, j - 1);
        x4[u] = Lt[l * kSchurW + row];
        y4[u] = Lt[l * kSchurW + p];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (l0 + u < j) c -= x4[u] * y4[u];            // uniform
    }
    double djj, ij;
    root_recip(mx, djj, ij);
    c = lane == p ? djj : div_by(c, djj, ij);
    if (lane == p) { ld = djj; id = ij; }
    if (on) Lt[j * kSchurW + lane] = c;
    if (on && pos > j) dg -= c * c;
    wave_sync();
    ++rank;
  }
  // right-hand side on the pivot rows, null components from eta0
  double x = (on && pos >= rank) ? e0[row] : 0.0;
  double t = on ? Sr[nc] - hv[row] : 0.0;
  for (int q = rank; q < nc; ++q) {
    const int pq = __builtin_amdgcn_readlane(ord, q);
    t -= Sr[pq] * lane_d(x, pq);
  }
  if (pos < rank) x = t;
  // everything in place order from here: lane l the unknown of place l, Lt[l]
  // the factor's column l by place
  for (int l0 = 0; l0 < rank; l0 += 8) {
    double x8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x8[u] = Lt[min(l0 + u, rank - 1) * kSchurW + row];
    wave_sync();
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (on && l0 + u < rank) Lt[(l0 + u) * kSchurW + pos] = x8[u];
  }
  wave_sync();
  x = push_d(x, pos);
  ld = push_d(ld, pos);
  id = push_d(id, pos);
  for (int l0 = 0; l0 < rank; l0 += 8) {              // L11 z = rhs
    double lv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) lv[u] = Lt[min(l0 + u, rank - 1) * kSchurW + row];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int l = l0 + u;
      if (l >= rank) break;                           // uniform
      const double z = div_by(x, ld, id), xl = lane_d(z, l);
      x = lane == l ? z : (lane > l && lane < rank ? x - lv[u] * xl : x);
    }
  }
  // L11^T y = z, each unknown's sum in ascending order of places
  auto back = [&](double y) {
    for (int i0 = (rank - 1) & ~7; i0 >= 0; i0 -= 8) {
      double lv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) lv[u] = Lt[min(i0 + u, rank - 1) * kSchurW + row];
#pragma unroll
      for (int u = 7; u >= 0; --u) {
        const int i = i0 + u;
        if (i >= rank) continue;                      // uniform
        double s = lane_d(y, i);
        for (int l = i + 1; l < rank; ++l) s -= lane_d(lv[u], l) * lane_d(y, l);
        s = div_by(s, lane_d(ld, i), lane_d(id, i));
        y = lane == i ? s : y;
      }
    }
    return y;
  };
  x = back(x);
  if (on) rr[ord] = x;
  // null directions: v_piv = -L11^-T L21^T e_t, v_t = 1
  const int nd = min(nc - rank, kMaxNull);
  for (int q = 0; q < nd; ++q) {
    double v = lane < rank ? -Lt[lane * kSchurW + rank + q] : (lane == rank + q ? 1.0 : 0.0);
    v = back(v);
    if (on) nul[q * nul_stride + ord] = v;
  }
  return nd;
}

// leading dimension of Kf in LDS: odd where the space allows (a column then
// spreads over the banks)
__host__ __device__ __forceinline__ int kf_ld(int k) { return k <= 100 ? (k | 1) : k; }

// rows staged at a time by the factor-space path: [b | V | pad | 1 / d]
__host__ __device__ __forceinline__ int stage_stride(int k, int ncol) {
  return 4 * ((k + ncol + 3) / 4) + 4;
}
__host__ __device__ __forceinline__ int stage_rows(int k, int G) {
  // as many of 64 rows as fit beside Kf in 144 KB, at least 16
  const int left = 144 * 1024 - 8 * k * kf_ld(k);
  const int r = left / (8 * stage_stride(k, G + 3));
  return r >= 64 ? 64 : r >= 32 ? 32 : 16;
}

}  // namespace fqp
