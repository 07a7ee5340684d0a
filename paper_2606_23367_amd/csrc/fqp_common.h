// Device-side layout shared by the fqp kernels (gfx950).
//
// Book state lives in HBM as account-major float32 arrays [m][n] (an
// account's row of assets is contiguous), so a wavefront half reading 32
// consecutive assets of one account issues one 128-byte line.  The factor
// block B~ = [B | A^T | 1 | 0-pad] is float32 [n][kp] with kp a multiple of
// 32: B (k columns), one one-hot column per exposure group (bands enter the
// x-update as extra low-rank directions), one column of ones (its
// contraction gives 1^T Delta^-1 r for the budget border), zero padding.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fqp {

constexpr int kTM = 32;        // accounts per workgroup tile (MFMA M)
constexpr int kWaves = 4;      // waves per workgroup
constexpr int kRowsPerChunk = 32 * kWaves;  // rows per chunk (MFMA N x waves)
constexpr int kMaxKp = 192;    // padded factor width limit
constexpr int kMaxK = 128;     // factor limit (polish keeps K_F in LDS)
constexpr int kMaxG = 64;      // exposure groups limit
constexpr int kMaxKpBf = 96;   // widest factor block of the bf16-split passes
                               // (their B~ and p operands stay in registers)

// per-account float parameters, [m][kNPar]
enum AccPar {
  P_GAMMA = 0, P_RHO, P_KAPPA, P_LAM, P_NU, P_LB, P_UB, P_TAU,
  P_ALPHA, P_RHOB, P_CLASS, P_HASTAX, kNPar = 12
};

// ---------------------------------------------------------------------------
// separable proximal step of phi_i + lam|. - w0| + box  (float32)
//
// For a convex piecewise-linear g with kinks c_1 < ... < c_m and slopes
// s_0 < ... < s_m, argmin_z g(z) + (rho/2)(z - v)^2 is
//   min(v - s_0/rho, max(c_1, min(v - s_1/rho, max(c_2, ... max(c_m,
//       v - s_m/rho)))))
// and adding the box [lb, ub] clips the result (1-D convexity).
// ---------------------------------------------------------------------------
struct TaxLots {
  float b1, b2, b3;        // cumulative sale breakpoints
  float s0, s1, s2, s3;    // lot slopes (non-decreasing)
};

__device__ __forceinline__ float prox_plain(float v, float w0, float th,
                                            float lb, float ub) {
  // kink at w0 with slopes -th*rho, +th*rho (th = (kappa+lam)/rho)
  float z = fminf(v + th, fmaxf(w0, v - th));
  return fminf(fmaxf(z, lb), ub);
}

__device__ __forceinline__ float prox_taxed(float v, float w0, float th,
                                            float irho, const TaxLots& t,
                                            float lb, float ub) {
  // kinks w0-b3 < w0-b2 < w0-b1 < w0; slopes (times 1/rho):
  //   -(th + s3/rho), -(th + s2/rho), -(th + s1/rho), -(th + s0/rho), +th
  float acc = v - th;
  acc = fmaxf(w0, acc);
  acc = fminf(v + th + t.s0 * irho, acc);
  acc = fmaxf(w0 - t.b1, acc);
  acc = fminf(v + th + t.s1 * irho, acc);
  acc = fmaxf(w0 - t.b2, acc);
  acc = fminf(v + th + t.s2 * irho, acc);
  acc = fmaxf(w0 - t.b3, acc);
  acc = fminf(v + th + t.s3 * irho, acc);
  return fminf(fmaxf(acc, lb), ub);
}

// one safeguarded Newton step on turnover(lam) = tau from the summed
// turnover gt and free count nft at lam; updates the bracket [lo, hi_b], the
// best multiplier known to be feasible and returns the next multiplier
__device__ __forceinline__ float cap_step(float gt, float nft, float tau, float rho, float lam,
                                          float& lo, float& hi_b, float& best_feas,
                                          bool& done) {
  const float tol = 1e-6f * fmaxf(tau, 1e-6f);
  if (gt <= tau) { hi_b = lam; best_feas = lam; } else { lo = lam; }
  done = fabsf(gt - tau) <= tol || (lam == 0.f && gt <= tau);
  float nl = lam;
  if (!done) {
    nl = (nft > 0.f) ? lam + rho * (gt - tau) / nft : NAN;
    if (gt <= tau && !(nl > 0.f) && lo == 0.f && lam > 0.f) {
      nl = 0.f;                        // try the unconstrained multiplier
    } else if (!(nl > lo && nl < hi_b)) {
      nl = isfinite(hi_b) ? 0.5f * (lo + hi_b) : fmaxf(2.f * lam, lam + 1e-4f);
    }
    if (isfinite(hi_b) && hi_b - lo <= 1e-6f * hi_b && lo > 0.f) { done = true; nl = hi_b; }
  }
  return fmaxf(nl, 0.f);
}

// the multiplier the search hands on: never one whose turnover is known to
// exceed tau
__device__ __forceinline__ float cap_result(float lam, bool done, float best_feas) {
  return (!done && isfinite(best_feas)) ? best_feas : lam;
}

__device__ __forceinline__ int popc_below(uint32_t word, int bit) {
  return __popc(word & ((1u << bit) - 1u));
}

// a double held by one lane, to all (the lane is uniform)
__device__ __forceinline__ double lane_d(double x, int l) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// a / b from a reciprocal ib of b that is right to the last place: the quotient
// with one correction (Markstein's step), three operations in a chain of them.
// Correctly rounded where ib is; root_recip's ib is a rounded Newton step, which
// is that in all but rare cases, but not proven to be: the bound is one unit in the
// last place, for finite a, b and quotient (b or a * ib infinite gives no number,
// where a division gave 0 or infinity)
__device__ __forceinline__ double div_by(double a, double b, double ib) {
  const double q = a * ib;
  return fma(fma(-b, q, a), ib, q);
}

// sqrt(a) and its reciprocal (a normal, positive, finite) from one estimate,
// each within a unit in the last place: a third of the chain of a root and a
// division
__device__ __forceinline__ void root_recip(double a, double& d, double& id) {
  double y = __builtin_amdgcn_rsq(a);
  y = fma(0.5 * y, fma(-a * y, y, 1.0), y);
  y = fma(0.5 * y, fma(-a * y, y, 1.0), y);
  double s = a * y;
  s = fma(0.5 * y, fma(-s, s, a), s);
  d = s;
  id = fma(y, fma(-s, y, 1.0), y);
}

// Cholesky factor of the k x k matrix L (lower triangle, LDS, k <= 128,
// leading dimension ld) by the whole workgroup, in panels of 8 columns: wave
// 0 factors a panel with its rows in registers (pivots and multipliers pass
// by readlane: no LDS or barrier inside it), then every thread updates a slice
// of the trailing block by the panel's eight columns.  inv[j] takes 1 / L_jj.
// A column at a time with two barriers took 46 us at k = 60, one wave reading
// finished columns from LDS 29 us at k = 46; panels take 19 and 11 us.  Ends with a
// barrier.
__device__ inline void chol_factor(double* L, int k, int ld, double* inv) {
  const int tid = threadIdx.x, nt = (int)blockDim.x;
  for (int p0 = 0; p0 < k; p0 += 8) {
    if (tid < 64) {
      const int i0 = p0 + tid, i1 = p0 + 64 + tid;
      const int nb = min(8, k - p0);
      double r0[8], r1[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        r0[c] = (c < nb && i0 < k && c <= tid) ? L[i0 * ld + p0 + c] : 0.0;
        r1[c] = (c < nb && i1 < k) ? L[i1 * ld + p0 + c] : 0.0;
      }
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (c >= nb) break;                                   // uniform
        double d, id;
        root_recip(fmax(lane_d(r0[c], c), 1e-300), d, id);
        r0[c] = tid == c ? d : div_by(r0[c], d, id);
        r1[c] = div_by(r1[c], d, id);
        if (tid == c) inv[p0 + c] = id;
#pragma unroll
        for (int e = c + 1; e < 8; ++e) {
          const double m = lane_d(r0[c], e);                  // L[p0 + e][p0 + c]
          r0[e] -= r0[c] * m;
          r1[e] -= r1[c] * m;
        }
      }
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if (c < nb && i0 < k && c <= tid) L[i0 * ld + p0 + c] = r0[c];
        if (c < nb && i1 < k) L[i1 * ld + p0 + c] = r1[c];
      }
    }
    __syncthreads();
    const int b0 = p0 + 8, m = k - b0;
    if (m > 0) {
      for (int e = tid; e < m * m; e += nt) {
        const int i = b0 + e / m, l = b0 + e % m;
        if (l > i) continue;
        const double *ri = L + i * ld + p0, *rl = L + l * ld + p0;
        double s = L[i * ld + l];
#pragma unroll
        for (int c = 0; c < 8; ++c) s -= ri[c] * rl[c];
        L[i * ld + l] = s;
      }
      __syncthreads();
    }
  }
}

// Y <- L^-T L^-1 Y for the k x ncol matrix Y (row-major, any memory), L
// lower (k <= 128, leading dimension ld), inv its inverse diagonal.  Columns
// are independent: wave q solves columns q, q + nwaves, ... with lane i holding
// rows i and i + 64; a solved entry passes by readlane, and the entries of L
// of eight steps are loaded before the first is used.  A pattern without free
// rows leaves nothing to solve (k = 0: L and inv have no entry to read).  Ends
// with a barrier.
__device__ inline void chol_solve_cols(const double* L, int k, int ld, const double* inv, double* Y,
                                       int ncol) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = (int)(blockDim.x >> 6);
  if (k <= 0) {                                               // uniform
    __syncthreads();
    return;
  }
  const int l0 = min(lane, k - 1), l1 = min(lane + 64, k - 1);
  const bool two = k > 64;                                    // uniform
  // the lane's own pivots and their reciprocals: each step's quotient is formed
  // in the lane that holds the entry, and passes from there
  const double d0 = L[l0 * ld + l0], e0 = inv[l0], d1 = L[l1 * ld + l1], e1 = inv[l1];
  for (int c = wv; c < ncol; c += nw) {
    double y0 = (lane < k) ? Y[lane * ncol + c] : 0.0;
    double y1 = (lane + 64 < k) ? Y[(lane + 64) * ncol + c] : 0.0;
    for (int j0 = 0; j0 < k; j0 += 8) {                       // L z = y
      double a0[8], a1[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = min(j0 + u, k - 1);
        a0[u] = L[l0 * ld + j];
        a1[u] = two ? L[l1 * ld + j] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = j0 + u;
        if (j >= k) break;                                    // uniform
        if (j < 64) {
          const double z = div_by(y0, d0, e0), zj = lane_d(z, j);
          y0 = lane == j ? z : (lane > j ? y0 - a0[u] * zj : y0);
          y1 -= a1[u] * zj;
        } else {
          const double z = div_by(y1, d1, e1), zj = lane_d(z, j - 64);
          y1 = lane == j - 64 ? z : (lane > j - 64 ? y1 - a1[u] * zj : y1);
        }
      }
    }
    for (int j0 = (k - 1) & ~7; j0 >= 0; j0 -= 8) {           // L^T x = z
      double a0[8], a1[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = min(j0 + u, k - 1);
        a0[u] = L[j * ld + min(lane, j)];
        a1[u] = two ? L[j * ld + min(lane + 64, j)] : 0.0;
      }
#pragma unroll
      for (int u = 7; u >= 0; --u) {
        const int j = j0 + u;
        if (j >= k) continue;                                 // uniform
        if (j < 64) {
          const double z = div_by(y0, d0, e0), xj = lane_d(z, j);
          y0 = lane == j ? z : (lane < j ? y0 - a0[u] * xj : y0);
        } else {
          const double z = div_by(y1, d1, e1), xj = lane_d(z, j - 64);
          y1 = lane == j - 64 ? z : (lane < j - 64 ? y1 - a1[u] * xj : y1);
          y0 -= a0[u] * xj;                                   // every row i < 64 <= j
        }
      }
    }
    if (lane < k) Y[lane * ncol + c] = y0;
    if (lane + 64 < k) Y[(lane + 64) * ncol + c] = y1;
  }
  __syncthreads();
}

}  // namespace fqp
