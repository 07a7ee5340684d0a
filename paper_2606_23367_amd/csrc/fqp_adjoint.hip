// KKT adjoint of the certified solutions (gfx950, float64).
//
// For a certified account the optimum of the build's Eq. 1 instance solves
// the reduced equality system of its active pattern (fixed coordinates at
// bounds / kinks, free coordinates F inside linear pieces, binding budget /
// bands / cap rows C_F):
//
//   gamma Sigma_FF w_F + C_F^T eta = mu_F - slope_F - gamma Sigma_FX w_X,
//   C_F w_F = h.
//
// Differentiating, for a loss L with gradient c = dL/dw the adjoint solves
//   [gamma Sigma_FF  C_F^T; C_F  0] [v; xi] = [c_F; 0],   v = 0 off F,
// and then  dL/dmu = eta v  and  dL/dB = -sum_a gamma_a (v_a (F B^T e_a)^T +
// e_a (F B^T v_a)^T)  with e = w - w_b (Sigma e changes by dB F B^T e +
// B F dB^T e; the halfspace rows are data of their own).  The constraint
// rows C_F are the budget, the binding band and halfspace rows and the cap.
// The solve reuses the polish's factor-space structure: Kf = diag(f)^-1 +
// B_F^T D_F^-1 B_F in LDS, Schur complement on the constraint rows.
#include <algorithm>

#include "fqp_common.h"
#include "fqp_dense.h"
#include "fqp_kernels.h"
#include "../../include/fqp.h"

namespace fqp {

enum PStateA { PA_CAP = 0, PA_NF, PA_NX, PA_NC, PA_DONE, PA_ROUNDS, PA_BACT0, PA_BACT1 };

__device__ __forceinline__ bool band_on(const int* ps, int g) {
  return g < 32 ? ((ps[PA_BACT0] >> g) & 1) : ((ps[PA_BACT1] >> (g - 32)) & 1);
}

// One workgroup per account: v (= dL/dmu) and the factor vectors F B^T w,
// F B^T v used by the dL/dB product.  Bound by its serial parts (two
// factorisations, the substitutions).  256 threads with 33 + 48 sums each over
// rows staged 16 at a time, a factorisation step per column and serial sums over
// the rows took 300 us at 128 x 5,000 (10 free rows) and 1,296 us at 160 free
// rows; 65 and 111 now.
__global__ __launch_bounds__(kPT) void adjoint_solve_kernel(AdjArgs A) {
  extern __shared__ double smem_d[];
  __shared__ double s_h[kSchurW], s_e0[kSchurW], s_xi[kMaxG + 3], s_inv[kMaxK], s_sol[kMaxK];
  const int k = A.k, G = A.G, n = A.n;
  const int a = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  constexpr int kW = kPT / 64;
  double* v = A.dmu + (size_t)a * n;
  for (int i = tid; i < n; i += kPT) v[i] = 0.0;
  if (A.status[a] != FQP_SOLVED) {
    for (int j = tid; j < 2 * k; j += kPT) A.yvw[(size_t)a * 2 * k + j] = 0.0;
    return;
  }
  const int* ps = A.pstate + (size_t)a * kPStateStride;
  const int nF = ps[PA_NF], nX = ps[PA_NX];
  const int cap_on = ps[PA_CAP];
  const int32_t* flist = A.flist + (size_t)a * n;
  const double gam = A.par[(size_t)a * kNPar + P_GAMMA];
  const double* c = A.dLdw + (size_t)a * n;
  const double* w = A.w + (size_t)a * n;
  int nb = 0;
  for (int g = 0; g < G; ++g) nb += band_on(ps, g) ? 1 : 0;
  const int nc = 1 + nb + (cap_on ? 1 : 0);
  const int ncol = nc + 1;
  double* Waug = A.wk + (size_t)a * A.wk_stride;
  double* Y = Waug + (size_t)k * (G + 3);
  double* CV = Y + (size_t)k * (G + 3);
  double* S = CV + (size_t)(G + 3) * (G + 3);

  // ---- one pass over the free rows: Kf = diag(1/f) + sum_F b b^T / d (lower
  // triangle), Waug = sum_F b V^T / d, CV = sum_F V V^T / d, V = [C_i, c_i].  A
  // 4 x 4 register tile a thread: the first ntile threads on Kf, the last on
  // X^T D^-1 V, X = [b | V]
  const int ld = kf_ld(k), SR = stage_rows(k, G), SS = stage_stride(k, ncol);
  double* Kf = smem_d;
  double* stg = Kf + k * ld;                // [SR][SS], 1 / d_i at index SS - 4
  const int kx = k + ncol, xt = (kx + 3) >> 2, vt = (ncol + 3) >> 2;
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
        int i = 0;
        double c_r = 0.0, w_r = 0.0, w0_r = 0.0, d_r = 1.0;
        if (tid < rows) {
          i = flist[f0 + tid];
          c_r = c[i];
          w_r = w[i];
          w0_r = A.w0in[(size_t)a * n + i];
          d_r = (double)A.d[i];
        }
        for (int e = tid; e < rows * k; e += kPT) {
          const int rr = e / k, j = e % k;
          stg[rr * SS + j] = (double)A.Bt[(size_t)flist[f0 + rr] * A.kp + j];
        }
        __syncthreads();
        if (tid < rows) {
          double* x = stg + tid * SS;
          double* vv = x + k;
          vv[0] = 1.0;
          int col = 1;
          for (int g = 0; g < G; ++g) {
            if (!band_on(ps, g)) continue;
            vv[col++] = row_coef(A, i, g);
          }
          // side of w0 of the piece the free coordinate lies in
          if (cap_on) vv[col++] = (w_r > w0_r) ? 1.0 : -1.0;
          vv[col] = c_r;
          x[SS - 4] = 1.0 / d_r;
          for (int q = kx; q < 4 * xt; ++q) x[q] = 0.0;
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
              Waug[j * ncol + l] = acc[q * 4 + s];
              Y[j * ncol + l] = acc[q * 4 + s];
            } else {
              CV[(j - k) * ncol + l] = acc[q * 4 + s];
            }
          }
      }
    }
  }
  __syncthreads();
  // ---- Y = Kf^-1 Waug, S = C H^-1 [C^T | c] --------------------------------
  chol_factor(Kf, k, ld, s_inv);
  chol_solve_cols(Kf, k, ld, s_inv, Y, ncol);
  const bool sl = nc <= kSchurW;
  double* Sd = sl ? smem_d : S;             // over Kf
  for (int e = tid; e < nc * ncol; e += kPT) {
    const int p = e / ncol, q = e % ncol;
    double s = CV[p * ncol + q];
#pragma unroll 8
    for (int j = 0; j < k; ++j) s -= Waug[j * ncol + p] * Y[j * ncol + q];
    Sd[p * ncol + q] = s / gam;
  }
  if (tid < kSchurW) { s_h[tid] = 0.0; s_e0[tid] = 0.0; }
  __syncthreads();
  // S xi = C H^-1 c (h = 0), S PSD: pivoted Cholesky, the components the
  // free rows do not pin are set to 0 (they do not change v)
  if (sl) {
    if (tid < 64)
      schur_solve_wave(nc, ncol, smem_d, s_h, s_e0, smem_d + nc * ncol, s_xi, S, G + 3);
  } else if (tid == 0) {
    double* Sm = CV;
    int perm[kMaxG + 3];
    double dmax = 0.0;
    for (int p = 0; p < nc; ++p) {
      perm[p] = p;
      dmax = fmax(dmax, S[p * ncol + p]);
      for (int q = 0; q < nc; ++q) Sm[p * nc + q] = S[p * ncol + q];
    }
    int rank = 0;
    for (int j = 0; j < nc; ++j) {
      int best = j;
      for (int p = j + 1; p < nc; ++p)
        if (Sm[p * nc + p] > Sm[best * nc + best]) best = p;
      if (!(Sm[best * nc + best] > 1e-12 * dmax)) break;
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
    double x[kMaxG + 3];
    for (int j = 0; j < nc; ++j) x[j] = (j < rank) ? S[perm[j] * ncol + nc] : 0.0;
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
    for (int j = 0; j < nc; ++j) s_xi[perm[j]] = x[j];
  }
  __syncthreads();
  for (int j = tid; j < k; j += kPT) {
    double s = Y[j * ncol + nc];
    for (int p = 0; p < nc; ++p) s -= Y[j * ncol + p] * s_xi[p];
    s_sol[j] = s;
  }
  __syncthreads();
  // ---- v_i = (c_i - C_i^T xi - b_i . sol) / (gamma d_i), 16 threads a row
  for (int t0 = 0; t0 < nF; t0 += kPT / 16) {
    const int t = min(t0 + (tid >> 4), nF - 1), q = tid & 15;
    const int i = flist[t];
    double bs = 0.0;
    for (int j = q; j < k; j += 16) bs += (double)A.Bt[(size_t)i * A.kp + j] * s_sol[j];
    bs = row_red(bs, SumOp());
    if (q == 0 && t0 + (tid >> 4) < nF) {
      double ct = s_xi[0];
      int col = 1;
      for (int g = 0; g < G; ++g) {
        if (!band_on(ps, g)) continue;
        ct += row_coef(A, i, g) * s_xi[col];
        ++col;
      }
      if (cap_on) ct += ((w[i] > (double)A.w0in[(size_t)a * n + i]) ? 1.0 : -1.0) * s_xi[col];
      v[i] = (c[i] - ct - bs) / (gam * (double)A.d[i]);
    }
  }
  __syncthreads();
  // ---- F B^T w (free + nonzero fixed rows) and F B^T v (free rows): eight rows
  // a wave at a time, its lanes the columns; the waves' partials meet in LDS
  {
    const int j0 = min(lane, k - 1), j1 = min(lane + 64, k - 1);
    const bool two = k > 64;                               // uniform
    const int cnt = nF + nX;
    double w0 = 0.0, w1 = 0.0, v0 = 0.0, v1 = 0.0;
    for (int t0 = 8 * wv; t0 < cnt; t0 += 8 * kW) {
      double wt[8], vt8[8];
      float b0[8], b1[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = min(t0 + u, cnt - 1);
        const int i = flist[t < nF ? t : n - 1 - (t - nF)];
        const float* row = A.Bt + (size_t)i * A.kp;
        const bool on = t0 + u < cnt;
        const double wi = w[i], vi = v[i];
        wt[u] = on ? wi : 0.0;
        vt8[u] = on && t < nF ? vi : 0.0;
        b0[u] = row[j0];
        b1[u] = two ? row[j1] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        w0 += (double)b0[u] * wt[u];
        v0 += (double)b0[u] * vt8[u];
        w1 += (double)b1[u] * wt[u];
        v1 += (double)b1[u] * vt8[u];
      }
    }
    double* red = smem_d;                                  // [2][kW][k]
    if (lane < k) { red[wv * k + lane] = w0; red[(kW + wv) * k + lane] = v0; }
    if (lane + 64 < k) { red[wv * k + lane + 64] = w1; red[(kW + wv) * k + lane + 64] = v1; }
    __syncthreads();
    for (int e = tid; e < 2 * k; e += kPT) {
      const int j = e % k, r = e / k;
      double s = 0.0;
      for (int q = 0; q < kW; ++q) s += red[(r * kW + q) * k + j];
      if (r == 0 && A.wb) s -= A.ywb[(size_t)a * k + j];   // e = w - w_b
      A.yvw[(size_t)a * 2 * k + e] = gam * (double)A.f[j] * s;   // gamma F B^T e, gamma F B^T v
    }
  }
}

// dL/dB[i][j] = -sum_a ( v_a,i (gamma F B^T w_a)_j + e_a,i (gamma F B^T v_a)_j )
// a product of depth 2 m in float64 on the matrix cores: a wave owns a tile of
// 16 rows and 16 factors and takes four accounts a step (accounts in order:
// deterministic), loads of four steps in flight.  One workgroup per 64 rows
// walking the accounts with two barriers each was 246 us at 128 x 5,000 x 60;
// 21 now, bound by the latency of its loads.
typedef double d4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void adjoint_db_kernel(AdjArgs A) {
  const int k = A.k, n = A.n, m = A.m;
  const int nct = (k + 15) >> 4;
  const int lane = threadIdx.x & 63;
  const int tile = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  const int r0 = (tile / nct) * 16, c0 = (tile % nct) * 16;
  if (r0 >= n) return;
  // operands: lane l holds row (factor) l & 15 of account l >> 4 of a step
  const int i = min(r0 + (lane & 15), n - 1), j = min(c0 + (lane & 15), k - 1);
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int a0 = 0; a0 < m; a0 += 16) {
    double av[4], aw[4], yv[4], yw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int a = a0 + 4 * u + (lane >> 4), ac = min(a, m - 1);
      const size_t off = (size_t)ac * n + i;
      const double vi = A.dmu[off], wi = A.w[off];
      const double wb = A.wb ? (double)A.wb[off] : 0.0;
      const double y0 = A.yvw[(size_t)ac * 2 * k + j], y1 = A.yvw[(size_t)ac * 2 * k + k + j];
      // (an uncertified account has no gradient, and its weights may be anything)
      const bool on = a < m && A.status[ac] == FQP_SOLVED;
      av[u] = on ? vi : 0.0;
      aw[u] = on ? wi - wb : 0.0;
      yv[u] = on ? y0 : 0.0;
      yw[u] = on ? y1 : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], yv[u], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[u], yw[u], acc, 0, 0, 0);
    }
  }
  // result: lane l holds factor l & 15 of rows l >> 4, + 4, + 8, + 12
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int row = r0 + (lane >> 4) + 4 * q, col = c0 + (lane & 15);
    if (row < n && col < k) A.dB[(size_t)row * k + col] = -acc[q];
  }
}

// dL/dmu = eta dL/dmu' (mu' = eta mu + gamma Sigma w_b), after dL/dB used v
__global__ void adjoint_eta_kernel(AdjArgs A) {
  const size_t total = (size_t)A.m * A.n;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (size_t)gridDim.x * blockDim.x)
    A.dmu[e] *= (double)A.eta[e / A.n];
}

hipError_t launch_adjoint(const AdjArgs& A, hipStream_t st) {
  // Kf and the staged rows; over them the constraint system and the list sums
  const size_t factor = (size_t)A.k * kf_ld(A.k) +
                        (size_t)stage_rows(A.k, A.G) * stage_stride(A.k, A.G + 3);
  const size_t schur = (size_t)kSchurW * (2 * kSchurW + 1), sums = 2 * (kPT / 64) * (size_t)A.k;
  const size_t smem = sizeof(double) * std::max(factor, std::max(schur, sums));
  hipError_t e = hipFuncSetAttribute((const void*)adjoint_solve_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     153 * 1024);   // at k = 128 and the most rows
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(adjoint_solve_kernel, dim3(A.m), dim3(kPT), smem, st, A);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int tiles = ((A.n + 15) / 16) * ((A.k + 15) / 16);
  hipLaunchKernelGGL(adjoint_db_kernel, dim3((tiles + 3) / 4), dim3(256), 0, st, A);
  e = hipGetLastError();
  if (e != hipSuccess || !A.eta) return e;
  hipLaunchKernelGGL(adjoint_eta_kernel, dim3(1024), dim3(256), 0, st, A);
  return hipGetLastError();
}

}  // namespace fqp
