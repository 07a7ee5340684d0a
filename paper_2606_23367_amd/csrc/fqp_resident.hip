// Account-resident iterations (gfx950): a block of ADMM iterations of one
// account in one workgroup, for books whose factor block one compute unit
// can stream in a few microseconds.
//
// The four passes of fqp_iter.hip cost a launch's latency chain each (8 to
// 20 us an iteration however small the book).  Here the workgroup of an
// account runs every iteration of a block itself: the state stays in LDS,
// the factor-space solve in registers and LDS, and the only stream is B~
// from the XCD's L2 (64 B a clock and compute unit: what bounds the kernel
// at the larger sizes; the instruction stream runs at about the same rate).
//
// One pass over B~ serves both products.  A tile of 64 rows is held as
//   lane (c = lane & 3, r = lane >> 2):  rows 16 u + r (u = 0..3), columns
//   c + 4 q (q < KQ),
// so that (B~ p)_i needs the sum over a quad of lanes only (DPP), after which
// lane (c, r) owns row 16 c + r: it forms v' = w + alpha Delta^-1 (nu -
// (B~ p)_i), the prox step and R', the quad passes its four R' around (DPP)
// and the same registers of B~ accumulate t = B~^T R'.  The sums over the 16
// lanes of a column class are taken once per iteration.  (With a turnover
// cap the multiplier search stands between the products: two passes.)
//
// Measured, us an iteration (four passes before): 1 account x 100 names 13.2 ->
// 1.5; 128 x 481 (21 columns) 18 -> 2.4; 128 x 2,000 (51) 25.8 -> 7.5, 3.0 of
// them the L2 stream; 128 x 5,000 (71) 36.5 -> 17.0, 9.5 the stream.  About
// 1.5 us are the three barriers of the factor-space solve.
//
// B~ is stored in that order: float4 (u = 0..3) per [tile][q][lane], 1 KB a
// wave and load.  All arithmetic is float32 as in the float32 passes, the
// factor-space solve float64 as in ksolve_kernel.
#include <type_traits>

#include "fqp_common.h"
#include "fqp_kernels.h"
#include "../../include/fqp.h"

namespace fqp {

// quad permutation of a float (DPP): PERM = 4 x 2-bit source lanes
template <int PERM>
__device__ __forceinline__ float quad(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), PERM, 0xf, 0xf, true));
}
constexpr int kQx1 = 0xB1;               // [1, 0, 3, 2]
constexpr int kQx2 = 0x4E;               // [2, 3, 0, 1]

template <int PERM>
__device__ __forceinline__ double quad_d(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, PERM, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), PERM, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// rotation by N lanes within each row of 16 (DPP)
template <int N>
__device__ __forceinline__ float ror(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x120 + N, 0xf, 0xf, true));
}
// sum over the wave: DPP rotations within the rows of 16 lanes, the four row
// sums through scalar registers (no LDS round trip)
template <int N>
__device__ __forceinline__ double ror_d(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + N, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + N, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double x) {
  x += ror_d<1>(x);
  x += ror_d<2>(x);
  x += ror_d<4>(x);
  x += ror_d<8>(x);
  return (lane_d(x, 0) + lane_d(x, 16)) + (lane_d(x, 32) + lane_d(x, 48));
}
__device__ __forceinline__ float wave_sum(float x) {
  x += ror<1>(x);
  x += ror<2>(x);
  x += ror<4>(x);
  x += ror<8>(x);
  const int b = __builtin_bit_cast(int, x);
  auto at = [&](int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, l)); };
  return (at(0) + at(16)) + (at(32) + at(48));
}

// the account's trade lines as the passes read them: {mu, w0, lb, ub} per
// row (rows n .. npr - 1: zeros) and, for books with tax lots, the index of
// the row's lot record or -1
__global__ __launch_bounds__(256) void resident_rows_kernel(ResRowArgs A) {
  const int a = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  if (i >= A.npr) return;
  float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
  int ix = -1;
  if (i < A.n) {
    const size_t wi = (size_t)a * A.W + (i >> 5), off = (size_t)a * A.n + i;
    const int b = i & 31;
    const bool el = A.elig == nullptr || ((A.elig[wi] >> b) & 1u);
    r.x = A.mu[off];
    asset_box(A, off, el, A.lb[a], A.ub[a], r.z, r.w);
    const uint32_t hw = A.hold[wi];
    if ((hw >> b) & 1u) {
      const int j = A.hold_ptr[a] + A.hold_pre[wi] + popc_below(hw, b);
      const float4 rec = A.hold_rec[2 * j];
      r.y = rec.x;
      if (rec.y > 0.f) ix = j;
    }
  }
  const size_t o = (size_t)a * A.npr + i;
  A.rows[o] = r;
  if (A.lot) A.lot[o] = ix;
}

// B~ in the tile order above (zeros past row n and column kp)
__global__ __launch_bounds__(256) void resident_bq_kernel(int n, int kp, int KQ, int ntile,
                                                          const float* Bt, float4* Bq) {
  const int total = ntile * KQ * 64;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int lane = e & 63, q = (e >> 6) % KQ, tile = (e >> 6) / KQ;
  const int col = (lane & 3) + 4 * q;
  float x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = tile * 64 + 16 * u + (lane >> 2);
    x[u] = (row < n && col < kp) ? Bt[(size_t)row * kp + col] : 0.f;
  }
  Bq[e] = make_float4(x[0], x[1], x[2], x[3]);
}

// the row's z at threshold th, from its line and (ix >= 0) its lots
struct ResLine {
  float4 r;              // {mu, w0, lb, ub}
  int ix;
  TaxLots t;
};

__device__ __forceinline__ float res_prox(const ResLine& L, bool lots, float v, float th,
                                          float irho) {
  float z = fminf(v + th, fmaxf(L.r.y, v - th));
  z = fminf(fmaxf(z, L.r.z), L.r.w);
  if (lots && L.ix >= 0) z = prox_taxed(v, L.r.y, th, irho, L.t, L.r.z, L.r.w);
  return z;
}

// the lots of a taxed row
__device__ __forceinline__ void res_lots(const ResArgs& A, const int* s_ix, bool lots, int row,
                                         ResLine& L) {
  L.ix = -1;
  if (lots) {
    L.ix = s_ix[row];
    if (L.ix >= 0) {
      const float4 r0 = A.hold_rec[2 * L.ix], r1 = A.hold_rec[2 * L.ix + 1];
      L.t.b1 = r0.y; L.t.b2 = r0.z; L.t.b3 = r0.w;
      L.t.s0 = r1.x; L.t.s1 = r1.y; L.t.s2 = r1.z; L.t.s3 = r1.w;
    }
  }
}

template <int KQ, int NTHR>
__global__ __launch_bounds__(NTHR) void resident_kernel(ResArgs A, int count) {
  constexpr int NW = NTHR / 64, KC = 4 * KQ;
  extern __shared__ float smem[];
  __shared__ float s_t[4 * NW][KC];       // parts of t, one per wave and row of 16 lanes
  __shared__ double s_td[KC];             // t, with the constraint rows' terms
  __shared__ float s_p[KC];               // back-projection coefficients
  __shared__ double s_y[kMaxG];           // rho_b (zb - vb) of the constraint rows
  __shared__ float s_zb[kMaxG], s_vb[kMaxG];
  __shared__ float s_g[2][NW], s_n[2][NW];
  const int slot = blockIdx.x;
  if (slot >= *A.m_act) return;
  const int a = A.act[slot];
  const int tid = threadIdx.x, lane = tid & 63;
  // (uniform: the tiles' addresses stay in scalar registers)
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = A.n, k = A.k, G = A.G, kg = k + G;
  float* s_w = smem;                                        // [npr] v or w of every row
  int* s_ix = reinterpret_cast<int*>(s_w + A.npr);          // [npr] with tax lots
  float* s_mb = s_w + (A.lot ? 2 : 1) * (size_t)A.npr;      // [kg + 1][G]
  float* par = A.par + (size_t)a * kNPar;
  const int cls = A.ncls == 1 ? 0 : (int)par[P_CLASS];
  const float rho = par[P_RHO], irho = 1.f / rho, kap = par[P_KAPPA], gam = par[P_GAMMA];
  const float alpha = par[P_ALPHA], rhob = par[P_RHOB], tau = par[P_TAU];
  const bool capped = isfinite(tau);
  const bool lots = A.lot != nullptr && par[P_HASTAX] != 0.f;
  float lam = capped ? par[P_LAM] : 0.f;
  const float* Kinv = A.Kinv + (size_t)cls * A.kp * A.kp;
  const float* qv = A.qvec + (size_t)cls * A.kp;
  const float4* rows = A.rows + (size_t)a * A.npr;
  float* vg = A.v + (size_t)a * n;

  // state and tables into LDS
  for (int i = tid; i < A.npr; i += NTHR) {
    s_w[i] = i < n ? vg[i] : 0.f;
    if (A.lot) s_ix[i] = A.lot[(size_t)a * A.npr + i];
  }
  for (int e = tid; e < (kg + 1) * G; e += NTHR) {
    const int j = e / G, g = e % G;
    s_mb[e] = j < kg ? A.mbg[((size_t)cls * A.kp + j) * G + g]
                     : A.cvec[(size_t)cls * A.kp + k + g];
  }
  for (int g = tid; g < G; g += NTHR) {
    const float zb = A.zb[(size_t)a * G + g], vb = A.vb[(size_t)a * G + g];
    s_zb[g] = zb;
    s_vb[g] = vb;
    s_y[g] = (double)rhob * ((double)zb - (double)vb);
  }
  for (int j = tid; j < KC; j += NTHR) { s_p[j] = 0.f; s_td[j] = 0.0; }
  // column j = tid >> 2 of K^-1: entries l = (tid & 3) + 4 i
  const int cj = tid >> 2, c4 = tid & 3;
  float kreg[KQ];
#pragma unroll
  for (int i = 0; i < KQ; ++i) {
    const int l = c4 + 4 * i;
    kreg[i] = (cj < kg && l < kg) ? Kinv[l * A.kp + cj] : 0.f;
  }
  const double q0 = lane < kg ? (double)qv[lane] : 0.0;
  const double q1 = lane + 64 < kg ? (double)qv[lane + 64] : 0.0;
  const double qj = cj < kg ? (double)qv[cj] : 0.0;
  const double sig1 = A.sig1[cls];
  float nu = 0.f;
  __syncthreads();

  const int own = (lane & 3) * 16 + (lane >> 2);            // the lane's row of a tile
  const bool h2 = lane & 2, h1 = lane & 1;
  float th = (kap + lam) * irho;
  float acc[KQ];

  const auto bq = __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(A.Bq), (short)0,
                                                    A.ntile * KQ * 1024, 0x00027000);
  // one pass over the account's rows: X: v = w + alpha Delta^-1 (nu - B~ p)
  // first; P: z, R' and w of that v, R' contracted into acc; out: v and z to
  // global memory
  auto pass = [&](auto X, auto P, bool out) {
    constexpr bool kX = decltype(X)::value, kP = decltype(P)::value;
    float p[KQ];
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      p[q] = kX ? s_p[(lane & 3) + 4 * q] : 0.f;
      if (kP) acc[q] = 0.f;
    }
    // a tile's registers are loaded for the next tile as the second product
    // reads them for the last time (the passes that have one), its line and
    // d with them: the L2 stream runs under the arithmetic
    float4 b[KQ];
    // (buffer loads: one offset register per lane, the tile's offset scalar)
    auto load = [&](int tile, int q) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(bq, lane * 16, tile * (KQ * 1024) + q * 1024, 0);
      return __builtin_bit_cast(float4, x);
    };
    float d_n = 1.f;
    float4 r_n = make_float4(0.f, 0.f, 0.f, 0.f);
    auto row_loads = [&](int tile) {
      const int row = tile * 64 + own;
      d_n = A.d[min(row, n - 1)];
      if (kP || out) r_n = rows[row];
    };
    if (wv < A.ntile) {
#pragma unroll
      for (int q = 0; q < KQ; ++q) b[q] = load(wv, q);
      row_loads(wv);
    }
    for (int tile = wv; tile < A.ntile; tile += NW) {
      const int row = tile * 64 + own;
      const int next = min(tile + NW, A.ntile - 1);
      const float d_i = d_n;
      ResLine L;
      L.r = r_n;
      if (kP || out) res_lots(A, s_ix, lots, row, L);
      if (kP) row_loads(next);
      float v = s_w[row];
      const float iD = __builtin_amdgcn_rcpf(gam * d_i + rho);
      if (kX) {
        float x0 = 0.f, x1 = 0.f, x2 = 0.f, x3 = 0.f;
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
          x0 += b[q].x * p[q];
          x1 += b[q].y * p[q];
          x2 += b[q].z * p[q];
          x3 += b[q].w * p[q];
          if (!kP && (q % 3 == 2 || q == KQ - 1)) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = q - q % 3; r <= q; ++r) b[r] = load(next, r);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (!kP) row_loads(next);
        // the quad's four partials of rows u = 0..3: lane c keeps u = c
        const float y0 = (h2 ? x2 : x0) + quad<kQx2>(h2 ? x0 : x2);
        const float y1 = (h2 ? x3 : x1) + quad<kQx2>(h2 ? x1 : x3);
        const float x = (h1 ? y1 : y0) + quad<kQx1>(h1 ? y0 : y1);
        v = row < n ? v + alpha * iD * (nu - x) : 0.f;
      }
      if (kP) {
        const float z = res_prox(L, lots, v, th, irho);
        const float Rp = (L.r.x + rho * (z - (v - z))) * iD;
        s_w[row] = v + alpha * (Rp - z);
        const float Rm = row < n ? Rp : 0.f;
        const float r0 = quad<0x00>(Rm), r1 = quad<0x55>(Rm), r2 = quad<0xAA>(Rm),
                    r3 = quad<0xFF>(Rm);
        // (the barriers keep a register's reload behind its last use: hoisted
        // ahead of it the loads would need a second set of registers)
#pragma unroll
        for (int q = 0; q < KQ; ++q) {
          acc[q] = fmaf(b[q].w, r3, fmaf(b[q].z, r2, fmaf(b[q].y, r1, fmaf(b[q].x, r0, acc[q]))));
          if (q % 3 == 2 || q == KQ - 1) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = q - q % 3; r <= q; ++r) b[r] = load(next, r);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
        s_w[row] = v;
        if (out && row < n) {
          vg[row] = v;
          if (!capped) A.zs[(size_t)a * n + row] = res_prox(L, lots, v, th, irho);
        }
      }
    }
  };

  // the exact cap multiplier of the v in s_w (every lane on its own rows)
  auto search = [&]() {
    float lo = 0.f, hi_b = INFINITY, best_feas = INFINITY;
    bool done = false;
    for (int it = 0; it < 48 && !done; ++it) {              // done is uniform
      const float t1 = (kap + lam) * irho;
      float g = 0.f, nf = 0.f;
      for (int tile = wv; tile < A.ntile; tile += NW) {
        const int row = tile * 64 + own;
        ResLine L;
        L.r = rows[row];
        res_lots(A, s_ix, lots, row, L);
        const float z = res_prox(L, lots, s_w[row], t1, irho);
        g += fabsf(z - L.r.y);
        bool kink = (z == L.r.y) || z <= L.r.z || z >= L.r.w;
        if (lots && L.ix >= 0)
          kink = kink || (z == L.r.y - L.t.b1) || (z == L.r.y - L.t.b2) || (z == L.r.y - L.t.b3);
        nf += kink ? 0.f : 1.f;
      }
      g = wave_sum(g);
      nf = wave_sum(nf);
      const int buf = it & 1;
      if (lane == 0) { s_g[buf][wv] = g; s_n[buf][wv] = nf; }
      __syncthreads();
      float gt = 0.f, nft = 0.f;
#pragma unroll
      for (int q = 0; q < NW; ++q) { gt += s_g[buf][q]; nft += s_n[buf][q]; }
      lam = cap_step(gt, nft, tau, rho, lam, lo, hi_b, best_feas, done);
    }
    lam = cap_result(lam, done, best_feas);                 // the same in every thread
    th = (kap + lam) * irho;
    __syncthreads();                                        // s_g, s_n free again
  };

  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  for (int it = 0; it < count; ++it) {
    if (capped) {
      if (it > 0) pass(yes, no, false);
      search();
      pass(no, yes, false);
    } else if (it == 0) {
      pass(no, yes, false);
    } else {
      pass(yes, yes, false);
    }
    // t: over the four lanes of a column class in each row of 16 lanes (DPP),
    // then over the rows and the waves, four threads a column
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      float s = acc[q];
      s += ror<4>(s);
      s += ror<8>(s);
      if ((lane & 15) < 4) s_t[4 * wv + (lane >> 4)][(lane & 3) + 4 * q] = s;
    }
    __syncthreads();
    if (cj <= kg) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < NW; ++q) t += (double)s_t[4 * q + c4][cj];
      const float* mb = s_mb + cj * G;
      for (int g = c4; g < G; g += 4) t += (double)mb[g] * s_y[g];
      t += quad_d<kQx2>(t);
      t += quad_d<kQx1>(t);
      if (c4 == 0) s_td[cj] = t;
    }
    __syncthreads();
    // nu = (1 - s0 + q^T t) / sigma1, in every wave; p = K^-1 t + nu q, four
    // lanes a column
    double qt = q0 * s_td[min(lane, KC - 1)] + q1 * s_td[min(lane + 64, KC - 1)];
    qt = wave_sum(qt);
    const double nud = (1.0 - s_td[kg] + qt) / sig1;
    nu = (float)nud;
    if (cj < kg) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < KQ; ++i) {
        // (opaque: the conversions stay here, not in registers of their own
        // across the passes)
        float kv = kreg[i];
        asm volatile("" : "+v"(kv));
        s += (double)kv * s_td[c4 + 4 * i];          // (kreg is 0 past column kg - 1)
      }
      s += quad_d<kQx2>(s);
      s += quad_d<kQx1>(s);
      if (c4 == 0) {
        const float pj = (float)(s + nud * qj);
        if (cj < k) {
          s_p[cj] = pj;
        } else {
          // constraint row g: A x = p' / rho_b, its ADMM step
          const int g = cj - k;
          const float zb = s_zb[g], vb = s_vb[g];
          s_p[cj] = pj - rhob * (zb - vb);
          const float ax = pj / rhob;
          const float zh = alpha * ax + (1.f - alpha) * zb;
          const float zn = fminf(fmaxf(zh + vb, A.blo[(size_t)a * G + g]), A.bhi[(size_t)a * G + g]);
          const float vn = vb + zh - zn;
          s_zb[g] = zn;
          s_vb[g] = vn;
          s_y[g] = (double)rhob * ((double)zn - (double)vn);
        }
      }
    }
    __syncthreads();
  }
  pass(yes, no, true);
  if (capped) {
    // z of the final v at its own multiplier, the input of the polish
    search();
    for (int tile = wv; tile < A.ntile; tile += NW) {
      const int row = tile * 64 + own;
      if (row < n) {
        ResLine L;
        L.r = rows[row];
        res_lots(A, s_ix, lots, row, L);
        A.zs[(size_t)a * n + row] = res_prox(L, lots, s_w[row], th, irho);
      }
    }
  }
  for (int g = tid; g < G; g += NTHR) {
    A.zb[(size_t)a * G + g] = s_zb[g];
    A.vb[(size_t)a * G + g] = s_vb[g];
  }
  if (tid == 0) {
    if (capped) par[P_LAM] = lam;
    par[P_NU] = nu;
    A.iters[a] += count;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int resident_kq(int kw) {
  const int q = (kw + 3) / 4;
  return q <= 6 ? 6 : q <= 8 ? 8 : q <= 11 ? 11 : q <= 14 ? 14 : q <= 18 ? 18 : q <= 21 ? 21 : 24;
}

// Which books: the resident block wins while one compute unit streams the
// account's share of B~ faster than four launches drain.  Both sides in us
// an iteration, fitted to measurements over n = 64 .. 16,384, 6 .. 96 columns, 1 ..
// 4,096 accounts, 100 held names an account and all of them (resident / four
// passes):
//   no cap:  100 x 6, 1 account 1.5 / 13.2;  481 x 21, 128 accounts 2.4 / 18;
//            2,000 x 51, 128: 7.5 / 26;  5,000 x 71, 128: 17 / 37;
//            128 x 6, 4,096: 23 / 60;  10,000 x 81, 1: 32 / 26, 128: 36 / 46
//            8,192 x 56, 1,024: 88 / 68 with 100 held names, / 133 with all
//   caps:    481 x 21, 128: 6.3 / 22;  2,000 x 51, 128: 19 / 29;
//            4,000 x 41, 1: 25 / 21, 128: 26 / 29;  10,000 x 81: 76 / 29
//            2,048 x 6, 512: 48 / 39 with lots on every name, 27 / 34 without
// A capped account streams B~ twice and searches its rows, their lots from
// memory past the first few hundred; more accounts than compute units take
// further rounds of workgroups.  The four passes cost by the launches and the
// workgroups an account takes, and by the entries: four times as much an entry
// where PROX cannot hold the held names in LDS or walks per-asset bounds, or with
// float32 contractions (at one price for all, books of few held names took blocks
// up to 1.46 times as long).
bool resident_fits(int n, int kw, int G, bool lots, int m, int ncap, int max_held, bool asset_box,
                   bool split, int n_cu) {
  if (kw > 96) return false;
  const int tiles = (n + 63) / 64;
  const size_t smem = sizeof(float) * ((size_t)tiles * 64 * (lots ? 2 : 1) + (size_t)kw * G);
  if (smem > 140 * 1024) return false;
  const double stream = 0.011 * tiles * resident_kq(kw);
  const double rounds = n_cu > 0 ? (double)((m + n_cu - 1) / n_cu) : 1.0;
  const double far_lots = lots && max_held > 512 ? 0.004 * (max_held - 512) : 0.0;
  const double res = rounds * (ncap > 0 ? 3.5 + 2.0 * stream + 0.0022 * n + far_lots
                                        : 1.6 + stream * (lots ? 1.05 : 1.0));
  const double entry = max_held > 1024 || asset_box || !split ? 1.2e-5 : 3e-6;
  const double four = 13.0 + 0.1 * kw + (m > 8 ? 4.0 : 0.0) + 6e-4 * n +
                      (ncap > 0 ? 7e-6 * (double)n * m : entry * (double)n * m + 0.01 * m);
  return res < 0.95 * four;
}

static size_t resident_smem(const ResArgs& A) {
  return sizeof(float) * ((size_t)A.npr * (A.lot ? 2 : 1) + (size_t)(A.k + A.G + 1) * A.G);
}

template <int KQ, int NTHR>
static hipError_t launch_resident_t(const ResArgs& A, int m_total, int count, hipStream_t st) {
  const size_t smem = resident_smem(A);
  hipError_t e = hipFuncSetAttribute((const void*)resident_kernel<KQ, NTHR>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 140 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((resident_kernel<KQ, NTHR>), dim3(m_total), dim3(NTHR), smem, st, A, count);
  return hipGetLastError();
}

hipError_t launch_resident(const ResArgs& A, int KQ, int m_total, int count, hipStream_t st) {
  switch (KQ) {
    case 6: return launch_resident_t<6, 1024>(A, m_total, count, st);
    case 8: return launch_resident_t<8, 512>(A, m_total, count, st);
    case 11: return launch_resident_t<11, 512>(A, m_total, count, st);
    case 14: return launch_resident_t<14, 512>(A, m_total, count, st);
    case 18: return launch_resident_t<18, 512>(A, m_total, count, st);
    case 21: return launch_resident_t<21, 512>(A, m_total, count, st);
    case 24: return launch_resident_t<24, 512>(A, m_total, count, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_resident_setup(const ResRowArgs& A, int kp, int KQ, const float* Bt, float4* Bq,
                                 hipStream_t st) {
  const int ntile = A.npr / 64;
  hipLaunchKernelGGL(resident_bq_kernel, dim3((ntile * KQ * 64 + 255) / 256), dim3(256), 0, st,
                     A.n, kp, KQ, ntile, Bt, Bq);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(resident_rows_kernel, dim3((A.npr + 255) / 256, A.m), dim3(256), 0, st, A);
  return hipGetLastError();
}

}  // namespace fqp
