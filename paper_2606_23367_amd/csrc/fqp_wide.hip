// Fused iteration pass of wide books (gfx950): the float32 passes PROJECT,
// PROX and CONTRACT of fqp_iter.hip in one launch, for few accounts without
// turnover caps over many assets.
//
// Without a cap the prox step needs nothing but the row's own v, so the
// back-projection of one iteration, the prox step and the contraction of the
// next run on one 128-row chunk of B~ while it is in LDS: B~ is read from
// HBM once an iteration instead of twice, and the per-account PROX launch
// (one workgroup an account: 423 us at 8 x 384,800) is gone.
//
// The products run on v_mfma_f32_16x16x4 (16 accounts; half the padding of
// the 32-account tiles).  A float32 MFMA is a chain of fused multiply-adds in
// ascending k (checked against fmaf chains bit for bit), so every sum keeps
// the order of the four passes -- the back-projection over ascending
// columns, the contraction over ascending rows of each 32-row strip per wave,
// chunk after chunk, the strips in order -- and the iterates are the same
// numbers bit for bit.
//
// 512 threads: wave w takes rows 16 w .. 16 w + 15 of a chunk through the
// back-projection and the prox step, then strip w / 2 (32 rows) and half
// w % 2 of the columns through the contraction.  The next chunk is loaded into
// registers while the current one is worked on (50 to 80 KB in flight a compute
// unit).  Columns are stored permuted within groups of 16 (column 4 i + j at
// 4 j + i), so that four k-steps of the back-projection's operand are one
// 16-byte LDS read; rows are kp + 4 words apart (those reads are free of bank
// conflicts).
//
// Bound by the phases of a chunk, one workgroup a compute unit: of 5.7 us at
// 8 x 384,800 x 160 the back-projection is 2.1 (1.1 of it the matrix pipe), the
// prox step 1.2, the contraction 0.7, the chunk's way into LDS 0.5 and the three
// barriers 1.2; no wave waits for memory.  84 us a launch with every column
// streamed and the rows' own data loaded after the back-projection, 77 now.
#include "fqp_common.h"
#include "fqp_kernels.h"
#include "../../include/fqp.h"

namespace fqp {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWdAcc = 16;                // accounts (MFMA rows)
constexpr int kWdT = 512;                 // threads

// position of a column within its group of 16
__host__ __device__ __forceinline__ int wide_pos(int col) {
  return (col & ~15) + 4 * (col & 3) + ((col >> 2) & 3);
}

// Columns of B~ kept in memory: without halfspace rows the factor columns (in
// fours), as the one-hot band columns follow from the labels and the last
// column is 1; else all of them.  That is 154 MB instead of 246 at 384,800 x (100
// factors + 50 bands): a third less to stream, and it stays in the 256 MB
// last-level cache from one iteration to the next.
__host__ __device__ __forceinline__ int wide_cols(int k, int kp, int H) {
  return H > 0 ? kp : (k + 3) & ~3;
}

// Bp, per 128-row chunk: [whole groups of 16 columns][128 rows][16, permuted],
// then [fours of columns left][128 rows][4]
__global__ __launch_bounds__(256) void wide_perm_kernel(int n, int npad, int kp, int kc,
                                                        const float* Bt, float* Bp) {
  const size_t total = (size_t)npad * kc;
  const int per = kRowsPerChunk * kc, full = (kc >> 4) * kRowsPerChunk * 16;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
    const int ch = (int)(e / per), x = (int)(e % per);
    int rr, col;
    if (x < full) {
      const int p = x & 15;
      rr = (x >> 4) % kRowsPerChunk;
      // (the permutation is its own inverse)
      col = (x >> 4) / kRowsPerChunk * 16 + 4 * (p & 3) + (p >> 2);
    } else {
      const int y = x - full;
      rr = (y >> 2) % kRowsPerChunk;
      col = (kc & ~15) + (y >> 2) / kRowsPerChunk * 4 + (y & 3);
    }
    const int row = ch * kRowsPerChunk + rr;
    Bp[e] = row < n ? Bt[(size_t)row * kp + col] : 0.f;
  }
}

template <int NT>                         // kp = 16 NT
__global__ __launch_bounds__(kWdT) void wide_kernel(WideArgs A, int do_x, int do_p) {
  constexpr int kp = 16 * NT, S = kp + 4, NH = NT / 2;
  extern __shared__ float smem[];
  float* Bs = smem;                                             // [128][S]
  float* Rs = Bs + kRowsPerChunk * S;                           // [128][16] R'
  float4* Acc = reinterpret_cast<float4*>(Rs + kRowsPerChunk * kWdAcc);   // [16][2]
  int* Aid = reinterpret_cast<int*>(Acc + 2 * kWdAcc);          // [16] account, -1: none
  int* Hp = Aid + kWdAcc;                                       // [16] first held record
  const int m_act = *A.m_act;
  const TileMap tm = tile_map(m_act, A.n, gridDim.x, blockIdx.x);
  if (!tm.active) return;                                       // one tile: m_act <= 16
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, q4 = lane >> 4;
  const int n = A.n;
  if (tid < kWdAcc) {
    // MFMA row 4 q + r takes the list's account 4 r + q: a lane's four rows are
    // filled one after another over all lanes, so that few accounts take few
    // rounds of the prox step (1.75 us a chunk for four rounds, of 5.8)
    const int j = 4 * (tid & 3) + (tid >> 2);
    const int a = j < m_act ? A.act[j] : -1;
    Aid[tid] = a;
    Hp[tid] = a >= 0 ? A.hold_ptr[a] : 0;
    float4 c0 = make_float4(1.f, 1.f, 0.f, 0.f), c1 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a >= 0) {
      const float* p = A.par + (size_t)a * kNPar;
      const float rho = p[P_RHO], irho = 1.f / rho, kap = p[P_KAPPA], lam = 0.f;
      c0 = make_float4(rho, irho, p[P_GAMMA], (kap + lam) * irho);
      c1 = make_float4(p[P_LB], p[P_UB], p[P_NU], p[P_ALPHA]);
    }
    Acc[2 * tid] = c0;
    Acc[2 * tid + 1] = c1;
  }
  __syncthreads();
  const int rounds = (m_act + 3) >> 2;                          // of the lanes' accounts (uniform)
  // p of MFMA row l16, columns 4 s + q4
  float p[kp / 4];
  {
    const int a = Aid[l16];
#pragma unroll
    for (int s = 0; s < kp / 4; ++s)
      p[s] = (do_x && a >= 0) ? A.pp[(size_t)a * kp + 4 * s + q4] : 0.f;
  }
  floatx4 T[NH];
#pragma unroll
  for (int c = 0; c < NH; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) T[c][r] = 0.f;
  const float* src = do_x ? A.zs : A.v;
  // the row tile's chunks; the first one's loads
  const int c_end = min(tm.chunks, (n - tm.row_begin + kRowsPerChunk - 1) / kRowsPerChunk);
  // a chunk: a float4 a thread of each whole group of 16 columns (row tid / 4),
  // one of a four of columns left (row tid % 128), the label of row tid
  static_assert(4 * kRowsPerChunk == kWdT, "a group of 16 columns is a float4 a thread");
  const int kc = A.kc, fg = kc >> 4, pq = (kc & 15) >> 2;       // uniform
  const int pr = tid & (kRowsPerChunk - 1), pi = tid >> 7;      // row and four of the columns left
  floatx4 buf[NT], left;
  int label = -1;
  // the wave's rows 16 w + l16 of the chunk, accounts 4 q4 + r
  float d_n = 1.f, sv_n[4] = {}, mu_n[4] = {};
  uint32_t ew_n[4] = {}, hw_n[4] = {};
  int hp_n[4] = {};
  auto fetch = [&](int ch) {
    const int row0 = tm.row_begin + ch * kRowsPerChunk;
    const floatx4* g = reinterpret_cast<const floatx4*>(A.Bp) + (size_t)row0 * (kc >> 2);
#pragma unroll
    for (int u = 0; u < NT; ++u)
      if (u < fg) buf[u] = g[u * kWdT + tid];
    // (threads without one read the first: no branch around a load in flight)
    left = g[pi < pq ? fg * kWdT + tid : 0];
    if (A.group) label = A.group[min(row0 + pr, n - 1)];         // uniform
    const int rc = min(row0 + 16 * w + l16, n - 1);
    d_n = A.d[rc];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r >= rounds) break;                                   // uniform
      const int a = max(Aid[4 * q4 + r], 0);                    // (an empty slot reads account 0)
      const size_t off = (size_t)a * n + rc, wi = (size_t)a * A.W + (rc >> 5);
      sv_n[r] = src[off];
      mu_n[r] = A.mu[off];
      ew_n[r] = A.elig ? A.elig[wi] : 0xffffffffu;
      hw_n[r] = A.hold[wi];
      hp_n[r] = A.hold_pre[wi];
    }
  };
  // the columns not in memory: bands from the labels as chunks pass, the column
  // of ones (rows past n have R' = 0 and no output)
  if (kc < kp)
    for (int e = tid; e < kRowsPerChunk * (kp - kc); e += kWdT) {
      const int col = kc + e % (kp - kc);
      Bs[e / (kp - kc) * S + wide_pos(col)] = col == A.one ? 1.f : 0.f;
    }
  int hot = -1;                             // row tid's one, from the last chunk
  if (c_end > 0) fetch(0);
  for (int ch = 0; ch < c_end; ++ch) {
    const int r0 = tm.row_begin + ch * kRowsPerChunk;
    __syncthreads();                                            // the last chunk's reads are done
#pragma unroll
    for (int u = 0; u < NT; ++u)
      if (u < fg) *reinterpret_cast<floatx4*>(Bs + (tid >> 2) * S + 16 * u + 4 * (tid & 3)) = buf[u];
    if (pi < pq) {
      float* b = Bs + pr * S + 16 * fg + pi;
      b[0] = left.x; b[4] = left.y; b[8] = left.z; b[12] = left.w;
    }
    if (kc < kp && tid < kRowsPerChunk) {
      float* b = Bs + tid * S;
      if (hot >= 0) b[hot] = 0.f;
      const int col = A.k + label;
      hot = label >= 0 && label < A.Gl && col >= kc ? wide_pos(col) : -1;
      if (hot >= 0) b[hot] = 1.f;
    }
    __syncthreads();
    // ---- back-projection and prox step: rows 16 w + l16, accounts 4 q4 + r
    const int row = r0 + 16 * w + l16;
    const bool row_ok = row < n;
    const float d_i = row_ok ? d_n : 1.f;
    float sv[4], mu[4];
    uint32_t ew[4], hw[4];
    int hp[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sv[r] = sv_n[r]; mu[r] = mu_n[r]; ew[r] = ew_n[r]; hw[r] = hw_n[r]; hp[r] = hp_n[r];
    }
    if (ch + 1 < c_end) fetch(ch + 1);
    floatx4 X;
#pragma unroll
    for (int r = 0; r < 4; ++r) X[r] = 0.f;
    if (do_x) {
      const float* bs = Bs + (16 * w + l16) * S + 4 * q4;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const floatx4 b = *reinterpret_cast<const floatx4*>(bs + 16 * t);
        X = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * t], b.x, X, 0, 0, 0);
        X = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * t + 1], b.y, X, 0, 0, 0);
        X = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * t + 2], b.z, X, 0, 0, 0);
        X = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * t + 3], b.w, X, 0, 0, 0);
      }
    }
    float Rp[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 4 * q4 + r, a = Aid[m];
      Rp[r] = 0.f;
      if (r < rounds && a >= 0 && row_ok) {
        const float4 c0 = Acc[2 * m], c1 = Acc[2 * m + 1];
        const float rho = c0.x, gam = c0.z, alpha = c1.w;
        float v = sv[r];
        const float iDelta = __builtin_amdgcn_rcpf(gam * d_i + rho);
        if (do_x) v = sv[r] + alpha * iDelta * (c1.z - X[r]);
        const size_t off = (size_t)a * n + row;
        const RowInfo ri = row_info_w(A, off, row, c1.x, c1.y, ew[r], hw[r], hp[r], Hp[m]);
        const float z = prox_row(ri, v, c0.w, c0.y, nullptr);
        if (do_p) {
          const float u = v - z;
          const float Rv = (mu[r] + rho * (z - u)) * iDelta;
          A.zs[off] = v + alpha * (Rv - z);
          Rp[r] = Rv;
        } else {
          A.v[off] = v;
          A.zs[off] = z;
        }
      }
    }
    if (!do_p) continue;                                        // uniform
    *reinterpret_cast<float4*>(Rs + (16 * w + l16) * kWdAcc + 4 * q4) =
        make_float4(Rp[0], Rp[1], Rp[2], Rp[3]);
    __syncthreads();
    // ---- contraction: strip w / 2, column tiles (w % 2) NH ...
    const int strip = 32 * (w >> 1), ct = (w & 1) * NH;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int rr = strip + 4 * s + q4;
      const float av = Rs[rr * kWdAcc + l16];
#pragma unroll
      for (int c = 0; c < NH; ++c)
        T[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(
            av, Bs[rr * S + 16 * (ct + c) + 4 * (l16 & 3) + (l16 >> 2)], T[c], 0, 0, 0);
    }
  }
  if (!do_p) return;
  __syncthreads();                                              // all waves are done with Bs
  float* red = Bs;                                              // [4][16][kp]
#pragma unroll
  for (int c = 0; c < NH; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      red[((w >> 1) * kWdAcc + 4 * q4 + r) * kp + 16 * ((w & 1) * NH + c) + l16] = T[c][r];
  __syncthreads();
  for (int e = tid; e < kWdAcc * kp; e += kWdT) {
    const int m = e / kp, c = e % kp;
    const int a = Aid[m];
    if (a < 0) continue;
    const float s = red[(0 * kWdAcc + m) * kp + c] + red[(1 * kWdAcc + m) * kp + c] +
                    red[(2 * kWdAcc + m) * kp + c] + red[(3 * kWdAcc + m) * kp + c];
    A.part[((size_t)tm.rt * A.m_total + a) * kp + c] = s;
  }
}

int wide_columns(int k, int kp, int H) { return wide_cols(k, kp, H); }

// Which books: no account has a turnover cap (its search needs every row
// between the two products), the accounts fit one MFMA tile, and the
// contractions are the float32 ones (the bf16-split passes sum in another
// order).  Below about 8,000 rows a workgroup's fill and drain outweigh the
// launches saved.
bool wide_fits(int n, int kp, int m, int ncap, bool split) {
  return !split && ncap == 0 && m <= kWdAcc && n >= 8192 && kp >= 64;
}

template <int NT>
static hipError_t launch_wide_t(const WideArgs& A, int nblk, int do_x, int do_p, hipStream_t st) {
  constexpr size_t smem = sizeof(float) * ((size_t)kRowsPerChunk * (16 * NT + 4) +
                                           kRowsPerChunk * kWdAcc + 8 * kWdAcc) +
                          2 * sizeof(int) * kWdAcc;
  hipError_t e = hipFuncSetAttribute((const void*)wide_kernel<NT>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((wide_kernel<NT>), dim3(nblk), dim3(kWdT), smem, st, A, do_x, do_p);
  return hipGetLastError();
}

hipError_t launch_wide(const WideArgs& A, int nblk, int do_x, int do_p, hipStream_t st) {
  switch (A.kp) {
    case 64: return launch_wide_t<4>(A, nblk, do_x, do_p, st);
    case 96: return launch_wide_t<6>(A, nblk, do_x, do_p, st);
    case 128: return launch_wide_t<8>(A, nblk, do_x, do_p, st);
    case 160: return launch_wide_t<10>(A, nblk, do_x, do_p, st);
    case 192: return launch_wide_t<12>(A, nblk, do_x, do_p, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_wide_setup(int n, int k, int kp, int H, const float* Bt, float* Bp,
                             hipStream_t st) {
  const int npad = ((n + kRowsPerChunk - 1) / kRowsPerChunk) * kRowsPerChunk;
  const int kc = wide_cols(k, kp, H);
  const size_t total = (size_t)npad * kc;
  const unsigned blocks = (unsigned)((total + 255) / 256 < 8192 ? (total + 255) / 256 : 8192);
  hipLaunchKernelGGL(wide_perm_kernel, dim3(blocks), dim3(256), 0, st, n, npad, kp, kc, Bt, Bp);
  return hipGetLastError();
}

}  // namespace fqp
