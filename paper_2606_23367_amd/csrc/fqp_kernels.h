// Kernel argument blocks and launchers (internal to libfqp).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fqp_common.h"

namespace fqp {

struct IterArgs {
  int n, W;                  // assets, bitmask words per account
  int m_total;               // accounts in the book (partials are indexed by id)
  const int* m_act;          // device: number of active accounts
  const int* act;            // device: active account ids [m_act]
  const float* Bt;           // [n][kp]
  const float* d;            // [n]
  const float* mu;           // [m][n]
  float* v;                  // [m][n]  ADMM state v = xh + u
  const uint32_t* elig;      // [m][W] or null
  const uint32_t* hold;      // [m][W]
  const int32_t* hold_pre;   // [m][W]
  const int32_t* hold_ptr;   // [m+1]
  const float* hold_w0;      // [nnz_h]
  const int32_t* hold_tax;   // [nnz_h]
  const float* tax_brk;      // [nnz_t][3]
  const float* tax_slope;    // [nnz_t][4]
  const float4* hold_rec;    // [nnz_h][2]: {w0, b1, b2, b3}, {s0, s1, s2, s3}; b1 < 0: no lots
  int npad;                  // rows of the bf16 copies of B~ (n padded to whole chunks)
  const uint16_t* bt_hi;     // npad x kp bf16 hi part of B~, PROJECT operand order
  const uint16_t* bt_lo;     // its lo part
  const uint16_t* btt_hi;    // npad x kp bf16 hi part of B~, CONTRACT operand order
  const uint16_t* btt_lo;    // its lo part
  const float* pp;           // [m][kp]
  const float* par;          // [m][kNPar]
  float* par_rw;             // same array, written by the cap kernel
  float* part;               // [row tiles][m][kp] (at most one per 128-row chunk)
  const float* lbv;          // [m][n] per-asset bounds, or null (the
  const float* ubv;          //   account's scalars P_LB / P_UB)
  float* zs;                 // [m][n] w = v + alpha (Delta^-1 r - z) of the
                             // current iterate: PROX writes it, PROJECT adds
                             // the back-projection; before a polish it holds
                             // z = prox(v; lam*) instead (PROX in z mode)
  float* rp;                 // [m][npad] R' = r / Delta of the current iterate
                             // (PROX writes rows < n, CONTRACT reads it)
};

struct KArgs {
  int kp, k, G, n, nblk, m_total;    // nblk: workgroups of the CONTRACT pass
  int nblk_p;                        // workgroups of the PROJECT pass
  int ncls;                          // gamma classes (1: no per-account class lookup)
  const int* m_act;
  const int* act;
  const float* part;
  float* par;                // [m][kNPar]
  float* pp;                 // [m][kp]
  const float* Kinv;         // [ncls][kp][kp]
  const float* cvec;         // [ncls][kp]
  const float* qvec;         // [ncls][kp]
  const float* sig1;         // [ncls]
  const float* mbg;          // [ncls][kp][G]
  float* zb;                 // [m][G]
  float* vb;                 // [m][G]
  const float* blo;          // [m][G]
  const float* bhi;          // [m][G]
  int* iters;                // [m]
};

// Work split of the two iteration passes for the current number of active
// accounts: the grid's workgroups are spread over the active 32-account
// tiles, and each tile's rows are cut into as many row tiles as it gets
// workgroups (whole 128-row chunks), so a short active list still fills the
// chip.  The k-space solve uses the same split to find the partials.
struct TileMap {
  int tile, rt, n_rt, chunks, row_begin;
  bool active;
};
__device__ __forceinline__ TileMap tile_map(int m_act, int n, int nblk, int lin) {
  const int tiles = (m_act + kTM - 1) / kTM;
  const int total_chunks = (n + kRowsPerChunk - 1) / kRowsPerChunk;
  int r = tiles > 0 ? nblk / tiles : 1;
  r = r < 1 ? 1 : (r > total_chunks ? total_chunks : r);
  const int cpt = (total_chunks + r - 1) / r;        // chunks per row tile
  TileMap t;
  t.n_rt = (total_chunks + cpt - 1) / cpt;
  t.chunks = cpt;
  t.tile = lin / t.n_rt;
  t.rt = lin % t.n_rt;
  t.row_begin = t.rt * cpt * kRowsPerChunk;
  t.active = t.tile < tiles;
  return t;
}

hipError_t configure_iter_kernels();
// workgroups of one iteration pass (mode) resident on one compute unit at
// once; 0 if the runtime cannot tell
int iter_blocks_per_cu(int kp, int prec, int mode);
// ev0 / ev1 (optional): events stamped at the start and the end of the
// kernel's own execution (not of the queue around it)
hipError_t launch_iter(const IterArgs& A, int kp, int mode, int prec, dim3 grid,
                       hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t launch_split_bt(int n, int npad, int kp, const float* Bt, uint16_t* bh, uint16_t* bl,
                           uint16_t* bth, uint16_t* btl, hipStream_t st);
// the per-account PROX pass (cap multiplier, then R' and w; zmode: z): the
// register-resident layout needs n <= 16384, at most 2048 held rows in
// every account and no per-asset bounds
bool cap_resident_fits(int n, int max_held);
hipError_t launch_prox(const IterArgs& A, int m_total, bool resident, int zmode,
                       hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
hipError_t launch_ksolve(const KArgs& A, int m_total, hipStream_t st);
// Bq: [ceil(k / 4)][n] float4, the first k columns by fours
hipError_t launch_build_bt(int n, int k, int G, int H, int kp, const float* B,
                           const int32_t* group, const float* half, float* Bt, float* Bq,
                           hipStream_t st);
hipError_t launch_gram(int n, int kp, int kg, int nparts, int rows_per_blk, const float* Bt,
                       const float* d, double gamma, double rho, double* part, hipStream_t st);
hipError_t launch_kfactor(int k, int G, int kp, int nparts, const double* part, const float* f,
                          double gamma, double rho_b, double* Kw, float* Kinv, float* c,
                          float* q, float* sig, float* mbg, hipStream_t st);

// ---- account-resident iterations -------------------------------------------
// the trade lines and lot indices of every row, [m][npr] (npr: rows padded
// to whole 64-row tiles)
struct ResRowArgs {
  int n, npr, W, m;
  const float* mu;
  const float* lb;
  const float* ub;
  const float* lbv;          // [m][n] per-asset bounds or null
  const float* ubv;
  const uint32_t* elig;
  const uint32_t* hold;
  const int32_t* hold_pre;
  const int32_t* hold_ptr;
  const float4* hold_rec;
  float4* rows;              // [m][npr] out: {mu, w0, lb, ub}
  int32_t* lot;              // [m][npr] out: lot record or -1; null without tax
};

struct ResArgs {
  int n, npr, ntile, k, G, kp, ncls;
  const int* m_act;
  const int* act;
  const float4* Bq;          // B~ in tile order (fqp_resident.hip)
  const float4* rows;
  const int32_t* lot;
  const float4* hold_rec;
  const float* d;
  float* v;                  // [m][n] ADMM state
  float* zs;                 // [m][n] z of the state a block ends with
  float* par;
  const float* Kinv;
  const float* cvec;
  const float* qvec;
  const float* sig1;
  const float* mbg;
  float* zb;
  float* vb;
  const float* blo;
  const float* bhi;
  int* iters;
};
// quarter of the padded factor width the resident kernel is compiled for
int resident_kq(int kw);
// whether a book of m accounts runs its blocks account-resident: kw = used
// columns of B~, ncap = accounts with a turnover cap, max_held = the most names
// one account holds, asset_box: per-asset bounds, split: the passes' contractions
// are the bf16-split ones
bool resident_fits(int n, int kw, int G, bool lots, int m, int ncap, int max_held, bool asset_box,
                   bool split, int n_cu);
hipError_t launch_resident_setup(const ResRowArgs& A, int kp, int KQ, const float* Bt, float4* Bq,
                                 hipStream_t st);
hipError_t launch_resident(const ResArgs& A, int KQ, int m_total, int count, hipStream_t st);

// ---- fused pass of wide books (fqp_wide.hip) -----------------------------------
struct WideArgs {
  int n, W, k, kp, m_total;
  int kc, Gl, one;           // columns of B~ in Bp (wide_cols), bands, the column of ones
  const int32_t* group;      // [n] labels (with bands)
  const int* m_act;
  const int* act;
  const float* Bp;           // the columns in memory, by 128-row chunks (wide_perm_kernel)
  const float* d;
  const float* mu;
  const float* lbv;          // [m][n] per-asset bounds or null
  const float* ubv;
  const uint32_t* elig;
  const uint32_t* hold;
  const int32_t* hold_pre;
  const int32_t* hold_ptr;
  const float4* hold_rec;
  const float* pp;           // [m][kp]
  const float* par;
  float* v;                  // [m][n]
  float* zs;                 // [m][n] w between the launches of a block, z after it
  float* part;               // [row tiles][m][kp]
};
bool wide_fits(int n, int kp, int m, int ncap, bool split);
int wide_columns(int k, int kp, int H);
hipError_t launch_wide_setup(int n, int k, int kp, int H, const float* Bt, float* Bp,
                             hipStream_t st);
// one launch of an iteration block over nblk row tiles: do_x applies the last
// factor-space solve, do_p takes the prox step and contracts (else v and z
// are written)
hipError_t launch_wide(const WideArgs& A, int nblk, int do_x, int do_p, hipStream_t st);

// ---- packing / validation -------------------------------------------------
struct PackArgs {
  int n, W, m, G;            // G: constraint rows (bands, then halfspaces)
  int Gl;                    // band rows (finite bounds required)
  const float* lbv;          // [m][n] per-asset bounds or null
  const float* ubv;
  const float* eta;          // [m] or null
  const float* mu;
  const float* w0;
  const float* lb;
  const float* ub;
  const uint32_t* elig;
  const float* gamma;
  const float* kappa;
  const float* tau;
  const float* blo;
  const float* bhi;
  const int32_t* tax_ptr;
  const int32_t* tax_asset;
  const float* tax_brk;
  const float* tax_slope;
  // outputs
  uint32_t* hold;
  int32_t* hold_pre;
  int32_t* hold_cnt;        // [m]
  int32_t* hold_ptr;        // [m+2]: prefix [m+1], then the largest count
  float* hold_w0;
  int32_t* hold_tax;
  int32_t* status;          // [m]
  float* par;               // [m][kNPar]
  // pinned host memory (device address) or null: [0] the total of held names,
  // [1] the most held names of one account, [4] the accounts with a finite
  // turnover cap, stored by the scan
  int32_t* host_counts;
};
hipError_t launch_pack_count(const PackArgs& A, hipStream_t st);
hipError_t launch_pack_scan(const PackArgs& A, hipStream_t st);
hipError_t launch_pack_fill(const PackArgs& A, hipStream_t st);
hipError_t launch_pack_rec(const PackArgs& A, float4* rec, int total, hipStream_t st);

// ---- polish / certification (float64) -------------------------------------
// ints of polish bookkeeping per account
constexpr int kPStateStride = 16;

struct PolishArgs {
  int n, k, G, kp, W, m_total;  // G: constraint rows, bands then halfspaces
  int Gl;                    // band rows, one-hot by label; rows Gl..G-1 are
                             // the halfspace columns k + Gl.. of B~
  const float* lbv;          // [m][n] per-asset bounds or null
  const float* ubv;
  const double* obj_const;   // [m] (gamma/2) w_b^T Sigma w_b, or null
  const double* mu64;        // [m][n] mu' = eta mu + gamma Sigma w_b in float64
                             // (with a benchmark or eta; mu holds it in float32)
  const int* m_act;
  const int* act;
  const float* Bt;           // [n][kp] (first k columns = B)
  const float* f;            // [k]
  const float* d;            // [n]
  const int32_t* group;      // [n] or null
  const float4* Bq;          // [ceil(k / 4)][n] the factor columns by fours
  const float* half;         // [G - Gl][n] halfspace rows or null
  const float* mu;           // [m][n]
  const float* z;            // [m][n]  ADMM iterate
  const uint32_t* elig;
  const uint32_t* hold;
  const int32_t* hold_pre;
  const float4* hold_rec;    // [nnz_h][2] packed held records (as IterArgs)
  const int32_t* hold_ptr;
  const float* hold_w0;
  const int32_t* hold_tax;
  const float* tax_brk;
  const float* tax_slope;
  const float* par;          // [m][kNPar]
  const float* zb;           // [m][G] ADMM band state
  const float* vb;           // [m][G] ADMM band scaled duals
  const float* blo;
  const float* bhi;
  int8_t* code;              // [m][n] active-set codes
  int8_t* code_next;         // [m][n] refinement proposals
  int32_t* flist;            // [m][n] free list
  double* wk;                // [m][wk_stride] per-account scratch
  size_t wk_stride;
  double* wout;              // [m][n] polished weights (caller output)
  double* gbase;             // [m][n] gamma (Sigma w)_i - mu_i of the pattern
  double* mult;              // [m][2 + G] nu, lam_cap, lam_band
  int32_t* pstate;           // [m][kPStateStride] polish bookkeeping
  double eps_prim, eps_dual, eps_comp;
  int first_round;           // classify from z when nonzero
  int nf_gate;               // skip patterns with more free rows (0: never)
  int nf_small;              // larger free sets wait for a repeated pattern
  int* pcount;               // [2] reduced solves formed, attempts gated
  int max_prop;              // a failed pattern with more proposals stops refining
  int n_rb;                  // row blocks of the gradient-base pass
  double* gpart;             // [m][n_rb][4] its per-block reductions
  int n_sb;                  // row blocks of the other row passes
  int32_t* fseg;             // [m][n] per-block free / nonzero fixed rows
  double* rpart;             // [m][n_sb][polish_rpart_stride] pattern partials
  double* spart;             // [m][n_sb][4] null-direction sweep partials
  double* cpart;             // [m][n_sb][8] diagnostic partials
};
// whether one workgroup per account runs a pass's rounds (launch_polish_pass)
bool polish_pass_fits(int n, int k, int G);
hipError_t launch_polish_solve(const PolishArgs& A, hipStream_t st);
// pact / pm_act: the accounts of act / m_act that neither certified nor stalled;
// host_count (pinned host memory, device address, or null) also receives the count
hipError_t launch_polish_list(const int* m_act, const int* act, const int32_t* pstate, int* pact,
                              int* pm_act, int* host_count, hipStream_t st);
size_t polish_wk_stride(int k, int G);
int polish_row_blocks(int n);
int polish_pass_blocks(int n);
int polish_rpart_stride(int k, int G);

// ---- KKT adjoint (float64) ---------------------------------------------------
struct AdjArgs {
  int n, k, G, kp, m;        // G: constraint rows (as PolishArgs)
  int Gl;
  const float* wb;           // [m][n] benchmark weights or null
  const float* eta;          // [m] return scale or null
  const double* ywb;         // [m][k] B^T w_b (with wb)
  const float* Bt;
  const float* f;
  const float* d;
  const int32_t* group;
  const float* w0in;         // [m][n] caller's w0
  const float* par;
  const int32_t* status;     // [m] statuses of the last solve
  const int32_t* pstate;
  const int32_t* flist;
  const int8_t* code;
  const double* w;           // [m][n] weights of the last solve
  const double* dLdw;        // [m][n]
  double* dmu;               // [m][n] out
  double* dB;                // [n][k] out
  double* yvw;               // [m][2k] scratch
  double* wk;
  size_t wk_stride;
};
hipError_t launch_adjoint(const AdjArgs& A, hipStream_t st);

// ---- the rest of Eq. 1 -------------------------------------------------------
// box of (account a, asset i) of an eligible asset: the per-asset bounds
// when the book has them, else the account's scalars (excluded: [0, 0])
template <typename Args>
__device__ __forceinline__ void asset_box(const Args& A, size_t off, bool el, float lbp,
                                          float ubp, float& lb, float& ub) {
  if (!el) { lb = 0.f; ub = 0.f; return; }
  lb = A.lbv ? A.lbv[off] : lbp;
  ub = A.ubv ? A.ubv[off] : ubp;
}

struct RowInfo {
  float lb, ub, w0;
  bool taxed;
  TaxLots t;
};

__device__ __forceinline__ float prox_row(const RowInfo& ri, float v, float th, float irho,
                                          bool* at_kink) {
  float zn;
  if (ri.taxed) {
    zn = prox_taxed(v, ri.w0, th, irho, ri.t, ri.lb, ri.ub);
    if (at_kink)
      *at_kink = (zn == ri.w0) || (zn == ri.w0 - ri.t.b1) || (zn == ri.w0 - ri.t.b2) ||
                 (zn == ri.w0 - ri.t.b3) || zn <= ri.lb || zn >= ri.ub;
  } else {
    zn = prox_plain(v, ri.w0, th, ri.lb, ri.ub);
    if (at_kink) *at_kink = (zn == ri.w0) || zn <= ri.lb || zn >= ri.ub;
  }
  return zn;
}

// box, w0 and tax lots of (account a, row) from its eligibility word, its
// holding word and the holding prefix word (already loaded) and the
// account's first record hptr: one more dependent load, only for held rows
template <typename Args>
__device__ __forceinline__ RowInfo row_info_w(const Args& A, size_t off, int row, float lbp,
                                              float ubp, uint32_t ew, uint32_t hw, int hpre,
                                              int hptr) {
  RowInfo ri;
  const int b = row & 31;
  const bool el = (ew >> b) & 1u;
  asset_box(A, off, el, lbp, ubp, ri.lb, ri.ub);
  ri.w0 = 0.f;
  ri.taxed = false;
  if ((hw >> b) & 1u) {
    const int idx = hptr + hpre + popc_below(hw, b);
    const float4 r0 = A.hold_rec[2 * idx], r1 = A.hold_rec[2 * idx + 1];
    ri.w0 = r0.x;
    ri.taxed = r0.y > 0.f;
    ri.t.b1 = r0.y; ri.t.b2 = r0.z; ri.t.b3 = r0.w;
    ri.t.s0 = r1.x; ri.t.s1 = r1.y; ri.t.s2 = r1.z; ri.t.s3 = r1.w;
  }
  return ri;
}

// the linear term of the polish and certificate: mu' in float64 when the
// book has a benchmark term, else the caller's mu
__device__ __forceinline__ double mu_at(const PolishArgs& A, size_t off) {
  return A.mu64 ? A.mu64[off] : (double)A.mu[off];
}

// coefficient of constraint row g at asset i: band rows (g < Gl) are
// one-hot by label, halfspace rows are the columns k + g of B~
template <typename Args>
__device__ __forceinline__ double row_coef(const Args& A, int i, int g) {
  return g < A.Gl ? (A.group[i] == g ? 1.0 : 0.0) : (double)A.Bt[(size_t)i * A.kp + A.k + g];
}

// mu' = eta mu + gamma Sigma w_b and (gamma/2) w_b^T Sigma w_b per account
// (the benchmark term of Eq. 1 expanded)
hipError_t launch_benchmark_prep(int m, int n, int k, const float* B, const float* f,
                                 const float* d, const float* mu, const float* wb,
                                 const float* eta, const float* gamma, double* ywb,
                                 double* part, float* mu_out, double* mu64_out,
                                 double* obj_const, hipStream_t st);
int benchmark_row_blocks(int n);
// the band bounds then the halfspace bounds, [m][G + H]
hipError_t launch_concat_rows(int m, int G, int H, const float* blo, const float* bhi,
                              const float* hlo, const float* hhi, float* lo, float* hi,
                              hipStream_t st);

}  // namespace fqp
