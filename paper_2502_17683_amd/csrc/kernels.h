// Internal launchers shared by the translation units of libthccp.so.
// Not part of the public C-ABI (include/thccp.h).
//
// Every kernel of the sweep is "grouped": one launch serves a table of
// independent problems (the CPDs of a batch; a single CPD is a group of
// one).  Argument tables live in device memory (the plan's workspace);
// `offs` tables hold the prefix sums of each problem's workgroup count.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "common.h"

namespace thccp {

// ---------------------------------------------------------------- GEMM
// C[M x N] = alpha * op(A)[M x K] * op(B)[K x N] + beta * C, row-major C.
//   a_t = false: A[i*lda + k];  a_t = true: A[k*lda + i]   (A stored K x M)
//   b_t = false: B[k*ldb + j];  b_t = true: B[j*ldb + k]   (B stored N x K)
//   B2 != nullptr: every B element is B1[.] * B2[.] (single products only).
//   C2 != nullptr: the result is also written to C2 (same ldc).
//   done != nullptr: the problem is skipped once *done is set.
//   gate != nullptr: the problem is skipped unless *gate == want (per-problem
//   choice between the split-BF16 and the FP64 path).
//   lower != 0: tiles strictly above the diagonal are skipped (C is only
//   needed on and below it, as in a symmetric rank-k update); for square
//   C only the lower tiles are launched (see gemm_tile_count).
//   P1 != nullptr: P1 = C o H1 as well (ldc; H1 == C: the square), P2
//   likewise with H2: the pair operand of a later product, formed while C
//   is in registers.
//   slices > 1: tiles at or past nfull are split over K (gemm_plan_slices);
//   part: their partial tiles, cnt: one zeroed counter each.
//   vec: C, C2, H and P take 16-byte accesses.
template <typename T>
struct GemmArgs {
  int M, N, K;
  const T* A; int lda;
  const T* B1; const T* B2; int ldb;
  T* C; int ldc; T* C2;
  T alpha, beta;
  const int32_t* done;
  const int32_t* gate = nullptr;
  int32_t want = 0;
  int32_t lower = 0;
  const T* H1 = nullptr; T* P1 = nullptr;
  const T* H2 = nullptr; T* P2 = nullptr;
  int32_t nfull = 0, slices = 1;
  void* part = nullptr;
  int32_t* cnt = nullptr;
  int32_t vec = 0;
  int32_t kdiag = 0;   // op(B) is zero above row n0 of column block n0 / 64: K starts there
  int32_t mirror = 0;  // with lower and op(A) = A^T: C is symmetric, and its upper tiles are stored as well
};
struct GemmF64 {
  int M, N, K;
  const double* A; int lda; bool a_t;
  const double* B1; const double* B2; int ldb; bool b_t;
  double* C; int ldc;
  double alpha, beta;
};
struct GemmF32 {
  int M, N, K;
  const float* A; int lda; bool a_t;
  const float* B1; const float* B2; int ldb; bool b_t;
  float* C; int ldc;
  float alpha, beta;
};
void gemm_f64(hipStream_t s, const GemmF64& g);
void gemm_f32(hipStream_t s, const GemmF32& g);
// C = X^T X (n x n, X stored K x n): the lower tiles are computed and stored
// on both sides, which gives the bits of the whole product.
void syrk_f64(hipStream_t s, int n, int K, const double* X, int ld, double* C, int ldc);
// Two independent products, op(A) = A^T of the first and op(B) = B^T of the
// second, side by side where their shapes allow it.
void gemm_f32_two(hipStream_t s, const GemmF32& g, const GemmF32& h);
// Tiles of one GEMM; a lower-triangle GEMM (lower != 0, square) launches
// only the T (T + 1) / 2 tiles on and below the diagonal.
inline int gemm_tile_count(int M, int N, int bm, int lower = 0) {
  const int tm = (M + bm - 1) / bm, tn = (N + bm - 1) / bm;
  return lower && M == N ? tm * (tm + 1) / 2 : tm * tn;
}
// First k of slice z of `slices` (multiples of 32, so that every tile form
// cuts K at the same places).
__host__ __device__ inline int gemm_slice_k(int K, int slices, int z) {
  const long b = (K + 31) / 32;
  const int k = (int)(b * z / slices) * 32;
  return k < K ? k : K;
}
// Whether the direct-load tiles can take this product: 16-byte aligned
// operands whose leading dimensions, and K where an operand is contiguous
// along k, are multiples of a 16-byte chunk.
template <typename T>
bool gemm_tile_ok(const GemmArgs<T>& g, bool a_t, bool b_t);
// Chooses nfull and slices of a product of a plan (part and cnt are the
// caller's: (tiles - nfull) slices bm^2 elements and tiles - nfull zeroed
// counters).
template <typename T>
void gemm_plan_slices(GemmArgs<T>& g);
// Workgroups of a product in tile form bm.
template <typename T>
int gemm_units(const GemmArgs<T>& g, int bm);
// Tile form (32, 64 or 128) of a grouped launch.
template <typename T>
int gemm_tile_form(const std::vector<GemmArgs<T>>& v);
// Tests: forces the tile form of products prepared afterwards, wherever it
// is one of the product's own (0: the rule and the autotuner decide);
// returns the previous value.
int set_tile_force(int bm);
int get_tile_force();
// Grouped launch: tab[nprob] products with identical (a_t, b_t) flags, all
// of them gemm_tile_ok, in tile form bm; offs[nprob + 1] prefix sums of
// gemm_units.
template <typename T>
void gemm_group(hipStream_t s, const GemmArgs<T>* tab, const int* offs, int nprob, int units, bool a_t, bool b_t,
                int bm);
// Whether C and its companions take 16-byte accesses (sets g.vec).
template <typename T>
void gemm_set_vec(GemmArgs<T>& g);

// -------------------------------------------------- Cholesky / triangular solve
// One problem of the blocked factorisation and row solves.  V: Tp x Tp
// row-major (Tp = 64 nblk); the diagonal blocks of L go to ldiag (nblk
// 64 x 64 blocks), the diagonal of L to diagL; M: n x Tp right-hand sides.
template <typename T>
struct StepProb {
  T* V;
  T* ldiag;
  T* diagL;
  T* M;
  DevState* st;
  int nblk;
  int n;
  int32_t* flow;   // ready flags of the dataflow solves, ceil(n / 64) x nblk
  int32_t* cflow;  // ready flags of the dataflow factorisation, nblk^2 + 2 nblk,
                   // then CU_SLOTS per-compute-unit counters
  T* dpart;        // diagonal blocks updated through column k - 2, nblk x 64 x 64
  int32_t* bflow;  // ready flags of the dataflow backward solve, ceil(n / 64) x nblk
  // Inverse form (null: off): the forward solve also takes the rows of the
  // identity, whose solution L^{-T} goes to the upper blocks of E (Tp x Tp,
  // zero below), and the backward solve F = G L^{-1} is one product.
  T* E = nullptr;
  // The Grams whose Hadamard product is V, R x R (null: V is formed already):
  // the dataflow factorisation multiplies them as it loads its tiles.
  const T *g0 = nullptr, *g1 = nullptr, *g2 = nullptr;
  int R = 0;
};
// Per-compute-unit counters of the dataflow factorisation (an XCC, shader
// engine, shader array and CU index from the hardware id registers).
constexpr int CU_SLOTS = 2048;
enum StepMode {
  STEP_CHOL = 0,
  STEP_FWD = 1,
  STEP_BWD = 2,
  STEP_CHOL_FWD = 3,
  STEP_FLOW_RESET = 4,     // clears the backward solve's ready flags (one workgroup per problem)
  STEP_BWD_FLOW = 5,       // the whole one-level backward solve as one dataflow launch
  STEP_CFLOW_RESET = 6,    // clears the ready flags of the factorisation and of both solves
  STEP_CHOL_FWD_FLOW = 7,  // one-level factorisation + forward solve as one dataflow launch
  STEP_BWD_PREP = 8,       // per pair of block columns, the products of L the paired solve needs
  STEP_BWD_PAIR = 9        // the one-level backward solve as one dataflow launch, in block pairs
};

// Two-level blocking: the 64-wide block columns are grouped into panels of
// pw blocks.  Inside a panel the step kernel works one block column per
// launch (panel-local updates only); after a panel, one grouped GEMM applies
// its rank-(64 pw) update to everything right of it (factorisation, forward
// solve) or left of it (backward solve).  pw >= nblk is the one-level form:
// every step updates the whole trailing matrix.
// One step launch: factorisation step tc of panel pc and solve step tf of
// panel pf (a negative panel or step: none).  Factorisation step t of panel
// p updates the panel's remaining block columns with block column
// pw p - 1 + t (when inside the panel) and factors block column pw p + t;
// forward step t likewise for the right-hand sides; backward step t solves
// block column b1 - t of the panel (b1 its last block) after updating the
// panel's columns left of it.
struct StepCfg {
  int pw;
  int pc, tc;
  int pf, tf;
  int strip = 0;  // STEP_CHOL_FWD_FLOW in FP64: diagonal blocks by the strip factorisation
};
inline int panel_count(int nblk, int pw) { return (nblk + pw - 1) / pw; }
// Workgroups of problem (nblk, n) in a launch of `mode` with `cfg`.
int step_tiles(int mode, int nblk, int n, StepCfg cfg);
// Workgroup order of a grouped dataflow launch (STEP_CHOL_FWD_FLOW,
// STEP_BWD_FLOW, STEP_BWD_PAIR) over problems of nblk[p] blocks and n[p]
// rows: segments of one (problem, block column), block column by block
// column across the problems (ascending for the factorisation, from each
// problem's last column down for the backward solve), so every problem
// advances at the same pace and every wait is on a lower workgroup id.
// STEP_BWD_PAIR: segments of one (problem, pair of block columns), pairs
// from the last column down; per row tile the workgroup of the pair's upper
// block, then that of its lower block.  The one wait on a higher id is the
// upper block's wait for the lower block's first action (its right-hand
// side read), which waits on nothing.  inv[p]: the problem is in the
// inverse form.  Int triples (first workgroup, problem, column or pair),
// then (total workgroups, -1, -1).
std::vector<int> flow_segments(int mode, const std::vector<int>& nblk, const std::vector<int>& n,
                               const std::vector<char>& inv);
inline bool is_flow_mode(int mode) {
  return mode == STEP_CHOL_FWD_FLOW || mode == STEP_BWD_FLOW || mode == STEP_BWD_PAIR;
}
// Polls a dataflow wait makes before it gives up (negative: the default);
// returns the previous value.  Applies to launches enqueued afterwards.
int set_flow_spin_limit(int polls);
// Form of the one-level backward solve for schedules built afterwards:
// 0 (default) two block columns per dependency hop (STEP_BWD_PREP +
// STEP_BWD_PAIR), 1 one block column per hop (STEP_BWD_FLOW); returns the
// previous value.
int set_bwd_form(int form);
int get_bwd_form();
// Launches one step of `mode`.  offs: nprob + 1 prefix sums of the
// problems' workgroups, or for a dataflow mode the segment table, with
// nprob its segment count.
template <typename T>
void step_group(hipStream_t s, int mode, const StepProb<T>* probs, const int* offs, int nprob, int total_tiles,
                StepCfg cfg, int retry_pass);
// The panel update GEMM of panel p for one problem (false: none needed):
//   PG_SYRK  V[c0:, c0:] -= L[c0:, panel] L[c0:, panel]^T (lower tiles),
//   PG_FWD   M[:, c0:]   -= G[:, panel] L[c0:, panel]^T,
//   PG_BWD   M[:, :b0]   -= X[:, panel] L[panel, :b0],
// with c0 the first column after the panel and b0 its first column.  SYRK
// and FWD take (a_t, b_t) = (false, true), BWD (false, false).
enum PanelGemm { PG_SYRK = 0, PG_FWD = 1, PG_BWD = 2 };
template <typename T>
bool panel_gemm(int kind, const StepProb<T>& q, int pw, int p, GemmArgs<T>& g);

// Launch order of a blocked solve with panel width pw for problems of up
// to max_nblk blocks: step launches (mode >= 0) and panel GEMM launches
// (mode < 0, up to two PanelGemm kinds in one grouped launch).
//   SCHED_CHOL      factorisation: per panel, its steps, then its SYRK.
//   SCHED_CHOL_FWD  factorisation fused with the forward solve.  With
//                   panels, the latter runs one panel behind: the launches
//                   of panel p also run the forward steps of panel p - 1, and
//                   one GEMM launch holds the SYRK of panel p and the
//                   forward update of panel p - 1.  One-level (pw >=
//                   max_nblk): one block column behind.
//   SCHED_FWD       forward solve alone;  SCHED_BWD  backward solve (panels
//                   from the last one down; one level: a flag reset, then
//                   STEP_BWD_PREP and the dataflow launch STEP_BWD_PAIR, or
//                   the dataflow launch STEP_BWD_FLOW; set_bwd_form).
enum SolveSched { SCHED_CHOL = 0, SCHED_CHOL_FWD = 1, SCHED_FWD = 2, SCHED_BWD = 3 };
struct SolveItem {
  int mode;
  StepCfg cfg;
  int g_kind[2];
  int g_panel[2];
};
std::vector<SolveItem> solve_schedule(int sched, int max_nblk, int pw);

// ------------------------------------------------------------- element-wise
// The ready flags of a problem's dataflow solves.  Clear before a solve: the
// launch that closes one (normalise_group) clears them for the next.
struct FlowFlags {
  int32_t *flow, *cflow, *bflow;
  int nflow, ncflow;
};
template <typename T>
struct FormVArgs {
  T* V; const T* g0; const T* g1; const T* g2; DevState* st; int Tp; int R;
  FlowFlags flags;  // cleared beside V (the first pass only)
};
template <typename T>
void form_v_group(hipStream_t s, const FormVArgs<T>* tab, int nprob, int max_Tp, int retry_pass);
template <typename T>
void retry_prepare_group(hipStream_t s, const FormVArgs<T>* tab, int nprob, int allow_fallback);

template <typename T>
struct NormArgs {
  const T* Msol; T* F; T* lam; const T* Msave; double* inner_part; DevState* st; int n; int R; int ld;
  int from_F = 0;  // inverse form: the solution is in F already (normalised in place)
  FlowFlags flags;
};
// slow: the problems in the damped-retry pass have theirs in Msol all the same.
template <typename T>
void normalise_group(hipStream_t s, const NormArgs<T>* tab, int nprob, int max_R, int slow);
// Tied model: <G, G~> partials lam[k] sum_s F3[s,k] M3[s,k] (F3 passed as
// Msol, M3 as Msave; F unused).
template <typename T>
void tied_inner_group(hipStream_t s, const NormArgs<T>* tab, int nprob, int max_R);

template <typename T>
struct FitArgs {
  const T* g[4]; const T* lam; const double* inner_part; double* row_part; double* fit_hist; DevState* st;
  int R; int ld;
};
template <typename T>
void fit_group(hipStream_t s, const FitArgs<T>* tab, int nprob, int max_R, int hist_cap, double tol,
               double fit_floor, int guard, double cond_limit, int rule_every);
// Non-fit sweep of a split-BF16 plan: sweep counter and precision guard.
void sweep_tick_group(hipStream_t s, DevState* const* st_tab, int nprob, int guard, double cond_limit);
// Precision guard bookkeeping (split-BF16 plans):
//   cond_track: st->cond_max = max(st->cond_max, (max diagL / min diagL)^2)
//   after each mode's factorisation; guard_begin: reset at sweep start.
template <typename T>
struct CondArgs {
  const T* diagL; DevState* st; int R;
};
template <typename T>
void cond_track_group(hipStream_t s, const CondArgs<T>* tab, int nprob);
void guard_begin_group(hipStream_t s, DevState* const* st_tab, int nprob);
// Sets path = 1 (FP64) and clears promote for the listed problems.
void set_path_group(hipStream_t s, DevState* const* st_tab, int nprob, const int32_t* flags_dev);

// Factor checkpoint: copies (dir = 0) F -> Fsave and st -> st_save, or back.
struct CkptArgs {
  void* a[4];
  void* b[4];
  size_t bytes[4];
  DevState* st;
  DevState* st_save;
  const int32_t* gate;  // non-NULL: copy only while *gate == want
  int32_t want;
};
// Copies a[m] -> b[m] (dir 0) or back (dir 1), bytes[m] each, and the
// device state with them; with st or st_save NULL only the regions (the
// tied model's factor copies, the right-hand-side backups of the solve).
void checkpoint_group(hipStream_t s, const CkptArgs* tab, int nprob, int dir);

void hadamard_inplace_f64(hipStream_t s, double* A, const double* B, size_t count);
void transposed_dot_f64(hipStream_t s, const double* P, const double* Q, int R, int ld, double* partials,
                        double* out);
void fill_bytes(hipStream_t s, void* p, size_t bytes);
template <typename T>
void hadamard(hipStream_t s, const T* a, const T* b, T* out, size_t count);
template <typename T>
void copy_rows_f64(hipStream_t s, const double* src, int rows, int cols, T* dst, int ld);
void state_reset(hipStream_t s, DevState* st, double* norm2_src, double fit_target);
void cast_f64_to_f32(hipStream_t s, const double* a, float* b, size_t count);
void copy_normalised_init(hipStream_t s, const double* src, int n, int R, int ld, double* dst);
void lt_scale_rows(hipStream_t s, const double* X, const double* eps, int n, int r, double t, double sign,
                   double* out);

}  // namespace thccp
