// Learned warm start for CP-ALS (gfx950).
//
// With a diagonal core the THC form is already an exact CP decomposition
// whose columns are the grid columns X_m[:, P] (eq. THC), so an initial CP
// is built from R_cp selected grid columns, each scaled.  A three-layer
// network scores every grid point from eight features of (X0, Z, S) and
// predicts a log-scale; the top-R_cp grid points by score become the
// initial factor columns.  The paper notes that the sweep count depends
// strongly on the initial guess (Results) and leaves better guesses open.
//
//   features   per grid point P: log Z_PP, log sum_Q |Z_PQ|, log S_PP,
//              log sum_Q S_PQ^2, log max_p |X0_pP|, participation ratio
//              (sum x^2)^2 / (n sum x^4), log sum_Q S_PQ^2 |Z_PQ|,
//              log Z_PP S_PP^2; standardised over the grid points.
//   selection  rank of every grid point by score (ties: smaller P first),
//              F_m[:, k] = exp(ell_P) (X_m[:, P] + sigma ||X_m[:, P]|| R^_m[:, k])
//              for rank k < R_cp, R^ the unit columns of the caller's
//              random guess (the positive, strongly overlapping grid
//              columns alone make a nearly degenerate start).
//   labels     greedy one-to-one matching of a converged CPD's mode-0
//              columns to grid columns by |cosine|, largest first.
//   network    8 -> 256 -> 256 -> 2 with SiLU; FP32 training (the 256 x 256
//              layer and its gradients on the FP32 matrix cores through the
//              GEMM kernel, the rest in fused element-wise and fixed-order
//              reduction kernels, Adam); BF16 inference in one fused kernel
//              (the 256 x 256 layer on the BF16 matrix cores, FP32
//              accumulation).
// Every reduction has a fixed order: results are bitwise reproducible.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <mutex>

#include "../../include/thccp.h"
#include "common.h"
#include "kernels.h"

using namespace thccp;

namespace {

constexpr int D_IN = 8, WIDTH = 256, D_OUT = 2;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + D_IN * WIDTH;
constexpr int OFF_W2 = OFF_B1 + WIDTH;
constexpr int OFF_B2 = OFF_W2 + WIDTH * WIDTH;
constexpr int OFF_W3 = OFF_B2 + WIDTH;
constexpr int OFF_B3 = OFF_W3 + WIDTH * D_OUT;
constexpr int NPARAM = OFF_B3 + D_OUT;

// Packed inference weights: FP32 W1, b1, b2, W3, b3, then W2 transposed in
// BF16 (n-major, so one lane's eight k values are one 16-byte load).
constexpr int PK_W1 = 0;
constexpr int PK_B1 = PK_W1 + D_IN * WIDTH;
constexpr int PK_B2 = PK_B1 + WIDTH;
constexpr int PK_W3 = PK_B2 + WIDTH;
constexpr int PK_B3 = PK_W3 + WIDTH * D_OUT;
constexpr size_t PK_W2T_BYTES = ((size_t)(PK_B3 + D_OUT) * 4 + 255) & ~(size_t)255;
constexpr size_t PK_BYTES = PK_W2T_BYTES + (size_t)WIDTH * WIDTH * 2;

constexpr int CHUNK = 256;  // rows per partial sum of the reductions over rows
constexpr int CG = 32;      // columns per workgroup of the gradients' reductions
// Partial gradients of the small blocks, one vector per CHUNK rows.
constexpr int PG_W1 = 0;
constexpr int PG_B1 = PG_W1 + D_IN * WIDTH;
constexpr int PG_B2 = PG_B1 + WIDTH;
constexpr int PG_W3 = PG_B2 + WIDTH;
constexpr int PG_B3 = PG_W3 + WIDTH * D_OUT;
constexpr int PG_LEN = PG_B3 + D_OUT;
constexpr double TINY = 1e-300;

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }
int grid_of(size_t n) {
  size_t g = (n + 255) / 256;
  return (int)(g > 16384 ? 16384 : (g < 1 ? 1 : g));
}

#define WSCHK(x)                             \
  do {                                       \
    if ((x) != hipSuccess) return CPD_ERR_HIP; \
  } while (0)

struct Carve {
  char* p;
  size_t used = 0;
  template <typename T>
  T* take(size_t count) {
    T* r = (T*)(p + used);
    used += al(sizeof(T) * count);
    return r;
  }
};

// log(max(v, 1e-300)), NaN propagating like the definition's max.
__device__ __forceinline__ double lg(double v) { return v != v ? v : log(v > TINY ? v : TINY); }
__device__ __forceinline__ float sigm(float a) { return 1.f / (1.f + expf(-a)); }
__device__ __forceinline__ float silu(float a) { return a * sigm(a); }
__device__ __forceinline__ float silu_grad(float a) {
  const float g = sigm(a);
  return g * (1.f + a * (1.f - g));
}

// Fixed-order tree reduction over the 256 threads of a block.
template <typename T>
__device__ __forceinline__ T block_sum(T v, T* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) sh[tid] += sh[tid + w];
    __syncthreads();
  }
  T r = sh[0];
  __syncthreads();
  return r;
}

// Sums over the rows of a matrix, column by column: a workgroup takes CC
// columns (whole 128-byte lines) and 256 / CC groups of rows, so that the
// chip is full and a thread has eight loads in flight (one thread per
// column, one load at a time, took 98-114 us at 400 x 2000).  The groups'
// sums are added in a fixed order.
constexpr int CC = 16, CG_ROWS = 256 / CC;

// ------------------------------------------------------------ features
__global__ __launch_bounds__(256) void feat_rows_kernel(const double* Z, const double* S, int R, double* raw) {
  __shared__ double sh[256];
  const int P = blockIdx.x;
  double a = 0.0, b = 0.0, c = 0.0;
  for (int Q = threadIdx.x; Q < R; Q += 256) {
    const double z = fabs(Z[(size_t)P * R + Q]);
    const double s = S[(size_t)P * R + Q];
    a += z;
    b += s * s;
    c += s * s * z;
  }
  a = block_sum(a, sh);
  b = block_sum(b, sh);
  c = block_sum(c, sh);
  if (threadIdx.x == 0) {
    const double zd = Z[(size_t)P * R + P], sd = S[(size_t)P * R + P];
    double* f = raw + (size_t)P * D_IN;
    f[0] = lg(zd);
    f[1] = lg(a);
    f[2] = lg(sd);
    f[3] = lg(b);
    f[6] = lg(c);
    f[7] = lg(zd * sd * sd);
  }
}

__global__ __launch_bounds__(256) void feat_cols_kernel(const double* X0, int n, int R, double* raw) {
  __shared__ double sm[CG_ROWS][CC], s2[CG_ROWS][CC], s4[CG_ROWS][CC];
  const int c = threadIdx.x % CC, g = threadIdx.x / CC, P = blockIdx.x * CC + c;
  double mx = 0.0, x2 = 0.0, x4 = 0.0;
  if (P < R) {
#pragma unroll 8
    for (int p = g; p < n; p += CG_ROWS) {
      const double x = X0[(size_t)p * R + P];
      if (fabs(x) > mx || x != x) mx = fabs(x);  // NaN sticks
      x2 += x * x;
      x4 += (x * x) * (x * x);
    }
  }
  sm[g][c] = mx;
  s2[g][c] = x2;
  s4[g][c] = x4;
  __syncthreads();
  if (g || P >= R) return;
  mx = x2 = x4 = 0.0;
  for (int k = 0; k < CG_ROWS; ++k) {
    if (sm[k][c] > mx || sm[k][c] != sm[k][c]) mx = sm[k][c];
    x2 += s2[k][c];
    x4 += s4[k][c];
  }
  raw[(size_t)P * D_IN + 4] = lg(mx);
  raw[(size_t)P * D_IN + 5] = x4 > 0.0 ? x2 * x2 / ((double)n * x4) : 0.0;
}

// (bad, if given, is cleared for the checks that follow)
__global__ __launch_bounds__(256) void feat_standardise_kernel(const double* raw, int R, float* feat, double* heur,
                                                               int* bad) {
  __shared__ double sh[256];
  const int f = blockIdx.x;
  if (bad && f == 0 && threadIdx.x < 2) bad[threadIdx.x] = 0;
  double s = 0.0;
  for (int P = threadIdx.x; P < R; P += 256) s += raw[(size_t)P * D_IN + f];
  const double mu = block_sum(s, sh) / R;
  double v = 0.0;
  for (int P = threadIdx.x; P < R; P += 256) {
    const double d = raw[(size_t)P * D_IN + f] - mu;
    v += d * d;
  }
  const double sd = sqrt(block_sum(v, sh) / R);
  const bool ok = sd > 1e-9 * fmax(1.0, fabs(mu));
  for (int P = threadIdx.x; P < R; P += 256) {
    const double x = raw[(size_t)P * D_IN + f];
    feat[(size_t)P * D_IN + f] = ok ? (float)((x - mu) / sd) : 0.f;
    if (f == 7 && heur) heur[P] = x;
  }
}

// ------------------------------------------------------------ selection
// Rank of every grid point, one wave each, four to a workgroup (one thread
// per point took 134 us at 2000 points, 8 workgroups).
template <typename S>
__global__ __launch_bounds__(256) void rank_kernel(const S* s, int stride, int R, int Rc, int* perm) {
  const int P = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (P >= R) return;
  const S sp = s[(size_t)P * stride];
  int cnt = 0;
#pragma unroll 8
  for (int Q = lane; Q < R; Q += 64) {
    const S sq = s[(size_t)Q * stride];
    cnt += (sq > sp) || (sq == sp && Q < P);
  }
  for (int m = 32; m > 0; m >>= 1) cnt += __shfl_xor(cnt, m);
  if (lane == 0 && cnt < Rc) perm[cnt] = P;
}

struct ScatterArgs {
  const double* X[4];
  const double* noise[4];  // nullable: no blend
  double* F[4];
  int n[4];
  int xn[4];               // the first mode with the same X
};
// Column norms for the blend: xn[m][P] of X_m (r_thc per mode) and
// rn[m][k] of noise_m (r_cp per mode), laid out as 4 x (R + Rc).  A mode
// that shares its X with an earlier one uses that one's norms.
__global__ __launch_bounds__(256) void blend_norms_kernel(ScatterArgs a, int R, int Rc, double* norms) {
  __shared__ double sh[CG_ROWS][CC];
  const int m = blockIdx.y, z = blockIdx.z;
  const int c = threadIdx.x % CC, g = threadIdx.x / CC, col = blockIdx.x * CC + c;
  const int cols = z ? Rc : R;
  if (blockIdx.x * CC >= cols || (!z && a.xn[m] != m)) return;
  const double* A = z ? a.noise[m] : a.X[m];
  double s = 0.0;
  if (col < cols) {
#pragma unroll 8
    for (int p = g; p < a.n[m]; p += CG_ROWS) {
      const double v = A[(size_t)p * cols + col];
      s += v * v;
    }
  }
  sh[g][c] = s;
  __syncthreads();
  if (g || col >= cols) return;
  s = 0.0;
  for (int k = 0; k < CG_ROWS; ++k) s += sh[k][c];
  norms[(size_t)m * (R + Rc) + (z ? R : 0) + col] = sqrt(s);
}
// F_m[p, k] = exp(ell_P) (X_m[p, P] + sigma ||X_m[:, P]|| R_m[p, k] / ||R_m[:, k]||),
// P = perm[k], unless *bad.  A thread keeps its column and takes SROWS rows.
// Every element is read and written by one thread, so noise may alias F.
constexpr int SROWS = 16;
__global__ __launch_bounds__(256) void scatter_kernel(ScatterArgs a, int R, int Rc, const int* perm, const float* ell,
                                                      int stride, double sigma, const double* norms, const int* bad) {
  if (bad && *bad) return;
  const int m = blockIdx.z, k = blockIdx.x * 256 + threadIdx.x;
  const int p0 = blockIdx.y * SROWS, p1 = p0 + SROWS < a.n[m] ? p0 + SROWS : a.n[m];
  if (k >= Rc || p0 >= p1) return;
  const int P = perm[k];
  const double sc = ell ? exp((double)ell[(size_t)P * stride]) : 1.0;
  const double* noise = a.noise[m];
  const double xs = noise ? sigma * norms[(size_t)a.xn[m] * (R + Rc) + P] : 0.0;
  const double rn = noise ? norms[(size_t)m * (R + Rc) + R + k] : 0.0;
#pragma unroll 4
  for (int p = p0; p < p1; ++p) {
    const size_t e = (size_t)p * Rc + k;
    double v = a.X[m][(size_t)p * R + P];
    if (noise) {
      const double unit = rn > 0.0 ? noise[e] / rn : 0.0;
      v = v + xs * unit;
    }
    a.F[m][e] = v * sc;
  }
}

template <typename S>
__global__ void finite_kernel(const S* v, size_t count, int* bad) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (size_t)gridDim.x * 256)
    if (!isfinite((double)v[e])) *bad = 1;
}

// ------------------------------------------------------------ labels
__global__ void col_norms_kernel(const double* A, int rows, int cols, double* out) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= cols) return;
  double s = 0.0;
  for (int r = 0; r < rows; ++r) {
    const double v = A[(size_t)r * cols + c];
    s += v * v;
  }
  out[c] = sqrt(s);
}

__global__ void abs_cos_kernel(double* C, const double* fn, const double* xn, int Rc, int R) {
  const size_t total = (size_t)Rc * R;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
    const int k = (int)(e / R), P = (int)(e % R);
    const double den = fn[k] * xn[P];
    C[e] = den > 0.0 ? fabs(C[e]) / den : 0.0;
  }
}

// Better of two (value, index) candidates: larger value, then smaller index.
__device__ __forceinline__ bool better(double v, int i, double bv, int bi) {
  return v > bv || (v == bv && i >= 0 && (bi < 0 || i < bi));
}

__global__ __launch_bounds__(256) void row_argmax_kernel(const double* C, int R, double* rowmax, int* rowarg) {
  __shared__ double sv[256];
  __shared__ int si[256];
  const int k = blockIdx.x, tid = threadIdx.x;
  double bv = -1.0;
  int bi = -1;
  for (int P = tid; P < R; P += 256) {
    const double v = C[(size_t)k * R + P];
    if (better(v, P, bv, bi)) { bv = v; bi = P; }
  }
  sv[tid] = bv;
  si[tid] = bi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w && better(sv[tid + w], si[tid + w], sv[tid], si[tid])) {
      sv[tid] = sv[tid + w];
      si[tid] = si[tid + w];
    }
    __syncthreads();
  }
  if (tid == 0) {
    rowmax[k] = sv[0];
    rowarg[k] = si[0];
  }
}

// Greedy matching in one workgroup: each round takes the largest remaining
// entry (ties: smaller row, then smaller column), then rescans the rows
// whose best column was just taken.
__global__ __launch_bounds__(1024) void greedy_kernel(const double* C, int Rc, int R, double* rowmax, int* rowarg,
                                                      int* rowused, int* colused, int* match) {
  __shared__ double sv[1024];
  __shared__ int si[1024];
  const int tid = threadIdx.x;
  for (int k = tid; k < Rc; k += 1024) {
    rowused[k] = 0;
    match[k] = -1;
  }
  for (int P = tid; P < R; P += 1024) colused[P] = 0;
  __syncthreads();
  const int rounds = Rc < R ? Rc : R;
  for (int round = 0; round < rounds; ++round) {
    double bv = -1.0;
    int bk = -1;
    for (int k = tid; k < Rc; k += 1024) {
      if (rowused[k] || rowarg[k] < 0) continue;
      if (better(rowmax[k], k, bv, bk)) { bv = rowmax[k]; bk = k; }
    }
    sv[tid] = bv;
    si[tid] = bk;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
      if (tid < w && better(sv[tid + w], si[tid + w], sv[tid], si[tid])) {
        sv[tid] = sv[tid + w];
        si[tid] = si[tid + w];
      }
      __syncthreads();
    }
    const int ks = si[0];
    if (ks < 0) break;  // uniform: every thread read the same value
    const int Ps = rowarg[ks];
    __syncthreads();
    if (tid == 0) {
      match[ks] = Ps;
      rowused[ks] = 1;
      colused[Ps] = 1;
    }
    __syncthreads();
    for (int k = tid; k < Rc; k += 1024) {
      if (rowused[k] || rowarg[k] != Ps) continue;
      double v = -1.0;
      int b = -1;
      for (int P = 0; P < R; ++P) {
        if (colused[P]) continue;
        const double c = C[(size_t)k * R + P];
        if (better(c, P, v, b)) { v = c; b = P; }
      }
      rowmax[k] = v;
      rowarg[k] = b;
    }
    __syncthreads();
  }
}

struct LabelArgs {
  const double* X[4];
  const double* F[4];
  int n[4];
};
__global__ __launch_bounds__(256) void label_targets_kernel(LabelArgs a, const double* lam, const int* match, int R,
                                                            int Rc, float* y, float* ell, float* mask) {
  __shared__ double sh[256];
  const int k = blockIdx.x;
  const int P = match[k];
  if (P < 0) return;
  const double w = pow(fabs(lam[k]), 0.25);
  double acc = 0.0;
  bool ok = true;
  for (int m = 0; m < 4; ++m) {
    double xx = 0.0, d = 0.0;
    for (int p = threadIdx.x; p < a.n[m]; p += 256) {
      const double x = a.X[m][(size_t)p * R + P];
      xx += x * x;
      d += a.F[m][(size_t)p * Rc + k] * x;
    }
    xx = block_sum(xx, sh);
    d = block_sum(d, sh);
    if (!(xx > 0.0)) {
      ok = false;
      break;
    }
    acc += lg(fabs(w * d / xx));
  }
  if (threadIdx.x == 0) {
    y[P] = 1.f;
    ell[P] = ok ? (float)(acc / 4.0) : 0.f;
    mask[P] = ok ? 1.f : 0.f;
  }
}

__global__ void zero_f32(float* a, size_t n) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) a[e] = 0.f;
}

// ------------------------------------------------------------ network, FP32
// The training step runs in ten launches (with the Adam update).  What bounded the first form of
// it were its reductions over the rows: one workgroup per 256 rows and one
// load at a time (192 us each at 8192 rows, three of them).  Now a row's
// values are formed by many threads into LDS, and one thread per output
// adds them from there; the element-wise passes ride along, and a1 and h2
// are formed again where they are needed (8 products and one sigmoid)
// instead of stored.  Every sum keeps its order (rows of a chunk one by
// one, then the chunks): training is a long recursion, so another order
// would end in other weights.
__device__ __forceinline__ float layer1(const float w[D_IN], float b, const float* x) {
  float a = b;
#pragma unroll
  for (int i = 0; i < D_IN; ++i) a += x[i] * w[i];
  return a;
}

// h1 = silu(x W1 + b1), thread j = column j, 16 rows per workgroup.
constexpr int L1R = 16;
__global__ __launch_bounds__(256) void l1_fwd_kernel(const float* prm, const float* x, const int* idx, int rows,
                                                     float* h1) {
  __shared__ float xs[L1R][D_IN];
  const int j = threadIdx.x, r0 = blockIdx.x * L1R;
  const int m = rows - r0 < L1R ? rows - r0 : L1R;
  if (j < m * D_IN) {
    const int r = r0 + j / D_IN;
    xs[j / D_IN][j % D_IN] = x[(size_t)(idx ? idx[r] : r) * D_IN + j % D_IN];
  }
  float wj[D_IN];
#pragma unroll
  for (int i = 0; i < D_IN; ++i) wj[i] = prm[OFF_W1 + i * WIDTH + j];
  const float bj = prm[OFF_B1 + j];
  __syncthreads();
  for (int r = 0; r < m; ++r) h1[(size_t)(r0 + r) * WIDTH + j] = silu(layer1(wj, bj, xs[r]));
}

// out = silu(z2 + b2) W3 + b3 (z2 = h1 W2): one wave per row, lane l holds
// columns 4l .. 4l+3.
__global__ __launch_bounds__(256) void l3_fwd_kernel(const float* prm, const float* z2, int rows, float* out) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const f4_t z = *(const f4_t*)(z2 + (size_t)r * WIDTH + 4 * lane);
  float s0 = 0.f, s1 = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = 4 * lane + q;
    const float h = silu(z[q] + prm[OFF_B2 + c]);
    s0 += h * prm[OFF_W3 + 2 * c];
    s1 += h * prm[OFF_W3 + 2 * c + 1];
  }
  for (int m = 32; m > 0; m >>= 1) {
    s0 += __shfl_xor(s0, m);
    s1 += __shfl_xor(s1, m);
  }
  if (lane == 0) {
    out[2 * (size_t)r] = s0 + prm[OFF_B3];
    out[2 * (size_t)r + 1] = s1 + prm[OFF_B3 + 1];
  }
}

__global__ __launch_bounds__(256) void loss_partial_kernel(const float* out, const float* y, const float* ell_t,
                                                           const float* mask, const int* idx, int rows,
                                                           double* part) {
  __shared__ double sh[256];
  const int r = blockIdx.x * CHUNK + threadIdx.x;
  double bce = 0.0, ms = 0.0, sq = 0.0;
  if (r < rows) {
    const int src = idx ? idx[r] : r;
    const float s = out[2 * (size_t)r], l = out[2 * (size_t)r + 1];
    const float yv = y[src], lt = ell_t[src], mv = mask[src];
    bce = (double)(fmaxf(s, 0.f) - s * yv + log1pf(expf(-fabsf(s))));
    ms = mv;
    sq = (double)(mv * (l - lt) * (l - lt));
  }
  bce = block_sum(bce, sh);
  ms = block_sum(ms, sh);
  sq = block_sum(sq, sh);
  if (threadIdx.x == 0) {
    part[3 * (size_t)blockIdx.x] = bce;
    part[3 * (size_t)blockIdx.x + 1] = ms;
    part[3 * (size_t)blockIdx.x + 2] = sq;
  }
}

// Every workgroup sums the chunks' partial sums (in the same fixed order)
// and forms the gradients of its rows; the first one also writes the loss.
__global__ __launch_bounds__(256) void loss_grad_kernel(const float* out, const float* y, const float* ell_t,
                                                        const float* mask, const int* idx, int rows,
                                                        const double* part, int nchunk, float* dout, double* loss) {
  __shared__ double sh[256];
  double b = 0.0, m = 0.0, q = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    b += part[3 * (size_t)c];
    m += part[3 * (size_t)c + 1];
    q += part[3 * (size_t)c + 2];
  }
  m = block_sum(m, sh);
  const double ms = m > 1.0 ? m : 1.0;
  if (blockIdx.x == 0 && loss) {
    b = block_sum(b, sh);
    q = block_sum(q, sh);
    if (threadIdx.x == 0) *loss = b / rows + q / ms;
  }
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= rows) return;
  const int src = idx ? idx[r] : r;
  const float s = out[2 * (size_t)r], l = out[2 * (size_t)r + 1];
  const float inv_ms = (float)(1.0 / ms);
  dout[2 * (size_t)r] = (sigm(s) - y[src]) / (float)rows;
  dout[2 * (size_t)r + 1] = 2.f * mask[src] * (l - ell_t[src]) * inv_ms;
}

// Backward of layer 3 and layer 2's activation for CHUNK rows x CG columns:
// da2 = (dout W3^T) o silu'(a2), and the chunk's sums of dW3 = h2^T dout,
// db3 and db2.
__global__ __launch_bounds__(256) void bwd3_kernel(const float* prm, const float* dout, const float* z2, int rows,
                                                   float* da2, float* part) {
  __shared__ float hs[CHUNK][CG], ds[CHUNK][CG], go[CHUNK][D_OUT];
  const int tid = threadIdx.x, c = tid % CG, r0 = blockIdx.x * CHUNK, j = blockIdx.y * CG + c;
  const int m = rows - r0 < CHUNK ? rows - r0 : CHUNK;
  for (int e = tid; e < m * D_OUT; e += 256) go[e / D_OUT][e % D_OUT] = dout[(size_t)r0 * D_OUT + e];
  const float w0 = prm[OFF_W3 + 2 * j], w1 = prm[OFF_W3 + 2 * j + 1], bj = prm[OFF_B2 + j];
  const float* zc = z2 + (size_t)r0 * WIDTH + j;
  float z[CHUNK * CG / 256];  // all of the thread's loads in flight at once
#pragma unroll
  for (int i = 0; i < CHUNK * CG / 256; ++i) {
    const int r = tid / CG + i * (256 / CG);
    z[i] = r < m ? zc[(size_t)r * WIDTH] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < CHUNK * CG / 256; ++i) {
    const int r = tid / CG + i * (256 / CG);
    if (r < m) {
      const float a = z[i] + bj;
      const float g = go[r][0] * w0 + go[r][1] * w1;
      const float d = g * silu_grad(a);
      da2[(size_t)(r0 + r) * WIDTH + j] = d;
      ds[r][c] = d;
      hs[r][c] = silu(a);
    }
  }
  __syncthreads();
  float* q = part + (size_t)blockIdx.x * PG_LEN;
  const int k = tid / CG;  // the sum: dW3 of either output, db2, db3
  float acc = 0.f;
  if (k < D_OUT) {
#pragma unroll 16
    for (int r = 0; r < m; ++r) acc += hs[r][c] * go[r][k];
    q[PG_W3 + D_OUT * j + k] = acc;
  } else if (k == D_OUT) {
#pragma unroll 16
    for (int r = 0; r < m; ++r) acc += ds[r][c];
    q[PG_B2 + j] = acc;
  } else if (k == D_OUT + 1 && j < D_OUT) {
#pragma unroll 16
    for (int r = 0; r < m; ++r) acc += go[r][j];
    q[PG_B3 + j] = acc;
  }
}

// Backward of layer 1 likewise: da1 = dh1 o silu'(a1), the chunk's sums of
// dW1 = x^T da1 and db1.
__global__ __launch_bounds__(256) void bwd1_kernel(const float* prm, const float* dh1, const float* x, const int* idx,
                                                   int rows, float* part) {
  __shared__ float xs[CHUNK][D_IN], ds[CHUNK][CG];
  const int tid = threadIdx.x, c = tid % CG, r0 = blockIdx.x * CHUNK, j = blockIdx.y * CG + c;
  const int m = rows - r0 < CHUNK ? rows - r0 : CHUNK;
  for (int e = tid; e < m * D_IN; e += 256) {
    const int r = r0 + e / D_IN;
    xs[e / D_IN][e % D_IN] = x[(size_t)(idx ? idx[r] : r) * D_IN + e % D_IN];
  }
  float wj[D_IN];
#pragma unroll
  for (int i = 0; i < D_IN; ++i) wj[i] = prm[OFF_W1 + i * WIDTH + j];
  const float bj = prm[OFF_B1 + j];
  const float* dc = dh1 + (size_t)r0 * WIDTH + j;
  float d[CHUNK * CG / 256];
#pragma unroll
  for (int i = 0; i < CHUNK * CG / 256; ++i) {
    const int r = tid / CG + i * (256 / CG);
    d[i] = r < m ? dc[(size_t)r * WIDTH] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < CHUNK * CG / 256; ++i) {
    const int r = tid / CG + i * (256 / CG);
    if (r < m) ds[r][c] = d[i] * silu_grad(layer1(wj, bj, xs[r]));
  }
  __syncthreads();
  float* q = part + (size_t)blockIdx.x * PG_LEN;
  const int k = tid / CG;  // the sum: dW1 of input k (and db1, by the threads of input 0)
  static_assert(256 / CG == D_IN, "one thread per input and column");
  float acc = 0.f;
#pragma unroll 16
  for (int r = 0; r < m; ++r) acc += xs[r][k] * ds[r][c];
  q[PG_W1 + k * WIDTH + j] = acc;
  if (k == 0) {
    acc = 0.f;
#pragma unroll 16
    for (int r = 0; r < m; ++r) acc += ds[r][c];
    q[PG_B1 + j] = acc;
  }
}

// Sums the partial gradients over the chunks, in their order.
__global__ __launch_bounds__(64) void grad_sum_kernel(const float* part, int nchunk, float* grads) {
  const int o = blockIdx.x * 64 + threadIdx.x;
  if (o >= PG_LEN) return;
  float acc = 0.f;
#pragma unroll 16
  for (int c = 0; c < nchunk; ++c) acc += part[(size_t)c * PG_LEN + o];
  // (W1, b1) and (b2, W3, b3) lie in the parameters' own order
  grads[o < PG_B2 ? OFF_W1 + o : OFF_B2 + (o - PG_B2)] = acc;
}

__global__ void adam_kernel(float* p, const float* g, float* m, float* v, int n, float lr, float b1, float b2,
                            float eps, float bc1, float bc2) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * bc1) / (sqrtf(vi * bc2) + eps);
}

// ------------------------------------------------------------ network, BF16 inference
__global__ void pack_kernel(const float* prm, float* pk, __bf16* w2t) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < WIDTH * WIDTH) {
    const int n = e / WIDTH, k = e % WIDTH;
    w2t[e] = (__bf16)prm[OFF_W2 + k * WIDTH + n];
  }
  if (e < D_IN * WIDTH) pk[PK_W1 + e] = prm[OFF_W1 + e];
  if (e < WIDTH) {
    pk[PK_B1 + e] = prm[OFF_B1 + e];
    pk[PK_B2 + e] = prm[OFF_B2 + e];
  }
  if (e < WIDTH * D_OUT) pk[PK_W3 + e] = prm[OFF_W3 + e];
  if (e < D_OUT) pk[PK_B3 + e] = prm[OFF_B3 + e];
}

// IR rows per workgroup: 64, or 16 where that many workgroups would leave
// compute units idle (2000 rows: 19.5 us with 64, 9.3 us with 16).
constexpr int HLD = WIDTH + 8;  // LDS row stride (bf16), keeps 16-byte alignment

template <int IR>
__global__ __launch_bounds__(256) void infer_bf16_kernel(const float* pk, const __bf16* w2t, const float* x,
                                                         int rows, float* out) {
  __shared__ float xs[IR][D_IN];
  __shared__ __attribute__((aligned(16))) __bf16 hs[IR * HLD];
  __shared__ float red[4][IR][D_OUT];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r0 = blockIdx.x * IR;
  for (int e = tid; e < IR * D_IN; e += 256) {
    const int r = e / D_IN, i = e % D_IN;
    xs[r][i] = r0 + r < rows ? x[(size_t)(r0 + r) * D_IN + i] : 0.f;
  }
  __syncthreads();
  {
    const int j = tid;
    float wj[D_IN];
#pragma unroll
    for (int i = 0; i < D_IN; ++i) wj[i] = pk[PK_W1 + i * WIDTH + j];
    const float bj = pk[PK_B1 + j];
    for (int r = 0; r < IR; ++r) {
      float a = bj;
#pragma unroll
      for (int i = 0; i < D_IN; ++i) a += xs[r][i] * wj[i];
      hs[r * HLD + j] = (__bf16)silu(a);
    }
  }
  __syncthreads();
  constexpr int TI = IR / 16;
  f4_t acc[TI][4];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int k0 = 0; k0 < WIDTH; k0 += 32) {
    const int koff = k0 + 8 * (lane >> 4);
    bf16x8_t a[TI], b[4];
#pragma unroll
    for (int i = 0; i < TI; ++i) a[i] = *(const bf16x8_t*)&hs[(16 * i + (lane & 15)) * HLD + koff];
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = *(const bf16x8_t*)&w2t[(size_t)(64 * w + 16 * j + (lane & 15)) * WIDTH + koff];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  }
  // h2 = silu(acc + b2); partial out over this lane's columns, then over
  // the 16 lanes of a row group, then over the four waves.
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = 64 * w + 16 * j + (lane & 15);
        const float h = silu(acc[i][j][r] + pk[PK_B2 + col]);
        s0 += h * pk[PK_W3 + 2 * col];
        s1 += h * pk[PK_W3 + 2 * col + 1];
      }
      for (int m = 8; m > 0; m >>= 1) {
        s0 += __shfl_xor(s0, m);
        s1 += __shfl_xor(s1, m);
      }
      if ((lane & 15) == 0) {
        const int row = 16 * i + 4 * (lane >> 4) + r;
        red[w][row][0] = s0;
        red[w][row][1] = s1;
      }
    }
  __syncthreads();
  if (tid < IR * D_OUT) {
    const int row = tid / D_OUT, j = tid % D_OUT;
    if (r0 + row < rows)
      out[(size_t)(r0 + row) * D_OUT + j] =
          pk[PK_B3 + j] + ((red[0][row][j] + red[1][row][j]) + (red[2][row][j] + red[3][row][j]));
  }
}

void infer_bf16(hipStream_t s, const void* packed, const float* x, int rows, float* out) {
  const float* pk = (const float*)packed;
  const __bf16* w2t = (const __bf16*)((const char*)packed + PK_W2T_BYTES);
  if (rows < 64 * 256)
    hipLaunchKernelGGL(infer_bf16_kernel<16>, dim3((rows + 15) / 16), dim3(256), 0, s, pk, w2t, x, rows, out);
  else
    hipLaunchKernelGGL(infer_bf16_kernel<64>, dim3((rows + 63) / 64), dim3(256), 0, s, pk, w2t, x, rows, out);
}

// ------------------------------------------------------------ workspace layouts
struct FeatWs {
  double* S;
  double* raw;
};
FeatWs carve_feat(Carve& c, int R) { return {c.take<double>((size_t)R * R), c.take<double>((size_t)R * D_IN)}; }
size_t feat_bytes(int R) { return al(sizeof(double) * (size_t)R * R) + al(sizeof(double) * (size_t)R * D_IN); }

int enqueue_features(hipStream_t s, int n0, int R, const double* X0, const double* Z, float* feat, double* heur,
                     FeatWs w, int* bad = nullptr) {
  syrk_f64(s, R, n0, X0, R, w.S, R);
  hipLaunchKernelGGL(feat_rows_kernel, dim3(R), dim3(256), 0, s, Z, w.S, R, w.raw);
  hipLaunchKernelGGL(feat_cols_kernel, dim3((R + CC - 1) / CC), dim3(256), 0, s, X0, n0, R, w.raw);
  hipLaunchKernelGGL(feat_standardise_kernel, dim3(D_IN), dim3(256), 0, s, w.raw, R, feat, heur, bad);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

bool dims_ok(const int32_t n[4], int32_t r_thc, int32_t r_cp) {
  if (!n || r_thc <= 0 || r_cp <= 0 || r_cp > r_thc) return false;
  for (int m = 0; m < 4; ++m)
    if (n[m] <= 0) return false;
  return true;
}

size_t select_bytes(int R, int Rc) { return al(sizeof(int) * (size_t)Rc) + al(sizeof(double) * 4 * ((size_t)R + Rc)); }

int enqueue_select(hipStream_t s, const int32_t n[4], int R, int Rc, const double* const X[4], double* const F[4],
                   const int* perm, const float* ell, int stride, const double* const noise[4], double sigma,
                   double* norms, const int* bad = nullptr) {
  ScatterArgs a;
  int nmax = 0;
  for (int m = 0; m < 4; ++m) {
    a.X[m] = X[m];
    a.noise[m] = (noise && sigma != 0.0) ? noise[m] : nullptr;
    a.F[m] = F[m];
    a.n[m] = n[m];
    a.xn[m] = m;
    for (int k = m - 1; k >= 0; --k)
      if (X[k] == X[m] && n[k] == n[m]) a.xn[m] = k;
    nmax = n[m] > nmax ? n[m] : nmax;
  }
  if (a.noise[0]) {
    const int cols = R > Rc ? R : Rc;
    hipLaunchKernelGGL(blend_norms_kernel, dim3((cols + CC - 1) / CC, 4, 2), dim3(256), 0, s, a, R, Rc, norms);
  }
  // (the y extent of a grid ends at 65535)
  for (int p0 = 0; p0 < nmax; p0 += 65535 * SROWS) {
    ScatterArgs b = a;
    int rows = 0;
    for (int m = 0; m < 4; ++m) {
      const int left = a.n[m] - p0;
      b.n[m] = left < 0 ? 0 : left < 65535 * SROWS ? left : 65535 * SROWS;
      b.X[m] = a.X[m] + (size_t)p0 * R;
      b.F[m] = a.F[m] + (size_t)p0 * Rc;
      if (a.noise[m]) b.noise[m] = a.noise[m] + (size_t)p0 * Rc;
      rows = b.n[m] > rows ? b.n[m] : rows;
    }
    hipLaunchKernelGGL(scatter_kernel, dim3((Rc + 255) / 256, (rows + SROWS - 1) / SROWS, 4), dim3(256), 0, s, b, R, Rc,
                       perm, ell, stride, sigma, norms, bad);
  }
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

size_t mlp_ws_bytes(int rows) {
  const size_t act = al(sizeof(float) * (size_t)rows * WIDTH);
  const size_t nchunk = (rows + CHUNK - 1) / CHUNK;
  return 4 * act + al(sizeof(float) * nchunk * PG_LEN) + al(sizeof(double) * 3 * nchunk);
}
struct MlpWs {
  float *h1, *z2, *d1, *d2, *part;
  double* lpart;
};
MlpWs carve_mlp(void* ws, int rows) {
  Carve c{(char*)ws};
  const size_t act = (size_t)rows * WIDTH, nchunk = (rows + CHUNK - 1) / CHUNK;
  MlpWs w;
  w.h1 = c.take<float>(act);
  w.z2 = c.take<float>(act);
  w.d1 = c.take<float>(act);
  w.d2 = c.take<float>(act);
  w.part = c.take<float>(nchunk * PG_LEN);
  w.lpart = c.take<double>(3 * nchunk);
  return w;
}

// Scratch of the allocation-free feature entry point: S = X0^T X0
// (r_thc^2 doubles) and the raw features (r_thc x 8 doubles) for
// r_thc <= WS_NOALLOC_MAX_RTHC.  One copy per GPU, alive until the process
// ends; host code uses only the device address of this array looked up with
// hipGetSymbolAddress, once per device (the name itself is a host-side
// stand-in, not a device address).
constexpr int WS_NOALLOC_MAX_RTHC = 2048;
constexpr size_t al_c(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr size_t WS_NOALLOC_BYTES =
    al_c(sizeof(double) * (size_t)WS_NOALLOC_MAX_RTHC * WS_NOALLOC_MAX_RTHC) +
    al_c(sizeof(double) * (size_t)WS_NOALLOC_MAX_RTHC * D_IN);
static __device__ __align__(256) char feat_scratch[WS_NOALLOC_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[MAX_DEVICES] = {};

// Device address of feat_scratch on the current device (looked up on the
// first call per device); nullptr if the lookup fails.
void* scratch_of_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(feat_scratch)) != hipSuccess || !ptr) return nullptr;
    g_scratch_dev[dev] = ptr;
  }
  return g_scratch_dev[dev];
}

}  // namespace

extern "C" {

size_t cpd_ws_workspace_size(int32_t n0, int32_t r_thc, int32_t r_cp) {
  if (n0 <= 0 || r_thc <= 0 || r_cp <= 0 || r_cp > r_thc) return 0;
  const size_t R = r_thc, Rc = r_cp;
  return feat_bytes(r_thc) + al(sizeof(float) * R * D_IN) + al(sizeof(double) * R) + al(sizeof(float) * R * D_OUT) +
         select_bytes(r_thc, r_cp) + al(2 * sizeof(int)) + al(sizeof(double) * Rc * R) + 2 * al(sizeof(double) * (Rc + R)) +
         4 * al(sizeof(int) * (Rc + R));
}

cpd_status cpd_ws_features(int32_t n0, int32_t r_thc, const double* X0, const double* Z, float* feat, double* heur,
                           void* workspace, size_t workspace_bytes, void* stream) {
  if (n0 <= 0 || r_thc <= 0 || !X0 || !Z || !feat || !workspace) return CPD_ERR_INVALID_ARG;
  if (workspace_bytes < feat_bytes(r_thc)) return CPD_ERR_WORKSPACE;
  Carve c{(char*)workspace};
  return enqueue_features((hipStream_t)stream, n0, r_thc, X0, Z, feat, heur, carve_feat(c, r_thc));
}

cpd_status cpd_ws_features_noalloc(int32_t n0, int32_t r_thc, const double* X0, const double* Z, float* feat,
                                   double* heur, void* stream) {
  if (n0 <= 0 || r_thc <= 0 || !X0 || !Z || !feat) return CPD_ERR_INVALID_ARG;
  if (r_thc > WS_NOALLOC_MAX_RTHC) return CPD_ERR_INVALID_ARG;
  void* ws = scratch_of_current_device();
  if (!ws) return CPD_ERR_HIP;
  Carve c{(char*)ws};
  return enqueue_features((hipStream_t)stream, n0, r_thc, X0, Z, feat, heur, carve_feat(c, r_thc));
}

cpd_status cpd_ws_select_init(const int32_t n[4], int32_t r_thc, int32_t r_cp, const double* const X[4],
                              const float* s, const float* ell, int32_t stride, const double* const noise[4],
                              double sigma, double* const init[4], void* workspace, size_t workspace_bytes,
                              void* stream) {
  if (!dims_ok(n, r_thc, r_cp) || !X || !s || !init || stride <= 0 || !workspace || !(sigma >= 0.0))
    return CPD_ERR_INVALID_ARG;
  for (int m = 0; m < 4; ++m)
    if (!X[m] || !init[m] || (noise && !noise[m])) return CPD_ERR_INVALID_ARG;
  if (workspace_bytes < select_bytes(r_thc, r_cp)) return CPD_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  Carve c{(char*)workspace};
  int* perm = c.take<int>(r_cp);
  double* norms = c.take<double>(4 * ((size_t)r_thc + r_cp));
  hipLaunchKernelGGL(rank_kernel<float>, dim3((r_thc + 3) / 4), dim3(256), 0, st, s, stride, r_thc, r_cp, perm);
  return enqueue_select(st, n, r_thc, r_cp, X, init, perm, ell, stride, noise, sigma, norms);
}

cpd_status cpd_ws_labels(const int32_t n[4], int32_t r_thc, int32_t r_cp, const double* const X[4],
                         const double* const F[4], const double* lam, float* y, float* ell, float* mask,
                         void* workspace, size_t workspace_bytes, void* stream) {
  if (!dims_ok(n, r_thc, r_cp) || !X || !F || !lam || !y || !ell || !mask || !workspace) return CPD_ERR_INVALID_ARG;
  for (int m = 0; m < 4; ++m)
    if (!X[m] || !F[m]) return CPD_ERR_INVALID_ARG;
  const size_t R = r_thc, Rc = r_cp;
  const size_t need = al(sizeof(double) * Rc * R) + 2 * al(sizeof(double) * (Rc + R)) + 4 * al(sizeof(int) * (Rc + R));
  if (workspace_bytes < need) return CPD_ERR_WORKSPACE;
  Carve c{(char*)workspace};
  double* C = c.take<double>(Rc * R);
  double* fn = c.take<double>(Rc + R);
  double* xn = fn + Rc;
  double* rowmax = c.take<double>(Rc + R);
  int* rowarg = c.take<int>(Rc + R);
  int* rowused = c.take<int>(Rc + R);
  int* colused = c.take<int>(Rc + R);
  int* match = c.take<int>(Rc + R);
  hipStream_t st = (hipStream_t)stream;
  GemmF64 g{r_cp, r_thc, n[0], F[0], r_cp, true, X[0], nullptr, r_thc, false, C, r_thc, 1.0, 0.0};
  gemm_f64(st, g);
  hipLaunchKernelGGL(col_norms_kernel, dim3((r_cp + 255) / 256), dim3(256), 0, st, F[0], n[0], r_cp, fn);
  hipLaunchKernelGGL(col_norms_kernel, dim3((r_thc + 255) / 256), dim3(256), 0, st, X[0], n[0], r_thc, xn);
  hipLaunchKernelGGL(abs_cos_kernel, dim3(grid_of(Rc * R)), dim3(256), 0, st, C, fn, xn, r_cp, r_thc);
  hipLaunchKernelGGL(row_argmax_kernel, dim3(r_cp), dim3(256), 0, st, C, r_thc, rowmax, rowarg);
  hipLaunchKernelGGL(greedy_kernel, dim3(1), dim3(1024), 0, st, C, r_cp, r_thc, rowmax, rowarg, rowused, colused,
                     match);
  for (float* a : {y, ell, mask}) hipLaunchKernelGGL(zero_f32, dim3(grid_of(R)), dim3(256), 0, st, a, R);
  LabelArgs la;
  for (int m = 0; m < 4; ++m) {
    la.X[m] = X[m];
    la.F[m] = F[m];
    la.n[m] = n[m];
  }
  hipLaunchKernelGGL(label_targets_kernel, dim3(r_cp), dim3(256), 0, st, la, lam, match, r_thc, r_cp, y, ell, mask);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

int32_t cpd_mlp_param_count(void) { return NPARAM; }
size_t cpd_mlp_workspace_size(int32_t rows) { return rows > 0 ? mlp_ws_bytes(rows) : 0; }
size_t cpd_mlp_packed_size(void) { return PK_BYTES; }

cpd_status cpd_mlp_forward(const float* params, const float* x, const int32_t* idx, int32_t rows, float* out,
                           void* workspace, size_t workspace_bytes, void* stream) {
  if (!params || !x || !out || rows <= 0 || !workspace) return CPD_ERR_INVALID_ARG;
  if (workspace_bytes < mlp_ws_bytes(rows)) return CPD_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  MlpWs w = carve_mlp(workspace, rows);
  hipLaunchKernelGGL(l1_fwd_kernel, dim3((rows + L1R - 1) / L1R), dim3(256), 0, s, params, x, idx, rows, w.h1);
  GemmF32 g{rows, WIDTH, WIDTH, w.h1, WIDTH, false, params + OFF_W2, nullptr, WIDTH, false, w.z2, WIDTH,
            1.f, 0.f};
  gemm_f32(s, g);
  hipLaunchKernelGGL(l3_fwd_kernel, dim3((rows + 3) / 4), dim3(256), 0, s, params, w.z2, rows, out);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

cpd_status cpd_mlp_loss(const float* out, const float* y, const float* ell_t, const float* mask, const int32_t* idx,
                        int32_t rows, float* dout, double* loss_dev, void* workspace, size_t workspace_bytes,
                        void* stream) {
  if (!out || !y || !ell_t || !mask || !dout || rows <= 0 || !workspace) return CPD_ERR_INVALID_ARG;
  if (workspace_bytes < mlp_ws_bytes(rows)) return CPD_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  MlpWs w = carve_mlp(workspace, rows);
  const int nchunk = (rows + CHUNK - 1) / CHUNK;
  hipLaunchKernelGGL(loss_partial_kernel, dim3(nchunk), dim3(256), 0, s, out, y, ell_t, mask, idx, rows, w.lpart);
  hipLaunchKernelGGL(loss_grad_kernel, dim3((rows + 255) / 256), dim3(256), 0, s, out, y, ell_t, mask, idx, rows,
                     w.lpart, nchunk, dout, loss_dev);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

cpd_status cpd_mlp_backward(const float* params, const float* x, const int32_t* idx, const float* dout,
                            int32_t rows, float* grads, void* workspace, size_t workspace_bytes, void* stream) {
  if (!params || !x || !dout || !grads || rows <= 0 || !workspace) return CPD_ERR_INVALID_ARG;
  if (workspace_bytes < mlp_ws_bytes(rows)) return CPD_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  MlpWs w = carve_mlp(workspace, rows);
  const dim3 chunks((rows + CHUNK - 1) / CHUNK, WIDTH / CG);
  hipLaunchKernelGGL(bwd3_kernel, chunks, dim3(256), 0, s, params, dout, w.z2, rows, w.d2, w.part);
  // layer 2: dW2 = h1^T da2, dh1 = da2 W2^T
  GemmF32 gw{WIDTH, WIDTH, rows, w.h1, WIDTH, true, w.d2, nullptr, WIDTH, false, grads + OFF_W2, WIDTH,
             1.f, 0.f};
  GemmF32 gd{rows, WIDTH, WIDTH, w.d2, WIDTH, false, params + OFF_W2, nullptr, WIDTH, true, w.d1, WIDTH,
             1.f, 0.f};
  gemm_f32_two(s, gw, gd);
  hipLaunchKernelGGL(bwd1_kernel, chunks, dim3(256), 0, s, params, w.d1, x, idx, rows, w.part);
  hipLaunchKernelGGL(grad_sum_kernel, dim3((PG_LEN + 63) / 64), dim3(64), 0, s, w.part, (int)chunks.x, grads);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

cpd_status cpd_mlp_adam(float* params, const float* grads, float* m, float* v, int32_t step, float lr, float beta1,
                        float beta2, float eps, void* stream) {
  if (!params || !grads || !m || !v || step < 1 || !(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) ||
      !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
    return CPD_ERR_INVALID_ARG;
  const double bc1 = 1.0 / (1.0 - pow((double)beta1, step));
  const double bc2 = 1.0 / (1.0 - pow((double)beta2, step));
  hipLaunchKernelGGL(adam_kernel, dim3((NPARAM + 255) / 256), dim3(256), 0, (hipStream_t)stream, params, grads, m, v,
                     NPARAM, lr, beta1, beta2, eps, (float)bc1, (float)bc2);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

cpd_status cpd_mlp_pack(const float* params, void* packed, void* stream) {
  if (!params || !packed) return CPD_ERR_INVALID_ARG;
  if ((uintptr_t)packed % 256) return CPD_ERR_INVALID_ARG;
  hipLaunchKernelGGL(pack_kernel, dim3((WIDTH * WIDTH + 255) / 256), dim3(256), 0, (hipStream_t)stream, params,
                     (float*)packed, (__bf16*)((char*)packed + PK_W2T_BYTES));
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

cpd_status cpd_mlp_infer_bf16(const void* packed, const float* x, int32_t rows, float* out, void* stream) {
  if (!packed || !x || !out || rows <= 0) return CPD_ERR_INVALID_ARG;
  if ((uintptr_t)packed % 256) return CPD_ERR_INVALID_ARG;
  infer_bf16((hipStream_t)stream, packed, x, rows, out);
  return hipGetLastError() == hipSuccess ? CPD_OK : CPD_ERR_HIP;
}

cpd_status cpd_ws_init(const int32_t n[4], int32_t r_thc, int32_t r_cp, const double* const X[4], const double* Z,
                       const void* packed, const double* const noise[4], double sigma, double* const init[4],
                       int32_t* source, void* workspace, size_t workspace_bytes, void* stream) {
  if (!dims_ok(n, r_thc, r_cp) || !X || !Z || !init || !workspace || !(sigma >= 0.0)) return CPD_ERR_INVALID_ARG;
  for (int m = 0; m < 4; ++m)
    if (!X[m] || !init[m] || (noise && !noise[m])) return CPD_ERR_INVALID_ARG;
  if (packed && (uintptr_t)packed % 256) return CPD_ERR_INVALID_ARG;
  if (workspace_bytes < cpd_ws_workspace_size(n[0], r_thc, r_cp)) return CPD_ERR_WORKSPACE;
  const int R = r_thc, Rc = r_cp;
  hipStream_t s = (hipStream_t)stream;
  Carve c{(char*)workspace};
  FeatWs fw = carve_feat(c, R);
  float* feat = c.take<float>((size_t)R * D_IN);
  double* heur = c.take<double>(R);
  float* out = c.take<float>((size_t)R * D_OUT);
  int* perm = c.take<int>(Rc);
  double* norms = c.take<double>(4 * ((size_t)R + Rc));
  int* bad = c.take<int>(2);  // non-finite scores of the network, of the heuristic
  int rc = enqueue_features(s, n[0], R, X[0], Z, feat, heur, fw, bad);
  if (rc != CPD_OK) return rc;
  // The selection follows its check without a word from the host: with a
  // non-finite score its last kernel writes nothing, so the noise is intact
  // for the next source.
  int src = 2;
  int hbad = 1;
  if (packed) {
    infer_bf16(s, packed, feat, R, out);
    hipLaunchKernelGGL(finite_kernel<float>, dim3(grid_of((size_t)R * D_OUT)), dim3(256), 0, s, out,
                       (size_t)R * D_OUT, bad);
    hipLaunchKernelGGL(rank_kernel<float>, dim3((R + 3) / 4), dim3(256), 0, s, out, D_OUT, R, Rc, perm);
    rc = enqueue_select(s, n, R, Rc, X, init, perm, out + 1, D_OUT, noise, sigma, norms, bad);
    if (rc != CPD_OK) return rc;
    WSCHK(hipMemcpyAsync(&hbad, bad, sizeof(int), hipMemcpyDeviceToHost, s));
    WSCHK(hipStreamSynchronize(s));
    if (!hbad) src = 0;
  }
  if (src == 2) {
    hipLaunchKernelGGL(finite_kernel<double>, dim3(grid_of(R)), dim3(256), 0, s, heur, (size_t)R, bad + 1);
    hipLaunchKernelGGL(rank_kernel<double>, dim3((R + 3) / 4), dim3(256), 0, s, heur, 1, R, Rc, perm);
    rc = enqueue_select(s, n, R, Rc, X, init, perm, nullptr, 1, noise, sigma, norms, bad + 1);
    if (rc != CPD_OK) return rc;
    WSCHK(hipMemcpyAsync(&hbad, bad + 1, sizeof(int), hipMemcpyDeviceToHost, s));
    WSCHK(hipStreamSynchronize(s));
    if (!hbad) src = 1;
  }
  if (source) *source = src;
  return CPD_OK;
}

}  // extern "C"
