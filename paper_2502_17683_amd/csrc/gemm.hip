// Dense GEMM on the 16x16x4 FP64 / FP32 matrix cores.
//
// This one kernel family carries every FP64 / FP32 contraction of the
// matrix-free MTTKRP (projection X^T F, core product Z (W o W),
// back-projection X (W o Y)), the Gram matrices F^T F, the set-up products
// and the FP32 layers of the warm-start network.
//
// Two forms:
//   - direct-load tiles (FP64 and FP32, gemm_tile_ok): operands go from
//     global memory straight into LDS, and are read from there 16 bytes a
//     lane (below).  Every product of a plan takes this form.
//   - register-staged 64 x 64 tiles, 256 threads = 2 x 2 waves, k-step 16
//     through LDS in k-major form, the next k-tile prefetched into
//     registers: single products of the other shapes and alignments.  It
//     also takes a Hadamard pair operand, which cpd_test_gemm alone still
//     passes (the pair operands of a plan are formed in the epilogue of the
//     product before).
#include "kernels.h"
#include "mfma.h"

namespace thccp {

template <typename T, int BM, int BN, bool AT, bool BT, bool HAD>
__device__ __forceinline__ void gemm_body(const GemmArgs<T>& p, int bid_in, int nblocks) {
  constexpr int BK = 16;
  constexpr int WTM = BM / 2, WTN = BN / 2;
  constexpr int TI = WTM / 16, TJ = WTN / 16;
  constexpr int PAD = 1;  // odd row stride: the k-contiguous A stores hit distinct banks
  constexpr int AE = BM * BK / 256, BE = BN * BK / 256;
  typedef typename Acc4<T>::type acc_t;
  __shared__ T As[BK][BM + PAD];
  __shared__ T Bs[BK][BN + PAD];

  int tm, tn;
  grouped_tile(xcd_remap(bid_in, nblocks), (p.M + BM - 1) / BM, (p.N + BN - 1) / BN, 8, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wm = wid >> 1, wn = wid & 1;
  const gptr<const T> gA = as_global(p.A), gB1 = as_global(p.B1), gB2 = as_global(p.B2);
  const gptr<T> gC = as_global(p.C);

  // Operand loads are unconditional: interior tiles (the whole k-tile in
  // range) load without checks; edge tiles read offset 0 for an
  // out-of-range element and zero it at the LDS store from the validity
  // bits.  The Hadamard product is also formed at the LDS store, so nothing
  // waits on the prefetch until the current k-tile's products are issued.
  T ra[AE], rb[BE], rb2[HAD ? BE : 1];
  uint32_t va = 0, vb = 0;
  const bool interior = m0 + BM <= p.M && n0 + BN <= p.N;
  auto load = [&](int k0) {
    if (interior && k0 + BK <= p.K) {
      va = vb = ~0u;
#pragma unroll
      for (int e = 0; e < AE; ++e) {
        const int idx = tid + e * 256;
        int i, k;
        if (AT) { i = idx % BM; k = idx / BM; } else { k = idx % BK; i = idx / BK; }
        ra[e] = AT ? gA[(size_t)(k0 + k) * p.lda + m0 + i] : gA[(size_t)(m0 + i) * p.lda + k0 + k];
      }
#pragma unroll
      for (int e = 0; e < BE; ++e) {
        const int idx = tid + e * 256;
        int j, k;
        if (BT) { k = idx % BK; j = idx / BK; } else { j = idx % BN; k = idx / BN; }
        const size_t off = BT ? (size_t)(n0 + j) * p.ldb + k0 + k : (size_t)(k0 + k) * p.ldb + n0 + j;
        rb[e] = gB1[off];
        if constexpr (HAD) rb2[e] = gB2[off];
      }
      return;
    }
    va = 0;
    vb = 0;
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const int idx = tid + e * 256;
      int i, k;
      if (AT) { i = idx % BM; k = idx / BM; } else { k = idx % BK; i = idx / BK; }
      const int gi = m0 + i, gk = k0 + k;
      const bool ok = gi < p.M && gk < p.K;
      const size_t off = ok ? (AT ? (size_t)gk * p.lda + gi : (size_t)gi * p.lda + gk) : 0;
      ra[e] = gA[off];
      va |= (uint32_t)ok << e;
    }
#pragma unroll
    for (int e = 0; e < BE; ++e) {
      const int idx = tid + e * 256;
      int j, k;
      if (BT) { k = idx % BK; j = idx / BK; } else { j = idx % BN; k = idx / BN; }
      const int gj = n0 + j, gk = k0 + k;
      const bool ok = gj < p.N && gk < p.K;
      const size_t off = ok ? (BT ? (size_t)gj * p.ldb + gk : (size_t)gk * p.ldb + gj) : 0;
      rb[e] = gB1[off];
      if constexpr (HAD) rb2[e] = gB2[off];
      vb |= (uint32_t)ok << e;
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int e = 0; e < AE; ++e) {
      const int idx = tid + e * 256;
      int i, k;
      if (AT) { i = idx % BM; k = idx / BM; } else { k = idx % BK; i = idx / BK; }
      As[k][i] = (va >> e) & 1 ? ra[e] : T(0);
    }
#pragma unroll
    for (int e = 0; e < BE; ++e) {
      const int idx = tid + e * 256;
      int j, k;
      if (BT) { k = idx % BK; j = idx / BK; } else { j = idx % BN; k = idx / BN; }
      T v = rb[e];
      if constexpr (HAD) {
        // keeps the product (and the wait for both loads) here, after the
        // current k-tile's matrix-core products
        T w = rb2[e];
        asm volatile("" : "+v"(v), "+v"(w));
        v *= w;
      }
      Bs[k][j] = (vb >> e) & 1 ? v : T(0);
    }
  };

  acc_t acc[TI][TJ];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b) acc[a][b] = acc_t{0, 0, 0, 0};

  const int nk = (p.K + BK - 1) / BK;
  load(0);
  store();
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) load((kt + 1) * BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int k = kk + (lane >> 4);
      T af[TI], bf[TJ];
#pragma unroll
      for (int a = 0; a < TI; ++a) af[a] = As[k][wm * WTM + a * 16 + (lane & 15)];
#pragma unroll
      for (int b = 0; b < TJ; ++b) bf[b] = Bs[k][wn * WTN + b * 16 + (lane & 15)];
#pragma unroll
      for (int a = 0; a < TI; ++a)
#pragma unroll
        for (int b = 0; b < TJ; ++b) acc[a][b] = mfma4(af[a], bf[b], acc[a][b]);
    }
    __syncthreads();
    if (kt + 1 < nk) {
      store();
      __syncthreads();
    }
  }

#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * WTM + a * 16 + dsub_row<T>(lane, r);
        const int col = n0 + wn * WTN + b * 16 + (lane & 15);
        if (row < p.M && col < p.N) {
          const size_t off = (size_t)row * p.ldc + col;
          T v = p.alpha * acc[a][b][r];
          if (p.beta != T(0)) v += p.beta * gC[off];
          gC[off] = v;
        }
      }
}

template <typename T, int BM, int BN, bool AT, bool BT, bool HAD>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs<T> p) {
  gemm_body<T, BM, BN, AT, BT, HAD>(p, blockIdx.x, gridDim.x);
}


// ---------------------------------------------------------------------
// Direct-load tiles.  BM x BN tiles, WM x WN waves, k-steps of BKB bytes
// of k (128: 16 doubles or 32 floats), ST LDS stages of which ST - 1 are in
// flight while one is multiplied.  buffer_load_dwordx4 ... lds moves 16
// bytes a lane (V = 2 doubles or 4 floats) without staging registers; a
// lane past the end of K reads an offset outside the buffer's bound, which
// writes zeros, so K needs no multiple of the k-step.  Rows past the edge
// read a clamped in-range address and feed only elements that are not
// stored.  (The compiler waits for the new loads before the reads of the
// present stage; global_load_lds with the zeros from a branch does not, and
// measured the same or 2% slower: the other workgroups of the unit cover
// the wait.)
//
// What bounds it: the FP64 matrix instruction takes 64 cycles, so 16 of
// them (a 64 x 64 wave tile and 4 of k) leave ~1000 cycles for a few LDS
// reads; the loss is in waits.  So:
//   - one barrier per k-step, with a plain s_barrier (a fenced one would
//     wait for the loads of the next stages);
//   - few LDS reads without bank conflicts.  An operand contiguous along
//     its row index r is kept as [k][r]; one 16-byte read of a lane brings
//     V adjacent rows, which feed V different 16-row tiles (tile a of a
//     group of V holds rows V i + a, i = 0..15), so that a lane's results
//     are adjacent columns of C as well.  An operand contiguous along k is
//     kept as [r][k] with the 16-byte chunks of a row XORed by r: the 16
//     rows of a read then lie in 16 different chunks of the banks;
//   - the fragments of the next 4 of k are read before the products of the
//     present ones.
// Every tile form adds the products of one element in the order of k, four
// to an instruction, as the register-staged form does: a result depends
// neither on the tile form nor on the path.
//
// Measured on the MI355X (FP64): 4096^3 63-66 TFLOP/s with 64 x 64 tiles,
// 70.6 with 128 x 128 tiles of eight waves (66.5 at 4000^3, two rounds of
// 512); the register-to-LDS form before it reached 49 with a Hadamard pair
// and 59 without.  500 x 400 x 500: 46 us -> 22 us with 64 x 64 tiles (56
// workgroups), 10.5 us with 32 x 32 tiles (208 workgroups, four stages in
// flight).  FP32: 1000^3 62 us -> 26 us.
//
// Split K: a tile at or past nfull is computed by `slices` workgroups.
// Each stores its partial tile device-coherently and then counts itself;
// the last one sums the partial tiles in slice order, whichever it is, so
// the result is reproducible, and sets the counter back to zero.  Nobody
// waits for anybody.
namespace {
template <typename T>
struct Chunk;
template <>
struct Chunk<double> {
  static constexpr int V = 2;
  typedef double vec __attribute__((ext_vector_type(2)));
};
template <>
struct Chunk<float> {
  static constexpr int V = 4;
  typedef float vec __attribute__((ext_vector_type(4)));
};
typedef __attribute__((address_space(3))) void* lds_vptr;
}  // namespace

// Tile forms.
struct TileBig {    // 128 x 128, eight waves of 32 x 64, two workgroups per compute unit
  static constexpr int BM = 128, BN = 128, WM = 4, WN = 2, BKB = 128, ST = 2, WPE = 4;
};
struct TileMid {    // 64 x 64, four waves of 32 x 32, four workgroups per compute unit (32 KB of LDS each and a flag)
  static constexpr int BM = 64, BN = 64, WM = 2, WN = 2, BKB = 128, ST = 2, WPE = 4;
};
struct TileSmall {  // 32 x 32, four waves of 16 x 16, long k-steps, four stages
  static constexpr int BM = 32, BN = 32, WM = 2, WN = 2, BKB = 256, ST = 4, WPE = 2;
};
struct TileLong {   // 32 x 32 with twice the k-step: few tiles, long K, both operands contiguous along their rows
  static constexpr int BM = 32, BN = 32, WM = 2, WN = 2, BKB = 512, ST = 2, WPE = 2;
};

// Chunk c of row r of a k-contiguous operand lies in slot c ^ chunk_swizzle(r)
// of the row (8 or 16 chunks: half or the whole of the 64 banks).
template <int KP>
__device__ __forceinline__ int chunk_swizzle(int r) {
  static_assert(KP == 8 || KP == 16, "128- or 256-byte rows");
  return KP == 8 ? (r >> 1) & 7 : r & 15;
}

// The share of one thread in the loads of an operand tile of R rows.
template <typename T, int R, int BK, bool KC, int NT>
struct OperandLoad {
  static constexpr int V = Chunk<T>::V;
  static constexpr int KP = BK / V;  // 16-byte chunks of one row along k
  static constexpr int PER = R * BK / V / NT;
  static_assert(PER * NT * V == R * BK, "whole loads");
  uint32_t off[PER];
  int kof[PER];
  __device__ __forceinline__ void init(int r0, int rows, int ld, int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int c = i * NT + tid;
      if constexpr (KC) {
        const int r = c / KP, kp = (c % KP) ^ chunk_swizzle<KP>(r);
        off[i] = (uint32_t)(((size_t)(min(r0 + r, rows - 1) - r0) * ld + kp * V) * sizeof(T));
        kof[i] = kp * V;
      } else {
        const int k = c / (R / V), rv = c % (R / V);
        off[i] = (uint32_t)(((size_t)k * ld + (min(r0 + rv * V, (rows - 1) / V * V) - r0)) * sizeof(T));
        kof[i] = k;
      }
    }
  }
  // base: the operand at (r0, k0); left: the k's from k0 on (past them: zeros)
  __device__ __forceinline__ void issue(const T* base, int left, T* stage, int w) const {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, 0x7ffffff0, 0x00020000);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_vptr)(stage + (size_t)(i * NT + w * 64) * V), 16,
                                               kof[i] < left ? off[i] : 0xfffffff0u, 0, 0, 0);
  }
};

// The fragments of one operand for the 16-row tiles of a wave.
template <typename T, int R, int BK, bool KC, int TI>
struct OperandFrag {
  static constexpr int V = Chunk<T>::V;
  static constexpr int F = KC ? 1 : (TI < V ? TI : V);  // tiles fed by one read
  typedef T vr __attribute__((ext_vector_type(F)));
  // k's 4 q .. 4 q + 3 of the stage, rows from r0 on
  static __device__ __forceinline__ void read(T f[TI], const T* stage, int q, int r0, int lane) {
    const int k = 4 * q + (lane >> 4), l = lane & 15;
    if constexpr (KC) {
      constexpr int KP = BK / V;
#pragma unroll
      for (int a = 0; a < TI; ++a) {
        const int r = r0 + 16 * a + l;
        f[a] = stage[(r * KP + ((k / V) ^ chunk_swizzle<KP>(r))) * V + k % V];
      }
    } else {
#pragma unroll
      for (int a = 0; a < TI; a += F) {
        const vr v = *(const vr*)(stage + k * R + r0 + 16 * a + F * l);
#pragma unroll
        for (int i = 0; i < F; ++i) f[a + i] = v[i];
      }
    }
  }
  // row (from r0) of index i (0..15) of tile a
  static __device__ __forceinline__ int row(int a, int i) { return a / F * (16 * F) + i * F + a % F; }
};

template <typename T, typename C, bool AT, bool BT>
__device__ __forceinline__ void gemm_tile_body(const GemmArgs<T>& p, int local, T* lds, int& last) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BM = C::BM, BN = C::BN, ST = C::ST, NT = 64 * C::WM * C::WN, V = Chunk<T>::V;
  constexpr int BK = C::BKB / (int)sizeof(T);
  constexpr int WTM = BM / C::WM, WTN = BN / C::WN, TI = WTM / 16, TJ = WTN / 16;
  constexpr int SA = BM * BK, STG = SA + BN * BK;
  typedef typename Acc4<T>::type acc_t;
  typedef OperandLoad<T, BM, BK, !AT, NT> LoadA;
  typedef OperandLoad<T, BN, BK, BT, NT> LoadB;
  typedef OperandFrag<T, BM, BK, !AT, TI> FragA;
  typedef OperandFrag<T, BN, BK, BT, TJ> FragB;
  constexpr int LPS = LoadA::PER + LoadB::PER;  // loads of a wave per stage
  // fragments held: of the present 4 of k and of the next D - 1, so that a
  // read has some 200 cycles of products to return in
  constexpr int D = TI * TJ >= 4 ? 2 : BK / 4 < 8 ? BK / 4 : 8;
  if (p.done && *p.done) return;
  if (p.gate && *p.gate != p.want) return;
  const int tiles_n = (p.N + BN - 1) / BN, tiles_m = (p.M + BM - 1) / BM;
  const bool lower = p.lower && p.M == p.N;
  const int ntiles = lower ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int nfull = p.slices > 1 ? p.nfull : ntiles;
  // unsplit tiles first, then the slices of the others
  int tile, slice = 0, kbeg = 0, kend = p.K;
  if (local < nfull) {
    tile = p.kdiag ? local : xcd_remap(local, nfull);
  } else {
    tile = nfull + (local - nfull) / p.slices;
    slice = (local - nfull) % p.slices;
    kbeg = gemm_slice_k(p.K, p.slices, slice);
    kend = gemm_slice_k(p.K, p.slices, slice + 1);
  }
  int m0, n0;
  if (lower) {
    // the lower tiles in row order (row r holds r + 1)
    int r = (int)((sqrtf(8.f * (float)tile + 1.f) - 1.f) * 0.5f);
    while ((r + 1) * (r + 2) / 2 <= tile) ++r;
    while (r * (r + 1) / 2 > tile) --r;
    m0 = r * BM;
    n0 = (tile - r * (r + 1) / 2) * BN;
  } else if (p.kdiag) {
    // the columns with the longest sums first
    m0 = tile % tiles_m * BM;
    n0 = tile / tiles_m * BN;
  } else {
    int tm, tn;
    grouped_tile(tile, tiles_m, tiles_n, 8, tm, tn);
    m0 = tm * BM;
    n0 = tn * BN;
  }
  if (p.kdiag) kbeg = n0 & ~63;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int wm = w / C::WN, wn = w % C::WN;

  LoadA la;
  LoadB lb;
  la.init(m0, p.M, p.lda, tid);
  lb.init(n0, p.N, p.ldb, tid);
  const size_t strideA = AT ? (size_t)BK * p.lda : BK, strideB = BT ? BK : (size_t)BK * p.ldb;
  const T* gA = AT ? p.A + (size_t)kbeg * p.lda + m0 : p.A + (size_t)m0 * p.lda + kbeg;
  const T* gB = BT ? p.B1 + (size_t)n0 * p.ldb + kbeg : p.B1 + (size_t)kbeg * p.ldb + n0;
  const int nk = (kend - kbeg + BK - 1) / BK;
  int left = kend - kbeg, wst = 0;
  // past the last k-tile the loads bring zeros into a stage nobody reads,
  // which keeps the wait counts constant
  auto issue = [&]() {
    la.issue(gA, left, lds + wst * STG, w);
    lb.issue(gB, left, lds + wst * STG + SA, w);
    left -= BK;
    if (left > 0) {
      gA += strideA;
      gB += strideB;
    }
    wst = wst == ST - 1 ? 0 : wst + 1;
  };

  acc_t acc[TI][TJ];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < ST - 1; ++i) issue();
  int rst = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // this wave's loads of k-tile kt have landed; the barrier makes every
    // wave's visible and ends all reads of the stage that is loaded next
    __asm__ volatile("s_waitcnt vmcnt(%0)" ::"n"((ST - 2) * LPS) : "memory");
    __builtin_amdgcn_s_barrier();
    __asm__ volatile("" ::: "memory");
    issue();
    const T* sA = lds + rst * STG;
    const T* sB = sA + SA;
    rst = rst == ST - 1 ? 0 : rst + 1;
    T af[D][TI], bf[D][TJ];
#pragma unroll
    for (int q = 0; q < D - 1; ++q) {
      FragA::read(af[q], sA, q, wm * WTM, lane);
      FragB::read(bf[q], sB, q, wn * WTN, lane);
    }
#pragma unroll
    for (int q = 0; q < BK / 4; ++q) {
      if (q + D - 1 < BK / 4) {
        FragA::read(af[(q + D - 1) % D], sA, q + D - 1, wm * WTM, lane);
        FragB::read(bf[(q + D - 1) % D], sB, q + D - 1, wn * WTN, lane);
      }
      if (D > 2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < TI; ++a)
#pragma unroll
        for (int b = 0; b < TJ; ++b) acc[a][b] = mfma4(af[q % D][a], bf[q % D][b], acc[a][b]);
      if (D > 2) __builtin_amdgcn_sched_barrier(0);
    }
  }
  // no load into LDS may outlive the workgroup
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");

  if (local >= nfull) {
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    constexpr int SC1 = 16;  // cache policy: device-coherent
    constexpr int W16 = 4 * (int)sizeof(T) / 16, TILE = BM * BN;
    T* part = (T*)p.part + (size_t)(tile - nfull) * p.slices * TILE;
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(part + (size_t)slice * TILE), (short)0,
                                                                  TILE * (int)sizeof(T), 0x00020000);
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b) {
        struct Q { u4 v[W16]; };
        const Q x = __builtin_bit_cast(Q, acc[a][b]);
#pragma unroll
        for (int h = 0; h < W16; ++h)
          __builtin_amdgcn_raw_buffer_store_b128(x.v[h], rs, (((a * TJ + b) * W16 + h) * NT + tid) * 16, 0, SC1);
      }
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* cnt = p.cnt + (tile - nfull);
    if (tid == 0) {
      last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == p.slices - 1;
      if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last) return;
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
    for (int z = 0; z < p.slices; ++z) {
      rs = __builtin_amdgcn_make_buffer_rsrc((void*)(part + (size_t)z * TILE), (short)0, TILE * (int)sizeof(T),
                                             0x00020000);
#pragma unroll
      for (int a = 0; a < TI; ++a)
#pragma unroll
        for (int b = 0; b < TJ; ++b) {
          struct Q { u4 v[W16]; } x;
#pragma unroll
          for (int h = 0; h < W16; ++h)
            x.v[h] = __builtin_amdgcn_raw_buffer_load_b128(rs, (((a * TJ + b) * W16 + h) * NT + tid) * 16, 0, SC1);
          acc[a][b] += __builtin_bit_cast(acc_t, x);
        }
    }
  }

  // C = alpha A B + beta C, its copy, and the Hadamard products that the
  // next products of the sweep take as their operand
  const gptr<T> gC = as_global(p.C), gC2 = as_global(p.C2);
  const gptr<const T> gH1 = as_global(p.H1), gH2 = as_global(p.H2);
  const gptr<T> gP1 = as_global(p.P1), gP2 = as_global(p.P2);
  constexpr int FB = FragB::F;
  typedef T vb __attribute__((ext_vector_type(FB)));
  if (AT && p.mirror && m0 != n0) {
    // the transposed tile above the diagonal (AT: a lane's tiles of A are
    // adjacent rows of C)
    constexpr int FA = FragA::F;
    typedef T va __attribute__((ext_vector_type(FA)));
#pragma unroll
    for (int b = 0; b < TJ; ++b) {
      const int col = n0 + wn * WTN + FragB::row(b, lane & 15);
      if (col >= p.N) continue;
#pragma unroll
      for (int a = 0; a < TI; a += FA)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + wm * WTM + FragA::row(a, dsub_row<T>(lane, r));
          const size_t off = (size_t)col * p.ldc + row;
          va v;
#pragma unroll
          for (int i = 0; i < FA; ++i) v[i] = p.alpha * acc[a + i][b][r];
          if (p.vec && row + FA <= p.M) {
            *(gptr<va>)(gC + off) = v;
          } else {
#pragma unroll
            for (int i = 0; i < FA; ++i)
              if (row + i < p.M) gC[off + i] = v[i];
          }
        }
    }
  }
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = m0 + wm * WTM + FragA::row(a, dsub_row<T>(lane, r));
      if (row >= p.M) continue;
#pragma unroll
      for (int b = 0; b < TJ; b += FB) {
        const int col = n0 + wn * WTN + FragB::row(b, lane & 15);
        const size_t off = (size_t)row * p.ldc + col;
        vb v;
#pragma unroll
        for (int i = 0; i < FB; ++i) v[i] = p.alpha * acc[a][b + i][r];
        if (FB > 1 && p.vec && col + FB <= p.N) {
          if (p.beta != T(0)) v += p.beta * *(const gptr<const vb>)(gC + off);
          *(gptr<vb>)(gC + off) = v;
          if (p.C2) *(gptr<vb>)(gC2 + off) = v;
          if (p.P1) *(gptr<vb>)(gP1 + off) = v * (p.H1 == p.C ? v : *(const gptr<const vb>)(gH1 + off));
          if (p.P2) *(gptr<vb>)(gP2 + off) = v * (p.H2 == p.C ? v : *(const gptr<const vb>)(gH2 + off));
        } else {
#pragma unroll
          for (int i = 0; i < FB; ++i) {
            if (col + i >= p.N) continue;
            const size_t o = off + i;
            T x = v[i];
            if (p.beta != T(0)) x += p.beta * gC[o];
            gC[o] = x;
            if (p.C2) gC2[o] = x;
            if (p.P1) gP1[o] = x * (p.H1 == p.C ? x : gH1[o]);
            if (p.P2) gP2[o] = x * (p.H2 == p.C ? x : gH2[o]);
          }
        }
      }
    }
#endif
}

// Bytes of LDS of a tile form.
template <typename C>
constexpr int tile_lds() {
  return C::ST * (C::BM + C::BN) * C::BKB;
}

template <typename T, typename C, bool AT, bool BT>
__global__ __launch_bounds__(64 * C::WM * C::WN, C::WPE) void gemm_tile_kernel(GemmArgs<T> p) {
  __shared__ __attribute__((aligned(1024))) char lds[tile_lds<C>()];
  __shared__ int last;
  gemm_tile_body<T, C, AT, BT>(p, blockIdx.x, (T*)lds, last);
}
// Two independent products in one launch: workgroups below n1 take p (form
// C1, op(A) = A^T), the others q (form C2, op(B) = B^T).
template <typename T, typename C1, typename C2>
__global__ __launch_bounds__(256, 2) void gemm_tile_two_kernel(GemmArgs<T> p, GemmArgs<T> q, int n1) {
  static_assert(C1::WM * C1::WN == 4 && C2::WM * C2::WN == 4, "256 threads");
  __shared__ __attribute__((aligned(1024))) char lds[tile_lds<C1>() > tile_lds<C2>() ? tile_lds<C1>() : tile_lds<C2>()];
  __shared__ int last;
  if ((int)blockIdx.x < n1) {
    __builtin_amdgcn_s_setprio(3);  // the launch ends with these
    gemm_tile_body<T, C1, true, false>(p, blockIdx.x, (T*)lds, last);
  } else {
    gemm_tile_body<T, C2, false, true>(q, blockIdx.x - n1, (T*)lds, last);
  }
}
// Grouped form: workgroup -> (problem, local unit) through the prefix sums.
template <typename T, typename C, bool AT, bool BT>
__global__ __launch_bounds__(64 * C::WM * C::WN, C::WPE) void gemm_tile_group_kernel(const GemmArgs<T>* tab,
                                                                                      const int* offs, int nprob) {
  __shared__ __attribute__((aligned(1024))) char lds[tile_lds<C>()];
  __shared__ int last;
  int pid = 0;
  while (pid + 1 < nprob && (int)blockIdx.x >= offs[pid + 1]) ++pid;
  const GemmArgs<T> p = tab[pid];
  gemm_tile_body<T, C, AT, BT>(p, blockIdx.x - offs[pid], (T*)lds, last);
}

template <typename T>
bool gemm_tile_ok(const GemmArgs<T>& g, bool a_t, bool b_t) {
  constexpr int V = Chunk<T>::V;
  auto al16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  // 32-bit offsets inside a tile, and whole 16-byte chunks along the
  // contiguous index: along k, K itself; along the rows, the row length
  // (the last chunk of a row may reach past M or N, not past lda or ldb)
  const long span = 128L * (g.lda > g.ldb ? g.lda : g.ldb) * (long)sizeof(T);
  return g.M > 0 && g.N > 0 && g.K > 0 && !g.B2 && g.lda % V == 0 && g.ldb % V == 0 && span < (1L << 31) &&
         (a_t ? (g.M + V - 1) / V * V <= g.lda : g.K % V == 0) &&
         (b_t ? g.K % V == 0 : (g.N + V - 1) / V * V <= g.ldb) && al16(g.A) && al16(g.B1);
}
template bool gemm_tile_ok<double>(const GemmArgs<double>&, bool, bool);
template bool gemm_tile_ok<float>(const GemmArgs<float>&, bool, bool);

template <typename T>
void gemm_set_vec(GemmArgs<T>& g) {
  const uintptr_t all = (uintptr_t)g.C | (uintptr_t)g.C2 | (uintptr_t)g.H1 | (uintptr_t)g.P1 | (uintptr_t)g.H2 |
                        (uintptr_t)g.P2;
  g.vec = (all & 15) == 0 && g.ldc % Chunk<T>::V == 0;
}
template void gemm_set_vec<double>(GemmArgs<double>&);
template void gemm_set_vec<float>(GemmArgs<float>&);

// Units (workgroups) of g in tile form bm.
template <typename T>
int gemm_units(const GemmArgs<T>& g, int bm) {
  const int t = gemm_tile_count(g.M, g.N, bm, g.lower);
  return g.slices > 1 ? g.nfull + (t - g.nfull) * g.slices : t;
}
template int gemm_units<double>(const GemmArgs<double>&, int);
template int gemm_units<float>(const GemmArgs<float>&, int);

// K slices of one product, from its own shape alone (a problem gives the
// same bits alone and in any group).
//   - At least 256 tiles of 64: the tiles past a whole number per compute
//     unit are split, so that the last round is shared by all units
//     (800 x 4000 x 4000: 819 = 3 x 256 + 51 tiles, 51 x 5 slices).
//   - Fewer: all of its tiles, into as many slices of at least 128 k as
//     give 256 workgroups of 32 x 32 tiles (100 x 400 x 500: 52 tiles).
// FP64 only: the sums of an FP32 plan keep the one order of k, since its
// factors would follow another order's rounding by some 1e-6.
template <typename T>
void gemm_plan_slices(GemmArgs<T>& g) {
  const int t64 = gemm_tile_count(g.M, g.N, 64, g.lower);
  g.slices = 1;
  g.nfull = 0;
  if (sizeof(T) == 4) return;
  if (t64 >= 256) {
    const int rest = t64 % 256;
    if (!rest) return;
    int s = 256 / rest;
    s = s < g.K / 256 ? s : g.K / 256;
    if (s > 8) s = 8;
    if (s < 2) return;
    g.nfull = t64 - rest;
    g.slices = s;
    return;
  }
  const int t32 = gemm_tile_count(g.M, g.N, 32, g.lower);
  int s = 256 / t32;
  s = s < g.K / 128 ? s : g.K / 128;
  if (s > 8) s = 8;
  if (s >= 2) g.slices = s;
}
template void gemm_plan_slices<double>(GemmArgs<double>&);
template void gemm_plan_slices<float>(GemmArgs<float>&);

static int g_tile_force = 0;  // host side, tests only: 0 the rule decides
int set_tile_force(int bm) {
  const int prev = g_tile_force;
  g_tile_force = bm == 32 || bm == 64 || bm == 128 ? bm : 0;
  return prev;
}
int get_tile_force() { return g_tile_force; }

// Tile form of a launch.  A split product with unsplit tiles runs in the
// form its split is made for (64); otherwise the largest form that gives
// every compute unit work:
//   - 32 below 256 tiles of 64 (a 64-tile alone on its unit waits for its
//     loads; 500 x 400 x 500: 22 us against 10.5 us);
//   - 128 where two full rounds of it exist and its last round wastes less
//     than its higher rate gives (4000 x 4000: 1024 tiles of 128 are four
//     for each unit, 66.5 against 62 TFLOP/s; 1920 x 15360: 1800 are eight
//     for some units, 62 against 64).
template <typename T>
int gemm_tile_form(const std::vector<GemmArgs<T>>& v) {
  long t64 = 0, t128 = 0;
  bool tail = false, split = false;
  for (auto& g : v) {
    t64 += gemm_tile_count(g.M, g.N, 64, g.lower);
    t128 += gemm_tile_count(g.M, g.N, 128, g.lower);
    split = split || g.slices > 1;
    tail = tail || (g.slices > 1 && g.nfull > 0);
  }
  if (g_tile_force && !tail) return g_tile_force;
  if (t64 < 256) return 32;
  if (tail || split || t128 < 512) return 64;
  return 4.0 * ((t128 + 255) / 256) / 1.06 < (double)((t64 + 255) / 256) ? 128 : 64;
}
template int gemm_tile_form<double>(const std::vector<GemmArgs<double>>&);
template int gemm_tile_form<float>(const std::vector<GemmArgs<float>>&);

template <typename T, typename C>
static void launch_tile_group(hipStream_t s, const GemmArgs<T>* tab, const int* offs, int nprob, int units, bool at,
                              bool bt) {
  const dim3 grid(units), block(64 * C::WM * C::WN);
  if (at && !bt) hipLaunchKernelGGL((gemm_tile_group_kernel<T, C, true, false>), grid, block, 0, s, tab, offs, nprob);
  else if (!at && !bt)
    hipLaunchKernelGGL((gemm_tile_group_kernel<T, C, false, false>), grid, block, 0, s, tab, offs, nprob);
  else hipLaunchKernelGGL((gemm_tile_group_kernel<T, C, false, true>), grid, block, 0, s, tab, offs, nprob);
}

template <typename T>
void gemm_group(hipStream_t s, const GemmArgs<T>* tab, const int* offs, int nprob, int units, bool a_t, bool b_t,
                int bm) {
  if (units <= 0) return;
  if (bm == 128) launch_tile_group<T, TileBig>(s, tab, offs, nprob, units, a_t, b_t);
  else if (bm == 64) launch_tile_group<T, TileMid>(s, tab, offs, nprob, units, a_t, b_t);
  else launch_tile_group<T, TileSmall>(s, tab, offs, nprob, units, a_t, b_t);
}
template void gemm_group<double>(hipStream_t, const GemmArgs<double>*, const int*, int, int, bool, bool, int);
template void gemm_group<float>(hipStream_t, const GemmArgs<float>*, const int*, int, int, bool, bool, int);

template <typename T, typename C>
static void launch_tile_single(hipStream_t s, const GemmArgs<T>& a, bool at, bool bt) {
  const dim3 grid(gemm_units(a, C::BM)), block(64 * C::WM * C::WN);
  if (at && bt) hipLaunchKernelGGL((gemm_tile_kernel<T, C, true, true>), grid, block, 0, s, a);
  else if (at) hipLaunchKernelGGL((gemm_tile_kernel<T, C, true, false>), grid, block, 0, s, a);
  else if (bt) hipLaunchKernelGGL((gemm_tile_kernel<T, C, false, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gemm_tile_kernel<T, C, false, false>), grid, block, 0, s, a);
}

template <typename T>
static void launch_staged(hipStream_t s, const GemmArgs<T>& a, bool at, bool bt, bool had) {
  const dim3 grid(gemm_tile_count(a.M, a.N, 64)), block(256);
#define THCCP_GEMM_CASE(AT_, BT_, HAD_)                                                 \
  if (at == AT_ && bt == BT_ && had == HAD_) {                                          \
    hipLaunchKernelGGL((gemm_kernel<T, 64, 64, AT_, BT_, HAD_>), grid, block, 0, s, a); \
    return;                                                                             \
  }
  THCCP_GEMM_CASE(false, false, false)
  THCCP_GEMM_CASE(true, false, false)
  THCCP_GEMM_CASE(false, false, true)
  THCCP_GEMM_CASE(true, false, true)
  THCCP_GEMM_CASE(false, true, false)
  THCCP_GEMM_CASE(true, true, false)
#undef THCCP_GEMM_CASE
}

template <typename T>
static void gemm_dispatch(hipStream_t s, GemmArgs<T> a, bool at, bool bt) {
  if (a.M <= 0 || a.N <= 0) return;
  if (!gemm_tile_ok(a, at, bt)) {
    launch_staged<T>(s, a, at, bt, a.B2 != nullptr);
    return;
  }
  gemm_set_vec(a);
  const int bm = gemm_tile_form<T>({a});
  if (bm == 128) launch_tile_single<T, TileBig>(s, a, at, bt);
  else if (bm == 64) launch_tile_single<T, TileMid>(s, a, at, bt);
  else launch_tile_single<T, TileSmall>(s, a, at, bt);
}

void gemm_f64(hipStream_t s, const GemmF64& g) {
  GemmArgs<double> a{g.M, g.N, g.K, g.A, g.lda, g.B1, g.B2, g.ldb, g.C, g.ldc, nullptr, g.alpha, g.beta, nullptr};
  gemm_dispatch<double>(s, a, g.a_t, g.b_t);
}

// dW = A^T B (M x N, few tiles, long K) and dX = C D^T.  The 16 x 16 tiles
// of dW are chains of K / 4 dependent products (their order of K is kept),
// so only 64 workgroups run; at 256 x 256 x 8192 that is 64 us with the
// LDS reads eight products ahead (84 us one product ahead), beside the other
// product (17 us alone at 8192 x 256 x 256) 78 us.
void gemm_f32_two(hipStream_t s, const GemmF32& g, const GemmF32& h) {
  GemmArgs<float> a{g.M, g.N, g.K, g.A, g.lda, g.B1, g.B2, g.ldb, g.C, g.ldc, nullptr, g.alpha, g.beta, nullptr};
  GemmArgs<float> b{h.M, h.N, h.K, h.A, h.lda, h.B1, h.B2, h.ldb, h.C, h.ldc, nullptr, h.alpha, h.beta, nullptr};
  if (!g.a_t || g.b_t || h.a_t || !h.b_t || !gemm_tile_ok(a, true, false) || !gemm_tile_ok(b, false, true)) {
    gemm_f32(s, g);
    gemm_f32(s, h);
    return;
  }
  gemm_set_vec(a);
  gemm_set_vec(b);
  const int n1 = gemm_units(a, TileLong::BM), n2 = gemm_units(b, TileMid::BM);
  hipLaunchKernelGGL((gemm_tile_two_kernel<float, TileLong, TileMid>), dim3(n1 + n2), dim3(256), 0, s, a, b, n1);
}

void syrk_f64(hipStream_t s, int n, int K, const double* X, int ld, double* C, int ldc) {
  GemmArgs<double> a{n, n, K, X, ld, X, nullptr, ld, C, ldc, nullptr, 1.0, 0.0, nullptr};
  if (gemm_tile_ok(a, true, false)) {
    a.lower = 1;
    a.mirror = 1;
  }
  gemm_dispatch<double>(s, a, true, false);
}

void gemm_f32(hipStream_t s, const GemmF32& g) {
  GemmArgs<float> a{g.M, g.N, g.K, g.A, g.lda, g.B1, g.B2, g.ldb, g.C, g.ldc, nullptr, g.alpha, g.beta, nullptr};
  gemm_dispatch<float>(s, a, g.a_t, g.b_t);
}

}  // namespace thccp
