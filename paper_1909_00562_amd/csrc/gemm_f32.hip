// fp32 matrix products for the AS_F32 path (fp32 operands, products summed in
// fp64 so that each output is rounded once; fp64 matrix cores, LDS tiled), the
// split-K combine kernel shared with the bf16 path, and the tile planner.
#include <type_traits>

#include "common.h"
#include "db_reduce_dev.h"
#include "gemm.h"

namespace asx {

struct GemmDevF {
  const float* A[kMaxSeg];
  const float* B[kMaxSeg];
  int64_t lda, ldb, sA, sB;   // the same for all segments, like K
  int K, nseg;
  int M, N;
  float* C;
  float* C_lo;
  float* C_dact;
  const int32_t* copy_pos;   // row n of C also goes to row copy_pos[n] of C_copy, and of C_dact there alone (or null)
  float* C_copy;
  int64_t ldc, sC;
  const float* bias;
  const float* gate;
  int64_t ldg;
  int act_tanh, accumulate;
  uint32_t drop_thr;
  float drop_scale;
  uint64_t drop_seed;
  int splits;
  float* partial;
  int kper;
  int tiles_n;
  const int32_t* M_dev;   // device-side row count / reduction length (or null), clamped to M / K[0]
  const int32_t* K_dev;
};

__device__ __forceinline__ int dev_bound_f(const int32_t* count, int bound) {
  if (!count) return bound;
  const int v = *count;
  return v < 0 ? 0 : (v < bound ? v : bound);
}

// ---- fp32 products on the fp64 matrix cores ------------------------------------------
// v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16] as doubles; accumulator register r of
// lane l is row 4 * r + l / 16, column l % 16.  Operands stay float in memory and in LDS (half the bytes) and are
// widened after the fragment read, which is exact; products and sums are fp64 as in scalar code, so an output is
// rounded once.  Which four reduction indices meet in one instruction is free as long as both operands agree: lane
// group q = l / 16 takes k = 4 q + j for instruction j, so a lane's four values are one 16-byte LDS read.
//
// Block: 256 threads as 2 x 2 waves, reduction tiles of FK, two LDS stages.  The next PF tiles are on their way in
// registers (PF = 4 at 32 x 32, where a tile is short against a load's latency and the registers are there; 2 at 64 x 64).
// LDS rows are padded to FLD floats: 16 rows at one k then start in 16 different groups of 4 banks.
//
// Large products are bound by the fp64 matrix rate: 61 TFLOP/s at 4096^3 (the vendor's fp64 product reaches 62 on the
// same part; the scalar fp64 form this replaced ran at 17).  Small ones are bound by the steps of one wave: 64 matrix
// cycles x 8, 16 conversions and a barrier per tile of a 32 x 32 block.  64 x 2048 x 512 in 4 splits: 55 -> 9.4 us.
constexpr int FK = 32;
constexpr int FLD = FK + 4;

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// ROWS x FK tiles of one operand: global -> registers -> LDS [row][k].  KC: the reduction index is contiguous (a thread
// takes 4 consecutive k of a row); else a thread takes 4 consecutive rows of one k and scatters them.  Nothing branches
// (with branches around the loads the compiler waits for every load in flight at each of them): reduction indices
// outside the operand are read from `safe`, an address inside it, and stored as zero; rows outside are read from row 0
// and stay as they are, they only reach elements of C that are not stored.
// VEC: 16-byte loads; the host has checked that a group of four is all inside or all outside the operand.
template <int ROWS, bool KC, bool VEC>
struct F32Loader {
  static constexpr int NV = ROWS * FK / 4 / 256;
  const float* ptr[NV];
  int last[NV];   // !KC, scalar loads: rows behind the first of the four that are inside
  static __device__ __forceinline__ int row_of(int tid, int j) {
    return KC ? (tid >> 3) + 32 * j : (tid & 7) * 4 + 32 * j;
  }
  static __device__ __forceinline__ int k_of(int tid) { return KC ? (tid & 7) * 4 : tid >> 3; }
  // X: element (0, k0) of the rows; rows_left >= 1 of them are inside the operand
  __device__ __forceinline__ void init(const float* X, int64_t ld, int rows_left, int tid) {
    const int k = k_of(tid);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int row = row_of(tid, j) < rows_left ? row_of(tid, j) : 0;
      ptr[j] = KC ? X + (int64_t)row * ld + k : X + (int64_t)k * ld + row;
      last[j] = rows_left - 1 - row;
    }
  }
  __device__ __forceinline__ void load(f32x4_t (&r)[NV], const float* safe, int k_left, int64_t step, int tid) {
    const int k = k_of(tid);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      if constexpr (VEC) {
        r[j] = *reinterpret_cast<const f32x4_t*>(k < k_left ? ptr[j] : safe);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float* q = ptr[j] + (KC || e <= last[j] ? e : last[j]);
          r[j][e] = *(k + (KC ? e : 0) < k_left ? q : safe);
        }
      }
      ptr[j] += step;
    }
  }
  static __device__ __forceinline__ void store(const f32x4_t (&r)[NV], float* lds, int k_left, int tid) {
    const int k = k_of(tid);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int row = row_of(tid, j);
      f32x4_t v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = k + (KC && !VEC ? e : 0) < k_left ? r[j][e] : 0.f;
      if constexpr (KC) {
        *reinterpret_cast<f32x4_t*>(lds + row * FLD + k) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) lds[(row + e) * FLD + k] = v[e];
      }
    }
  }
};

template <int BM, int BN> constexpr int f32_smem_floats = 2 * (BM + BN) * FLD;
template <int BM, int BN, int PF, bool AKC, bool BKC, bool AVEC, bool BVEC>
__device__ __forceinline__ void gemm_f32_block(GemmDevF p, int pid, int z, float* smem) {
  constexpr bool COPY = false;
#include "gemm_f32_block.inc"
}
// (COPY: an instance of its own; as a branch of all of them it cost every product half a microsecond)
template <int BM, int BN, int PF, bool AKC, bool BKC, bool AVEC, bool BVEC, bool COPY>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmDevF p) {
  __shared__ __align__(16) float smem[f32_smem_floats<BM, BN>];
  int pid = blockIdx.x;
  const int z = blockIdx.z;
#include "gemm_f32_block.inc"
}

// Block tile edge (64 or 32) for nz products of M x N.  With four blocks and more on every compute unit the 64 x 64 tile
// is the faster one (4096^3: 2.25 ms = 61 TFLOP/s against 2.43 ms with 32 x 32); below that there are too few waves to
// cover the loads, and the four times as many blocks of 32 x 32 win by far: 1286 x 512 x 16000 0.70 -> 0.53 ms,
// 64 x 2048 x 512 28 -> 11 us.  (128 x 64 was never the fastest: 2.43 ms at 4096^3.)
static int f32_tile(int M, int N, int nz) {
  return (int64_t)((M + 63) / 64) * ((N + 63) / 64) * nz >= 1024 ? 64 : 32;
}

bool gemm_f32_small(int M, int N, int nz) { return f32_tile(M, N, nz) == 32; }

template <int BM, int BN, int PF, bool AKC, bool BKC>
static hipError_t launch_f32_tile(GemmDevF& d, int batch, bool avec, bool bvec, hipStream_t st) {
  d.tiles_n = (d.N + BN - 1) / BN;
  dim3 grid((d.M + BM - 1) / BM * d.tiles_n, 1, batch * d.splits);
#define ASX_F32_C(AV, BV, CP) hipLaunchKernelGGL((gemm_f32_kernel<BM, BN, PF, AKC, BKC, AV, BV, CP>), grid, dim3(256), 0, st, d)
#define ASX_F32(AV, BV)                                   \
  do {                                                    \
    if (AKC && BKC && d.copy_pos) ASX_F32_C(AV, BV, (AKC && BKC)); \
    else ASX_F32_C(AV, BV, false);                        \
  } while (0)
  if (d.copy_pos && !(AKC && BKC)) return hipErrorInvalidValue;
  if (avec && bvec) ASX_F32(true, true);
  else if (avec) ASX_F32(true, false);
  else if (bvec) ASX_F32(false, true);
  else ASX_F32(false, false);
#undef ASX_F32_C
#undef ASX_F32
  return hipGetLastError();
}
template <bool AKC, bool BKC>
static hipError_t launch_f32_oriented(GemmDevF& d, int batch, bool avec, bool bvec, hipStream_t st) {
  return f32_tile(d.M, d.N, batch * d.splits) == 64 ? launch_f32_tile<64, 64, 2, AKC, BKC>(d, batch, avec, bvec, st)
                                                    : launch_f32_tile<32, 32, 4, AKC, BKC>(d, batch, avec, bvec, st);
}

// checks of a product and its description for the kernels; avec, bvec: 16-byte loads of the operand
static hipError_t f32_describe(const GemmArgs& g, GemmDevF& d, bool& avec, bool& bvec) {
  if (g.M < 1 || g.N < 1 || g.batch < 1 || g.splits < 1 || g.c_bf16 || g.nseg < 1 || g.K[g.nseg - 1] < 1) return hipErrorInvalidValue;
  if (g.splits > 1 && (g.K[1] != 0 || g.partial == nullptr)) return hipErrorInvalidValue;
  if (g.splits > 1 && (g.C_dact || g.drop_thr)) return hipErrorInvalidValue;
  if (g.drop_thr && g.batch != 1) return hipErrorInvalidValue;
  if (g.copy_pos && (!g.C_copy || g.batch != 1 || g.splits != 1 || g.M_dev || g.accumulate)) return hipErrorInvalidValue;
  avec = bvec = true;
  for (int s = 0; s < kMaxSeg; ++s) {
    d.A[s] = reinterpret_cast<const float*>(g.A[s]);
    d.B[s] = reinterpret_cast<const float*>(g.B[s]);
    if (g.K[s] > 0) {
      if (g.lda[s] != g.lda[0] || g.ldb[s] != g.ldb[0] || g.sA[s] != g.sA[0] || g.sB[s] != g.sB[0] || g.K[s] != g.K[0] || s >= g.nseg)
        return hipErrorInvalidValue;
      // 16-byte loads: groups of four start aligned and do not straddle the operand's edge (a reduction length or row
      // count read on the device counts rows, which are the other index of the operands that use it)
      auto vec_ok = [&](const void* X, int64_t ld, int64_t stride, bool kc, int rows) {
        return !((ld | stride | (kc ? g.K[s] : rows)) & 3) && !(reinterpret_cast<uintptr_t>(X) & 15);
      };
      avec = avec && vec_ok(g.A[s], g.lda[s], g.sA[s], g.a_kc, g.M) && !(g.a_kc && g.K_dev) && !(!g.a_kc && g.M_dev);
      bvec = bvec && vec_ok(g.B[s], g.ldb[s], g.sB[s], g.b_kc, g.N) && !(g.b_kc && g.K_dev);
    }
  }
  d.lda = g.lda[0];
  d.ldb = g.ldb[0];
  d.sA = g.sA[0];
  d.sB = g.sB[0];
  d.K = g.K[0];
  d.nseg = g.nseg;
  d.M = g.M;
  d.N = g.N;
  d.C = reinterpret_cast<float*>(g.C);
  d.C_lo = reinterpret_cast<float*>(g.C_lo);
  d.C_dact = g.C_dact;
  d.copy_pos = g.copy_pos;
  d.C_copy = reinterpret_cast<float*>(g.C_copy);
  d.ldc = g.ldc;
  d.sC = g.sC;
  d.bias = reinterpret_cast<const float*>(g.bias);
  d.gate = g.gate;
  d.ldg = g.ldg;
  d.act_tanh = g.act_tanh;
  d.drop_thr = g.drop_thr;
  d.drop_scale = g.drop_scale;
  d.drop_seed = g.drop_seed;
  d.accumulate = g.accumulate;
  d.splits = g.splits;
  d.partial = g.partial;
  if (g.M_dev && g.batch != 1) return hipErrorInvalidValue;
  if (g.K_dev && g.K[1] != 0) return hipErrorInvalidValue;
  d.M_dev = g.M_dev;
  d.K_dev = g.K_dev;
  const int ktiles = (g.K[0] + FK - 1) / FK;
  d.kper = ((ktiles + g.splits - 1) / g.splits) * FK;
  if (g.splits > 1 && (int64_t)d.kper * (g.splits - 1) >= g.K[0]) return hipErrorInvalidValue;
  return hipSuccess;
}

hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t st) {
  GemmDevF d;
  bool avec, bvec;
  const hipError_t e = f32_describe(g, d, avec, bvec);
  if (e != hipSuccess) return e;
  if (g.a_kc && g.b_kc) return launch_f32_oriented<true, true>(d, g.batch, avec, bvec, st);
  if (g.a_kc && !g.b_kc) return launch_f32_oriented<true, false>(d, g.batch, avec, bvec, st);
  if (!g.a_kc && !g.b_kc) return launch_f32_oriented<false, false>(d, g.batch, avec, bvec, st);
  return hipErrorInvalidValue;  // (A strided, B contiguous) is not used by the path
}

// ---- several products in one launch: their blocks of 32 x 32 one product behind the other ----
template <bool AKC, bool BKC, bool AVEC, bool BVEC = AVEC> struct F32Member {
  GemmDevF d;
  int tiles, blocks;   // blocks: of the grid, a multiple of 8 so that a product's blocks keep their XCDs
  void set(const GemmDevF& dev, int batch) {
    d = dev;
    d.tiles_n = (d.N + 31) / 32;
    tiles = (d.M + 31) / 32 * d.tiles_n;
    blocks = (tiles * batch * d.splits + 7) / 8 * 8;
  }
  __device__ __forceinline__ void run(int id, int nz, float* smem) const {
    const int z = id / tiles;
    if (z < nz) gemm_f32_block<32, 32, 4, AKC, BKC, AVEC, BVEC>(d, id - z * tiles, z, smem);
  }
};
struct F32Sums {   // column sums of dlogits beside the products that read it
  DbReduce d;
  int blocks;
  __device__ __forceinline__ void run(int id, int, float* smem) const {
    if (id * kDbColumns < d.V) db_reduce_block<256>(d, id, smem);
  }
};
struct F32Counts {
  int nz[kMaxTogether];
};
template <int I, typename F, typename... R>
__device__ __forceinline__ void run_f32_member(int id, const F32Counts& n, float* smem, const F& f, const R&... rest) {
  if constexpr (sizeof...(R) > 0) {
    if (id >= f.blocks) return run_f32_member<I + 1>(id - f.blocks, n, smem, rest...);
  }
  f.run(id, n.nz[I], smem);
}
template <typename... M> __global__ __launch_bounds__(256) void gemm_f32_together_kernel(F32Counts n, M... m) {
  __shared__ __align__(16) float smem[f32_smem_floats<32, 32>];
  static_assert(sizeof(smem) >= kDbSmem, "the column sums' share");
  run_f32_member<0>(blockIdx.x, n, smem, m...);
}
template <typename... M> static hipError_t launch_f32_grid(const F32Counts& n, hipStream_t st, const M&... m) {
  int64_t blocks = 0;
  for (int64_t b : {(int64_t)m.blocks...}) blocks += b;
  if (blocks > (1 << 24)) return hipErrorNotSupported;
  hipLaunchKernelGGL(gemm_f32_together_kernel<M...>, dim3((unsigned)blocks), dim3(256), 0, st, n, m...);
  return hipGetLastError();
}
template <typename... M>
static hipError_t launch_f32_members(const GemmArgs* g, const GemmDevF* d, const DbReduce* sums, hipStream_t st, M... m) {
  F32Counts n{};
  int i = 0;
  ((m.set(d[i], g[i].batch), n.nz[i] = g[i].batch * g[i].splits, ++i), ...);
  if constexpr (sizeof...(M) == 2) {
    if (sums) return launch_f32_grid(n, st, m..., F32Sums{*sums, (sums->V + kDbColumns - 1) / kDbColumns});
  }
  return sums ? hipErrorNotSupported : launch_f32_grid(n, st, m...);
}
// VEC: 16-byte loads of every operand but, without VEC_LAST, the A of the last of three
template <bool VEC, bool VEC_LAST>
static hipError_t launch_f32_together_with(const GemmArgs* g, const GemmDevF* d, int n, const DbReduce* sums, hipStream_t st) {
  using TN = F32Member<false, false, VEC>;
  using NN = F32Member<true, false, VEC>;
  using NT = F32Member<true, true, VEC>;
  const bool nn = g[1].a_kc && !g[1].b_kc, nt = g[1].a_kc && g[1].b_kc;
  if constexpr (VEC == VEC_LAST) {
    bool tn = true;
    for (int i = 1; i < n; ++i) tn = tn && !g[i].a_kc && !g[i].b_kc;
    if (tn && n == 2) return launch_f32_members(g, d, sums, st, TN(), TN());
    if (tn && n == 3) return launch_f32_members(g, d, sums, st, TN(), TN(), TN());
    if (tn && n == 4) return launch_f32_members(g, d, sums, st, TN(), TN(), TN(), TN());
    if (n == 2 && nn) return launch_f32_members(g, d, sums, st, TN(), NN());
    if (n == 3 && nn && g[2].a_kc && !g[2].b_kc) return launch_f32_members(g, d, sums, st, TN(), NN(), NN());
  }
  if (n == 3 && nt && !g[2].a_kc && !g[2].b_kc)
    return launch_f32_members(g, d, sums, st, TN(), NT(), F32Member<false, false, VEC_LAST, VEC>());
  return hipErrorNotSupported;
}
// Products that all go to 32 x 32 tiles; hipErrorNotSupported for the other combinations.  A training step of 32 rows x 64 units x
// 1000 words, a launch each / the four groups: 105 / 87 us; of 1920 x 512 x 16000, whose products fill the chip: 1656 / 1650.
static hipError_t launch_gemm_f32_together(const GemmArgs* g, int n, const DbReduce* sums, hipStream_t st) {
  if (n < 2 || n > kMaxTogether || g[0].a_kc || g[0].b_kc) return hipErrorNotSupported;
  GemmDevF d[kMaxTogether];
  bool vec = true, vec_last = true;
  for (int i = 0; i < n; ++i) {
    bool avec, bvec;
    const hipError_t e = f32_describe(g[i], d[i], avec, bvec);
    if (e != hipSuccess) return e;
    if (g[i].copy_pos || !gemm_f32_small(g[i].M, g[i].N, g[i].batch * g[i].splits)) return hipErrorNotSupported;
    vec = vec && bvec && (avec || (i == 2 && n == 3));   // (source positions, the rows of the last A, are rarely a multiple of four)
    vec_last = vec_last && avec && bvec;
  }
  if (vec_last) return launch_f32_together_with<true, true>(g, d, n, sums, st);
  if (vec && n == 3 && g[1].b_kc) return launch_f32_together_with<true, false>(g, d, n, sums, st);
  return launch_f32_together_with<false, false>(g, d, n, sums, st);
}

// ---- split-K combine: C = epilogue(sum_s partial[b*splits+s]) in fixed order --
struct CombineDev {
  const float* partial;
  int splits, M, N;
  void *C, *C_lo;
  float* C_dact;
  int64_t ldc, sC;
  const void* bias;
  const float* gate;
  int64_t ldg;
  int act_tanh, accumulate;
  uint32_t drop_thr;
  float drop_scale;
  uint64_t drop_seed;
  const int32_t* M_dev;
  const int32_t* row_pos;   // row n of C is row row_pos[n] of the product, zeros where that is negative
  const int32_t* copy_pos;  // row n of C also goes to row copy_pos[n] of C_copy, and of C_dact there alone (or null)
  void* C_copy;
  int dyn_ktiles, dyn_blocks;
};

// Bound by memory: splits x 4 bytes read per element, 4 to 12 more for the gate and the outputs.  V columns per thread, the
// gate and up to four splits requested together, 16-byte accesses throughout.  12145 of 16384 rows x 2048, two splits, gate
// and remainder, back to their rows: 148 us behind the product that has just written the partial sums (an element at a time,
// and the rows in a pass of their own, 207 + 39), 102 with everything in memory (4.2 TB/s; a copy of as much 5.2); 4287 of 6400
// x 1024, three splits: 26.6 us (56 + 9), 27.0 from memory.  One split after the other instead of together: 238 and 46.
template <typename TIn, bool OUT_BF16, int V>
__global__ __launch_bounds__(256) void splitk_combine_kernel(CombineDev p) {
  constexpr int Q = V > 4 ? 4 : V;            // columns of a vector access
  typedef float vec_t __attribute__((ext_vector_type(Q)));
  const int64_t mn = (int64_t)p.M * p.N;      // extent of one partial
  const int Mv = dev_bound_f(p.M_dev, p.M);
  int splits = p.splits;
  if (p.dyn_ktiles > 0)   // the product chose its split from the row count: the same choice here
    splits = pp_dyn_splits(((Mv + 255) / 256) * ((p.N + 255) / 256), p.dyn_ktiles, splits, p.dyn_blocks);
  const int batch = blockIdx.y;
  const int64_t total = (int64_t)(p.row_pos ? p.M : Mv) * (p.N / V);   // groups of V columns
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    int row;
    if constexpr (V > 1) row = (int)((uint32_t)i / (uint32_t)(p.N / V));   // (the launcher has checked the range)
    else row = (int)(i / p.N);
    const int col = (int)(i - (int64_t)row * (p.N / V)) * V;
    const int src = p.row_pos ? p.row_pos[row] : row;   // rows >= Mv were not written
    const int64_t ci = (int64_t)batch * p.sC + (int64_t)row * p.ldc + col;
    auto get = [&](const float* from, float (&x)[V]) {
#pragma unroll
      for (int k = 0; k < V / Q; ++k) {
        const vec_t o = *reinterpret_cast<const vec_t*>(from + k * Q);
#pragma unroll
        for (int e = 0; e < Q; ++e) x[k * Q + e] = o[e];
      }
    };
    float v[V], dact[V], gate[V];
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = dact[e] = 0.f;
    if (src >= 0 && src < Mv) {
      const float* P = p.partial + (int64_t)batch * splits * mn + (int64_t)src * p.N + col;
      if (p.gate) get(p.gate + (int64_t)src * p.ldg + col, gate);   // ahead of the sums: in flight with them
      auto add = [&](auto count, const float* from) {               // `count` splits, requested together
        constexpr int S = decltype(count)::value;
        float x[S][V];
#pragma unroll
        for (int u = 0; u < S; ++u) get(from + (int64_t)u * mn, x[u]);
#pragma unroll
        for (int u = 0; u < S; ++u)
#pragma unroll
          for (int e = 0; e < V; ++e) v[e] += x[u][e];
      };
      int s = 0;
      for (; s + 4 <= splits; s += 4) add(std::integral_constant<int, 4>{}, P + (int64_t)s * mn);
      if ((splits - s) == 3) add(std::integral_constant<int, 3>{}, P + (int64_t)s * mn);
      else if ((splits - s) == 2) add(std::integral_constant<int, 2>{}, P + (int64_t)s * mn);
      else if ((splits - s) == 1) add(std::integral_constant<int, 1>{}, P + (int64_t)s * mn);
      if (p.bias)
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] += ld_elem<TIn>(reinterpret_cast<const TIn*>(p.bias), col + e);
      if (p.act_tanh)
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = tanhf(v[e]);
#pragma unroll
      for (int e = 0; e < V; ++e) dact[e] = 1.f - v[e] * v[e];
      if (p.drop_thr) {
        const uint64_t flat = (uint64_t)row * p.N + col;
        if constexpr (V >= 4) {   // N % 4 == 0: whole blocks of the generator
#pragma unroll
          for (int k = 0; k < V / 4; ++k) {
            uint32_t w[4];
            dropout_words4((flat >> 2) + k, p.drop_seed, w);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float sc = w[e] >= p.drop_thr ? p.drop_scale : 0.f;
              v[4 * k + e] *= sc;
              dact[4 * k + e] *= sc;
            }
          }
        } else {
          const float sc = dropout_mult(flat, p.drop_seed, p.drop_thr, p.drop_scale);
          v[0] *= sc;
          dact[0] *= sc;
        }
      }
      if (p.gate)
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] *= gate[e];
    }
    const int copy = p.copy_pos ? p.copy_pos[row] : -1;
    const int64_t cc = (int64_t)copy * p.ldc + col;
    auto put = [&](void* dst, int64_t at, const float (&x)[V]) {   // floats
#pragma unroll
      for (int k = 0; k < V / Q; ++k) {
        vec_t o;
#pragma unroll
        for (int e = 0; e < Q; ++e) o[e] = x[k * Q + e];
        *reinterpret_cast<vec_t*>(reinterpret_cast<float*>(dst) + at + k * Q) = o;
      }
    };
    if (p.C_dact && (copy >= 0 || !p.copy_pos)) put(p.C_dact, p.copy_pos ? cc : ci, dact);
    if constexpr (OUT_BF16) {
      uint32_t hi[V], lo[V];
#pragma unroll
      for (int e = 0; e < V; ++e) {
        hi[e] = f32_to_bf16_bits(v[e]);
        lo[e] = f32_to_bf16_bits(v[e] - bf16_bits_to_f32(hi[e]));
      }
      auto put16 = [&](void* dst, int64_t at, const uint32_t (&x)[V]) {
        uint16_t* d = reinterpret_cast<uint16_t*>(dst) + at;
        static_assert(V == 8, "16-byte stores");
        *reinterpret_cast<uint4*>(d) = make_uint4(x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16));
      };
      put16(p.C, ci, hi);
      if (copy >= 0) put16(p.C_copy, cc, hi);
      if (p.C_lo) put16(p.C_lo, ci, lo);
    } else {
      if (p.accumulate) {
        float x[V];
        get(reinterpret_cast<const float*>(p.C) + ci, x);
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] += x[e];
      }
      put(p.C, ci, v);
      if (copy >= 0) put(p.C_copy, cc, v);
      if (p.C_lo) {   // partial sums were already rounded to fp32
        const float z[V] = {};
        put(p.C_lo, ci, z);
      }
    }
  }
}

hipError_t launch_splitk_combine(const GemmArgs& g, bool in_bf16, hipStream_t st) {
  if (g.row_pos && (g.batch != 1 || g.accumulate || g.drop_thr || g.C_dact)) return hipErrorInvalidValue;
  if (g.copy_pos && (!g.C_copy || g.batch != 1 || g.accumulate || g.row_pos)) return hipErrorInvalidValue;
  CombineDev d;
  d.partial = g.partial;
  d.splits = g.splits;
  d.M = g.M;
  d.N = g.N;
  d.C = g.C;
  d.C_lo = g.C_lo;
  d.C_dact = g.C_dact;
  d.ldc = g.ldc;
  d.sC = g.sC;
  d.bias = g.bias;
  d.gate = g.gate;
  d.ldg = g.ldg;
  d.act_tanh = g.act_tanh;
  d.accumulate = g.accumulate;
  d.drop_thr = g.drop_thr;
  d.drop_scale = g.drop_scale;
  d.drop_seed = g.drop_seed;
  d.M_dev = g.M_dev;
  d.row_pos = g.row_pos;
  d.copy_pos = g.copy_pos;
  d.C_copy = g.C_copy;
  // a split chosen by the persistent kernel (dyn_split): its reduction tiles and its grid, as that launch had them
  d.dyn_ktiles = g.dyn_split ? (g.K[0] + 63) / 64 : 0;
  d.dyn_blocks = g.dyn_split ? pp_grid_blocks(((g.M + 255) / 256) * ((g.N + 255) / 256) * g.splits) : 0;
  // groups of V columns: every row of what is read and written starts on a whole vector, and the group's index fits 32 bits
  // for the division.  bf16 widths are multiples of 8.
  const int V = g.c_bf16 ? 8 : 4;
  auto al = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const bool vec = g.N % V == 0 && g.ldc % V == 0 && g.sC % V == 0 && al(g.partial) && al(g.C) && al(g.C_lo) && al(g.C_dact) && al(g.C_copy) &&
                   (!g.gate || (g.ldg % 4 == 0 && al(g.gate))) && (int64_t)g.M * g.N / V < (int64_t)1 << 32;
  int64_t blocks = ((int64_t)g.M * g.N / (vec ? V : 1) + 255) / 256;
  if (blocks > 1 << 17) blocks = 1 << 17;
  const dim3 grid((unsigned)blocks, g.batch);
#define ASX_COMBINE(TIN, BF, W) hipLaunchKernelGGL((splitk_combine_kernel<TIN, BF, W>), grid, dim3(256), 0, st, d)
  if (in_bf16) {
    if (!vec) return hipErrorInvalidValue;
    if (g.c_bf16) ASX_COMBINE(uint16_t, true, 8);
    else ASX_COMBINE(uint16_t, false, 4);
  } else if (vec) {
    ASX_COMBINE(float, false, 4);
  } else {
    ASX_COMBINE(float, false, 1);
  }
#undef ASX_COMBINE
  return hipGetLastError();
}

// ---- planner ----------------------------------------------------------------
// Cost model (seconds) that decides whether a bf16 product gets 256x256 tiles, and its reduction split then, on a
// 256-CU part: blocks run in rounds of `slots` (one 256x256 block or two 128x128 blocks per CU); a round costs the
// block's flops at the per-CU rate the kernel sustains plus a fixed prologue/epilogue; a split adds the round trip
// of its fp32 partial sums through HBM and one more launch.  The 128x128 rate is that of an earlier kernel: with the
// present one's it would draw products with several rounds of 256x256 tiles away from the kernel that is faster there.
static double plan_cost(int M, int N, int K, int batch, int tile, int splits) {
  const double cus = 256.0;
  const double rate = tile == 256 ? 3.9e12 : 1.35e12;      // flop/s of one resident block
  const double slots = tile == 256 ? cus : 2.0 * cus;
  const double fixed = tile == 256 ? 8e-6 : 5e-6;
  const double blocks = (double)((M + tile - 1) / tile) * ((N + tile - 1) / tile) * batch * splits;
  const double rounds = (double)(int64_t)((blocks + slots - 1) / slots);
  const double kblk = (double)((K + splits - 1) / splits);
  double t = rounds * (2.0 * tile * tile * kblk / rate + fixed);
  if (splits > 1) t += 2.0 * splits * (double)M * N * batch * 4.0 / 4e12 + 8e-6;
  return t;
}

// Microseconds of the kernels of gemm_tile.hip, from what they measure.  A split adds the round trip of its partial sums
// and a launch.
static double plan_split_us(int M, int N, int batch, int splits) {
  return splits > 1 ? 2.0 * splits * (double)M * N * batch * 4.0 / 4e6 + 4.5 : 0.0;
}
// 64 x 64: 0.26 us per reduction tile and compute unit however many blocks share it, 0.8 per block.  (1920 x 512 x 1024 NN
// 9.1 measured, 10.0 by this; 128 x 1024 x 3072 NT 14.5, 18.3; 2257 x 1000 x 1000 NN 19.3, 19.9; 1024 x 1024 x 6400 TN 30.8,
// 31.8; 6400 x 1024 x 3072 NT 73.3, 98.)
static double plan_us_64(int M, int N, int ktiles, int batch, int splits) {
  const int64_t blocks = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch * splits;
  return (double)((blocks + 255) / 256) * (0.26 * ((ktiles + splits - 1) / splits) + 0.8) + 5.0 +
         plan_split_us(M, N, batch, splits);
}
// 128 x 128: 0.7 us per reduction tile with a compute unit to itself, 1.05 with two blocks on one.  (2257 x 1000 x 1000 NN
// 18.1, 18.2; 6400 x 1024 x 1024 NN 23.5, 25.3, NT 22.8, 25.3; x 2048 NN 37.5, 42.1; 16000 x 512 x 1286 TN 28.0, 30.5; 1286 x
// 16000 x 512 NT 39.3, 39.7, the 256 x 256 kernel 35.2.)  These are the rates of the loop that read a tile's fragments first;
// the one that reads them between the matrix instructions takes 0.58 and 0.9.  They stand because the choices do: over 89
// sizes of 16 to 16000 in every form, with every tile and ten splits timed, the plan is 0.5 % behind the best on average and
// 9 % at most (48 x 376 x 8168 NN: 32 splits, 11.1 us, 16 10.2).
static double plan_us_128(int M, int N, int ktiles, int batch, int splits) {
  const int64_t blocks = (int64_t)((M + 127) / 128) * ((N + 127) / 128) * batch * splits;
  const int k = (ktiles + splits - 1) / splits;
  const double t = blocks <= 256 ? 0.7 * k + 1.5 : (double)((blocks + 511) / 512) * (1.05 * k + 3.0);
  return t + 5.5 + plan_split_us(M, N, batch, splits);
}

// 256 x 256, a round of blocks or less: 0.9 to 1.6 us per reduction tile, the more compute units share the memory and the
// power.  Its combine moves the partial sums at 5.7 TB/s, and 6.5 us at least.  (2048 x 2048 x 16384 TN in 4 splits 147
// measured, 140 by this; two of them in 2 splits 255, 242; 6144 x 512 x 6400 TN in 5 65, 67; 4096 x 1024 x 6400 TN in 4 73,
// 78: with 128 x 128 73 too, and less ahead of another product; 1280 x 1024 x 32000 NN in 12 100, 102; 3776 x 512 x 27403 NN
// in 8 135, 120; 4096^3 TN 116, 110.  plan_cost puts the first two at 187 and 325.)
static double plan_us_256(int M, int N, int ktiles, int batch, int splits) {
  const int64_t blocks = (int64_t)((M + 255) / 256) * ((N + 255) / 256) * batch * splits;
  const int k = (ktiles + splits - 1) / splits;
  return (0.9 + 0.7 * (double)blocks / 256.0) * k + 7.5 + (splits > 1 ? 8.0 * splits * M * N * batch / 5.7e6 + 6.5 : 0.0);
}

// A split's sum is rounded to fp32, an undivided one is fp64 to the end: at most one split per 256 reduction indices (by
// sixteens), 32 in all, and 768 blocks of 64 x 64, however many more the compute units could take.
static int f32_most_splits(int M, int N, int K, int batch) {
  const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch;
  if (tiles >= 384) return 1;
  const int slices = (K + 15) / 16;
  int64_t most = (768 + tiles - 1) / tiles;
  if (most > slices / 16) most = slices / 16;
  if (most > 32) most = 32;
  if (most <= 1) return 1;
  const int per = (int)((slices + most - 1) / most);
  return (slices + per - 1) / per;
}

GemmPlan gemm_plan(int M, int N, int K, int batch, bool bf16, bool allow_split, bool multi_segment, bool counted) {
  GemmPlan pl;
  pl.tile = kTile128;
  pl.splits = 1;
  if (!bf16) {
    if (multi_segment) allow_split = false;
    // fp32 path: split while there are fewer than ten 32 x 32 blocks per compute unit.  Measured (1 / 2 / 4 / 8 splits):
    // 1286 x 512 x 16000 531 / 507 / 453 / 431 us, 512 x 512 x 1920 35 / 32 / 31 / 33 us, 64 x 512 x 2048 36 / 23 / 16 /
    // 13 us; 16000 x 512 x 1286 (8000 blocks) only loses.
    const int64_t tiles = (int64_t)((M + 31) / 32) * ((N + 31) / 32) * batch;
    if (allow_split) {
      const int ktiles = (K + FK - 1) / FK;
      int64_t want = 2560 / tiles;
      const int most = f32_most_splits(M, N, K, batch);
      if (want > most) want = most;
      if (want > 1) {
        const int per = (int)((ktiles + want - 1) / want);
        pl.splits = (ktiles + per - 1) / per;
      }
    }
    return pl;
  }
  const int ktiles = (K + 63) / 64;
  double best = 1e30;
  for (int tile = 128; tile <= 256; tile += 128) {
    if (tile == 256 && (M < 192 || N < 192)) continue;   // most of a 256-row tile would be padding
    const int smax = allow_split ? (ktiles / 4 < 32 ? (ktiles / 4 > 1 ? ktiles / 4 : 1) : 32) : 1;
    for (int want = 1; want <= smax; ++want) {
      const int per = (ktiles + want - 1) / want;
      const int s = (ktiles + per - 1) / per;            // no empty split
      if (s != want) continue;
      if (tile == 256 && s > 1 && multi_segment) continue;
      const double c = plan_cost(M, N, K, batch, tile, s);
      if (c < best) {
        best = c;
        pl.tile = tile == 256 ? kTile256 : kTile128;
        pl.splits = s;
      }
    }
  }
  // Which of the two shapes of gemm_tile.hip, if they are faster than 256 x 256.  With more than a round of 256 x 256
  // tiles that kernel stays: it writes a tile while the next one is on its way, which the models leave out
  // (2257 x 32003 x 1000: 174 us, 231 with 128 x 128, 184 by the model).
  double now = 1e30;
  if (pl.tile == kTile256) {
    if ((int64_t)((M + 255) / 256) * ((N + 255) / 256) * batch * pl.splits > 256) return pl;
    // (A count takes whole tiles or reduction tiles out of the plan, fewer blocks the larger they are: smaller tiles win
    // earlier.  dlogits W_out over half of 800 rows, 1024 x 32000: a training step of 332 us, 377 with 256 x 256.)
    now = counted ? 0.9 * best * 1e6 : plan_us_256(M, N, ktiles, batch, pl.splits);
  }
  const int smax = allow_split ? (ktiles / 4 < 32 ? (ktiles / 4 > 1 ? ktiles / 4 : 1) : 32) : 1;
  for (int want = 1; want <= smax; ++want) {
    const int per = (ktiles + want - 1) / want, s = (ktiles + per - 1) / per;
    if (s != want) continue;
    for (int tile = 64; tile <= 128; tile += 64) {
      const double c = tile == 64 ? plan_us_64(M, N, ktiles, batch, s) : plan_us_128(M, N, ktiles, batch, s);
      if (c < now) {
        now = c;
        pl.tile = tile == 64 ? kTile64 : kTile128;
        pl.splits = s;
      }
    }
  }
  return pl;
}

// h_c = tanh(W_c [ctx ; h_dec]) of N rows.  Segments: ctx (+ remainder), h_dec.  Each is cut into reduction tiles of its own,
// so the length to plan a split for counts whole tiles per segment: planned over 3 * H, sizes like H = 584 got a split with no
// tiles left.
// Few rows whose tiles would need a split over blocks and a combine launch, with a reduction that is short for one block: the
// planner splits from 449 units on, up to 127 rows of 456 units and 113 of 512.  us, split and combined / few: 456 units, 1 row
// 7.6 / 4.2, 113 8.7 / 5.6; 512, 1 7.6 / 4.5, 16 8.0 / 5.4, 40 8.4 / 6.8, 113 8.6 / 6.9; past the line 576, 16 8.3 / 6.7, 40 8.6 / 8.7,
// 640, 40 8.7 / 10.5, 1024, 16 8.9 / 8.8, 40 9.3 / 11.8.  (Fewer units are not split, and stay with the tiles.)
GemmPlan plan_hc(int N, int H, bool bf16) {
  const GemmPlan p = gemm_plan(N, H, bf16 ? 3 * ((H + 63) / 64 * 64) : 2 * H, 1, bf16, true, true);
  return bf16 && N <= 128 && H <= 512 && p.splits > 1 ? GemmPlan{kTileFew, 1} : p;
}
// d_h_dec += dQ W_a^T of N rows: as for h_c, and here without a split to save.  us, 64 x 64 tiles / few: 128 units, 1 row 4.1 /
// 3.3, 128 rows 4.7 / 4.0; 256, 40 4.9 / 4.6; 512, 17 5.8 / 5.5, 40 6.0 / 6.5, 128 6.2 / 6.6; 640, 17 6.3 / 5.9, 40 6.4 / 6.7; 768, 40
// 6.8 / 6.4, 128 7.0 / 6.5; 1024, 1 7.2 / 4.4, 128 7.8 / 6.5; 1280, 128 8.6 / 10.6.
GemmPlan plan_dh(int N, int H, bool bf16) {
  const GemmPlan p = gemm_plan(N, H, H, 1, bf16, false);
  const bool few = bf16 && N <= 128 && H <= 1024 && (N <= 32 || H <= 256 || H >= 768);
  return few && p.tile == kTile64 ? GemmPlan{kTileFew, 1} : p;
}

hipError_t launch_gemm(const GemmArgs& g, bool in_bf16, GemmTile tile, hipStream_t st) {
  if (g.row_pos && g.splits <= 1) return hipErrorInvalidValue;
  hipError_t e = in_bf16 ? launch_gemm_bf16(g, tile, st) : launch_gemm_f32(g, st);
  if (e != hipSuccess) return e;
  if (g.splits > 1) e = launch_splitk_combine(g, in_bf16, st);
  return e;
}

hipError_t launch_gemm_joint(const GemmArgs* g, const GemmTile* tile, int n, bool in_bf16, hipStream_t st, const DbReduce* sums) {
  for (int i = 0; i < n; ++i)
    if (g[i].row_pos && g[i].splits <= 1) return hipErrorInvalidValue;
  hipError_t e = in_bf16 ? launch_gemm_bf16_together(g, tile, n, sums, st) : launch_gemm_f32_together(g, n, sums, st);
  for (int i = 0; i < n && e == hipSuccess; ++i)
    if (g[i].splits > 1) e = launch_splitk_combine(g[i], in_bf16, st);
  return e;
}
hipError_t launch_gemm_together(const GemmArgs* g, const GemmTile* tile, int n, bool in_bf16, hipStream_t st) {
  hipError_t e = launch_gemm_joint(g, tile, n, in_bf16, st);
  if (e != hipErrorNotSupported) return e;
  e = hipSuccess;
  for (int i = 0; i < n && e == hipSuccess; ++i) e = launch_gemm(g[i], in_bf16, tile[i], st);
  return e;
}

}  // namespace asx
