// The stacked LSTM on the matrix cores (gfx950): one launch per WAVEFRONT of layer-steps.
//
// Layer l can take step t as soon as it has its own state of step t - 1 and the output of layer l - 1 at step t.  All
// layer-steps (l, d - l) are therefore independent and go into one launch; the input product is folded into the
// step as a second segment of the reduction, so that nothing else has to run between two launches (layer 0: unless
// ls_input_apart).
//
// A wavefront is a skinny product (B columns, typically 128) on the critical path, bound by the way from the caches to
// the registers and by what any launch costs, not by the matrix cores:
//   * no LDS staging: a wave loads matrix fragments straight into registers, 1 KiB per load from contiguous memory
//     (fragment tiles, lstm_wave.h), with the next PF reduction steps in flight;
//   * the reduction is split over the four waves of a block (wave w takes steps w, w + 4, ...), so no byte is loaded
//     twice by a block; the partial tiles meet in LDS and are added in wave order.  Every block shape adds in the same
//     order: results do not depend on the shape chosen, nor on how many sentences share the batch;
//   * the WEIGHT rows are the rows of the matrix instruction and the sentences its columns.  A lane then holds four
//     rows for its sentence: forward the four gates of one unit (and over four tiles those of four consecutive units),
//     backward four consecutive units.  The whole cell is lane-local and its memory accesses are vectors.
//   * bf16 storage: h enters as a (value, rounding remainder) pair that shares the weight fragment, without which
//     rounding compounds over steps and layers.  Gate gradients enter the backward products as plain bf16.
//   * fp32 storage: fp64 matrix instructions on operands widened after the load, as in gemm_f32.hip.
//
// 4 layers x 1024 units x 128 sentences, full wavefronts: 25.1 us forward, 27.6 backward (27.3 and 28.9 before the cells
// were shortened: functions above the kernels, dropout and the backward tanh while the first fragments are on their way,
// column sums by rotations in registers, 16 MB of stores of which the gates go past the caches).  Forward, launch and first
// loads 3.5, reduction 12.5 (weights that all come from the L2 save 1.6), cells the rest, 5 of it the stores.  64 MB of
// weights and 1 MB (forward) or 1.5 MB (backward) of fragments per compute unit make the reduction.  A launch per layer and
// step took 10.5 us each, 42 for what a wavefront does, and the input products another 90 per layer.  Tried without gain: weights streamed past the caches (34.6 / 40.7 us), other tile orders
// of the weights, two to four slots (30.0 / 28.9 / 28.4), 64 x 64 and 64 x 32 forward blocks (33.5, 34.0).
#include "common.h"
#include "lstm_wave.h"
#include "wave_pipe.h"

namespace asx {

typedef uint32_t ls_u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t ls_u32x2_t __attribute__((ext_vector_type(2)));
typedef double ls_f64x4_t __attribute__((ext_vector_type(4)));

constexpr int LS_KS = 4;   // waves per block = ways a reduction is split

// Matrix instruction of one fragment pair.  Row of the tile that register r of a lane in group q = lane / 16 holds:
// 4 q + r (bf16) or 4 r + q (fp64).
template <typename TE> struct LsMma;
template <> struct LsMma<uint16_t> {
  typedef f32x4_t acc_t;
  typedef float sum_t;
  typedef ls_u32x2_t raw4_t;
  static constexpr bool kPair = true;
  static __device__ __forceinline__ void mma(acc_t& acc, ls_u32x4_t a, ls_u32x4_t b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), acc,
                                                  0, 0, 0);
  }
  // tile row that lane group q holds in register r
  static __host__ __device__ __forceinline__ int q_of_row(int rho) { return rho >> 2; }
  static __host__ __device__ __forceinline__ int r_of_row(int rho) { return rho & 3; }
};
template <> struct LsMma<float> {
  typedef ls_f64x4_t acc_t;
  typedef double sum_t;
  typedef f32x4_t raw4_t;
  static constexpr bool kPair = false;
  static __device__ __forceinline__ void mma(acc_t& acc, ls_u32x4_t a, ls_u32x4_t b) {
    const f32x4_t af = __builtin_bit_cast(f32x4_t, a), bf = __builtin_bit_cast(f32x4_t, b);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)af[e], (double)bf[e], acc, 0, 0, 0);
  }
  static __host__ __device__ __forceinline__ int q_of_row(int rho) { return rho & 3; }
  static __host__ __device__ __forceinline__ int r_of_row(int rho) { return rho >> 2; }
};

// The cell's functions without branches or IEEE divisions: with one wave per SIMD nothing hides the vector instructions of
// a cell (4 x 1024 units x 128 sentences, forward wavefronts: 2 us of 27 less than with expf, tanhf and divisions).  Error in
// units of the last place, over every float of a binade, here and with those: no binade of either function has a larger
// maximum or mean.  Largest, sigmoid 1.72 and 2.20 (2.62 below -16; past -87 results less than the smallest normal number,
// which 1 / (1 + expf) loses), tanh 1.03 and 1.41; mean over N(0, s^2), s = 0.1 / 1 / 10, sigmoid 0.266 / 0.280 / 0.283 and 0.458 /
// 0.397 / 0.418, tanh 0.250 / 0.257 / 0.166 and 0.251 / 0.275 / 0.169.
// e^-a, 0 <= a <= 104 or NaN
__device__ __forceinline__ float ls_exp_neg(float a) {
  constexpr float kLog2e = 1.44269504088896f, kLog2eLo = 1.925963033500e-8f;
  const float n = __builtin_rintf(-a * kLog2e);
  const float f = __builtin_fmaf(-a, kLog2eLo, __builtin_fmaf(-a, kLog2e, -n));
  return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}
// x / (1 + e), 0 <= e <= 1: a Newton step from the reciprocal instruction whose remainder counts the rounding of 1 + e in
__device__ __forceinline__ float ls_over_1p(float x, float e) {
  const float d = 1.f + e, lo = e - (d - 1.f), r = __builtin_amdgcn_rcpf(d), q = x * r;
  return __builtin_fmaf(__builtin_fmaf(-q, lo, __builtin_fmaf(-q, d, x)), r, q);
}
__device__ __forceinline__ float ls_sigmoid(float a) {
  const float m = __builtin_fabsf(a), e = ls_exp_neg(m > 104.f ? 104.f : m);   // (NaN stays; e^-104 rounds to 0)
  return ls_over_1p(a < 0.f ? e : 1.f, e);
}
// |a| < 0.625: a + a^3 P(a^2), P the minimax polynomial of (tanh(a) / a - 1) / a^2 (relative error of the whole 1.6e-10 before
// rounding); else 1 - 2 e^-2a / (1 + e^-2a)
__device__ __forceinline__ float ls_tanh(float a) {
  const float m = __builtin_fabsf(a), b = m > 20.f ? 20.f : m;
  const float e = ls_exp_neg(b + b), t = __builtin_fmaf(-2.f * e, ls_over_1p(1.f, e), 1.f);
  const float u = a * a;
  float q = __builtin_fmaf(u, 0x1.1ace3ep-9f, -0x1.0c895ep-7f);
  q = __builtin_fmaf(u, q, 0x1.63ad18p-6f);
  q = __builtin_fmaf(u, q, -0x1.b9f220p-5f);
  q = __builtin_fmaf(u, q, 0x1.11107cp-3f);
  q = __builtin_fmaf(u, q, -0x1.555554p-2f);
  const float s = __builtin_fmaf(u * m, q, m);
  return __builtin_copysignf(m < 0.625f ? s : t, a);
}
// sum over the 16 lanes of a row (lanes l, l ^ 8, then ^ 4, ^ 2, ^ 1: rotations add the same pairs), without the LDS pipe
template <int N> __device__ __forceinline__ float ls_row_ror(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float ls_row_sum(float v) {
  v += ls_row_ror<8>(v);
  v += ls_row_ror<4>(v);
  v += ls_row_ror<2>(v);
  v += ls_row_ror<1>(v);
  return v;
}
__device__ __forceinline__ int ls_len(const int32_t* lengths, int b, int T) {
  const int n = lengths[b];
  return n < 0 ? 0 : (n > T ? T : n);
}

// Four consecutive elements, of which n are inside.  VEC (H % 4 == 0): all four are, and aligned.
template <bool VEC> __device__ __forceinline__ f32x4_t ls_ld4(const float* p, int n) {
  if constexpr (VEC) {
    return *reinterpret_cast<const f32x4_t*>(p);
  } else {
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) v[e] = p[e];
    return v;
  }
}
template <bool VEC> __device__ __forceinline__ void ls_st4(float* p, const f32x4_t& v, int n) {
  if constexpr (VEC) {
    *reinterpret_cast<f32x4_t*>(p) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) p[e] = v[e];
  }
}
// the same past the caches, for what no wavefront reads again
template <bool VEC> __device__ __forceinline__ void ls_st4_away(float* p, const f32x4_t& v, int n) {
  if constexpr (VEC) {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4_t*>(p));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) p[e] = v[e];
  }
}
// bf16 storage implies VEC (H % 8 == 0); raw: four elements as loaded
template <bool VEC> __device__ __forceinline__ ls_u32x2_t ls_ldraw4(const uint16_t* p, int) {
  return *reinterpret_cast<const ls_u32x2_t*>(p);
}
template <bool VEC> __device__ __forceinline__ f32x4_t ls_ldraw4(const float* p, int n) { return ls_ld4<VEC>(p, n); }
__device__ __forceinline__ f32x4_t ls_widen4(const f32x4_t& v) { return v; }
__device__ __forceinline__ f32x4_t ls_widen4(const ls_u32x2_t& w) {
  const f32x4_t v = {lo_bf16(w[0]), hi_bf16(w[0]), lo_bf16(w[1]), hi_bf16(w[1])};
  return v;
}
template <bool VEC> __device__ __forceinline__ void ls_st4(uint16_t* p, const f32x4_t& v, int) {
  const ls_u32x2_t w = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
  *reinterpret_cast<ls_u32x2_t*>(p) = w;
}
template <typename TE> __device__ __forceinline__ f32x4_t ls_rest(const f32x4_t& v) {
  f32x4_t r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = v[e] - round_elem<TE>(v[e]);
  return r;
}
// multipliers of the four elements from flat index i on (VEC: i % 4 == 0)
template <bool VEC> __device__ __forceinline__ f32x4_t ls_drop4(uint64_t i, uint64_t seed, uint32_t thr, float scale) {
  f32x4_t m;
  if constexpr (VEC) {
    uint32_t w[4];
    dropout_words4(i >> 2, seed, w);
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = w[e] >= thr ? scale : 0.f;
  } else {
#pragma unroll 1
    for (int e = 0; e < 4; ++e) {
      const float x = dropout_mult(i + e, seed, thr, scale);
      m[0] = e == 0 ? x : m[0]; m[1] = e == 1 ? x : m[1]; m[2] = e == 2 ? x : m[2]; m[3] = e == 3 ? x : m[3];
    }
  }
  return m;
}
// offset (elements) of reduction index k, k % 4 == 0, of column b in fragment tiles of nct column tiles
template <typename TE> __device__ __forceinline__ int64_t ls_tile_off(int k, int b, int nct) {
  constexpr int V = LsGeom<TE>::kVec, K = LsGeom<TE>::kKStep;
  return (((int64_t)(k / K) * nct + (b >> 4)) * 64 + (k % K) / V * 16 + (b & 15)) * V + k % V;
}

// 16 bytes per lane from a wave-uniform address and an unsigned lane offset: the form that needs no 64-bit address
// arithmetic and no address registers per load
__device__ __forceinline__ ls_u32x4_t ls_frag(const char* base, uint32_t lane16) {
  return *reinterpret_cast<const ls_u32x4_t*>(base + lane16);
}

// Blocks of a wavefront: nslices (layer, row block) slices of the weights x nbt batch blocks.  Consecutive blocks go
// round-robin to the 8 XCDs.  An XCD gets a contiguous run of slices with all their batch blocks: its L2 fetches a
// slice of the weights once, and the state of few layers only.
__device__ __forceinline__ bool ls_block_of(int nslices, int nbt, int& slice, int& bt) {
  const int per = (nslices + 7) >> 3, xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int s = idx / nbt;
  slice = xcd * per + s;
  bt = idx - s * nbt;
  return slice < nslices;
}
static inline unsigned ls_grid(int64_t nslices, int64_t nbt) { return (unsigned)((nslices + 7) / 8 * 8 * nbt); }

// ---- operands as tiles -------------------------------------------------------------
template <typename TE>
__device__ __forceinline__ void ls_copy_chunk(char* dst, const TE* src, int n) {
  constexpr int V = LsGeom<TE>::kVec;
  if (n >= V && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
    *reinterpret_cast<ls_u32x4_t*>(dst) = *reinterpret_cast<const ls_u32x4_t*>(src);
    return;
  }
#pragma unroll
  for (int e = 0; e < V; ++e) reinterpret_cast<TE*>(dst)[e] = e < n ? src[e] : (TE)0;
}

// Initial state of layer l: as tiles, and where the backward pass looks for it.  padding: only the zeros behind the reduction.
template <typename TE>
__device__ __forceinline__ void ls_prep_state(const LsFwd& p, int l, int64_t first, int64_t stride, bool padding) {
  typedef LsMma<TE> M;
  constexpr int V = LsGeom<TE>::kVec, KST = LsGeom<TE>::kKStep;
  const int H = p.H, B = p.B, L = p.L, nct = (B + 15) >> 4;
  const int64_t BH = (int64_t)B * H;
  const int64_t n = (int64_t)((H + KST - 1) / KST) * nct * 64;
  TE* hE = reinterpret_cast<TE*>(p.hE) + (int64_t)l * (p.T + 1) * BH;
  float* cs = p.cs + (int64_t)l * (p.T + 1) * BH;
  for (int64_t i = first; i < n; i += stride) {
    const int lane = (int)(i & 63), k = (int)((i >> 6) / nct) * KST + (lane >> 4) * V;
    const int64_t tile = i >> 6;
    const int b = (int)(tile % nct) * 16 + (lane & 15);
    if (padding && k < H) continue;
    alignas(16) TE hi[V], lo[V];
    // a chunk of V units inside, its rows aligned: whole vectors (one step of 4 x 1024 units x 128 sentences: 8.6 -> 5.3 us)
    const bool whole = H % V == 0 && b < B && k < H;
    if (whole) {
      const int64_t row = (int64_t)b * H + k, idx = (int64_t)l * BH + row;
      f32x4_t h[V / 4], c[V / 4];
#pragma unroll
      for (int v = 0; v < V / 4; ++v) {
        h[v] = p.h0 ? *reinterpret_cast<const f32x4_t*>(p.h0 + idx + 4 * v) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        c[v] = p.c0 ? *reinterpret_cast<const f32x4_t*>(p.c0 + idx + 4 * v) : f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int v = 0; v < V / 4; ++v) {
        ls_st4<true>(p.hf + idx + 4 * v, h[v], 4);
        ls_st4<true>(cs + row + 4 * v, c[v], 4);
        ls_st4<true>(hE + row + 4 * v, h[v], 4);
        ls_st4<true>(hi + 4 * v, h[v], 4);
        ls_st4<true>(lo + 4 * v, ls_rest<TE>(h[v]), 4);
      }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
      if (whole) break;
      const bool in = b < B && k + e < H;
      const int64_t idx = (int64_t)l * BH + (int64_t)(in ? b : 0) * H + (in ? k + e : 0);
      const float h = in && p.h0 ? p.h0[idx] : 0.f;
      st_elem<TE>(hi, e, h);
      st_elem<TE>(lo, e, h - round_elem<TE>(h));
      if (in) {
        const float c = p.c0 ? p.c0[idx] : 0.f;
        p.hf[idx] = h;
        cs[idx - (int64_t)l * BH] = c;
        st_elem<TE>(hE, idx - (int64_t)l * BH, h);
      }
    }
    auto put = [&](char* base, const TE (&v)[V]) {
      *reinterpret_cast<ls_u32x4_t*>(base + i * 16) = *reinterpret_cast<const ls_u32x4_t*>(v);
    };
    put(p.hF_hi + 2 * l * p.h_stride, hi);
    if constexpr (M::kPair) put(p.hF_lo + 2 * l * p.h_stride, lo);
    if (k >= H) {   // reduction padding: zero in every slot
      alignas(16) const TE z[V] = {};
      put(p.hF_hi + (2 * l + 1) * p.h_stride, z);
      if constexpr (M::kPair) put(p.hF_lo + (2 * l + 1) * p.h_stride, z);
      if (l + 1 < L)
        for (int sl = 0; sl < 2; ++sl) {
          put(p.oF_hi + (2 * l + sl) * p.h_stride, z);
          if constexpr (M::kPair) put(p.oF_lo + (2 * l + sl) * p.h_stride, z);
        }
    }
  }
}

// ---- forward ---------------------------------------------------------------------
// Block: 16 * NI gate rows (4 * NI hidden units) x 16 * NJ sentences.  Tile 4 g + ii of a block, row rho: unit
// u0 + 16 g + 4 q + ii, gate r, (q, r) = the lane group and register that hold row rho.  ROWS: weights are read as the
// caller's rows (64 bytes of a row per load), each used once by the call; steps of the reduction, their waves and the order
// inside a step are those of the tiles, so that a step by itself gives the bits it has in a sequence (whole lines of a row
// per step: 4 x 1024 units x 128 sentences 114.7 us for 116.9, 4 x 192 units x 116 sentences 75.5 for 73.8, and other bits).
// ROWS = 2: layer 0 of ls_reads_states.  APART: layer 0 finds the input product and the
// bias in the gates' place.
template <typename TE, int NI, int NJ, int PF, int ROWS, bool VEC, bool APART, bool PACKED>
__global__ __launch_bounds__(64 * LS_KS) void ls_wave_fwd_kernel(LsFwd p, int d, int l_lo, int n_layers) {
  typedef LsMma<TE> M;
  typedef typename M::acc_t acc_t;
  constexpr int NG = NI / 4, V = LsGeom<TE>::kVec, KST = LsGeom<TE>::kKStep;
  static_assert(NI % 4 == 0, "four tiles hold the gates of four consecutive units per lane");
  __shared__ acc_t red[LS_KS * NI * NJ * 64];   // [wave][i][j][lane]
  const uint32_t lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane >> 4, c = lane & 15;
  const uint32_t lane16 = lane * 16u;
  const int H = p.H, B = p.B, nct = (B + 15) >> 4;
  const int nut = (H + 4 * NI - 1) / (4 * NI), nbt = (B + 16 * NJ - 1) / (16 * NJ);
  constexpr bool DIRECT = ROWS == 2;
  if constexpr (DIRECT) {   // blocks past the layer's: the states of the others as tiles
    const int own = (n_layers * nut + 7) / 8 * 8 * nbt, extra = (int)blockIdx.x - own;
    if (extra >= 0) {
      const int per = ((int)gridDim.x - own) / p.L, job = extra / per;
      ls_prep_state<TE>(p, job, (int64_t)(extra - job * per) * blockDim.x + threadIdx.x, (int64_t)per * blockDim.x, job == 0);
      return;
    }
  }
  int slice, bt;
  if (!ls_block_of(n_layers * nut, nbt, slice, bt)) return;
  const int l = l_lo + slice / nut, u0 = (slice % nut) * 4 * NI, b0 = bt * 16 * NJ;
  const int t = d - l;
  const int Kin = l == 0 ? p.I : H;
  const int64_t BH = (int64_t)B * H;

  // what the cells need from memory is requested ahead of the product
  constexpr int NTASK = (NG * NJ + LS_KS - 1) / LS_KS;   // (g, j) pairs, dealt out to the waves
  // (lanes and tasks without a cell read the last one: no branch around a load that is to stay in flight)
  constexpr bool packed = PACKED;
  int len[NTASK], wrd[NTASK];     // packed: row of the sentence's first word
  f32x4_t cp[NTASK], hp[NTASK];   // hp (DIRECT): the initial state itself
  typename M::raw4_t bias[NTASK][4];
  const float* c_prev = DIRECT && p.c0 ? p.c0 + l * BH : p.cs + ((int64_t)l * (p.T + 1) + t) * BH;
  const float* h_prev = p.h0 ? p.h0 + l * BH : c_prev;
  const TE* bl = reinterpret_cast<const TE*>(p.bias[l]);
#pragma unroll
  for (int k = 0; k < NTASK; ++k) {
    const int task = wave + k * LS_KS, g = task / NJ, j = task % NJ;
    const int b = b0 + 16 * j + c, unit0 = u0 + 16 * g + 4 * q;
    const int bs = b < B ? b : B - 1, us = unit0 < H ? unit0 : (H - 1) & ~3;
    if constexpr (packed) {
      len[k] = p.lengths[bs];
      wrd[k] = p.words.start[bs];
    }
    cp[k] = ls_ld4<VEC>(c_prev + (int64_t)bs * H + us, H - us);
    if constexpr (DIRECT) hp[k] = ls_ld4<VEC>(h_prev + (int64_t)bs * H + us, H - us);
#pragma unroll
    for (int e = 0; e < 4; ++e) bias[k][e] = ls_ldraw4<VEC>(bl + (int64_t)e * H + us, H - us);
  }

  acc_t acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;

  // Segments: own state, then the input.  x is exact in the storage type, it has no remainder.  The widest block reduces
  // the two segments of layer 0 one after the other, the second without remainders (one loop for both spilled 32
  // registers: 4 x 1024 units x 128 sentences 1508 -> 1410 us).  In the smaller ones the refill between two loops costs
  // more (a step by itself 147 -> 148 us for four layers): they load zeroed tiles as the remainder and branch around its
  // product, a block of its own behind the one the loads are spread over (0 * inf would be NaN; the weight cleared by a
  // mask instead, 50 x 128 x 512 units x 4 took 699 us, 681 so).
  constexpr bool TWO = M::kPair && NI * NJ >= 32;
  const bool apart = APART && l == 0;
  const int n0 = (H + KST - 1) / KST, n1 = apart ? 0 : (Kin + KST - 1) / KST;
  const int64_t cstep = (int64_t)nct * kLsTile;
  const char* h_hi = p.hF_hi + (2 * l + (t & 1)) * p.h_stride;
  const char* h_lo = M::kPair ? p.hF_lo + (2 * l + (t & 1)) * p.h_stride : nullptr;
  const char* i_hi = DIRECT ? reinterpret_cast<const char*>(p.x) : l == 0 ? p.xF + t * p.x_stride : p.oF_hi + (2 * (l - 1) + (t & 1)) * p.h_stride;
  const bool no_rest = !TWO && !APART && l == 0;   // the input's remainder: zeroed tiles (DIRECT: the input again)
  const char* i_lo = !M::kPair ? nullptr : DIRECT ? i_hi : no_rest ? p.zeros : p.oF_lo + (2 * (l - 1) + (t & 1)) * p.h_stride;
  const int64_t lstep1 = no_rest ? 0 : cstep;
  int64_t ctoff[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int ct = (b0 >> 4) + j;
    ctoff[j] = (ct < nct ? ct : nct - 1) * kLsTile;   // columns past the batch repeat the last tile; not stored
  }
  const char* w0 = reinterpret_cast<const char*>(p.W_hh[l]) + (ROWS ? 0 : (int64_t)(u0 / 16) * n0 * 4 * kLsTile);
  const char* w1 = reinterpret_cast<const char*>(p.W_ih[l]) + (ROWS ? 0 : (int64_t)(u0 / 16) * n1 * 4 * kLsTile);
  // DIRECT: the caller's initial state as float, split into value and remainder after the load, and his input's rows
  int wrow[NI];
  int64_t hrow[NJ], xrow[NJ];
  const char* h_f32 = reinterpret_cast<const char*>(h_prev);
  if constexpr (DIRECT) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int b = b0 + 16 * j + c, bs = b < B ? b : B - 1;
      hrow[j] = (int64_t)bs * H * 4;
      xrow[j] = (int64_t)bs * p.I * sizeof(TE);
    }
  }
  if constexpr (ROWS) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int unit = u0 + 16 * (i / 4) + 4 * M::q_of_row(c) + (i & 3);
      wrow[i] = M::r_of_row(c) * H + (unit < H ? unit : H - 1);   // rows past the layer repeat the last unit; not stored
    }
  }
  ls_u32x4_t wf[PF][NI], hf[PF][NJ], lf[PF][M::kPair ? NJ : 1];
  auto load = [&](int slot, int step, bool rest = true) {   // rest: the remainders too
    const int s = wave + step * LS_KS;
    const bool in = s >= n0;
    const int k = in ? s - n0 : s;
    if constexpr (ROWS) {
      const int K = in ? Kin : H, kk = k * KST + q * V;
      const char* wb = (in ? w1 : w0) + (int64_t)(kk < K ? kk : 0) * sizeof(TE);
#pragma unroll
      for (int i = 0; i < NI; ++i)
        wf[slot][i] = *reinterpret_cast<const ls_u32x4_t*>(wb + (int64_t)wrow[i] * K * sizeof(TE));
    } else {
      const char* wb = (in ? w1 : w0) + k * (4 * kLsTile);
      const int64_t group = (int64_t)(in ? n1 : n0) * (4 * kLsTile);
#pragma unroll
      for (int i = 0; i < NI; ++i)
        wf[slot][i] = ls_frag(wb + (i / 4) * group + (i % 4) * kLsTile, lane16);
    }
    if constexpr (DIRECT) {
      const int K = in ? Kin : H, kk = k * KST + q * V, kc = kk < K ? kk : 0;
      const char *hb = in ? i_hi : h_f32, *lb = in ? i_lo : h_f32 + 16;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int64_t off = in ? xrow[j] + kc * (int)sizeof(TE) : hrow[j] + kc * 4;
        hf[slot][j] = *reinterpret_cast<const ls_u32x4_t*>(hb + off);
        if constexpr (M::kPair) lf[slot][j] = *reinterpret_cast<const ls_u32x4_t*>(lb + off);
      }
      return;
    }
    const char* hb = (in ? i_hi : h_hi) + k * cstep;
#pragma unroll
    for (int j = 0; j < NJ; ++j) hf[slot][j] = ls_frag(hb + ctoff[j], lane16);
    if (M::kPair && rest) {
      const char* lb = in ? i_lo + k * lstep1 : h_lo + k * cstep;
#pragma unroll
      for (int j = 0; j < NJ; ++j) lf[slot][j] = ls_frag(lb + ctoff[j], lane16);
    }
  };
  auto mul = [&](int slot, int step, bool rest = true) {
    const int s = wave + step * LS_KS;
    if constexpr (ROWS) {   // chunks past a row's end were read from its start (DIRECT: both operands cleared, 0 * inf)
      const int K = s >= n0 ? Kin : H, kk = (s >= n0 ? s - n0 : s) * KST + q * V;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) wf[slot][i][e] = kk < K ? wf[slot][i][e] : 0u;
      const bool state = s < n0, live = kk < K && (!state || p.h0);
#pragma unroll
      for (int j = 0; j < (DIRECT ? NJ : 0); ++j) {
        if constexpr (M::kPair) {
          const f32x4_t h0 = __builtin_bit_cast(f32x4_t, hf[slot][j]), h1 = __builtin_bit_cast(f32x4_t, lf[slot][j]);
          const f32x4_t r0 = ls_rest<TE>(h0), r1 = ls_rest<TE>(h1);
          const ls_u32x4_t hi = {pack_bf16(h0[0], h0[1]), pack_bf16(h0[2], h0[3]), pack_bf16(h1[0], h1[1]), pack_bf16(h1[2], h1[3])};
          const ls_u32x4_t lo = {pack_bf16(r0[0], r0[1]), pack_bf16(r0[2], r0[3]), pack_bf16(r1[0], r1[1]), pack_bf16(r1[2], r1[3])};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            hf[slot][j][e] = live ? state ? hi[e] : hf[slot][j][e] : 0u;
            lf[slot][j][e] = live ? state ? lo[e] : lf[slot][j][e] : 0u;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) hf[slot][j][e] = live ? hf[slot][j][e] : 0u;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) M::mma(acc[i][j], wf[slot][i], hf[slot][j]);
    if constexpr (M::kPair) {   // (a plain condition cost the fp32 wavefronts 0.5 us in copies of accumulators)
      if (rest) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) M::mma(acc[i][j], wf[slot][i], lf[slot][j]);
      }
    }
  };
  // while the first fragments are on their way: the dropout multipliers of the cells
  const bool drop = p.drop_thr && l + 1 < p.L;
  f32x4_t dm[NTASK];
  auto masks = [&]() {
    if (!drop) return;
#pragma unroll
    for (int k = 0; k < NTASK; ++k) {
      const int task = wave + k * LS_KS, g = task / NJ, j = task % NJ;
      dm[k] = ls_drop4<VEC>(((uint64_t)l * p.T + t) * (uint64_t)BH + (uint64_t)((int64_t)(b0 + 16 * j + c) * H) +
                                (uint64_t)(u0 + 16 * g + 4 * q), p.drop_seed, p.drop_thr, p.drop_scale);
    }
  };
  constexpr int NP = M::kPair ? 2 : 1, NM = M::kPair ? 2 * NI * NJ : 4 * NI * NJ;
  const int own = own_steps<LS_KS>(n0 + n1, wave);
  if constexpr (TWO) {
    const int own0 = l == 0 ? own_steps<LS_KS>(n0, wave) : own;
    wave_reduce<PF, NI + NP * NJ, NM>(own0, load, mul, NoRest(), masks);
    wave_reduce<PF, NI + NJ, NM / 2>(
        own - own0, [&](int slot, int i) { load(slot, own0 + i, false); },
        [&](int slot, int i) { mul(slot, own0 + i, false); });
  } else if constexpr (M::kPair && !APART) {
    wave_reduce<PF, NI + NP * NJ, NM / 2>(
        own, load, [&](int slot, int i) { mul(slot, i, false); },
        [&](int slot, int i) {
          if (l == 0 && wave + i * LS_KS >= n0) return;
#pragma unroll
          for (int ii = 0; ii < NI; ++ii)
#pragma unroll
            for (int j = 0; j < NJ; ++j) M::mma(acc[ii][j], wf[slot][ii], lf[slot][j]);
        },
        masks);
  } else {
    wave_reduce<PF, NI + NP * NJ, NM>(own, load, mul, NoRest(), masks);
  }

#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) red[((wave * NI + i) * NJ + j) * 64 + lane] = acc[i][j];
  __syncthreads();

  const bool last = t + 1 == p.T;
#pragma unroll
  for (int k = 0; k < NTASK; ++k) {
    const int task = wave + k * LS_KS, g = task / NJ, j = task % NJ;
    const int b = b0 + 16 * j + c, unit0 = u0 + 16 * g + 4 * q;
    if (task >= NG * NJ || b >= B || unit0 >= H) continue;
    const int n = H - unit0;
    float* G = p.gates + ((int64_t)l * p.T + t) * 4 * BH + (int64_t)b * 4 * H + unit0;
    f32x4_t gi, gf, gg, go, cn, hn, bias4[4];
    if constexpr (DIRECT) {
      if (!p.c0) cp[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if (!p.h0) hp[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    if (apart) {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias4[e] = ls_ld4<VEC>(G + (int64_t)e * H, n);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) bias4[e] = ls_widen4(bias[k][e]);
    }
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      acc_t v = red[((4 * g + ii) * NJ + j) * 64 + lane];
#pragma unroll
      for (int w = 1; w < LS_KS; ++w) v += red[((w * NI + 4 * g + ii) * NJ + j) * 64 + lane];
      float a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = (float)(v[e] + (typename M::sum_t)bias4[e][ii]);
      gi[ii] = ls_sigmoid(a[0]);
      gf[ii] = ls_sigmoid(a[1]);
      gg[ii] = ls_tanh(a[2]);
      go[ii] = ls_sigmoid(a[3]);
      // (which product is rounded by itself is not left to the compiler: block shapes would differ)
      cn[ii] = __builtin_fmaf(gf[ii], cp[k][ii], gi[ii] * gg[ii]);
      hn[ii] = go[ii] * ls_tanh(cn[ii]);
    }
    const int64_t idx = (int64_t)b * H + unit0;
    if constexpr (packed) {
      len[k] = len[k] < 0 ? 0 : (len[k] > p.T ? p.T : len[k]);
      if (t >= len[k]) {   // a padded step leaves everything as it is: no product and no cell reads this sentence's columns again
        if (l + 1 == p.L) ls_st4<VEC>(reinterpret_cast<TE*>(p.y) + (int64_t)t * BH + idx, f32x4_t{0.f, 0.f, 0.f, 0.f}, n);
        if (len[k] == 0 && t == 0 && p.cT) ls_st4<VEC>(p.cT + l * BH + idx, cp[k], n);   // (not by the preparation, which reads c0)
        continue;
      }
    }
    if constexpr (DIRECT) {   // what the preparation leaves elsewhere
      ls_st4<VEC>(p.cs + (int64_t)l * (p.T + 1) * BH + idx, cp[k], n);
      ls_st4<VEC>(reinterpret_cast<TE*>(p.hE) + (int64_t)l * (p.T + 1) * BH + idx, hp[k], n);
    }
    ls_st4_away<VEC>(G, gi, n);
    ls_st4_away<VEC>(G + H, gf, n);
    ls_st4_away<VEC>(G + 2 * (int64_t)H, gg, n);
    ls_st4_away<VEC>(G + 3 * (int64_t)H, go, n);
    if constexpr (!packed) len[k] = ls_len(p.lengths, b, p.T);
    const bool valid = packed || t < len[k];
    const int64_t foff = ls_tile_off<TE>(unit0, b, nct);
    TE* hFn_hi = reinterpret_cast<TE*>(p.hF_hi + (2 * l + ((t + 1) & 1)) * p.h_stride) + foff;
    TE* hFn_lo = reinterpret_cast<TE*>(p.hF_lo + (2 * l + ((t + 1) & 1)) * p.h_stride) + foff;
    if constexpr (!VEC) {   // units past H: reduction padding of the next step, kept zero
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e >= n) hn[e] = 0.f;
    }
    f32x4_t o = {0.f, 0.f, 0.f, 0.f}, hv;
    if (valid) {   // what the next layer reads
      o = hn;
      if (drop) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = dm[k][e] != 0.f ? o[e] * dm[k][e] : 0.f;
      }
      hv = hn;
      if (t + 1 == len[k]) {   // the final state
        ls_st4<VEC>(p.hf + l * BH + idx, hn, n);
        if (packed && p.cT) ls_st4<VEC>(p.cT + l * BH + idx, cn, n);
      }
      if constexpr (!DIRECT) {
        ls_st4<true>(hFn_hi, hn, 4);
        if constexpr (M::kPair) ls_st4<true>(hFn_lo, ls_rest<TE>(hn), 4);
      }
    } else if constexpr (DIRECT) {
      cn = cp[k];
      hv = hp[k];
      ls_st4<VEC>(p.hf + l * BH + idx, hv, n);
    } else {       // padded step: the state passes through, the output is 0
      cn = cp[k];
      hv = ls_widen4(ls_ldraw4<true>(reinterpret_cast<const TE*>(h_hi) + foff, 4));
      ls_st4<true>(hFn_hi, hv, 4);
      if constexpr (M::kPair) ls_st4<true>(hFn_lo, ls_widen4(ls_ldraw4<true>(reinterpret_cast<const TE*>(h_lo) + foff, 4)), 4);
    }
    ls_st4<VEC>(p.cs + ((int64_t)l * (p.T + 1) + t + 1) * BH + idx, cn, n);
    if (!packed && last && p.cT) ls_st4<VEC>(p.cT + l * BH + idx, cn, n);
    const int64_t row = packed ? wrd[k] + t : (int64_t)t * B + b;   // of the word (states: of the next one, behind the initial ones)
    if (!packed || t + 1 < len[k])
      ls_st4<VEC>(reinterpret_cast<TE*>(p.hE) + (int64_t)l * (p.T + 1) * BH + (B + row + packed) * H + unit0, hv, n);
    if (l + 1 < p.L) {
      ls_st4<VEC>(reinterpret_cast<TE*>(p.out) + ((int64_t)l * p.T * B + row) * H + unit0, o, n);
      const int64_t slot = (2 * l + (t & 1)) * p.h_stride;
      ls_st4<true>(reinterpret_cast<TE*>(p.oF_hi + slot) + foff, o, 4);
      if constexpr (M::kPair) ls_st4<true>(reinterpret_cast<TE*>(p.oF_lo + slot) + foff, ls_rest<TE>(o), 4);
    } else {
      ls_st4<VEC>(reinterpret_cast<TE*>(p.y) + (int64_t)t * BH + idx, o, n);
    }
  }
}

// ---- backward --------------------------------------------------------------------
// Block: 16 * NI hidden units x 16 * NJ sentences of layer l at step t.  Two sums per output, over the 4H gate rows:
// da_{t+1} W_hh of the layer itself (the gradient through its own state) and da_t W_ih of the layer above (the gradient
// of its output; the top layer reads the caller's dy).  The gradient w.r.t. h_t is the former where step t + 1 was a
// word of the sentence, else what came in for the final state (sentences are right-padded, so the steps of a sentence
// are a prefix).  t = -1: the first sum alone, written out as the gradient of the initial state.
template <typename TE, int NI, int NJ, int PF, bool VEC, bool PACKED>
__global__ __launch_bounds__(64 * LS_KS) void ls_wave_bwd_kernel(LsBwd p, int d, int l_lo, int n_layers) {
  typedef LsMma<TE> M;
  typedef typename M::acc_t acc_t;
  constexpr int KST = LsGeom<TE>::kKStep;
  static_assert(PF % 2 == 0, "a slot belongs to one of the two sums");
  __shared__ acc_t red[2 * LS_KS * NI * NJ * 64];   // [sum][wave][i][j][lane]
  const uint32_t lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane >> 4, c = lane & 15;
  const uint32_t lane16 = lane * 16u;
  const int H = p.H, B = p.B, nct = (B + 15) >> 4;
  const int nut = (H + 16 * NI - 1) / (16 * NI), nbt = (B + 16 * NJ - 1) / (16 * NJ);
  int slice, bt;
  if (!ls_block_of(n_layers * nut, nbt, slice, bt)) return;
  const int l = l_lo + slice / nut, u0 = (slice % nut) * 16 * NI, b0 = bt * 16 * NJ;
  const int t = p.T - 1 - (d - (p.L - 1 - l));
  const bool top = l + 1 == p.L;
  const int64_t BH = (int64_t)B * H;

  // the inputs of the cell derivative are requested ahead of the products
  constexpr int NTASK = (NI * NJ + LS_KS - 1) / LS_KS;
  // (lanes and tasks without a cell read the last one, and what is absent is read from cs: no branch around a load
  // that is to stay in flight)
  f32x4_t gi[NTASK], gf[NTASK], gg[NTASK], go[NTASK], cp[NTASK], cn[NTASK], dy[NTASK], dcs[NTASK], carried[NTASK];
  constexpr bool packed = PACKED;
  int len[NTASK], wrd[NTASK];   // packed: row of the sentence's first word
  const int tc0 = t < 0 ? 0 : t;
  const float* cs_t = p.cs + ((int64_t)l * (p.T + 1) + tc0) * BH;
  const float* dc_in = t + 1 < p.T ? p.dcs : p.dcT;
  const float* dc_src = dc_in ? dc_in + l * BH : cs_t;
  const float* dh_src = p.dhT ? p.dhT + l * BH : cs_t;
  const float* dy_src = top ? p.dy + (int64_t)tc0 * BH : cs_t;
#pragma unroll
  for (int k = 0; k < NTASK; ++k) {
    const int task = wave + k * LS_KS, i = task / NJ, j = task % NJ;
    const int b = b0 + 16 * j + c, unit0 = u0 + 16 * i + 4 * q;
    const int bs = b < B ? b : B - 1, us = unit0 < H ? unit0 : (H - 1) & ~3, n = H - us;
    const int64_t idx = (int64_t)bs * H + us;
    const float* G = p.gates + ((int64_t)l * p.T + tc0) * 4 * BH + (int64_t)bs * 4 * H + us;
    len[k] = p.lengths[bs];
    if constexpr (packed) wrd[k] = p.words.start[bs];
    gi[k] = ls_ld4<VEC>(G, n);
    gf[k] = ls_ld4<VEC>(G + H, n);
    gg[k] = ls_ld4<VEC>(G + 2 * (int64_t)H, n);
    go[k] = ls_ld4<VEC>(G + 3 * (int64_t)H, n);
    cp[k] = ls_ld4<VEC>(cs_t + idx, n);
    cn[k] = ls_ld4<VEC>(cs_t + BH + idx, n);
    dy[k] = ls_ld4<VEC>(dy_src + idx, n);
    dcs[k] = ls_ld4<VEC>(dc_src + idx, n);
    carried[k] = ls_ld4<VEC>(dh_src + idx, n);
  }

  acc_t acc[2][NI][NJ];   // own state, output
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[s][i][j][r] = 0;

  // back through the mask the forward step put on this layer's output
  const bool drop = p.drop_thr && !top;
  auto mask = [&](int k) {
    const int task = wave + k * LS_KS, i = task / NJ, j = task % NJ;
    return ls_drop4<VEC>(((uint64_t)l * p.T + tc0) * (uint64_t)BH + (uint64_t)((int64_t)(b0 + 16 * j + c) * H) +
                             (uint64_t)(u0 + 16 * i + 4 * q), p.drop_seed, p.drop_thr, p.drop_scale);
  };
  // while the first fragments are on their way: tanh of the cell states, and in whole vectors the mask (an element at a time it
  // is four blocks of the generator, only where a sentence has the step: 219 units 13.0 us a wavefront ahead, 12.6 so)
  f32x4_t tc[NTASK], dm[NTASK];
  auto ahead = [&]() {
#pragma unroll
    for (int k = 0; k < NTASK; ++k) {
#pragma unroll
      for (int e = 0; e < 4; ++e) tc[k][e] = ls_tanh(cn[k][e]);
      if constexpr (VEC)
        if (drop) dm[k] = mask(k);
    }
  };
  const int ng = 4 * ls_gate_stride<TE>(H) / KST;
  const int n0 = t + 1 < p.T ? ng : 0, n1 = !top && t >= 0 ? ng : 0;
  if (n0 + n1 == 0) ahead();
  if (n0 + n1 > 0) {
    const int64_t cstep = (int64_t)nct * kLsTile, wrow = ng * kLsTile;
    const char* w0 = p.WT_hh[l] + u0 / 16 * wrow;
    const char* w1 = p.WT_up[l] + u0 / 16 * wrow;
    const char* g0 = p.dGF + (2 * l + ((t + 1) & 1)) * p.g_stride;
    const char* g1 = p.dGF + (2 * (l + 1) + (t & 1)) * p.g_stride;
    int64_t ctoff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int ct = (b0 >> 4) + j;
      ctoff[j] = (ct < nct ? ct : nct - 1) * kLsTile;
    }
    ls_u32x4_t wf[PF][NI], df[PF][NJ];
    auto fetch = [&](int slot, bool in, int k) {
      const char* wb = (in ? w1 : w0) + k * kLsTile;
#pragma unroll
      for (int i = 0; i < NI; ++i) wf[slot][i] = ls_frag(wb + i * wrow, lane16);
      const char* gb = (in ? g1 : g0) + k * cstep;
#pragma unroll
      for (int j = 0; j < NJ; ++j) df[slot][j] = ls_frag(gb + ctoff[j], lane16);
    };
    auto add = [&](int slot, int sum) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) M::mma(acc[sum][i][j], wf[slot][i], df[slot][j]);
    };
    // Both sums: their steps alternate, so that the slot says which sum a step belongs to (PF is even).
    constexpr int NL = NI + NJ, NM = M::kPair ? NI * NJ : 4 * NI * NJ;
    const int own = own_steps<LS_KS>(ng, wave);
    if (n0 > 0 && n1 > 0) {
      wave_reduce<PF, NL, NM>(
          2 * own, [&](int slot, int i) { fetch(slot, (i & 1) != 0, wave + (i >> 1) * LS_KS); },
          [&](int slot, int) { add(slot, slot & 1); }, NoRest(), ahead);
    } else {
      const bool in = n0 == 0;
      wave_reduce<PF, NL, NM>(
          own, [&](int slot, int i) { fetch(slot, in, wave + i * LS_KS); }, [&](int slot, int) { add(slot, 0); }, NoRest(),
          ahead);
      if (in) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            acc[1][i][j] = acc[0][i][j];
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[0][i][j][r] = 0;
          }
      }
    }
  }
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) red[(((s * LS_KS + wave) * NI + i) * NJ + j) * 64 + lane] = acc[s][i][j];
  __syncthreads();

  const int GS = ls_gate_stride<TE>(H);
#pragma unroll
  for (int k = 0; k < NTASK; ++k) {
    const int task = wave + k * LS_KS, i = task / NJ, j = task % NJ;
    const int b = b0 + 16 * j + c, unit0 = u0 + 16 * i + 4 * q;
    if (task >= NI * NJ || unit0 >= H) continue;   // lanes past the batch stay for the column sums
    const int n = H - unit0;
    const int64_t idx = (int64_t)b * H + unit0;
    f32x4_t sum[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      acc_t v = red[((s * LS_KS * NI + i) * NJ + j) * 64 + lane];
#pragma unroll
      for (int w = 1; w < LS_KS; ++w) v += red[(((s * LS_KS + w) * NI + i) * NJ + j) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[s][e] = (float)v[e];
    }
    len[k] = len[k] < 0 ? 0 : (len[k] > p.T ? p.T : len[k]);
    f32x4_t dh;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (!dc_in) dcs[k][e] = 0.f;
      if (!p.dhT) carried[k][e] = 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) dh[e] = t + 1 < len[k] ? sum[0][e] : carried[k][e];
    if (t < 0) {
      if (b < B) ls_st4<VEC>(p.dh0 + l * BH + idx, dh, n);
      continue;
    }
    f32x4_t da[4];
    const bool cell = b < B && t < len[k];
    if (cell) {
      if (!top) {
        dy[k] = sum[1];
        if (drop) {
          if constexpr (!VEC) dm[k] = mask(k);
#pragma unroll
          for (int e = 0; e < 4; ++e) dy[k][e] = dm[k][e] != 0.f ? dy[k][e] * dm[k][e] : 0.f;
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float dd = dy[k][e] + dh[e];
        const float dc = dcs[k][e] + dd * go[k][e] * (1.f - tc[k][e] * tc[k][e]);
        da[0][e] = dc * gg[k][e] * gi[k][e] * (1.f - gi[k][e]);
        da[1][e] = dc * cp[k][e] * gf[k][e] * (1.f - gf[k][e]);
        da[2][e] = dc * gi[k][e] * (1.f - gg[k][e] * gg[k][e]);
        da[3][e] = dd * tc[k][e] * go[k][e] * (1.f - go[k][e]);
        dcs[k][e] = dc * gf[k][e];
      }
      if constexpr (!VEC) {   // units past H: reduction padding of the products that read these, kept zero
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e >= n) da[0][e] = da[1][e] = da[2][e] = da[3][e] = 0.f;
      }
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) da[g][e] = 0.f;
    }
    if (b < B && (!packed || cell || t + 1 == p.T)) ls_st4<VEC>(p.dcs + l * BH + idx, dcs[k], n);
    if (packed ? cell : b < B) {   // (packed: a padded step has no row, and its column of the tiles adds to sums nobody reads)
      const int64_t row = packed ? wrd[k] + t : (int64_t)t * B + b;
      TE* dG = reinterpret_cast<TE*>(p.dG) + ((int64_t)l * p.T * B + row) * 4 * H + unit0;
      TE* dGF = reinterpret_cast<TE*>(p.dGF + (2 * l + (t & 1)) * p.g_stride);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        ls_st4<VEC>(dG + (int64_t)g * H, da[g], n);
        ls_st4<true>(dGF + ls_tile_off<TE>(g * GS + unit0, b, nct), da[g], 4);
      }
    }
    // bias gradient: sums over the tile's sentences, added up over the steps in an accumulator of the tile's own
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        da[g][e] = ls_row_sum(da[g][e]);
      }
    if (c < 4 && (b0 >> 4) + j < nct) {
      const f32x4_t mine = c == 0 ? da[0] : c == 1 ? da[1] : c == 2 ? da[2] : da[3];
      float* acc_p = p.dbacc + ((int64_t)l * nct + (b0 >> 4) + j) * 4 * H + (int64_t)c * H + unit0;
      f32x4_t old = {0.f, 0.f, 0.f, 0.f};
      if (t + 1 < p.T) old = ls_ld4<VEC>(acc_p, n);
      ls_st4<VEC>(acc_p, old + mine, n);
    }
  }
}

// Row of every sentence's first word, by a block of 256 threads: prefix sums of the lengths, 256 sentences at a time.
__device__ __forceinline__ void ls_word_starts(int32_t* start, const int32_t* lengths, int T, int B) {
  __shared__ int total[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int base = 0;
  for (int b0 = 0; b0 < B; b0 += 256) {
    const int own = b0 + tid < B ? ls_len(lengths, b0 + tid, T) : 0;
    int v = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(v, d, 64);
      v += lane >= d ? up : 0;
    }
    if (lane == 63) total[wave] = v;
    __syncthreads();
    int before = base, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      before += w < wave ? total[w] : 0;
      all += total[w];
    }
    if (b0 + tid < B) start[b0 + tid] = before + v - own;
    base += all;
    __syncthreads();   // the totals are rewritten
  }
  if (tid == 0) start[B] = base;
}

// Jobs (blockIdx.y): 0 .. L-1 states of a layer, L the input x, then (unless w_rows) W_hh and W_ih of each layer; packed: at the
// end the rows of the sentences.
template <typename TE>
__global__ __launch_bounds__(256) void ls_prep_fwd_kernel(LsFwd p, LsPrepFwd s, int jobs) {
  typedef LsMma<TE> M;
  constexpr int V = LsGeom<TE>::kVec, KST = LsGeom<TE>::kKStep;
  const int job = blockIdx.y, H = p.H, B = p.B, L = p.L, nct = (B + 15) >> 4;
  const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
  const int64_t BH = (int64_t)B * H;
  if (p.words.start && job == jobs - 1) {
    if (blockIdx.x == 0) ls_word_starts(p.words.start, p.lengths, p.T, B);
  } else if (job < L) {
    ls_prep_state<TE>(p, job, first, stride, false);
  } else if (job == L) {
    if (p.x_apart) return;
    const int nks = (p.I + KST - 1) / KST;
    const int64_t per = (int64_t)nks * nct * 64, n = per * p.T;
    const TE* x = reinterpret_cast<const TE*>(p.x);
    for (int64_t i = first; i < n; i += stride) {
      const int t = (int)(i / per);
      const int64_t r = i - t * per, tile = r >> 6;
      const int lane = (int)(r & 63), k = (int)(tile / nct) * KST + (lane >> 4) * V;
      const int b = (int)(tile % nct) * 16 + (lane & 15);
      const bool in = b < B && k < p.I;
      ls_copy_chunk<TE>(const_cast<char*>(p.xF) + t * p.x_stride + r * 16,
                        x + ((int64_t)t * B + (in ? b : 0)) * p.I + (in ? k : 0), in ? p.I - k : 0);
    }
    if (M::kPair)
      for (int64_t i = first; i < (int64_t)nct * 64; i += stride)
        *reinterpret_cast<ls_u32x4_t*>(const_cast<char*>(p.zeros) + i * 16) = ls_u32x4_t{0u, 0u, 0u, 0u};
  } else {
    const int l = (job - L - 1) >> 1;
    const bool hh = ((job - L - 1) & 1) == 0;
    if (p.x_apart && l == 0 && !hh) return;
    const int K = hh || l > 0 ? H : p.I, ntw = (H + 31) / 32 * 8;
    const TE* W = reinterpret_cast<const TE*>(hh ? s.W_hh[l] : s.W_ih[l]);
    char* dst = reinterpret_cast<char*>(const_cast<void*>(hh ? p.W_hh[l] : p.W_ih[l]));
    const int nks = (K + KST - 1) / KST;
    const int64_t n = (int64_t)nks * ntw * 64;
    for (int64_t i = first; i < n; i += stride) {
      const int64_t tile = i >> 6;
      const int lane = (int)(i & 63), k = (int)((tile >> 2) % nks) * KST + (lane >> 4) * V;
      const int ug = (int)((tile >> 2) / nks), ii = (int)(tile & 3);
      const int unit = 16 * ug + 4 * M::q_of_row(lane & 15) + ii, gate = M::r_of_row(lane & 15);
      const bool in = unit < H && k < K;
      ls_copy_chunk<TE>(dst + i * 16, W + ((int64_t)gate * H + (in ? unit : 0)) * K + (in ? k : 0), in ? K - k : 0);
    }
  }
}

// n elements of a row by a wave
template <typename TE> __device__ __forceinline__ void ls_copy_row(TE* dst, const TE* src, int n) {
  constexpr int V = 16 / (int)sizeof(TE);
  const int lane = threadIdx.x & 63;
  if (n % V == 0) {
    for (int u = lane * V; u < n; u += 64 * V) *reinterpret_cast<ls_u32x4_t*>(dst + u) = *reinterpret_cast<const ls_u32x4_t*>(src + u);
  } else {
    for (int u = lane; u < n; u += 64) dst[u] = src[u];
  }
}
// What the products over all words read and no wavefront writes, a wave per row: rows of x and of the positions; or the states
// before each sentence's first word.
template <typename TE> __device__ __forceinline__ void ls_prep_words(const LsPrepBwd& s, bool inputs) {
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), waves = (int64_t)gridDim.x * 4;
  const int B = s.B, H = s.H;
  if (inputs) {
    for (int64_t i = wave; i < (int64_t)s.T * B; i += waves) {
      const int t = (int)(i / B), b = (int)(i - (int64_t)t * B), row = s.words.start[b] + t;
      const bool word = row < s.words.start[b + 1];
      if ((threadIdx.x & 63) == 0) s.words.pos[i] = word ? row : -1;
      if (word) ls_copy_row<TE>(reinterpret_cast<TE*>(s.words.x) + (int64_t)row * s.I, reinterpret_cast<const TE*>(s.x) + i * s.I, s.I);
    }
  } else {
    for (int64_t i = wave; i < (int64_t)s.L * B; i += waves) {
      const int l = (int)(i / B), b = (int)(i - (int64_t)l * B), row = s.words.start[b];
      TE* hE = reinterpret_cast<TE*>(s.hE) + (int64_t)l * (s.T + 1) * B * H;
      if (row < s.words.start[b + 1]) ls_copy_row<TE>(hE + ((int64_t)B + row) * H, hE + (int64_t)b * H, H);
    }
  }
}

// blockIdx.y: the weight.  Tile row rho of tile i: unit 16 i + 4 q + r.  Packed: two more for the rows of words.
template <typename TE>
__global__ __launch_bounds__(256) void ls_prep_bwd_kernel(LsPrepBwd s) {
  typedef LsMma<TE> M;
  constexpr int V = LsGeom<TE>::kVec, KST = LsGeom<TE>::kKStep;
  const int H = s.H;
  if ((int)blockIdx.y >= s.n) {
    ls_prep_words<TE>(s, blockIdx.y == s.n);
    return;
  }
  const TE* W = reinterpret_cast<const TE*>(s.W[blockIdx.y]);
  char* dst = s.tiles[blockIdx.y];
  const int GS = ls_gate_stride<TE>(H), ntu = (H + 63) / 64 * 4;
  const int nks = 4 * GS / KST;
  const int64_t n = (int64_t)nks * ntu * 64;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t tile = i >> 6;
    const int lane = (int)(i & 63), rho = lane & 15, k = (int)(tile % nks) * KST + (lane >> 4) * V;
    const int unit = 16 * (int)(tile / nks) + 4 * M::q_of_row(rho) + M::r_of_row(rho);
    const int gate = k / GS, u = k - gate * GS;   // GS % V == 0: a chunk lies inside one gate
    TE v[V];
#pragma unroll
    for (int e = 0; e < V; ++e)
      v[e] = unit < H && u + e < H ? W[((int64_t)gate * H + u + e) * H + unit] : (TE)0;
#pragma unroll
    for (int e = 0; e < V; ++e) reinterpret_cast<TE*>(dst + i * 16)[e] = v[e];
  }
}

__global__ __launch_bounds__(256) void ls_bias_reduce_kernel(const float* __restrict__ dbacc, LsBiasOut o, int nct,
                                                             int cols) {
  const int col = blockIdx.x * 256 + threadIdx.x, l = blockIdx.y;
  if (col >= cols) return;
  const float* a = dbacc + (int64_t)l * nct * cols + col;
  float s = 0.f;
#pragma unroll 8
  for (int ct = 0; ct < nct; ++ct) s += a[(int64_t)ct * cols];
  o.db[l][col] = s;
}

// ---- launches ----------------------------------------------------------------------
// One step: making tiles (64 bytes moved per 16 used once) costs more than the rows' half-used lines do.  128 sentences, 1024
// units: 16 us per layer from rows, 13 from tiles and 7 to make them.  From two steps on the tiles are read again.
template <typename TE> bool ls_reads_weight_rows(int T, int I, int H) {
  return T == 1 && I % LsGeom<TE>::kVec == 0 && H % LsGeom<TE>::kVec == 0;
}

// One step in blocks of 16 sentences: layer 0 reads x and the initial state where they are, a lane's 32 bytes of the state split
// into value and remainder after the load, and blocks behind its own make the tiles of the other layers' states.  That costs a
// layer-step 1 to 4 us, the more bytes a block reads, and saves a launch: a decoder step of 2 x 512 units, 16 sentences 49.8 -> 47.5
// us, 2 x 128 units, 182 sentences 56.4 -> 53.6; blocks of 32 sentences, 4 x 1024 units, 128 sentences 138.6 / 140.0 (all
// layers from their rows 154).
template <typename TE> bool ls_reads_states(int H, int B) {
  return (int64_t)((H + 15) / 16) * ((B + 31) / 32) < (LsMma<TE>::kPair ? 192 : 512);
}

// Folded into the wavefronts, the input product of layer 0 lengthens a chain of T dependent launches by what I reduction
// indices take (0.7 us a launch at I = 512); as one product ahead of them it costs a launch and the round trip of the gates.
// With more than one layer a launch has reductions of 2 H in it anyway.  The number of sentences has no part in the rule: the
// two ways add in different orders, and a sentence's result must not depend on its batch.  Forward, us, folded / apart, at
// T x B, I -> H:
//   L = 1  50 x 16, 512 -> 64: 317 / 304, 1024 -> 256: 373 / 336, 4096 -> 256: 594 / 349, 512 -> 1024: 409 / 404,
//          256 -> 128: 308 / 324; 50 x 128, 512 -> 512: 396 / 392, 512 -> 1024: 516 / 526, 1024 -> 1024: 568 / 546;
//          10 x 512, 512 -> 256: 91 / 99, 2048 -> 512: 208 / 174; 3 x 128, 1024 -> 256: 32 / 36
//   L = 2  50 x 128, 512 -> 256: 363 / 363, 512 -> 512: 467 / 481, 1024 -> 1024: 968 / 1014; 20 x 256, 2048 -> 512: 406 /
//          317; 3 x 128, 2048 -> 512: 59 / 61
//   L = 4  50 x 128, 512 -> 1024: 1385 / 1521, 1024 -> 512: 783 / 727
// fp32 storage is always folded: the matrix instructions bound it, and a sum over both segments is rounded once.
template <typename TE> bool ls_input_apart(int T, int I, int H, int L) {
  return LsMma<TE>::kPair && T > 1 && (int64_t)T * (I - 256) >= 6000 && I >= (L > 1 ? 2 * H : H);
}

// Rows of words alone shorten the products over all steps by the share of padding (30 % where lengths are even over 0.4 T .. T, half
// over 1 .. T) and save a padded step its stores; the rows of x and of the initial states, the way back of dx and rows of a wavefront
// that lie apart cost 4 to 60 us, the more words there are.  So where the weight gradients have enough to do, and enough per word.
// Forward and backward, us, a row per position / per word with lengths over 1 .. T, then over 0.4 T .. T; multiplications of the weight
// gradients, of them per word:
//   bf16  64 x 192, 64 -> 2 x 128      3e9, 2.3e5   896 / 962      891 / 960      60 x 128, 256 -> 2 x 256   8e9, 1.0e6    952 / 962    945 / 965
//         60 x 64, 128 -> 4 x 256      7e9, 2.0e6   992 / 999      987 / 998      64 x 192, 256 -> 4 x 256   3e10, 2.1e6   1473 / 1411  1467 / 1439
//         32 x 64, 512 -> 512          4e9, 2.1e6   506 / 504      503 / 506      32 x 128, 512 -> 512       9e9, 2.1e6    565 / 558    562 / 563
//         50 x 32, 512 -> 4 x 512      1e10, 8.4e6  982 / 979      978 / 986      60 x 64, 512 -> 2 x 512    2e10, 4.2e6   1120 / 1114  1114 / 1118
//         64 x 12, 64 -> 1024          3e9, 4.5e6   1028 / 1029    1020 / 1023    64 x 48, 64 -> 1024        1e10, 4.5e6   1175 / 1167  1168 / 1168
//         40 x 64, 512 -> 2 x 640      2e10, 6.4e6  908 / 892      905 / 904      50 x 64, 512 -> 4 x 1024   1e11, 3.1e7   2234 / 2116  2231 / 2164
//   fp32  60 x 128, 64 -> 2 x 128      2e9, 2.3e5   1109 / 1096    1107 / 1133    30 x 64, 192 -> 192        6e8, 2.9e5    549 / 550    548 / 552
//         24 x 16, 256 -> 384          4e8, 9.8e5   541 / 545      541 / 546      10 x 64, 256 -> 384        6e8, 9.8e5    287 / 281    286 / 284
//         24 x 64, 512 -> 2 x 128      7e8, 4.6e5   543 / 539      542 / 548      24 x 48, 256 -> 2 x 384    2e9, 2.2e6    819 / 770    819 / 788
// (Either way in instances of their own: a choice made in the wavefront kernels cost each launch 0.2 us.  One block finds the rows of
// the sentences.)
template <typename TE> bool ls_packed(int T, int B, int I, int H, int L) {
  const double word = 4.0 * H * (I + H + (L - 1) * 2.0 * H), work = (double)T * B * word;   // multiplications of the weight gradients
  return T > 1 && B <= 16384 && work >= (LsMma<TE>::kPair ? 8e9 : 4e8) && word >= (LsMma<TE>::kPair ? 2e6 : 3e5);
}

template <typename TE> hipError_t launch_ls_prep_fwd(const LsFwd& p, const LsPrepFwd& q, hipStream_t st) {
  constexpr int KST = LsGeom<TE>::kKStep;
  const int64_t nct = ls_batch_tiles(p.B);
  int64_t n = ls_ksteps<TE>(p.H) * nct * 64;   // largest job, in chunks
  const int I = p.x_apart ? 0 : p.I;
  const int64_t nx = (int64_t)ls_ksteps<TE>(I) * nct * 64 * p.T;
  if (nx > n) n = nx;
  if (!p.w_rows) {
    const int64_t nw = (int64_t)((I > p.H ? I : p.H) + KST - 1) / KST * ls_gate_tiles(p.H) * 64;
    if (nw > n) n = nw;
  }
  int64_t gx = (n + 255) / 256;
  if (gx > 1024) gx = 1024;
  const int jobs = p.L + 1 + (p.w_rows ? 0 : 2 * p.L) + (p.words.start ? 1 : 0);
  hipLaunchKernelGGL(ls_prep_fwd_kernel<TE>, dim3((unsigned)gx, jobs), dim3(256), 0, st, p, q, jobs);
  return hipGetLastError();
}
template <typename TE> hipError_t launch_ls_prep_bwd(const LsPrepBwd& q, hipStream_t st) {
  const int jobs = q.n + (q.words.start ? 2 : 0);
  if (jobs < 1) return hipSuccess;
  const int64_t n = (int64_t)(4 * ls_gate_stride<TE>(q.H) / LsGeom<TE>::kKStep) * ls_unit_tiles(q.H) * 64;
  int64_t gx = (n + 255) / 256;
  if (gx > 1024) gx = 1024;
  hipLaunchKernelGGL(ls_prep_bwd_kernel<TE>, dim3((unsigned)gx, jobs), dim3(256), 0, st, q);
  return hipGetLastError();
}
__global__ __launch_bounds__(256) void ls_copy_kernel(LsCopy c) {
  const int j = blockIdx.y;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(c.src[j]);
  uint32_t* dst = reinterpret_cast<uint32_t*>(c.dst[j]);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < c.words[j]; i += (int64_t)gridDim.x * 256) dst[i] = src[i];
}
hipError_t launch_ls_copy(const LsCopy& c, hipStream_t st) {
  hipLaunchKernelGGL(ls_copy_kernel, dim3(256, c.n), dim3(256), 0, st, c);
  return hipGetLastError();
}
hipError_t launch_ls_bias_reduce(const float* dbacc, const LsBiasOut& o, int L, int nct, int cols, hipStream_t st) {
  hipLaunchKernelGGL(ls_bias_reduce_kernel, dim3((cols + 255) / 256, L), dim3(256), 0, st, dbacc, o, nct, cols);
  return hipGetLastError();
}

// One step: how many steps of the weight rows, which come from memory, a wave of the smaller blocks has in flight; K: the
// layer's input width.  With PF in flight PF - 1 - n % PF loads of n steps are past the end and waited for with the others: three of
// four in flight where four divides n.  There, up to eight steps (what registers hold of 16 x 16 blocks), all are requested at once and
// none is past the end; else six in flight where they save two such loads.  A layer-step of H units from H, 16 x 16 blocks, us
// with four / six / all: n = 1 (64) 5.8 / 6.7, 4 (256) 7.8 / 7.1 / 6.8, 5 (320) 8.0 / 7.5 / 7.6, 6 (384) 8.1 / 9.8 / 8.0, 7 (448) 8.2 / 9.8 /
// 8.8, 8 (512) 10.1 / - / 9.2, 10 (640) 9.8 / 10.0, 12 (768) 11.8 / 12.7, 14 (896) 11.9 / 12.8, 16 (1024) 14.0 / 13.2, 17 (1088) 14.1 / 13.3,
// 20 (1280) 16.3 / 16.4, 22 (1408) 16.2 / 16.2; 16 x 32 blocks, 8 (512) 10.8 / 11.1, 14 13.4 / 15.0, 16 16.0 / 15.6.  (Eight: 4 x 1024
// units x 128 sentences 75.4, six 68.5.  Layer 0 of ls_reads_states, which splits the states it loads: four, 256 -> 512 units 9.9,
// all at once 11.4.)
static int ls_row_steps(int K, int H) {   // of a wave
  constexpr int KST = LsGeom<uint16_t>::kKStep;
  return ((H + KST - 1) / KST + (K + KST - 1) / KST + LS_KS - 1) / LS_KS;
}
int ls_row_steps_in_flight(int K, int H) {
  const int n = ls_row_steps(K, H);
  return 5 - n % 6 + 2 <= 3 - n % 4 ? 6 : 4;
}

template <typename TE, int NI, int NJ, int PF, int PF_ROWS = PF>
static hipError_t ls_fwd_shape(const LsFwd& p, int d, int l_lo, int nl, hipStream_t st) {
  const unsigned grid = ls_grid((int64_t)nl * ((p.H + 4 * NI - 1) / (4 * NI)), (p.B + 16 * NJ - 1) / (16 * NJ));
  // one step, layer 0: blocks behind its own prepare the states of the other layers
  const int64_t chunks = (int64_t)ls_ksteps<TE>(p.H) * ls_batch_tiles(p.B) * 64, per = (chunks + 64 * LS_KS - 1) / (64 * LS_KS);
  const unsigned others = p.direct && l_lo == 0 && p.L > 1 ? (unsigned)(p.L * (per < 64 ? per : 64)) : 0;
  const bool packed = p.words.start != nullptr;
#define ASX_FWD_P(ROWS, VEC, APART, PACKED)                                                                          \
  hipLaunchKernelGGL((ls_wave_fwd_kernel<TE, NI, NJ, ROWS ? PF_ROWS : PF, ROWS, VEC, APART, PACKED>), dim3(grid + others), dim3(64 * LS_KS), \
                     0, st, p, d, l_lo, nl)
#define ASX_FWD(ROWS, VEC, APART)                                         \
  do {                                                                    \
    if (ROWS == 0 && packed) ASX_FWD_P(ROWS, VEC, APART, (ROWS == 0));    \
    else ASX_FWD_P(ROWS, VEC, APART, false);                              \
  } while (0)
  if (p.x_apart && p.w_rows) return hipErrorInvalidValue;   // (ls_input_apart: not with one step)
  if constexpr (NJ == 1 && PF_ROWS == PF) {
    if (p.direct && l_lo == 0) {
      ASX_FWD(2, true, false);   // (widths are whole vectors)
      return hipGetLastError();
    }
  }
  if (p.w_rows) ASX_FWD(1, true, false);
  else if (LsMma<TE>::kPair && p.x_apart && l_lo == 0) ASX_FWD(0, true, LsMma<TE>::kPair);
  else if (LsMma<TE>::kPair || p.H % 4 == 0) ASX_FWD(0, true, false);
  else ASX_FWD(0, LsMma<TE>::kPair, false);
#undef ASX_FWD
#undef ASX_FWD_P
  return hipGetLastError();
}
template <typename TE, int NI, int NJ, int PF>
static hipError_t ls_bwd_shape(const LsBwd& p, int d, int l_lo, int nl, hipStream_t st) {
  const unsigned grid = ls_grid((int64_t)nl * ((p.H + 16 * NI - 1) / (16 * NI)), (p.B + 16 * NJ - 1) / (16 * NJ));
  constexpr bool kAnyVec = LsMma<TE>::kPair;   // (bf16 widths are whole vectors)
  const bool vec = kAnyVec || p.H % 4 == 0;
  auto k = p.words.start ? (vec ? ls_wave_bwd_kernel<TE, NI, NJ, PF, true, true> : ls_wave_bwd_kernel<TE, NI, NJ, PF, kAnyVec, true>)
                         : (vec ? ls_wave_bwd_kernel<TE, NI, NJ, PF, true, false> : ls_wave_bwd_kernel<TE, NI, NJ, PF, kAnyVec, false>);
  hipLaunchKernelGGL(k, dim3(grid), dim3(64 * LS_KS), 0, st, p, d, l_lo, nl);
  return hipGetLastError();
}

template <typename TE> hipError_t launch_ls_wave_fwd(const LsFwd& p, int d, hipStream_t st) {
  const int l_lo = d - p.T + 1 > 0 ? d - p.T + 1 : 0, l_hi = d < p.L - 1 ? d : p.L - 1;   // 0 <= d - l < T
  const int nl = l_hi - l_lo + 1;
  if (nl < 1) return hipErrorInvalidValue;
  const int64_t b64 = (p.B + 63) / 64, b32 = (p.B + 31) / 32;
  // The largest block that still gives most compute units one: larger blocks load less per output (128 gate rows x 64
  // sentences: 512 bytes per reduction index for 8192 outputs).  1024 units x 128 sentences, 64 x 32 blocks against 128 x 64:
  // three layers 27.5 us (768 blocks) and 28.0 (192), four 34.0 (1024) and 29.4 (256).
  if constexpr (LsMma<TE>::kPair) {
    if (nl * ((p.H + 31) / 32) * b64 >= 192) return ls_fwd_shape<TE, 8, 4, 3>(p, d, l_lo, nl, st);
    const int64_t blocks = nl * ((p.H + 15) / 16) * b32;   // (ls_reads_states: the same line)
    const int K = l_lo == 0 ? p.I : p.H, pf = p.w_rows ? ls_row_steps_in_flight(K, p.H) : 4;   // (one step: one layer)
    // (six take the registers of a second block of 16 x 32: not where compute units get one)
    if (blocks >= 192 && pf == 6 && blocks <= 256) return ls_fwd_shape<TE, 4, 2, 4, 6>(p, d, l_lo, nl, st);
    if (blocks >= 192) return ls_fwd_shape<TE, 4, 2, 4>(p, d, l_lo, nl, st);
    if (p.direct && l_lo == 0) return ls_fwd_shape<TE, 4, 1, 4>(p, d, l_lo, nl, st);
    if (p.w_rows) {
      const int n = ls_row_steps(K, p.H);   // all at once: a slot more than steps
      if (n == 4) return ls_fwd_shape<TE, 4, 1, 4, 5>(p, d, l_lo, nl, st);
      if (n == 8) return ls_fwd_shape<TE, 4, 1, 4, 9>(p, d, l_lo, nl, st);
    }
    return pf == 6 ? ls_fwd_shape<TE, 4, 1, 4, 6>(p, d, l_lo, nl, st) : ls_fwd_shape<TE, 4, 1, 4>(p, d, l_lo, nl, st);
  } else {   // (ls_reads_states: the same line)
    if (nl * ((p.H + 15) / 16) * b32 >= 512) return ls_fwd_shape<TE, 4, 2, 4>(p, d, l_lo, nl, st);
    return ls_fwd_shape<TE, 4, 1, 4>(p, d, l_lo, nl, st);
  }
}

template <typename TE> hipError_t launch_ls_wave_bwd(const LsBwd& p, int d, hipStream_t st) {
  const int dl = p.L - 1;                              // layer l takes step T - 1 - (d - (dl - l))
  const int tail = p.dh0 ? p.T : p.T - 1;              // largest d - (dl - l)
  const int l_hi = dl - (d - tail > 0 ? d - tail : 0), l_lo = dl - (d < dl ? d : dl);
  const int nl = l_hi - l_lo + 1;
  if (nl < 1) return hipErrorInvalidValue;
  const int64_t b32 = (p.B + 31) / 32;
  // as forward; four layers of 1024 units x 128 sentences in 256 blocks of 64 x 32: 32.4 us, 512 of 32 x 32: 33.7, 128 of
  // 64 x 64: 43.4 (before the loads were spread)
  if constexpr (LsMma<TE>::kPair) {
    if (nl * ((p.H + 63) / 64) * b32 >= 192) return ls_bwd_shape<TE, 4, 2, 4>(p, d, l_lo, nl, st);
    if (nl * ((p.H + 31) / 32) * b32 >= 192) return ls_bwd_shape<TE, 2, 2, 4>(p, d, l_lo, nl, st);
    return ls_bwd_shape<TE, 1, 2, 4>(p, d, l_lo, nl, st);
  } else {
    if (nl * ((p.H + 15) / 16) * b32 >= 512) return ls_bwd_shape<TE, 1, 2, 4>(p, d, l_lo, nl, st);
    return ls_bwd_shape<TE, 1, 1, 4>(p, d, l_lo, nl, st);
  }
}

#define ASX_LS(TE)                                                                                  \
  template bool ls_reads_weight_rows<TE>(int, int, int);                                            \
  template bool ls_reads_states<TE>(int, int);                                                      \
  template bool ls_packed<TE>(int, int, int, int, int);                                             \
  template bool ls_input_apart<TE>(int, int, int, int);                                             \
  template hipError_t launch_ls_prep_fwd<TE>(const LsFwd&, const LsPrepFwd&, hipStream_t);          \
  template hipError_t launch_ls_prep_bwd<TE>(const LsPrepBwd&, hipStream_t);                        \
  template hipError_t launch_ls_wave_fwd<TE>(const LsFwd&, int, hipStream_t);                       \
  template hipError_t launch_ls_wave_bwd<TE>(const LsBwd&, int, hipStream_t);
ASX_LS(uint16_t)
ASX_LS(float)
#undef ASX_LS

}  // namespace asx
