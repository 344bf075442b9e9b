// Fused attention for the batched path, bf16 storage (section 3.2, Eq. 1-3): one workgroup per
// (sentence b, block of 16 or 32 decoder steps) computes
//   score[t,s] = (q_hi + q_lo)[t,b,:] . h_enc[s,b,:]      (Eq. 2; q = h_dec W_a as value + rounding remainder)
//   alpha[t,:] = softmax over s < src_len[b], exactly 0 elsewhere   (Eq. 1)
//   ctx[t,b,:] = sum_s alpha[t,s] h_enc[s,b,:]             (Eq. 3; alpha enters as value + remainder)
// without the scores ever leaving the compute unit.
// The same kernel with BWD = true is the first half of the attention backward pass, which has the same shape:
//   dalpha[t,s] = (dC_hi + dC_lo)[t,b,:] . h_enc[s,b,:]
//   dscore[t,:] = alpha[t,:] * (dalpha[t,:] - sum_s alpha[t,s] dalpha[t,s])      (softmax Jacobian)
//   dQ[t,b,:]   = sum_s dscore[t,s] h_enc[s,b,:]
// (dscore also leaves as bf16 value / remainder for the product that forms d_h_enc).
//
// A few hundred KiB per workgroup: what counts is that they are requested early and by many waves, so eight waves share a
// workgroup, none of them waits for another inside a phase, and phase 3's first operand is requested before phase 1.
// Phase 1 (scores): matrix fragments straight from global memory into registers.  A wave takes pairs of 32-wide reduction
//   steps (whole 128-byte lines of its rows), a pair ahead on its way; pairs w, w + 8, ... go to wave w, and the eight
//   partial sums are added in wave order whatever T and B are.
// Phase 2 (softmax): one wavefront per row, shuffle reductions, all rows of a wave at once; alpha goes to global memory
//   (float, and the bf16 value / remainder copies the backward pass reads) and to LDS as the row operand of phase 3.
// Phase 3 (context): the reduction runs over source positions, so h_enc_b is the strided operand: a wave brings its chunks
//   of 64 columns (32 where S > 64) as stored into two LDS slots of its own, directly, and reads them transposing.
// One workgroup per 32 decoder steps where that makes 192 of them, else per 16, so that more compute units have one
// (us, 32 / 16 steps: 64 / 128 workgroups of S 30 H 512 10.2 / 7.5, 122 / 183 of S 43 H 1000 16.3 / 12.8, 256 / 512 of S 50
// H 1024 20.8 / 24.4, 512 / 1024 of S 64 H 2048 104 / 129); S > 64: 16, by the LDS.  Four waves, two workgroups per compute
// unit: 8.4, 13.8, 23.3, 107.  The kernel this replaced, four waves that brought both operands through LDS a tile ahead in
// registers: 20.6, 32.8, 36.4, 104 forward and 17.3, -, 33.5, 108 backward (now 6.2, -, 18.1, 91); T 80 S 80 B 128 H 1024
// 69 and 66, now 43 and 43; T 1 S 50 B 128 H 1024 29, now 9.5.
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "lds_limit.h"
#include "gemm_dev.h"
#include "row_list_dev.h"

namespace asx {

namespace {

typedef uint32_t af_u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) void af_glb_void_t;

constexpr int AF_NW = 8;        // waves of a workgroup
constexpr int kGridY = 65535;   // a grid's limit in y

// alpha operand blocks: rows of 64 elements (128 bytes), chunk c of row r at chunk c ^ (r & 7) ^ ((r >> 3) & 1)
__device__ __forceinline__ uint32_t kc_off(int row, int chunk) {
  return (uint32_t)(row * 128 + ((chunk ^ (row & 7) ^ ((row >> 3) & 1)) << 4));
}

struct AttnFwdArgs {
  const uint16_t *q_hi, *q_lo, *h_enc;   // row operand of phase 1 as value / remainder (q, or dC for BWD), encoder states
  const int32_t* src_len;
  float* alpha32;                        // forward: written; BWD: read
  uint16_t *alphaE, *alphaE_lo;          // [B,T,ldS] copies of the row result (alpha, or dscore for BWD)
  uint16_t *ctx, *ctx_lo;                // phase-3 result (ctx + remainder, or dQ with ctx_lo = null for BWD)
  uint8_t* attn_mask;
  int T, S, B, H;
  int64_t ldS;
  int y0;                                // first block of decoder steps of this launch
};
struct AttnFwdMore : AttnFwdArgs {
  int32_t* zero;                         // cleared, if not null
  RowList list;                          // made by the blocks x = B, y = 0 of the first launch, if wanted
};

// LDS of a workgroup of 16 RT decoder steps x 16 ST source positions: a slot of NT x 16 columns of encoder states per wave;
// the score partial sums, later a second slot per wave; the row results
template <int RT, int ST> struct AttnLds {
  static constexpr int kRows = 16 * RT, kSld = 16 * ST + 4;
  static constexpr int kNT = ST <= 4 ? 4 : 2, kRB = kNT * 32;           // slot rows: bytes
  static constexpr int kSlot = 16 * ST * kRB, kPart = kRows * kSld * 4;  // bytes per wave
  static constexpr int kX = AF_NW * kSlot, kA = kX + AF_NW * (kPart > kSlot ? kPart : kSlot);
  static constexpr int kBlk = kRows * 128, kKB = (16 * ST + 63) / 64;
  static constexpr int kBytes = kA + 2 * kKB * kBlk;
  static_assert(kBytes <= 160 * 1024, "LDS of a compute unit");
};

// 16-byte piece c of slot row k is kept at c ^ slot_swizzle(k): the four rows of a transposing read lie in different banks
template <int NT> __device__ __forceinline__ int slot_swizzle(int k) { return NT == 4 ? (k & 2) << 1 : 0; }

// Args: AttnFwdMore where the forward pass has either to do, an instance of its own: its arguments and tests cost the others 0.3 us (53 x
// 52, H 256 7.2 / 6.9, 29 x 7, H 192 6.1 / 5.8).
template <bool BWD, int RT, int ST, typename Args>
__global__ __launch_bounds__(64 * AF_NW) void attn_fused_kernel(Args p) {
  typedef AttnLds<RT, ST> Lds;
  constexpr int NW = AF_NW, ROWS = Lds::kRows, SLD = Lds::kSld, KB = Lds::kKB, NT = Lds::kNT, RB = Lds::kRB;
  extern __shared__ __align__(1024) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  if constexpr (std::is_same<Args, AttnFwdMore>::value) {
    if (p.zero && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *p.zero = 0;
    if (blockIdx.x == (unsigned)p.B) {
      if (blockIdx.y == 0) row_list_block<64 * AF_NW>(p.list, reinterpret_cast<int*>(smem));
      return;
    }
  }
  const int b = blockIdx.x, t0 = (p.y0 + blockIdx.y) * ROWS;
  const int T = p.T, S = p.S, H = p.H;
  const int64_t BH = (int64_t)p.B * H;
  int L = p.src_len[b];
  L = L < 0 ? 0 : (L > S ? S : L);
  const int last = L > 0 ? L - 1 : 0;   // source rows past the sentence are read from its last word: their weights are 0
  const uint16_t* he = p.h_enc + (int64_t)b * H;

  // ---------------- phase 3's first chunk of encoder states, requested first --------------------------------------
  const int nk3 = (L + 31) >> 5, nch = (H + 16 * NT - 1) / (16 * NT);   // reduction steps of 32 source positions; chunks
  auto load_chunk = [&](int c, unsigned char* slot) {
    constexpr int CPR = RB / 16, RPL = 64 / CPR;   // 16-byte pieces of a row, rows per load
    const int kr = lane / CPR, col = c * 16 * NT + ((lane % CPR) ^ slot_swizzle<NT>(kr)) * 8;
    const uint16_t* src = he + (col < H ? col : 0);
    for (int i = 0; i < 32 / RPL * nk3; ++i) {
      const int k = i * RPL + kr;
      __builtin_amdgcn_global_load_lds((af_glb_void_t*)(src + (k < L ? k : last) * BH), (lds_void_t*)(slot + i * 1024), 16, 0, 0);
    }
  };
  if (wave < nch) load_chunk(wave, smem + wave * Lds::kSlot);
  constexpr int RPW = ROWS / NW;        // rows of phase 2 per wave
  float al[RPW][KB];                    // BWD: their weights
  if constexpr (BWD) {
#pragma unroll
    for (int r = 0; r < RPW; ++r)
#pragma unroll
      for (int h = 0; h < KB; ++h) {
        const int t = t0 + wave * RPW + r, s = lane + 64 * h;
        al[r][h] = p.alpha32[((int64_t)b * T + (t < T ? t : T - 1)) * S + (s < S ? s : 0)];
      }
  }

  // ---------------- phase 1: scores -------------------------------------------------------------------------------
  {
    const uint16_t *qh[RT], *ql[RT], *hr[ST];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int t = t0 + 16 * r + c16;
      const int64_t off = (int64_t)(t < T ? t : T - 1) * BH + (int64_t)b * H;
      qh[r] = p.q_hi + off;
      ql[r] = p.q_lo + off;
    }
#pragma unroll
    for (int j = 0; j < ST; ++j) {
      const int s = 16 * j + c16;
      hr[j] = he + (s < L ? s : last) * BH;
    }
    f32x4_t acc[RT][ST];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int j = 0; j < ST; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[r][j][e] = 0.f;
    // Steps 2 i and 2 i + 1 of a pair go through register slots 0 and 1: a pair ahead is on its way.
    af_u32x4_t fq[2][RT], fl[2][RT], fh[2][ST];
    auto load = [&](int slot, int i) {  // half `slot` of the wave's i-th pair
      const int k = (2 * (wave + i * NW) + slot) * 32 + q4 * 8, kk = k < H ? k : 0;
#pragma unroll
      for (int j = 0; j < ST; ++j) fh[slot][j] = *reinterpret_cast<const af_u32x4_t*>(hr[j] + kk);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        fq[slot][r] = *reinterpret_cast<const af_u32x4_t*>(qh[r] + kk);
        fl[slot][r] = *reinterpret_cast<const af_u32x4_t*>(ql[r] + kk);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](int slot, int i) {
      const int k0 = (2 * (wave + i * NW) + slot) * 32;
      if (k0 + 32 > H) {                // reduction indices past the end were read from the row's start
        const bool in = k0 + q4 * 8 < H;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int j = 0; j < ST; ++j) fh[slot][j][e] = in ? fh[slot][j][e] : 0u;
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            fq[slot][r][e] = in ? fq[slot][r][e] : 0u;
            fl[slot][r][e] = in ? fl[slot][r][e] : 0u;
          }
        }
      }
#pragma unroll
      for (int j = 0; j < ST; ++j) {
        const bf16x8_t a = __builtin_bit_cast(bf16x8_t, fh[slot][j]);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8_t, fq[slot][r]), acc[r][j], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8_t, fl[slot][r]), acc[r][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    const int npair = (H + 63) / 64, n = npair > wave ? (npair - wave + NW - 1) / NW : 0;
    if (n > 0) {
      load(0, 0);
      load(1, 0);
      for (int i = 0; i + 1 < n; ++i) {
        mul(0, i);
        load(0, i + 1);
        mul(1, i);
        load(1, i + 1);
      }
      mul(0, n - 1);
      mul(1, n - 1);
    }
    float* part = reinterpret_cast<float*>(smem + Lds::kX) + wave * (ROWS * SLD);
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int j = 0; j < ST; ++j)
        *reinterpret_cast<f32x4_t*>(part + (16 * r + c16) * SLD + 16 * j + 4 * q4) = acc[r][j];
  }
  __syncthreads();

  // ---------------- phase 2: masked softmax rows, or the softmax Jacobian ------------------------------------------
  unsigned char* a_hi = smem + Lds::kA;             // [KB][rows][64] value
  unsigned char* a_lo = a_hi + KB * Lds::kBlk;      // same, rounding remainder
  {
    const float* part = reinterpret_cast<const float*>(smem + Lds::kX);
    float x[RPW][KB], a[RPW][KB];
#pragma unroll
    for (int r = 0; r < RPW; ++r)
#pragma unroll
      for (int h = 0; h < KB; ++h) {
        const int s = lane + 64 * h;
        const float* q = part + (wave * RPW + r) * SLD + (s < 16 * ST ? s : 0);
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += q[w * (ROWS * SLD)];
        x[r][h] = v;
      }
    if constexpr (!BWD) {
#pragma unroll
      for (int r = 0; r < RPW; ++r) {
        float m = -INFINITY, sum = 0.f;
#pragma unroll
        for (int h = 0; h < KB; ++h) m = lane + 64 * h < L ? fmaxf(m, x[r][h]) : m;
        m = wave_max(m);
#pragma unroll
        for (int h = 0; h < KB; ++h) {
          a[r][h] = lane + 64 * h < L ? expf(x[r][h] - m) : 0.f;   // masked positions: exactly 0
          sum += a[r][h];
        }
        sum = wave_sum(sum);
        const float inv = L > 0 ? 1.f / sum : 0.f;
#pragma unroll
        for (int h = 0; h < KB; ++h) a[r][h] *= inv;
      }
    } else {
      // alpha is 0 at masked positions, so dscore is exactly 0 there
#pragma unroll
      for (int r = 0; r < RPW; ++r) {
        float dot = 0.f;
#pragma unroll
        for (int h = 0; h < KB; ++h) {
          const bool in = lane + 64 * h < L && t0 + wave * RPW + r < T;
          al[r][h] = in ? al[r][h] : 0.f;
          x[r][h] = in ? x[r][h] : 0.f;
          dot += al[r][h] * x[r][h];
        }
        dot = wave_sum(dot);
#pragma unroll
        for (int h = 0; h < KB; ++h) a[r][h] = al[r][h] * (x[r][h] - dot);
      }
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r)
#pragma unroll
      for (int h = 0; h < KB; ++h) {
        const int row = wave * RPW + r, t = t0 + row, s = lane + 64 * h;
        const uint32_t hb = f32_to_bf16_bits(a[r][h]);
        const uint32_t lb = f32_to_bf16_bits(a[r][h] - bf16_bits_to_f32(hb));
        const uint32_t o = (uint32_t)(h * Lds::kBlk) + kc_off(row, (s & 63) >> 3) + (uint32_t)(s & 7) * 2;
        *reinterpret_cast<uint16_t*>(a_hi + o) = (uint16_t)hb;   // operand of phase 3 (zeros beyond the valid positions)
        *reinterpret_cast<uint16_t*>(a_lo + o) = (uint16_t)lb;
        if (t < T) {
          if constexpr (!BWD)
            if (s < S) p.alpha32[((int64_t)b * T + t) * S + s] = a[r][h];
          if (s < p.ldS) {
            p.alphaE[((int64_t)b * T + t) * p.ldS + s] = (uint16_t)hb;
            p.alphaE_lo[((int64_t)b * T + t) * p.ldS + s] = (uint16_t)lb;
          }
        }
      }
    if (!BWD && p.attn_mask && t0 == 0)
      for (int s = tid; s < S; s += 64 * NW) p.attn_mask[(int64_t)b * S + s] = s < L ? 1 : 0;
  }
  __builtin_amdgcn_s_waitcnt(0);   // the first chunk has landed (each wave reads its own slots only)
  __syncthreads();                 // row results complete; the partial sums are dead from here on

  // ---------------- phase 3: context vectors, each wave over its 64-column chunks of H ------------------------------
  // Transposing reads: lane j of a 16-lane group presents four columns of k-row j / 4 and gets four k of the column that
  // is its row of the matrix instruction.  Tile i's rows 4 q .. 4 q + 3 are the columns 32 (i / 2) + 8 q + 4 (i % 2) ..: a
  // lane then holds eight consecutive columns of its decoder step in two tiles.
  uint32_t fb[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int k = q4 * 8 + (c16 >> 2), piece = (4 * (i >> 1) + (lane & 3)) ^ slot_swizzle<NT>(k);
    fb[i] = (uint32_t)(k * RB + piece * 16 + (i & 1) * 8);
  }
  int par = 0;
  for (int c = wave; c < nch; c += NW, par ^= 1) {
    const unsigned char* slot = smem + par * Lds::kX + wave * Lds::kSlot;
    if (c + NW < nch) load_chunk(c + NW, smem + (par ^ 1) * Lds::kX + wave * Lds::kSlot);
    f32x4_t acc[RT][NT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[r][i][e] = 0.f;
    for (int ks = 0; ks < nk3; ++ks) {
      bf16x8_t f[NT];
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        union { s16x4_t h[2]; bf16x8_t v; } u;
        u.h[0] = lds_read_tr((lds_s16x4_t*)(lds_void_t*)(slot + fb[i] + ks * 32 * RB));
        u.h[1] = lds_read_tr((lds_s16x4_t*)(lds_void_t*)(slot + fb[i] + ks * 32 * RB + 4 * RB));
        f[i] = u.v;
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const uint32_t o = (uint32_t)((ks >> 1) * Lds::kBlk) + kc_off(16 * r + c16, (ks & 1) * 4 + q4);
        const bf16x8_t ah = *reinterpret_cast<const bf16x8_t*>(a_hi + o), alo = *reinterpret_cast<const bf16x8_t*>(a_lo + o);
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[i], ah, acc[r][i], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < NT; ++i) acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[i], alo, acc[r][i], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);   // the next chunk has landed; this one's stores are not waited for until the next time
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int t = t0 + 16 * r + c16;
#pragma unroll
      for (int g = 0; g < NT / 2; ++g) {
        const int col = c * 16 * NT + g * 32 + q4 * 8;
        if (t >= T || col >= H) continue;
        af_u32x4_t hv, lv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x4_t& v4 = acc[r][2 * g + (e >> 1)];
          const float v0 = v4[2 * (e & 1)], v1 = v4[2 * (e & 1) + 1];
          const uint32_t h0 = f32_to_bf16_bits(v0), h1 = f32_to_bf16_bits(v1);
          hv[e] = h0 | (h1 << 16);
          lv[e] = pack_bf16(v0 - bf16_bits_to_f32(h0), v1 - bf16_bits_to_f32(h1));
        }
        const int64_t o = (int64_t)t * BH + (int64_t)b * H + col;
        *reinterpret_cast<af_u32x4_t*>(p.ctx + o) = hv;
        if constexpr (!BWD) *reinterpret_cast<af_u32x4_t*>(p.ctx_lo + o) = lv;
      }
    }
  }
}

}  // namespace

bool attn_fwd_fused_supported(int S, int H) { return S >= 1 && S <= 128 && (H % 8) == 0; }

template <bool BWD, int RT, int ST, typename Args> static hipError_t launch_attn_shape(Args p, hipStream_t st) {
  auto k = attn_fused_kernel<BWD, RT, ST, Args>;
  constexpr int smem = AttnLds<RT, ST>::kBytes;
  static LdsLimit limit;
  const hipError_t e = limit.raise(reinterpret_cast<const void*>(k), smem);
  if (e != hipSuccess) return e;
  const int ny = (p.T + 16 * RT - 1) / (16 * RT);
  for (p.y0 = 0; p.y0 < ny; p.y0 += kGridY) {   // (more than a million decoder steps: several launches)
    int list = 0;
    if constexpr (std::is_same<Args, AttnFwdMore>::value) list = p.y0 == 0 && p.list.targets ? 1 : 0;
    hipLaunchKernelGGL(k, dim3(p.B + list, ny - p.y0 < kGridY ? ny - p.y0 : kGridY), dim3(64 * AF_NW), smem, st, p);
    const hipError_t launched = hipGetLastError();
    if (launched != hipSuccess) return launched;
  }
  return hipSuccess;
}
template <bool BWD, typename Args> static hipError_t launch_attn_fused(const Args& p, hipStream_t st) {
  if (!attn_fwd_fused_supported(p.S, p.H) || p.B < 1 || p.T < 1 || p.ldS < p.S || p.ldS > 128) return hipErrorInvalidValue;
  // (the order of every sum is the same in all of them; the figures are at the head of this file)
  if (p.S > 64) return launch_attn_shape<BWD, 1, 8>(p, st);
  const bool wide = (int64_t)p.B * ((p.T + 31) / 32) >= 192;
  if (p.S > 32) return wide ? launch_attn_shape<BWD, 2, 4>(p, st) : launch_attn_shape<BWD, 1, 4>(p, st);
  return wide ? launch_attn_shape<BWD, 2, 2>(p, st) : launch_attn_shape<BWD, 1, 2>(p, st);
}

hipError_t launch_attn_fwd_fused(const void* q_hi, const void* q_lo, const void* h_enc, const int32_t* src_len, int B,
                                 int T, int S, int H, float* alpha32, void* alphaE, void* alphaE_lo, int64_t ldS,
                                 void* ctx, void* ctx_lo, uint8_t* attn_mask, const RowList& list, int32_t* zero, hipStream_t st) {
  AttnFwdMore p{};
  p.zero = zero;
  p.list = list;
  p.q_hi = reinterpret_cast<const uint16_t*>(q_hi);
  p.q_lo = reinterpret_cast<const uint16_t*>(q_lo);
  p.h_enc = reinterpret_cast<const uint16_t*>(h_enc);
  p.src_len = src_len;
  p.alpha32 = alpha32;
  p.alphaE = reinterpret_cast<uint16_t*>(alphaE);
  p.alphaE_lo = reinterpret_cast<uint16_t*>(alphaE_lo);
  p.ctx = reinterpret_cast<uint16_t*>(ctx);
  p.ctx_lo = reinterpret_cast<uint16_t*>(ctx_lo);
  p.attn_mask = attn_mask;
  p.T = T; p.S = S; p.B = B; p.H = H;
  p.ldS = ldS;
  return zero || list.targets ? launch_attn_fused<false>(p, st) : launch_attn_fused<false>(static_cast<const AttnFwdArgs&>(p), st);
}

hipError_t launch_attn_bwd_fused(const void* dC_hi, const void* dC_lo, const void* h_enc, const int32_t* src_len,
                                 int B, int T, int S, int H, const float* alpha32, void* dscoreE, void* dscoreE_lo,
                                 int64_t ldS, void* dQ, hipStream_t st) {
  AttnFwdArgs p{};
  p.q_hi = reinterpret_cast<const uint16_t*>(dC_hi);
  p.q_lo = reinterpret_cast<const uint16_t*>(dC_lo);
  p.h_enc = reinterpret_cast<const uint16_t*>(h_enc);
  p.src_len = src_len;
  p.alpha32 = const_cast<float*>(alpha32);
  p.alphaE = reinterpret_cast<uint16_t*>(dscoreE);
  p.alphaE_lo = reinterpret_cast<uint16_t*>(dscoreE_lo);
  p.ctx = reinterpret_cast<uint16_t*>(dQ);
  p.ctx_lo = nullptr;
  p.attn_mask = nullptr;
  p.T = T; p.S = S; p.B = B; p.H = H;
  p.ldS = ldS;
  return launch_attn_fused<true>(p, st);
}

}  // namespace asx
