// Fused attention for fp32 storage (section 3.2, Eq. 1-3), the forward pass and the first half of the backward pass: what
// attn_fused.hip does for bf16, one workgroup per (sentence, 16 decoder steps), on the fp64 matrix cores.
//   score[t,s] = (q + q_lo)[t,b,:] . h_enc[s,b,:]    alpha[t,:] = softmax over s < src_len[b]    ctx = sum_s alpha[t,s] h_enc[s,b,:]
//   BWD: dalpha = (dC + dC_lo) . h_enc    dscore = alpha (dalpha - sum alpha dalpha)    dQ = sum_s dscore[t,s] h_enc[s,b,:]
// Products and sums are fp64 and rounded to float where the separate launches (two batched products and the row kernel) store
// floats.  Value and remainder of the row operand are added before the product, exactly: half its matrix instructions.
//
// The time is launches and a few memory latencies, so fragments come straight into registers, a step ahead:
//   phase 1: a wave takes every fourth step of 16 reduction indices (lane group q: indices 4 q .. 4 q + 3, a 16-byte load); the
//     four partial sums meet in LDS;  phase 2: a wavefront per row;  phase 3: a wave takes 64 columns of h_enc_b at a time, lane
//     n of a group columns 4 n .. 4 n + 3, so that loads and stores are 16 bytes.
// us, three launches / one: 4 x 8 steps, S 8, H 64 14.8 / 6.0 forward, 13.8 / 4.8 backward; 64 x 30, S 30, H 512 33 / 15.4 and 34 /
// 14.4.  A training step of 32 rows x 64 units 78.8 / 65.6.
#include "common.h"
#include "kernels.h"
#include "lds_limit.h"
#include "row_list_dev.h"

namespace asx {
namespace {

typedef double a32_f64x4_t __attribute__((ext_vector_type(4)));
constexpr int kRows = 16, kWaves = 4, kThreads = 64 * kWaves, kMaxS = 128;

struct AttnF32Args {
  const float *q, *q_lo, *h_enc;   // row operand of phase 1 as value and remainder (q, or dC for BWD); encoder states
  const int32_t* src_len;
  float* alpha32;                  // forward: written; BWD: read
  float *out, *out_lo;             // [B,T,ldS] row result (alpha, or dscore for BWD) and its remainder, which is zero
  float *ctx, *ctx_lo;             // phase 3: context and remainder, or dQ with ctx_lo = null
  uint8_t* attn_mask;
  int T, S, B, H;
  int64_t ldS;
  int32_t* zero;
  RowList list;
};

// four consecutive elements, of which n >= 1 are inside (VEC: all of them, aligned); the others repeat the last
template <bool VEC> __device__ __forceinline__ f32x4_t ld4(const float* p, int n) {
  if constexpr (VEC) return *reinterpret_cast<const f32x4_t*>(p);
  f32x4_t v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = p[e < n ? e : n - 1];
  return v;
}
template <bool VEC> __device__ __forceinline__ void st4(float* p, const f32x4_t& v, int n) {
  if constexpr (VEC) {
    *reinterpret_cast<f32x4_t*>(p) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) p[e] = v[e];
  }
}

// up to 16 ST source positions; VEC: H % 4 == 0
template <bool BWD, int ST, bool VEC>
__global__ __launch_bounds__(kThreads) void attn_f32_kernel(AttnF32Args p) {
  constexpr int SP = 16 * ST, LD = SP + 4;
  extern __shared__ __align__(16) unsigned char smem[];
  double* part = reinterpret_cast<double*>(smem);                  // [wave][row][LD]
  float* rows = reinterpret_cast<float*>(part + kWaves * kRows * LD);   // [row][LD]: alpha, or dscore
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q4 = lane >> 4, n = lane & 15;
  if constexpr (!BWD) {
    if (p.zero && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *p.zero = 0;
    if (blockIdx.x == (unsigned)p.B) {
      if (blockIdx.y == 0) row_list_block<kThreads>(p.list, reinterpret_cast<int*>(smem));
      return;
    }
  }
  const int b = blockIdx.x, T = p.T, S = p.S, H = p.H;
  const int64_t BH = (int64_t)p.B * H;
  int L = p.src_len[b];
  L = L < 0 ? 0 : (L > S ? S : L);
  const int last = L > 0 ? L - 1 : 0;   // positions past the sentence are read from its last word: their weights are 0
  const float* he = p.h_enc + (int64_t)b * H;
  const int nh = (H + 15) >> 4;
  for (int t0 = blockIdx.y * kRows; t0 < T; t0 += gridDim.y * kRows) {
    // ---- phase 1
    a32_f64x4_t acc[ST];
#pragma unroll
    for (int j = 0; j < ST; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[j][r] = 0.0;
    {
      const int t = t0 + n;
      const int64_t off = (int64_t)(t < T ? t : T - 1) * BH + (int64_t)b * H;
      const float *qh = p.q + off, *ql = p.q_lo + off, *hr[ST];
#pragma unroll
      for (int j = 0; j < ST; ++j) {
        const int s = 16 * j + n;
        hr[j] = he + (s < L ? s : last) * BH;
      }
      f32x4_t fq, fl, fh[ST];
      auto load = [&](int i) {
        const int k = i * 16 + 4 * q4, kk = k < H ? k : 0;
        fq = ld4<VEC>(qh + kk, H - kk);
        fl = ld4<VEC>(ql + kk, H - kk);
#pragma unroll
        for (int j = 0; j < ST; ++j) fh[j] = ld4<VEC>(hr[j] + kk, H - kk);
      };
      if (wave < nh) load(wave);
      for (int i = wave; i < nh; i += kWaves) {
        const int left = H - (i * 16 + 4 * q4);   // past the end: both operands cleared (0 * inf)
        double a[4];
        f32x4_t h[ST];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = (VEC ? 0 : e) < left ? (double)fq[e] + (double)fl[e] : 0.0;
#pragma unroll
        for (int j = 0; j < ST; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) h[j][e] = (VEC ? 0 : e) < left ? fh[j][e] : 0.f;
        load(i + kWaves < nh ? i + kWaves : i);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < ST; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], (double)h[j][e], acc[j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < ST; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[(wave * kRows + 4 * r + q4) * LD + 16 * j + n] = acc[j][r];
    __syncthreads();
    // ---- phase 2: rows wave, wave + 4, ...; lane: positions lane and lane + 64
    constexpr int NS = SP > 64 ? 2 : 1;
    for (int r = wave; r < kRows; r += kWaves) {
      const int t = t0 + r;
      if (t >= T) {
        for (int s = lane; s < SP; s += 64) rows[r * LD + s] = 0.f;
        continue;
      }
      const int64_t row = (int64_t)b * T + t;
      float x[NS], v[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int s = lane + 64 * u;
        double d = 0.0;
        if (s < SP)
#pragma unroll
          for (int w = 0; w < kWaves; ++w) d += part[(w * kRows + r) * LD + s];
        x[u] = (float)d;
      }
      if constexpr (!BWD) {
        float m = -INFINITY, sum = 0.f;
#pragma unroll
        for (int u = 0; u < NS; ++u)
          if (lane + 64 * u < L) m = fmaxf(m, x[u]);
        m = wave_max(m);
#pragma unroll
        for (int u = 0; u < NS; ++u) {
          v[u] = lane + 64 * u < L ? expf(x[u] - m) : 0.f;
          sum += v[u];
        }
        sum = wave_sum(sum);
        const float inv = L > 0 ? 1.f / sum : 0.f;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
          v[u] = lane + 64 * u < L ? v[u] * inv : 0.f;   // masked positions: exactly 0
          if (lane + 64 * u < S) p.alpha32[row * S + lane + 64 * u] = v[u];
        }
        if (p.attn_mask && t == 0)
          for (int s = lane; s < S; s += 64) p.attn_mask[(int64_t)b * S + s] = s < L ? 1 : 0;
      } else {
        float a[NS], dot = 0.f;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
          const int s = lane + 64 * u;
          a[u] = s < L ? p.alpha32[row * S + s] : 0.f;
          dot += s < L ? a[u] * x[u] : 0.f;
        }
        dot = wave_sum(dot);
#pragma unroll
        for (int u = 0; u < NS; ++u) v[u] = lane + 64 * u < L ? a[u] * (x[u] - dot) : 0.f;
      }
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int s = lane + 64 * u;
        if (s < SP) rows[r * LD + s] = v[u];
        if (s < p.ldS) {
          p.out[row * p.ldS + s] = v[u];
          p.out_lo[row * p.ldS + s] = 0.f;
        }
      }
    }
    __syncthreads();
    // ---- phase 3: tile c of a wave's four holds columns 4 n + c of its 64
    const int nk = (L + 15) >> 4;
    for (int c0 = wave * 64; c0 < H; c0 += kWaves * 64) {
      const int col = c0 + 4 * n, cc = col < H ? col : 0;
      a32_f64x4_t o[4];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[c][r] = 0.0;
      f32x4_t h[4];
      auto load = [&](int k) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int s = k * 16 + 4 * q4 + e;
          h[e] = ld4<VEC>(he + (s < L ? s : last) * BH + cc, H - cc);
        }
      };
      if (nk > 0) load(0);
      for (int k = 0; k < nk; ++k) {
        const f32x4_t a = *reinterpret_cast<const f32x4_t*>(rows + n * LD + k * 16 + 4 * q4);
        f32x4_t g[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < 4; ++c) g[e][c] = k * 16 + 4 * q4 + e < L ? h[e][c] : 0.f;   // (its weight is 0, the word may be infinite)
        load(k + 1 < nk ? k + 1 : k);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < 4; ++c) o[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[e], (double)g[e][c], o[c], 0, 0, 0);
      }
      if (col >= H) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int t = t0 + 4 * r + q4;
        if (t >= T) continue;
        f32x4_t v, lo;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          v[c] = (float)o[c][r];
          lo[c] = (float)(o[c][r] - (double)v[c]);
        }
        const int64_t at = (int64_t)t * BH + (int64_t)b * H + col;
        st4<VEC>(p.ctx + at, v, H - col);
        if (p.ctx_lo) st4<VEC>(p.ctx_lo + at, lo, H - col);
      }
    }
    __syncthreads();   // the next rows overwrite the weights
  }
}

template <bool BWD, int ST> hipError_t launch_shape(const AttnF32Args& p, hipStream_t st) {
  constexpr int SP = 16 * ST, smem = kRows * (SP + 4) * (kWaves * 8 + 4);
  static_assert(smem >= kRowListSmem, "the row list's share");
  const bool vec = p.H % 4 == 0;
  auto k = vec ? attn_f32_kernel<BWD, ST, true> : attn_f32_kernel<BWD, ST, false>;
  static LdsLimit limits[2];
  LdsLimit& limit = limits[vec];
  const hipError_t e = limit.raise(reinterpret_cast<const void*>(k), smem);
  if (e != hipSuccess) return e;
  const int ny = (p.T + kRows - 1) / kRows;
  const dim3 grid(p.B + (!BWD && p.list.targets ? 1 : 0), ny < 65535 ? ny : 65535);   // (more steps: a block takes several)
  hipLaunchKernelGGL(k, grid, dim3(kThreads), smem, st, p);
  return hipGetLastError();
}
template <bool BWD> hipError_t launch_any(const AttnF32Args& p, hipStream_t st) {
  if (!attn_f32_fused_supported(p.S, p.H) || p.B < 1 || p.T < 1 || p.ldS < p.S || p.ldS > kMaxS) return hipErrorInvalidValue;
  if (p.S <= 16) return launch_shape<BWD, 1>(p, st);
  if (p.S <= 32) return launch_shape<BWD, 2>(p, st);
  if (p.S <= 64) return launch_shape<BWD, 4>(p, st);
  return launch_shape<BWD, 8>(p, st);
}
}  // namespace

// More than 64 source positions: a wave's eight tiles a step and each row's sweeps over the columns are one chain per workgroup, longer
// than three launches where there is more than one sweep (256 columns) and few workgroups.  A training step, us, separate / fused, 16
// steps of S 128: H 256, 1 sentence 119.6 / 112.2, 32 156.9 / 151.9; H 320, 1 131.5 / 133.7, 16 148.3 / 155.4; 512, 16 193.1 / 197.6; 1024, 4
// 274.0 / 295.4; 2048, 4 549.9 / 603.8.  With 64 and more workgroups it would win there too (43 sentences x 48 steps, H 512 of 72
// positions 446 / 416), but a sentence's attention must not depend on how many share its batch.  S 64: H 2048, 1 524.0 / 496.3, 16
// 806.7 / 778.5, 4096, 4 1075.6 / 1024.9.
bool attn_f32_fused_supported(int S, int H) { return S >= 1 && (S <= 64 || (S <= kMaxS && H <= 256)); }

hipError_t launch_attn_f32_fwd(const float* q, const float* q_lo, const float* h_enc, const int32_t* src_len, int B, int T, int S,
                               int H, float* alpha32, float* alphaE, float* alphaE_lo, int64_t ldS, float* ctx, float* ctx_lo,
                               uint8_t* attn_mask, const RowList& list, int32_t* zero, hipStream_t st) {
  AttnF32Args p{};
  p.q = q; p.q_lo = q_lo; p.h_enc = h_enc; p.src_len = src_len;
  p.alpha32 = alpha32; p.out = alphaE; p.out_lo = alphaE_lo;
  p.ctx = ctx; p.ctx_lo = ctx_lo; p.attn_mask = attn_mask;
  p.T = T; p.S = S; p.B = B; p.H = H; p.ldS = ldS;
  p.zero = zero; p.list = list;
  return launch_any<false>(p, st);
}
hipError_t launch_attn_f32_bwd(const float* dC, const float* dC_lo, const float* h_enc, const int32_t* src_len, int B, int T, int S,
                               int H, const float* alpha32, float* dscore, float* dscore_lo, int64_t ldS, float* dQ, hipStream_t st) {
  AttnF32Args p{};
  p.q = dC; p.q_lo = dC_lo; p.h_enc = h_enc; p.src_len = src_len;
  p.alpha32 = const_cast<float*>(alpha32); p.out = dscore; p.out_lo = dscore_lo;
  p.ctx = dQ;
  p.T = T; p.S = S; p.B = B; p.H = H; p.ldS = ldS;
  return launch_any<true>(p, st);
}

}  // namespace asx
