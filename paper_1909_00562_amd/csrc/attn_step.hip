// Attention for ONE decoder step (T = 1), fused: scores (Eq. 2), masked softmax (Eq. 1) and context vector (Eq. 3) of
// section 3.2 in one kernel, one workgroup per sentence, and the backward pass of the same.
//   score[s] = query[b] . key[s,b]      alpha = softmax_{s < src_len[b]}      ctx = sum_s alpha[s] h_enc[s,b]
// Per-step mode (decoding, scoring, the input-feeding variant of the paper's section 4, where step t+1 needs the
// attentional state of step t): query h_t, key K'[s,b,:] = W_a h_enc[s,b,:] (float), computed once per batch of
// sentences.  Backward of a training step with T = 1: with query dC and key h_enc the scores are dalpha;
//   dscore = alpha (dalpha - alpha . dalpha)    dQ = sum_s dscore[s] h_enc[s,b]
//   d_h_enc[s,b] = alpha[s] dC[b] + dscore[s] Q[b]
// One row per sentence leaves nothing for matrix instructions; what counts is that the sentence's S x H block is
// requested at once: 16 waves, four source positions per wave in flight.  128 x 50 x 1024, bf16: per-step mode 11 us (19 with
// eight waves and two positions); backward 14 us, where d_h_enc alone as a batched product of rank one takes 25.
#include "common.h"
#include "kernels.h"
#include "lds_limit.h"

namespace asx {

typedef uint32_t st_u32x4_t __attribute__((ext_vector_type(4)));
constexpr int kStepThreads = 1024, kStepWaves = kStepThreads / 64;
constexpr size_t kStepSmem = 150 * 1024;

template <typename T> __device__ __forceinline__ void st_unpack(const st_u32x4_t& q, float (&f)[16 / sizeof(T)]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const uint32_t w = q[v];
    if constexpr (sizeof(T) == 2) {
      f[2 * v] = lo_bf16(w);
      f[2 * v + 1] = hi_bf16(w);
    } else {
      f[v] = __builtin_bit_cast(float, w);
    }
  }
}

struct AttnStep {
  const void *query, *query_lo;   // [B,H] storage type: value, optional remainder
  const void* key;                // [S,B,H] TK
  const void* h_enc;              // [S,B,H] storage type
  const int32_t* src_len;
  int B, S, H;
  int G;                          // groups of the context sum (0: element-wise form)
  float* alpha;                   // [B,S]: written; BWD: read
  void *ctx, *ctx_lo;             // [B,H] storage type: ctx and optional remainder; BWD: dQ
  uint8_t* attn_mask;             // optional
  int32_t* zero;                  // cleared, if not null
  const void *q, *q_lo;           // BWD: Q [B,H] as value and remainder
  float* d_h_enc;                 // BWD: [S,B,H]
};

template <typename TK, typename TE, bool BWD>
__global__ __launch_bounds__(kStepThreads) void attn_step_kernel(AttnStep p) {
  extern __shared__ __align__(16) float sm[];   // query [H], row results [S], BWD: alpha [S], partial sums [G][H]
  const int B = p.B, S = p.S, H = p.H;
  float* hs = sm;
  float* sc = sm + H;
  float* al = sc + S;             // BWD only
  float* part = BWD ? al + S : al;
  __shared__ float red[2 * kStepWaves];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!BWD && p.zero && b == 0 && tid == 0) *p.zero = 0;
  int L = p.src_len[b];
  L = L < 0 ? 0 : (L > S ? S : L);
  const TE* query = reinterpret_cast<const TE*>(p.query) + (int64_t)b * H;
  const TE* query_lo = reinterpret_cast<const TE*>(p.query_lo) + (int64_t)b * H;
  for (int c = tid; c < H; c += kStepThreads)
    hs[c] = ld_elem<TE>(query, c) + (p.query_lo ? ld_elem<TE>(query_lo, c) : 0.f);
  if constexpr (BWD)
    for (int s = tid; s < S; s += kStepThreads) al[s] = p.alpha[(int64_t)b * S + s];
  __syncthreads();

  // scores: one wavefront per source position, four positions at a time, lanes across H
  constexpr int VK = 16 / (int)sizeof(TK), NU = 4;
  const TK* key = reinterpret_cast<const TK*>(p.key) + (int64_t)b * H;
  const int64_t BH = (int64_t)B * H;
  for (int s0 = wave; s0 < L; s0 += NU * kStepWaves) {
    float acc[NU];
    const TK* row[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int s = s0 + u * kStepWaves;
      acc[u] = 0.f;
      row[u] = key + (s < L ? s : s0) * BH;   // past the end: the first position again, not stored
    }
    if (H % VK == 0) {
#pragma unroll 2
      for (int c = lane * VK; c < H; c += 64 * VK) {
        st_u32x4_t k[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) k[u] = *reinterpret_cast<const st_u32x4_t*>(row[u] + c);
        float h[VK];
#pragma unroll
        for (int v = 0; v < VK; v += 4) {
          const f32x4_t h4 = *reinterpret_cast<const f32x4_t*>(hs + c + v);
          h[v] = h4[0]; h[v + 1] = h4[1]; h[v + 2] = h4[2]; h[v + 3] = h4[3];
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          float f[VK];
          st_unpack<TK>(k[u], f);
#pragma unroll
          for (int v = 0; v < VK; ++v) acc[u] += f[v] * h[v];
        }
      }
    } else {
      for (int c = lane; c < H; c += 64)
#pragma unroll
        for (int u = 0; u < NU; ++u) acc[u] += ld_elem<TK>(row[u], c) * hs[c];
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const float a = wave_sum(acc[u]);
      if (lane == 0 && s0 + u * kStepWaves < L) sc[s0 + u * kStepWaves] = a;
    }
  }
  __syncthreads();

  if constexpr (!BWD) {   // masked softmax over the L valid positions
    float m = -INFINITY;
    for (int s = tid; s < L; s += kStepThreads) m = fmaxf(m, sc[s]);
    m = wave_max(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int i = 1; i < kStepWaves; ++i) m = fmaxf(m, red[i]);
    float sum = 0.f;
    for (int s = tid; s < L; s += kStepThreads) sum += expf(sc[s] - m);
    sum = wave_sum(sum);
    if (lane == 0) red[kStepWaves + wave] = sum;
    __syncthreads();
    sum = 0.f;
#pragma unroll
    for (int i = 0; i < kStepWaves; ++i) sum += red[kStepWaves + i];
    const float inv = L > 0 ? 1.f / sum : 0.f;
    for (int s = tid; s < S; s += kStepThreads) {   // a thread reads and writes its own positions only
      const float a = s < L ? expf(sc[s] - m) * inv : 0.f;   // masked positions: exactly 0
      p.alpha[(int64_t)b * S + s] = a;
      if (p.attn_mask) p.attn_mask[(int64_t)b * S + s] = s < L ? 1 : 0;
      sc[s] = a;
    }
  } else {                // softmax Jacobian
    float dot = 0.f;
    for (int s = tid; s < L; s += kStepThreads) dot += al[s] * sc[s];
    dot = wave_sum(dot);
    if (lane == 0) red[wave] = dot;
    __syncthreads();
    dot = 0.f;
#pragma unroll
    for (int i = 0; i < kStepWaves; ++i) dot += red[i];
    for (int s = tid; s < S; s += kStepThreads) sc[s] = s < L ? al[s] * (sc[s] - dot) : 0.f;
  }
  __syncthreads();

  // context: the threads form G groups; a group covers all of H with 16-byte vectors and takes every G-th
  // source position; the G partial sums are added in a fixed order
  constexpr int VEC = 16 / (int)sizeof(TE);
  const TE* h_enc = reinterpret_cast<const TE*>(p.h_enc) + (int64_t)b * H;
  TE* ctx = reinterpret_cast<TE*>(p.ctx) + (int64_t)b * H;
  TE* ctx_lo = reinterpret_cast<TE*>(p.ctx_lo) + (int64_t)b * H;
  auto put = [&](int c, float v) {
    st_elem<TE>(ctx, c, v);
    if (p.ctx_lo) st_elem<TE>(ctx_lo, c, v - round_elem<TE>(v));
  };
  if (p.G > 0) {
    const int per = H / VEC, G = p.G;     // threads of one group
    const int grp = tid / per, c = (tid - grp * per) * VEC;
    if (grp < G) {
      float acc[VEC];
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
#pragma unroll 8
      for (int s = grp; s < L; s += G) {
        float f[VEC];
        st_unpack<TE>(*reinterpret_cast<const st_u32x4_t*>(h_enc + s * BH + c), f);
        const float a = sc[s];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += a * f[v];
      }
#pragma unroll
      for (int v = 0; v < VEC; ++v) part[grp * H + c + v] = acc[v];
    }
    __syncthreads();
    for (int cc = tid; cc < H; cc += kStepThreads) {
      float acc = 0.f;
      for (int g = 0; g < G; ++g) acc += part[g * H + cc];
      put(cc, acc);
    }
  } else {
    for (int c = tid; c < H; c += kStepThreads) {
      float acc = 0.f;
      for (int s = 0; s < L; ++s) acc += sc[s] * ld_elem<TE>(h_enc, s * BH + c);
      put(c, acc);
    }
  }
  if constexpr (BWD) {   // gradient of the encoder states: the sentence's rows are written by its workgroup alone
    const TE* q = reinterpret_cast<const TE*>(p.q) + (int64_t)b * H;
    const TE* q_lo = reinterpret_cast<const TE*>(p.q_lo) + (int64_t)b * H;
    float* out = p.d_h_enc + (int64_t)b * H;
    const int per = H / 4;   // H % 8 == 0 (bf16 storage)
    const int side = per < kStepThreads ? kStepThreads / per : 1;   // positions side by side
    const int step = per < kStepThreads ? per : kStepThreads;
    const int ss = tid / step;
    for (int c4 = tid - ss * step; c4 < per && ss < side; c4 += step) {
      const int c = c4 * 4;
      const f32x4_t dc = *reinterpret_cast<const f32x4_t*>(hs + c);
      f32x4_t qv;
#pragma unroll
      for (int e = 0; e < 4; ++e) qv[e] = ld_elem<TE>(q, c + e) + ld_elem<TE>(q_lo, c + e);
      for (int s = ss; s < S; s += side) {
        const float a = al[s], d = sc[s];
        f32x4_t o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = a * dc[e] + d * qv[e];
        *reinterpret_cast<f32x4_t*>(out + s * BH + c) = o;
      }
    }
  }
}

// groups of the context sum, by what the threads and the LDS allow
static int step_groups(int S, int H, int vec, bool bwd, size_t& smem) {
  int G = 0;
  if (H % vec == 0 && H / vec <= kStepThreads) {
    G = kStepThreads / (H / vec);
    if (G > 8) G = 8;
  }
  const size_t base = ((size_t)H + (bwd ? 2 : 1) * (size_t)S) * sizeof(float);
  while (G > 0 && base + (size_t)G * H * sizeof(float) > kStepSmem) --G;
  smem = base + (size_t)G * H * sizeof(float);
  return G;
}

template <typename TK, typename TE, bool BWD>
static hipError_t launch_step(AttnStep p, hipStream_t st) {
  size_t smem = 0;
  p.G = step_groups(p.S, p.H, 16 / (int)sizeof(TE), BWD, smem);
  if (smem > kStepSmem) return hipErrorInvalidValue;
  auto k = attn_step_kernel<TK, TE, BWD>;
  if (smem > 48 * 1024) {
    static LdsLimit limit;
    const hipError_t e = limit.raise(reinterpret_cast<const void*>(k), (int)kStepSmem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3(p.B), dim3(kStepThreads), smem, st, p);
  return hipGetLastError();
}

hipError_t launch_attn_step(const void* h_t, const float* kprime, const void* h_enc, const int32_t* src_len, int B,
                            int S, int H, float* alpha, void* ctx, void* ctx_lo, bool e_bf16, uint8_t* attn_mask,
                            int32_t* zero, hipStream_t st) {
  AttnStep p{};
  p.zero = zero;
  p.query = h_t;
  p.key = kprime;
  p.h_enc = h_enc;
  p.src_len = src_len;
  p.B = B; p.S = S; p.H = H;
  p.alpha = alpha; p.ctx = ctx; p.ctx_lo = ctx_lo; p.attn_mask = attn_mask;
  return e_bf16 ? launch_step<float, uint16_t, false>(p, st) : launch_step<float, float, false>(p, st);
}

bool attn_one_step_bwd_supported(int T, int S, int H) {
  size_t smem = 0;
  step_groups(S, H, 8, true, smem);
  return T == 1 && H % 8 == 0 && smem <= kStepSmem;
}
hipError_t launch_attn_one_step_bwd(const void* dC_hi, const void* dC_lo, const void* h_enc, const int32_t* src_len,
                                    int B, int S, int H, const float* alpha, const void* q_hi, const void* q_lo, void* dQ,
                                    float* d_h_enc, hipStream_t st) {
  AttnStep p{};
  p.query = dC_hi; p.query_lo = dC_lo;
  p.key = p.h_enc = h_enc;
  p.src_len = src_len;
  p.B = B; p.S = S; p.H = H;
  p.alpha = const_cast<float*>(alpha);
  p.ctx = dQ;
  p.q = q_hi; p.q_lo = q_lo; p.d_h_enc = d_h_enc;
  return launch_step<uint16_t, uint16_t, true>(p, st);
}

}  // namespace asx
