// Fused Adam update of one parameter tensor (paper section 4.2, "Parameter
// settings"; Kingma and Ba, Algorithm 1).  One streaming pass: per element 16
// bytes read (gradient, both moments, master weight), 12 written back and the
// 2- or 4-byte copy in the storage type of the forward pass; HBM-bound.  Nothing but
// that copy is read again soon: the other streams go past the caches where they would not stay there.
// 33.5M elements, bf16 copy, after other work: 200 us as a grid-stride loop through the caches, 191 with one vector
// per thread, 184 past the caches too (5.5 TB/s); repeated on one tensor 199, 190, 156.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"
#include "kernels.h"

namespace asx {

template <bool NT> __device__ __forceinline__ f32x4_t adam_ld(const float* p, size_t i) {
  const f32x4_t* q = reinterpret_cast<const f32x4_t*>(p) + i;
  return NT ? __builtin_nontemporal_load(q) : *q;
}
template <bool NT> __device__ __forceinline__ void adam_st(float* p, size_t i, const f32x4_t& v) {
  f32x4_t* q = reinterpret_cast<f32x4_t*>(p) + i;
  if constexpr (NT) __builtin_nontemporal_store(v, q);
  else *q = v;
}

template <bool OUT_BF16, bool HAS_OUT, bool NT>
__global__ __launch_bounds__(256) void adam_step_kernel(size_t n4, size_t n, const float* __restrict__ grad,
                                                        float* __restrict__ master, float* __restrict__ m,
                                                        float* __restrict__ v, void* __restrict__ wout, float lr,
                                                        float beta1, float beta2, float eps, float inv_bc1,
                                                        float inv_bc2) {
  const float omb1 = 1.f - beta1, omb2 = 1.f - beta2;
  auto upd = [&](float g, float& mm, float& vv, float& w) {
    mm = beta1 * mm + omb1 * g;
    vv = beta2 * vv + omb2 * g * g;
    w -= lr * (mm * inv_bc1) / (sqrtf(vv * inv_bc2) + eps);
  };
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    const f32x4_t g4 = adam_ld<NT>(grad, i);
    f32x4_t m4 = adam_ld<NT>(m, i);
    f32x4_t v4 = adam_ld<NT>(v, i);
    f32x4_t w4 = adam_ld<NT>(master, i);
    float mm[4] = {m4[0], m4[1], m4[2], m4[3]}, vv[4] = {v4[0], v4[1], v4[2], v4[3]};
    float w[4] = {w4[0], w4[1], w4[2], w4[3]};
#pragma unroll
    for (int c = 0; c < 4; ++c) upd(g4[c], mm[c], vv[c], w[c]);
    adam_st<NT>(m, i, f32x4_t{mm[0], mm[1], mm[2], mm[3]});
    adam_st<NT>(v, i, f32x4_t{vv[0], vv[1], vv[2], vv[3]});
    adam_st<NT>(master, i, f32x4_t{w[0], w[1], w[2], w[3]});
    if constexpr (HAS_OUT) {
      if constexpr (OUT_BF16)
        reinterpret_cast<uint2*>(wout)[i] = make_uint2(pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3]));
      else
        reinterpret_cast<f32x4_t*>(wout)[i] = f32x4_t{w[0], w[1], w[2], w[3]};
    }
  }
  // ragged tail (n % 4 elements), one thread each
  const size_t t = n4 * 4 + (size_t)blockIdx.x * 256 + threadIdx.x;
  if (t < n) {
    float mm = m[t], vv = v[t], w = master[t];
    upd(grad[t], mm, vv, w);
    m[t] = mm;
    v[t] = vv;
    master[t] = w;
    if constexpr (HAS_OUT) {
      if constexpr (OUT_BF16) reinterpret_cast<uint16_t*>(wout)[t] = (uint16_t)f32_to_bf16_bits(w);
      else reinterpret_cast<float*>(wout)[t] = w;
    }
  }
}

hipError_t launch_adam_step(size_t n, const float* grad, float* master, float* m, float* v, void* wout,
                            bool out_bf16, float lr, float beta1, float beta2, float eps, float inv_bc1,
                            float inv_bc2, hipStream_t st) {
  const size_t n4 = n / 4;
  size_t blocks = (n4 + 255) / 256;
  // One vector per thread: blocks that come and go keep the streams in step, a grid-stride loop of resident blocks drifts
  // apart (32.8M elements past the caches: 16 blocks per compute unit 175 us, 64 of them 162, one vector each 157).
  if (blocks > (size_t)1 << 20) blocks = (size_t)1 << 20;
  if (blocks < 1) blocks = 1;
  dim3 grid((unsigned)blocks), blk(256);
  // Past the caches only where a tensor's streams exceed the 256 MB memory-side cache: below, a next update that follows at
  // once finds them there (8.2M elements: 45 us through the caches, 50 past them).  Above, it still finds some (12.6M: 54
  // and 62 us, 18.9M: 88 and 92, 21M: 111 and 101), but after a training step's other work it does not (12.6M: 73 and 62).
  const bool nt = n * 28 > (size_t)256 << 20;
#define ASX_ADAM(BF, HO) \
  if (nt) ASX_ADAM_NT(BF, HO, true); \
  else ASX_ADAM_NT(BF, HO, false)
#define ASX_ADAM_NT(BF, HO, NT) \
  hipLaunchKernelGGL((adam_step_kernel<BF, HO, NT>), grid, blk, 0, st, n4, n, grad, master, m, v, wout, lr, beta1, beta2, \
                     eps, inv_bc1, inv_bc2)
  if (!wout) {
    ASX_ADAM(false, false);
  } else if (out_bf16) {
    ASX_ADAM(true, true);
  } else {
    ASX_ADAM(false, true);
  }
#undef ASX_ADAM_NT
#undef ASX_ADAM
  return hipGetLastError();
}

}  // namespace asx
