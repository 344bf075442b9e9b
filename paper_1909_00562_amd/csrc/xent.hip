// Vocabulary softmax cross-entropy (Eq. 5-6 of section 3.2) without ever
// forming the probability matrix: a streaming statistics pass (online max /
// sum-exp, target logit, argmax) and an in-place pass that turns the stored
// logits into dlogits = g*(p - onehot) while summing the columns for db_out.
// Both passes are pure HBM streams: 16-byte loads/stores, fp32 arithmetic.
#include <type_traits>

#include "common.h"
#include "db_reduce_dev.h"
#include "gemm.h"
#include "kernels.h"

namespace asx {

// 16-byte load of data that is read once (streamed past the caches)
typedef uint32_t xe_u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16_stream(const void* p) {
  const xe_u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const xe_u32x4_t*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void st16_stream(void* p, const uint4& q) {
  const xe_u32x4_t v = {q.x, q.y, q.z, q.w};
  __builtin_nontemporal_store(v, reinterpret_cast<xe_u32x4_t*>(p));
}

template <typename TE> struct Vec;
template <> struct Vec<uint16_t> { static constexpr int N = 8; };
template <> struct Vec<float> { static constexpr int N = 4; };

template <typename TE>
__device__ __forceinline__ void unpack(const uint4& q, float (&f)[Vec<TE>::N]) {
  if constexpr (sizeof(TE) == 2) {
    f[0] = lo_bf16(q.x); f[1] = hi_bf16(q.x); f[2] = lo_bf16(q.y); f[3] = hi_bf16(q.y);
    f[4] = lo_bf16(q.z); f[5] = hi_bf16(q.z); f[6] = lo_bf16(q.w); f[7] = hi_bf16(q.w);
  } else {
    f[0] = __builtin_bit_cast(float, q.x); f[1] = __builtin_bit_cast(float, q.y);
    f[2] = __builtin_bit_cast(float, q.z); f[3] = __builtin_bit_cast(float, q.w);
  }
}
template <typename TE>
__device__ __forceinline__ uint4 pack(const float (&f)[Vec<TE>::N]) {
  uint4 q;
  if constexpr (sizeof(TE) == 2) {
    q.x = pack_bf16(f[0], f[1]); q.y = pack_bf16(f[2], f[3]);
    q.z = pack_bf16(f[4], f[5]); q.w = pack_bf16(f[6], f[7]);
  } else {
    q.x = __builtin_bit_cast(uint32_t, f[0]); q.y = __builtin_bit_cast(uint32_t, f[1]);
    q.z = __builtin_bit_cast(uint32_t, f[2]); q.w = __builtin_bit_cast(uint32_t, f[3]);
  }
  return q;
}

// running (max, sum of exp relative to max, lowest index of the max)
struct RowStat {
  float m, s;
  int idx;
};
__device__ __forceinline__ RowStat combine(const RowStat& a, const RowStat& b) {
  RowStat r;
  r.m = fmaxf(a.m, b.m);
  const float sa = a.m == r.m ? 1.f : __expf(a.m - r.m);
  const float sb = b.m == r.m ? 1.f : __expf(b.m - r.m);
  r.s = a.s * sa + b.s * sb;
  r.idx = a.m > b.m ? a.idx : (b.m > a.m ? b.idx : (a.idx < b.idx ? a.idx : b.idx));
  return r;
}

// UNR loads in flight per thread, all streaming (4 to 8 in flight measure the same).  A plain read stream with the
// same grid and loads moves 6.8 TB/s on this part when it runs alone; the first form of this kernel, which updated
// the running maximum and its index per element, reached 5.4 inside the step, this one 5.7: a wave's
// vector instruction occupies its 16-lane SIMD for four cycles, so every operation per element counts.  Per
// element this form spends: one shift / mask to widen bf16, half a v_max3, one fused multiply-add into the base-2
// exponent, one v_exp_f32, one add.  The running maximum is updated once per group of UNR vectors instead of per
// vector, and the arg max is tracked at vector granularity (column of the first vector of the thread that attains
// the maximum); the element inside that vector is found once per row by re-reading 16 bytes.
template <typename TE, int UNR = 8>
__global__ __launch_bounds__(256) void xent_stats_kernel(const TE* __restrict__ logits, int64_t ldV, int V,
                                                        const int32_t* __restrict__ targets, int pad_id,
                                                        float* __restrict__ lse, float* __restrict__ tok_loss_ws,
                                                        float* __restrict__ tok_loss, int32_t* __restrict__ argmax,
                                                        uint8_t* __restrict__ tgt_mask,
                                                        const int32_t* __restrict__ rows,
                                                        const int32_t* __restrict__ n_act) {
  constexpr int VEC = Vec<TE>::N;
  constexpr float L2E = 1.4426950408889634f;
  constexpr uint32_t NEG_INF_WORD = sizeof(TE) == 2 ? 0xff80ff80u : 0xff800000u;   // -inf in every element
  // compacted rows (rows != null): logits row r belongs to position rows[r]; lse and the workspace loss are
  // indexed by r, the caller's per-position outputs by the position
  const int n = blockIdx.x, tid = threadIdx.x;
  if (rows && n >= *n_act) return;
  const int pos = rows ? rows[n] : n;
  const TE* x = logits + (int64_t)n * ldV;
  RowStat st{-INFINITY, 0.f, 0x7fffffff};   // idx: column of the first element of the vector holding the first maximum
  // one group = UNR vectors of this thread, 256 * VEC columns apart; GUARD: the group may reach past the row
  auto group = [&](int v0, auto guard) {
    constexpr bool GUARD = decltype(guard)::value;
    // UNR independent 16-byte loads per thread are issued before any of them is used: a row is read once, so
    // the only way to cover the memory latency is to have enough bytes in flight per compute unit
    uint4 q[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int v = v0 + u * 256 * VEC;
      if constexpr (GUARD) {
        q[u] = make_uint4(NEG_INF_WORD, NEG_INF_WORD, NEG_INF_WORD, NEG_INF_WORD);   // a vector past the row: all -inf
        if (v < V) q[u] = ld16_stream(x + v);
      } else {
        q[u] = ld16_stream(x + v);
      }
    }
    float f[UNR][VEC], vm[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int v = v0 + u * 256 * VEC;
      unpack<TE>(q[u], f[u]);
      if constexpr (GUARD) {
        if (v < V && v + VEC > V) {           // the one ragged vector of a row whose length is not a multiple of VEC
#pragma unroll
          for (int i = 0; i < VEC; ++i)
            if (v + i >= V) f[u][i] = -INFINITY;
        }
      }
      float a = f[u][0];
#pragma unroll
      for (int i = 1; i + 1 < VEC; i += 2) a = fmaxf(fmaxf(a, f[u][i]), f[u][i + 1]);   // v_max3_f32
      if constexpr (VEC % 2 == 0) a = fmaxf(a, f[u][VEC - 1]);
      vm[u] = a;
    }
    float gm = fmaxf(fmaxf(vm[0], vm[1]), vm[2]);
#pragma unroll
    for (int u = 3; u + 1 < UNR; u += 2) gm = fmaxf(fmaxf(gm, vm[u]), vm[u + 1]);
    if constexpr (UNR % 2 == 0) gm = fmaxf(gm, vm[UNR - 1]);
    if (gm > st.m) {                          // strict: an equal maximum further right does not move the arg max
      st.s *= __builtin_amdgcn_exp2f((st.m - gm) * L2E);   // exp2(-inf) = 0 the first time
      st.m = gm;
      int first = 0;
#pragma unroll
      for (int u = UNR - 1; u >= 0; --u)      // lowest u (= lowest column of this thread) attaining gm
        if (vm[u] == gm) first = u;
      st.idx = v0 + first * 256 * VEC;
    }
    const float mb = -st.m * L2E;
    float e0 = 0.f, e1 = 0.f;                 // two chains: the adds do not wait on each other
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int i = 0; i < VEC; i += 2) {
        e0 += __builtin_amdgcn_exp2f(__builtin_fmaf(f[u][i], L2E, mb));
        e1 += __builtin_amdgcn_exp2f(__builtin_fmaf(f[u][i + 1], L2E, mb));
      }
    st.s += e0 + e1;
  };
  static_assert(UNR >= 3, "group maximum is taken with v_max3");
  constexpr int STEP = 256 * VEC * UNR;
  int v0 = tid * VEC;
  for (; v0 + (UNR - 1) * 256 * VEC + VEC <= V; v0 += STEP) group(v0, std::false_type{});
  if (v0 < V) group(v0, std::true_type{});
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    RowStat other;
    other.m = __shfl_xor(st.m, o, 64);
    other.s = __shfl_xor(st.s, o, 64);
    other.idx = __shfl_xor(st.idx, o, 64);
    st = combine(st, other);
  }
  __shared__ RowStat ws[4];
  if ((tid & 63) == 0) ws[tid >> 6] = st;
  __syncthreads();
  if (tid == 0) {
    RowStat r = combine(combine(ws[0], ws[1]), combine(ws[2], ws[3]));
    // the vectors of a row are disjoint column ranges, so the lowest vector column among equal maxima holds the
    // lowest arg max; find the element inside it
    int amax = 0;
    if (r.idx < V) {
      float f[VEC];
      unpack<TE>(*reinterpret_cast<const uint4*>(x + r.idx), f);
      int k = VEC - 1;
#pragma unroll
      for (int i = VEC - 1; i >= 0; --i)
        if (r.idx + i < V && f[i] == r.m) k = i;
      amax = r.idx + k;
    }
    const float l = r.m + logf(r.s);
    const int y = targets[pos];
    const bool nonpad = (y != pad_id) && (y >= 0) && (y < V);
    const float loss = nonpad ? l - ld_elem<TE>(x, y) : 0.f;
    lse[n] = l;
    tok_loss_ws[n] = loss;
    if (tok_loss) tok_loss[pos] = loss;
    if (argmax) argmax[pos] = amax;
    if (tgt_mask) tgt_mask[pos] = nonpad ? 1 : 0;
  }
}

// loss_sum and n_tok by one block of 1024 threads; order fixed
template <typename Load>
__device__ __forceinline__ void loss_reduce_block(Load loss, const int32_t* targets, int N, int V, int pad_id, float* loss_sum,
                                                  int32_t* n_tok, const int32_t* n_act, double* sd, int* sc) {
  const int tid = threadIdx.x;
  double acc = 0.0;
  int cnt = 0;
  if (n_act) {   // compacted rows: the first *n_act entries are the non-pad positions
    const int na = *n_act;
    for (int i = tid; i < na; i += 1024) acc += (double)loss(i);
    cnt = tid == 0 ? na : 0;
  } else {
    for (int i = tid; i < N; i += 1024) {
      acc += (double)loss(i);
      const int y = targets[i];
      cnt += ((y != pad_id) && (y >= 0) && (y < V)) ? 1 : 0;
    }
  }
  sd[tid] = acc;
  sc[tid] = cnt;
  __syncthreads();
  for (int o = 512; o >= 64; o >>= 1) {
    if (tid < o) { sd[tid] += sd[tid + o]; sc[tid] += sc[tid + o]; }
    __syncthreads();
  }
  if (tid >= 64) return;
  acc = sd[tid];
  cnt = sc[tid];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {   // the same tree inside one wave
    acc += __shfl_down(acc, o, 64);
    cnt += __shfl_down(cnt, o, 64);
  }
  if (tid == 0) { *loss_sum = (float)acc; *n_tok = cnt; }
}
__global__ __launch_bounds__(1024) void loss_reduce_kernel(const float* __restrict__ tok_loss_ws,
                                                          const int32_t* __restrict__ targets, int N, int V,
                                                          int pad_id, float* loss_sum, int32_t* n_tok,
                                                          const int32_t* __restrict__ n_act) {
  __shared__ double sd[1024];
  __shared__ int sc[1024];
  loss_reduce_block([&](int i) { return tok_loss_ws[i]; }, targets, N, V, pad_id, loss_sum, n_tok, n_act, sd, sc);
}

// Few rows: the statistics of the projection's tiles instead of the logits themselves, a wavefront per row, and the loss by the
// block that is through last.
constexpr int kFinishRows = 16;
__global__ __launch_bounds__(1024) void xent_finish_kernel(XentFinish p) {
  __shared__ double sd[1024];
  __shared__ int sc[1024];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, n = blockIdx.x * kFinishRows + (tid >> 6);
  const int rows = p.rows ? (*p.n_act < p.N ? *p.n_act : p.N) : p.N;
  if (n < rows) {
    const int pos = p.rows ? p.rows[n] : n;
    const int y = p.targets[pos];
    const bool nonpad = (y != p.pad_id) && (y >= 0) && (y < p.V);
    const float at = nonpad ? ld_elem<uint16_t>(reinterpret_cast<const uint16_t*>(p.logits) + (int64_t)n * p.ldV, y) : 0.f;
    RowStat st{-INFINITY, 0.f, 0x7fffffff};
    const TileStat* t = p.stats + (int64_t)n * p.parts;
    for (int i = lane; i < p.parts; i += 256) {
      TileStat q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = t[i + 64 * u < p.parts ? i + 64 * u : i];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + 64 * u < p.parts) st = combine(st, RowStat{q[u].m, q[u].s, q[u].idx});
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      RowStat other;
      other.m = __shfl_xor(st.m, o, 64);
      other.s = __shfl_xor(st.s, o, 64);
      other.idx = __shfl_xor(st.idx, o, 64);
      st = combine(st, other);
    }
    if (lane == 0) {
      const float l = st.m + logf(st.s), loss = nonpad ? l - at : 0.f;
      p.lse[n] = l;
      __hip_atomic_store(p.tok_loss_ws + n, loss, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (p.tok_loss) p.tok_loss[pos] = loss;
      if (p.argmax) p.argmax[pos] = st.idx < p.V ? st.idx : 0;
      if (p.tgt_mask) p.tgt_mask[pos] = nonpad ? 1 : 0;
    }
  }
  if (gridDim.x > 1) {
    __builtin_amdgcn_s_waitcnt(0);   // the wave's losses are where every XCD sees them (stored past the caches)
    __syncthreads();
    if (tid == 0)
      last = __hip_atomic_fetch_add(p.ticket, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    __syncthreads();
    if (!last) return;
  } else {
    __syncthreads();
  }
  loss_reduce_block([&](int i) { return __hip_atomic_load(p.tok_loss_ws + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                    p.targets, p.N, p.V, p.pad_id, p.loss_sum, p.n_tok, p.n_act, sd, sc);
}

// RU rows in flight per thread; NT: 1 = streaming loads, 2 = streaming stores, 3 = both.  Measured on
// 12288 x 128000 bf16: (4, 0) 4.93 TB/s, (4, 3) 5.02, (8, 3) 5.09; a plain device copy moves 4.7-5.3.
template <typename TE, int RU = 8, int NT = 3>
__global__ __launch_bounds__(256) void xent_dlogits_kernel(TE* __restrict__ logits, int64_t ldV, int N, int V,
                                                          const int32_t* __restrict__ targets, int pad_id,
                                                          const float* __restrict__ lse, float g, int RB,
                                                          float* __restrict__ db_partial,
                                                          const int32_t* __restrict__ rows,
                                                          const int32_t* __restrict__ n_act) {
  constexpr int VEC = Vec<TE>::N;
  const int c0 = (blockIdx.x * 256 + threadIdx.x) * VEC;
  if (c0 >= ldV) return;
  if (rows) N = *n_act;                 // compacted rows: row r belongs to position rows[r]
  const int r0 = blockIdx.y * RB;
  if (rows && r0 >= N) return;          // past the last row: db_reduce does not read these column sums
  const int r1 = r0 + RB < N ? r0 + RB : N;
  float cs[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) cs[i] = 0.f;
  for (int r = r0; r < r1; r += RU) {   // RU rows of loads in flight per thread
    uint4 q[RU];
    bool live[RU];
    int y[RU];
    float l[RU];
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int rr = r + u;
      live[u] = false;
      y[u] = -1;
      l[u] = 0.f;
      q[u] = make_uint4(0, 0, 0, 0);
      if (rr < r1) {
        y[u] = targets[rows ? rows[rr] : rr];
        live[u] = (y[u] != pad_id) && (y[u] >= 0) && (y[u] < V);
        if (live[u]) {                      // pad rows are not read, only zeroed
          l[u] = lse[rr];
          q[u] = (NT & 1) ? ld16_stream(logits + (int64_t)rr * ldV + c0)
                          : *reinterpret_cast<const uint4*>(logits + (int64_t)rr * ldV + c0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int rr = r + u;
      if (rr >= r1) break;
      float f[VEC], d[VEC];
      unpack<TE>(q[u], f);
#pragma unroll
      for (int i = 0; i < VEC; ++i) {
        float v = 0.f;
        if (live[u] && c0 + i < V) v = g * (__expf(f[i] - l[u]) - (c0 + i == y[u] ? 1.f : 0.f));
        d[i] = v;
        cs[i] += v;
      }
      if (NT & 2) st16_stream(logits + (int64_t)rr * ldV + c0, pack<TE>(d));
      else *reinterpret_cast<uint4*>(logits + (int64_t)rr * ldV + c0) = pack<TE>(d);
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i)
    if (c0 + i < V) db_partial[(int64_t)blockIdx.y * V + c0 + i] = cs[i];
}

__global__ __launch_bounds__(1024) void db_reduce_kernel(DbReduce p) {
  __shared__ float red[kDbSmem / sizeof(float)];
  db_reduce_block<1024>(p, blockIdx.x, red);
}

// ---- launchers ----------------------------------------------------------------
hipError_t launch_xent_stats(const void* logits, int64_t ldV, bool e_bf16, int N, int V,
                             const int32_t* targets, int pad_id, float* lse, float* tok_loss_ws,
                             float* tok_loss, int32_t* argmax, uint8_t* tgt_mask, const int32_t* rows,
                             const int32_t* n_act, hipStream_t st) {
  if (e_bf16)
    hipLaunchKernelGGL(xent_stats_kernel<uint16_t>, dim3(N), dim3(256), 0, st,
                       reinterpret_cast<const uint16_t*>(logits), ldV, V, targets, pad_id, lse, tok_loss_ws,
                       tok_loss, argmax, tgt_mask, rows, n_act);
  else
    hipLaunchKernelGGL(xent_stats_kernel<float>, dim3(N), dim3(256), 0, st,
                       reinterpret_cast<const float*>(logits), ldV, V, targets, pad_id, lse, tok_loss_ws, tok_loss,
                       argmax, tgt_mask, rows, n_act);
  return hipGetLastError();
}

hipError_t launch_xent_finish(const XentFinish& p, hipStream_t st) {
  hipLaunchKernelGGL(xent_finish_kernel, dim3((p.N + kFinishRows - 1) / kFinishRows), dim3(1024), 0, st, p);
  return hipGetLastError();
}

hipError_t launch_loss_reduce(const float* tok_loss_ws, const int32_t* targets, int N, int V, int pad_id,
                              float* loss_sum, int32_t* n_tok, const int32_t* n_act, hipStream_t st) {
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(1024), 0, st, tok_loss_ws, targets, N, V, pad_id, loss_sum,
                     n_tok, n_act);
  return hipGetLastError();
}

int xent_rows_per_block(int N, int V, bool e_bf16) {
  const int vec = e_bf16 ? 8 : 4;
  const int64_t ldV = ((int64_t)V + 7) / 8 * 8;
  const int64_t strips = (ldV + 256 * vec - 1) / (256 * vec);
  // About 32768 blocks, of 16 rows and more: short-lived blocks keep to one neighbourhood of rows, long ones drift apart
  // (16384 x 128000, three quarters words, with the column sums' reduction: 252 rows 1285 us, 128 1243, 64 1227, 32
  // 1206; 6400 x 32000: 28 rows 119 us, 16 118.5, 8 140).  Eight rows where 16 would leave fewer than 2048 blocks.  The
  // blocks' column sums take V floats each (16384 x 128000: 262 MB at 32 rows, 33 at 252), where the partial sums of the
  // products go afterwards.
  int64_t rb = ((int64_t)N * strips + 32767) / 32768;
  const int64_t least = (int64_t)N * strips >= 16 * 2048 ? 16 : 8;
  if (rb < least) rb = least;
  if (rb > 256) rb = 256;
  return (int)((rb + 3) / 4 * 4);
}

hipError_t launch_xent_dlogits(void* logits, int64_t ldV, bool e_bf16, int N, int V, const int32_t* targets,
                               int pad_id, const float* lse, float g, float* db_partial, const int32_t* rows,
                               const int32_t* n_act, hipStream_t st) {
  const int vec = e_bf16 ? 8 : 4;
  const int RB = xent_rows_per_block(N, V, e_bf16);
  dim3 grid((unsigned)((ldV + 256 * vec - 1) / (256 * vec)), (N + RB - 1) / RB);
  if (e_bf16)
    hipLaunchKernelGGL(xent_dlogits_kernel<uint16_t>, grid, dim3(256), 0, st, reinterpret_cast<uint16_t*>(logits),
                       ldV, N, V, targets, pad_id, lse, g, RB, db_partial, rows, n_act);
  else
    hipLaunchKernelGGL(xent_dlogits_kernel<float>, grid, dim3(256), 0, st, reinterpret_cast<float*>(logits), ldV, N,
                       V, targets, pad_id, lse, g, RB, db_partial, rows, n_act);
  return hipGetLastError();
}

hipError_t launch_db_reduce(const DbReduce& d, hipStream_t st) {
  hipLaunchKernelGGL(db_reduce_kernel, dim3((d.V + kDbColumns - 1) / kDbColumns), dim3(1024), 0, st, d);
  return hipGetLastError();
}

}  // namespace asx
