// bf16 products with few 128 x 128 output tiles (gfx950): 64 x 64 block tile, NST-stage LDS ring.
//
// A product of a hundred rows and a thousand columns is 8 tiles of 128 x 128; each of these walks the whole reduction
// on one compute unit at that unit's LDS and matrix rate (0.45 us per 64 reduction elements) while the others idle.
// Here there are four times as many blocks with a quarter of the work per reduction tile, and the loads run NST - 1
// tiles ahead, which the shorter tile needs: HBM -> LDS directly in every orientation, one barrier per tile, no branch
// and the same number of loads in flight at every wait (past the last tile they read out of range, i.e. zeros).
//   * reduction-contiguous operand: LDS [64 rows][64 k] as in gemm_bf16.hip;
//   * strided operand: LDS [64 k][64 columns] as in memory, fragments by transposing reads.  A 16-lane group reads four
//     k-rows x 32 bytes; the 32-byte segments of a row are XOR-swizzled with (k >> 1) & 3, so that k-rows two apart
//     (256 bytes, all banks) do not meet.
#include "common.h"
#include "gemm.h"
#include "gemm_dev.h"

#include <type_traits>

namespace asx {

constexpr int GS_TILE = 64 * ROWB;         // bytes of an operand tile
constexpr int GS_STAGE = 2 * GS_TILE;
constexpr int GS_LD = 68;                  // floats per row of the write-out staging

// 64 k-rows x 64 columns of a strided operand: two loads per wave, eight k-rows each
struct StridedLoader64 {
  uint32_t voff[2];
  int k;
  __device__ __forceinline__ void init(int64_t ld, int cols_left, int wave, int lane) {
    k = 8 * wave + (lane >> 3);
    const int pc = lane & 7, seg = (pc >> 1) ^ ((lane >> 4) & 3);
    const int col = (seg * 2 + (pc & 1)) * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j) voff[j] = col < cols_left ? (uint32_t)(((int64_t)(k + 32 * j) * ld + col) * 2) : kOob;
  }
  __device__ __forceinline__ void load(int j, const __amdgpu_buffer_rsrc_t& rs, int k_left, unsigned char* lds_tile,
                                       int wave) const {
    const uint32_t off = k + 32 * j < k_left ? voff[j] : kOob;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(lds_tile + (wave + 4 * j) * 1024), 16, off, 0, 0, 0);
  }
};

// Fragment of the 16x16x32 instruction: 16 rows (columns) from row0 on x 32 reduction elements, step ks of the tile.
template <bool KC> __device__ __forceinline__ uint32_t gs_frag_base(int row0, int lane) {
  if constexpr (KC) {
    const int row = row0 + (lane & 15);
    return (uint32_t)(row * ROWB + (((lane >> 4) ^ (row & 7) ^ ((row >> 3) & 1)) << 4));
  } else {
    const int k = (lane >> 4) * 8 + ((lane & 15) >> 2);   // this lane presents four columns of k-rows k and k + 4
    const int cb = (row0 + (lane & 3) * 4) * 2;
    return (uint32_t)(k * 128 + (((cb >> 5) ^ ((k >> 1) & 3)) << 5) + (cb & 31));
  }
}
template <bool KC> __device__ __forceinline__ bf16x8_t gs_frag(const unsigned char* tile, uint32_t base, int ks) {
  if constexpr (KC) {
    return *reinterpret_cast<const bf16x8_t*>(tile + (base ^ (uint32_t)(ks << 6)));
  } else {
    union { s16x4_t h[2]; bf16x8_t v; } u;
    u.h[0] = lds_read_tr((lds_s16x4_t*)(lds_void_t*)(tile + base + ks * 4096));
    u.h[1] = lds_read_tr((lds_s16x4_t*)(lds_void_t*)(tile + (base ^ 64u) + ks * 4096 + 512));
    return u.v;
  }
}

// Epilogue of four consecutive columns of a row
__device__ __forceinline__ void gs_store4(const GemmDev& p, int out_bf16, int batch, int z, int row, int col,
                                          const f32x4_t& v) {
  const int nc = p.N - col < 4 ? p.N - col : 4;   // columns inside
  const bool vec = p.vec_ok != 0;                 // all four are inside C's rows (or their padding) and aligned
  float x[4] = {v[0], v[1], v[2], v[3]};
  if (p.splits > 1) {
    float* dst = p.partial + ((int64_t)z * p.M + row) * p.N + col;
    if (vec) {
      *reinterpret_cast<f32x4_t*>(dst) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nc) dst[e] = x[e];
    }
    return;
  }
  float dact[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (p.bias && e < nc) x[e] += bf16_bits_to_f32(p.bias[col + e]);
    if (p.act_tanh) x[e] = tanhf(x[e]);
    dact[e] = 1.f - x[e] * x[e];
  }
  if (p.drop_thr) {
    const uint64_t at = (uint64_t)row * p.N + col;
    uint32_t w[4];
    if (vec) dropout_words4(at >> 2, p.drop_seed, w);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float m = vec ? (w[e] >= p.drop_thr ? p.drop_scale : 0.f)
                          : dropout_mult(at + e, p.drop_seed, p.drop_thr, p.drop_scale);
      x[e] *= m;
      dact[e] *= m;
    }
  }
  if (p.gate) {
    const float* gp = p.gate + (int64_t)row * p.ldg + col;
    if (vec) {
      const f32x4_t g4 = *reinterpret_cast<const f32x4_t*>(gp);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] *= g4[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nc) x[e] *= gp[e];
    }
  }
  const int64_t ci = (int64_t)batch * p.sC + (int64_t)row * p.ldc + col;
  if (out_bf16) {
    uint32_t hb[4];
    float lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      hb[e] = f32_to_bf16_bits(x[e]);
      lo[e] = x[e] - bf16_bits_to_f32(hb[e]);
    }
    uint16_t* C = reinterpret_cast<uint16_t*>(p.C) + ci;
    if (vec) {
      const u32x2_t o = {hb[0] | (hb[1] << 16), hb[2] | (hb[3] << 16)};
      *reinterpret_cast<u32x2_t*>(C) = o;
      if (p.C_lo) {
        const u32x2_t ol = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3])};
        *reinterpret_cast<u32x2_t*>(p.C_lo + ci) = ol;
      }
      if (p.C_dact) {
        const f32x4_t od = {dact[0], dact[1], dact[2], dact[3]};
        *reinterpret_cast<f32x4_t*>(p.C_dact + ci) = od;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nc) {
          C[e] = (uint16_t)hb[e];
          if (p.C_lo) p.C_lo[ci + e] = (uint16_t)f32_to_bf16_bits(lo[e]);
          if (p.C_dact) p.C_dact[ci + e] = dact[e];
        }
    }
  } else {
    float* C = reinterpret_cast<float*>(p.C) + ci;
    if (vec) {
      f32x4_t o = {x[0], x[1], x[2], x[3]};
      if (p.accumulate) o += *reinterpret_cast<const f32x4_t*>(C);
      *reinterpret_cast<f32x4_t*>(C) = o;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < nc) C[e] = p.accumulate ? x[e] + C[e] : x[e];
    }
  }
}

template <bool AKC, bool BKC, int NST>
__global__ __launch_bounds__(256) void gemm_bf16_small_kernel(GemmDev p, int out_bf16) {
  static_assert((NST & (NST - 1)) == 0 && NST >= 4, "ring of a power of two; the staging needs 17 KiB");
  extern __shared__ __align__(1024) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int Mv = dev_bound(p.M_dev, p.M), K0 = dev_bound(p.K_dev, p.K[0]);
  const int tiles_m = (Mv + 63) / 64, nt = tiles_m * p.tiles_n;   // the grid was sized for p.M
  int pid = blockIdx.x;
  if (pid >= nt) return;                                          // the whole block, before any barrier
  {  // each XCD gets a contiguous run of tiles, walked in groups of 8 tile rows
    const int xcd = pid & 7, idx = pid >> 3, per = nt >> 3, rem = nt & 7;
    pid = xcd * per + (xcd < rem ? xcd : rem) + idx;
  }
  const int gid = pid / (8 * p.tiles_n), first_m = gid * 8;
  const int gm = tiles_m - first_m < 8 ? tiles_m - first_m : 8;
  const int in_g = pid - gid * 8 * p.tiles_n;
  const int m0 = (first_m + in_g % gm) * 64, n0 = (in_g / gm) * 64;
  const int z = blockIdx.z, batch = z / p.splits, split = z - batch * p.splits;

  // reduction tiles of this block: [t0, t1) of the sequence that runs through the segments one after the other
  int nk = 0, seg = 0, skip = 0;
#pragma unroll
  for (int s = 0; s < kMaxSeg; ++s) nk += ((s == 0 ? K0 : p.K[s]) + BK - 1) / BK;
  if (p.splits > 1) {
    const int per = p.K_dev ? (nk + p.splits - 1) / p.splits : p.kper / BK;
    skip = split * per;
    nk = nk - skip < per ? nk - skip : per;
    for (int left = (K0 + BK - 1) / BK; seg < kMaxSeg - 1 && skip >= left; left = (p.K[seg] + BK - 1) / BK) {
      skip -= left;
      ++seg;
    }
  }
  typename std::conditional<AKC, DirectLoader<64, 4>, StridedLoader64>::type la;
  typename std::conditional<BKC, DirectLoader<64, 4>, StridedLoader64>::type lb;
  la.init(p.lda[0], Mv - m0, wave, lane);
  lb.init(p.ldb[0], p.N - n0, wave, lane);
  const int64_t stepA = AKC ? BK : BK * p.lda[0], stepB = BKC ? BK : BK * p.ldb[0];
  const int64_t offA = AKC ? (int64_t)m0 * p.lda[0] : m0, offB = BKC ? (int64_t)n0 * p.ldb[0] : n0;
  int k_left = (seg == 0 ? K0 : p.K[seg]) - skip * BK;
  const uint16_t* cA = p.A[seg] + (int64_t)batch * p.sA[seg] + offA + skip * stepA;
  const uint16_t* cB = p.B[seg] + (int64_t)batch * p.sB[seg] + offB + skip * stepB;
  auto issue = [&](int stage) {   // the tile under the cursor
    if (k_left <= 0) {            // on to the next segment, if there is one
      do { ++seg; } while (seg < kMaxSeg && p.K[seg] <= 0);
      if (seg < kMaxSeg) {
        cA = p.A[seg] + (int64_t)batch * p.sA[seg] + offA;
        cB = p.B[seg] + (int64_t)batch * p.sB[seg] + offB;
        k_left = p.K[seg];
      } else {
        seg = kMaxSeg - 1;        // all loads below are out of range
      }
    }
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(cA), rb = make_rsrc(cB);
    unsigned char* as = smem + stage * GS_STAGE;
#pragma unroll
    for (int j = 0; j < 2; ++j) la.load(j, ra, k_left, as, wave);
#pragma unroll
    for (int j = 0; j < 2; ++j) lb.load(j, rb, k_left, as + GS_TILE, wave);
    cA += stepA;
    cB += stepB;
    k_left -= BK;
  };
  uint32_t fa[2], fb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    fa[i] = gs_frag_base<AKC>(wm + 16 * i, lane);
    fb[i] = gs_frag_base<BKC>(wn + 16 * i, lane);
  }
  f32x4_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // s_waitcnt vmcnt(4 (NST - 2)): four loads per wave and tile, the oldest tile has landed
  constexpr int kFly = 4 * (NST - 2), kWaitOldest = (kFly & 15) | ((kFly >> 4) << 14) | 0x0f70;
  for (int t = 0; t < NST - 1; ++t) issue(t);
  for (int t = 0; t < nk; ++t) {
    __builtin_amdgcn_s_waitcnt(kWaitOldest);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();   // tile t is in LDS, and every wave is done with tile t - 1, whose stage is refilled
    __builtin_amdgcn_sched_barrier(0);
    issue((t + NST - 1) & (NST - 1));
    const unsigned char* as = smem + (t & (NST - 1)) * GS_STAGE;
    bf16x8_t a[2][2], b[2][2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[ks][i] = gs_frag<AKC>(as, fa[i], ks);
        b[ks][i] = gs_frag<BKC>(as + GS_TILE, fb[i], ks);
      }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], b[ks][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }

  // write-out through LDS, rows of 64 columns; the loads past the last tile have to land before their stages are reused
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  float* stage = reinterpret_cast<float*>(smem);
  const int q = lane >> 4, c = lane & 15;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) stage[(wm + 16 * i + 4 * q + r) * GS_LD + wn + 16 * j + c] = acc[i][j][r];
  __syncthreads();
  const int col = n0 + (tid & 15) * 4;
#pragma unroll 1
  for (int r = tid >> 4; r < 64; r += 16)
    if (m0 + r < Mv && col < p.N)
      gs_store4(p, out_bf16, batch, z, m0 + r, col,
                *reinterpret_cast<const f32x4_t*>(stage + r * GS_LD + (tid & 15) * 4));
}

template <bool AKC, bool BKC, int NST>
static hipError_t launch_small(const GemmDev& d, int out_bf16, hipStream_t st) {
  constexpr int smem = NST * GS_STAGE;
  auto kfn = gemm_bf16_small_kernel<AKC, BKC, NST>;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const dim3 grid((d.M + 63) / 64 * d.tiles_n, 1, d.nz);
  hipLaunchKernelGGL(kfn, grid, dim3(256), smem, st, d, out_bf16);
  return hipGetLastError();
}

hipError_t launch_gemm_bf16_small(const GemmDev& d, bool a_kc, bool b_kc, bool out_bf16, hipStream_t st) {
  if (a_kc && b_kc) return launch_small<true, true, 4>(d, out_bf16, st);
  if (a_kc && !b_kc) return launch_small<true, false, 4>(d, out_bf16, st);
  if (!a_kc && !b_kc) return launch_small<false, false, 4>(d, out_bf16, st);
  return hipErrorInvalidValue;  // (A strided, B contiguous) is not used by the path
}

}  // namespace asx
