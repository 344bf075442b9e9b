// bf16 products that do not fill the 256 x 256 kernels (gfx950): square block tiles of 64 or 128, an NST-stage LDS ring.
//
// 64 x 64 tiles, four stages: a product of a hundred rows and a thousand columns is 8 tiles of 128 x 128, each of which
// walks the whole reduction on one compute unit while the others idle; there are four times as many blocks with a
// quarter of the work per reduction tile.  0.26 us per 64 reduction elements and compute unit, its LDS traffic (16 KiB in,
// 32 KiB out), however many blocks share it.
// 128 x 128 tiles: 0.58 us per 64 reduction elements with a compute unit to itself (four stages; 0.5 where a quarter of the
// units have one), 0.85 to 0.95 for two blocks that share one (two stages each: 64 KiB of LDS per block).  Rates and the
// choice between the shapes: gemm_plan.
// Loads go HBM -> LDS directly in every orientation, NST tiles ahead, one barrier per tile, no branch and the same number of
// loads in flight at every wait; the last tiles have a loop without loads (LACED) or read out of range, i.e. zeros.
// What bounds it is the stream of loads: without fragment reads and matrix instructions a tile takes 0.57 us (32 KiB per
// compute unit, 57 bytes a nanosecond), contiguous operands or a fifth stage change nothing, operands that all blocks share
// 0.49.  The rest was the chain barrier -> fragment reads -> matrix instructions of a wave that has its SIMD to itself, so
// the reads of half a tile run between the matrix instructions of the half before (gemm_tile_laced: where that is faster).
// Without / with, and without loads past the end: 4096 x 1024 x 6400 TN 70.1 / 63.9 us, 1024 x 1024 x 6400 TN 62.0 / 54.0, 6400 x
// 1024 x 3072 NT 53.5 / 49.9, 2257 x 1000 x 3000 NT 38.2 / 36.0, 6400 x 1024 x 2048 NN 40.9 / 38.7.  At most 256 registers per wave
// keep the accumulators out of the other register half, from which the compiler copies them around every matrix instruction
// of that loop.
//   * reduction-contiguous operand: LDS [rows][64 k] as in gemm_bf16.hip;
//   * strided operand: LDS [64 k][columns] as in memory, fragments by transposing reads.  A 16-lane group reads four
//     k-rows x 32 bytes; the 32-byte segments of a row are XOR-swizzled so that the four land in different banks.
#include "common.h"
#include "db_reduce_dev.h"
#include "gemm.h"
#include "gemm_dev.h"
#include "lds_limit.h"
#include "wave_pipe.h"

#include <type_traits>

namespace asx {

// 64 k-rows x COLS columns of a strided operand, 1 KiB per wave-wide load
template <int COLS> struct StridedLoader {
  static constexpr int RPL = 512 / COLS, NL = COLS / 32;   // k-rows per load, loads per wave
  uint32_t voff[NL];
  int k;
  // 32-byte segments of k-row k are stored at segment ^ swizzle(k)
  static __device__ __forceinline__ int swizzle(int k) { return COLS == 64 ? (k >> 1) & 3 : k & 3; }
  __device__ __forceinline__ void init(int64_t ld, int cols_left, int wave, int lane) {
    constexpr int CPR = COLS / 8;   // 16-byte chunks of a row
    k = RPL * wave + lane / CPR;
    const int pc = lane % CPR, seg = (pc >> 1) ^ swizzle(lane / CPR);   // (4 RPL j and RPL wave are multiples of 4)
    const int col = (seg * 2 + (pc & 1)) * 8;
#pragma unroll
    for (int j = 0; j < NL; ++j)
      voff[j] = col < cols_left ? (uint32_t)(((int64_t)(k + 4 * RPL * j) * ld + col) * 2) : kOob;
  }
  __device__ __forceinline__ void load(int j, const __amdgpu_buffer_rsrc_t& rs, int k_left, unsigned char* lds_tile,
                                       int wave) const {
    const uint32_t off = k + 4 * RPL * j < k_left ? voff[j] : kOob;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(lds_tile + (wave + 4 * j) * 1024), 16, off, 0, 0, 0);
  }
};

// Fragment of the 16x16x32 instruction: 16 rows (columns) from row0 on x 32 reduction elements, step ks of the tile.
template <bool KC, int COLS> __device__ __forceinline__ uint32_t gs_frag_base(int row0, int lane) {
  if constexpr (KC) {
    const int row = row0 + (lane & 15);
    return (uint32_t)(row * ROWB + (((lane >> 4) ^ (row & 7) ^ ((row >> 3) & 1)) << 4));
  } else {
    const int k = (lane >> 4) * 8 + ((lane & 15) >> 2);   // this lane presents four columns of k-rows k and k + 4
    const int cb = (row0 + (lane & 3) * 4) * 2;
    return (uint32_t)(k * COLS * 2 + (((cb >> 5) ^ StridedLoader<COLS>::swizzle(k)) << 5) + (cb & 31));
  }
}
template <bool KC, int COLS> __device__ __forceinline__ bf16x8_t gs_frag(const unsigned char* tile, uint32_t base, int ks) {
  if constexpr (KC) {
    return *reinterpret_cast<const bf16x8_t*>(tile + (base ^ (uint32_t)(ks << 6)));
  } else {
    constexpr uint32_t flip = COLS == 64 ? 64u : 0u;      // k-row k + 4 has another swizzle in 128-byte rows
    union { s16x4_t h[2]; bf16x8_t v; } u;
    u.h[0] = lds_read_tr((lds_s16x4_t*)(lds_void_t*)(tile + base + ks * COLS * 64));
    u.h[1] = lds_read_tr((lds_s16x4_t*)(lds_void_t*)(tile + (base ^ flip) + ks * COLS * 64 + COLS * 8));
    return u.v;
  }
}

// What sets an instance of a tile kernel apart (with the choices made in the kernel its other products were 1 to 8 % slower)
enum TileExtra { kNoExtra, kSecond, kCopy, kStats, kPast };   // C_second; copy_pos; row_stats; past_caches

// Epilogue of four consecutive columns of a row, in whole vectors
template <bool COPY>
__device__ __forceinline__ void gs_finish4(const GemmDev& p, int out_bf16, int batch, int row, int col, f32x4_t v,
                                           const f32x4_t& bias4) {
  const int64_t ci = (int64_t)batch * p.sC + (int64_t)row * p.ldc + col;
  v += bias4;
  if (p.act_tanh) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = tanhf(v[e]);
  }
  f32x4_t dact = 1.f - v * v;
  if (p.drop_thr) {
    uint32_t w[4];
    dropout_words4(((uint64_t)row * p.N + col) >> 2, p.drop_seed, w);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float m = w[e] >= p.drop_thr ? p.drop_scale : 0.f;
      v[e] *= m;
      dact[e] *= m;
    }
  }
  if (p.gate) v *= *reinterpret_cast<const f32x4_t*>(p.gate + (int64_t)row * p.ldg + col);
  const int copy = COPY ? p.copy_pos[row] : -1;
  const int64_t cc = (int64_t)copy * p.ldc + col;
  if (p.C_dact && (copy >= 0 || !COPY)) *reinterpret_cast<f32x4_t*>(p.C_dact + (COPY ? cc : ci)) = dact;
  if (out_bf16) {
    uint32_t hb[4];
    float lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      hb[e] = f32_to_bf16_bits(v[e]);
      lo[e] = v[e] - bf16_bits_to_f32(hb[e]);
    }
    const u32x2_t o = {hb[0] | (hb[1] << 16), hb[2] | (hb[3] << 16)};
    *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(p.C) + ci) = o;
    if (COPY && copy >= 0) *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(p.C_copy) + cc) = o;
    if (p.C_lo) {
      const u32x2_t ol = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3])};
      *reinterpret_cast<u32x2_t*>(p.C_lo + ci) = ol;
    }
  } else {
    float* C = reinterpret_cast<float*>(p.C) + ci;
    if (p.accumulate) v += *reinterpret_cast<const f32x4_t*>(C);
    *reinterpret_cast<f32x4_t*>(C) = v;
    if (COPY && copy >= 0) *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(p.C_copy) + cc) = v;
  }
}
// The same element by element: nc columns inside, nothing aligned
template <bool COPY>
__device__ __forceinline__ void gs_finish_ragged(const GemmDev& p, int out_bf16, int batch, int z, int row, int col,
                                                 const f32x4_t& v) {
  const int nc = p.N - col < 4 ? p.N - col : 4;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (e >= nc) continue;
    float x = v[e];
    if (p.splits > 1) {
      p.partial[((int64_t)z * p.M + row) * p.N + col + e] = x;
      continue;
    }
    if (p.bias) x += bf16_bits_to_f32(p.bias[col + e]);
    if (p.act_tanh) x = tanhf(x);
    float dact = 1.f - x * x;
    if (p.drop_thr) {
      const float m = dropout_mult((uint64_t)row * p.N + col + e, p.drop_seed, p.drop_thr, p.drop_scale);
      x *= m;
      dact *= m;
    }
    if (p.gate) x *= p.gate[(int64_t)row * p.ldg + col + e];
    const int64_t ci = (int64_t)batch * p.sC + (int64_t)row * p.ldc + col + e;
    const int copy = COPY ? p.copy_pos[row] : -1;
    const int64_t cc = (int64_t)copy * p.ldc + col + e;
    if (p.C_dact && (copy >= 0 || !COPY)) p.C_dact[COPY ? cc : ci] = dact;
    if (out_bf16) {
      const uint32_t hb = f32_to_bf16_bits(x);
      reinterpret_cast<uint16_t*>(p.C)[ci] = (uint16_t)hb;
      if (COPY && copy >= 0) reinterpret_cast<uint16_t*>(p.C_copy)[cc] = (uint16_t)hb;
      if (p.C_lo) p.C_lo[ci] = (uint16_t)f32_to_bf16_bits(x - bf16_bits_to_f32(hb));
    } else {
      float* C = reinterpret_cast<float*>(p.C);
      C[ci] = p.accumulate ? x + C[ci] : x;
      if (COPY && copy >= 0) reinterpret_cast<float*>(p.C_copy)[cc] = x;
    }
  }
}

// Softmax statistics of a staged row's BM columns by four lanes, which take every fourth vector: few steps across lanes, which
// is what the time goes to (16 and 32 lanes with a vector each, 128 x 32000 x 1024: 17.9 -> 22.4 us).
template <int CTRL> __device__ __forceinline__ float gs_quad(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;
template <int BM> __device__ __forceinline__ TileStat gs_stats(const float* row, int part, int col0, int ncols) {
  constexpr float L2E = 1.4426950408889634f;
  constexpr int NV = BM / 16;
  f32x4_t x[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) x[i] = *reinterpret_cast<const f32x4_t*>(row + (part + 4 * i) * 4);
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x[i][e] = (part + 4 * i) * 4 + e < ncols ? bf16_bits_to_f32(f32_to_bf16_bits(x[i][e])) : -INFINITY;
    m = fmaxf(fmaxf(m, x[i][0]), x[i][1]);
    m = fmaxf(fmaxf(m, x[i][2]), x[i][3]);
  }
  m = fmaxf(m, gs_quad<kQuadXor1>(m));
  m = fmaxf(m, gs_quad<kQuadXor2>(m));
  const bool any = m > -INFINITY;   // (a part of a row without a finite value adds nothing, unless NaN makes it so)
  const float mb = any ? -m * L2E : 0.f;
  float s0 = 0.f, s1 = 0.f;
  int idx = 0x7fffffff;
#pragma unroll
  for (int i = NV - 1; i >= 0; --i)
#pragma unroll
    for (int e = 3; e >= 0; --e) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(x[i][e], L2E, mb));
      if (e & 1) s1 += p;
      else s0 += p;
      idx = x[i][e] == m ? (part + 4 * i) * 4 + e : idx;
    }
  float s = s0 + s1;
  s += gs_quad<kQuadXor1>(s);
  s += gs_quad<kQuadXor2>(s);
  idx = any && idx != 0x7fffffff ? col0 + idx : 0x7fffffff;
  int o = __builtin_amdgcn_update_dpp(0, idx, kQuadXor1, 0xf, 0xf, false);
  idx = o < idx ? o : idx;
  o = __builtin_amdgcn_update_dpp(0, idx, kQuadXor2, 0xf, 0xf, false);
  idx = o < idx ? o : idx;
  return TileStat{m, s, idx, 0};
}

// Block `id` of a launch's tiles of all batches and splits; dynamic LDS: NST * 2 * 32 TW * ROWB bytes.  (p by value: by reference the
// instances take five registers more and 182 x 51130 x 128 18.7 us for 17.2.)
template <int TW, bool AKC, bool BKC, int NST, bool LACED, TileExtra EXTRA>
__device__ __forceinline__ void gemm_bf16_tile_block(GemmDev p, int out_bf16, int id) {
  extern __shared__ __align__(1024) unsigned char smem[];
  constexpr int BM = 32 * TW, TILE = BM * ROWB, STAGE = 2 * TILE;   // square block tile; bytes of an operand tile, a stage
  constexpr int NL = TW, LD = BM + 4;                               // loads per wave, operand and tile; staging row (floats)
  static_assert((NST & (NST - 1)) == 0 && NST * STAGE >= 64 * LD * 4, "ring of a power of two; write-out staging");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * 16 * TW, wn = (wave & 1) * 16 * TW;
  const int Mv = dev_bound(p.M_dev, p.M), K0 = dev_bound(p.K_dev, p.K);
  const int tiles_m = (Mv + BM - 1) / BM, nt = tiles_m * p.tiles_n;   // the grid was sized for p.M
  // Each XCD gets a contiguous run of the tiles of all products (batches, splits), a product's walked in groups of 8 tile rows: its
  // L2 then brings an operand of a batch, or a split's part of both operands, from memory once.
  const int total = nt * p.nz, xcd = id & 7, per = total >> 3, rem = total & 7;
  if ((id >> 3) >= per + (xcd < rem)) return;                     // the whole block, before any barrier
  int pid = xcd * per + (xcd < rem ? xcd : rem) + (id >> 3), z = 0;
  if (p.nz > 1) {
    z = __builtin_amdgcn_readfirstlane(pid / nt);
    pid -= z * nt;
  }
  const int gid = pid / (8 * p.tiles_n), first_m = gid * 8;
  const int gm = tiles_m - first_m < 8 ? tiles_m - first_m : 8;
  const int in_g = pid - gid * 8 * p.tiles_n;
  const int m0 = (first_m + in_g % gm) * BM, n0 = (in_g / gm) * BM;
  const int batch = z / p.splits, split = z - batch * p.splits;
  const bool second = EXTRA == kSecond && batch == 1;                      // segment 0 alone, to C_second
  const int nseg = second ? 1 : p.nseg;

  // reduction tiles of this block: [t0, t1) of the sequence that runs through the segments one after the other
  const int ks = (p.K + BK - 1) / BK;
  int nk = (K0 + BK - 1) / BK + (nseg - 1) * ks, seg = 0, skip = 0;
  if (p.splits > 1) {
    const int per = p.K_dev ? (nk + p.splits - 1) / p.splits : p.kper / BK;
    skip = split * per;
    nk = nk - skip < per ? nk - skip : per;
    for (; seg < nseg - 1 && skip >= ks; ++seg) skip -= ks;   // (K0 = K where there are more segments than one)
  }
  typename std::conditional<AKC, DirectLoader<BM, 4>, StridedLoader<BM>>::type la;
  typename std::conditional<BKC, DirectLoader<BM, 4>, StridedLoader<BM>>::type lb;
  la.init(p.lda, Mv - m0, wave, lane);
  lb.init(p.ldb, p.N - n0, wave, lane);
  const int64_t stepA = AKC ? BK : BK * p.lda, stepB = BKC ? BK : BK * p.ldb;
  const int64_t offA = AKC ? (int64_t)m0 * p.lda : m0, offB = BKC ? (int64_t)n0 * p.ldb : n0;
  int k_left = K0 - skip * BK;
  const uint16_t* cA = p.A[seg] + (int64_t)batch * p.sA + offA + skip * stepA;
  const uint16_t* cB = p.B[seg] + (int64_t)batch * p.sB + offB + skip * stepB;
  auto issue = [&](int stage) {   // the tile under the cursor
    if (k_left <= 0) {            // on to the next segment, if there is one
      if (++seg < nseg) {
        cA = p.A[seg] + (int64_t)batch * p.sA + offA;
        cB = p.B[seg] + (int64_t)batch * p.sB + offB;
        k_left = p.K;
      } else {
        seg = nseg - 1;           // all loads below are out of range
      }
    }
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(cA), rb = make_rsrc(cB);
    unsigned char* as = smem + stage * STAGE;
#pragma unroll
    for (int j = 0; j < NL; ++j) la.load(j, ra, k_left, as, wave);
#pragma unroll
    for (int j = 0; j < NL; ++j) lb.load(j, rb, k_left, as + TILE, wave);
    cA += stepA;
    cB += stepB;
    k_left -= BK;
  };
  uint32_t fa[TW], fb[TW];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    fa[i] = gs_frag_base<AKC, BM>(wm + 16 * i, lane);
    fb[i] = gs_frag_base<BKC, BM>(wn + 16 * i, lane);
  }
  f32x4_t acc[TW][TW];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // Two sets of fragments, one per half (32 reduction elements) of a tile.  LACED: the reads of a half run between the matrix
  // instructions of the half before it; else all reads of a tile come first and the other blocks of the compute unit run
  // meanwhile.  s_waitcnt vmcnt: 2 NL loads per wave and tile, all but NST - 2 (LACED, ahead of the first barrier: NST - 1)
  // tiles have landed.  The sums are the same.
  constexpr int kFly = 2 * NL * (NST - 2), kFly0 = 2 * NL * (NST - 1);
  constexpr int kWaitNext = (kFly & 15) | ((kFly >> 4) << 14) | 0x0070, kWaitOldest = kWaitNext | 0x0f00;
  constexpr int kWaitFirst = (kFly0 & 15) | ((kFly0 >> 4) << 14) | 0x0f70;
  bf16x8_t a[2][TW], b[2][TW];
  auto read = [&](int stage, int ks, int i) {
    const unsigned char* as = smem + stage * STAGE;
    b[ks][i] = gs_frag<BKC, BM>(as + TILE, fb[i], ks);
    a[ks][i] = gs_frag<AKC, BM>(as, fa[i], ks);
  };
  auto mul = [&](int ks, int i) {
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][i], b[ks][j], acc[i][j], 0, 0, 0);
  };
  if constexpr (LACED) {
    static_assert(NST == 2 || NST == 4, "the waits of the last tiles");
    if (nk >= NST) {
      for (int t = 0; t < NST; ++t) issue(t);
      __builtin_amdgcn_s_waitcnt(kWaitFirst);
    } else {
      for (int t = 0; t < nk; ++t) issue(t);
      __builtin_amdgcn_s_waitcnt(0x0f70);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < TW; ++i) read(0, 0, i);
    int t = 0;
    for (; t + NST < nk; ++t) {
      const int cur = t & (NST - 1);
#pragma unroll
      for (int i = 0; i < TW; ++i) {
        read(cur, 1, i);
        mul(0, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(kWaitNext);   // own loads of tile t + 1 have landed, own reads of tile t are in registers
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();            // tile t + 1 is in LDS, and every wave is done with tile t, whose stage is refilled
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TW; ++i) read((t + 1) & (NST - 1), 0, i);
      issue(cur);
#pragma unroll
      for (int i = 0; i < TW; ++i) mul(1, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    // The last NST tiles: nothing more to load.  (Loads past the end would be waited for before the write-out: 0.4 us, a tenth
    // of a short product.)
    for (; t < nk; ++t) {
#pragma unroll
      for (int i = 0; i < TW; ++i) {
        read(t & (NST - 1), 1, i);
        mul(0, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (t + 1 < nk) {
        const int behind = nk - 2 - t;         // tiles on their way after t + 1
        if (NST > 2 && behind >= 2) __builtin_amdgcn_s_waitcnt(kWaitNext);
        else if (NST > 2 && behind == 1) __builtin_amdgcn_s_waitcnt(((2 * NL) & 15) | (((2 * NL) >> 4) << 14) | 0x0070);
        else __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TW; ++i) read((t + 1) & (NST - 1), 0, i);
      }
#pragma unroll
      for (int i = 0; i < TW; ++i) mul(1, i);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    for (int t = 0; t < NST - 1; ++t) issue(t);
    for (int t = 0; t < nk; ++t) {
      __builtin_amdgcn_s_waitcnt(kWaitOldest);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();            // tile t is in LDS, and every wave is done with tile t - 1, whose stage is refilled
      __builtin_amdgcn_sched_barrier(0);
      issue((t + NST - 1) & (NST - 1));
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < TW; ++i) read(t & (NST - 1), ks, i);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < TW; ++i) mul(ks, i);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // write-out through LDS, rows of 64 columns; the loads past the last tile have to land before their stages are reused
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  float* stage = reinterpret_cast<float*>(smem);
  const int q = lane >> 4, c = lane & 15;
  constexpr int VPR = BM / 4;                 // groups of four columns per row
  const int col = n0 + (tid % VPR) * 4;
  const bool fuse = p.splits <= 1;
  if (second) out_bf16 = 0;
  const bool plain = p.vec_ok && (!fuse || second || (EXTRA != kCopy && !p.act_tanh && !p.drop_thr && !p.gate && !p.C_lo && !p.C_dact));
  f32x4_t bias4 = {0.f, 0.f, 0.f, 0.f};
  float bias1[TW];   // kStats: added on the way into LDS
  if constexpr (EXTRA == kStats) {
#pragma unroll
    for (int j = 0; j < TW; ++j) bias1[j] = p.bias && n0 + wn + 16 * j + c < p.N ? bf16_bits_to_f32(p.bias[n0 + wn + 16 * j + c]) : 0.f;
  }
  if (EXTRA != kStats && fuse && p.bias)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < p.N) bias4[e] = bf16_bits_to_f32(p.bias[col + e]);
  constexpr int RP = 256 / VPR, RU = 4;       // rows per sweep of the block, sweeps whose reads go together
#pragma unroll 1
  for (int half = 0; half < BM / 64; ++half) {   // 64 rows at a time
    if (wm / 64 == half) {
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            stage[(wm % 64 + 16 * i + 4 * q + r) * LD + wn + 16 * j + c] = EXTRA == kStats ? acc[i][j][r] + bias1[j] : acc[i][j][r];
    }
    __syncthreads();
    const int left = Mv - m0 - half * 64 < 64 ? Mv - m0 - half * 64 : 64;   // rows inside (may be none)
    if constexpr (EXTRA == kStats) {
      const TileStat t = gs_stats<BM>(stage + (tid >> 2) * LD, tid & 3, n0, p.N - n0);
      if ((tid & 3) == 0 && (tid >> 2) < left) p.row_stats[(int64_t)(m0 + half * 64 + (tid >> 2)) * p.tiles_n + n0 / BM] = t;
    }
    if (plain) {   // bias and accumulation only: nothing tested per row but the bounds
#pragma unroll
      for (int r0 = 0; r0 < 64; r0 += RU * RP) {
        f32x4_t v[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u)
          v[u] = *reinterpret_cast<const f32x4_t*>(stage + (r0 + u * RP + tid / VPR) * LD + (tid % VPR) * 4);
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const int r = r0 + u * RP + tid / VPR, row = m0 + half * 64 + r;
          if (r >= left || col >= p.N) continue;
          if (!fuse) {
            *reinterpret_cast<f32x4_t*>(p.partial + ((int64_t)z * p.M + row) * p.N + col) = v[u];
            continue;
          }
          const int64_t ci = (int64_t)batch * p.sC + (int64_t)row * p.ldc + col;
          v[u] += bias4;
          if (out_bf16) {
            const u32x2_t o = {pack_bf16(v[u][0], v[u][1]), pack_bf16(v[u][2], v[u][3])};
            *reinterpret_cast<u32x2_t*>(reinterpret_cast<uint16_t*>(p.C) + ci) = o;
          } else {
            float* C = (second ? p.C_second : reinterpret_cast<float*>(p.C)) + ci;
            if (p.accumulate) v[u] += *reinterpret_cast<const f32x4_t*>(C);
            if (EXTRA == kPast) __builtin_nontemporal_store(v[u], reinterpret_cast<f32x4_t*>(C));
            else *reinterpret_cast<f32x4_t*>(C) = v[u];
          }
        }
      }
    } else if (col < p.N) {
#pragma unroll 1
      for (int r0 = tid / VPR; r0 < left; r0 += RP) {
        const int row = m0 + half * 64 + r0;
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(stage + r0 * LD + (tid % VPR) * 4);
        if (p.vec_ok) gs_finish4<EXTRA == kCopy>(p, out_bf16, batch, row, col, v, bias4);
        else gs_finish_ragged<EXTRA == kCopy>(p, out_bf16, batch, z, row, col, v);
      }
    }
    if (half + 1 < BM / 64) __syncthreads();
  }
}

template <int TW, bool AKC, bool BKC, int NST, bool LACED, TileExtra EXTRA>
__global__ __launch_bounds__(256, LACED ? 2 : 1) void gemm_bf16_tile_kernel(GemmDev p, int out_bf16) {
  gemm_bf16_tile_block<TW, AKC, BKC, NST, LACED, EXTRA>(p, out_bf16, blockIdx.x);
}

template <int TW, bool AKC, bool BKC, int NST, bool LACED, TileExtra EXTRA = kNoExtra>
static hipError_t launch_tile_shape(const GemmDev& d, int out_bf16, hipStream_t st) {
  constexpr int BM = 32 * TW, smem = NST * 2 * BM * ROWB;
  auto kfn = gemm_bf16_tile_kernel<TW, AKC, BKC, NST, LACED, EXTRA>;
  static LdsLimit limit;
  const hipError_t e = limit.raise(reinterpret_cast<const void*>(kfn), smem);
  if (e != hipSuccess) return e;
  const int64_t blocks = (int64_t)d.tiles_m * d.tiles_n * d.nz;
  if (blocks > (1 << 24)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks);
  hipLaunchKernelGGL(kfn, grid, dim3(256), smem, st, d, out_bf16);
  return hipGetLastError();
}

// Reads first and laced, us, 128 x 128 tiles (64 x 64 where it says so): up to 256 blocks 1024 x 1024 x 6400 TN 62.6 / 53.8, 2257 x
// 1000 x 1000 NN 20.8 / 18.0, 1920 x 1024 x 384 NT 13.2 / 12.2; 64: 128 x 1024 x 3072 NT 16.9 / 14.5, 1024 x 1024 x 6400 TN 31.3 /
// 30.7.  More, A contiguous: 6400 x 1024 x 3072 NT 52.1 / 48.9, 600 x 8000 x 256 NT 13.8 / 13.4, 6400 x 1024 x 2048 NN 40.5 / 37.9, x
// 256 15.0 / 14.1; 64: 6400 x 1024 x 1024 NT 33.7 / 30.6, 8192 x 1024 x 1024 NN 39.2 / 36.3.  More, both strided, where two blocks
// share a compute unit's transposing reads: 16000 x 512 x 1286 28.0 / 29.1, 9000 x 640 x 3000 44.2 / 47.9, 4096 x 2048 x 2048 35.3 /
// 36.2; 64: 2048 x 768 x 1500 13.8 / 14.5, 4096 x 1024 x 6400 84.8 / 91.1.
bool gemm_tile_laced(bool a_kc, int64_t blocks) { return a_kc || blocks <= 256; }

// both operands strided
template <TileExtra EXTRA> static hipError_t launch_tile_tn(const GemmDev& d, GemmTile tile, int out_bf16, hipStream_t st) {
  if (!gemm_tile_laced(false, (int64_t)d.tiles_m * d.tiles_n * d.nz))
    return tile == kTile64 ? launch_tile_shape<2, false, false, 4, false, EXTRA>(d, out_bf16, st)
                           : launch_tile_shape<4, false, false, 2, false, EXTRA>(d, out_bf16, st);
  return tile == kTile64 ? launch_tile_shape<2, false, false, 4, true, EXTRA>(d, out_bf16, st)
                         : launch_tile_shape<4, false, false, 4, true, EXTRA>(d, out_bf16, st);   // (a block per compute unit)
}
// A contiguous
template <bool BKC>
static hipError_t launch_tile_form(const GemmDev& d, GemmTile tile, int out_bf16, hipStream_t st) {
  constexpr bool AKC = true;
  const int64_t blocks = (int64_t)d.tiles_m * d.tiles_n * d.nz;
  // (launch_gemm_bf16: 64 x 64 only)
  if constexpr (!BKC) {
    if (d.C_second) return launch_tile_shape<2, AKC, BKC, 4, true, kSecond>(d, out_bf16, st);
  }
  if constexpr (BKC) {
    if (d.row_stats) {
      if (tile == kTile64) return launch_tile_shape<2, AKC, BKC, 4, true, kStats>(d, out_bf16, st);
      return blocks <= 256 ? launch_tile_shape<4, AKC, BKC, 4, true, kStats>(d, out_bf16, st) : hipErrorInvalidValue;
    }
    if (d.copy_pos) {
      if (tile == kTile64) return launch_tile_shape<2, AKC, BKC, 4, true, kCopy>(d, out_bf16, st);
      return blocks <= 256 ? launch_tile_shape<4, AKC, BKC, 4, true, kCopy>(d, out_bf16, st)
                           : launch_tile_shape<4, AKC, BKC, 2, true, kCopy>(d, out_bf16, st);
    }
  }
  if (d.copy_pos) return hipErrorInvalidValue;
  if (tile == kTile64) return launch_tile_shape<2, AKC, BKC, 4, true>(d, out_bf16, st);
  // 128 KiB of LDS where no compute unit gets a second block anyway
  if (blocks <= 256) return launch_tile_shape<4, AKC, BKC, 4, true>(d, out_bf16, st);
  return launch_tile_shape<4, AKC, BKC, 2, true>(d, out_bf16, st);
}

// ---- several products in one launch ------------------------------------------------
// Independent products of one pass that each leave the chip half empty, or are over before a launch is: their blocks one
// product behind the other in one grid, 64 x 64 tiles (64 KiB of LDS, two blocks on a compute unit).  The product whose blocks
// walk the longest reduction comes first; the short blocks of the others fill in behind it.  A training step, apart / together
// (dW_c with dC and dH1; dW_a with the last product of d_h_dec and d_h_enc): 1920 x 512 271 / 252 us, one step of 128 x 1024
// 200 / 193, 6400 x 1024 (the latter three, 104 us of it apart) 1387 / 1377.
template <int TW, bool AKC, bool BKC, int NST, bool LACED, TileExtra EXTRA = kNoExtra>
struct TileMember {
  GemmDev d;
  int out_bf16, blocks;   // blocks: of the grid, a multiple of 8 so that a product's blocks keep their XCDs
  static constexpr int kSmem = NST * 2 * 32 * TW * ROWB;
  void set(const GemmDev& dev, bool obf) {
    d = dev;
    out_bf16 = obf;
    blocks = (d.tiles_m * d.tiles_n * d.nz + 7) / 8 * 8;
  }
  __device__ __forceinline__ void run(int id) const {
    gemm_bf16_tile_block<TW, AKC, BKC, NST, LACED, EXTRA>(d, out_bf16, id);
  }
};
template <typename F, typename... R>
__device__ __forceinline__ void run_member(int id, const F& f, const R&... rest) {
  if constexpr (sizeof...(R) > 0) {
    if (id >= f.blocks) return run_member(id - f.blocks, rest...);
  }
  f.run(id);
}
// last_first: the blocks of the last product come first
template <typename... M> __global__ __launch_bounds__(256, 2) void gemm_bf16_together_kernel(int last_first, M... m) {
  run_member(last_first ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x, m...);
}
template <typename... M> static hipError_t launch_members(bool last_first, hipStream_t st, const M&... m) {
  constexpr int sizes[] = {M::kSmem...};
  int smem = 0;
  for (int v : sizes) smem = v > smem ? v : smem;
  auto kfn = gemm_bf16_together_kernel<M...>;
  static LdsLimit limit;
  const hipError_t e = limit.raise(reinterpret_cast<const void*>(kfn), smem);
  if (e != hipSuccess) return e;
  int64_t blocks = 0;
  for (int64_t b : {(int64_t)m.blocks...}) blocks += b;
  if (blocks > (1 << 24)) return hipErrorNotSupported;
  hipLaunchKernelGGL(kfn, dim3((unsigned)blocks), dim3(256), smem, st, (int)last_first, m...);
  return hipGetLastError();
}
// column sums of dlogits beside the products that read it
struct SumsMember {
  DbReduce d;
  int blocks;
  static constexpr int kSmem = kDbSmem;
  void set(const DbReduce& sums) {
    d = sums;
    blocks = ((d.V + kDbColumns - 1) / kDbColumns + 7) / 8 * 8;
  }
  __device__ __forceinline__ void run(int id) const {
    extern __shared__ __align__(1024) unsigned char smem[];
    if (id * kDbColumns < d.V) db_reduce_block<256>(d, id, reinterpret_cast<float*>(smem));
  }
};
using MemberTN = TileMember<2, false, false, 4, false>;
using MemberTNLaced = TileMember<2, false, false, 4, true>;
using MemberTN128 = TileMember<4, false, false, 2, false>;
using MemberTNPast = TileMember<2, false, false, 4, false, kPast>;
using MemberTNLacedPast = TileMember<2, false, false, 4, true, kPast>;
using MemberTN128Past = TileMember<4, false, false, 2, false, kPast>;
using MemberNN = TileMember<2, true, false, 4, true>;
using MemberNN128 = TileMember<4, true, false, 2, true>;
using MemberNNSecond = TileMember<2, true, false, 4, true, kSecond>;
using MemberNT = TileMember<2, true, true, 4, true>;

static int tile_ktiles(const GemmDev& d) {   // reduction tiles of a block
  return (d.nseg * ((d.K + BK - 1) / BK) + d.splits - 1) / d.splits;
}
template <typename TN, typename NN, typename TNPast>
static hipError_t launch_with_sums(const GemmDev* d, const TileForm* f, const DbReduce& sums, hipStream_t st) {
  if constexpr (!std::is_same<TN, TNPast>::value) {
    if (d[0].past_caches) return launch_with_sums<TNPast, NN, TNPast>(d, f, sums, st);
  }
  TN tn;
  NN nn;
  SumsMember s;
  tn.set(d[0], f[0].out_bf16);
  nn.set(d[1], f[1].out_bf16);
  s.set(sums);
  return launch_members(false, st, nn, tn, s);
}
template <typename First, typename TN>
static hipError_t launch_together_with(const GemmDev* d, const TileForm* f, int n, hipStream_t st) {
  First tn;
  tn.set(d[0], f[0].out_bf16);
  if (n == 2 && f[1].a_kc && !f[1].b_kc && d[1].C_second) {
    MemberNNSecond nn;
    nn.set(d[1], f[1].out_bf16);
    return launch_members(tile_ktiles(d[1]) > tile_ktiles(d[0]), st, tn, nn);
  }
  if (n >= 2 && f[1].a_kc && f[1].b_kc) {
    MemberNT nt;
    nt.set(d[1], f[1].out_bf16);
    if (n == 2) return launch_members(false, st, tn, nt);
    TN last;
    last.set(d[2], f[2].out_bf16);
    if (n == 3 && !f[2].a_kc && !f[2].b_kc) return launch_members(false, st, tn, nt, last);
  }
  for (int i = 1; i < n; ++i)
    if (f[i].a_kc || f[i].b_kc) return hipErrorNotSupported;
  TN more[kMaxTogether - 1];
  for (int i = 1; i < n; ++i) more[i - 1].set(d[i], f[i].out_bf16);
  if (n == 2) return launch_members(false, st, tn, more[0]);
  if (n == 3) return launch_members(false, st, tn, more[0], more[1]);
  if (n == 4) return launch_members(false, st, tn, more[0], more[1], more[2]);
  return hipErrorNotSupported;
}
// past the caches: all of them, the first alone, or none
template <typename TN, typename TNPast>
static hipError_t launch_together_any(const GemmDev* d, const TileForm* f, int n, hipStream_t st) {
  int past = 0;
  for (int i = 0; i < n; ++i) past += d[i].past_caches ? 1 : 0;
  if (past == n) return launch_together_with<TNPast, TNPast>(d, f, n, st);
  return d[0].past_caches ? launch_together_with<TNPast, TN>(d, f, n, st) : launch_together_with<TN, TN>(d, f, n, st);
}
hipError_t launch_gemm_bf16_tiles_together(const GemmDev* d, const TileForm* f, int n, const DbReduce* sums, hipStream_t st) {
  if (n < 2 || f[0].a_kc || f[0].b_kc) return hipErrorNotSupported;
  if (sums) {
    if (n != 2 || !f[1].a_kc || f[1].b_kc || d[1].C_second) return hipErrorNotSupported;
    if (f[1].tile == kTile128) return f[0].tile == kTile128 ? launch_with_sums<MemberTN128, MemberNN128, MemberTN128Past>(d, f, *sums, st) : hipErrorNotSupported;
    return f[0].tile == kTile128 ? launch_with_sums<MemberTN128, MemberNN, MemberTN128Past>(d, f, *sums, st)
                                 : launch_with_sums<MemberTN, MemberNN, MemberTNPast>(d, f, *sums, st);
  }
  int64_t blocks = 0;
  for (int i = 0; i < n; ++i) {
    if (f[i].tile != kTile64) return hipErrorNotSupported;
    blocks += (int64_t)d[i].tiles_m * d[i].tiles_n * d[i].nz;
  }
  return gemm_tile_laced(false, blocks) ? launch_together_any<MemberTNLaced, MemberTNLacedPast>(d, f, n, st)
                                        : launch_together_any<MemberTN, MemberTNPast>(d, f, n, st);
}

// ---- few rows ----------------------------------------------------------------------
// 16 columns x 16 NJ rows per block, the reduction split over its eight waves (wave w takes steps w, w + 8, ...), fragments
// straight from the operands' rows into registers, PF - 1 lines ahead; the partial tiles meet in LDS and are added in wave
// order, and the epilogue follows.  A hundred rows and a thousand columns are a few tiles of 64 x 64: those need a split over
// blocks to fill the chip, and a split needs a second launch that reads the partial sums back.  What bounds this one is its
// launch and one or two memory latencies: 16 x 512 x 1536 5.4 us, 8.0 split and combined.
// The columns of B are the rows of the matrix instruction, so that a lane holds four consecutive columns of a row of C.
constexpr int kFewWaves = 8;
// (by value: a choice between variables that a lambda refers to would keep them in memory)
__device__ __forceinline__ const uint16_t* few_pick(int seg, const uint16_t* a, const uint16_t* b, const uint16_t* c) {
  return seg == 0 ? a : seg == 1 ? b : c;
}
template <int NJ, bool COPY>
__global__ __launch_bounds__(64 * kFewWaves) void gemm_bf16_few_kernel(GemmDev p, int out_bf16, int nseg) {
  constexpr int PF = 4;
  __shared__ f32x4_t red[kFewWaves * NJ * 64];   // [wave][row tile][lane]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = lane >> 4, c = lane & 15;
  // an XCD gets a contiguous run of column blocks with all their row blocks: its L2 fetches a row of B once
  const int nbm = (p.M + 16 * NJ - 1) / (16 * NJ), nbn = (p.N + 15) / 16, per = (nbn + 7) / 8;
  const int idx = blockIdx.x >> 3, bn = (blockIdx.x & 7) * per + idx / nbm;
  if (bn >= nbn) return;
  const int n0 = bn * 16, m0 = (idx % nbm) * 16 * NJ, K = p.K, nk = (K + 63) / 64;
  const int col = n0 + c < p.N ? n0 + c : p.N - 1;   // columns and rows outside repeat the last one; not stored
  const int64_t boff = (int64_t)col * p.ldb;
  int64_t aoff[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) aoff[j] = (int64_t)(m0 + 16 * j + c < p.M ? m0 + 16 * j + c : p.M - 1) * p.lda;
  const uint16_t *A0 = p.A[0], *A1 = p.A[1], *A2 = p.A[2], *B0 = p.B[0], *B1 = p.B[1], *B2 = p.B[2];
  f32x4_t acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // A step is a whole 128-byte line of every row, two matrix instructions: lane group q takes bytes 32 q .. 32 q + 31.
  u32x4_t bf[PF][2], af[PF][NJ][2];
  auto segment = [&](int step) { return (wave + step * kFewWaves >= nk) + (wave + step * kFewWaves >= 2 * nk); };
  auto first = [&](int step) { return (wave + step * kFewWaves - segment(step) * nk) * 64; };   // reduction index of a step
  auto load = [&](int slot, int step) {
    const int seg = segment(step), k0 = first(step);
    const uint16_t *A = few_pick(seg, A0, A1, A2), *B = few_pick(seg, B0, B1, B2);
    const int k = k0 + q * 16, ko[2] = {k < K ? k : k0, k + 8 < K ? k + 8 : k0};   // past the row's end: the line's start
    // the two halves of a line one behind the other, while it is on its way
#pragma unroll
    for (int h = 0; h < 2; ++h) bf[slot][h] = *reinterpret_cast<const u32x4_t*>(B + boff + ko[h]);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) af[slot][j][h] = *reinterpret_cast<const u32x4_t*>(A + aoff[j] + ko[h]);
  };
  auto mul = [&](int slot, int step) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool in = first(step) + q * 16 + h * 8 < K;   // chunks past the end: both operands cleared (0 * inf)
      u32x4_t b = bf[slot][h];
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = in ? b[e] : 0u;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        u32x4_t a = af[slot][j][h];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = in ? a[e] : 0u;
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, b), __builtin_bit_cast(bf16x8_t, a),
                                                         acc[j], 0, 0, 0);
      }
    }
  };
  wave_reduce<PF, 2 * (NJ + 1), 2 * NJ>(own_steps<kFewWaves>(nk * nseg, wave), load, mul);
#pragma unroll
  for (int j = 0; j < NJ; ++j) red[(wave * NJ + j) * 64 + lane] = acc[j];
  __syncthreads();
  if (wave >= NJ) return;
  f32x4_t v = red[wave * 64 + lane];
#pragma unroll
  for (int w = 1; w < kFewWaves; ++w) v += red[(w * NJ + wave) * 64 + lane];
  const int row = m0 + 16 * wave + c, ccol = n0 + 4 * q;
  if (row >= p.M || ccol >= p.N) return;
  if (!p.vec_ok) {
    gs_finish_ragged<COPY>(p, out_bf16, 0, 0, row, ccol, v);
    return;
  }
  f32x4_t bias4 = {0.f, 0.f, 0.f, 0.f};
  if (p.bias)
#pragma unroll
    for (int e = 0; e < 4; ++e) bias4[e] = bf16_bits_to_f32(p.bias[ccol + e]);
  gs_finish4<COPY>(p, out_bf16, 0, row, ccol, v, bias4);
}
hipError_t launch_gemm_bf16_few(const GemmDev& d, bool out_bf16, hipStream_t st) {
  const int nseg = d.nseg;
  if (nseg > 3 || d.splits != 1) return hipErrorInvalidValue;
  const int nj = d.M > 16 ? 2 : 1;
  const int64_t nbm = (d.M + 16 * nj - 1) / (16 * nj), per = ((d.N + 15) / 16 + 7) / 8;
  const dim3 grid((unsigned)(8 * per * nbm));
  auto kfn = nj == 2 ? (d.copy_pos ? gemm_bf16_few_kernel<2, true> : gemm_bf16_few_kernel<2, false>)
                     : (d.copy_pos ? gemm_bf16_few_kernel<1, true> : gemm_bf16_few_kernel<1, false>);
  hipLaunchKernelGGL(kfn, grid, dim3(64 * kFewWaves), 0, st, d, (int)out_bf16, nseg);
  return hipGetLastError();
}

hipError_t launch_gemm_bf16_tile(const GemmDev& d, GemmTile tile, bool a_kc, bool b_kc, bool out_bf16, hipStream_t st) {
  if (a_kc && b_kc) return launch_tile_form<true>(d, tile, out_bf16, st);
  if (a_kc && !b_kc) return launch_tile_form<false>(d, tile, out_bf16, st);
  if (!a_kc && !b_kc && !d.copy_pos)
    return d.past_caches ? launch_tile_tn<kPast>(d, tile, out_bf16, st) : launch_tile_tn<kNoExtra>(d, tile, out_bf16, st);
  return hipErrorInvalidValue;  // (A strided, B contiguous) is not used by the path
}

}  // namespace asx
