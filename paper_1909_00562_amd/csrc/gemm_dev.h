// Device-side description of a bf16 product and the addressing helpers its kernels share.
#pragma once
#include "common.h"
#include "gemm.h"

namespace asx {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

struct GemmDev {
  const uint16_t* A[kMaxSeg];
  const uint16_t* B[kMaxSeg];
  int64_t lda, ldb, sA, sB;   // the same for all segments, like K: every byte of the arguments costs a launch time (80 of them
  int K, nseg;                // 0.2 us a product of the smallest sizes)
  int M, N;
  int n_out;   // columns the vector write-out covers: N, or N rounded up to 4 where C's rows have padding
  int past_caches;
  void* C;
  uint16_t* C_lo;
  float* C_dact;
  int64_t ldc, sC;
  const int32_t* copy_pos; // row n of C also goes to row copy_pos[n] of C_copy, and of C_dact there alone (or null)
  void* C_copy;
  TileStat* row_stats;     // softmax statistics of a row's part of a tile (or null)
  float* C_second;         // batch of two: where the product of segment 0 alone goes (or null)
  const uint16_t* bias;
  const float* gate;
  int64_t ldg;
  int act_tanh, accumulate;
  uint32_t drop_thr;
  float drop_scale;
  uint64_t drop_seed;
  int splits;
  float* partial;
  int tiles_m, tiles_n;
  int group;   // tile rows per group of the persistent kernel's tile walk
  int kper;    // reduction elements per split, multiple of 64
  int vec_ok;  // rows of C (and C_lo, C_dact, gate) allow 8/16-byte vector access
  const int32_t* M_dev;   // device-side row count (or null): min(*M_dev, M) rows are valid
  const int32_t* K_dev;   // device-side reduction length of segment 0 (or null)
  int nz;                 // batch * splits
  int dyn_split;          // splits is the bound of a split chosen in the kernel from the row count (pp kernel)
};

// Results of a batch that lie apart, an argument of the one instance that writes them (in GemmDev its 128 bytes cost every
// product 0.2 us).
struct GemmApart {
  void* C[kMaxApart];
};
struct GemmNotApart {};

// size made by an earlier kernel of the stream, clamped to the bound the launch was sized for
__device__ __forceinline__ int dev_bound(const int32_t* count, int bound) {
  if (!count) return bound;
  const int v = *count;
  return v < 0 ? 0 : (v < bound ? v : bound);
}

constexpr uint32_t kOob = 0x80000000u;  // offset outside every buffer resource below

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base) {
  // raw buffer, 2 GiB range: offsets >= 2^31 (kOob) read as zero
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
}

constexpr int BK = 64;                  // reduction elements per LDS tile row
constexpr int ROWB = BK * 2;            // bytes per LDS tile row

typedef __attribute__((address_space(3))) void lds_void_t;
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// Transposing LDS read.  The parameter is __restrict__ for the compiler's wait insertion: without alias information on
// the instruction it takes every HBM -> LDS load in flight for a possible writer of what is read and waits for all of
// them (s_waitcnt vmcnt(0) ahead of the first such read of a tile), although the tiles in flight are other ones.  The
// waits that are needed are written out in the kernels, ahead of the barrier that hands a tile over.
__device__ __forceinline__ s16x4_t lds_read_tr(lds_s16x4_t* __restrict__ p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(p);
}

// ---- reduction-contiguous operand: HBM -> LDS, no registers ----------------------
// The tile's ROWS rows are split into groups of 8 rows (1 KiB of LDS); one wave-wide
// 16-byte load fills one group.  Per-lane byte offsets relative to element
// (row0, k0) are computed once per kernel; rows beyond the operand get kOob.
template <int ROWS, int NW>
struct DirectLoader {
  static constexpr int NL = ROWS / 8 / NW;   // loads per wave and tile
  uint32_t voff[NL];
  int chunk8;                                // first reduction element of this lane's chunk
  __device__ __forceinline__ void init(int64_t ld, int rows_left, int wave, int lane) {
    static_assert(NW % 2 == 0, "swizzle below assumes the parity of the row group is the wave's");
    const int rl = lane >> 3;                        // row inside the group
    const int chunk = (lane & 7) ^ rl ^ (wave & 1);  // logical 16-byte chunk that belongs in LDS slot `lane`
    chunk8 = chunk * 8;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int r = (wave + NW * j) * 8 + rl;
      voff[j] = r < rows_left ? (uint32_t)(((int64_t)r * ld + chunk * 8) * 2) : kOob;
    }
  }
  // X points at element (row0, k0); k_left = reduction elements left from k0
  __device__ __forceinline__ void load(int j, const __amdgpu_buffer_rsrc_t& rs, int k_left, unsigned char* lds_tile,
                                       int wave) const {
    const uint32_t off = chunk8 < k_left ? voff[j] : kOob;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(lds_tile + (wave + NW * j) * 1024), 16, off, 0, 0, 0);
  }
};

// the 64 x 64 and 128 x 128 kernel (gemm_tile.hip); d as launch_gemm_bf16 has filled it in
hipError_t launch_gemm_bf16_tile(const GemmDev& d, GemmTile tile, bool a_kc, bool b_kc, bool out_bf16, hipStream_t st);
// Several products in one launch; hipErrorNotSupported where there is no kernel for the combination.  64 x 64 tiles: {both
// strided, A contiguous with C_second}, {both strided, both contiguous}, the latter with another of both strided,
// two to four of both strided.  64 x 64 or
// 128 x 128: {both strided, A contiguous}, sums beside them.
struct TileForm {
  bool a_kc, b_kc, out_bf16;
  GemmTile tile;
};
hipError_t launch_gemm_bf16_tiles_together(const GemmDev* d, const TileForm* f, int n, const DbReduce* sums, hipStream_t st);
// whether that kernel's fragment reads run between its matrix instructions
bool gemm_tile_laced(bool a_kc, int64_t blocks);
// the kernel for few rows: both operands reduction-contiguous, up to three segments of the same length, no split, no batch
hipError_t launch_gemm_bf16_few(const GemmDev& d, bool out_bf16, hipStream_t st);

}  // namespace asx
