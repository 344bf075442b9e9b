// Kernels of the stacked LSTM (lstm_wave.hip), as the entry points in lstm.hip drive them.
//
// One launch advances every layer that has work: layer l handles step t = d - l of wavefront d (forward; backward the
// mirror image), so L layers x T steps take T + L - 1 launches.  A layer-step is one product over two segments, the
// layer's own state and what it gets from its neighbour, and the cell.
//
// Operands are kept as FRAGMENT TILES: 16 rows x kKStep reduction indices = 64 lanes x 16 bytes = 1 KiB, in the order
// in which a wave's lanes hold them for the matrix instruction (lane l: row l % 16, the l / 16-th group of kVec
// consecutive reduction indices), laid out [reduction step][tile].  Reduction steps are padded with zeros.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace asx {

constexpr int kLsMaxLayers = 16;
constexpr int64_t kLsTile = 1024;   // bytes of a fragment tile

template <typename TE> struct LsGeom;
template <> struct LsGeom<uint16_t> { static constexpr int kVec = 8, kKStep = 32; };   // bf16
template <> struct LsGeom<float> { static constexpr int kVec = 4, kKStep = 16; };

// forward gate rows: 16 hidden units are 4 tiles of 16 rows; padded to whole groups of 32 units
inline int ls_gate_tiles(int H) { return (H + 31) / 32 * 8; }
// backward unit rows, padded to whole groups of 64 units
inline int ls_unit_tiles(int H) { return (H + 63) / 64 * 4; }
inline int ls_batch_tiles(int B) { return (B + 15) / 16; }
template <typename TE> inline int ls_ksteps(int K) { return (K + LsGeom<TE>::kKStep - 1) / LsGeom<TE>::kKStep; }
// reduction index of (gate, unit) in the backward products: gate * ls_gate_stride + unit
template <typename TE> __host__ __device__ inline int ls_gate_stride(int H) {
  return (H + LsGeom<TE>::kVec - 1) / LsGeom<TE>::kVec * LsGeom<TE>::kVec;
}

// Addresses in bytes or typed pointers; strides in elements of the pointer's type (bytes for char*).
// Sequences (ls_packed): what the products over all steps read (gate gradients, states, outputs, x) is kept per word, without
// rows for padding: sentence b's words are rows start[b] .. start[b + 1).  Otherwise a row per position, t B + b.
struct LsWords {
  int32_t* start;   // [B + 1], or null
  int32_t* pos;     // [T, B] row of a position, -1 where there is no word (made by the backward pass, as x)
  void* x;          // the input's rows of words, storage type
};
template <typename TE> bool ls_packed(int T, int B, int I, int H, int L);

struct LsFwd {
  LsWords words;
  // weights of layer l: fragment tiles made by launch_ls_prep_fwd, or the caller's rows (w_rows)
  const void *W_hh[kLsMaxLayers], *W_ih[kLsMaxLayers];
  const void* bias[kLsMaxLayers];
  const char *xF, *zeros;          // input of layer 0 as tiles, one block of x_stride bytes per step; zeroed tiles
  int64_t x_stride;
  char *hF_hi, *hF_lo;             // [L][2 slots][h_stride bytes]: h_{t-1} in slot t & 1 (lo: bf16 storage only)
  char *oF_hi, *oF_lo;             // [L - 1][2 slots][h_stride bytes]: output of step t (what layer l + 1 reads), slot t & 1
  int64_t h_stride;
  float *gates, *cs;               // [L][T,B,4H] i, f, g, o; [L][T+1,B,H] cell states
  void *hE, *out;                  // [L][T+1,B,H] states (packed: [B,H] initial ones, then the one before each word), [L - 1][T,B,H] outputs,
                                   // per word where packed; storage type
  void* y;                         // [T,B,H] output of the top layer
  float *hf, *cT;                  // [L][B,H] final h: h0 from the prepare launch, overwritten at a sentence's last step; final c (or null)
  const int32_t* lengths;
  int T, B, I, H, L;
  int w_rows;                      // one step: the caller's weight rows are read
  int direct;                      // one step: layer 0 reads x, h0 and c0, and prepares the states of the other layers
  const void* x;                   // the caller's
  const float *h0, *c0;            // the caller's initial states (null: zeros)
  int x_apart;                     // layer 0: gates hold x W_ih^T + b when a wavefront starts (x and W_ih are not read)
  uint32_t drop_thr;               // dropout on the outputs below the top layer; 0: none
  float drop_scale;
  uint64_t drop_seed;
};

struct LsBwd {
  LsWords words;
  const char *WT_hh[kLsMaxLayers], *WT_up[kLsMaxLayers];   // tiles of W_hh[l]^T and of W_ih[l + 1]^T
  const float *gates, *cs, *dy, *dhT, *dcT;                // dhT, dcT [L][B,H] may be null
  float* dcs;                                              // [L][B,H] running gradient w.r.t. c (ends as dc0)
  float* dh0;                                              // [L][B,H] or null
  void* dG;                                                // [L][T,B,4H] gate gradients, per word where packed; storage type
  char* dGF;                                               // [L][2 slots][g_stride bytes]: the same as tiles, slot t & 1
  int64_t g_stride;
  float* dbacc;                                            // [L][batch tiles][4H]: column sums of the gate gradients
  const int32_t* lengths;
  int T, B, H, L;
  uint32_t drop_thr;
  float drop_scale;
  uint64_t drop_seed;
};

// Before the first wavefront, unless p.direct: states of step 0 (h0, c0 may be null = zeros), x and, unless p.w_rows, the
// weights as tiles (W_hh, W_ih: the caller's rows; p.W_*: where the tiles go).
struct LsPrepFwd {
  const void *W_hh[kLsMaxLayers], *W_ih[kLsMaxLayers];
};
// up to three arrays of 4-byte words
struct LsCopy {
  const void* src[3];
  void* dst[3];
  int64_t words[3];
  int n;
  void add(const void* s, void* d, int64_t bytes) { src[n] = s; dst[n] = d; words[n++] = bytes / 4; }
};
hipError_t launch_ls_copy(const LsCopy& c, hipStream_t st);
template <typename TE> hipError_t launch_ls_prep_fwd(const LsFwd& p, const LsPrepFwd& q, hipStream_t st);
// tiles of n transposed [4H,H] weights (W_hh[l], W_ih[l + 1]) into the places p.WT_* point to
struct LsPrepBwd {
  const void* W[2 * kLsMaxLayers];
  char* tiles[2 * kLsMaxLayers];
  int n, H;
  // packed (words.start not null): behind the weights, rows of x, of the initial states and of the positions
  LsWords words;
  const void* x;
  void* hE;
  int T, B, I, L;
  void add(const void* w, const char* t) { W[n] = w; tiles[n++] = const_cast<char*>(t); }
};
template <typename TE> hipError_t launch_ls_prep_bwd(const LsPrepBwd& q, hipStream_t st);
// wavefront d = 0 .. T + L - 2
template <typename TE> hipError_t launch_ls_wave_fwd(const LsFwd& p, int d, hipStream_t st);
// wavefront d = 0 .. T + L - 2 + (dh0 != null)
template <typename TE> hipError_t launch_ls_wave_bwd(const LsBwd& p, int d, hipStream_t st);
// db[l][col] = sum over batch tiles of dbacc
struct LsBiasOut {
  float* db[kLsMaxLayers];
};
hipError_t launch_ls_bias_reduce(const float* dbacc, const LsBiasOut& o, int L, int nct, int cols, hipStream_t st);
// Whether the input product of layer 0 is one product over all steps ahead of the wavefronts.
template <typename TE> bool ls_input_apart(int T, int I, int H, int L);
// Whether forward wavefronts read the caller's weight rows instead of tiles made from them.
template <typename TE> bool ls_reads_weight_rows(int T, int I, int H);
// Whether layer 0 of one step reads the caller's initial state and input instead of tiles made from them.
template <typename TE> bool ls_reads_states(int H, int B);
// Reduction steps of those rows that a wave has in flight in the smaller blocks (bf16; K: input width of the layer).
int ls_row_steps_in_flight(int K, int H);

}  // namespace asx
