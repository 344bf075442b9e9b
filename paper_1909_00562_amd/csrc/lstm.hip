// Stacked LSTM without input feeding (section 3.2, Fig. 3; cell as stated in
// include/lstm_stack.h): forward and backward over all steps of one side, entry
// points, workspace and schedule.
//
// The layer-steps of one wavefront (layer l at step d - l) run as one launch, input
// product, recurrent product and cell together (lstm_wave.hip; a wide x has its product
// over all steps ahead of them).  Backward walks the wavefronts the other way; the weight
// gradients and the gradient of x are then large products over all steps at once.
// Right-padded sentences keep their state at steps t >= lengths[b]; their gate gradients
// are zero rows, so the large products need no masking, or (ls_packed) have no rows at all.
#include "../../include/lstm_stack.h"

#include <vector>

#include "common.h"
#include "gemm.h"
#include "kernels.h"
#include "lstm_wave.h"
#include "status.h"

namespace asx {
namespace {

constexpr size_t kAlignL = 256;
size_t upl(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct LsLayout {
  size_t e;
  int64_t TB, BH;
  int64_t x_stride, h_stride, g_stride;   // bytes of one step's operand as fragment tiles
  size_t gates, cs, hE, out, dG;          // [L] (out: [L - 1]) blocks each
  size_t hf, dcs, dbacc, partial, total;
  size_t start, pos, xw, dx_rows;         // packed: rows of the sentences and positions, of the words of x and of its gradient
  bool packed;
  size_t h0_copy;                         // T = 1: h0 and c0 where an output lies on top of them
  size_t xF, zeros, hF[2], oF[2], dGF;    // fragment tiles; [0] value, [1] remainder (bf16 storage)
  std::vector<size_t> Wf_hh, Wf_ih, Wb_hh, Wb_up;   // weights as tiles, per layer
  std::vector<GemmPlan> p_dwi;
  std::vector<size_t> dw_at;               // partial sums of the weight gradients that are not batched, behind `partial`
  GemmPlan p_dwh, p_dx, p_gx;
  bool dw_past;   // the weight gradients that are not batched past the caches
  bool dwh_batched, dwi_batched;   // dW_hh of all layers, dW_ih of all but the first, in one launch
  bool x_apart;   // the input product of layer 0 ahead of the wavefronts
  bool w_rows;    // forward wavefronts read the caller's weight rows
  bool direct;    // and layer 0 his initial state and input
  int group;      // T = 1, backward: wavefronts whose weights are tiles at the same time
};

bool ls_shape_ok(const ls_shape* s) {
  if (!s) return false;
  if (s->T < 1 || s->B < 1 || s->I < 1 || s->H < 1 || s->L < 1 || s->L > 16) return false;
  if (s->dtype != AS_F32 && s->dtype != AS_BF16) return false;
  if (!(s->dropout_p >= 0.f && s->dropout_p < 1.f)) return false;
  if (s->dtype == AS_BF16 && ((s->I % 8) != 0 || (s->H % 8) != 0)) return false;
  if ((int64_t)s->T * s->B > (1 << 24) || s->H > (1 << 16) || s->I > (1 << 16)) return false;
  if ((int64_t)s->T * s->B * 4 * s->H > ((int64_t)1 << 34)) return false;
  return true;
}

// Weights of the backward pass as tiles.  With one step (T = 1) a weight is used by one wavefront alone, so that places for
// a few wavefronts' (32 MiB of them, one wavefront's two at least) do for all layers: they are filled again in between.
// (Four layers of 1024 units, 128 sentences: 62 MiB of workspace where tiles of all weights make it 86.  Places for one
// wavefront alone, 46 MiB: forward and backward with one sentence 242 us, 224 with two.)
int ls_one_step_group(size_t weight) {
  const size_t g = ((size_t)32 << 20) / (2 * weight);
  return g < 1 ? 1 : (g < kLsMaxLayers ? (int)g : kLsMaxLayers);
}

template <typename TE, typename Take> void ls_fwd_tiles(const ls_shape* s, LsLayout& L, Take take) {
  const int T = s->T, I = s->I, H = s->H, NL = s->L;
  const size_t nct = ls_batch_tiles(s->B);
  const int copies = sizeof(TE) == 2 ? 2 : 1;
  L.x_apart = ls_input_apart<TE>(T, I, H, NL);
  L.w_rows = ls_reads_weight_rows<TE>(T, I, H);
  L.direct = L.w_rows && ls_reads_states<TE>(H, s->B);
  L.x_stride = L.x_apart ? 0 : (int64_t)(ls_ksteps<TE>(I) * nct * kLsTile);
  L.h_stride = (int64_t)(ls_ksteps<TE>(H) * nct * kLsTile);
  L.xF = take((size_t)L.x_stride * T);
  L.zeros = take(nct * kLsTile);
  L.h0_copy = take(L.direct ? 2 * (size_t)NL * s->B * H * 4 : 0);
  for (int k = 0; k < copies; ++k) {
    L.hF[k] = take((size_t)L.h_stride * 2 * NL);
    L.oF[k] = take((size_t)L.h_stride * 2 * (NL - 1));
  }
  for (int k = copies; k < 2; ++k) L.hF[k] = L.oF[k] = 0;
  for (int l = 0; l < NL; ++l) {
    const size_t row = L.w_rows ? 0 : ls_gate_tiles(H) * kLsTile;
    L.Wf_hh.push_back(take(ls_ksteps<TE>(H) * row));
    L.Wf_ih.push_back(take(ls_ksteps<TE>(l > 0 ? H : L.x_apart ? 0 : I) * row));
  }
}
template <typename TE, typename Take> void ls_bwd_tiles(const ls_shape* s, LsLayout& L, Take take) {
  const int H = s->H, NL = s->L;
  const size_t gk = 4 * (size_t)ls_gate_stride<TE>(H) / LsGeom<TE>::kKStep, weight = gk * ls_unit_tiles(H) * kLsTile;
  L.g_stride = (int64_t)(gk * ls_batch_tiles(s->B) * kLsTile);
  L.dGF = take((size_t)L.g_stride * 2 * NL);
  L.group = s->T > 1 ? NL : ls_one_step_group(weight);
  auto places = [&](int n) { return take((L.group < n ? L.group : n) * weight); };
  const size_t hh = places(NL), up = places(NL - 1);
  for (int l = 0; l < NL; ++l) {   // wavefront NL - l reads W_hh[l], the one before it W_ih[l + 1]
    L.Wb_hh.push_back(hh + (NL - 1 - l) % L.group * weight);
    L.Wb_up.push_back(l + 1 < NL ? up + (NL - 2 - l) % L.group * weight : 0);
  }
}

LsLayout make_ls_layout(const ls_shape* s) {
  LsLayout L;
  const bool bf = s->dtype == AS_BF16;
  const int T = s->T, B = s->B, I = s->I, H = s->H, NL = s->L;
  L.e = bf ? 2 : 4;
  L.TB = (int64_t)T * B;
  L.BH = (int64_t)B * H;
  const int TB = (int)L.TB;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += upl(bytes, kAlignL);
    return o;
  };
  size_t pb = 0;
  auto mx = [&](size_t v) { if (v > pb) pb = v; };
  // Several layers' weight gradients together fill the compute units with tiles of 256 x 256, whose operands are read half
  // as often as those of 128 x 128: where rounds of the compute units are two thirds full or more.  Four layers of 1024
  // units, 6400 rows: 473 us as seven products, 330 so.  The number of rows has no part in it: from 1 to 65536 of them, 2 to 16
  // layers of 704 to 2048 units, no pass was slower (forward and backward 16 x 1024, one row 955 -> 728 us; backward 3 x 1024,
  // 65536 rows 15.7 -> 15.3 ms, two thirds of a round in 2 x 1216 units, 16384 rows, 3.49 -> 3.32).
  auto batched = [&](int n) {
    const int64_t tiles = (int64_t)((4 * H + 255) / 256) * ((H + 255) / 256) * n, rounds = (tiles + 255) / 256;
    return bf && n > 1 && 3 * tiles >= 2 * 256 * rounds;
  };
  L.dwh_batched = batched(NL);
  L.dwi_batched = batched(NL - 1);
  for (int l = 0; l < NL; ++l) {
    const int Il = l == 0 ? I : H;
    L.p_dwi.push_back(gemm_plan(4 * H, Il, TB, 1, bf, true));
  }
  L.p_dwh = gemm_plan(4 * H, H, TB, 1, bf, true);
  // the others, up to kMaxTogether in a launch, whose partial sums are alive together
  size_t beside = 0;
  auto one = [&](int cols, const GemmPlan& p) {
    if (L.dw_at.size() % kMaxTogether == 0) beside = 0;
    L.dw_at.push_back(beside);
    beside += upl(gemm_partial_bytes(4 * H, cols, 1, p.splits), kAlignL);
    mx(beside);
  };
  size_t dw_bytes = 0;
  for (int l = 0; l < NL; ++l) {
    const int Il = l == 0 ? I : H;
    if (!L.dwh_batched) one(H, L.p_dwh);
    if (!L.dwi_batched || l == 0) one(Il, L.p_dwi[l]);
    dw_bytes += (L.dwh_batched ? 0 : (size_t)16 * H * H) + (L.dwi_batched && l > 0 ? 0 : (size_t)16 * H * Il);
  }
  // From a quarter of the L2s together on; smaller ones are the same either way.  Forward and backward, us, plain / past, alone; with a
  // running sum; with Adam behind it: 256 -> 2 x 256, 30 x 16 (4 MB) 417.9 / 417.7; 431.3 / 431.2; 431.9 / 432.1; 512 -> 512, 32 x 64 (8
  // MB) 507 / 506; 535 / 526; 545.7 / 545.9; 256 -> 2 x 512, 24 x 16 (15 MB) 416.8 / 415.6; 433.7 / 432.9; 460.7 / 462.4; 512 -> 1024, 32
  // x 32 (25 MB) 638 / 613; 656 / 654; 677.5 / 676.3; 512 -> 2 x 768, 20 x 32 (35 MB) 496 / 473; 523.6 / 522.2; 551.7 / 549.9; 512 -> 2 x
  // 1024, 20 x 16 (59 MB) 542 / 516; 580.5 / 576.9; 629 / 632.
  L.dw_past = dw_bytes >= (size_t)8 << 20;
  // The reduction split of the gradient of x is a function of the widths alone: with a split chosen from the row
  // count, a sentence's gradients would depend (in the last fp32 bit) on how many sentences share its batch.
  L.p_dx = gemm_plan(TB, I, 4 * H, 1, bf, false);
  if (bf) {
    const int ktiles = (4 * H + 63) / 64, want = I >= 1024 ? 2 : 4;
    L.p_dx.splits = ktiles / 8 < 1 ? 1 : (ktiles / 8 < want ? ktiles / 8 : want);
    L.p_dx.tile = kTile256;
    if (H <= 256 && I <= 512) L.p_dx = {kTile64, 1};   // few rows or many: 768 x 128 x 512 17.4 -> 6.2 us
  }
  mx(gemm_partial_bytes(TB, I, 1, L.p_dx.splits));
  L.p_gx = gemm_plan(TB, 4 * H, I, 1, bf, false);
  // what the forward pass leaves for the backward pass
  L.gates = take((size_t)NL * TB * 4 * H * 4);
  L.cs = take((size_t)NL * (T + 1) * L.BH * 4);
  L.hE = take((size_t)NL * (T + 1) * L.BH * L.e);
  L.out = take((size_t)(NL - 1) * TB * H * L.e);
  L.packed = bf ? ls_packed<uint16_t>(T, B, I, H, NL) : ls_packed<float>(T, B, I, H, NL);
  L.start = take(L.packed ? (size_t)(B + 1) * 4 : 0);
  // one area for what only the forward and what only the backward pass needs
  const size_t area = off;
  L.hf = take((size_t)NL * L.BH * 4);
  if (bf) ls_fwd_tiles<uint16_t>(s, L, take);
  else ls_fwd_tiles<float>(s, L, take);
  const size_t end = off;
  off = area;
  L.dG = take((size_t)NL * TB * 4 * H * L.e);
  L.dcs = take((size_t)NL * L.BH * 4);
  L.dbacc = take((size_t)NL * ls_batch_tiles(B) * 4 * H * 4);
  L.partial = take(pb);
  L.pos = take(L.packed ? (size_t)TB * 4 : 0);
  L.xw = take(L.packed ? (size_t)TB * I * L.e : 0);
  L.dx_rows = take(L.packed && L.p_dx.splits == 1 ? (size_t)TB * I * 4 : 0);
  if (bf) ls_bwd_tiles<uint16_t>(s, L, take);
  else ls_bwd_tiles<float>(s, L, take);
  if (off < end) off = end;
  L.total = off;
  return L;
}

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

as_status check_ptr_array(const void* const* arr, int n, const char* name) {
  if (!arr) return set_error(AS_ERR_NULL, "%s is NULL", name);
  for (int l = 0; l < n; ++l) {
    if (!arr[l]) return set_error(AS_ERR_NULL, "%s[%d] is NULL", name, l);
    if (!al16(arr[l])) return set_error(AS_ERR_ALIGN, "%s[%d] = %p is not 16-byte aligned", name, l, arr[l]);
  }
  return AS_OK;
}

as_status check_ls(const ls_shape* s, void* ws, size_t ws_bytes, LsLayout* L) {
  if (!s) return set_error(AS_ERR_NULL, "shape is NULL");
  if (s->dtype != AS_F32 && s->dtype != AS_BF16) return set_error(AS_ERR_DTYPE, "unknown dtype %d", s->dtype);
  if (s->dtype == AS_BF16 && s->T >= 1 && s->B >= 1 && s->I >= 1 && s->H >= 1 && ((s->I % 8) != 0 || (s->H % 8) != 0))
    return set_error(AS_ERR_ALIGN, "AS_BF16 needs I %% 8 == 0 and H %% 8 == 0 (I=%d H=%d)", s->I, s->H);
  if (!ls_shape_ok(s))
    return set_error(AS_ERR_SHAPE, "bad shape T=%d B=%d I=%d H=%d L=%d dropout_p=%g", s->T, s->B, s->I, s->H, s->L,
                     (double)s->dropout_p);
  if (!ws) return set_error(AS_ERR_NULL, "workspace is NULL");
  if (!al16(ws)) return set_error(AS_ERR_ALIGN, "workspace %p is not 16-byte aligned", ws);
  *L = make_ls_layout(s);
  if (ws_bytes < L->total) return set_error(AS_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, L->total);
  return AS_OK;
}

#define LS_TRY(expr)                                                                            \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess) return set_error(AS_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

bool ranges_meet(const void* a, int64_t na, const void* b, int64_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}

template <typename TE>
as_status ls_fwd(const ls_shape* s, const LsLayout& L, const char* x, const int32_t* lengths,
                 const void* const* W_ih, const void* const* W_hh, const void* const* b, const float* h0,
                 const float* c0, char* y, float* hT, float* cT, char* w, hipStream_t st) {
  LsFwd f{};
  LsPrepFwd q{};
  f.T = s->T; f.B = s->B; f.I = s->I; f.H = s->H; f.L = s->L;
  if (L.packed) f.words.start = reinterpret_cast<int32_t*>(w + L.start);
  f.x_apart = L.x_apart;
  f.w_rows = L.w_rows;
  for (int l = 0; l < s->L; ++l) {
    q.W_hh[l] = W_hh[l];
    q.W_ih[l] = W_ih[l];
    f.W_hh[l] = f.w_rows ? W_hh[l] : w + L.Wf_hh[l];
    f.W_ih[l] = f.w_rows ? W_ih[l] : w + L.Wf_ih[l];
    f.bias[l] = b[l];
  }
  f.x = x; f.h0 = h0; f.c0 = c0;
  f.xF = w + L.xF; f.zeros = w + L.zeros; f.x_stride = L.x_stride;
  f.hF_hi = w + L.hF[0]; f.hF_lo = w + L.hF[1];
  f.oF_hi = w + L.oF[0]; f.oF_lo = w + L.oF[1];
  f.h_stride = L.h_stride;
  f.gates = reinterpret_cast<float*>(w + L.gates);
  f.cs = reinterpret_cast<float*>(w + L.cs);
  f.hE = w + L.hE; f.out = w + L.out; f.y = y;
  f.hf = hT ? hT : reinterpret_cast<float*>(w + L.hf);
  f.cT = cT;
  f.lengths = lengths;
  // dropout sits between the layers: on what layer l+1 reads, never on the top layer's output
  f.drop_thr = s->dropout_p > 0.f ? (uint32_t)((double)s->dropout_p * 4294967296.0) : 0u;
  f.drop_scale = 1.f / (1.f - s->dropout_p);
  f.drop_seed = s->dropout_seed;
  f.direct = L.direct;
  if (f.direct) {
    // Read by every block of a layer while others of its launch write the outputs: where the caller has an output on top of an
    // input, from a copy.
    const int64_t states = s->L * L.BH * 4, xbytes = L.TB * s->I * (int64_t)sizeof(TE);
    const void* outs[] = {y, hT, cT};
    const int64_t sizes[] = {L.TB * s->H * (int64_t)sizeof(TE), states, states};
    auto overwritten = [&](const void* in, int64_t bytes) {
      bool hit = false;
      for (int k = 0; in && k < 3; ++k) hit = hit || (outs[k] && ranges_meet(in, bytes, outs[k], sizes[k]));
      return hit;
    };
    LsCopy c{};
    auto safe = [&](const void* in, int64_t bytes, char* place) -> const void* {
      if (!overwritten(in, bytes)) return in;
      c.add(in, place, bytes);
      return place;
    };
    f.x = safe(x, xbytes, w + L.xF);
    f.h0 = static_cast<const float*>(safe(h0, states, w + L.h0_copy));
    if (c0 != cT)   // (a cell's state is read and written by the same lane)
      f.c0 = static_cast<const float*>(safe(c0, states, w + L.h0_copy + states));
    if (c.n) LS_TRY(launch_ls_copy(c, st));
  } else {
    LS_TRY(launch_ls_prep_fwd<TE>(f, q, st));
  }
  if (L.x_apart) {   // x W_ih^T + b of layer 0, all steps
    GemmArgs g;
    g.seg(x, s->I, 0, W_ih[0], s->I, 0, s->I);
    g.a_kc = true; g.b_kc = true;
    g.M = (int)L.TB; g.N = 4 * s->H; g.bias = b[0];
    g.C = f.gates; g.ldc = 4 * s->H; g.c_bf16 = false;
    LS_TRY(launch_gemm(g, sizeof(TE) == 2, L.p_gx.tile, st));
  }
  for (int d = 0; d < s->T + s->L - 1; ++d) LS_TRY(launch_ls_wave_fwd<TE>(f, d, st));
  return AS_OK;
}

template <typename TE>
as_status ls_bwd(const ls_shape* s, const LsLayout& L, const char* x, const int32_t* lengths,
                 const void* const* W_ih, const void* const* W_hh, const float* dy, const float* dhT,
                 const float* dcT, char* w, float* dx, float* const* dW_ih, float* const* dW_hh, float* const* db,
                 float* dh0, float* dc0, hipStream_t st) {
  constexpr bool bf = sizeof(TE) == 2;
  const int T = s->T, B = s->B, I = s->I, H = s->H, NL = s->L;
  const int TB = (int)L.TB;
  float* partial = reinterpret_cast<float*>(w + L.partial);
  LsBwd r{};
  LsPrepBwd q{};
  LsBiasOut o{};
  for (int l = 0; l < NL; ++l) {
    r.WT_hh[l] = w + L.Wb_hh[l];
    r.WT_up[l] = w + L.Wb_up[l];
    o.db[l] = db[l];
  }
  r.gates = reinterpret_cast<const float*>(w + L.gates);
  r.cs = reinterpret_cast<const float*>(w + L.cs);
  r.dy = dy; r.dhT = dhT; r.dcT = dcT;
  const int32_t* n_words = nullptr;
  if (L.packed) {
    q.words = r.words = LsWords{reinterpret_cast<int32_t*>(w + L.start), reinterpret_cast<int32_t*>(w + L.pos), w + L.xw};
    q.x = x; q.hE = w + L.hE;
    q.T = T; q.B = B; q.I = I; q.L = NL;
    n_words = r.words.start + B;
  }
  r.dcs = dc0 ? dc0 : reinterpret_cast<float*>(w + L.dcs);
  r.dh0 = dh0;
  r.dG = w + L.dG;
  r.dGF = w + L.dGF; r.g_stride = L.g_stride;
  r.dbacc = reinterpret_cast<float*>(w + L.dbacc);
  r.lengths = lengths;
  r.T = T; r.B = B; r.H = H; r.L = NL;
  r.drop_thr = s->dropout_p > 0.f ? (uint32_t)((double)s->dropout_p * 4294967296.0) : 0u;
  r.drop_scale = 1.f / (1.f - s->dropout_p);
  r.drop_seed = s->dropout_seed;
  q.H = H;
  if (T > 1) {
    for (int l = 0; l < NL; ++l) q.add(W_hh[l], r.WT_hh[l]);
    for (int l = 0; l + 1 < NL; ++l) q.add(W_ih[l + 1], r.WT_up[l]);
    LS_TRY(launch_ls_prep_bwd<TE>(q, st));
  }
  const int waves = T + NL - 1 + (dh0 ? 1 : 0);
  for (int d = 0; d < waves; ++d) {
    if (T == 1 && d > 0 && (d - 1) % L.group == 0) {   // wavefront e: layer NL - 1 - e, and the initial state of NL - e
      q.n = 0;
      for (int e = d; e < d + L.group && e < waves; ++e) {
        if (e < NL) q.add(W_ih[NL - e], r.WT_up[NL - 1 - e]);
        if (dh0) q.add(W_hh[NL - e], r.WT_hh[NL - e]);
      }
      LS_TRY(launch_ls_prep_bwd<TE>(q, st));
    }
    LS_TRY(launch_ls_wave_bwd<TE>(r, d, st));
  }
  const size_t h_first = L.packed ? (size_t)L.BH * L.e : 0;   // packed: behind the initial states
  LS_TRY(launch_ls_bias_reduce(r.dbacc, o, NL, ls_batch_tiles(B), 4 * H, st));
  {
    const char *dG = w + L.dG, *hE = w + L.hE + h_first, *out = w + L.out;
    const int64_t sG = (int64_t)TB * 4 * H;
    auto together = [&](int n, const char* a, const char* b, int64_t sB, float* const* dW) {
      GemmArgs g;
      g.seg(a, 4 * H, sG, b, H, sB, TB);
      g.a_kc = false; g.b_kc = false;
      g.M = 4 * H; g.N = H; g.batch = n;
      g.K_dev = n_words;
      g.C_of = reinterpret_cast<void* const*>(dW); g.ldc = H; g.c_bf16 = false;
      return launch_gemm(g, bf, kTile256, st);
    };
    if (L.dwh_batched) LS_TRY(together(NL, dG, hE, (int64_t)(T + 1) * L.BH, dW_hh));
    if (L.dwi_batched) LS_TRY(together(NL - 1, dG + sG * L.e, out, (int64_t)TB * H, dW_ih + 1));
  }
  GemmArgs g[kMaxTogether];
  GemmTile tiles[kMaxTogether];
  int n = 0, made = 0;
  // dW = sum_t da_t^T (what came in), Il columns
  auto add = [&](const char* dG, const char* in, int Il, float* dW, const GemmPlan& p) {
    g[n] = GemmArgs();
    g[n].seg(dG, 4 * H, 0, in, Il, 0, TB);
    g[n].a_kc = false; g[n].b_kc = false;
    g[n].M = 4 * H; g[n].N = Il;
    g[n].K_dev = n_words;
    g[n].C = dW; g[n].ldc = Il; g[n].c_bf16 = false;
    g[n].past_caches = L.dw_past;
    g[n].splits = p.splits; g[n].partial = partial + L.dw_at[made++] / sizeof(float);
    tiles[n++] = p.tile;
    if (n < kMaxTogether && made < (int)L.dw_at.size()) return hipSuccess;
    const hipError_t e = n > 1 ? launch_gemm_together(g, tiles, n, bf, st) : launch_gemm(g[0], bf, tiles[0], st);
    n = 0;
    return e;
  };
  for (int l = 0; l < NL; ++l) {
    const char* dG = w + L.dG + (size_t)l * TB * 4 * H * L.e;
    const char* hE = w + L.hE + h_first + (size_t)l * (T + 1) * L.BH * L.e;
    const char* xin = l == 0 ? (L.packed ? w + L.xw : x) : w + L.out + (size_t)(l - 1) * TB * H * L.e;
    if (!L.dwh_batched) LS_TRY(add(dG, hE, H, dW_hh[l], L.p_dwh));
    if (!L.dwi_batched || l == 0) LS_TRY(add(dG, xin, l == 0 ? I : H, dW_ih[l], L.p_dwi[l]));
  }
  {  // gradient of x, all steps: da W_ih of the bottom layer (bf16: the gate gradients as rounded)
    GemmArgs g;
    g.seg(w + L.dG, 4 * H, 0, W_ih[0], I, 0, 4 * H);
    g.a_kc = true; g.b_kc = false;
    g.M = TB; g.N = I;
    const bool rows = L.packed && L.p_dx.splits == 1;   // (a split's combine puts the rows at their places)
    g.M_dev = n_words;
    g.row_pos = L.packed && !rows ? r.words.pos : nullptr;
    g.C = rows ? reinterpret_cast<float*>(w + L.dx_rows) : dx; g.ldc = I; g.c_bf16 = false;
    g.splits = L.p_dx.splits; g.partial = partial;
    LS_TRY(launch_gemm(g, bf, L.p_dx.tile, st));
    if (rows) LS_TRY(launch_scatter_rows(r.words.pos, TB, w + L.dx_rows, dx, nullptr, nullptr, (int64_t)I * 4, st));
  }
  return AS_OK;
}
}  // namespace
}  // namespace asx

using namespace asx;

extern "C" {

size_t lstm_stack_workspace_bytes(const ls_shape* shape) {
  if (!ls_shape_ok(shape)) return 0;
  return make_ls_layout(shape).total;
}

as_status lstm_stack_fwd(const ls_shape* s, const void* x, const int32_t* lengths, const void* const* W_ih,
                         const void* const* W_hh, const void* const* b, const float* h0, const float* c0, void* y,
                         float* hT, float* cT, void* workspace, size_t workspace_bytes, void* hip_stream) {
  LsLayout L;
  as_status rc = check_ls(s, workspace, workspace_bytes, &L);
  if (rc != AS_OK) return rc;
  if (!x || !lengths || !y) return set_error(AS_ERR_NULL, "a required pointer is NULL");
  const void* ptrs[] = {x, lengths, y, h0, c0, hT, cT};
  for (const void* p : ptrs)
    if (p && !al16(p)) return set_error(AS_ERR_ALIGN, "pointer %p is not 16-byte aligned", p);
  if ((rc = check_ptr_array(W_ih, s->L, "W_ih")) != AS_OK) return rc;
  if ((rc = check_ptr_array(W_hh, s->L, "W_hh")) != AS_OK) return rc;
  if ((rc = check_ptr_array(b, s->L, "b")) != AS_OK) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  char* w = reinterpret_cast<char*>(workspace);
  if (s->dtype == AS_BF16)
    return ls_fwd<uint16_t>(s, L, reinterpret_cast<const char*>(x), lengths, W_ih, W_hh, b, h0, c0,
                            reinterpret_cast<char*>(y), hT, cT, w, st);
  return ls_fwd<float>(s, L, reinterpret_cast<const char*>(x), lengths, W_ih, W_hh, b, h0, c0,
                       reinterpret_cast<char*>(y), hT, cT, w, st);
}

as_status lstm_stack_bwd(const ls_shape* s, const void* x, const int32_t* lengths, const void* const* W_ih,
                         const void* const* W_hh, const float* dy, const float* dhT, const float* dcT,
                         void* workspace, size_t workspace_bytes, float* dx, float* const* dW_ih,
                         float* const* dW_hh, float* const* db, float* dh0, float* dc0, void* hip_stream) {
  LsLayout L;
  as_status rc = check_ls(s, workspace, workspace_bytes, &L);
  if (rc != AS_OK) return rc;
  if (!x || !lengths || !dy || !dx) return set_error(AS_ERR_NULL, "a required pointer is NULL");
  const void* ptrs[] = {x, lengths, dy, dhT, dcT, dx, dh0, dc0};
  for (const void* p : ptrs)
    if (p && !al16(p)) return set_error(AS_ERR_ALIGN, "pointer %p is not 16-byte aligned", p);
  if ((rc = check_ptr_array(W_ih, s->L, "W_ih")) != AS_OK) return rc;
  if ((rc = check_ptr_array(W_hh, s->L, "W_hh")) != AS_OK) return rc;
  if ((rc = check_ptr_array(reinterpret_cast<const void* const*>(dW_ih), s->L, "dW_ih")) != AS_OK) return rc;
  if ((rc = check_ptr_array(reinterpret_cast<const void* const*>(dW_hh), s->L, "dW_hh")) != AS_OK) return rc;
  if ((rc = check_ptr_array(reinterpret_cast<const void* const*>(db), s->L, "db")) != AS_OK) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  char* w = reinterpret_cast<char*>(workspace);
  if (s->dtype == AS_BF16)
    return ls_bwd<uint16_t>(s, L, reinterpret_cast<const char*>(x), lengths, W_ih, W_hh, dy, dhT, dcT, w, dx, dW_ih,
                            dW_hh, db, dh0, dc0, st);
  return ls_bwd<float>(s, L, reinterpret_cast<const char*>(x), lengths, W_ih, W_hh, dy, dhT, dcT, w, dx, dW_ih, dW_hh,
                       db, dh0, dc0, st);
}

}  // extern "C"
