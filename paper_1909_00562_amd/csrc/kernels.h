// Launchers of the row-wise kernels (masked attention softmax, vocabulary
// softmax cross-entropy).  All enqueue on `st` and return the launch status.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace asx {

// Row compaction (rows / n_act below, both null = off): logits, lse and tok_loss_ws hold only the *n_act rows
// whose target is not padding, row r being position rows[r]; N stays the bound the launch is sized for.
// Position n -> row_pos[n] (its compacted row, -1 at padding), the list rows[0 .. *n_act) of positions in
// increasing order, *n_act; optional per-position outputs: tgt_mask everywhere, tok_loss = 0 and
// argmax = pad_id at padding (the statistics kernel fills the other positions).  Made by an extra block of the attention.
// (zero, in the launchers of the attention: a word they clear for a later kernel of the pass, or null)
struct RowList {
  const int32_t* targets;   // null: no list wanted
  int N, V, pad_id;
  int32_t *row_pos, *rows, *n_act;
  uint8_t* tgt_mask;
  float* tok_loss;
  int32_t* argmax;
};

// Eq. 1: alpha[b,t,:] = softmax(score[b,t,:]) over s < clamp(src_len[b],0,S),
// exactly 0 elsewhere.  Writes alpha32 [B,T,S], a copy in the storage type
// alphaE [B,T,ldS] (columns S..ldS-1 zero), if non-null the rounding remainder
// alphaE_lo = alpha - alphaE in the storage type, and, if non-null, attn_mask [B,S].
hipError_t launch_attn_softmax_rows(const float* score, const int32_t* src_len, int B, int T, int S,
                                    float* alpha32, void* alphaE, void* alphaE_lo, int64_t ldS, bool e_bf16,
                                    uint8_t* attn_mask, const RowList& list, int32_t* zero, hipStream_t st);
// Softmax Jacobian: dscore = alpha * (dalpha - sum_s alpha*dalpha), storage type, [B,T,ldS] zero
// padded; dscoreE_lo (optional) receives the rounding remainder.
hipError_t launch_attn_softmax_rows_bwd(const float* alpha32, const float* dalpha, int B, int T, int S,
                                        void* dscoreE, void* dscoreE_lo, int64_t ldS, bool e_bf16,
                                        hipStream_t st);

// Eq. 1-3 fused for the batched path, bf16 storage, S <= 128 (attn_fwd_fused_supported): q_hi / q_lo [T,B,H] (Q = h_dec
// W_a as value and rounding remainder), h_enc [S,B,H] -> alpha32 [B,T,S], alphaE / alphaE_lo [B,T,ldS] (zero padded),
// ctx / ctx_lo [T,B,H], optional attn_mask [B,S].  One workgroup per (sentence, 16 or 32 decoder steps).
bool attn_fwd_fused_supported(int S, int H);
hipError_t launch_attn_fwd_fused(const void* q_hi, const void* q_lo, const void* h_enc, const int32_t* src_len, int B,
                                 int T, int S, int H, float* alpha32, void* alphaE, void* alphaE_lo, int64_t ldS,
                                 void* ctx, void* ctx_lo, uint8_t* attn_mask, const RowList& list, int32_t* zero, hipStream_t st);
// First half of the attention backward pass with the same kernel: dC_hi / dC_lo [T,B,H], alpha32 [B,T,S] (read) ->
// dscoreE / dscoreE_lo [B,T,ldS] (softmax Jacobian, zero padded) and dQ [T,B,H] = dscore . h_enc (value only).
hipError_t launch_attn_bwd_fused(const void* dC_hi, const void* dC_lo, const void* h_enc, const int32_t* src_len,
                                 int B, int T, int S, int H, const float* alpha32, void* dscoreE, void* dscoreE_lo,
                                 int64_t ldS, void* dQ, hipStream_t st);

// dst_x[r] = src_x[rows[r]], r < *n_act; rows of bytes_x bytes (multiples of 4); the second array is optional
hipError_t launch_gather_rows(const int32_t* rows, const int32_t* n_act, int N, const void* src0, void* dst0,
                              int64_t bytes0, const void* src1, void* dst1, int64_t bytes1, hipStream_t st);
// dst_x[n] = src_x[row_pos[n]], zeros where row_pos[n] < 0; all N rows of dst are written; second array optional
hipError_t launch_scatter_rows(const int32_t* row_pos, int N, const void* src0, void* dst0, const void* src1,
                               void* dst1, int64_t bytes, hipStream_t st);

// The same two for fp32 storage.
bool attn_f32_fused_supported(int S, int H);
hipError_t launch_attn_f32_fwd(const float* q, const float* q_lo, const float* h_enc, const int32_t* src_len, int B, int T, int S,
                               int H, float* alpha32, float* alphaE, float* alphaE_lo, int64_t ldS, float* ctx, float* ctx_lo,
                               uint8_t* attn_mask, const RowList& list, int32_t* zero, hipStream_t st);
hipError_t launch_attn_f32_bwd(const float* dC, const float* dC_lo, const float* h_enc, const int32_t* src_len, int B, int T, int S,
                               int H, const float* alpha32, float* dscore, float* dscore_lo, int64_t ldS, float* dQ, hipStream_t st);

// Eq. 5-6 per row n of logits [N,ldV]: lse, loss, argmax, target mask.
hipError_t launch_xent_stats(const void* logits, int64_t ldV, bool e_bf16, int N, int V,
                             const int32_t* targets, int pad_id, float* lse, float* tok_loss_ws,
                             float* tok_loss, int32_t* argmax, uint8_t* tgt_mask, const int32_t* rows,
                             const int32_t* n_act, hipStream_t st);
// The same and the loss from the statistics of the projection's tiles (GemmArgs::row_stats, `parts` per row).  ticket: zero
// when the kernel starts (any more blocks than one).
struct XentFinish {
  const struct TileStat* stats;
  const void* logits;
  int64_t ldV;
  int parts, N, V;
  const int32_t* targets;
  int pad_id;
  float *lse, *tok_loss_ws, *tok_loss;
  int32_t* argmax;
  uint8_t* tgt_mask;
  const int32_t *rows, *n_act;
  float* loss_sum;
  int32_t *n_tok, *ticket;
};
hipError_t launch_xent_finish(const XentFinish& p, hipStream_t st);
// loss_sum = sum(tok_loss_ws) in double, n_tok = number of non-pad targets (= *n_act when given); fixed order.
hipError_t launch_loss_reduce(const float* tok_loss_ws, const int32_t* targets, int N, int V, int pad_id,
                              float* loss_sum, int32_t* n_tok, const int32_t* n_act, hipStream_t st);

// rows of logits handled by one block of the dlogits kernel (also sizes db_partial)
int xent_rows_per_block(int N, int V, bool e_bf16);
// dlogits = g * (exp(logit - lse) - onehot) on non-pad rows, 0 on pad rows and on
// columns V..ldV-1, in place; db_partial[rb][v] = column sums of row block rb.
hipError_t launch_xent_dlogits(void* logits, int64_t ldV, bool e_bf16, int N, int V, const int32_t* targets,
                               int pad_id, const float* lse, float g, float* db_partial, const int32_t* rows,
                               const int32_t* n_act, hipStream_t st);
// db_out[v] = sum_rb db_partial[rb][v], rb < nrb; with n_act (and rb_rows rows per block) only over the row blocks that
// hold compacted rows (the others are not written)
struct DbReduce {
  const float* db_partial;
  int nrb, V;
  float* db_out;
  const int32_t* n_act;
  int rb_rows;
};
hipError_t launch_db_reduce(const DbReduce& d, hipStream_t st);

// One decoder step of attention, fused (Eq. 1-3 with T = 1): kprime [S,B,H] float = W_a h_enc, h_t [B,H],
// h_enc [S,B,H]; writes alpha [B,S] float, ctx [B,H] (+ optional rounding remainder ctx_lo), optional attn_mask.
hipError_t launch_attn_step(const void* h_t, const float* kprime, const void* h_enc, const int32_t* src_len, int B,
                            int S, int H, float* alpha, void* ctx, void* ctx_lo, bool e_bf16, uint8_t* attn_mask,
                            int32_t* zero, hipStream_t st);
// Backward pass of attention for a training step with T = 1, bf16 storage: alpha as saved by the forward pass, dC [B,H] and
// Q = h_dec W_a [B,H] as value and remainder -> dQ [B,H] and d_h_enc [S,B,H] (all of it).
bool attn_one_step_bwd_supported(int T, int S, int H);
hipError_t launch_attn_one_step_bwd(const void* dC_hi, const void* dC_lo, const void* h_enc, const int32_t* src_len,
                                    int B, int S, int H, const float* alpha, const void* q_hi, const void* q_lo, void* dQ,
                                    float* d_h_enc, hipStream_t st);

// Measurement aid: plain streams over `rows` chunks of `row_bytes` bytes (a multiple of 16).  kind 0: read-only with
// the statistics kernel's load pattern, buf2 receives 4 words per row; kind 1: copy buf -> buf2 and kind 2:
// in-place read-modify-write of buf, both with the dlogits kernel's grid and loads in flight.
hipError_t launch_stream_probe(int kind, void* buf, void* buf2, int rows, size_t row_bytes, hipStream_t st);

// Adam, bias corrections passed as inv_bc1 = 1 / (1 - beta1^step), inv_bc2 likewise; wout optional.
hipError_t launch_adam_step(size_t n, const float* grad, float* master, float* m, float* v, void* wout,
                            bool out_bf16, float lr, float beta1, float beta2, float eps, float inv_bc1,
                            float inv_bc2, hipStream_t st);

}  // namespace asx
