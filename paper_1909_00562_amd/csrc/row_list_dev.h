// The list of non-pad positions (row compaction), made by one block beside other work that comes before its first reader.
#pragma once
#include "kernels.h"

namespace asx {

constexpr int kRowListSmem = 64 * (int)sizeof(int);

// 4096 targets at a time: a wave's votes for 64 consecutive positions are one of 64 counts, whose prefix sums every wave takes
// for itself.  Fixed order, no atomics.  (A launch of its own with 1024 targets at a time was 5 us of 1920 targets, 10 of 6400.)
template <int THREADS> __device__ __forceinline__ void row_list_block(const RowList& p, int* counts) {
  constexpr int NW = THREADS / 64, PER = 64 / NW;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int base = 0;
  for (int n0 = 0; n0 < p.N; n0 += 4096) {
    bool live[PER];
    int before[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int n = n0 + j * THREADS + tid;
      const int y = p.targets[n < p.N ? n : p.N - 1];
      live[j] = n < p.N && y != p.pad_id && y >= 0 && y < p.V;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const unsigned long long votes = __ballot(live[j]);
      before[j] = __popcll(votes & ((1ull << lane) - 1ull));
      if (lane == 0) counts[j * NW + wave] = __popcll(votes);
    }
    __syncthreads();
    const int own = counts[lane];
    int sum = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int up = __shfl_up(sum, o, 64);
      sum += lane >= o ? up : 0;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int n = n0 + j * THREADS + tid, pos = base + __shfl(sum - own, j * NW + wave, 64) + before[j];
      if (n >= p.N) continue;
      p.row_pos[n] = live[j] ? pos : -1;
      if (live[j]) p.rows[pos] = n;
      if (p.tgt_mask) p.tgt_mask[n] = live[j] ? 1 : 0;
      if (!live[j]) {
        if (p.tok_loss) p.tok_loss[n] = 0.f;
        if (p.argmax) p.argmax[n] = p.pad_id;
      }
    }
    base += __shfl(sum, 63, 64);
    __syncthreads();   // the counts are rewritten by the next slice
  }
  if (tid == 0) *p.n_act = base;
}

}  // namespace asx
