// Column sums of dlogits (db_out) from those of its row blocks: a block of a launch of its own, or beside the products that
// read dlogits.
#pragma once
#include "kernels.h"

namespace asx {

constexpr int kDbColumns = 64;   // columns of a block
constexpr int kDbSmem = 16 * kDbColumns * (int)sizeof(float);

// 64 columns x 16 phases: phase p adds the row blocks p, p + 16, ... of its column, eight loads in flight per thread, and the
// sixteen sums meet in LDS; the order of the additions does not depend on the number of threads.  (Four phases with a load at
// a time took 17 us for 240 row blocks of 16000 columns, 160 of them with rows.)
template <int THREADS> __device__ __forceinline__ void db_reduce_block(const DbReduce& p, int block, float* red) {
  constexpr int PT = 16 * kDbColumns / THREADS;   // phases of a thread
  const int c = threadIdx.x % kDbColumns, phase = threadIdx.x / kDbColumns;
  const int v = block * kDbColumns + c;
  int nrb = p.nrb;
  if (p.n_act) {
    const int used = (*p.n_act + p.rb_rows - 1) / p.rb_rows;
    nrb = used < nrb ? used : nrb;
  }
  float s[PT];
#pragma unroll
  for (int k = 0; k < PT; ++k) s[k] = 0.f;
  if (v < p.V) {
    if constexpr (PT == 1) {
#pragma unroll 8
      for (int r = phase; r < nrb; r += 16) s[0] += p.db_partial[(int64_t)r * p.V + v];
    } else {
#pragma unroll 2
      for (int r0 = phase; r0 < nrb; r0 += 16) {
        float x[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) {
          const int r = r0 + k * (16 / PT);
          x[k] = p.db_partial[(int64_t)(r < nrb ? r : r0) * p.V + v];
        }
#pragma unroll
        for (int k = 0; k < PT; ++k)
          if (r0 + k * (16 / PT) < nrb) s[k] += x[k];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < PT; ++k) red[(phase + k * (16 / PT)) * kDbColumns + c] = s[k];
  __syncthreads();
  if (phase == 0 && v < p.V) {
    float sum = s[0];
#pragma unroll
    for (int q = 1; q < 16; ++q) sum += red[q * kDbColumns + c];
    p.db_out[v] = sum;
  }
}

}  // namespace asx
