// Row compaction for the vocabulary part of the path (Eq. 5-6 and its backward).
// A target position that is padding contributes nothing to the loss or to any
// gradient, so the three products over the vocabulary and the two cross-entropy
// passes need only the rows n = t*B + b whose target is a word.  The list of them is made beside the attention of the forward pass
// (row_list_dev.h), on the device: nothing is copied to the host and the stream is never synchronised.  The products write the
// rows of h_c, of the saved tanh derivative and of dz to their places themselves; the 256 x 256 kernels do not, for them these
// kernels gather the rows into a dense [n_act, H] block and scatter the rows of dz back to their time-major places with
// zeros at the padding rows.
#include "common.h"
#include "kernels.h"

namespace asx {

// bytes of one row are a multiple of 4; 16-byte vectors when they are a multiple of 16 (row starts are then aligned)
__device__ __forceinline__ void copy_row(const unsigned char* __restrict__ src, unsigned char* __restrict__ dst,
                                         int64_t bytes, int tid, int nthreads) {
  if ((bytes & 15) == 0) {
    for (int64_t i = (int64_t)tid * 16; i < bytes; i += (int64_t)nthreads * 16)
      *reinterpret_cast<uint4*>(dst + i) = *reinterpret_cast<const uint4*>(src + i);
  } else {
    for (int64_t i = (int64_t)tid * 4; i < bytes; i += (int64_t)nthreads * 4)
      *reinterpret_cast<uint32_t*>(dst + i) = *reinterpret_cast<const uint32_t*>(src + i);
  }
}
__device__ __forceinline__ void zero_row(unsigned char* __restrict__ dst, int64_t bytes, int tid, int nthreads) {
  if ((bytes & 15) == 0) {
    for (int64_t i = (int64_t)tid * 16; i < bytes; i += (int64_t)nthreads * 16)
      *reinterpret_cast<uint4*>(dst + i) = make_uint4(0, 0, 0, 0);
  } else {
    for (int64_t i = (int64_t)tid * 4; i < bytes; i += (int64_t)nthreads * 4)
      *reinterpret_cast<uint32_t*>(dst + i) = 0u;
  }
}

// dst_x[r] = src_x[rows[r]] for r < *n_act, two arrays per launch (row sizes in bytes; src1 may be null)
__global__ __launch_bounds__(256) void gather_rows_kernel(const int32_t* __restrict__ rows,
                                                         const int32_t* __restrict__ n_act,
                                                         const unsigned char* __restrict__ src0,
                                                         unsigned char* __restrict__ dst0, int64_t bytes0,
                                                         const unsigned char* __restrict__ src1,
                                                         unsigned char* __restrict__ dst1, int64_t bytes1) {
  const int r = blockIdx.x;
  if (r >= *n_act) return;
  const int64_t n = rows[r];
  copy_row(src0 + n * bytes0, dst0 + (int64_t)r * bytes0, bytes0, threadIdx.x, 256);
  if (src1) copy_row(src1 + n * bytes1, dst1 + (int64_t)r * bytes1, bytes1, threadIdx.x, 256);
}

// dst_x[n] = src_x[row_pos[n]] where row_pos[n] >= 0, else zeros; every row of dst is written
__global__ __launch_bounds__(256) void scatter_rows_kernel(const int32_t* __restrict__ row_pos,
                                                          const unsigned char* __restrict__ src0,
                                                          unsigned char* __restrict__ dst0,
                                                          const unsigned char* __restrict__ src1,
                                                          unsigned char* __restrict__ dst1, int64_t bytes) {
  const int64_t n = blockIdx.x;
  const int64_t r = row_pos[n];
  if (r >= 0) {
    copy_row(src0 + r * bytes, dst0 + n * bytes, bytes, threadIdx.x, 256);
    if (src1) copy_row(src1 + r * bytes, dst1 + n * bytes, bytes, threadIdx.x, 256);
  } else {
    zero_row(dst0 + n * bytes, bytes, threadIdx.x, 256);
    if (src1) zero_row(dst1 + n * bytes, bytes, threadIdx.x, 256);
  }
}

hipError_t launch_gather_rows(const int32_t* rows, const int32_t* n_act, int N, const void* src0, void* dst0,
                              int64_t bytes0, const void* src1, void* dst1, int64_t bytes1, hipStream_t st) {
  if ((bytes0 & 3) || (bytes1 & 3)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_rows_kernel, dim3(N), dim3(256), 0, st, rows, n_act,
                     reinterpret_cast<const unsigned char*>(src0), reinterpret_cast<unsigned char*>(dst0), bytes0,
                     reinterpret_cast<const unsigned char*>(src1), reinterpret_cast<unsigned char*>(dst1), bytes1);
  return hipGetLastError();
}

hipError_t launch_scatter_rows(const int32_t* row_pos, int N, const void* src0, void* dst0, const void* src1,
                               void* dst1, int64_t bytes, hipStream_t st) {
  if (bytes & 3) return hipErrorInvalidValue;
  hipLaunchKernelGGL(scatter_rows_kernel, dim3(N), dim3(256), 0, st, row_pos,
                     reinterpret_cast<const unsigned char*>(src0), reinterpret_cast<unsigned char*>(dst0),
                     reinterpret_cast<const unsigned char*>(src1), reinterpret_cast<unsigned char*>(dst1), bytes);
  return hipGetLastError();
}

}  // namespace asx
