// psl_kern.h -- host-side launchers of libpsl's kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "psl_dev.h"

namespace psl {

// ----- primitives.hip ------------------------------------------------------
// Exclusive prefix sum of in[0..n) into out (in == out allowed); the total
// is written to *total (device pointer) when total != nullptr. ws must hold
// scan_ws_ints(n) ints.
size_t scan_ws_ints(int64_t n);
void scan_excl(const int32_t* in, int32_t* out, int64_t n, int32_t* total, int32_t* ws, hipStream_t s);

#define RX_TILE 2048  // keys a workgroup counts and moves

// One stable counting-sort pass by the digit (key >> shift) & (2^bits - 1),
// bits <= 8. vals_in == nullptr means value = index. ws: radix_ws_ints(n).
size_t radix_ws_ints(int64_t n);
void radix_pass(const uint32_t* keys_in, const int32_t* vals_in, uint32_t* keys_out, int32_t* vals_out,
                int64_t n, int shift, int bits, int32_t* ws, hipStream_t s);

// The same pass moving a payload of a row index and a value with each key;
// rows_in == nullptr takes row rowid1[p + 1] for item p. Buffers must not
// alias. ws: radix_ws_ints(n); counted: it holds the tiles' counts of the
// pass's digits already (count of digit d in tile t at d * tiles + t).
void radix_pass_payload(const uint32_t* keys_in, const int32_t* rows_in, const int32_t* rowid1,
                        const double* vals_in, uint32_t* keys_out, int32_t* rows_out, double* vals_out, int64_t n,
                        int shift, int bits, bool counted, int32_t* ws, hipStream_t s);

// out[i] = v (32-bit words)
void fill_i32(int32_t* out, int32_t v, int64_t n, hipStream_t s);

#define PW_TILE 2048

// Sum of one aligned tile x[0..2048) (elements at or beyond lim read as 0) by
// the whole block: eight contiguous leaves per thread (tree of 8), a butterfly
// over the wave (tree of 64 such groups), then the four wave sums as
// (w0 + w1) + (w2 + w3). Every thread returns the sum.
__device__ __forceinline__ double tile_sum(const double* x, int64_t lim) {
  __shared__ double ws[PSL_BLOCK / PSL_WAVE];
  int64_t base = (int64_t)threadIdx.x * 8;
  double v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = base + k < lim ? x[base + k] : 0.0;
  double s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
  s = group_sum<PSL_WAVE>(s);
  if (lane_id() == 0) ws[threadIdx.x >> 6] = s;
  __syncthreads();
  double t = (ws[0] + ws[1]) + (ws[2] + ws[3]);
  __syncthreads();
  return t;
}

// Canonical pairwise tree sum of x[0..n) into *out (device), ws: pairwise_ws_doubles(n).
size_t pairwise_ws_doubles(int64_t n);
void pairwise_sum(const double* x, int64_t n, double* out, double* ws, hipStream_t s);

// out[k] = +0-canonical (off[k] + canonical pairwise sum of x[seg[k]..seg[k+1]))
// for k < K; the tree of every segment starts at the segment's first element.
// seg is given on the device and on the host; segments of more than
// 2048 * 2048 elements are summed by pairwise_sum (ws: pairwise_ws_doubles + 1).
void segmented_pairwise_sum(const double* x, const int32_t* seg_dev, const int32_t* seg_host, int K,
                            const double* off, double* out, double* ws, hipStream_t s);

}  // namespace psl
