// HIP kernels of one pruning step on the stored entries of W_F (Section 4.2, Eq. 8 and Eq. 9):
//   w' = w - eta (dL/dw + lambda sign w)                (SGD step on L + lambda |w|_1, Eq. 9 with Eq. 7)
//   T(w') = 0 if |w'| (|dL/dw| + beta) < eps, else w'   (Eq. 8, gradient taken at the point of the step)
// and the new per-position CSR without the entries T zeroed.  Arithmetic in fp32, one rounding per
// operation: g + lambda*sign(w), one fused multiply-add for w', |g| + beta, the product with |w'|.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "swconv_rows.hpp"

namespace swconv {

__device__ __forceinline__ float pruned_value(float w, float g, float eta, float lambda, float eps, float beta,
                                              bool* drop) {
  const float sgn = w > 0.0f ? 1.0f : (w < 0.0f ? -1.0f : 0.0f);
  const float step = __fadd_rn(g, __fmul_rn(lambda, sgn));
  const float wn = __fmaf_rn(-eta, step, w);
  *drop = __fmul_rn(fabsf(wn), __fadd_rn(fabsf(g), beta)) < eps;
  return wn;
}

// The two entry-wise kernels give a row 16 lanes (rows of the pruned layers have 5 to 40 entries): the lanes of a
// wave then read whole lines of the CSR arrays, and a row of 25 entries is two rounds of independent loads.
// With one thread per row every load of a wave touched 64 lines and a row was a chain of 25 loads; with the
// serial scan, the step took 77 us on the 13 824 rows and 354 k entries of the 256 -> 384, F(4x4,3x3) layer; none of
// its launches moves more than 7 MB.

// The lanes of the calling lane's row that say `keep`, as a 16-bit mask.
__device__ __forceinline__ unsigned kept_in_row(bool keep) {
  return (unsigned)(__ballot(keep) >> (threadIdx.x & 48u)) & 0xffffu;
}

// Updates the row's values (0 where dropped) and counts what it keeps; the count goes to
// rowptr_out[row + 1] (rowptr_out[0] = 0).  LOCAL: not the count but -1 - (the count of the workgroup's rows up to and
// including this one), one turn per workgroup (rows <= kPruneLocalRows): what prune_compact_kernel<true> starts from.
template <bool LOCAL>
__global__ __launch_bounds__(256) void prune_update_kernel(int64_t rows, const int32_t* __restrict__ rowptr,
                                                           const float* __restrict__ vals,
                                                           const float* __restrict__ grad, float eta, float lambda,
                                                           float eps, float beta, float* __restrict__ updated,
                                                           int32_t* __restrict__ rowptr_out) {
  __shared__ int32_t counts[kPruneRows];
  const int lane = threadIdx.x % kPruneRowLanes;
  if (blockIdx.x == 0 && threadIdx.x == 0) rowptr_out[0] = 0;
  for (int64_t row0 = (int64_t)blockIdx.x * kPruneRows; row0 < rows; row0 += (int64_t)gridDim.x * kPruneRows) {
    const int64_t row = row0 + threadIdx.x / kPruneRowLanes;
    const int32_t q0 = row < rows ? rowptr[row] : 0, q1 = row < rows ? rowptr[row + 1] : 0;
    int kept = 0;
    for_row_chunks<kPruneRowLanes>(q0, q1, [&](uint32_t i, uint32_t n) {  // the 16 lanes of a row stay together
      bool drop = true;
      if (i + lane < n) {
        const size_t q = (size_t)q0 + i + lane;
        const float wn = pruned_value(vals[q], grad[q], eta, lambda, eps, beta, &drop);
        updated[q] = drop ? 0.0f : wn;
      }
      kept += __popc(kept_in_row(!drop));
    });
    if constexpr (LOCAL) {
      if (lane == 0) counts[threadIdx.x / kPruneRowLanes] = kept;
      __syncthreads();
      if (threadIdx.x < kPruneRows) {
        int32_t sum = 0;
        for (int i = 0; i <= (int)threadIdx.x; ++i) sum += counts[i];
        if (row0 + threadIdx.x < rows) rowptr_out[row0 + threadIdx.x + 1] = -1 - sum;
      }
    } else if (row < rows && lane == 0) {
      rowptr_out[row + 1] = kept;
    }
  }
}

// Inclusive scan of rowptr_out[1 .. rows] in place: one workgroup of 1024 threads takes 16 x 1024 values at a
// time, all loads in flight at once, scans every run of 64 in its wave and the 256 runs' totals in LDS.  (A
// device-wide scan would need storage between its launches that the entry point does not have.)  For more than
// kPruneLocalRows rows only: below, prune_compact_kernel<true> does without.
__global__ __launch_bounds__(1024) void prune_scan_kernel(int64_t rows, int32_t* __restrict__ rowptr_out) {
  constexpr int U = 16, W = 1024 / 64;
  __shared__ int32_t run[U * W];  // run j * W + w: the values of wave w in the j-th 1024
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t carry = 0;
  for (int64_t base = 0; base < rows; base += U * 1024) {
    int32_t v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int64_t i = base + j * 1024 + threadIdx.x;
      v[j] = i < rows ? rowptr_out[i + 1] : 0;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const int32_t up = __shfl_up(v[j], d);
        if (lane >= d) v[j] += up;
      }
    __syncthreads();  // every thread has read the totals of the round before
    if (lane == 63)
#pragma unroll
      for (int j = 0; j < U; ++j) run[j * W + wave] = v[j];
    __syncthreads();
    if (wave == 0) {  // 256 totals: four consecutive ones per lane
      int32_t r[4], sum = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) sum += r[k] = run[lane * 4 + k];
      int32_t incl = sum;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int32_t up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
      }
      int32_t at = incl - sum;
#pragma unroll
      for (int k = 0; k < 4; ++k) run[lane * 4 + k] = at += r[k];  // inclusive
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int64_t i = base + j * 1024 + threadIdx.x;
      const int before = j * W + wave - 1;
      if (i < rows) rowptr_out[i + 1] = carry + v[j] + (before >= 0 ? run[before] : 0);
    }
    carry += run[U * W - 1];
  }
}

// Copies the kept entries (in their order) to the compacted arrays.  An entry is kept exactly when
// prune_update_kernel kept it: the decision is taken again from the same inputs.
// LOCAL, without a scan between the two launches: a workgroup adds up what the workgroups before it keep, from the last
// entry of each in rowptr_out, and puts its own entries right.  Others may have done so already: a non-negative entry is
// a row pointer, the sum up to there, a negative one -1 - the workgroup's own sum.  Either says the same, so nobody
// waits for anybody; the sum starts behind the last of the workgroups whose entry is a row pointer.  13 824 rows:
// 864 workgroups read 432 entries on average (three launches of 4.0 + 7.2 + 4.3 us -> two of 4.0 + 6.2).
template <bool LOCAL>
__global__ __launch_bounds__(256) void prune_compact_kernel(int64_t rows, const int32_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ colidx,
                                                            const float* __restrict__ vals,
                                                            const float* __restrict__ grad, float eta, float lambda,
                                                            float eps, float beta,
                                                            int32_t* __restrict__ rowptr_out,
                                                            int32_t* __restrict__ colidx_out,
                                                            float* __restrict__ vals_out) {
  const int lane = threadIdx.x % kPruneRowLanes;
  __shared__ int32_t first_out[kPruneRows + 1];  // LOCAL: row pointers of the workgroup's rows and of the next one
  if constexpr (LOCAL) {
    __shared__ int32_t part[kPruneThreads / 64], last[kPruneThreads / 64];
    const int64_t row0 = (int64_t)blockIdx.x * kPruneRows;
    const int groups = (int)blockIdx.x;  // before this one, all of kPruneRows rows
    // the last group whose entry is a row pointer, and the sums of the groups behind it
    int done = -1;
    int32_t v[kPruneLocalTurns];
#pragma unroll
    for (int u = 0; u < kPruneLocalTurns; ++u) {
      const int g = u * kPruneThreads + (int)threadIdx.x;
      v[u] = g < groups ? __hip_atomic_load(rowptr_out + (int64_t)(g + 1) * kPruneRows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : -1;
      if (v[u] >= 0) done = g;
    }
    for (int d = 32; d > 0; d >>= 1) done = max(done, __shfl_xor(done, d));
    if ((threadIdx.x & 63) == 0) last[threadIdx.x >> 6] = done;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kPruneThreads / 64; ++w) done = max(done, last[w]);
    int32_t sum = 0;
#pragma unroll
    for (int u = 0; u < kPruneLocalTurns; ++u) {
      const int g = u * kPruneThreads + (int)threadIdx.x;
      if (g == done) sum += v[u];
      if (g > done && g < groups) sum += -1 - v[u];
    }
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    int32_t before = 0;
#pragma unroll
    for (int w = 0; w < kPruneThreads / 64; ++w) before += part[w];
    if (threadIdx.x == 0) first_out[0] = before;
    if (threadIdx.x < kPruneRows && row0 + threadIdx.x < rows) {
      const int32_t end = before + (-1 - rowptr_out[row0 + threadIdx.x + 1]);
      first_out[threadIdx.x + 1] = end;
      __hip_atomic_store(rowptr_out + row0 + threadIdx.x + 1, end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
  for (int64_t row0 = (int64_t)blockIdx.x * kPruneRows; row0 < rows; row0 += (int64_t)gridDim.x * kPruneRows) {
    const int64_t row = row0 + threadIdx.x / kPruneRowLanes;
    const int32_t q0 = row < rows ? rowptr[row] : 0, q1 = row < rows ? rowptr[row + 1] : 0;
    int32_t dst = row >= rows ? 0 : LOCAL ? first_out[threadIdx.x / kPruneRowLanes] : rowptr_out[row];
    for_row_chunks<kPruneRowLanes>(q0, q1, [&](uint32_t i, uint32_t n) {
      bool drop = true;
      float wn = 0.0f;
      int32_t c = 0;
      if (i + lane < n) {
        const size_t q = (size_t)q0 + i + lane;
        c = colidx[q];
        wn = pruned_value(vals[q], grad[q], eta, lambda, eps, beta, &drop);
      }
      const unsigned kept = kept_in_row(!drop);
      if (!drop) {
        const int32_t at = dst + __popc(kept & ((1u << lane) - 1u));
        colidx_out[at] = c;
        vals_out[at] = wn;
      }
      dst += __popc(kept);
    });
  }
}

// Fine-tuning with the sparsity pattern fixed (Section 4.3): only the values of W_F change.  Every
// (offset, weight) pair of a packed stream takes its weight from the caller's CSR value array
// through the pair's index into that array; padding pairs (index -1) keep +0.0f.
// All packed copies of W_F in one launch: small layers' take less time than a launch does (48 -> 128 channels, two
// streams of 64 positions: 2.8 us each, 3.2 together; 384 -> 384: 5.7 each, 8.7).
constexpr int kRefreshStreams = 3;
struct RefreshStreams {
  uint32_t* pairs[kRefreshStreams];
  const int32_t* index[kRefreshStreams];
  uint32_t n_pairs[kRefreshStreams];
  uint32_t first_block[kRefreshStreams + 1];  // of 256 pairs; a stream that is not there has none
};
__global__ __launch_bounds__(256) void refresh_values_kernel(RefreshStreams s, const float* __restrict__ vals) {
  const int i = blockIdx.x < s.first_block[1] ? 0 : blockIdx.x < s.first_block[2] ? 1 : 2;
  const uint32_t e = (blockIdx.x - s.first_block[i]) * 256u + threadIdx.x;
  if (e >= s.n_pairs[i]) return;
  const int32_t q = s.index[i][e];
  if (q >= 0) s.pairs[i][2 * (size_t)e + 1] = __float_as_uint(vals[q]);
}

}  // namespace swconv
