// Row counts -> row pointers, shared by the mask and the grouping kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fgscan {

constexpr int kScanThreads = 1024;
constexpr int kScanSteps = 8;   // counts per thread and pass

// indptr[0] = 0, indptr[r + 1] = count[0] + .. + count[r].  One workgroup; a count is at most 2^24.  Bound: latency (the
// rows are a few tens of thousands at most).  A wave takes 512 consecutive counts of a pass, 64 at a time, so that loads and
// stores are coalesced; its eight prefixes over the lanes are independent of each other (64 counts fit 32 bits) and one
// barrier per pass passes the waves' totals on.  6144 rows 14 -> 5 us, 22296 rows 47 -> 12 us against a
// pass of 1024 counts with a twenty-barrier prefix in LDS.
static __global__ void __launch_bounds__(kScanThreads) row_pointers_kernel(const unsigned* count, int64_t rows, int64_t* indptr) {
  constexpr int WAVES = kScanThreads / 64;
  __shared__ unsigned long long wave_total[2][WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  unsigned long long carry = 0;   // (the same in all threads)
  if (tid == 0) indptr[0] = 0;
  int par = 0;
  for (int64_t base = 0; base < rows; base += kScanThreads * kScanSteps, par ^= 1) {
    const int64_t r0 = base + wv * (64 * kScanSteps) + lane;
    unsigned incl[kScanSteps];
#pragma unroll
    for (int s = 0; s < kScanSteps; s++) incl[s] = r0 + 64 * s < rows ? count[r0 + 64 * s] : 0u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1)
#pragma unroll
      for (int s = 0; s < kScanSteps; s++) {
        const unsigned up = __shfl_up(incl[s], off);
        incl[s] += lane >= off ? up : 0u;
      }
    unsigned long long before[kScanSteps], total = 0;   // counts of this wave's earlier steps; of all its steps
#pragma unroll
    for (int s = 0; s < kScanSteps; s++) {
      before[s] = total;
      total += (unsigned)__builtin_amdgcn_readlane((int)incl[s], 63);
    }
    if (lane == 0) wave_total[par][wv] = total;
    __syncthreads();   // (the other half of wave_total is written in the next pass, so one barrier per pass is enough)
    unsigned long long first = carry;
    for (int w = 0; w < WAVES; w++) {
      const unsigned long long t = wave_total[par][w];
      first += w < wv ? t : 0ull;
      carry += t;
    }
#pragma unroll
    for (int s = 0; s < kScanSteps; s++)
      if (r0 + 64 * s < rows) indptr[r0 + 64 * s + 1] = (int64_t)(first + before[s] + incl[s]);
  }
}

inline void launch_row_pointers(const unsigned* count, int64_t rows, int64_t* indptr, hipStream_t stream) {
  hipLaunchKernelGGL(row_pointers_kernel, dim3(1), dim3(kScanThreads), 0, stream, count, rows, indptr);
}

}  // namespace fgscan
