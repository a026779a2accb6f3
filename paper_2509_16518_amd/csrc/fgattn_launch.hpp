// Host-side launcher template: occupancy-sized persistent grid, opt-in to large dynamic LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

#include "fgattn.h"
#include "fgattn_args.hpp"

namespace fg {

// Workgroups of `lds` bytes that a compute unit holds by its LDS.  It is given out in pieces of 1280 bytes, which the runtime's
// occupancy call does not round up to: of 32768 bytes it promises five, four are resident; of 16384 ten, nine are.  A
// workgroup of the grid that is not resident keeps the item it begins with from everybody else until another one exits
// (three heads of 16384 tokens at 32x32 on 1280 workgroups, of which 1024 were resident, 415 us, on 1024 323; 12 heads of
// 32760 tokens at 32x32 3.81 -> 3.38 ms).
inline int resident_by_lds(int lds) {
  constexpr int kLdsBytes = 160 * 1024, kLdsPiece = 1280;
  return kLdsBytes / ((lds + kLdsPiece - 1) / kLdsPiece * kLdsPiece);
}

template <typename Kernel>
int launch_variant(Kernel kernel, int lds_bytes, const FwdArgs& a, int cus, hipStream_t stream, int* grid_only,
                   int* occ_cache, int wgs_per_cu_cap = 0, int threads = 256) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return FGATTN_E_DEVICE;
  static std::mutex cache_mutex;   // one per kernel variant: first calls from several host threads take turns
  std::unique_lock<std::mutex> lock(cache_mutex);
  if (occ_cache[dev] == 0) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            lds_bytes) != hipSuccess)
      return FGATTN_E_DEVICE;
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, threads, lds_bytes) != hipSuccess || occ < 1)
      return FGATTN_E_DEVICE;
    const int by_lds = resident_by_lds(lds_bytes);
    occ_cache[dev] = occ < by_lds ? occ : by_lds;
  }
  long long want = (long long)cus * (wgs_per_cu_cap > 0 && wgs_per_cu_cap < occ_cache[dev] ? wgs_per_cu_cap : occ_cache[dev]);
  lock.unlock();
  int grid = (int)(a.n_items < want || a.schedule == SCHED_DIRECT ? a.n_items : want);
  if (grid < 1) grid = 1;
  if (grid_only) {
    *grid_only = grid;
    return FGATTN_OK;
  }
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds_bytes, stream, a);
  return hipGetLastError() == hipSuccess ? FGATTN_OK : FGATTN_E_DEVICE;
}

}  // namespace fg
