// Forward-kernel instantiations for the 128-row query tile: d = 64 / 128; dense, one key per
// group, N keys per group.
#include "fgattn_fwd.hpp"
#include "fgattn_launch.hpp"

namespace fg {

static_assert(FwdCfg<128, 128>::NT == (128 <= 32 ? 128 : 128 == 64 ? 64 : 32), "host-side NT table out of date");

template <int D, int OCC>
static int launch_d(const FwdArgs& a, int cus, hipStream_t stream, int* grid_only) {
  static int occ[5][64];
  // Dense, all items at once: with a raised priority in the gather phase (1 head of 50000 tokens 1.33 -> 1.27 ms, at d = 64 4
  // heads of 16384 308 -> 299 us; 235 to 640 items 0-11% faster).  From a queue without: with it two and six rounds of 16384
  // keys gain 2-4%, six of 32760 lose 1% and at d = 64 1024 items a quarter.
  if (a.indptr == nullptr && a.schedule == SCHED_DIRECT)
    return launch_variant(fgattn_fwd_kernel<128, D, NMODE_DENSE, OCC, PART_ALL, false, 2, 2, 4, true>,
                          fwd_lds_bytes<128, D, NMODE_DENSE>(), a, cus, stream, grid_only, occ[4]);
  if (a.indptr == nullptr)
    return launch_variant(fgattn_fwd_kernel<128, D, NMODE_DENSE, OCC>, fwd_lds_bytes<128, D, NMODE_DENSE>(), a, cus, stream, grid_only, occ[0]);
  if (a.N == 1)
    return launch_variant(fgattn_fwd_kernel<128, D, NMODE_N1, OCC>, fwd_lds_bytes<128, D, NMODE_N1>(), a, cus, stream, grid_only, occ[1]);
  if (a.N > 0 && a.L % a.N == 0)
    return launch_variant(fgattn_fwd_kernel<128, D, NMODE_GROUPS, OCC>, fwd_lds_bytes<128, D, NMODE_GROUPS>(), a, cus, stream, grid_only, occ[2]);
  return launch_variant(fgattn_fwd_kernel<128, D, NMODE_GROUPS_SHORT, OCC>, fwd_lds_bytes<128, D, NMODE_GROUPS_SHORT>(), a, cus, stream, grid_only, occ[3]);
}

int launch_mt128(const FwdArgs& a, int d, int cus, hipStream_t stream, int* grid_only) {
  // d = 64 fits 168 registers, a budget of three waves per SIMD: three workgroups per compute unit (12 heads x 32760 tokens at
  // 128x8 1.108 -> 1.077 ms).  The dense kernel needs 157 and runs three with either budget, at the same speed.
  if (d == 64) return launch_d<64, 3>(a, cus, stream, grid_only);
  return launch_d<128, 2>(a, cus, stream, grid_only);
}

}  // namespace fg
