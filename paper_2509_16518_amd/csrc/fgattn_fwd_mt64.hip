// Forward-kernel instantiations for the 64-row query tile: d = 64 / 128; dense, one key per
// group, N keys per group.
#include "fgattn_fwd.hpp"
#include "fgattn_launch.hpp"

namespace fg {

static_assert(FwdCfg<64, 128>::NT == (64 <= 32 ? 128 : 64 == 64 ? 64 : 32), "host-side NT table out of date");

template <int D, int OCC>
static int launch_d(const FwdArgs& a, int cus, hipStream_t stream, int* grid_only) {
  static int occ[4][64];
  if (a.indptr == nullptr)
    // (with a raised priority in the gather phase: 2-6% faster in 12 of 14 sizes from 157 to 6144 items, 1% slower in two)
    return launch_variant(fgattn_fwd_kernel<64, D, NMODE_DENSE, OCC, PART_ALL, false, 2, 2, 4, true>, fwd_lds_bytes<64, D, NMODE_DENSE>(), a, cus, stream, grid_only, occ[0]);
  if (a.N == 1)
    return launch_variant(fgattn_fwd_kernel<64, D, NMODE_N1, OCC>, fwd_lds_bytes<64, D, NMODE_N1>(), a, cus, stream, grid_only, occ[1]);
  if (a.N > 0 && a.L % a.N == 0)
    return launch_variant(fgattn_fwd_kernel<64, D, NMODE_GROUPS, OCC>, fwd_lds_bytes<64, D, NMODE_GROUPS>(), a, cus, stream, grid_only, occ[2]);
  return launch_variant(fgattn_fwd_kernel<64, D, NMODE_GROUPS_SHORT, OCC>, fwd_lds_bytes<64, D, NMODE_GROUPS_SHORT>(), a, cus, stream, grid_only, occ[3]);
}

int launch_mt64(const FwdArgs& a, int d, int cus, hipStream_t stream, int* grid_only) {
  // d = 64 fits the 168 registers of three workgroups per compute unit instead of two (dense, 12 heads x 32760 tokens 3.89 ->
  // 3.53 ms, 16 heads x 2635 tokens 54 -> 43 us; lists of 8 keys per group with a short last one, 12 heads x 32764 tokens,
  // 1.71 -> 1.23 ms); that last variant spills one register, which it reloads once per item
  if (d == 64) return launch_d<64, 3>(a, cus, stream, grid_only);
  return launch_d<128, 2>(a, cus, stream, grid_only);
}

}  // namespace fg
