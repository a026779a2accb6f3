// Selection steps that one wave takes by itself, without barriers: included by fgmask.hip.
#pragma once

namespace fgm {

// LDS operations of a wave complete in order; this keeps the compiler from moving them past each other
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// `x` of another lane, by the wave's own data paths (no LDS): shifts within rows of 16 lanes, then the last lane of a row
// into the next row(s).  Lanes without a source get `none`.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned from_lane(unsigned x, unsigned none) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)none, (int)x, CTRL, ROWS, 0xf, false);
}
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

// inclusive prefix sum over the lanes
__device__ __forceinline__ unsigned lane_prefix(unsigned x) {
  x += from_lane<kRowShr1, 0xf>(x, 0u);
  x += from_lane<kRowShr2, 0xf>(x, 0u);
  x += from_lane<kRowShr4, 0xf>(x, 0u);
  x += from_lane<kRowShr8, 0xf>(x, 0u);
  x += from_lane<kRowBcast15, 0xa>(x, 0u);
  x += from_lane<kRowBcast31, 0xc>(x, 0u);
  return x;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long add_lane(unsigned long long x) {
  return x + (((unsigned long long)from_lane<CTRL, ROWS>((unsigned)(x >> 32), 0u) << 32) | from_lane<CTRL, ROWS>((unsigned)x, 0u));
}
__device__ __forceinline__ unsigned long long lane_prefix(unsigned long long x) {
  x = add_lane<kRowShr1, 0xf>(x);
  x = add_lane<kRowShr2, 0xf>(x);
  x = add_lane<kRowShr4, 0xf>(x);
  x = add_lane<kRowShr8, 0xf>(x);
  x = add_lane<kRowBcast15, 0xa>(x);
  return add_lane<kRowBcast31, 0xc>(x);
}
// largest value of the lanes (0 is the least)
__device__ __forceinline__ unsigned lane_max(unsigned x) {
  x = max(x, from_lane<kRowShr1, 0xf>(x, 0u));
  x = max(x, from_lane<kRowShr2, 0xf>(x, 0u));
  x = max(x, from_lane<kRowShr4, 0xf>(x, 0u));
  x = max(x, from_lane<kRowShr8, 0xf>(x, 0u));
  x = max(x, from_lane<kRowBcast15, 0xa>(x, 0u));
  x = max(x, from_lane<kRowBcast31, 0xc>(x, 0u));
  return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ unsigned long long lane_max(unsigned long long x) {
  const unsigned hi = lane_max((unsigned)(x >> 32));
  return ((unsigned long long)hi << 32) | lane_max((unsigned)(x >> 32) == hi ? (unsigned)x : 0u);
}
__device__ __forceinline__ unsigned long long of_lane(unsigned long long x, int lane) {   // (the lane's number is the same in all)
  return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), lane) << 32) |
         (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, lane);
}
// number of set bits of `lanes` below this lane
__device__ __forceinline__ unsigned lanes_below(uint64_t lanes) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)lanes, 0u));
}

// Mass of all BINS bins and, with `target_of(mass)` and the mass `before` them, the bin in which the running mass reaches that
// target; `before` becomes the mass before that bin.  Every lane reads BINS / 64 consecutive bins, which lie STRIDE words
// apart.  The last bin if the masses fall short.
template <int BINS, int STRIDE = 1, typename TargetOf>
__device__ __forceinline__ int crossing_bin(const unsigned long long* mass, unsigned long long& before, TargetOf&& target_of) {
  constexpr int PER = BINS / 64;
  const int lane = threadIdx.x & 63;
  unsigned long long own[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; i++) sum += own[i] = mass[(lane * PER + i) * STRIDE];
  const unsigned long long incl = lane_prefix(sum);
  const unsigned long long target = target_of(of_lane(incl, 63));
  unsigned long long run = before + incl - sum;
  const uint64_t reach = __builtin_amdgcn_ballot_w64(before + incl >= target);
  const int owner = reach ? __ffsll((unsigned long long)reach) - 1 : 63;
  int bin = PER - 1;
#pragma unroll
  for (int i = 0; i < PER - 1; i++)
    if (bin == PER - 1) {
      if (run + own[i] >= target) bin = i;
      else run += own[i];
    }
  before = of_lane(run, owner);
  return __builtin_amdgcn_readlane(lane * PER + bin, owner);
}

// The cut among the n <= 64 rank keys in cand[0 .. n), n > 0: ranked by counting (they are distinct), then the first at which the
// running mass, from `before` on, reaches the target; the last if it falls short.  `mass` takes 64 words of scratch.
__device__ __forceinline__ unsigned long long cut_of_few(unsigned long long* cand, int n, unsigned long long* mass,
                                                         unsigned long long before, unsigned long long target, float rmax) {
  const int lane = threadIdx.x & 63;
  const unsigned long long key = lane < n ? cand[lane] : 0ull;
  int rank = 0;
  for (int j = 0; j < n; j++) rank += of_lane(key, j) > key ? 1 : 0;
  wave_order();
  if (lane < n) {
    mass[rank] = weight_of(from_ordered((unsigned)(key >> 32)), rmax);
    cand[rank] = key;
  }
  wave_order();
  const unsigned long long incl = lane_prefix(lane < n ? mass[lane] : 0ull);
  const uint64_t reach = __builtin_amdgcn_ballot_w64(lane < n && before + incl >= target);
  const unsigned long long cut = cand[reach ? __ffsll((unsigned long long)reach) - 1 : n - 1];
  wave_order();
  return cut;
}

// The cut among the rank keys in [klo, khi], before which there is the mass `before`.  for_each(fn) calls fn(key, there is one) for
// all keys, by all lanes together.  Rounds of BINS bins over the range that holds the cut until 64 keys or fewer are left
// (one, by then, in a run of equal scores).  keep(key, do) is called, by all lanes together, for what turns out to lie above that range.
// TIGHT: a round begins with the range of the keys that there are, where going over them once more costs little: a run of equal scores
// then differs in the few bits of its ids, one round instead of six with every sum in the same bin.
template <int BINS, bool TIGHT, typename ForEach, typename Keep>
__device__ __forceinline__ unsigned long long cut_of_many(ForEach&& for_each, Keep&& keep, unsigned long long klo, unsigned long long khi,
                                                          unsigned long long* cand, unsigned long long* mass,
                                                          unsigned long long before, unsigned long long target, float rmax) {
  const int lane = threadIdx.x & 63;
  unsigned found = 0;
  for (int round = 0; round < 10; round++) {
    if constexpr (TIGHT) {
      unsigned long long most = 0ull, least = ~0ull;
      for_each([&](unsigned long long key, bool is) {
        const bool in = is && key >= klo && key <= khi;
        if (in && key > most) most = key;
        if (in && key < least) least = key;
      });
      most = lane_max(most);
      least = ~lane_max(~least);
      if (most >= least) {
        klo = least;
        khi = most;
      }
    }
    const unsigned long long span = khi - klo;
    const int bits = span == 0 ? 0 : 64 - __clzll((long long)span);
    constexpr int DIGIT = BINS == 512 ? 9 : 8;
    static_assert(BINS == 1 << DIGIT, "bins");
    const int shift = max(0, bits - DIGIT);
    for (int i = lane; i < BINS; i += 64) mass[i] = 0;
    wave_order();
    for_each([&](unsigned long long key, bool is) {
      if (is && key >= klo && key <= khi) atomicAdd(&mass[(khi - key) >> shift], weight_of(from_ordered((unsigned)(key >> 32)), rmax));
    });
    wave_order();
    const int bin = crossing_bin<BINS>(mass, before, [&](unsigned long long) { return target; });
    wave_order();
    const unsigned long long top = khi;   // (what lies above the range has been dealt with)
    khi -= (unsigned long long)bin << shift;
    const unsigned long long deep = (1ull << shift) - 1ull;
    if (khi - klo > deep) klo = khi - deep;
    found = 0;   // how many are in the bin, and the first 64 of them
    for_each([&](unsigned long long key, bool is) {
      keep(key, is && key > khi && key <= top);
      const bool in = is && key >= klo && key <= khi;
      const uint64_t lanes = __builtin_amdgcn_ballot_w64(in);
      const unsigned pos = found + lanes_below(lanes);
      if (in && pos < 64u) cand[pos] = key;
      found += (unsigned)__popcll(lanes);
    });
    wave_order();
    if (found <= 64u) break;
  }
  if (found == 0u) return ~0ull;   // (out of reach: the crossing bin has mass, hence members)
  const unsigned long long cut = cut_of_few(cand, (int)min(found, 64u), mass, before, target, rmax);
  const unsigned long long key = lane < (int)min(found, 64u) ? cand[lane] : 0ull;
  keep(key, lane < (int)min(found, 64u) && key >= cut);
  return cut;
}

}  // namespace fgm
