// Grouping of query tiles that attend to similar sets of key blocks (paper Sec. 4.2), on the device.
//
//   bitmap_kernel     CSR mask -> one bit row per query tile
//   distance_kernel   d(i, j) = popcount(row_i XOR row_j) for all tile pairs of a slice (Sec. 4.2's distance)
//   greedy_kernel     the section's heuristic: the first ungrouped tile becomes a representative and takes the
//                     R - 1 ungrouped tiles closest to it (equal distances: lower tile index first)
//   consecutive_kernel  "merge-consecutive": R consecutive tiles per group
//   union_kernel      per group: OR of the members' rows, its popcount
//   row_pointers_kernel  counts -> union_indptr (fgscan.hpp)
//   emit_kernel       per group: the union's key-block ids in ascending order and, per id, the bit mask of the
//                     members that selected it
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "fgattn.h"
#include "fgscan.hpp"

namespace fgg {

constexpr int kThreads = 256;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

static bool launched() { return hipGetLastError() == hipSuccess; }

// one workgroup per query tile: its bit row is built in LDS and written out whole
__global__ void __launch_bounds__(kThreads) bitmap_kernel(const int64_t* indptr, const int32_t* indices, int Gw,
                                                          uint32_t* bits) {
  extern __shared__ uint32_t row[];
  const int tid = threadIdx.x;
  const int64_t w = blockIdx.x;
  for (int i = tid; i < Gw; i += kThreads) row[i] = 0u;
  __syncthreads();
  const int64_t beg = indptr[w], end = indptr[w + 1];
  for (int64_t e = beg + tid; e < end; e += kThreads) {
    const int g = indices[e];
    atomicOr(&row[g >> 5], 1u << (g & 31));
  }
  __syncthreads();
  for (int i = tid; i < Gw; i += kThreads) bits[w * Gw + i] = row[i];
}

// 64 x 64 block of the distance matrix of one slice per workgroup, 32 x 32 per wave: |a ^ b| = |a| + |b| - 2 |a & b|, and |a & b|
// for all pairs is a matrix product over the bits.  A bit becomes a 4-bit float, 1.0 = 0b0010, by a shift and a mask: a word of
// 32 bits is a lane's whole operand of v_mfma_f32_32x32x64_f8f6f4, its bits in the order 4n, 4n + 1, 4n + 2, 4n + 3, which is the
// same in both factors and so changes nothing.  The sums are whole numbers far below 2^24: exact.  The matrix is symmetric: only
// blocks on and above the diagonal are computed, the others are written from them.  Rows of 36 words in LDS put the 16 rows that a
// quarter of a wave reads at once into different banks.  Bound: latency of the steps, then the writes (100 MB of these figures').
// 12 slices of 2048 tiles x 2048 key blocks: with population counts, 4 x 4 pairs per thread, 260 us; now 83, and no less
// with blocks of 128, which leave small slices with too few workgroups (8 of 293 tiles, the whole call 276 -> 283 us).
constexpr int kDist = 64;           // tiles per side of a block
constexpr int kDistWords = 32;      // words of a row per step
constexpr int kDistFlush = 1024;    // words after which sums of longer rows go to whole numbers

template <typename T>
__global__ void __launch_bounds__(kThreads) distance_kernel(const uint32_t* bits, int QB, int Gw, int ld, T* dist) {
  typedef int i32x8 __attribute__((ext_vector_type(8)));
  typedef float f32x16 __attribute__((ext_vector_type(16)));
  typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int PITCH = sizeof(T) == 2 ? kDist + 2 : kDist + 1;
  __shared__ alignas(16) uint32_t words[2 * kDist][36];
  __shared__ uint32_t ones[2 * kDist];   // set bits per row
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.y * kDist, j0 = blockIdx.x * kDist;
  if (j0 < i0) return;
  const uint32_t* base = bits + (int64_t)blockIdx.z * QB * Gw;
  // rows i0 .. and then j0 .., 16 bytes of a row per thread, fetched one step ahead of their use; rows past the end repeat
  // the last one (their distances are not written)
  const int lc = (tid & 7) * 4, lr = tid >> 3;
  constexpr int PASS = kThreads / 8, PER = 2 * kDist / PASS;
  u32x4 next[PER];
  uint32_t set[PER];
#pragma unroll
  for (int m = 0; m < PER; m++) set[m] = 0;
  auto fetch = [&](int w0) {
#pragma unroll
    for (int m = 0; m < PER; m++) {
      const int r = m * PASS + lr;
      const uint32_t* const row = base + (int64_t)min(r < kDist ? i0 + r : j0 + r - kDist, QB - 1) * Gw;
      if (w0 + kDistWords <= Gw) next[m] = *reinterpret_cast<const u32x4_any*>(row + w0 + lc);
      else
#pragma unroll
        for (int e = 0; e < 4; e++) next[m][e] = w0 + lc + e < Gw ? row[w0 + lc + e] : 0u;
    }
  };
  f32x16 acc;
  uint32_t whole[sizeof(T) == 4 ? 16 : 1];
#pragma unroll
  for (int r = 0; r < 16; r++) acc[r] = 0.f;
  if constexpr (sizeof(T) == 4)
#pragma unroll
    for (int r = 0; r < 16; r++) whole[r] = 0u;
  const int i_wave = (wave >> 1) * 32, j_wave = (wave & 1) * 32;
  const int ra = i_wave + (lane & 31), rb = kDist + j_wave + (lane & 31);
  auto operand = [](uint32_t w) {
    constexpr uint32_t ONE = 0x22222222u;
    const i32x8 v = {(int)((w << 1) & ONE), (int)(w & ONE), (int)((w >> 1) & ONE), (int)((w >> 2) & ONE), 0, 0, 0, 0};
    return v;   // (the last four registers are no part of a 4-bit operand)
  };
  fetch(0);
  for (int w0 = 0; w0 < Gw; w0 += kDistWords) {
#pragma unroll
    for (int m = 0; m < PER; m++) {
      *reinterpret_cast<u32x4*>(&words[m * PASS + lr][lc]) = next[m];
#pragma unroll
      for (int e = 0; e < 4; e++) set[m] += (uint32_t)__popc(next[m][e]);
    }
    __syncthreads();
    if (w0 + kDistWords < Gw) fetch(w0 + kDistWords);
    for (int c = 0; c < kDistWords && w0 + c < Gw; c += 8) {   // eight words: four for either half of the wave
      const int cc = c + (lane >> 5) * 4;
      const u32x4 av = *reinterpret_cast<const u32x4*>(&words[ra][cc]), bv = *reinterpret_cast<const u32x4*>(&words[rb][cc]);
#pragma unroll
      for (int e = 0; e < 4; e++)   // (4: both factors in 4-bit floats; no scales)
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(av[e]), operand(bv[e]), acc, 4, 4, 0, 0, 0, 0);
    }
    if constexpr (sizeof(T) == 4)
      if ((w0 & (kDistFlush - 1)) == kDistFlush - kDistWords)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          whole[r] += (uint32_t)acc[r];
          acc[r] = 0.f;
        }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < PER; m++) {
    uint32_t n = set[m];
    for (int off = 1; off < 8; off <<= 1) n += __shfl_xor(n, off);
    if ((tid & 7) == 0) ones[m * PASS + lr] = n;
  }
  __syncthreads();
  // through LDS, so that the block and its mirror image are both written in whole rows
  T (&block)[kDist][PITCH] = *reinterpret_cast<T (*)[kDist][PITCH]>(words);
  static_assert(sizeof(block) <= sizeof(words), "the block takes the place of the words");
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const int i = i_wave + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), j = j_wave + (lane & 31);
    uint32_t both = (uint32_t)acc[r];
    if constexpr (sizeof(T) == 4) both += whole[r];
    block[i][j] = (T)(ones[i] + ones[kDist + j] - 2 * both);
  }
  __syncthreads();
  T* out = dist + (int64_t)blockIdx.z * QB * ld;
  if constexpr (sizeof(T) == 2) {   // two to a lane: rows start 16-byte aligned and end in padding
    const int c = 2 * (lane & 31);
    for (int r = tid >> 5; r < kDist; r += kThreads / 32) {
      if (i0 + r < QB && j0 + c < QB)
        *reinterpret_cast<uint32_t*>(out + (int64_t)(i0 + r) * ld + j0 + c) = block[r][c] | (uint32_t)block[r][c + 1] << 16;
      if (j0 > i0 && j0 + r < QB && i0 + c < QB)
        *reinterpret_cast<uint32_t*>(out + (int64_t)(j0 + r) * ld + i0 + c) = block[c][r] | (uint32_t)block[c + 1][r] << 16;
    }
  } else {
    for (int r = wave; r < kDist; r += kThreads / 64) {
      if (i0 + r < QB && j0 + lane < QB) out[(int64_t)(i0 + r) * ld + j0 + lane] = block[r][lane];
      if (j0 > i0 && j0 + r < QB && i0 + lane < QB) out[(int64_t)(j0 + r) * ld + i0 + lane] = block[lane][r];
    }
  }
}

// distances of all pairs of tiles of every slice, rows `ld` apart
template <typename T>
static void launch_distances(const uint32_t* bits, T* dist, int slices, int QB, int Gw, int ld, hipStream_t stream) {
  const unsigned side = (unsigned)((QB + kDist - 1) / kDist);
  hipLaunchKernelGGL(distance_kernel<T>, dim3(side, side, (unsigned)slices), dim3(kThreads), 0, stream, bits, QB, Gw, ld, dist);
}

__global__ void __launch_bounds__(kThreads) consecutive_kernel(int QB, int R, int NG, int32_t* group_tiles) {
  const int local = blockIdx.x * kThreads + threadIdx.x;   // position g*R + r inside the slice = the tile index
  if (local < NG * R) group_tiles[(int64_t)blockIdx.y * NG * R + local] = local < QB ? local : -1;
}

// one workgroup per slice; `used` lives in LDS (one byte per tile)
__global__ void __launch_bounds__(kThreads) greedy_kernel(const uint32_t* dist, int QB, int R, int NG,
                                                          int32_t* group_tiles) {
  extern __shared__ unsigned char used[];
  __shared__ unsigned long long best[kThreads];
  __shared__ int seed_s;
  const int tid = threadIdx.x;
  const int slice = blockIdx.x;
  const uint32_t* D = dist + (int64_t)slice * QB * QB;
  int32_t* out = group_tiles + (int64_t)slice * NG * R;
  for (int i = tid; i < QB; i += kThreads) used[i] = 0;
  __syncthreads();
  int next = 0;   // every tile below `next` is used (the same value in all threads)
  for (int g = 0; g < NG; g++) {
    if (tid == 0) {
      int s = next;
      while (s < QB && used[s]) s++;
      seed_s = s;
      if (s < QB) used[s] = 1;
    }
    __syncthreads();
    const int seed = seed_s;
    next = seed + 1;
    if (tid == 0) out[g * R] = seed < QB ? seed : -1;
    const uint32_t* drow = D + (int64_t)(seed < QB ? seed : 0) * QB;
    for (int r = 1; r < R; r++) {
      // smallest (distance, index) among the unused tiles
      unsigned long long mine = ~0ull;
      if (seed < QB)
        for (int j = tid; j < QB; j += kThreads)
          if (!used[j]) {
            const unsigned long long key = ((unsigned long long)drow[j] << 32) | (unsigned)j;
            mine = key < mine ? key : mine;
          }
      best[tid] = mine;
      __syncthreads();
      for (int off = kThreads / 2; off > 0; off >>= 1) {
        if (tid < off) best[tid] = best[tid + off] < best[tid] ? best[tid + off] : best[tid];
        __syncthreads();
      }
      const unsigned long long win = best[0];
      __syncthreads();
      if (tid == 0) {
        if (win != ~0ull) {
          const int j = (int)(win & 0xFFFFFFFFu);
          used[j] = 1;
          out[g * R + r] = j;
        } else {
          out[g * R + r] = -1;
        }
      }
      __syncthreads();
    }
  }
}

// Minimum of a 32-bit value over the 64 lanes of a wave, returned in every lane: shifts within rows of 16
// lanes, then the last lane of a row broadcast into the next row(s); lanes without a source keep the identity.
__device__ __forceinline__ unsigned wave_min_u32(unsigned x) {
  constexpr unsigned ID = 0xFFFFFFFFu;
  auto shifted = [&](unsigned v, auto ctrl, auto row_mask, auto bank_mask) {
    return (unsigned)__builtin_amdgcn_update_dpp((int)ID, (int)v, decltype(ctrl)::value, decltype(row_mask)::value,
                                                 decltype(bank_mask)::value, false);
  };
  using std::integral_constant;
  unsigned y = min(x, shifted(x, integral_constant<int, 0x111>(), integral_constant<int, 0xf>(), integral_constant<int, 0xf>()));   // row_shr:1
  y = min(y, shifted(x, integral_constant<int, 0x112>(), integral_constant<int, 0xf>(), integral_constant<int, 0xf>()));            // row_shr:2
  y = min(y, shifted(x, integral_constant<int, 0x113>(), integral_constant<int, 0xf>(), integral_constant<int, 0xf>()));            // row_shr:3
  y = min(y, shifted(y, integral_constant<int, 0x114>(), integral_constant<int, 0xf>(), integral_constant<int, 0xe>()));            // row_shr:4
  y = min(y, shifted(y, integral_constant<int, 0x118>(), integral_constant<int, 0xf>(), integral_constant<int, 0xc>()));            // row_shr:8
  y = min(y, shifted(y, integral_constant<int, 0x142>(), integral_constant<int, 0xa>(), integral_constant<int, 0xf>()));            // row_bcast:15
  y = min(y, shifted(y, integral_constant<int, 0x143>(), integral_constant<int, 0xc>(), integral_constant<int, 0xf>()));            // row_bcast:31
  return (unsigned)__builtin_amdgcn_readlane((int)y, 63);
}

// Ascending order of a lane's keys (odd-even merge sort).
template <int N>
__device__ __forceinline__ void sort_keys(unsigned (&k)[N]) {
  static_assert(N == 4 || N == 8 || N == 16, "written out for these");
  auto order = [&](int i, int j) {
    const unsigned a = min(k[i], k[j]), b = max(k[i], k[j]);
    k[i] = a;
    k[j] = b;
  };
  auto four = [&](int o) {
    order(o, o + 1); order(o + 2, o + 3); order(o, o + 2); order(o + 1, o + 3); order(o + 1, o + 2);
  };
  auto eight = [&](int o) {
    four(o);
    four(o + 4);
    order(o, o + 4); order(o + 1, o + 5); order(o + 2, o + 6); order(o + 3, o + 7);
    order(o + 2, o + 4); order(o + 3, o + 5);
    order(o + 1, o + 2); order(o + 3, o + 4); order(o + 5, o + 6);
  };
  if constexpr (N == 4) {
    four(0);
  } else if constexpr (N == 8) {
    eight(0);
  } else {
    eight(0);
    eight(8);
#pragma unroll
    for (int i = 0; i < 8; i++) order(i, i + 8);
#pragma unroll
    for (int i = 4; i < 8; i++) order(i, i + 4);
    order(2, 4); order(3, 5); order(6, 8); order(7, 9); order(10, 12); order(11, 13);
#pragma unroll
    for (int i = 1; i < 15; i += 2) order(i, i + 1);
  }
}

// The same heuristic for slices of at most KPT * kThreads tiles whose (distance, index) pairs fit 32 bits (`jbits` for
// the index).  One workgroup per slice and one group after the other, so what counts is the chain of instructions per group
// (with 1024 threads, whose 16 waves repeat the parts that every wave needs, 975 us at the size below) and that no load is
// part of it:
//   - the next representative is one of the first R unused tiles after this one (at most R - 1 of them are picked), so the
//     distances of those R rows are fetched while this group picks.  One compute unit draws 10-20 bytes per ns from beyond
//     its L2, so the bytes count too: 16-bit distances where they fit, and only the tiles from the row's own on (those
//     before it are used by the time it represents a group); with whole rows of 32 bits 832 us;
//   - every lane sorts its own keys, and a wave takes its R - 1 smallest from the lanes' heads with a cross-lane minimum each;
//   - the waves' lists meet in LDS after the group's one barrier, where every lane ranks one entry against all of them: all
//     waves know the picks, and each keeps its own bitmap of used tiles, so nothing is published;
//   - nothing in a group waits for what the group itself has issued to memory (rows fetched ahead, members stored);
//   - no conditional moves in the chain: one that reads vcc takes four times an ordinary instruction's time.
// 12 slices of 2048 tiles, R = 8: 975 us with a barrier per pick and one row fetched ahead; 750 with minima over all of a lane's
// keys and over the lists for every pick; 650 with sorted heads and ranks; 592 without a wait for the rows fetched ahead; 500 with
// the bitmap in LDS, where a lane notes a pick with one addition (in registers a pick took two dozen instructions).
// T = uint16_t: rows start 16-byte aligned and hold at least 15 elements past QB (of any value); T = uint32_t: no such assumption.
template <typename T, int KPT, int R>
__global__ void __launch_bounds__(kThreads) greedy_small_kernel(const T* dist, int QB, int ld, int NG, int jbits,
                                                                int32_t* group_tiles) {
  constexpr int WAVES = kThreads / 64, PICKS = R - 1;
  static_assert(R >= 2 && R <= 8 && WAVES * PICKS <= 64, "a list entry per lane");
  static_assert(KPT * kThreads <= 64 * 64 && KPT <= 32, "64 words of the bitmap, and a bit per key");
  constexpr int ENTRIES = WAVES * PICKS, QUADS = (ENTRIES + 3) / 4;
  __shared__ alignas(16) unsigned lists[2][64];
  __shared__ int picks[8];   // by rank + 1; the first wave's
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = blockIdx.x;
  const T* D = dist + (int64_t)slice * QB * ld;
  int32_t* out = group_tiles + (int64_t)slice * NG * R;
  const unsigned jmask = (1u << jbits) - 1u;
  if (tid < 128) lists[tid >> 6][lane] = 0xFFFFFFFFu;   // (entries past WAVES * PICKS stay)
  // used tiles as bits, each wave's own copy; those past the end count as used
  __shared__ uint64_t used[WAVES][64];
  const int mine = QB - lane * 64;
  used[wv][lane] = mine >= 64 ? 0ull : mine <= 0 ? ~0ull : ~0ull << mine;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (LDS operations of a wave complete in order)
  uint64_t free_tiles = 0;   // unused ones of tiles 64 * lane .. + 63, as of the last look
  auto look = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    free_tiles = ~used[wv][lane];
  };
  auto unused_word = [&](int l) {   // of lane l, in scalar registers
    return ((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)(free_tiles >> 32), l) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)(unsigned)free_tiles, l);
  };
  auto mark = [&](int tile) { atomicOr(reinterpret_cast<unsigned*>(used[wv]) + (tile >> 5), 1u << (tile & 31)); };
  const int j0 = tid * KPT;   // this thread's tiles: j0 .. j0 + KPT - 1
  static_assert(KPT <= 32 && 32 % KPT == 0, "a thread's tiles lie in one word");
  const unsigned* const my_word = reinterpret_cast<const unsigned*>(used[wv]) + (j0 >> 5);   // (their bits, from bit j0 % 32 on)
  constexpr int WORDS = KPT * sizeof(T) / 4;
  struct Part { uint32_t w[WORDS]; };   // a thread's part of a row of distances
  const int reach = j0 < QB ? j0 + KPT : 0;   // this thread has a part of the rows of tiles below
  auto fetch = [&](Part& p, int tile) {
    if (reach <= tile) return;
    const char* const row_of = reinterpret_cast<const char*>(D + (int64_t)tile * ld);   // (a scalar base and a lane's offset)
    const T* src = reinterpret_cast<const T*>(row_of + (unsigned)j0 * (unsigned)sizeof(T));
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int i = 0; i < WORDS; i += 4) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(src + 2 * i);
#pragma unroll
        for (int e = 0; e < 4; e++) p.w[i + e] = v[e];
      }
    } else {
#pragma unroll
      for (int i = 0; i < WORDS; i++) p.w[i] = src[min(i, QB - 1 - j0)];
    }
  };
  Part row = {};         // of the representative
  fetch(row, 0);
#pragma unroll
  for (int i = 0; i < WORDS; i++) asm volatile("" : "+v"(row.w[i]));   // (has arrived: inside the loop nothing waits for it)
  __syncthreads();
  int seed = 0;
  int picked = -1;   // lane r of the first wave: the r-th member of the group before, stored one group late (see below)
  for (int g = 0; g < NG; g++) {   // (every group but the last takes R tiles, so the representative exists)
    if (lane == 0) mark(seed);
    look();
    const unsigned taken = *my_word >> (j0 & 31);   // bit i: tile j0 + i is used
    int cand[R];
    Part ahead[R] = {};
    {
      int l = seed >> 6;
      uint64_t free = unused_word(l);
#pragma unroll
      for (int c = 0; c < R; c++) {
        while (free == 0 && l < 63) free = unused_word(++l);
        cand[c] = free != 0 ? l * 64 + __builtin_ctzll(free) : QB;
        free &= free - 1;   // (zero stays zero)
        if (cand[c] < QB) fetch(ahead[c], cand[c]);
      }
    }
    // The wait for the next representative's row, at the end of a group, is for all operations before it too: a store of this
    // group's members there would be waited for as well.
    if (g > 0 && tid < R) out[(g - 1) * R + tid] = picked;
    unsigned key[KPT];   // (distance, index) of the unused tiles this thread owns, all ones otherwise
#pragma unroll
    for (int i = 0; i < KPT; i++) {
      const unsigned dv = sizeof(T) == 2 ? (row.w[i / 2] >> (16 * (i & 1))) & 0xFFFFu : row.w[i];
      key[i] = ((dv << jbits) | (unsigned)(j0 + i)) | (unsigned)__builtin_amdgcn_sbfe((int)taken, i, 1);
    }
    sort_keys(key);
    unsigned top = 0u;   // lane r: the wave's r-th smallest
#pragma unroll
    for (int r = 0; r < PICKS; r++) {
      const unsigned w = wave_min_u32(key[0]);
      top |= w & (unsigned)(((lane ^ r) - 1) >> 31);   // (all ones in lane r)
      if (r + 1 < PICKS && key[0] == w) {   // (keys are distinct: one lane, or all that have none left)
        asm volatile("" : "+v"(key[0]));    // (stays a branch)
#pragma unroll
        for (int i = 0; i < KPT - 1 && i < PICKS - 1 - r; i++) key[i] = key[i + 1];
        if (KPT - 1 < PICKS - 1 - r) key[KPT - 1] = 0xFFFFFFFFu;
      }
    }
    unsigned* const list = lists[g & 1];   // (read by every wave before it comes to the next group's barrier)
    if (lane < PICKS) list[wv * PICKS + lane] = top;
    __syncthreads();
    const unsigned a = list[lane];   // (all ones past the entries)
    const bool there = a != 0xFFFFFFFFu;
    unsigned rank = 0;
#pragma unroll
    for (int i = 0; i < QUADS; i++) {
      const u32x4 e = *reinterpret_cast<const u32x4*>(&list[4 * i]);
#pragma unroll
      for (int x = 0; x < 4; x++) {
        // (keys of 16-bit distances have a bit to spare: the sign of a difference, without a compare and its wait states)
        if constexpr (sizeof(T) == 2) rank += ((e[x] & 0x7FFFFFFFu) - (a & 0x7FFFFFFFu)) >> 31;
        else rank += e[x] < a ? 1u : 0u;
      }
    }
    const int got = min(PICKS, (int)__popcll(__builtin_amdgcn_ballot_w64(there)));
    if (there && rank < (unsigned)PICKS) {
      mark((int)(a & jmask));
      if (wv == 0) picks[1 + rank] = (int)(a & jmask);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (tid < R) picked = tid == 0 ? seed : tid <= got ? picks[tid] : -1;
    look();
    int next = QB;
    {
      int l = seed >> 6;
      uint64_t free = unused_word(l);
      while (free == 0 && l < 63) free = unused_word(++l);
      if (free != 0) next = l * 64 + __builtin_ctzll(free);
    }
    seed = next;
    if (seed >= QB || g + 1 == NG) {
      if (tid < R) out[g * R + tid] = picked;
    }
    if (seed >= QB) {   // all taken: what is left of the list (nothing, by its length) holds no tile
      for (int t = (g + 1) * R + tid; t < NG * R; t += kThreads) out[t] = -1;
      break;
    }
#pragma unroll
    for (int c = 0; c < R; c++)
      if (cand[c] == seed) row = ahead[c];
  }
}

template <typename T, int R>
static void launch_greedy_small(const T* dist, int slices, int QB, int ld, int NG, int jbits, int32_t* group_tiles,
                                hipStream_t stream) {
  const dim3 grid((unsigned)slices), block(kThreads);
  if (QB <= 4 * kThreads && sizeof(T) == 4)
    hipLaunchKernelGGL((greedy_small_kernel<T, 4 * (4 / sizeof(T)), R>), grid, block, 0, stream, dist, QB, ld, NG, jbits, group_tiles);
  else if (QB <= 8 * kThreads)
    hipLaunchKernelGGL((greedy_small_kernel<T, 8, R>), grid, block, 0, stream, dist, QB, ld, NG, jbits, group_tiles);
  else
    hipLaunchKernelGGL((greedy_small_kernel<T, 16, R>), grid, block, 0, stream, dist, QB, ld, NG, jbits, group_tiles);
}

// Distances in 16 bits where no distance is larger and the workspace (4 bytes per pair of tiles) has room for the stride:
// rows start 16-byte aligned and, by the odd multiple of 16 bytes added, on different memory channels.
static bool distances_fit_16(int64_t QB, int64_t G) { return G <= 0xFFFF && QB >= 128; }
static int distance_stride(int QB) { return ((QB + 7) & ~7) + 72; }   // 2 (QB + 79) <= 4 QB for QB >= 79

template <typename T>
static bool greedy_small(const uint32_t* bits, T* dist, int slices, int QB, int Gw, int ld, int R, int NG, int jbits,
                         int32_t* group_tiles, hipStream_t stream) {
  launch_distances(bits, dist, slices, QB, Gw, ld, stream);
  if (!launched()) return false;
  if (R == 2) launch_greedy_small<T, 2>(dist, slices, QB, ld, NG, jbits, group_tiles, stream);
  else if (R == 4) launch_greedy_small<T, 4>(dist, slices, QB, ld, NG, jbits, group_tiles, stream);
  else launch_greedy_small<T, 8>(dist, slices, QB, ld, NG, jbits, group_tiles, stream);
  return launched();
}

// one workgroup per group: OR of the members' rows into `ubits`, number of set bits into `count`
__global__ void __launch_bounds__(kThreads) union_kernel(const uint32_t* bits, const int32_t* group_tiles, int QB, int Gw,
                                                         int R, int NG, uint32_t* ubits, unsigned* count) {
  __shared__ unsigned red[kThreads];
  const int tid = threadIdx.x;
  const int64_t grp = blockIdx.x;
  const int slice = (int)(grp / NG);
  const uint32_t* base = bits + (int64_t)slice * QB * Gw;
  int tiles[8];
  for (int r = 0; r < 8; r++) tiles[r] = r < R ? group_tiles[grp * R + r] : -1;
  unsigned n = 0;
  for (int i = tid; i < Gw; i += kThreads) {
    uint32_t u = 0;
    for (int r = 0; r < 8; r++)
      if (tiles[r] >= 0) u |= base[(int64_t)tiles[r] * Gw + i];
    ubits[grp * Gw + i] = u;
    n += (unsigned)__popc(u);
  }
  red[tid] = n;
  __syncthreads();
  for (int off = kThreads / 2; off > 0; off >>= 1) {
    if (tid < off) red[tid] += red[tid + off];
    __syncthreads();
  }
  if (tid == 0) count[grp] = red[0];
}

// one workgroup per group: ids of the union in ascending order with their member masks
__global__ void __launch_bounds__(kThreads) emit_kernel(const uint32_t* bits, const uint32_t* ubits,
                                                        const int32_t* group_tiles, const int64_t* uindptr, int QB,
                                                        int Gw, int R, int NG, int32_t* uindices, uint8_t* umemb,
                                                        int64_t capacity) {
  __shared__ unsigned wave_tot[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t grp = blockIdx.x;
  const int slice = (int)(grp / NG);
  const uint32_t* base = bits + (int64_t)slice * QB * Gw;
  int tiles[8];
  for (int r = 0; r < 8; r++) tiles[r] = r < R ? group_tiles[grp * R + r] : -1;
  const int64_t out0 = uindptr[grp];
  unsigned run = 0;
  for (int w0 = 0; w0 < Gw; w0 += kThreads) {
    const int i = w0 + tid;
    const uint32_t u = i < Gw ? ubits[grp * Gw + i] : 0u;
    const unsigned n = (unsigned)__popc(u);
    unsigned incl = n;
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned up = __shfl_up(incl, off);
      if (lane >= off) incl += up;
    }
    if (lane == 63) wave_tot[wv] = incl;
    __syncthreads();
    unsigned before = run;
    for (int w2 = 0; w2 < wv; w2++) before += wave_tot[w2];
    const unsigned total = wave_tot[0] + wave_tot[1] + wave_tot[2] + wave_tot[3];
    __syncthreads();
    if (u != 0u) {
      uint32_t m[8];
      for (int r = 0; r < 8; r++) m[r] = tiles[r] >= 0 ? base[(int64_t)tiles[r] * Gw + i] : 0u;
      int64_t pos = out0 + before + incl - n;
      uint32_t rest = u;
      while (rest) {
        const int b = __ffs(rest) - 1;
        rest &= rest - 1;
        unsigned mask = 0;
        for (int r = 0; r < 8; r++) mask |= ((m[r] >> b) & 1u) << r;
        if (pos < capacity) {
          uindices[pos] = i * 32 + b;
          umemb[pos] = (uint8_t)mask;
        }
        pos++;
      }
    }
    run += total;
  }
}

struct Layout {
  int64_t slices, QB, G, Gw, R, NG, groups;
  size_t bits_off, ubits_off, count_off, dist_off, total;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static int layout_of(const fgattn_params* p, int mode, Layout* lo) {
  if (p == nullptr) return FGATTN_E_NULL;
  if (p->B < 1 || p->H < 1 || p->L < 1 || p->N < 1) return FGATTN_E_SHAPE;
  if (p->M != 16 && p->M != 32 && p->M != 64 && p->M != 128) return FGATTN_E_SHAPE;
  if (mode != FGATTN_GROUP_CONSECUTIVE && mode != FGATTN_GROUP_XOR) return FGATTN_E_FLAGS;
  if (p->L > (1 << 24)) return FGATTN_E_SHAPE;
  lo->slices = (int64_t)p->B * p->H;
  lo->QB = ((int64_t)p->L + p->M - 1) / p->M;
  lo->G = ((int64_t)p->L + p->N - 1) / p->N;
  lo->Gw = (lo->G + 31) / 32;
  lo->R = 128 / p->M;
  lo->NG = (lo->QB + lo->R - 1) / lo->R;
  lo->groups = lo->slices * lo->NG;
  if (lo->slices > 65535 || lo->slices * lo->QB > 0x7fffffffLL || lo->Gw * 4 > 60 * 1024 || lo->QB > 48 * 1024)
    return FGATTN_E_SHAPE;
  size_t off = 0;
  lo->bits_off = off;
  off = align256(off + (size_t)lo->slices * lo->QB * lo->Gw * 4);
  lo->ubits_off = off;
  off = align256(off + (size_t)lo->groups * lo->Gw * 4);
  lo->count_off = off;
  off = align256(off + (size_t)lo->groups * 4);
  lo->dist_off = off;
  if (mode == FGATTN_GROUP_XOR) off = align256(off + (size_t)lo->slices * lo->QB * lo->QB * 4);
  lo->total = off;
  return FGATTN_OK;
}

static int device_ok() {
  static int known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return FGATTN_E_DEVICE;
  if (known[dev] == 0) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return FGATTN_E_DEVICE;
    known[dev] = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : 2;
  }
  return known[dev] == 1 ? FGATTN_OK : FGATTN_E_DEVICE;
}

}  // namespace fgg

extern "C" {

size_t fgattn_group_workspace_bytes(const fgattn_params* p, int mode) {
  fgg::Layout lo;
  if (fgg::layout_of(p, mode, &lo) != FGATTN_OK) return 0;
  return lo.total;
}

int fgattn_group_select(const int64_t* mask_indptr, const int32_t* mask_indices, const fgattn_params* p, int mode,
                        int32_t* group_tiles, int64_t* union_indptr, void* workspace, size_t workspace_bytes,
                        void* stream_v) {
  using namespace fgg;
  Layout lo;
  int rc = layout_of(p, mode, &lo);
  if (rc) return rc;
  if (!mask_indptr || !mask_indices || !group_tiles || !union_indptr || !workspace) return FGATTN_E_NULL;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(union_indptr) & 7) ||
      (reinterpret_cast<uintptr_t>(group_tiles) & 3))
    return FGATTN_E_ALIGN;
  if (workspace_bytes < lo.total) return FGATTN_E_WORKSPACE;
  rc = device_ok();
  if (rc) return rc;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  char* ws = static_cast<char*>(workspace);
  uint32_t* bits = reinterpret_cast<uint32_t*>(ws + lo.bits_off);
  uint32_t* ubits = reinterpret_cast<uint32_t*>(ws + lo.ubits_off);
  unsigned* count = reinterpret_cast<unsigned*>(ws + lo.count_off);
  uint32_t* dist = reinterpret_cast<uint32_t*>(ws + lo.dist_off);
  const int QB = (int)lo.QB, Gw = (int)lo.Gw, R = (int)lo.R, NG = (int)lo.NG;

  hipLaunchKernelGGL(bitmap_kernel, dim3((unsigned)(lo.slices * lo.QB)), dim3(kThreads), (size_t)Gw * 4, stream, mask_indptr,
                     mask_indices, Gw, bits);
  if (!launched()) return FGATTN_E_DEVICE;
  // (128 rows are a group by themselves: the greedy order of groups of one is the order of the tiles)
  if (mode == FGATTN_GROUP_CONSECUTIVE || R == 1) {
    hipLaunchKernelGGL(consecutive_kernel, dim3((unsigned)((NG * R + kThreads - 1) / kThreads), (unsigned)lo.slices),
                       dim3(kThreads), 0, stream, QB, R, NG, group_tiles);
  } else {
    // a distance is at most twice the number of key blocks; with the tile index below it in 32 bits where it fits
    int jbits = 1;
    while ((1 << jbits) < QB) jbits++;
    const bool small = QB <= 16 * kThreads && (2 * lo.G + 1) < ((int64_t)1 << (32 - jbits));
    if (small && distances_fit_16(QB, lo.G)) {
      if (!greedy_small(bits, reinterpret_cast<uint16_t*>(dist), (int)lo.slices, QB, Gw, distance_stride(QB), R, NG, jbits,
                        group_tiles, stream))
        return FGATTN_E_DEVICE;
    } else if (small) {
      if (!greedy_small(bits, dist, (int)lo.slices, QB, Gw, QB, R, NG, jbits, group_tiles, stream)) return FGATTN_E_DEVICE;
    } else {
      launch_distances(bits, dist, (int)lo.slices, QB, Gw, QB, stream);
      if (!launched()) return FGATTN_E_DEVICE;
      hipLaunchKernelGGL(greedy_kernel, dim3((unsigned)lo.slices), dim3(kThreads), (size_t)QB, stream, dist, QB, R, NG,
                         group_tiles);
    }
  }
  if (!launched()) return FGATTN_E_DEVICE;
  hipLaunchKernelGGL(union_kernel, dim3((unsigned)lo.groups), dim3(kThreads), 0, stream, bits, group_tiles, QB, Gw, R, NG,
                     ubits, count);
  if (!launched()) return FGATTN_E_DEVICE;
  fgscan::launch_row_pointers(count, lo.groups, union_indptr, stream);
  return launched() ? FGATTN_OK : FGATTN_E_DEVICE;
}

int fgattn_group_emit(const fgattn_params* p, int mode, const int32_t* group_tiles, const int64_t* union_indptr,
                      int32_t* union_indices, uint8_t* union_members, int64_t capacity, const void* workspace,
                      size_t workspace_bytes, void* stream_v) {
  using namespace fgg;
  Layout lo;
  int rc = layout_of(p, mode, &lo);
  if (rc) return rc;
  if (!group_tiles || !union_indptr || !workspace || ((!union_indices || !union_members) && capacity > 0))
    return FGATTN_E_NULL;
  if (capacity < 0) return FGATTN_E_SHAPE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(union_indices) & 3))
    return FGATTN_E_ALIGN;
  if (workspace_bytes < lo.total) return FGATTN_E_WORKSPACE;
  rc = device_ok();
  if (rc) return rc;
  const char* ws = static_cast<const char*>(workspace);
  const uint32_t* bits = reinterpret_cast<const uint32_t*>(ws + lo.bits_off);
  const uint32_t* ubits = reinterpret_cast<const uint32_t*>(ws + lo.ubits_off);
  hipLaunchKernelGGL(emit_kernel, dim3((unsigned)lo.groups), dim3(kThreads), 0, static_cast<hipStream_t>(stream_v), bits,
                     ubits, group_tiles, union_indptr, (int)lo.QB, (int)lo.Gw, (int)lo.R, (int)lo.NG, union_indices,
                     union_members, capacity);
  return launched() ? FGATTN_OK : FGATTN_E_DEVICE;
}

}  // extern "C"
