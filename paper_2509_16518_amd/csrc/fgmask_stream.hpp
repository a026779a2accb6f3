// Top-p selection for many long rows without a buffer of scores: included by fgmask.hip.
//
// The scores of a row are formed three times by the matrix cores instead of once, and never reach memory: a score takes
// 2 d operations, less time than its four bytes take to memory and back, and the same products in the same order
// give the same bits each time.
//   sweep_kernel<D, false>  the largest and the smallest score of every row
//   mass_kernel             a histogram of mass over the row's range (LDS), as fixed-point weights
//   locate_kernel           the bin where the descending mass crosses the target, as two thresholds on a score's product
//   sweep_kernel<D, true>   the bits of all key blocks above that bin; a list of its members and their scores
//   settle_kernel           ranks the members, adds the bits of those at or above the cut
//   overfull_kernel         rows whose lists were too short: the range around the cut narrowed by further passes
// The matrix product has the keys in its rows and the queries in its columns, so a lane owns one query: its range, its
// thresholds and its place in the lists are plain registers, and the 32 lanes of a histogram update name 32 different
// banks.  Against scores in memory, both mask calls, with the same emit kernel: 12 heads x 512 rows of 32760 532 -> 365 us,
// 24 x 929 rows of 118800 8.57 -> 4.75 ms (per eight heads of it: sweep 0.20, mass 0.50, locate 0.012, sweep 0.41, settle 0.12 ms).
#pragma once

namespace fgm {

constexpr int kSweepRows = 256;      // query blocks of a sweep workgroup: four waves of 64
constexpr int kSweepStep = 2;        // key tiles between two barriers of a sweep
constexpr int kMassRows = 64;        // query blocks of a mass workgroup, which all its waves share
constexpr int kMassWaves = 8;        // waves of a mass workgroup, each with key tiles of its own
constexpr int kMassBins = 312;       // 64 rows x 312 bins x 8 bytes fill 156 of 160 KB of LDS
constexpr int kMassWords = 2 * kMassBins * 32;   // 64-bit words of a histogram: [row / 32][bin][row % 32]
constexpr int kSettleBins = 512;
constexpr int kOverfullThreads = 512;

struct Member {
  float score;
  unsigned id;
};
// What locate_kernel leaves for a row.  With x = (product of the row and a key block) * sign of the scale: the key block lies above the
// crossing bin if x >= above, in it or above it if x >= inside.
struct alignas(16) RowCut {
  float neg_above, neg_inside;       // (negated)
  unsigned lo, hi;                   // ordered bits of the scores that the bin can hold
  unsigned long long mass_above, target;
};

struct StreamArgs {
  const uint16_t* qp;                // block means of Q: [slice][QB][D]
  const uint16_t* kp;                // of K (or K itself)
  int64_t k_slice_stride, k_row_stride;   // elements
  float scale, top_p;
  int QB, G, Gw;
  int slice0, slices;                // of this chunk
  int units, segs, seg_tiles;        // sweep: workgroup rows of kSweepRows, stretches of key tiles, tiles of a stretch
  int tiles, steps;                  // mass: row tiles of kMassRows, steps (of kMassWaves key tiles) per row tile
  int pieces, turn, groups;          // pieces of a row tile's steps, pieces per workgroup, workgroups (a multiple of eight)
  int cap;                           // list entries per row and stretch
  unsigned* range;                   // [row] (max, min) as ordered bits
  unsigned long long* hist;          // [workgroup + row tile][kMassWords]
  RowCut* cuts;                      // [row of the chunk]
  uint2* counts;                     // [row of the chunk][stretch]: key blocks above the bin, members
  Member* lists;                     // [row of the chunk][stretch][cap]
  unsigned long long* cut;           // [row]
  unsigned* count;                   // [row]; 0 marks a row left to overfull_kernel
  uint32_t* keep_bits;               // [row][Gw]
  unsigned* overfull;                // not zero if there are such rows
};

// ---- arithmetic that several kernels have to agree on to the last bit (no contraction into fused operations) ----
// first value of a histogram bin's float form: 2^23 + bin has the bin in its low bits
constexpr float kBinBias = 8388608.0f;

// Finite and above zero.  By bits: the library is built without regard for NaN, so a comparison with one may turn out either way.
__device__ __forceinline__ bool positive_finite(float x) { return __float_as_uint(x) - 1u < 0x7F7FFFFFu; }
// bins per unit of score, negated; 0 for a row without a range to divide: equal scores, infinite ones, a range so narrow that the
// quotient is infinite.  All of such a row lies in bin 0.
__device__ __forceinline__ float neg_bins_per_score(float rmax, float rmin) {
#pragma clang fp contract(off)
  const float width = rmax - rmin, bins = (float)(kMassBins - 1) / width;
  return positive_finite(width) && positive_finite(bins) ? -bins : 0.0f;
}
// below = score - rmax (not positive).  The low 16 bits of the result are the bin, falling scores in rising bins (0 to
// kMassBins - 1; 0 also for the NaN that an infinite `below` makes of it).
__device__ __forceinline__ float biased_bin(float below, float neg_bins) { return __builtin_fmaf(below, neg_bins, kBinBias); }
// Rounds results of 64-bit floating point toward zero from here on (MODE register, bits 3:2), as mass_update needs.  (No other
// 64-bit float instruction may be in the kernel: the compiler would set the mode back ahead of it.)
__device__ __forceinline__ void round_f64_toward_zero() { __builtin_amdgcn_s_setreg(1 | (2 << 6) | (1 << 11), 3); }
// Of four scores: weight = weight_below(below) and place = bin * 256 + base.  2^-1074 is the unit of a 64-bit float without
// an exponent, so the product of e = exp2(..) with 2^(40 - 1074), rounded toward zero, holds trunc(2^40 e) as its bits: two
// instructions for five.  In one statement because the compiler does not know the mode; the instructions between an exponential
// and the use of its result are the wait states that the hardware asks for there, and four at a time keep results from
// being waited for.
__device__ __forceinline__ void mass_update(const float (&below)[4], float neg_bins, unsigned base, unsigned long long (&weight)[4], unsigned (&place)[4]) {
  float e0, e1, e2, e3;
  asm("v_exp_f32 %0, %12\n\t"
      "v_exp_f32 %1, %13\n\t"
      "v_exp_f32 %2, %14\n\t"
      "v_exp_f32 %3, %15\n\t"
      "v_mad_u32_u16 %4, %16, %20, %21\n\t"
      "v_mad_u32_u16 %5, %17, %20, %21\n\t"
      "v_mad_u32_u16 %6, %18, %20, %21\n\t"
      "v_mad_u32_u16 %7, %19, %20, %21\n\t"
      "v_cvt_f64_f32 %8, %0\n\t"
      "v_cvt_f64_f32 %9, %1\n\t"
      "v_cvt_f64_f32 %10, %2\n\t"
      "v_cvt_f64_f32 %11, %3\n\t"
      "v_mul_f64 %8, %8, %22\n\t"
      "v_mul_f64 %9, %9, %22\n\t"
      "v_mul_f64 %10, %10, %22\n\t"
      "v_mul_f64 %11, %11, %22"
      : "=&v"(e0), "=&v"(e1), "=&v"(e2), "=&v"(e3), "=&v"(place[0]), "=&v"(place[1]), "=&v"(place[2]), "=&v"(place[3]),
        "=&v"(weight[0]), "=&v"(weight[1]), "=&v"(weight[2]), "=&v"(weight[3])
      : "v"(below[0] * kLog2e), "v"(below[1] * kLog2e), "v"(below[2] * kLog2e), "v"(below[3] * kLog2e),
        "v"(biased_bin(below[0], neg_bins)), "v"(biased_bin(below[1], neg_bins)), "v"(biased_bin(below[2], neg_bins)),
        "v"(biased_bin(below[3], neg_bins)), "s"(256), "v"(base), "s"(1ull << 40));
}
__device__ __forceinline__ float score_of(float product, float scale) {
#pragma clang fp contract(off)
  return product * scale;
}
// Of n infinite scores, which weigh nothing, rank_row keeps the first where it sorts them and all where it counts them off.
__device__ __forceinline__ unsigned kept_of_infinite(unsigned n) { return n <= (unsigned)kCap ? 1u : n; }
__device__ __forceinline__ float below_max(float score, float rmax) {
#pragma clang fp contract(off)
  return score - rmax;
}

// ---------------------------------------------------------------------------------------------
// Sweep: 256 query blocks (64 per wave, B operand, kept in registers: each operand read from LDS serves two matrix instructions)
// against a stretch of key tiles of 32, read once per workgroup and passed through XOR-swizzled LDS (as in scores_kernel).
// Bound: the first by the matrix cores at the clock that the power limit leaves them (226 GFLOP in 0.20 ms, the rate of a large
// matrix product); the second, 0.41 ms, by vector instructions (61% of issue slots) and by waits around the members' stores.
//   EMIT false: each row's largest and smallest score, two atomics per row and workgroup.
//   EMIT true:  a bit per pair (above the crossing bin), and the members of the bin.  The sign of (threshold - product) is
//               shifted into a word per lane, two instructions per score and threshold.  A row belongs to one wave, so places
//               in its list are counted in registers.
// ---------------------------------------------------------------------------------------------
template <int D, bool EMIT>
__global__ void __launch_bounds__(256, 3) sweep_kernel(const StreamArgs a) {
  constexpr int STEPS = D / 16, ROWB = D * 2, CHUNKS = ROWB / 16, TILEB = 32 * ROWB, LPT = kSweepStep * TILEB / 16 / 256;
  __shared__ __attribute__((aligned(16))) unsigned char ktile[2][kSweepStep * TILEB];
  __shared__ f32x4 picks[EMIT ? 4 : 1][EMIT ? 4 : 1][64];   // a wave's products: [wave][register / 4][lane][register % 4]
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, g = lane >> 5;
  // (see kShareUnits: every XCD keeps to its own eighth of the stretches)
  int local_unit, seg;
  if (a.segs < 8) {
    local_unit = blockIdx.x / a.segs;
    seg = blockIdx.x - local_unit * a.segs;
  } else {
    const int xcd_segs = (a.segs + 7) >> 3, j = blockIdx.x >> 3;
    const int first = j / (xcd_segs * kShareUnits) * kShareUnits, r = j - first * xcd_segs;
    const int share = min(kShareUnits, a.units - first);
    local_unit = first + r % share;
    seg = r / share * 8 + (blockIdx.x & 7);
    if (seg >= a.segs) return;
  }
  const int per_slice = (a.QB + kSweepRows - 1) / kSweepRows;
  const int local_slice = local_unit / per_slice, slice = a.slice0 + local_slice;
  const int q0 = (local_unit - local_slice * per_slice) * kSweepRows + wv * 64;
  const bool busy = q0 < a.QB;   // (a wave past the last query block still helps with the tiles)
  auto swz = [](int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
  bf16x8 qf[2][STEPS];
#pragma unroll
  for (int grp = 0; grp < 2; grp++) {
    const char* src = reinterpret_cast<const char*>(a.qp + ((int64_t)slice * a.QB + min(q0 + 32 * grp + ln, a.QB - 1)) * D);
#pragma unroll
    for (int s = 0; s < STEPS; s++) qf[grp][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(src + (2 * s + g) * 16));
  }
  const char* kbase = reinterpret_cast<const char*>(a.kp + slice * a.k_slice_stride);
  i32x4 stage[LPT];
  auto fetch_tile = [&](int tile) {   // key blocks past the end repeat the last one
#pragma unroll
    for (int i = 0; i < LPT; i++) {
      const int ci = i * 256 + tid, row = ci / CHUNKS, c = ci % CHUNKS;
      stage[i] = *reinterpret_cast<const i32x4*>(kbase + (int64_t)min(tile * 32 + row, a.G - 1) * a.k_row_stride * 2 + c * 16);
    }
  };
  auto stash_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < LPT; i++) {
      const int ci = i * 256 + tid, row = ci / CHUNKS, c = ci % CHUNKS;
      *reinterpret_cast<i32x4*>(&ktile[buf][row * ROWB + ((c ^ swz(row)) * 16)]) = stage[i];
    }
  };
  const int tile0 = seg * a.seg_tiles;
  const int ntiles = min(a.seg_tiles, (a.G - tile0 * 32 + 31) / 32);   // >= 1 by the grid
  // range
  float most[2] = {-INFINITY, -INFINITY}, least[2] = {INFINITY, INFINITY};
  // bits and members: this lane's queries (of both groups, for the products), and row (group g, ln) (for the words)
  const float sign = a.scale < 0.0f ? -1.0f : 1.0f;
  float neg_above[2], neg_inside[2];
  unsigned list[2];            // first list entry of the queries
  unsigned listed = 0;         // members so far, of group 0 and (upper half) of group 1; the same in both lanes of a query
  unsigned kept = 0;
  unsigned words[4];
  uint32_t* bits_row = nullptr;
  bool row_ok = false;
  if constexpr (EMIT) {
#pragma unroll
    for (int grp = 0; grp < 2; grp++) {
      const int row = local_slice * a.QB + min(q0 + 32 * grp + ln, a.QB - 1);
      neg_above[grp] = a.cuts[row].neg_above;
      neg_inside[grp] = a.cuts[row].neg_inside;
      if (q0 + 32 * grp + ln >= a.QB) neg_above[grp] = neg_inside[grp] = -INFINITY;   // no row: nothing is at or above
      list[grp] = ((unsigned)row * (unsigned)a.segs + (unsigned)seg) * (unsigned)a.cap;
    }
    const int q = q0 + 32 * g + ln;
    row_ok = q < a.QB;
    bits_row = a.keep_bits + ((int64_t)slice * a.QB + min(q, a.QB - 1)) * a.Gw;
  }
  fetch_tile(tile0);
  stash_tile(0);
  __syncthreads();
  for (int t0 = 0; t0 < ntiles; t0 += kSweepStep) {
    if (t0 + kSweepStep < ntiles) fetch_tile(tile0 + t0 + kSweepStep);
    bool stashed = false;
#pragma unroll
    for (int sub = 0; sub < kSweepStep; sub++) {
      const int t = t0 + sub;
      if (!busy || t >= ntiles) break;
      const unsigned char* kt = ktile[(t0 / kSweepStep) & 1] + sub * TILEB;
      f32x16 acc[2];
#pragma unroll
      for (int r = 0; r < 16; r++) acc[0][r] = acc[1][r] = 0.0f;
#pragma unroll
      for (int s = 0; s < STEPS; s++) {
        const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(kt + ln * ROWB + (((2 * s + g) ^ swz(ln)) * 16)));
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[0][s], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[1][s], acc[1], 0, 0, 0);
      }
      if constexpr (!EMIT) {
#pragma unroll
        for (int grp = 0; grp < 2; grp++)
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            most[grp] = fmaxf(fmaxf(most[grp], acc[grp][r]), acc[grp][r + 1]);
            least[grp] = fminf(fminf(least[grp], acc[grp][r]), acc[grp][r + 1]);
          }
      } else {
        const int key0 = (tile0 + t) * 32;
        const unsigned valid = key0 + 32 <= a.G ? ~0u : ~0u >> (32 - (a.G - key0));   // (the same in all lanes)
        unsigned spread[2], member[2];
#pragma unroll
        for (int grp = 0; grp < 2; grp++) {
          unsigned not_above = 0, not_inside = 0;   // bit r: accumulator register r, key 8 (r / 4) + 4 g + r % 4 of the tile
#pragma unroll
          for (int r = 15; r >= 0; r--) {
            const float da = __builtin_fmaf(acc[grp][r], sign, neg_above[grp]), di = __builtin_fmaf(acc[grp][r], sign, neg_inside[grp]);
            not_above = __builtin_amdgcn_alignbit(not_above, __float_as_uint(da), 31);
            not_inside = __builtin_amdgcn_alignbit(not_inside, __float_as_uint(di), 31);
          }
          unsigned x = ~not_above & 0xFFFFu;
          x = (x | (x << 8)) & 0x00FF00FFu;
          spread[grp] = (x | (x << 4)) & 0x0F0F0F0Fu;
          unsigned m = not_above & ~not_inside & 0xFFFFu;
          if (valid != ~0u) {
            unsigned v = (valid >> (4 * g)) & 0x0F0F0F0Fu;
            v = (v | (v >> 4)) & 0x00FF00FFu;
            m &= (v | (v >> 8)) & 0xFFFFu;
          }
          member[grp] = m;
        }
        // lanes of the first half collect the words of group 0, of the second half those of group 1
        const auto halves = __builtin_amdgcn_permlane32_swap(spread[0], spread[1], false, false);
        const unsigned word = (halves[0] | (halves[1] << 4)) & valid;
        kept += (unsigned)__popc(word);
        words[t & 3] = word;
        if (row_ok) {
          uint32_t* const to = bits_row + tile0 + (t & ~3);
          if ((t & 3) == 3) {
            struct __attribute__((packed, aligned(4))) Four { uint32_t w[4]; };   // (rows start on 4-byte boundaries)
            *reinterpret_cast<Four*>(to) = Four{{words[0], words[1], words[2], words[3]}};
          } else if (t + 1 == ntiles) {
            to[0] = words[0];
            if ((t & 3) > 0) to[1] = words[1];
            if ((t & 3) > 1) to[2] = words[2];
          }
        }
        // The next tiles go to LDS before the members' stores of a step's last tile: after them, the wait for their loads (they complete
        // in order) would be one for these stores too, as it is for those of the step's first tile.
        if (!stashed && (sub == kSweepStep - 1 || t + 1 == ntiles)) {
          if (t0 + kSweepStep < ntiles) stash_tile((t0 / kSweepStep + 1) & 1);
          stashed = true;
        }
        if (__builtin_amdgcn_ballot_w64((member[0] | member[1]) != 0u) != 0) {
          const unsigned mine = (unsigned)__popc(member[0]) | ((unsigned)__popc(member[1]) << 16);
          const auto both = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);   // of the first half's lane, of the second's
          const unsigned start = listed + (g ? both[0] : 0u);
          listed += both[0] + both[1];
#pragma unroll
          for (int grp = 0; grp < 2; grp++) {
            unsigned pos = grp ? start >> 16 : start & 0xFFFFu, m = member[grp];
            // (which register it is differs from lane to lane: LDS can be indexed so; a selection tree takes 20 instructions)
#pragma unroll
            for (int r4 = 0; r4 < 4; r4++)
              picks[wv][r4][lane] = f32x4{acc[grp][4 * r4], acc[grp][4 * r4 + 1], acc[grp][4 * r4 + 2], acc[grp][4 * r4 + 3]};
            const float* const mine_at = reinterpret_cast<const float*>(&picks[wv][0][lane]);
            while (m != 0u && pos < (unsigned)a.cap) {
              const int r = __ffs(m) - 1;
              m &= m - 1;
              const float product = mine_at[(r >> 2) * 256 + (r & 3)];
              a.lists[list[grp] + pos] = Member{score_of(product, a.scale), (unsigned)(key0 + 8 * (r >> 2) + 4 * g + (r & 3))};
              pos++;
            }
          }
        }
      }
    }
    if (!stashed && t0 + kSweepStep < ntiles) stash_tile((t0 / kSweepStep + 1) & 1);   // (the buffer that was read before the last barrier)
    __syncthreads();
  }
  if (!busy) return;
  if constexpr (!EMIT) {
#pragma unroll
    for (int grp = 0; grp < 2; grp++) {
      const float hi = fmaxf(most[grp], __shfl_xor(most[grp], 32)), lo = fminf(least[grp], __shfl_xor(least[grp], 32));
      const float s0 = score_of(hi, a.scale), s1 = score_of(lo, a.scale);   // (rounding keeps the order)
      const int q = q0 + 32 * grp + ln;
      if (g == 0 && q < a.QB) {
        unsigned* rr = a.range + 2 * ((int64_t)slice * a.QB + q);
        atomicMax(rr, ordered_bits(fmaxf(s0, s1)));
        atomicMin(rr + 1, ordered_bits(fminf(s0, s1)));
      }
    }
  } else {
    if (row_ok) {
      const int row = local_slice * a.QB + q0 + 32 * g + ln;
      a.counts[(int64_t)row * a.segs + seg] = make_uint2(kept, g ? listed >> 16 : listed & 0xFFFFu);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Histogram of mass.  A workgroup of eight waves keeps 64 query blocks in registers (all waves the same) and their histograms
// in LDS, and walks over key tiles, eight at a step, one per wave, whose operands each wave loads for itself (a tile is
// used by no other wave; through LDS, whole rows at a time, the same loads take 532 us instead of 504 per eight heads of 118800
// rows).  Bound: vector instructions, eleven per score of which the exponential takes two slots and the conversion to
// 64 bits two (59% of issue slots; 25% more of them, with the weight formed by 32-bit operations, 7% more time), the
// histogram's updates (one per score, 8 clocks of LDS per 64) and the matrix instructions, which issue between them.
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kMassWaves * 64, 2) mass_kernel(const StreamArgs a) {
  constexpr int STEPS = D / 16, THREADS = kMassWaves * 64;
  __shared__ __attribute__((aligned(16))) struct {
    unsigned long long hist[kMassWords];
  } sh;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, g = lane >> 5;
  const int per_slice = (a.QB + kMassRows - 1) / kMassRows;
  round_f64_toward_zero();
  for (int i = tid * 2; i < kMassWords; i += THREADS * 2) *reinterpret_cast<ulonglong2*>(&sh.hist[i]) = ulonglong2{0ull, 0ull};
  // A row tile's keys are cut into `pieces`, and a workgroup takes `turn` consecutive pieces of the line of all of them (slice,
  // row tile, piece).  The line is dealt to the XCDs in eighths, so that the workgroups of an XCD that begin at the same of
  // the few places of K walk over it in step and it comes through L2 once for them.  (Any places: 7 TB/s of K from beyond L2.)
  const int group = (blockIdx.x & 7) * (a.groups >> 3) + (int)(blockIdx.x >> 3);
  const int last = min((group + 1) * a.turn, a.tiles * a.pieces);
  for (int piece = group * a.turn; piece < last;) {
    const int tile = piece / a.pieces, local_slice = tile / per_slice;
    const int first_piece = piece - tile * a.pieces, end_piece = min(last - tile * a.pieces, a.pieces);
    const int slice = a.slice0 + local_slice, q0 = (tile - local_slice * per_slice) * kMassRows;
    const int s0 = (int)((int64_t)first_piece * a.steps / a.pieces), s1 = (int)((int64_t)end_piece * a.steps / a.pieces);
    piece += end_piece - first_piece;
    bf16x8 qf[2][STEPS];
    float rmax[2], neg_bins[2];
#pragma unroll
    for (int grp = 0; grp < 2; grp++) {
      const int64_t row = (int64_t)slice * a.QB + min(q0 + 32 * grp + ln, a.QB - 1);
      const char* src = reinterpret_cast<const char*>(a.qp + row * D);
#pragma unroll
      for (int s = 0; s < STEPS; s++) qf[grp][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(src + (2 * s + g) * 16));
      rmax[grp] = from_ordered(a.range[2 * row]);
      neg_bins[grp] = neg_bins_per_score(rmax[grp], from_ordered(a.range[2 * row + 1]));
    }
    const char* kbase = reinterpret_cast<const char*>(a.kp + slice * a.k_slice_stride);
    i32x4 keys_a[STEPS], keys_b[STEPS];   // of even and odd steps from s0 on
    auto fetch = [&](i32x4 (&kf)[STEPS], int step) {   // key blocks past the end repeat the last one
      const char* src = kbase + (int64_t)min((step * kMassWaves + wv) * 32 + ln, a.G - 1) * a.k_row_stride * 2 + g * 16;
#pragma unroll
      for (int s = 0; s < STEPS; s++) kf[s] = *reinterpret_cast<const i32x4*>(src + s * 32);
    };
    const unsigned base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)sh.hist + ln * 8;
    // products of the wave's tile of a step (its keys are in kf), the next one's keys on their way; between(i) fills the
    // slots after each pair of matrix instructions with the work of the tile before
    auto products = [&](f32x16 (&acc)[2], const i32x4 (&kf)[STEPS], i32x4 (&kf_next)[STEPS], int next, auto&& between) {
#pragma unroll
      for (int r = 0; r < 16; r++) acc[0][r] = acc[1][r] = 0.0f;
      fetch(kf_next, next);
#pragma unroll
      for (int s = 0; s < STEPS; s++) {
        const bf16x8 k8 = __builtin_bit_cast(bf16x8, kf[s]);
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k8, qf[0][s], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k8, qf[1][s], acc[1], 0, 0, 0);
        between(s);
      }
    };
    // registers r .. r + 3 of a group's products into the histogram, or only the first n of them
    auto add = [&](const f32x16 (&acc)[2], int grp, int r, int n) {
      float below[4];
      unsigned long long weight[4];
      unsigned place[4];
#pragma unroll
      for (int i = 0; i < 4; i++) below[i] = below_max(score_of(acc[grp][r + i], a.scale), rmax[grp]);
      mass_update(below, neg_bins[grp], base + grp * (kMassBins * 256), weight, place);
#pragma unroll
      for (int i = 0; i < 4; i++)
        if (i < n)
          __hip_atomic_fetch_add((__attribute__((address_space(3))) unsigned long long*)(uintptr_t)place[i], weight[i], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // the tile of `step` (products in cur) into the histogram, and the products of the next one's into nxt
    auto one_step = [&](int step, const f32x16 (&cur)[2], f32x16 (&nxt)[2], const i32x4 (&kf)[STEPS], i32x4 (&kf_next)[STEPS]) {
      const int key0 = (step * kMassWaves + wv) * 32;
      constexpr int PER = 32 / STEPS;
      if (key0 + 32 <= a.G && step + 1 < s1) {
        products(nxt, kf, kf_next, min(step + 2, s1 - 1), [&](int slot_no) {
#pragma unroll
          for (int x = 0; x < PER; x += 4) add(cur, (slot_no * PER + x) >> 4, (slot_no * PER + x) & 15, 4);
          __builtin_amdgcn_sched_barrier(0);
        });
        return;
      }
#pragma unroll
      for (int grp = 0; grp < 2; grp++)
#pragma unroll
        for (int r = 0; r < 16; r += 4) add(cur, grp, r, a.G - (key0 + 2 * r + 4 * g));
      if (step + 1 < s1) products(nxt, kf, kf_next, min(step + 2, s1 - 1), [](int) {});
    };
    f32x16 even[2], odd[2];
    fetch(keys_a, s0);
    products(even, keys_a, keys_b, min(s0 + 1, s1 - 1), [](int) {});
    __syncthreads();   // the histogram is clear
#pragma unroll 1
    for (int step = s0; step < s1; step += 2) {
      one_step(step, even, odd, keys_b, keys_a);
      if (step + 1 < s1) one_step(step + 1, odd, even, keys_a, keys_b);
    }
    __syncthreads();
    unsigned long long* const out = a.hist + (int64_t)(group + tile) * kMassWords;
    for (int i = tid * 2; i < kMassWords; i += THREADS * 2) {
      *reinterpret_cast<ulonglong2*>(out + i) = *reinterpret_cast<const ulonglong2*>(&sh.hist[i]);
      *reinterpret_cast<ulonglong2*>(&sh.hist[i]) = ulonglong2{0ull, 0ull};
    }
  }
}

// ---------------------------------------------------------------------------------------------
// The crossing bin of 32 rows: the parts of their histograms are added, a prefix over the bins meets the target, and the
// bin's two edges become thresholds on the product (by bisection over all floats, with the arithmetic of the histogram).
// ---------------------------------------------------------------------------------------------
constexpr int kLocateParts = 24;   // threads per row
__global__ void __launch_bounds__(kLocateParts * 32) locate_kernel(const StreamArgs a) {
  constexpr int PARTS = kLocateParts, PER = kMassBins / PARTS;
  static_assert(kMassBins % PARTS == 0, "whole parts");
  __shared__ unsigned long long part_mass[PARTS][32];
  __shared__ unsigned crossing[32];
  __shared__ unsigned long long above[32], goal[32];
  __shared__ float edge[2][32];
  const int tid = threadIdx.x, ln = tid & 31, part = tid >> 5;
  const int tile = blockIdx.x >> 1, grp = blockIdx.x & 1;
  if (blockIdx.x == 0 && tid == 0) *a.overfull = 0;
  const int per_slice = (a.QB + kMassRows - 1) / kMassRows;
  const int local_slice = tile / per_slice, q = (tile - local_slice * per_slice) * kMassRows + 32 * grp + ln;
  unsigned long long mass[PER] = {};
  for (int group = tile * a.pieces / a.turn; group <= ((tile + 1) * a.pieces - 1) / a.turn; group++) {
    const unsigned long long* h = a.hist + (int64_t)(group + tile) * kMassWords + (grp * kMassBins + part * PER) * 32 + ln;
#pragma unroll
    for (int i = 0; i < PER; i++) mass[i] += h[i * 32];
  }
  unsigned long long mine = 0;
#pragma unroll
  for (int i = 0; i < PER; i++) mine += mass[i];
  part_mass[part][ln] = mine;
  if (tid < 32) crossing[tid] = kMassBins - 1;
  __syncthreads();
  unsigned long long run = 0, Z = 0;
  for (int p = 0; p < PARTS; p++) {
    if (p == part) run = Z;
    Z += part_mass[p][ln];
  }
  const double t = ceil((double)a.top_p * (double)Z);
  unsigned long long target = t < 1.0 ? 1ull : (unsigned long long)t;
  if (target > Z) target = Z;
  if (part == 0) {
    goal[ln] = target;
    above[ln] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; i++) {
    if (run < target && target <= run + mass[i]) {
      crossing[ln] = (unsigned)(part * PER + i);
      above[ln] = run;
    }
    run += mass[i];
  }
  __syncthreads();
  const bool ok = q < a.QB;
  const int64_t row = (int64_t)(a.slice0 + local_slice) * a.QB + min(q, a.QB - 1);
  const float rmax = from_ordered(a.range[2 * row]);
  const float mag = fabsf(a.scale);
  const float neg_bins = neg_bins_per_score(rmax, from_ordered(a.range[2 * row + 1]));
  const bool equal = a.range[2 * row] == a.range[2 * row + 1];
  if (part < 2 && neg_bins == 0.0f) {
    // all of the row lies in the bin; equal scores are no members, settle_kernel counts them off by id
    edge[part][ln] = part == 0 || equal ? INFINITY : -INFINITY;
  } else if (part < 2) {
    // the smallest x whose bin is below `limit` (part 0: above the crossing bin; part 1: in it or above).  (Scores of the
    // largest floats may be infinite, but neg_bins is not zero: nothing here is NaN.)
    const float limit = kBinBias + (float)(crossing[ln] + part);
    auto higher = [&](unsigned o) {
      return biased_bin(below_max(score_of(from_ordered(o), mag), rmax), neg_bins) < limit;
    };
    unsigned lo = ordered_bits(-3.402823466e38f), hi = ordered_bits(3.402823466e38f);
    float x;
    if (higher(lo)) {
      x = -INFINITY;
    } else if (!higher(hi)) {
      x = INFINITY;
    } else {   // not higher(lo), higher(hi)
      while (hi - lo > 1u) {
        const unsigned mid = lo + ((hi - lo) >> 1);
        if (higher(mid)) hi = mid;
        else lo = mid;
      }
      x = from_ordered(hi);
    }
    edge[part][ln] = x;
  }
  __syncthreads();
  if (part == 0 && ok) {
    RowCut c;
    const float xa = edge[0][ln], xi = edge[1][ln];
    c.neg_above = -xa;
    c.neg_inside = -xi;
    // ordered bits of the bin's scores: below that of the first one above it, not below that of its own first one
    c.hi = xa == INFINITY ? ordered_bits(rmax) : ordered_bits(score_of(xa, mag)) - 1u;
    c.lo = xi == -INFINITY ? 0u : ordered_bits(score_of(xi, mag));
    // (a row without a range has one bin; one with an infinite maximum has no weights either)
    c.mass_above = neg_bins == 0.0f ? 0ull : above[ln];
    c.target = fabsf(rmax) == INFINITY ? 0ull : goal[ln];
    a.cuts[(int64_t)local_slice * a.QB + q] = c;
  }
}

// ---------------------------------------------------------------------------------------------
// The cut of a row among the members of its crossing bin: one wave per row (cut_of_many).
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) settle_kernel(const StreamArgs a) {
  __shared__ unsigned long long all_mass[4][kSettleBins];
  __shared__ unsigned long long all_cand[4][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  unsigned long long* const mass = all_mass[wv];
  unsigned long long* const cand = all_cand[wv];
  const int rows = a.slices * a.QB;
  for (int local = blockIdx.x * 4 + wv; local < rows; local += gridDim.x * 4) {
    const int64_t row = (int64_t)a.slice0 * a.QB + local;
    const RowCut c = a.cuts[local];
    const unsigned highest = a.range[2 * row];
    const float rmax = from_ordered(highest);
    uint32_t* const bits_row = a.keep_bits + row * a.Gw;
    if (highest == a.range[2 * row + 1]) {   // equal scores, of weight 2^40: the first so many key blocks
      const unsigned keep = c.target != 0ull ? (unsigned)((c.target + (1ull << 40) - 1ull) >> 40) : kept_of_infinite((unsigned)a.G);
      for (int w = lane; w < a.Gw; w += 64) {
        const unsigned left = keep > 32u * (unsigned)w ? keep - 32u * (unsigned)w : 0u;
        bits_row[w] = left >= 32u ? ~0u : (1u << left) - 1u;
      }
      if (lane == 0) {
        a.cut[row] = rank_key(rmax, (int)keep - 1);
        a.count[row] = keep;
      }
      continue;
    }
    uint2 n = make_uint2(0u, 0u);   // of stretch `lane`
    if (lane < a.segs) n = a.counts[(int64_t)local * a.segs + lane];
    if (__builtin_amdgcn_ballot_w64(n.y > (unsigned)a.cap) != 0) {
      if (lane == 0) {
        a.count[row] = 0u;
        *a.overfull = 1u;   // (not counted: additions to one word take 12 ns each, 72 us for 6144 rows)
      }
      continue;
    }
    unsigned kept = n.x;
    for (int off = 32; off > 0; off >>= 1) kept += __shfl_xor(kept, off);
    const Member* const lists = a.lists + (int64_t)local * a.segs * a.cap;
    // fn(key, there is one), by all lanes together: half a wave per list (256 consecutive bytes), four pairs of lists and
    // two steps of each in flight
    auto for_each = [&](auto&& fn) {
      for (int seg = 0; seg < a.segs; seg += 8) {
        unsigned len[4], longest = 0;
        const Member* list[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int s0 = min(seg + 2 * e, 62);   // (stretches past the last have empty lists; 64 at most, an even number before the last)
          const unsigned n0 = seg + 2 * e < 64 ? (unsigned)__builtin_amdgcn_readlane((int)n.y, s0) : 0u;
          const unsigned n1 = seg + 2 * e < 64 ? (unsigned)__builtin_amdgcn_readlane((int)n.y, s0 + 1) : 0u;
          len[e] = lane < 32 ? n0 : n1;
          longest = max(longest, max(n0, n1));
          list[e] = lists + (int64_t)min(s0 + (lane >> 5), a.segs - 1) * a.cap;
        }
        for (unsigned base = 0; base < longest; base += 64) {
          Member m[2][4];
#pragma unroll
          for (int h = 0; h < 2; h++)
#pragma unroll
            for (int e = 0; e < 4; e++)
              if (base + 32 * h < longest) m[h][e] = list[e][min(base + 32 * h + (lane & 31), (unsigned)(a.cap - 1))];
#pragma unroll
          for (int h = 0; h < 2; h++)
#pragma unroll
            for (int e = 0; e < 4; e++)
              if (base + 32 * h < longest) fn(rank_key(m[h][e].score, (int)m[h][e].id), base + 32 * h + (lane & 31) < len[e]);
        }
      }
    };
    const unsigned long long cut_key = cut_of_many<kSettleBins, false>(
        for_each,
        [&](unsigned long long key, bool is) {
          const unsigned id = 0xFFFFFFFFu - (unsigned)key;
          if (is) atomicOr(&bits_row[id >> 5], 1u << (id & 31));
          kept += (unsigned)__popcll(__builtin_amdgcn_ballot_w64(is));
        },
        (unsigned long long)c.lo << 32, ((unsigned long long)c.hi << 32) | 0xFFFFFFFFull, cand, mass, c.mass_above, c.target, rmax);
    if (lane == 0) {
      a.cut[row] = cut_key;
      a.count[row] = kept;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Rows with more members in some stretch than its list takes (scores crowded beside a few that stand out, many equal ones; rows of
// nothing but equal scores don't come here): 32 or 8 rows per workgroup, their scores formed anew in every pass over the keys, a
// stretch of the key tiles per wave.
//   FIRST   (not where the listed scores differ) how many members there are, their smallest and largest score.  Taking it that they are
//           equal, their number ahead of a wave follows from what the sweep counted: the bits are written in the same pass.
//   NARROW  a histogram of the members' mass, its bins over the range of the listed ones, until the bin that holds the cut has few enough
//   COUNT   of members of a single score that was left after that, per wave
//   LAST    the bits above the cut's range; its members into a list in LDS, ranked by a wave each, or counted off if they are equal
// Bound: the chain of a tile (LDS, matrix instructions, scores) with two waves to a SIMD, about 1 us.  (Fetching further ahead
// changes nothing; with the operands read from LDS one after the other a pass takes a tenth more, straight from memory twice as
// long.)  Select call, from kept scores / with eight or four rows formed into memory for rank_row / now: 6144 rows of 32760 in two
// values 1.34 / 1.91 / 0.63 ms, crowded beside one large negative score 1.72 / 2.24 / 1.18; 20480 of 4095 0.76 / 2.10 / 0.47 and
// 1.24 / 2.11 / 0.72; 929 of 118800 0.97 / 1.74 / 0.85 and 1.18 / 1.92 / 1.22 (with FIRST for all and bins over the whole range
// 1.70).  Equal scores (settle_kernel), 6144 of 32760: 1.57 / 2.04 / 0.26.
// The matrix product has 32 columns.  With 8 ROWS a lane holds what the three lanes 8, 16 and 24 from it hold, and takes a quarter of
// it: workgroups enough where rows are few.
// ---------------------------------------------------------------------------------------------
template <int D, int ROWS>
__global__ void __launch_bounds__(kOverfullThreads, 2) overfull_kernel(const StreamArgs a) {
  constexpr int STEPS = D / 16, WAVES = kOverfullThreads / 64, ROWB = D * 2, CHUNKS = ROWB / 16, TILEB = 32 * ROWB, LPT = TILEB / 16 / 64;
  constexpr int DIGIT = ROWS == 32 ? 8 : 10, BINS = 1 << DIGIT, LIST = BINS;   // (64 KB of LDS)
  constexpr int PER = ROWS / 2;                                               // scores of a tile per lane
  enum { FIRST, NARROW, COUNT, LAST };                                        // steps
  static_assert(ROWS == 32 || ROWS == 8, "written out for these");
  if (*a.overfull == 0) return;
  __shared__ __attribute__((aligned(16))) unsigned char staged[WAVES][TILEB];   // a wave's own
  __shared__ unsigned long long hist[BINS][ROWS];   // then the lists of rank keys
  __shared__ unsigned long long mass[WAVES][kShortBins], cand[WAVES][64];
  __shared__ unsigned long long mass_above[ROWS], target[ROWS], cut_key[ROWS];
  __shared__ unsigned lo[ROWS], hi[ROWS], least[ROWS], most[ROWS], listed[ROWS], kept[ROWS];
  __shared__ unsigned members[WAVES][ROWS];
  __shared__ unsigned dense_lo[ROWS], dense_hi[ROWS];   // most members lie in here, as far as is known
  // a bit per row: to be selected; known to have members of different scores; range still too wide; one score, not counted; bits written
  __shared__ unsigned todo, differ, wide, single, done;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, g = lane >> 5, rl = lane % ROWS, part = ln / ROWS;
  const int per_slice = (a.QB + ROWS - 1) / ROWS, ktiles = (a.G + 31) / 32;
  // A wave's key tiles, in the order of ids: whole stretches of the sweep where these divide well, since the numbers of members that the
  // sweep counted in them then say how many are ahead of a wave's own.
  const bool counted = a.segs >= 2 * WAVES || a.segs == WAVES;
  const int s0 = a.segs * wv / WAVES, s1 = a.segs * (wv + 1) / WAVES;
  const int t0 = counted ? min(s0 * a.seg_tiles, ktiles) : (int)((int64_t)ktiles * wv / WAVES);
  const int t1 = counted ? min(s1 * a.seg_tiles, ktiles) : (int)((int64_t)ktiles * (wv + 1) / WAVES);
  // (an eighth of the rows per XCD, where there are workgroups enough: those of a slice read its keys at about the same time)
  const int64_t all = (int64_t)a.slices * per_slice;
  const int xcds = (gridDim.x & 7) == 0 ? 8 : 1, xcd = (int)blockIdx.x & (xcds - 1);
  const int e_end = (int)(all * (xcd + 1) / xcds), e_step = (int)gridDim.x / xcds;
  for (int e = (int)(all * xcd / xcds) + (int)blockIdx.x / xcds; e < e_end; e += e_step) {
    const int local_slice = e / per_slice, slice = a.slice0 + local_slice, q0 = (e - local_slice * per_slice) * ROWS;
    const int64_t row0 = (int64_t)slice * a.QB + q0;
    __syncthreads();   // the rows before these are done with the shared state
    if (tid == 0) todo = differ = wide = single = done = 0;
    __syncthreads();
    if (tid < ROWS && q0 + tid < a.QB && a.count[row0 + tid] == 0u) {
      const RowCut c = a.cuts[(int64_t)local_slice * a.QB + q0 + tid];
      lo[tid] = max(c.lo, 1u);   // (0 stands for key blocks past the end; no score has those bits)
      hi[tid] = c.hi;
      mass_above[tid] = c.mass_above;
      target[tid] = c.target;
      dense_lo[tid] = ~0u;
      dense_hi[tid] = 0u;
      atomicOr(&todo, 1u << tid);
    }
    __syncthreads();
    const unsigned rows = todo;
    if (rows == 0u) continue;   // (the same in all threads)
    const int64_t row = row0 + min(rl, a.QB - 1 - q0);
    if (counted) {   // some of the scores that the sweep has listed, a few of each stretch
      const int64_t first_list = ((int64_t)local_slice * a.QB + min(q0 + rl, a.QB - 1)) * a.segs;
      unsigned own = 0, small = ~0u, large = 0u;
      for (int seg = s0; seg < s1; seg++) {
        const unsigned n = a.counts[first_list + seg].y;
        own += n;
        if (n != 0u) {
          const unsigned at = (min(n, (unsigned)a.cap) - 1u) * (unsigned)(lane / ROWS) / (64u / ROWS - 1u);
          const unsigned o = ordered_bits(a.lists[(first_list + seg) * a.cap + at].score);
          small = min(small, o);
          large = max(large, o);
        }
      }
      if (lane < ROWS) members[wv][rl] = own;
      if (own != 0u) {
        atomicMin(&dense_lo[rl], small);
        atomicMax(&dense_hi[rl], large);
      }
      __syncthreads();
      if (tid < ROWS && ((rows >> tid) & 1u) && dense_lo[tid] < dense_hi[tid]) {   // not equal: no need to see whether they are
        unsigned n = 0;
        for (int w = 0; w < WAVES; w++) n += members[w][tid];
        atomicOr(&differ, 1u << tid);
        if (n > (unsigned)LIST) atomicOr(&wide, 1u << tid);
      }
      __syncthreads();
    }
    const float rmax = from_ordered(a.range[2 * row]);
    bf16x8 qf[STEPS];
    {
      const char* src = reinterpret_cast<const char*>(a.qp + row * D);
#pragma unroll
      for (int s = 0; s < STEPS; s++) qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(src + (2 * s + g) * 16));
    }
    const char* const kbase = reinterpret_cast<const char*>(a.kp + slice * a.k_slice_stride);
    const unsigned odd = (unsigned)-(part & 1), upper = (unsigned)-(part >> 1);
    unsigned char* const kt = staged[wv];
    // fn(tile, scores, ordered bits) of the lane's scores of every tile of the wave, the next tile's keys on their way: score i is
    // key 8 (r / 4) + 4 g + r % 4 of the tile with r = part * PER + i; the bits of those past the end are 0.  (The keys come in whole
    // rows and go through LDS: as operands straight from memory, 32 rows for every instruction, a pass takes three times as long.)
    auto pass = [&](auto&& fn) {
      auto swz = [](int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
      i32x4 stage[LPT];
      const int64_t lane_at = (lane / CHUNKS) * a.k_row_stride * 2 + lane % CHUNKS * 16;
      auto fetch = [&](int tile) {
        if (tile * 32 + 32 <= a.G) {   // (64-bit products by the scalar unit)
          const char* const at = kbase + (int64_t)tile * 32 * a.k_row_stride * 2;
#pragma unroll
          for (int i = 0; i < LPT; i++) stage[i] = *reinterpret_cast<const i32x4*>(at + (int64_t)i * (64 / CHUNKS) * a.k_row_stride * 2 + lane_at);
        } else {   // key blocks past the end repeat the last one
#pragma unroll
          for (int i = 0; i < LPT; i++) {
            const int ci = i * 64 + lane, row = ci / CHUNKS, c = ci % CHUNKS;
            stage[i] = *reinterpret_cast<const i32x4*>(kbase + (int64_t)min(tile * 32 + row, a.G - 1) * a.k_row_stride * 2 + c * 16);
          }
        }
      };
      if (t0 < t1) fetch(t0);
#pragma unroll 1
      for (int tile = t0; tile < t1; tile++) {
        wave_order();
#pragma unroll
        for (int i = 0; i < LPT; i++) {
          const int ci = i * 64 + lane, row = ci / CHUNKS, c = ci % CHUNKS;
          *reinterpret_cast<i32x4*>(kt + row * ROWB + ((c ^ swz(row)) * 16)) = stage[i];
        }
        wave_order();
        fetch(min(tile + 1, t1 - 1));
        i32x4 kf[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; s++) kf[s] = *reinterpret_cast<const i32x4*>(kt + ln * ROWB + (((2 * s + g) ^ swz(ln)) * 16));
        __builtin_amdgcn_sched_barrier(0);   // (all on their way; left to itself the compiler waits for each by itself)
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; r++) acc[r] = 0.0f;
#pragma unroll
        for (int s = 0; s < STEPS; s++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[s]), qf[s], acc, 0, 0, 0);
        float x[PER];
        unsigned o[PER];
#pragma unroll
        for (int i = 0; i < PER; i++) {
          float product = acc[i];
          if constexpr (ROWS == 8) {
            auto either = [](float lower_half, float upper_half, unsigned mask) {
              return __uint_as_float((__float_as_uint(upper_half) & mask) | (__float_as_uint(lower_half) & ~mask));
            };
            product = either(either(acc[i], acc[4 + i], odd), either(acc[8 + i], acc[12 + i], odd), upper);
          }
          x[i] = score_of(product, a.scale);
          const unsigned u = __float_as_uint(x[i]);
          o[i] = u ^ ((unsigned)((int)u >> 31) | 0x80000000u);   // (ordered_bits)
        }
        const int left = a.G - tile * 32;
        if (left < 32) {
#pragma unroll
          for (int i = 0; i < PER; i++) {
            const int r = part * PER + i;
            o[i] = 8 * (r / 4) + 4 * g + r % 4 < left ? o[i] : 0u;
          }
        }
        fn(tile, x, o);
      }
    };
    // so that a range gives at most BINS - 2 bins
    auto shift_for = [](unsigned range) {
      const int shift = max(0, 32 - __clz((int)range) - DIGIT);
      return (range >> shift) > (unsigned)(BINS - 3) ? shift + 1 : shift;
    };
    // a value of a row, combined over its lanes
    auto over_lanes = [&](unsigned v, auto&& combine) {
      if constexpr (ROWS == 8) {
        v = combine(v, (unsigned)__shfl_xor(v, 8));
        v = combine(v, (unsigned)__shfl_xor(v, 16));
      }
      return combine(v, (unsigned)__shfl_xor(v, 32));
    };
    uint32_t* const bits_row = a.keep_bits + row * a.Gw;
    unsigned act = rows & ~differ;   // rows that the step is about
    int step = FIRST;
    if (act == 0u) {
      act = wide;
      step = NARROW;
    }
    if (act == 0u) {
      act = rows;
      step = LAST;
    }
    __syncthreads();
    for (int round = 0; round < 16; round++) {   // (FIRST, a few times NARROW, COUNT, LAST)
      if (step == NARROW) {
        for (int i = tid; i < ROWS * BINS / 2; i += kOverfullThreads) reinterpret_cast<ulonglong2*>(hist)[i] = ulonglong2{0ull, 0ull};
        if (tid == 0) wide = 0;
      } else if (tid < ROWS && ((act >> tid) & 1u)) {
        least[tid] = ~0u;
        most[tid] = 0u;
        listed[tid] = 0;
        kept[tid] = 0;
        cut_key[tid] = ~0ull;
      }
      __syncthreads();
      const bool active = (act >> rl) & 1u;
      const unsigned from = active ? lo[rl] : ~0u, to = active ? hi[rl] : ~0u, span = to - from;   // (no score has the bits ~0)
      if (step == NARROW) {
        // bins over the dense part, and one each for what lies above and below it
        const unsigned high = active ? dense_hi[rl] : 0u;
        const int shift = active ? shift_for(high - dense_lo[rl]) : 0;
        pass([&](int, const float (&x)[PER], const unsigned (&o)[PER]) {
#pragma unroll
          for (int i = 0; i < PER; i++)
            if (o[i] - from <= span) {
              const unsigned bin = o[i] > high ? 0u : min((high - o[i]) >> shift, (unsigned)(BINS - 2)) + 1u;
              atomicAdd(&hist[bin][rl], weight_of(x[i], rmax));
            }
        });
        __syncthreads();
        for (int r = wv; r < ROWS; r += WAVES) {
          if (!((act >> r) & 1u)) continue;
          const unsigned high = dense_hi[r];
          const int bin_shift = shift_for(high - dense_lo[r]);
          unsigned long long before = mass_above[r];
          int bin = crossing_bin<BINS, ROWS>(&hist[0][r], before, [&](unsigned long long) { return target[r]; });
          if (lane == 0) {
            const unsigned whole_lo = lo[r], whole_hi = hi[r];
            if (bin == 0 && high == whole_hi) bin = 1;   // (nothing lies above: members without mass, of a target of zero)
            const unsigned below = (unsigned)max(bin - 1, 0) << bin_shift;
            const unsigned top = bin == 0 ? whole_hi : high - whole_lo > below ? high - below : whole_lo;
            const unsigned deep = (1u << bin_shift) - 1u;
            const unsigned bottom = bin == 0 ? high + 1u : bin == BINS - 1 || top - whole_lo <= deep ? whole_lo : top - deep;
            mass_above[r] = before;
            dense_hi[r] = hi[r] = top;
            dense_lo[r] = lo[r] = bottom;
            // how many members it has at most, by the weight of the least of them
            const unsigned long long weight = weight_of(from_ordered(bottom), from_ordered(a.range[2 * (row0 + r)]));
            const unsigned long long many = weight != 0ull ? hist[bin][r] / weight : ~0ull;
            if (top == bottom) atomicOr(&single, 1u << r);
            else if (many >= (unsigned long long)(LIST - LIST / 16)) atomicOr(&wide, 1u << r);
          }
        }
        __syncthreads();
      } else {
        // equal scores: so many of this wave's are kept, and the last one of all is the cut.  The first step takes it that they are equal.
        const bool ties = active && (step == FIRST ? counted : step == LAST && from == to), collect = active && step == LAST && !ties;
        int allowed = 0;
        bool last = false;
        unsigned equal_bits = 0;
        if (ties) {
          unsigned n = 0, ahead = 0;
          for (int w = 0; w < WAVES; w++) {
            if (w < wv) ahead += members[w][rl];
            n += members[w][rl];
          }
          // (if they are not, what the first step writes is overwritten)
          equal_bits = step == FIRST ? dense_hi[rl] : to;
          const unsigned long long weight = weight_of(from_ordered(equal_bits), rmax);
          unsigned long long need = target[rl] > mass_above[rl] ? target[rl] - mass_above[rl] : 1ull;
          need = weight != 0ull ? (need + weight - 1ull) / weight : kept_of_infinite(n);
          const unsigned keep = (unsigned)min(need, (unsigned long long)n), own = members[wv][rl];
          allowed = (int)min((int64_t)own, max((int64_t)keep - (int64_t)ahead, (int64_t)0));
          last = keep > ahead && keep <= ahead + own;
        }
        unsigned count = 0, n = 0, small = ~0u, large = 0u;
        pass([&](int tile, const float (&)[PER], const unsigned (&o)[PER]) {
          unsigned above = 0, in = 0;   // bit i: score i
#pragma unroll
          for (int i = PER - 1; i >= 0; i--) {   // (shifted in: an addition with carry each)
            above = above + above + (o[i] > to ? 1u : 0u);
            in = in + in + (o[i] - from <= span ? 1u : 0u);
          }
          n += (unsigned)__popc(in);
          if (step == FIRST) {
#pragma unroll
            for (int i = 0; i < PER; i++)
              if (o[i] - from <= span) {
                small = min(small, o[i]);
                large = max(large, o[i]);
              }
          }
          auto word_of = [&](unsigned v) {   // of all lanes of the row, by key
            if constexpr (ROWS == 32) {
              v = (v | (v << 8)) & 0x00FF00FFu;
              v = ((v | (v << 4)) & 0x0F0F0F0Fu) << (4 * g);
            } else {
              v <<= 8 * part + 4 * g;
            }
            return over_lanes(v, [](unsigned p, unsigned q) { return p | q; });
          };
          unsigned word = word_of(above);
          if (__builtin_amdgcn_ballot_w64(allowed != 0 && in != 0u) != 0) {
            unsigned equal = word_of(in);
            if (allowed != 0 && equal != 0u) {
              while (__popc(equal) > allowed) equal &= ~(0x80000000u >> __clz((int)equal));
              allowed -= __popc(equal);
              word |= equal;
              if (allowed == 0 && last) cut_key[rl] = rank_key_of_bits(equal_bits, tile * 32 + 31 - __clz((int)equal));
            }
          }
          if (active && lane < ROWS) {
            count += (unsigned)__popc(word);
            bits_row[tile] = word;
          }
          if (collect && in != 0u) {
            unsigned pos = atomicAdd(&listed[rl], (unsigned)__popc(in));
#pragma unroll
            for (int i = 0; i < PER; i++)
              if ((in >> i) & 1u) {
                const int r = part * PER + i;
                if (pos < (unsigned)LIST) hist[pos][rl] = rank_key_of_bits(o[i], tile * 32 + 8 * (r / 4) + 4 * g + r % 4);
                pos++;
              }
          }
        });
        n = over_lanes(n, [](unsigned p, unsigned q) { return p + q; });
        small = over_lanes(small, [](unsigned p, unsigned q) { return min(p, q); });
        large = over_lanes(large, [](unsigned p, unsigned q) { return max(p, q); });
        __syncthreads();   // (all have read the numbers of members)
        if (active && lane < ROWS) {
          atomicAdd(&kept[rl], count);
          members[wv][rl] = n;
          atomicMin(&least[rl], small);
          atomicMax(&most[rl], large);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the bits are in this L2 before those of listed members are added there
        __syncthreads();
        if (step == FIRST && tid < ROWS && active) {
          unsigned all_members = 0;
          for (int w = 0; w < WAVES; w++) all_members += members[w][tid];
          const bool equal = least[tid] == most[tid];
          if (equal && counted && least[tid] == dense_hi[tid]) atomicOr(&done, 1u << tid);
          if (!equal && all_members > (unsigned)LIST) atomicOr(&wide, 1u << tid);
          if (all_members != 0u) {
            dense_lo[tid] = lo[tid] = least[tid];
            dense_hi[tid] = hi[tid] = most[tid];
          }
        }
        if (step == COUNT && tid == 0) single = 0;
        __syncthreads();
      }
      if (step == LAST) break;
      act = wide;
      step = NARROW;
      if (act == 0u) {
        act = single;
        step = COUNT;
      }
      if (act == 0u) {
        act = rows & ~done;
        step = LAST;
        if (act == 0u) break;
      }
      __syncthreads();
    }
    for (int r = wv; r < ROWS; r += WAVES) {
      if (!((rows >> r) & 1u)) continue;
      const int64_t this_row = row0 + r;
      uint32_t* const bits_row = a.keep_bits + this_row * a.Gw;
      unsigned count = kept[r];
      unsigned long long cut = cut_key[r];
      const unsigned n = min(listed[r], (unsigned)LIST);
      if (n != 0u)
        cut = cut_of_many<kShortBins, true>(
            [&](auto&& fn) {
#pragma unroll 1
              for (unsigned i = lane; i < (n + 63u) / 64u * 64u; i += 64) fn(hist[min(i, n - 1u)][r], i < n);
            },
            [&](unsigned long long key, bool is) {
              const unsigned id = 0xFFFFFFFFu - (unsigned)key;
              if (is) atomicOr(&bits_row[id >> 5], 1u << (id & 31));
              count += (unsigned)__popcll(__builtin_amdgcn_ballot_w64(is));
            },
            (unsigned long long)lo[r] << 32, ((unsigned long long)hi[r] << 32) | 0xFFFFFFFFull, cand[wv], mass[wv], mass_above[r], target[r],
            from_ordered(a.range[2 * this_row]));
      if (lane == 0) {
        a.cut[this_row] = cut;
        a.count[this_row] = count;
      }
    }
  }
}

}  // namespace fgm
