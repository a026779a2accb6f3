// Mean-query/key top-p mask (paper Sec. 4.3 "Determining the Fine-grain Sparse Mask with Top-p
// Masking") for CDNA4: block means of Q and K, approximate attention between the block means,
// and per query block the smallest set of key blocks, most probable first, whose probability
// mass reaches p -- written straight into the CSR form the forward kernel reads.
//
// Kernels (all on the caller's stream):
//   pool_kernel        block means (fp32 running sum in row order, fp32 divide, one bf16 rounding)
//   scores_kernel      S = scale * Q_avg K_avg^T with bf16 MFMA, fp32 scores to the workspace
//   select_codes_kernel  rows of up to 131072 scores: persistent workgroups; the row is read once, a byte per score (its
//                      bin) stays in LDS; finds the CUT, the 64-bit key (score, then lower id first) of the last kept
//                      key block, without sorting the row, and leaves the kept set as one bit per key block
//   select_kernel      longer rows (or on request): the same selection, one workgroup per query block,
//                      every pass reading the row from device memory; leaves the same outputs
//   (fgmask_short.hpp)  rows of at most 1024 scores: scores and selection in one kernel, a wave per row
//   (fgmask_stream.hpp)  many long rows: the same selection from scores that are formed anew for each pass instead of kept
//   row_pointers_kernel  counts -> indptr (fgscan.hpp)
//   emit_bits_kernel   kept ids, ascending, into indices (from the bit rows)
//
// Where scores are kept, they are the only large intermediate (4 bytes per pair of query block and key block).  They are
// produced and consumed in chunks of whole score tiles (128 query blocks of one slice), scores_kernel and
// the selection kernel alternating over one buffer of bounded size; what outlives a chunk is one bit per pair.
//
// Selection works on integers so that it does not depend on the order of additions: the weight
// of a key block is exp2((s - max) * log2 e) in 2^-40 fixed point, the row's mass Z is the integer
// sum, and the kept set is the smallest prefix of the ranking whose integer mass reaches
// ceil(p * Z).  The ranking is never materialised: a histogram over the score range locates the
// bin in which the running mass crosses the target, only that bin's members are sorted.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "fgattn.h"
#include "fgscan.hpp"

namespace fgm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int kSelThreads = 256;
constexpr int kBins = 2048;
constexpr int kCap = 2048;          // members of the crossing bin that are sorted in LDS
// Rows of up to kRowCodesMax scores are selected by workgroups that read the row once and keep a byte per score in LDS.
constexpr int kRowBins = 1024;
constexpr int kRowCodesMax = 131072;
constexpr float kLog2e = 1.44269504088896340736f;

__device__ __forceinline__ unsigned ordered_bits(float s) {   // monotone: larger score, larger unsigned
  const unsigned u = __float_as_uint(s);
  return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float from_ordered(unsigned o) {
  const unsigned u = o ^ ((o >> 31) ? 0x80000000u : 0xFFFFFFFFu);
  return __uint_as_float(u);
}
// ---------------------------------------------------------------------------------------------
// Step 1: block means.  One thread per (block, pair of columns): the additions of a column run in
// row order, so every implementation of this reading produces the same bits.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint16_t mean_bf16(float acc, int n) {
  const float mean = __fdiv_rn(acc, (float)n);
  unsigned u = __float_as_uint(mean);
  u += 0x7FFFu + ((u >> 16) & 1u);   // nearest even; the inputs are finite
  return (uint16_t)(u >> 16);
}

struct PoolTensor {
  const uint16_t* x;
  int64_t sb, sh, sl;   // strides in elements
  int rows_per_block, nblocks;
  uint16_t* pooled;
};

// One wave per block, of Q first (blockIdx.x < q.nblocks), then of K.  Bound: latency for short inputs, where Q and K share a
// launch (12 heads x 9360 rows in blocks of 64: 2 x 6.2 us and the gap between -> 9.9), bytes for long ones (24 heads x
// 118800 rows of Q in blocks of 128: 182 us, 4 TB/s).  Sixteen rows are in flight.
__global__ void __launch_bounds__(64) pool_kernel(PoolTensor q, PoolTensor k, int H, int L, int d, unsigned* range_init) {
  const int c = threadIdx.x * 2;
  const bool of_k = (int)blockIdx.x >= q.nblocks;
  const PoolTensor& t = of_k ? k : q;
  const int blk = (int)blockIdx.x - (of_k ? q.nblocks : 0);
  const int slice = blockIdx.y;
  if (c >= d) return;
  // the Q part also resets the (max, min) pair of the score row this query block will own
  if (!of_k && c == 0) {
    range_init[2 * ((int64_t)slice * q.nblocks + blk)] = 0u;
    range_init[2 * ((int64_t)slice * q.nblocks + blk) + 1] = 0xFFFFFFFFu;
  }
  const int b = slice / H, h = slice - b * H;
  const int r0 = blk * t.rows_per_block;
  const int r1 = min(r0 + t.rows_per_block, L);
  const int64_t sl = t.sl;
  const uint16_t* p = t.x + b * t.sb + h * t.sh + (int64_t)r0 * sl + c;   // 4-byte aligned: strides are multiples of 8 elements
  float acc0 = 0.0f, acc1 = 0.0f;
  int r = r0;
  auto batch = [&](auto n) {
    constexpr int N = decltype(n)::value;
    for (; r + N <= r1; r += N, p += N * sl) {
      unsigned w[N];
#pragma unroll
      for (int i = 0; i < N; i++) w[i] = *reinterpret_cast<const unsigned*>(p + i * sl);
#pragma unroll
      for (int i = 0; i < N; i++) {
        acc0 = acc0 + __uint_as_float(w[i] << 16);
        acc1 = acc1 + __uint_as_float(w[i] & 0xFFFF0000u);
      }
    }
  };
  batch(std::integral_constant<int, 16>());
  batch(std::integral_constant<int, 8>());
  batch(std::integral_constant<int, 1>());
  const unsigned out = (unsigned)mean_bf16(acc0, r1 - r0) | ((unsigned)mean_bf16(acc1, r1 - r0) << 16);
  *reinterpret_cast<unsigned*>(t.pooled + ((int64_t)slice * t.nblocks + blk) * d + c) = out;
}

// ---------------------------------------------------------------------------------------------
// Step 2a: scores.  A workgroup owns 128 query blocks (32 per wave, A operand, kept in registers)
// and walks over tiles of 32 key blocks.  A tile is read from global memory once per workgroup,
// whole rows at a time (16 bytes per thread, next tile in flight during this tile's MFMAs), and
// passed through LDS, from where every wave takes it as its B operand; the 16-byte chunks of a row
// are XOR-swizzled so that both the row-wise writes and the column-wise operand reads are free of
// bank conflicts.  In the accumulator a register holds one query block and 32 consecutive key
// blocks across lanes, so every store covers whole 128-byte lines.  Bound: the writes of the scores (a kernel that
// only stores this pattern takes 173-188 us per GiB).  With a lane test and its branches around every store, and 160 lane
// exchanges per workgroup and wave for the ranges, it took 239 us for 805 MB (6144 rows of 32760), then 206; 301 us per GiB (rows of
// 118800, K shared as below), then 242.  (Calls of that size keep no scores now; 1024 rows of 32760, 134 MB, take 28 us.)
// ---------------------------------------------------------------------------------------------
// Tiles of a workgroup: with sixteen, the calls that come this way leave compute units idle or a second round nearly empty (both
// mask calls, 12 heads x 147 rows of 9360 scores 110 us, 98 with eight, 101 with four; 40 x 64 x 4096 85, 74, 75; 2 x 512 x 32760
// 113, 105, 107; 40 x 256 x 4096 142, 141, 140).
constexpr int kTilesPerGroup = 8;
// Workgroups go to the eight XCDs in turn.  With at least eight stretches of key blocks, every XCD keeps to its own eighth of
// them and takes a stretch for up to kShareUnits consecutive score tiles (of one slice, mostly) before the next one, so
// that the tiles read K through one L2 at about the same time.  (In the order of their indices they read it from device
// memory again, half as many bytes as they write: many rows of 118800 scores 337 us per GiB of scores, shared 301.)
constexpr int kShareUnits = 8;

template <int D>
__global__ void __launch_bounds__(256, 4) scores_kernel(const uint16_t* qp, const uint16_t* kp, int64_t k_slice_stride,
                                                      int64_t k_row_stride, int QB, int G, int Gs, float scale,
                                                      int unit0, int nunits, int YT, int segs, float* scores, unsigned* range) {
  constexpr int STEPS = D / 16;
  constexpr int ROWB = D * 2;                 // bytes of a row of K
  constexpr int CHUNKS = ROWB / 16;           // 16-byte chunks per row
  constexpr int TILEB = 32 * ROWB;
  constexpr int LPT = TILEB / 16 / 256;       // chunks per thread and tile
  static_assert(LPT >= 1, "a tile is at least one chunk per thread");
  __shared__ __attribute__((aligned(16))) unsigned char ktile[2][TILEB];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, g = lane >> 5;
  // which score tile of this chunk, and which stretch of its key blocks (see kShareUnits)
  int local_unit, seg;
  if (segs < 8) {
    local_unit = blockIdx.x / segs;
    seg = blockIdx.x - local_unit * segs;
  } else {
    const int xcd_segs = (segs + 7) >> 3, j = blockIdx.x >> 3;   // stretches of one XCD; its j-th workgroup
    const int first = j / (xcd_segs * kShareUnits) * kShareUnits, r = j - first * xcd_segs;
    const int share = min(kShareUnits, nunits - first);
    local_unit = first + r % share;
    seg = r / share * 8 + (blockIdx.x & 7);
    if (seg >= segs) return;
  }
  // unit = slice * YT + (tile of 128 query blocks inside the slice)
  const int unit = unit0 + local_unit;
  const int slice = unit / YT;
  const int qtile0 = (unit - slice * YT) * 128;
  const int q0 = qtile0 + wv * 32;   // (a wave past the last query block still helps with the tiles)
  const int tile0 = seg * kTilesPerGroup;
  auto swz = [](int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
  bf16x8 qf[STEPS];
  {
    const int qrow = min(q0 + ln, QB - 1);
    const char* src = reinterpret_cast<const char*>(qp + ((int64_t)slice * QB + qrow) * D);
#pragma unroll
    for (int s = 0; s < STEPS; s++) qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(src + (2 * s + g) * 16));
  }
  const char* kbase = reinterpret_cast<const char*>(kp + slice * k_slice_stride);
  i32x4 stage[LPT];
  auto fetch_tile = [&](int tile) {
#pragma unroll
    for (int i = 0; i < LPT; i++) {
      const int ci = i * 256 + tid, row = ci / CHUNKS, c = ci % CHUNKS;
      const int krow = min(tile * 32 + row, G - 1);
      stage[i] = *reinterpret_cast<const i32x4*>(kbase + (int64_t)krow * k_row_stride * 2 + c * 16);
    }
  };
  auto stash_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < LPT; i++) {
      const int ci = i * 256 + tid, row = ci / CHUNKS, c = ci % CHUNKS;
      *reinterpret_cast<i32x4*>(&ktile[buf][row * ROWB + ((c ^ swz(row)) * 16)]) = stage[i];
    }
  };
  // running range of the scores this lane produced, per accumulator register (= per query block); the minimum negated
  float vmax[16], vneg[16];
#pragma unroll
  for (int r = 0; r < 16; r++) {
    vmax[r] = -INFINITY;
    vneg[r] = -INFINITY;
  }
  // Key blocks past the end repeat the last one and query blocks past the end the last query block: neither changes a
  // range, and their scores land in the padding of a row and in rows of the tile that nobody reads.  So nothing in the loop
  // depends on a lane but its 32-bit offset; the row of register r is a scalar base.
  const bool busy = q0 < QB;   // (the same in all lanes of a wave)
  float* const rows = scores + ((int64_t)local_unit * 128 + wv * 32) * Gs + (int64_t)tile0 * 32;
  const unsigned lane_off = (unsigned)(4 * g) * (unsigned)Gs + (unsigned)ln;
  const int ntiles = min(kTilesPerGroup, (G - tile0 * 32 + 31) / 32);   // >= 1 by the grid
  fetch_tile(tile0);
  stash_tile(0);
  __syncthreads();
  for (int t = 0; t < ntiles; t++) {
    if (t + 1 < ntiles) fetch_tile(tile0 + t + 1);
    const unsigned char* kt = ktile[t & 1];
    if (busy) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; r++) acc[r] = 0.0f;
#pragma unroll
      for (int s = 0; s < STEPS; s++) {
        const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(kt + ln * ROWB + (((2 * s + g) ^ swz(ln)) * 16)));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[s], kf, acc, 0, 0, 0);
      }
      const unsigned off = lane_off + (unsigned)t * 32u;
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const float v = acc[r] * scale;
        vmax[r] = fmaxf(vmax[r], v);
        vneg[r] = fmaxf(vneg[r], -v);
        (rows + (int64_t)(8 * (r / 4) + r % 4) * Gs)[off] = v;
      }
    }
    if (t + 1 < ntiles) stash_tile((t + 1) & 1);   // (the buffer that was read in step t - 1, before the last barrier)
    __syncthreads();
  }
  if (!busy) return;
  // One (max, min) update per query block and wave.  The 16 registers meet over the 32 lanes that share their query
  // blocks by halves: a lane hands the half of its registers that its partner keeps to it and keeps the other, so after four
  // steps it holds one register's maximum of 16 lanes (15 exchanges instead of 80), and after the fifth of all 32.
  auto meet = [&](float (&x)[16]) {
#pragma unroll
    for (int b = 0; b < 4; b++) {
      const int half = 8 >> b;
      // (by bits: as `upper ? x[i] : x[i + half]` the compiler indexes the array and selects among all sixteen, 889 conditional
      // moves in all)
      const unsigned upper = (unsigned)-((ln >> b) & 1);
#pragma unroll
      for (int i = 0; i < half; i++) {
        const unsigned lower_half = __float_as_uint(x[i]), upper_half = __float_as_uint(x[i + half]), swap = (lower_half ^ upper_half) & upper;
        x[i] = fmaxf(__uint_as_float(lower_half ^ swap), __shfl_xor(__uint_as_float(upper_half ^ swap), 1 << b));
      }
    }
    return fmaxf(x[0], __shfl_xor(x[0], 16));
  };
  const float hi = meet(vmax), lo = -meet(vneg);
  const int r = ((ln & 1) << 3) | ((ln & 2) << 1) | ((ln & 4) >> 1) | ((ln & 8) >> 3);   // the register this lane ended up with
  const int qrow = q0 + 8 * (r / 4) + 4 * g + (r % 4);
  if (ln < 16 && qrow < QB) {
    unsigned* rr = range + 2 * ((int64_t)slice * QB + qrow);
    atomicMax(rr, ordered_bits(hi));
    atomicMin(rr + 1, ordered_bits(lo));
  }
}

// ---------------------------------------------------------------------------------------------
// Step 2b + 3: selection.
// ---------------------------------------------------------------------------------------------
// rank key of key block j with score s: higher score first, then lower id first
__device__ __forceinline__ unsigned long long rank_key_of_bits(unsigned ordered, int j) {
  return ((unsigned long long)ordered << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)j);
}
__device__ __forceinline__ unsigned long long rank_key(float s, int j) { return rank_key_of_bits(ordered_bits(s), j); }
// Weight of a score relative to the row maximum: trunc(2^40 * 2^((s - rmax) * log2 e)), 2^-40 fixed point.
// The bare exponential instruction differs from exp2f only below 2^-126, where the weight is zero either way.
// The products with powers of two are exact, and so is the split into a whole and a fractional part (the hardware
// has no float -> 64-bit integer conversion).
__device__ __forceinline__ unsigned long long weight_below(float below) {   // below = s - rmax
  const float x = __builtin_amdgcn_exp2f(below * kLog2e) * 256.0f;   // in [0, 2^8]; the weight is trunc(2^32 x)
  const unsigned hi = (unsigned)x;
  const unsigned lo = (unsigned)(__builtin_amdgcn_fractf(x) * 4294967296.0f);
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long weight_of(float s, float rmax) { return weight_below(s - rmax); }

// Visits every score of a row: four consecutive scores per thread and step (16-byte loads; rows start 16-byte
// aligned and their stride is a multiple of four floats), DEPTH steps in flight.
template <int THREADS, int DEPTH, typename Fn>
__device__ __forceinline__ void for_each_score(const float* s, int G, Fn&& fn) {
  constexpr int STEP = THREADS * 4;
  auto whole = [&](const float4& v, int j4) {
    fn(v.x, j4);
    fn(v.y, j4 + 1);
    fn(v.z, j4 + 2);
    fn(v.w, j4 + 3);
  };
  auto ragged = [&](const float4& v, int j4) {
    fn(v.x, j4);
    if (j4 + 1 < G) fn(v.y, j4 + 1);
    if (j4 + 2 < G) fn(v.z, j4 + 2);
    if (j4 + 3 < G) fn(v.w, j4 + 3);
  };
  int j4 = threadIdx.x * 4;
  if constexpr (DEPTH > 1) {
    for (; j4 + (DEPTH - 1) * STEP + 3 < G; j4 += DEPTH * STEP) {
      float4 v[DEPTH];
#pragma unroll
      for (int e = 0; e < DEPTH; e++) v[e] = *reinterpret_cast<const float4*>(s + j4 + e * STEP);
#pragma unroll
      for (int e = 0; e < DEPTH; e++) whole(v[e], j4 + e * STEP);
    }
  }
  for (; j4 < G; j4 += STEP) ragged(*reinterpret_cast<const float4*>(s + j4), j4);
}

}  // namespace fgm

#include "fgmask_wave.hpp"

namespace fgm {

// (Sums over a wave go by its own data paths, lane_prefix.  By shuffles through LDS, two for every 64-bit step, the sums of
// select_codes_kernel cost the whole of fgattn_mask_select and _emit 1-5%: 12 x 147 rows of 9360 scores 97.6 us, now 93.1; 40 x 64 rows
// of 4096 74.3, now 70.8; 512 rows of 32760 72.4, now 71.6)
// Exclusive prefix of `n` over the threads of the workgroup in thread order; *total gets the sum.
// wave_tot: THREADS / 64 words of shared memory.  Contains two barriers.
template <int THREADS>
__device__ __forceinline__ unsigned block_exclusive(unsigned n, unsigned* wave_tot, unsigned* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const unsigned incl = lane_prefix(n);
  if (lane == 63) wave_tot[wv] = incl;
  __syncthreads();
  unsigned before = 0;
  for (int w2 = 0; w2 < wv; w2++) before += wave_tot[w2];
  unsigned all = 0;
  for (int w2 = 0; w2 < THREADS / 64; w2++) all += wave_tot[w2];
  *total = all;
  __syncthreads();
  return before + incl - n;
}

template <int THREADS, int BINS, int CAP>
struct SelShared {
  unsigned long long mass[BINS];
  unsigned wave_tot[THREADS / 64];
  alignas(16) unsigned long long cand[CAP];
  unsigned long long wave_m[THREADS / 64];
  unsigned wave_n[THREADS / 64];
  unsigned long long mass_above, target, cut;
  unsigned n_above, bin, bin_cnt, ncand, klo, khi;
};

template <int THREADS, int BINS, int CAP>
__device__ __forceinline__ unsigned long long block_sum_u64(SelShared<THREADS, BINS, CAP>& sh, unsigned long long v) {
  v = lane_prefix(v);
  if ((threadIdx.x & 63) == 63) sh.wave_m[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long r = 0;
  for (int w2 = 0; w2 < THREADS / 64; w2++) r += sh.wave_m[w2];
  __syncthreads();
  return r;
}

// Exclusive prefix, in thread order, of a mass; *tm gets the mass of all threads.  Contains two barriers.
template <int THREADS, int BINS, int CAP>
__device__ __forceinline__ void block_exclusive_mass(SelShared<THREADS, BINS, CAP>& sh, unsigned long long m,
                                                     unsigned long long* em, unsigned long long* tm) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const unsigned long long im = lane_prefix(m);
  if (lane == 63) sh.wave_m[wv] = im;
  __syncthreads();
  unsigned long long bm = 0;
  for (int w2 = 0; w2 < wv; w2++) bm += sh.wave_m[w2];
  unsigned long long all = bm;
  for (int w2 = wv; w2 < THREADS / 64; w2++) all += sh.wave_m[w2];
  *tm = all;
  __syncthreads();
  *em = bm + im - m;
}

// Finds, in the histogram just built, the bin where the running mass (starting from mass_above) reaches the
// target; updates mass_above to exclude that bin and stores the bin.  Every thread owns BINS / THREADS consecutive
// bins; a prefix over the threads names the one owner whose bins contain the crossing.  FIRST: the histogram is
// that of the whole row; its mass Z sets the target ceil(top_p * Z) (at least 1, at most Z), and nothing lies above
// it yet.
template <bool FIRST, int THREADS, int BINS, int CAP>
__device__ __forceinline__ void locate_bin(SelShared<THREADS, BINS, CAP>& sh, float top_p) {
  const int tid = threadIdx.x;
  constexpr int PER = BINS / THREADS;
  const unsigned long long base = FIRST ? 0ull : sh.mass_above;
  unsigned long long target = FIRST ? 0ull : sh.target;
  unsigned long long local = 0;
  for (int i = 0; i < PER; i++) local += sh.mass[tid * PER + i];
  unsigned long long em, Z;
  block_exclusive_mass(sh, local, &em, &Z);
  if constexpr (FIRST) {   // every thread computes the same target
    const double t = ceil((double)top_p * (double)Z);
    target = t < 1.0 ? 1ull : (unsigned long long)t;
    if (target > Z) target = Z;
  }
  // the caller guarantees base < target <= base + (mass of this histogram); the two extra clauses only make sure
  // that some bin is named if that did not hold
  const unsigned long long lo = base + em;
  const bool mine = (lo < target && (target <= lo + local || tid == THREADS - 1)) || (tid == 0 && target <= lo);
  if (mine) {
    unsigned long long run = lo;
    int b = tid * PER;
    while (b < tid * PER + PER - 1 && run + sh.mass[b] < target) {
      run += sh.mass[b];
      b++;
    }
    sh.mass_above = run;
    sh.bin = (unsigned)b;
    if constexpr (FIRST) {
      sh.target = target;
      sh.n_above = 0;
    }
  }
  __syncthreads();
}

// Sorts cand[0 .. n2) (n2 a power of two above 64, unused entries zero) by descending key in LDS.  All threads call
// it; it ends with a barrier.
template <int THREADS, typename SH>
__device__ __forceinline__ void sort_candidates(SH& sh, int n2) {
  const int tid = threadIdx.x;
  for (int k = 2; k <= n2; k <<= 1)
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
      for (int i = tid; i < n2; i += THREADS) {
        const int l = i ^ jj;
        if (l > i) {
          const unsigned long long a = sh.cand[i], b = sh.cand[l];
          const bool desc = (i & k) == 0;
          if (desc ? (a < b) : (a > b)) {
            sh.cand[i] = b;
            sh.cand[l] = a;
          }
        }
      }
      __syncthreads();
    }
}

// Bin of a score in a histogram over a row's range [rmin, rmax] (collected by the scores kernel); bin 0 holds the largest
// scores, and inv = BINS / (rmax - rmin), 0 for a row of equal scores.
template <int BINS>
__device__ __forceinline__ float bins_per_score(float rmax, float rmin) {
  const float width = rmax - rmin;
  return width > 0.0f ? (float)BINS / width : 0.0f;
}
template <int BINS>
__device__ __forceinline__ unsigned value_bin_of(float v, float rmax, float inv) {
  return min((unsigned)((rmax - v) * inv), (unsigned)(BINS - 1));   // (rmax - v is not negative)
}

// where a score lies relative to bin `bin` of that histogram: -1 above, 0 inside, 1 below
template <int BINS>
__device__ __forceinline__ auto place_by_bin(unsigned bin, float rmax, float inv) {
  return [=](float v) -> int {
    const unsigned b = value_bin_of<BINS>(v, rmax, inv);
    return b < bin ? -1 : (b == bin ? 0 : 1);
  };
}

// The part of the selection after the row's histogram: sh holds the mass above the crossing bin, the target and n_above = 0, and
// place(score) says where a score lies, -1 above the bin, 0 in it, 1 below.  Called by all threads of the workgroup.  Writes
// the cut, the count and the kept set as one bit per key block (`keep_bits`, Gw words per row), from a row of scores `s` in
// device memory.
//
// Passes over the row: the scores ranked above the crossing bin are counted and written as bits straight away, the bin's
// members are collected; then the members are ranked, and the bits of those at or above the cut are added.  Only a crossing
// bin with more members than the sort holds takes further passes, and a last one that writes all bits from the cut.
template <int THREADS, int BINS, int CAP, int DEPTH, typename SH, typename Place>
__device__ __forceinline__ void rank_row(SH& sh, const float* s, int64_t row, float rmax, Place place, int G, float top_p,
                                         unsigned long long* cut, unsigned* count, uint32_t* keep_bits, int Gw) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // (see select_codes_kernel: nothing here is worth keeping from row to row)
  uint32_t* const bits_row = keep_bits + row * Gw;
  // All bits of the row from the cut (in sh.cut): set where the rank key is not below it.  A thread ranks four
  // consecutive key blocks, eight lanes make a word.
  auto write_all_bits = [&]() {
    __syncthreads();
    const unsigned long long c = sh.cut;
    const int last4 = (G - 1) & ~3;
    for (int base = 0; base < Gw * 32; base += DEPTH * THREADS * 4) {
      f32x4 v[DEPTH];
#pragma unroll
      for (int e = 0; e < DEPTH; e++) v[e] = *reinterpret_cast<const f32x4*>(s + min(base + (e * THREADS + tid) * 4, last4));
#pragma unroll
      for (int e = 0; e < DEPTH; e++) {
        const int j4 = base + (e * THREADS + tid) * 4;
        unsigned nib = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) nib |= j4 + i < G && rank_key(v[e][i], j4 + i) >= c ? 1u << i : 0u;
        unsigned word = nib << (4 * (tid & 7));
        word |= __shfl_xor(word, 1);
        word |= __shfl_xor(word, 2);
        word |= __shfl_xor(word, 4);
        if ((tid & 7) == 0 && (j4 >> 5) < Gw) bits_row[j4 >> 5] = word;
      }
    }
  };
  // The bits of everything above the crossing bin are in memory already (pass 2): add those of the collected
  // members cand[0 .. n) that are at or above the cut.  Those stores were made by other waves of this workgroup:
  // every wave waits until its own have completed before the barrier, so the atomics on the same words, which go to
  // the same L2, come after them (a device-wide fence would do too, but writes back the whole L2 on this chip).
  auto add_member_bits = [&](unsigned n) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const unsigned long long c = sh.cut;
    for (unsigned i = tid; i < n; i += THREADS) {
      const unsigned long long key = sh.cand[i];
      if (key >= c) {
        const unsigned id = 0xFFFFFFFFu - (unsigned)key;
        atomicOr(&bits_row[id >> 5], 1u << (id & 31));
      }
    }
  };

  // One pass: counts the scores ranked above the crossing bin and collects the rank keys of its members, as many
  // as fit the sort.  cls(v): -1 above the bin, 0 inside, +1 below or outside what was the bin before.  WITH_BITS:
  // "above" of a thread's four consecutive key blocks is a nibble of the row's bits, eight lanes make a word (every
  // word of the row is written once).  DEPTH 16-byte loads are in flight.
  auto count_and_collect = [&](auto&& cls, auto with_bits) {
    if (tid == 0) sh.ncand = 0;
    __syncthreads();
    unsigned na = 0;
    constexpr int STEP = THREADS * 4;
    const int last4 = (G - 1) & ~3;
    for (int base = 0; base < Gw * 32; base += DEPTH * STEP) {   // (the same trip count for all threads: they vote below)
      f32x4 v[DEPTH];   // (unconditional loads, of the last scores again past the end: under a test they become 4-byte loads)
#pragma unroll
      for (int e = 0; e < DEPTH; e++) v[e] = *reinterpret_cast<const f32x4*>(s + min(base + e * STEP + tid * 4, last4));
#pragma unroll
      for (int e = 0; e < DEPTH; e++) {
        const int j4 = base + e * STEP + tid * 4;
        const float x[4] = {v[e][0], v[e][1], v[e][2], v[e][3]};
        unsigned nib = 0, all = 0;
        uint64_t in[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int c = j4 + i < G ? cls(x[i]) : 1;
          nib |= c < 0 ? 1u << i : 0u;
          in[i] = __builtin_amdgcn_ballot_w64(c == 0);
          all += (unsigned)__popcll(in[i]);
        }
        if (all != 0u) {   // (one addition per wave for all its members: one each, to the same word, they are served one by one)
          unsigned first = 0;
          if ((tid & 63) == 0) first = atomicAdd(&sh.ncand, all);
          first = (unsigned)__builtin_amdgcn_readfirstlane((int)first);
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const unsigned pos = first + __builtin_amdgcn_mbcnt_hi((unsigned)(in[i] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in[i], 0u));
            if (((in[i] >> (tid & 63)) & 1u) && pos < (unsigned)CAP) sh.cand[pos] = rank_key(x[i], j4 + i);
            first += (unsigned)__popcll(in[i]);
          }
        }
        na += (unsigned)__popc(nib);
        if constexpr (decltype(with_bits)::value) {
          unsigned word = nib << (4 * (tid & 7));
          word |= __shfl_xor(word, 1);
          word |= __shfl_xor(word, 2);
          word |= __shfl_xor(word, 4);
          if ((tid & 7) == 0 && (j4 >> 5) < Gw) bits_row[j4 >> 5] = word;
        }
      }
    }
    const unsigned long long na_all = block_sum_u64(sh, (unsigned long long)na);   // (its barriers also order the atomics before the read of ncand)
    if (tid == 0) {
      sh.n_above += (unsigned)na_all;
      sh.bin_cnt = sh.ncand;
    }
    __syncthreads();
  };
  count_and_collect(place, std::true_type{});

  // The members of the crossing bin form a contiguous stretch of the ranking.  While there are too many to
  // sort, narrow the stretch: take the range [klo, khi] of their ordered score bits and histogram it again,
  // now linearly in those bits (every round divides the range by BINS, so a few rounds reach a single value).
  bool by_place = true;     // how the current bin is defined: place() == 0, or key range [klo, khi]
  bool bits_partial = true; // the bits in memory are those of pass 2 (everything above the first crossing bin)
  unsigned klo = 0, khi = 0;
  for (int round = 0; round < 6; round++) {
    if (sh.bin_cnt <= (unsigned)CAP) break;
    bits_partial = false;   // members of the first bin get ranked above the final one: all bits are rewritten at the end
    // range of ordered bits inside the current bin
    if (tid == 0) {
      sh.klo = 0xFFFFFFFFu;
      sh.khi = 0u;
    }
    __syncthreads();
    unsigned lo = 0xFFFFFFFFu, hi = 0u;
    for_each_score<THREADS, DEPTH>(s, G, [&, by_place, klo, khi](float v, int) {
      const unsigned o = ordered_bits(v);
      const bool in = by_place ? place(v) == 0 : (o >= klo && o <= khi);
      if (in) {
        lo = min(lo, o);
        hi = max(hi, o);
      }
    });
    atomicMin(&sh.klo, lo);
    atomicMax(&sh.khi, hi);
    __syncthreads();
    klo = sh.klo;
    khi = sh.khi;
    by_place = false;
    if (klo == khi) break;   // one score value left: a run of equal scores, handled by id below
    const unsigned long long R = (unsigned long long)(khi - klo) + 1ull;
    for (int i = tid; i < BINS; i += THREADS) sh.mass[i] = 0;
    __syncthreads();
    for_each_score<THREADS, DEPTH>(s, G, [&](float v, int) {
      const unsigned o = ordered_bits(v);
      if (o >= klo && o <= khi) {
        const int b = (int)(((unsigned long long)(khi - o) * BINS) / R);
        atomicAdd(&sh.mass[b], weight_of(v, rmax));
      }
    });
    __syncthreads();
    locate_bin<false>(sh, top_p);
    // ordered bits of the new bin b: khi - o in [ceil(b*R/BINS), ceil((b+1)*R/BINS) - 1]
    const unsigned long long b = sh.bin;
    const unsigned long long d_lo = (b * R + BINS - 1) / BINS;
    const unsigned long long d_hi = ((b + 1) * R + BINS - 1) / BINS - 1;
    const unsigned nkhi = khi - (unsigned)d_lo;
    const unsigned nklo = khi - (unsigned)(d_hi > (unsigned long long)(khi - klo) ? (khi - klo) : d_hi);
    const unsigned old_hi = khi;
    count_and_collect(
        [&](float v) {
          const unsigned o = ordered_bits(v);
          return (o > nkhi && o <= old_hi) ? -1 : ((o >= nklo && o <= nkhi) ? 0 : 1);
        },
        std::false_type{});
    khi = nkhi;
    klo = nklo;
    __syncthreads();
  }

  const unsigned bin_cnt = sh.bin_cnt;
  auto finish_bits = [&]() {
    if (bits_partial)
      add_member_bits(bin_cnt);
    else
      write_all_bits();
  };
  if (bin_cnt == 0) {   // unreachable (the crossing bin has mass, hence members); kept so that no path leaves the outputs unset
    if (tid == 0) {
      sh.cut = ~0ull;
      cut[row] = ~0ull;
      count[row] = sh.n_above;
    }
    finish_bits();
    return;
  }
  if (bin_cnt <= (unsigned)CAP) {
    // rank the members of the crossing bin (they are in cand[0 .. bin_cnt)) and walk their masses
    if (bin_cnt <= 64u) {
      // few members (the usual case): the first wave holds one each, ranks them by counting (the keys are
      // distinct), orders their masses by rank through LDS and finds the crossing with a prefix over its lanes
      if (tid < 64) {
        const int n = (int)bin_cnt;
        const unsigned long long key = tid < n ? sh.cand[tid] : 0ull;
        int rank = 0;
        for (int j = 0; j < n; j++) rank += of_lane(key, j) > key ? 1 : 0;
        if (tid < n) {
          sh.mass[rank] = weight_of(from_ordered((unsigned)(key >> 32)), rmax);
          sh.mass[64 + rank] = key;
        }
        const unsigned long long inc = lane_prefix(tid < n ? sh.mass[tid] : 0ull);   // (same wave: LDS accesses complete in order)
        const unsigned long long reached = __ballot(tid < n && sh.mass_above + inc >= sh.target);
        const int idx = reached ? __ffsll((long long)reached) - 1 : n - 1;   // (the last one if the masses fell short)
        if (tid == idx) {
          const unsigned long long c = sh.mass[64 + idx];
          sh.cut = c;
          cut[row] = c;
          count[row] = sh.n_above + (unsigned)idx + 1u;
        }
      }
      finish_bits();
      return;
    }
    int n2 = 128;
    while (n2 < (int)bin_cnt) n2 <<= 1;
    for (int i = (int)bin_cnt + tid; i < n2; i += THREADS) sh.cand[i] = 0ull;
    __syncthreads();
    sort_candidates<THREADS>(sh, n2);
    // first position where mass_above + (masses of cand[0..position]) reaches the target: every thread owns
    // CAP / THREADS consecutive candidates, a prefix over the threads names the owner of the crossing
    constexpr int PER = CAP / THREADS;
    const unsigned long long target = sh.target, base = sh.mass_above;
    const int lastc = (int)bin_cnt - 1;
    unsigned long long local = 0;
    for (int i = 0; i < PER; i++) {
      const int idx = tid * PER + i;
      if (idx <= lastc) local += weight_of(from_ordered((unsigned)(sh.cand[idx] >> 32)), rmax);
    }
    unsigned long long em;
    unsigned long long all;
    block_exclusive_mass(sh, local, &em, &all);
    const unsigned long long lo = base + em;
    // (the second clause names the last candidate if the masses fell short of the target, the third the first
    // one if the target was already reached; neither happens with a consistent histogram)
    const bool mine = (lo < target && (target <= lo + local || tid == lastc / PER)) || (tid == 0 && target <= lo);
    if (mine && tid * PER <= lastc) {
      unsigned long long run = lo;
      int idx = tid * PER;
      const int stop = min(lastc, tid * PER + PER - 1);
      while (idx < stop) {
        run += weight_of(from_ordered((unsigned)(sh.cand[idx] >> 32)), rmax);
        if (run >= target) break;
        idx++;
      }
      sh.cut = sh.cand[idx];
      cut[row] = sh.cand[idx];
      count[row] = sh.n_above + (unsigned)idx + 1u;
    }
    finish_bits();
    return;
  }

  // A run of more than CAP equal scores contains the crossing: all of them weigh the same, so the number
  // to keep follows by division, and they are taken in ascending id.
  const float v_eq = from_ordered(klo);
  const unsigned long long w_eq = weight_of(v_eq, rmax);
  unsigned long long need = sh.target > sh.mass_above ? sh.target - sh.mass_above : 1ull;
  unsigned long long t_keep = w_eq > 0 ? (need + w_eq - 1) / w_eq : (unsigned long long)bin_cnt;
  if (t_keep < 1) t_keep = 1;
  if (t_keep > bin_cnt) t_keep = bin_cnt;
  unsigned run = 0;   // members seen in the chunks before this one (the same in every thread)
  const int last4 = (G - 1) & ~3;
  f32x4 next = *reinterpret_cast<const f32x4*>(s + min(tid * 4, last4));
  for (int base = 0; base < G && (unsigned long long)run < t_keep; base += THREADS * 4) {
    const int j4 = base + tid * 4;
    const f32x4 v = next;
    next = *reinterpret_cast<const f32x4*>(s + min(j4 + THREADS * 4, last4));
    bool in[4];
#pragma unroll
    for (int e = 0; e < 4; e++) in[e] = j4 + e < G && ordered_bits(v[e]) == klo;
    unsigned total;
    unsigned pos = run + block_exclusive<THREADS>((unsigned)in[0] + in[1] + in[2] + in[3], sh.wave_tot, &total);
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (in[e] && (unsigned long long)(++pos) == t_keep) {
        sh.cut = rank_key(v_eq, j4 + e);
        cut[row] = rank_key(v_eq, j4 + e);
        count[row] = sh.n_above + (unsigned)t_keep;
      }
    run += total;
  }
  write_all_bits();   // (this path is only reached through the narrowing rounds)
}

// Selection for one query block; called by all threads of the workgroup.  One pass for the mass of the row and its histogram
// over the score range, then rank_row.
template <int THREADS, int BINS, int CAP, int DEPTH, typename SH>
__device__ __forceinline__ void select_row(SH& sh, const float* s, int64_t row, float rmax, float rmin, int G, float top_p,
                                           unsigned long long* cut, unsigned* count, uint32_t* keep_bits, int Gw) {
  const float inv = bins_per_score<BINS>(rmax, rmin);
  for (int i = threadIdx.x; i < BINS; i += THREADS) sh.mass[i] = 0;
  __syncthreads();
  for_each_score<THREADS, DEPTH>(s, G, [&](float v, int) { atomicAdd(&sh.mass[value_bin_of<BINS>(v, rmax, inv)], weight_of(v, rmax)); });
  __syncthreads();
  locate_bin<true>(sh, top_p);
  rank_row<THREADS, BINS, CAP, DEPTH>(sh, s, row, rmax, place_by_bin<BINS>(sh.bin, rmax, inv), G, top_p, cut, count, keep_bits, Gw);
}

// Row `local` of a chunk's score buffer that starts at score tile unit0: the (slice, query block) row it holds, or
// -1 for the unused rows of a slice's last tile.
__device__ __forceinline__ int64_t chunk_row(int64_t local, int unit0, int YT, int QB) {
  const int unit = unit0 + (int)(local >> 7);
  const int slice = unit / YT;
  const int qb = (unit - slice * YT) * 128 + (int)(local & 127);
  return qb < QB ? (int64_t)slice * QB + qb : -1;
}

// One workgroup per query block, rows read from device memory in every pass.
template <int THREADS, int BINS, int CAP>
__global__ void __launch_bounds__(THREADS) select_kernel(const float* scores, const unsigned* range, int unit0, int YT, int QB,
                                                         int G, int Gs, float top_p, unsigned long long* cut, unsigned* count,
                                                         uint32_t* keep_bits, int Gw) {
  __shared__ SelShared<THREADS, BINS, CAP> sh;
  const int64_t local = blockIdx.x;
  const int64_t row = chunk_row(local, unit0, YT, QB);
  if (row < 0) return;
  select_row<THREADS, BINS, CAP, 4>(sh, scores + local * Gs, row, from_ordered(range[2 * row]),
                                        from_ordered(range[2 * row + 1]), G, top_p, cut, count, keep_bits, Gw);
}

// Rows of at most MAXROW scores: the row is read from device memory ONCE.  That pass builds the mass histogram and leaves, in
// LDS, a byte per score: its bin divided by four.  The second pass works on the bytes alone, sixteen per lane and step: a
// smaller byte than the crossing bin's keeps the key block, an equal one makes it a member.  The members fetch their scores
// again by id; those above the crossing bin are kept, those in it are ranked.  The row's bits replace the bytes in LDS as
// they are read, so members add theirs with LDS atomics and the row of bits is written once.
// Bound: the first pass's vector instructions and LDS atomics (one 64-bit addition per score) and the latencies of the short
// phases between barriers, so what matters is how many waves a compute unit holds; bytes (16-bit bins before) let three
// workgroups of 512 threads share one for rows of up to 32768 scores instead of two, and let rows of up to 131072 in at all
// (before, they were read from memory in every pass).  Against select_kernel, which does that: 1024 rows of 32760 51 -> 36 us, 469 of
// 60000 61 -> 35, 782 of 100000 172 -> 132, 10240 of 2048 77 -> 52; fewer short rows, whose scores stay in the caches, are
// slower: 1764 of 9360 35 -> 47, 2560 of 4096 25 -> 31.  (The histogram's atomics are not what binds: without seven eighths of them it
// is no faster.)  Too many members for LDS are rare (many equal scores): such a row goes on from its histogram as in select_kernel,
// after the other rows (1024 rows of 32760 equal scores 217 us, there 202; 10240 of 2048 211 and 1814).  A launch of its own, which
// started those rows over, cost every call 2 us.
template <int THREADS, int MAXROW, int IDCAP, typename ID>
struct alignas(16) CodesShared {
  static constexpr int CAND = IDCAP * sizeof(ID) / 8;
  SelShared<THREADS, kRowBins, CAND> sel;   // (the ranked keys reuse the histogram's memory, the members' ids lie in sel.cand)
  alignas(16) uint32_t codes[MAXROW / 4];
};

template <int THREADS, int MAXROW, int IDCAP, typename ID, int WAVES_PER_SIMD>
__global__ void __launch_bounds__(THREADS, WAVES_PER_SIMD)
select_codes_kernel(const float* scores, const unsigned* range, int64_t chunk_rows, int unit0, int YT, int QB, int G, int Gs,
                    float top_p, unsigned long long* cut, unsigned* count, uint32_t* keep_bits, int Gw) {
  constexpr int BINS = kRowBins, CAP = THREADS;   // one ranked member per thread
  static_assert(IDCAP % THREADS == 0 && CAP <= BINS && BINS == 4 * 256 && MAXROW % 1024 == 0 && (sizeof(ID) > 2 || MAXROW <= 65536), "layout");
  __shared__ CodesShared<THREADS, MAXROW, IDCAP, ID> shm;
  auto& sh = shm.sel;
  unsigned long long* const keys = sh.mass;
  ID* const ids = reinterpret_cast<ID*>(sh.cand);
  bool left = false;   // some row had too many members
  for (int64_t local = blockIdx.x; local < chunk_rows; local += gridDim.x) {
    const int64_t row = chunk_row(local, unit0, YT, QB);
    if (row < 0) continue;   // (the same for all threads)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (what follows from the thread's number is formed anew for every row: kept, it spills)
    const float* s = scores + local * Gs;
    const float rmax = from_ordered(range[2 * row]), rmin = from_ordered(range[2 * row + 1]);
    uint32_t* const bits_row = keep_bits + row * Gw;
    const float inv = bins_per_score<BINS>(rmax, rmin);
    auto value_bin = [&](float v) -> unsigned { return value_bin_of<BINS>(v, rmax, inv); };
    __syncthreads();   // the row before this one is done with the shared state
    for (int i = tid; i < BINS; i += THREADS) sh.mass[i] = 0;
    if (tid == 0) {
      sh.ncand = 0;
      sh.bin_cnt = 0;
    }
    __syncthreads();

    // pass 1: four consecutive scores per thread and step, DEPTH steps in flight while DEPTH are processed.  The loads are
    // unconditional, 16 bytes of the row's padding or of its last scores again past the end (with a test around them the
    // compiler makes four 4-byte loads and four branches of each, and it takes a fifth more time).
    {
      constexpr int STEP = THREADS * 4, DEPTH = WAVES_PER_SIMD > 4 ? 2 : 4;
      auto one = [&](float v) -> unsigned {
        const unsigned b = value_bin(v);
        atomicAdd(&sh.mass[b], weight_of(v, rmax));
        return b;
      };
      auto store4 = [&](unsigned b0, unsigned b1, unsigned b2, unsigned b3, int j4) {
        const unsigned b01 = (b0 | (b1 << 16)) >> 2, b23 = (b2 | (b3 << 16)) >> 2;   // bytes 0 and 2 are the codes
        shm.codes[j4 >> 2] = __builtin_amdgcn_perm(b23, b01, 0x06040200u);
      };
      const int last4 = (G - 1) & ~3;   // the last four scores, or what is left of them
      auto load4 = [&](f32x4 (&x)[DEPTH], int j0) {
#pragma unroll
        for (int e = 0; e < DEPTH; e++) x[e] = *reinterpret_cast<const f32x4*>(s + min(j0 + e * STEP, last4));
      };
      f32x4 cur[DEPTH], nxt[DEPTH];
      load4(cur, tid * 4);
#pragma unroll 1
      for (int base = 0; base < G; base += DEPTH * STEP) {
        load4(nxt, base + DEPTH * STEP + tid * 4);
#pragma unroll
        for (int e = 0; e < DEPTH; e++) {
          const int j4 = base + e * STEP + tid * 4;
          if (base + (e + 1) * STEP <= G) {   // (the same in all threads)
            const unsigned b0 = one(cur[e][0]), b1 = one(cur[e][1]), b2 = one(cur[e][2]), b3 = one(cur[e][3]);
            store4(b0, b1, b2, b3, j4);
          } else if (j4 < G) {
            unsigned b[4] = {0u, 0u, 0u, 0u};   // (codes of positions past the end are never looked at)
#pragma unroll
            for (int i = 0; i < 4; i++)
              if (j4 + i < G) b[i] = one(cur[e][i]);
            store4(b[0], b[1], b[2], b[3], j4);
          }
        }
#pragma unroll
        for (int e = 0; e < DEPTH; e++) cur[e] = nxt[e];
      }
    }
    __syncthreads();
    locate_bin<true>(sh, top_p);

    // pass 2: sixteen codes per lane and step.  Per word of four, high bit of byte e: `less` says code e is below the crossing
    // one (by the subtraction of the low seven bits, which cannot borrow, and the high bits), `same` that it is equal; a dot
    // product with 1, 2, 4, 8 gathers the four bits.
    const unsigned fine = sh.bin, code = fine >> 2;
    unsigned n_codes;   // key blocks with a smaller code
    {
      constexpr unsigned H = 0x80808080u;
      const unsigned c4 = code * 0x01010101u, c4low = c4 & ~H, c_small = code < 128u ? ~0u : 0u;
      unsigned na = 0;
#pragma unroll 1
      for (int base = 0; base < G; base += THREADS * 16) {
        const int j16 = base + tid * 16;
        if (base + (tid & ~63) * 16 >= G) break;   // (the same in all lanes of a wave)
        const int left = G - j16;   // codes of this lane inside the row
        unsigned keep = 0, member = 0;
        if (left > 0) {
          const uint4 w4 = *reinterpret_cast<const uint4*>(&shm.codes[j16 >> 2]);
          const unsigned w[4] = {w4.x, w4.y, w4.z, w4.w};
          unsigned below[2] = {0u, 0u}, equal[2] = {0u, 0u};   // eight codes each, shifted left by seven
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const unsigned t = (w[r] | H) - c4low;
            const unsigned less = ~((t & (w[r] | c_small)) | (w[r] & c_small)) & H;
            const unsigned z = w[r] ^ c4;
            const unsigned same = ~(((z & ~H) + ~H) | z) & H;
            const unsigned weights = r & 1 ? 0x80402010u : 0x08040201u;
            below[r >> 1] = __builtin_amdgcn_udot4(less, weights, below[r >> 1], false);
            equal[r >> 1] = __builtin_amdgcn_udot4(same, weights, equal[r >> 1], false);
          }
          const unsigned inside = left >= 16 ? 0xFFFFu : (1u << left) - 1u;
          keep = ((below[0] >> 7) | (below[1] << 1)) & inside;
          member = ((equal[0] >> 7) | (equal[1] << 1)) & inside;
        }
        na += (unsigned)__popc(keep);
        unsigned word = keep << (16 * (tid & 1));
        word |= __shfl_xor(word, 1);
        // the word takes the place of the codes it stands for: every lane has read its own, and no other lane reads these
        if ((tid & 1) == 0 && left > 0) shm.codes[j16 >> 2] = word;
        if (__builtin_amdgcn_ballot_w64(member != 0u) != 0) {
          // places for the members of the whole wave with one atomic; a lane's own follow those of the lanes below it
          const unsigned m = (unsigned)__popc(member);
          unsigned pos = 0, all = 0;
#pragma unroll
          for (int b = 0; b < 5; b++) {   // (a count of at most 16, bit by bit)
            const uint64_t lanes = __builtin_amdgcn_ballot_w64((m >> b) & 1u);
            pos += __builtin_amdgcn_mbcnt_hi((unsigned)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)lanes, 0u)) << b;
            all += (unsigned)__popcll(lanes) << b;
          }
          unsigned first = 0;
          if ((tid & 63) == 0) first = atomicAdd(&sh.ncand, all);
          pos += (unsigned)__builtin_amdgcn_readfirstlane((int)first);
#pragma unroll 1
          while (member != 0u) {
            if (pos < (unsigned)IDCAP) ids[pos] = (ID)(j16 + __ffs(member) - 1);
            pos++;
            member &= member - 1;
          }
        }
      }
      n_codes = (unsigned)block_sum_u64(sh, (unsigned long long)na);   // (its barriers also order the bits and the ids)
    }
    const unsigned n_ids = sh.ncand;   // (read by all threads after the barriers of the sum)
    auto keep_bit = [&](unsigned id) { atomicOr(&shm.codes[(id >> 5) * 8], 1u << (id & 31)); };
    // members: above the crossing bin, in it (their rank keys are collected), or below it
    unsigned more = 0;
    if (n_ids <= (unsigned)IDCAP) {
      // (four scores of a thread in flight at once: one after the other, a row of 118800 with its 2000 members waits for
      // device memory three times)
      constexpr int PER = 4;
      static_assert(IDCAP % (PER * THREADS) == 0, "whole steps");
#pragma unroll 1
      for (unsigned base = 0; base < n_ids; base += PER * THREADS) {
        unsigned id[PER];
        float v[PER];
#pragma unroll
        for (int e = 0; e < PER; e++) id[e] = min((unsigned)ids[base + e * THREADS + tid], (unsigned)(G - 1));
#pragma unroll
        for (int e = 0; e < PER; e++)
          if (base + e * THREADS < n_ids) v[e] = s[id[e]];   // (the same in all threads)
#pragma unroll
        for (int e = 0; e < PER; e++) {
          if (base + e * THREADS + tid >= n_ids) continue;
          const unsigned b = value_bin(v[e]);
          if (b < fine) {
            keep_bit(id[e]);
            more++;
          } else if (b == fine) {
            const unsigned pos = atomicAdd(&sh.bin_cnt, 1u);
            if (pos < (unsigned)CAP) keys[pos] = rank_key(v[e], (int)id[e]);   // (the histogram is not needed any more)
          }
        }
      }
    }
    const unsigned n_above = n_codes + (unsigned)block_sum_u64(sh, (unsigned long long)more);
    const unsigned n = sh.bin_cnt;
    if (n_ids > (unsigned)IDCAP || n > (unsigned)CAP) {
      // too many members: the row goes on from its histogram below.  (A row that is done keeps at least one key block; the
      // state waits in the row's own bits, eight words at least here: a row that short has no more members than fit.)
      left = true;
      if (tid == 0) {
        count[row] = 0u;
        bits_row[0] = sh.bin;
        bits_row[1] = (uint32_t)sh.mass_above;
        bits_row[2] = (uint32_t)(sh.mass_above >> 32);
        bits_row[3] = (uint32_t)sh.target;
        bits_row[4] = (uint32_t)(sh.target >> 32);
      }
      continue;
    }
    // rank by counting (the keys are distinct), keys ordered by rank, crossing by a prefix of their masses over the threads.
    // As many threads as there are share the counting for a key, each over its part of the keys (with that and the members'
    // scores fetched together, rows of 118800 take 371 us per GiB of scores, 378 before).
    const unsigned long long key = tid < (int)n ? keys[tid] : 0ull;
    unsigned* const ranks = reinterpret_cast<unsigned*>(sh.cand);   // (the ids are not needed any more)
    static_assert(sizeof(sh.cand) >= THREADS * sizeof(unsigned), "a rank per thread");
    if (tid >= (int)n && tid < (((int)n + 7) & ~7)) keys[tid] = 0ull;   // (zeros up to a multiple of eight: below every key)
    ranks[tid] = 0u;
    __syncthreads();
    {
      const unsigned slots = max((n + 63u) & ~63u, 64u), parts = (unsigned)THREADS / slots;
      const unsigned part = (unsigned)tid / slots, slot = (unsigned)tid - part * slots;
      const unsigned per = (((n + 7u) >> 3) + parts - 1u) / parts * 8u;
      if (part < parts && slot < n) {
        const unsigned long long ranked = keys[slot];
        unsigned rank = 0;
#pragma unroll 1
        for (unsigned j = part * per; j < min(part * per + per, n); j += 8) {   // eight keys per step: four 16-byte reads in flight
          unsigned long long o[8];
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const ulonglong2 two = *reinterpret_cast<const ulonglong2*>(&keys[j + e]);
            o[e] = two.x;
            o[e + 1] = two.y;
          }
#pragma unroll
          for (int e = 0; e < 8; e++) rank += o[e] > ranked ? 1u : 0u;
        }
        if (rank != 0u) atomicAdd(&ranks[slot], rank);
      }
    }
    __syncthreads();   // all keys read: the ordered ones go back
    if (tid < (int)n) keys[ranks[tid]] = key;
    __syncthreads();
    {
      const unsigned long long mine = tid < (int)n ? keys[tid] : 0ull;
      const unsigned long long w = tid < (int)n ? weight_of(from_ordered((unsigned)(mine >> 32)), rmax) : 0ull;
      unsigned long long before, all;
      block_exclusive_mass(sh, w, &before, &all);
      const unsigned long long target = sh.target, base = sh.mass_above;
      // the first member at which the running mass reaches the target; the last one if the masses fell short (they do
      // not with a consistent histogram)
      const bool here = tid < (int)n && ((base + before < target && base + before + w >= target) ||
                                         (tid == (int)n - 1 && base + before + w < target) || (tid == 0 && base >= target));
      if (here) {
        sh.cut = mine;
        cut[row] = mine;
        count[row] = n_above + (unsigned)tid + 1u;
      }
      if (n == 0 && tid == 0) {   // unreachable (the crossing bin has mass, hence members); no output is left unset
        sh.cut = ~0ull;
        cut[row] = ~0ull;
        count[row] = n_above;
      }
    }
    __syncthreads();
    if (tid < (int)n && key >= sh.cut) keep_bit(0xFFFFFFFFu - (unsigned)key);
    __syncthreads();
#pragma unroll 1
    for (int wi = tid; wi < Gw; wi += THREADS) bits_row[wi] = shm.codes[wi * 8];
  }
  if (!left) return;   // (the same in all threads)
  // (a loop of its own: inside the one above, this path costs the usual one its registers)
  for (int64_t local = blockIdx.x; local < chunk_rows; local += gridDim.x) {
    const int64_t row = chunk_row(local, unit0, YT, QB);
    if (row < 0) continue;
    __syncthreads();   // the row before this one is done with the shared state; this one's words have been written
    if (count[row] != 0u) continue;
    const uint32_t* const state = keep_bits + row * Gw;
    if (threadIdx.x == 0) {
      sh.bin = state[0];
      sh.mass_above = state[1] | ((unsigned long long)state[2] << 32);
      sh.target = state[3] | ((unsigned long long)state[4] << 32);
      sh.n_above = 0;
    }
    __syncthreads();
    const float rmax = from_ordered(range[2 * row]), rmin = from_ordered(range[2 * row + 1]);
    rank_row<THREADS, BINS, CodesShared<THREADS, MAXROW, IDCAP, ID>::CAND, 2>(
        sh, scores + local * Gs, row, rmax, place_by_bin<BINS>(sh.bin, rmax, bins_per_score<BINS>(rmax, rmin)), G, top_p, cut, count, keep_bits, Gw);
  }
}

// Kept ids in ascending order, from the bit rows that the selection leaves.  Bound: the writes of the ids (4 bytes each: for
// 24 x 929 rows of 118800, 5.6 GB of ids, 1.27 ms; without the stores the kernel takes 0.64).  A wave takes a stretch of one
// row, a byte of it (eight key blocks) per lane and step.  A table gives the places of a byte's set bits, a prefix over the
// lanes where a lane's ids begin, and the ids go next to each other into the wave's own piece of LDS.  From there whole
// 128-byte lines go to memory, past the caches (nothing reads them soon); what is left over waits for the next ids.  No
// barrier and no loop over bits.  (A bit per lane, with the words handed out through scalar registers, takes twice the
// instructions, and 16-byte groups leave lines in parts: 12 heads x 512 rows of 32760 73 -> 55 us, 24 x 929 rows of 118800
// 1490-1640 -> 1210-1270 us.  A loop over each lane's bits runs as long as the fullest lane's: 91 and 1510 us.  Stores
// straight from the lanes whose bit is set make as many requests as full ones.)
// The first batch of a longer stretch goes through the caches: past them too, all waves begin their rows in step, 6144 rows of
// 32760 with 88% kept 139 us instead of 126, 3072 of 16384 35.4 instead of 30.2.  Stretches of one batch go past them (16252 rows of 1016
// with 90% kept 11.2 us, through them 11.7).  Written id by id, as it once was, the first batch costs 127, 31.5 and 13.1.
constexpr int kEmitBatch = 32;   // words of a row staged between two flushes
__global__ void __launch_bounds__(256) emit_bits_kernel(const uint32_t* keep_bits, int Gw, int seg_words, int segs, int64_t units,
                                                        const int64_t* indptr, int32_t* indices, int64_t capacity) {
  __shared__ alignas(16) int32_t stages[4][kEmitBatch * 32 + 40];
  // of every byte, the places of its set bits, ascending, a byte each; the rest are zero
  __shared__ uint2 places[256];
  {
    uint64_t p = 0;
    int n = 0;
#pragma unroll
    for (int b = 0; b < 8; b++)
      if ((threadIdx.x >> b) & 1u) p |= (uint64_t)b << (8 * n++);
    places[threadIdx.x] = make_uint2((unsigned)p, (unsigned)(p >> 32));
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t unit = (int64_t)blockIdx.x * 4 + wv;
  if (unit >= units) return;
  const int64_t row = unit / segs;
  const int w0 = (int)(unit - row * segs) * seg_words, w1 = min(w0 + seg_words, Gw);
  if (w0 >= w1) return;   // (the last stretches may be empty: all others are of even length)
  int32_t* const stage = stages[wv];
  const uint32_t* const bits = keep_bits + row * Gw;
  uint32_t words = w0 + lane < w1 ? bits[w0 + lane] : 0u;   // 64 words of the row, one a lane, fetched one ahead of their use
  unsigned before = 0;   // kept key blocks of the row ahead of this stretch
  for (int w = lane; w < w0; w += 64) before += (unsigned)__popc(bits[w]);
  if (w0 > 0)
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
  const int64_t out = indptr[row] + (unsigned)__builtin_amdgcn_readfirstlane((int)before);
  // stage[i] goes to indices[to + i]; indices + to lies on a 128-byte line, so up to 31 slots at the start are no ids
  unsigned skip = (unsigned)((reinterpret_cast<uintptr_t>(indices + out) >> 2) & 31);
  int64_t to = out - skip;
  unsigned fill = skip, begins = 32;   // slots of the stretch's first line, until it has been written
  for (int w = w0; w < w1; w += 64) {
    asm volatile("" : "+v"(words));   // (waits for these words here, and for the stores before them: after the next load is under way, for that too)
    const uint32_t next = w + 64 + lane < w1 ? bits[w + 64 + lane] : 0u;
    for (int half = 0; half < 64 && w + half < w1; half += kEmitBatch) {
#pragma unroll
      for (int i = 0; i < kEmitBatch; i += 16) {   // sixteen words at a step, a byte per lane (words past the end are zero)
        const unsigned word = (unsigned)__builtin_amdgcn_ds_bpermute((half + i + (lane >> 2)) * 4, (int)words);
        const unsigned byte = (word >> (8 * (lane & 3))) & 0xFFu, count = (unsigned)__popc(byte);
        const uint2 p = places[byte];
        const unsigned incl = lane_prefix(count);
        auto* const at = (volatile __attribute__((address_space(3))) int32_t*)(stage + fill + (incl - count));   // (in the order written)
        const int id = (w + half + i) * 32 + lane * 8;
        // Eight ids a lane, the last one first: what a lane writes past its count lands on places of lanes above it, which write
        // them again in a later one of these instructions (a lane without ids writes none, so "above" is by one instruction
        // at least), or past the last id, where the next step begins.
        if (count != 0u) {
          at[7] = id | (int)(p.y >> 24);
          at[6] = id | (int)((p.y >> 16) & 0xFFu);
          at[5] = id | (int)((p.y >> 8) & 0xFFu);
          at[4] = id | (int)(p.y & 0xFFu);
          at[3] = id | (int)(p.x >> 24);
          at[2] = id | (int)((p.x >> 16) & 0xFFu);
          at[1] = id | (int)((p.x >> 8) & 0xFFu);
          at[0] = id | (int)(p.x & 0xFFu);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        fill += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
      }
      // whole groups to memory (LDS operations of a wave complete in order)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const unsigned whole = fill & ~31u;
      if (whole != 0u) {
        if (to + (int64_t)whole <= capacity) {
          if ((unsigned)lane >= skip && (unsigned)lane < begins) indices[to + lane] = stage[lane];   // (none past the first flush)
          if (begins != 0u && w1 - w0 > kEmitBatch) {
            for (unsigned i = begins + 4 * lane; i < whole; i += 256)
              *reinterpret_cast<i32x4*>(indices + to + i) = *reinterpret_cast<const i32x4*>(stage + i);
          } else {
            for (unsigned i = begins + 4 * lane; i < whole; i += 256)
              __builtin_nontemporal_store(*reinterpret_cast<const i32x4*>(stage + i), reinterpret_cast<i32x4*>(indices + to + i));
          }
        } else {   // the end of the buffer
          for (unsigned i = lane; i < whole; i += 64)
            if (i >= skip && to + i < capacity) indices[to + i] = stage[i];
        }
        const int rest = stage[whole + (lane & 31)];   // (up to 31 ids; the array has the slots to spare)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane < 32) stage[lane] = rest;
        to += whole;
        fill &= 31;
        skip = 0;
        begins = 0;
      }
    }
    words = next;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (lane < (int)fill && lane >= (int)skip && to + lane < capacity) indices[to + lane] = stage[lane];
}

}  // namespace fgm

#include "fgmask_short.hpp"
#include "fgmask_stream.hpp"

namespace fgm {

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
// The score buffer takes whole tiles of 128 query-block rows; as many tiles as fit kScoreBudget, at least one.
constexpr size_t kScoreBudget = (size_t)1 << 30;

struct Layout {
  int64_t rows, QB, G, Gs, Gw, slices;
  int64_t YT, units, chunk_units;   // score tiles per slice, in all, and per chunk
  bool row_in_lds;   // rows of scores fit the LDS-row selection kernel
  size_t qp_off, kp_off, scores_off, cut_off, count_off, range_off, bits_off, total;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static int layout_of(const fgattn_params* p, Layout* lo) {
  if (p == nullptr) return FGATTN_E_NULL;
  if (p->B < 1 || p->H < 1 || p->L < 1 || p->N < 1) return FGATTN_E_SHAPE;
  if (p->d != 64 && p->d != 128) return FGATTN_E_SHAPE;
  if (p->M != 16 && p->M != 32 && p->M != 64 && p->M != 128) return FGATTN_E_SHAPE;
  if (p->L > (1 << 24)) return FGATTN_E_SHAPE;
  if (p->flags & ~31) return FGATTN_E_FLAGS;
  lo->slices = (int64_t)p->B * p->H;
  lo->QB = ((int64_t)p->L + p->M - 1) / p->M;
  lo->G = ((int64_t)p->L + p->N - 1) / p->N;
  lo->Gs = (lo->G + 31) & ~(int64_t)31;   // rows start on 128-byte lines
  lo->Gw = (lo->G + 31) / 32;
  lo->row_in_lds = lo->Gs <= kRowCodesMax && !(p->flags & FGATTN_FLAG_MASK_ROWS_IN_HBM);
  lo->rows = lo->slices * lo->QB;
  if (lo->rows > 0x7fffffffLL || lo->slices > 65535) return FGATTN_E_SHAPE;
  lo->YT = (lo->QB + 127) / 128;
  lo->units = lo->slices * lo->YT;
  const size_t tile_bytes = (size_t)128 * lo->Gs * 4;
  lo->chunk_units = (p->flags & FGATTN_FLAG_MASK_ONE_TILE_CHUNKS) ? 1 : (int64_t)(kScoreBudget / tile_bytes);
  if (lo->chunk_units < 1) lo->chunk_units = 1;
  if (lo->chunk_units > 65535) lo->chunk_units = 65535;   // (bounds the grids of a chunk whose rows are short)
  if (lo->chunk_units > lo->units) lo->chunk_units = lo->units;
  size_t off = 0;
  lo->qp_off = off;
  off = align256(off + (size_t)lo->rows * p->d * 2);
  lo->kp_off = off;
  if (p->N > 1 || p->B > 1) off = align256(off + (size_t)lo->slices * lo->G * p->d * 2);   // else K is read in place
  lo->scores_off = off;
  off = align256(off + (size_t)lo->chunk_units * tile_bytes);
  lo->cut_off = off;
  off = align256(off + (size_t)lo->rows * 8);
  lo->count_off = off;
  off = align256(off + (size_t)lo->rows * 4);
  lo->range_off = off;
  off = align256(off + (size_t)lo->rows * 8);
  lo->bits_off = off;
  off = align256(off + (size_t)lo->rows * lo->Gw * 4);
  lo->total = off;
  return FGATTN_OK;
}

// gfx950 or an error; *cus (if given) gets the number of compute units
static int device_ok(int* cus = nullptr) {
  static int known[64];   // 0 unknown, 1 gfx950, 2 other
  static int units[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return FGATTN_E_DEVICE;
  if (known[dev] == 0) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return FGATTN_E_DEVICE;
    units[dev] = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
    known[dev] = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : 2;
  }
  if (cus) *cus = units[dev];
  return known[dev] == 1 ? FGATTN_OK : FGATTN_E_DEVICE;
}

static bool launched() { return hipGetLastError() == hipSuccess; }

// Lays out the score buffer (`bytes` at `at`) for the selection without scores (fgmask_stream.hpp), in chunks of whole
// slices.  False where it does not fit, or where the selection from scores is the better one: with few scores the six kernels
// of a chunk are mostly set-up, the more so at head dim 128, where a score takes twice the matrix work, and with few rows, whose
// histograms are the same keys' work for less.  A histogram has to be worth its setting up for 64 rows, too.  The line, in units of
// 2^20 scores, between measured pairs (select call, us, from scores / without, masks of video-like and of random scores):
//   d = 64, from 2048 rows on   48: 2816 x 16384 (44) 95 / 96 and 98 / 105; 3328 x 16384 (52) 125 / 99 and 129 / 111
//           from 1024 rows on   54: 1875 x 30000 (53.6) 102 / 101 and 107 / 118; 1641 x 35000 (54.8) 132 / 110 and 146 / 129
//           below               72: 750 x 96000 (68.7) 163 / 168 and 176 / 196; 782 x 100000 (74.6) 209 / 173 and 222 / 204
//   d = 128, from 1024 rows on  72: 1470 x 47000 (65.9) 151 / 156 and 160 / 177; 1548 x 49500 (73.1) 184 / 166 and 192 / 187
//            below              96: 860 x 110000 (90.2) 242 / 241 and 259 / 272; 891 x 114000 (96.9) 261 / 245 and 280 / 277
static int64_t stream_min_scores(int d, int64_t rows) {
  const int64_t mi = d == 128 ? (rows < 1024 ? 96 : 72) : rows < 1024 ? 72 : rows < 2048 ? 54 : 48;
  return mi << 20;
}
constexpr int64_t kStreamMinRow = 2048;

static bool plan_stream(const Layout& lo, int d, char* at, size_t bytes, int cus, StreamArgs* a) {
  if (lo.G < kStreamMinRow || lo.rows * lo.G < stream_min_scores(d, lo.rows)) return false;
  const int64_t ktiles = (lo.G + 31) / 32, per_slice = (lo.QB + kSweepRows - 1) / kSweepRows, tiles = (lo.QB + kMassRows - 1) / kMassRows;
  a->steps = (int)((ktiles + kMassWaves - 1) / kMassWaves);
  for (int64_t chunks = 1; chunks <= lo.slices; chunks++) {
    const int64_t slices = (lo.slices + chunks - 1) / chunks, units = slices * per_slice, rows = slices * lo.QB;
    // sweep: one round of the three workgroups that a compute unit holds, if the rows allow; lists for an eighth of a stretch's
    // key blocks (about one in a hundred is a member)
    int64_t segs = (3 * (int64_t)cus + units - 1) / units;
    if (segs > 64) segs = 64;
    int64_t seg_tiles = ((ktiles + segs - 1) / segs + 3) & ~(int64_t)3;
    if (seg_tiles < 16) seg_tiles = 16;
    segs = (ktiles + seg_tiles - 1) / seg_tiles;
    // (A wave settles 64 lists; a list's places have 16 bits.  Many query blocks make few stretches, of more tiles than that: fewer slices
    // in a chunk then make more.)
    if (segs > 64 || seg_tiles > 2047) continue;
    const int64_t cap = seg_tiles * 32 / 8;
    // mass: one workgroup fits a compute unit; setting up a row tile and leaving its histogram cost it about six steps
    const int64_t most = cus & ~7;
    int64_t pieces = 1, turn = 1, least = INT64_MAX;
    for (int64_t n = 1; n <= 8 && n <= a->steps; n++) {
      const int64_t m = (slices * tiles * n + most - 1) / most, cost = m * ((a->steps + n - 1) / n) + 6 * (1 + (m + n - 1) / n);
      if (cost < least) {
        least = cost;
        pieces = n;
        turn = m;
      }
    }
    const int64_t groups = ((slices * tiles * pieces + turn - 1) / turn + 7) & ~(int64_t)7;
    size_t off = 256;
    const size_t cuts = off;
    off = align256(off + (size_t)rows * sizeof(RowCut));
    const size_t hist = off;
    off = align256(off + (size_t)(groups + slices * tiles) * kMassWords * 8);
    const size_t counts = off;
    off = align256(off + (size_t)(rows * segs) * sizeof(uint2));
    const size_t lists = off;
    off = align256(off + (size_t)(rows * segs * cap) * sizeof(Member));
    if (off > bytes) continue;
    a->slices = (int)slices;
    a->units = (int)units;
    a->segs = (int)segs;
    a->seg_tiles = (int)seg_tiles;
    a->tiles = (int)(slices * tiles);
    a->pieces = (int)pieces;
    a->turn = (int)turn;
    a->groups = (int)groups;
    a->cap = (int)cap;
    a->overfull = reinterpret_cast<unsigned*>(at);
    a->hist = reinterpret_cast<unsigned long long*>(at + hist);
    a->cuts = reinterpret_cast<RowCut*>(at + cuts);
    a->counts = reinterpret_cast<uint2*>(at + counts);
    a->lists = reinterpret_cast<Member*>(at + lists);
    return true;
  }
  return false;
}

template <int D>
static bool launch_stream(StreamArgs a, const Layout& lo, int cus, hipStream_t stream) {
  const int64_t per_slice = (lo.QB + kSweepRows - 1) / kSweepRows, tiles = (lo.QB + kMassRows - 1) / kMassRows;
  const int step = a.slices;
  for (int64_t slice0 = 0; slice0 < lo.slices; slice0 += step) {
    a.slice0 = (int)slice0;
    a.slices = (int)(lo.slices - slice0 < step ? lo.slices - slice0 : step);
    a.units = (int)(a.slices * per_slice);
    a.tiles = (int)(a.slices * tiles);
    const dim3 sweep((unsigned)((a.segs < 8 ? a.segs : (a.segs + 7) & ~7) * a.units));
    hipLaunchKernelGGL((sweep_kernel<D, false>), sweep, dim3(256), 0, stream, a);
    if (!launched()) return false;
    hipLaunchKernelGGL(mass_kernel<D>, dim3(a.groups), dim3(kMassWaves * 64), 0, stream, a);
    if (!launched()) return false;
    hipLaunchKernelGGL(locate_kernel, dim3(2 * a.tiles), dim3(kLocateParts * 32), 0, stream, a);
    if (!launched()) return false;
    hipLaunchKernelGGL((sweep_kernel<D, true>), sweep, dim3(256), 0, stream, a);
    if (!launched()) return false;
    const int64_t rows = (int64_t)a.slices * lo.QB, waves = (rows + 3) / 4;
    hipLaunchKernelGGL(settle_kernel, dim3((unsigned)(waves < 8 * cus ? waves : 8 * cus)), dim3(256), 0, stream, a);
    if (!launched()) return false;
    // One workgroup to a compute unit, 32 rows each where that is enough of them: rows of two values and crowded rows take, of 32 / of 8,
    // 0.32 / 0.40 and 0.53 / 0.55 ms with 65 workgroups of 32 (2063 rows of 33000, d = 64), 0.39 / 0.49 and 0.60 / 0.69 with 90 (3 x 938 of
    // 30000), 0.50 / 0.61 and 1.07 / 0.90 with 128 (8 x 512 of 32760), 0.63 / 0.89 and 1.17 / 1.28 with 192, but 1.01 / 0.85 and
    // 2.69 / 1.25 with 30 (929 of 118800).
    auto overfull = [&](auto rows) {
      int64_t over = a.slices * ((lo.QB + rows - 1) / rows);
      if (over > cus) over = cus;
      hipLaunchKernelGGL((overfull_kernel<D, decltype(rows)::value>), dim3((unsigned)((over + 7) & ~(int64_t)7)), dim3(kOverfullThreads), 0, stream, a);
    };
    if (a.slices * ((lo.QB + 31) / 32) >= cus / 4) overfull(std::integral_constant<int, 32>());
    else overfull(std::integral_constant<int, 8>());
    if (!launched()) return false;
  }
  return true;
}

}  // namespace fgm

extern "C" {

size_t fgattn_mask_workspace_bytes(const fgattn_params* p) {
  fgm::Layout lo;
  if (fgm::layout_of(p, &lo) != FGATTN_OK) return 0;
  return lo.total;
}

int fgattn_mask_select(const void* q, const void* k, const fgattn_params* p, float top_p, int64_t* mask_indptr,
                       void* workspace, size_t workspace_bytes, void* stream_v) {
  using namespace fgm;
  Layout lo;
  int rc = layout_of(p, &lo);
  if (rc) return rc;
  if (!q || !k || !mask_indptr || !workspace) return FGATTN_E_NULL;
  if (!(top_p > 0.0f) || !(top_p <= 1.0f) || !isfinite(p->scale)) return FGATTN_E_SCALE;
  if ((reinterpret_cast<uintptr_t>(q) & 15) || (reinterpret_cast<uintptr_t>(k) & 15) ||
      (reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(mask_indptr) & 7))
    return FGATTN_E_ALIGN;
  const int64_t strides[6] = {p->q_stride_b, p->q_stride_h, p->q_stride_l, p->k_stride_b, p->k_stride_h, p->k_stride_l};
  for (int i = 0; i < 6; i++)
    if (strides[i] < 0 || (strides[i] % 8) != 0) return FGATTN_E_STRIDE;
  if (p->q_stride_l < p->d || p->k_stride_l < p->d) return FGATTN_E_STRIDE;
  if (workspace_bytes < lo.total) return FGATTN_E_WORKSPACE;
  int cus = 1;
  rc = device_ok(&cus);
  if (rc) return rc;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  char* ws = static_cast<char*>(workspace);
  uint16_t* qp = reinterpret_cast<uint16_t*>(ws + lo.qp_off);
  uint16_t* kp = reinterpret_cast<uint16_t*>(ws + lo.kp_off);
  float* scores = reinterpret_cast<float*>(ws + lo.scores_off);
  unsigned long long* cut = reinterpret_cast<unsigned long long*>(ws + lo.cut_off);
  unsigned* count = reinterpret_cast<unsigned*>(ws + lo.count_off);
  unsigned* range = reinterpret_cast<unsigned*>(ws + lo.range_off);
  const uint16_t* qx = static_cast<const uint16_t*>(q);
  const uint16_t* kx = static_cast<const uint16_t*>(k);

  const PoolTensor pool_q = {qx, p->q_stride_b, p->q_stride_h, p->q_stride_l, p->M, (int)lo.QB, qp};
  const PoolTensor pool_k = {kx, p->k_stride_b, p->k_stride_h, p->k_stride_l, p->N, (int)lo.G, kp};
  const uint16_t* kmat = kp;
  int64_t k_slice_stride = lo.G * p->d, k_row_stride = p->d;
  const bool k_in_place = p->N == 1 && p->B == 1;   // a block of one row is the row itself; slices are then heads
  if (k_in_place) {
    kmat = kx;
    k_slice_stride = p->k_stride_h;
    k_row_stride = p->k_stride_l;
  }
  hipLaunchKernelGGL(pool_kernel, dim3((unsigned)(lo.QB + (k_in_place ? 0 : lo.G)), (unsigned)lo.slices), dim3(64), 0, stream,
                     pool_q, pool_k, p->H, p->L, p->d, range);
  if (!launched()) return FGATTN_E_DEVICE;
  uint32_t* keep_bits = reinterpret_cast<uint32_t*>(ws + lo.bits_off);
  if (lo.G <= kShortMax && !(p->flags & (FGATTN_FLAG_MASK_ROWS_IN_HBM | FGATTN_FLAG_MASK_ONE_TILE_CHUNKS))) {
    auto launch = [&](auto d, auto k) {
      hipLaunchKernelGGL((short_rows_kernel<decltype(d)::value, decltype(k)::value>),
                         dim3((unsigned)((lo.QB + kShortRows - 1) / kShortRows), (unsigned)lo.slices), dim3(kShortRows * 64), 0, stream, qp,
                         kmat, k_slice_stride, k_row_stride, (int)lo.QB, (int)lo.G, (int)lo.Gw, p->scale, top_p, cut, count, keep_bits);
    };
    auto launch_k = [&](auto d) {
      if (lo.G <= 64) launch(d, std::integral_constant<int, 1>());
      else if (lo.G <= 128) launch(d, std::integral_constant<int, 2>());
      else if (lo.G <= 256) launch(d, std::integral_constant<int, 4>());
      else if (lo.G <= 512) launch(d, std::integral_constant<int, 8>());
      else launch(d, std::integral_constant<int, 16>());
    };
    if (p->d == 128) launch_k(std::integral_constant<int, 128>());
    else launch_k(std::integral_constant<int, 64>());
    if (!launched()) return FGATTN_E_DEVICE;
    fgscan::launch_row_pointers(count, lo.rows, mask_indptr, stream);
    return launched() ? FGATTN_OK : FGATTN_E_DEVICE;
  }
  const unsigned gx = (unsigned)((lo.G + kTilesPerGroup * 32 - 1) / (kTilesPerGroup * 32));
  const size_t score_bytes = lo.cut_off - lo.scores_off;
  StreamArgs sa;
  if (!(p->flags & (FGATTN_FLAG_MASK_ROWS_IN_HBM | FGATTN_FLAG_MASK_ONE_TILE_CHUNKS)) &&
      plan_stream(lo, p->d, ws + lo.scores_off, score_bytes, cus, &sa)) {
    sa.qp = qp;
    sa.kp = kmat;
    sa.k_slice_stride = k_slice_stride;
    sa.k_row_stride = k_row_stride;
    sa.scale = p->scale;
    sa.top_p = top_p;
    sa.QB = (int)lo.QB;
    sa.G = (int)lo.G;
    sa.Gw = (int)lo.Gw;
    sa.range = range;
    sa.cut = cut;
    sa.count = count;
    sa.keep_bits = keep_bits;
    if (!(p->d == 128 ? launch_stream<128>(sa, lo, cus, stream) : launch_stream<64>(sa, lo, cus, stream)))
      return FGATTN_E_DEVICE;
    fgscan::launch_row_pointers(count, lo.rows, mask_indptr, stream);
    return launched() ? FGATTN_OK : FGATTN_E_DEVICE;
  }
  for (int64_t unit0 = 0; unit0 < lo.units; unit0 += lo.chunk_units) {
    const int64_t nunits = lo.units - unit0 < lo.chunk_units ? lo.units - unit0 : lo.chunk_units;
    const int64_t chunk_rows = nunits * 128;
    const dim3 sgrid((unsigned)((gx < 8 ? gx : (gx + 7) & ~7u) * nunits));
    if (p->d == 128)
      hipLaunchKernelGGL(scores_kernel<128>, sgrid, dim3(256), 0, stream, qp, kmat, k_slice_stride, k_row_stride, (int)lo.QB,
                         (int)lo.G, (int)lo.Gs, p->scale, (int)unit0, (int)nunits, (int)lo.YT, (int)gx, scores, range);
    else
      hipLaunchKernelGGL(scores_kernel<64>, sgrid, dim3(256), 0, stream, qp, kmat, k_slice_stride, k_row_stride, (int)lo.QB,
                         (int)lo.G, (int)lo.Gs, p->scale, (int)unit0, (int)nunits, (int)lo.YT, (int)gx, scores, range);
    if (!launched()) return FGATTN_E_DEVICE;
    if (lo.row_in_lds) {
      // As many persistent workgroups as LDS or registers let in: three per compute unit with the codes of 32768 scores, two
      // with 65536, one, of 1024 threads, with 131072.  Short rows are all latency: workgroups of 256, seven of them (10240
      // rows of 2048 scores 102 us with three workgroups of 512 per unit -> 52, 2560 of 4096 54 -> 31).
      auto launch = [&](auto kernel, int threads, int per_cu) {
        const int64_t fit = (int64_t)per_cu * cus;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(chunk_rows < fit ? chunk_rows : fit)), dim3(threads), 0, stream, scores, range,
                           chunk_rows, (int)unit0, (int)lo.YT, (int)lo.QB, (int)lo.G, (int)lo.Gs, top_p, cut, count, keep_bits,
                           (int)lo.Gw);
      };
      if (lo.Gs <= 4096)
        launch(select_codes_kernel<256, 4096, 2048, uint16_t, 7>, 256, 7);
      else if (lo.Gs <= 32768)
        launch(select_codes_kernel<512, 32768, 2048, uint16_t, 6>, 512, 3);
      else if (lo.Gs <= 65536)
        launch(select_codes_kernel<512, 65536, 2048, uint16_t, 4>, 512, 2);
      else
        launch(select_codes_kernel<1024, kRowCodesMax, 4096, uint32_t, 4>, 1024, 1);
    } else {
      hipLaunchKernelGGL((select_kernel<kSelThreads, kBins, kCap>), dim3((unsigned)chunk_rows), dim3(kSelThreads), 0, stream,
                         scores, range, (int)unit0, (int)lo.YT, (int)lo.QB, (int)lo.G, (int)lo.Gs, top_p, cut, count, keep_bits,
                         (int)lo.Gw);
    }
    if (!launched()) return FGATTN_E_DEVICE;
  }
  fgscan::launch_row_pointers(count, lo.rows, mask_indptr, stream);
  return launched() ? FGATTN_OK : FGATTN_E_DEVICE;
}

int fgattn_mask_emit(const fgattn_params* p, const int64_t* mask_indptr, int32_t* mask_indices, int64_t indices_capacity,
                     const void* workspace, size_t workspace_bytes, void* stream_v) {
  using namespace fgm;
  Layout lo;
  int rc = layout_of(p, &lo);
  if (rc) return rc;
  if (!mask_indptr || !workspace || (!mask_indices && indices_capacity > 0)) return FGATTN_E_NULL;
  if (indices_capacity < 0) return FGATTN_E_SHAPE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(mask_indices) & 3)) return FGATTN_E_ALIGN;
  if (workspace_bytes < lo.total) return FGATTN_E_WORKSPACE;
  int cus = 1;
  rc = device_ok(&cus);
  if (rc) return rc;
  const char* ws = static_cast<const char*>(workspace);
  // a wave per row, or several per row (each counts the bits ahead of its stretch): until two rounds of waves fill the chip,
  // with at least 4096 key blocks each, and until every SIMD has four, with at least 1024 each (250 rows of 4000 one wave per
  // row 7.8 us, four 5.3; 1000 rows 9.1 and 7.5; 3000 rows of 8000 with stretches that short 20, with two per row 17.6)
  auto stretches = [&](int64_t waves, int64_t words) {
    const int64_t by_waves = (waves + lo.rows - 1) / lo.rows, by_words = (lo.Gw + words - 1) / words;
    return by_waves < by_words ? by_waves : by_words;
  };
  const int64_t few = stretches(2 * 32 * (int64_t)cus, 128), more = stretches(4 * 4 * (int64_t)cus, 32), segs = few > more ? few : more;
  const int64_t seg_words = ((lo.Gw + segs - 1) / segs + 1) & ~(int64_t)1;
  const int64_t units = lo.rows * segs;
  hipLaunchKernelGGL(emit_bits_kernel, dim3((unsigned)((units + 3) / 4)), dim3(256), 0, static_cast<hipStream_t>(stream_v),
                     reinterpret_cast<const uint32_t*>(ws + lo.bits_off), (int)lo.Gw, (int)seg_words, (int)segs, units,
                     mask_indptr, mask_indices, indices_capacity);
  return launched() ? FGATTN_OK : FGATTN_E_DEVICE;
}

}  // extern "C"
