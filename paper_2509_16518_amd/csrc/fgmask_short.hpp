// Scores and top-p selection of short rows in one kernel: included by fgmask.hip.
#pragma once

namespace fgm {

constexpr int kShortRows = 8;     // query blocks of a workgroup, one per wave
constexpr int kShortBins = 256;
// Rows of more key blocks are selected by workgroups: with 32 scores per lane a compute unit holds one workgroup of these (both mask
// calls, 40 heads x 128 rows of 2048 96 us against 63, 24 x 929 of 1857 593 against 495, 12 x 1024 of 2048 219 against 153).
constexpr int kShortMax = 1024;

// A workgroup of eight waves forms the scores of eight query blocks of one slice (the waves take the tiles of 32 key blocks in
// turn; the matrix instruction's other 24 rows repeat a query block and are dropped), passes them through LDS, and each
// wave selects one row, K scores per lane, with nothing but its own registers and its own piece of LDS: range, a histogram of
// mass over it, the crossing bin's members ranked.  Bound: latency, which a scores kernel and a selection by workgroups paid for twice
// and with a barrier for every step.  Both mask calls: 12 heads x 147 rows of 147 scores 44.6 -> 23.6 us, 32 x 83 of 165 43.7 ->
// 20.7, 40 x 512 of 512 276 -> 204, 12 x 1024 of 1024 142 -> 122, 40 x 7425 of 929 2.33 -> 1.30 ms.
// Rows with more than 64 members of the crossing bin go on in cut_of_many (the select call alone, 12 x 1024 rows of 1024: equal scores
// 390 us when a round did not begin with the range of its keys and one bin took every addition, now 87; two values 137, now 90; by
// workgroups 239 and 127).
template <int D, int K>
__global__ void __launch_bounds__(kShortRows * 64) short_rows_kernel(const uint16_t* qp, const uint16_t* kp, int64_t k_slice_stride,
                                                                     int64_t k_row_stride, int QB, int G, int Gw, float scale,
                                                                     float top_p, unsigned long long* cut, unsigned* count,
                                                                     uint32_t* keep_bits) {
  constexpr int STEPS = D / 16;
  __shared__ float scores[kShortRows][K * 64];
  __shared__ unsigned long long all_mass[kShortRows][kShortBins];
  __shared__ unsigned long long all_cand[kShortRows][64];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ln = lane & 31, g = lane >> 5;
  const int slice = blockIdx.y, q0 = blockIdx.x * kShortRows;
  unsigned long long* const mass = all_mass[wv];
  unsigned long long* const cand = all_cand[wv];
  for (int i = lane; i < kShortBins; i += 64) mass[i] = 0;
  {
    const char* qsrc = reinterpret_cast<const char*>(qp + ((int64_t)slice * QB + min(q0 + min(ln, kShortRows - 1), QB - 1)) * D) + g * 16;
    const char* kbase = reinterpret_cast<const char*>(kp + slice * k_slice_stride) + g * 16;
    bf16x8 qf[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; s++) qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(qsrc + s * 32));
    for (int tile = wv; tile * 32 < G; tile += kShortRows) {
      const char* ksrc = kbase + (int64_t)min(tile * 32 + ln, G - 1) * k_row_stride * 2;
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; r++) acc[r] = 0.0f;
#pragma unroll
      for (int s = 0; s < STEPS; s++)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[s], __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(ksrc + s * 32)), acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; r++) scores[4 * g + r][tile * 32 + ln] = acc[r] * scale;   // (rows 0 to 7 of the product)
    }
  }
  __syncthreads();
  const int q = q0 + wv;
  if (q >= QB) return;
  const int64_t row = (int64_t)slice * QB + q;
  float x[K];
  bool is[K];
  unsigned hi = 0u, lo = 0u;   // largest ordered bits, and largest of the complement
#pragma unroll
  for (int k = 0; k < K; k++) {
    x[k] = scores[wv][k * 64 + lane];
    is[k] = k * 64 + lane < G;
    hi = max(hi, is[k] ? ordered_bits(x[k]) : 0u);
    lo = max(lo, is[k] ? ~ordered_bits(x[k]) : 0u);
  }
  hi = lane_max(hi);
  lo = ~lane_max(lo);
  const float rmax = from_ordered(hi), rmin = from_ordered(lo);
  const float inv = bins_per_score<kShortBins>(rmax, rmin);
  unsigned bins[K];
#pragma unroll
  for (int k = 0; k < K; k++) bins[k] = value_bin_of<kShortBins>(x[k], rmax, inv);
  if (inv != 0.0f) {
#pragma unroll
    for (int k = 0; k < K; k++)
      if (is[k]) atomicAdd(&mass[bins[k]], weight_of(x[k], rmax));
  } else {   // one bin for all: added up over the lanes (additions to the same word are served one by one)
    unsigned long long sum = 0;
#pragma unroll
    for (int k = 0; k < K; k++) sum += is[k] ? weight_of(x[k], rmax) : 0ull;
    sum = lane_prefix(sum);
    if (lane == 63) mass[0] = sum;
  }
  wave_order();
  unsigned long long before = 0, target = 0;
  const unsigned bin = (unsigned)crossing_bin<kShortBins>(mass, before, [&](unsigned long long Z) {
    const double t = ceil((double)top_p * (double)Z);
    target = t < 1.0 ? 1ull : (unsigned long long)t;
    if (target > Z) target = Z;
    return target;
  });
  wave_order();
  unsigned found = 0;   // members of the crossing bin, and the first 64 of them
#pragma unroll
  for (int k = 0; k < K; k++) {
    const bool in = is[k] && bins[k] == bin;
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(in);
    const unsigned pos = found + lanes_below(lanes);
    if (in && pos < 64u) cand[pos] = rank_key(x[k], k * 64 + lane);
    found += (unsigned)__popcll(lanes);
  }
  wave_order();
  unsigned long long c = ~0ull;
  if (found - 1u < 64u) {   // 1 to 64
    c = cut_of_few(cand, (int)found, mass, before, target, rmax);
  } else if (found != 0u) {
    c = cut_of_many<kShortBins, true>(
        [&](auto&& fn) {   // (from LDS again, not unrolled: the usual rows pay for this path with registers and code)
#pragma unroll 1
          for (int j = lane; j < K * 64; j += 64) {
            const float v = scores[wv][j];
            fn(rank_key(v, j), j < G && value_bin_of<kShortBins>(v, rmax, inv) == bin);
          }
        },
        [](unsigned long long, bool) {}, (unsigned long long)lo << 32, ((unsigned long long)hi << 32) | 0xFFFFFFFFull, cand, mass, before,
        target, rmax);   // (the row's own range: with infinite scores nothing weighs anything, and the first range that holds a key is it)
  }
  unsigned kept = 0;
  uint32_t* const bits_row = keep_bits + row * Gw;
#pragma unroll
  for (int k = 0; k < K; k++) {
    const uint64_t keep = __builtin_amdgcn_ballot_w64(is[k] && rank_key(x[k], k * 64 + lane) >= c);
    kept += (unsigned)__popcll(keep);
    if (lane < 2 && 2 * k + lane < Gw) bits_row[2 * k + lane] = lane == 0 ? (uint32_t)keep : (uint32_t)(keep >> 32);
  }
  if (lane == 0) {
    cut[row] = c;
    count[row] = kept;
  }
}

}  // namespace fgm
