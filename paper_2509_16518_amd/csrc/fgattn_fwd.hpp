// Forward kernel of fine-grained sparse attention for CDNA4 (gfx950, wave64).
//
// One persistent workgroup (4 waves) processes one work item at a time: a block of M query
// rows of one head against the compacted list of its active keys (paper Sec. 4.1, Fig. 1b).
// Per item: the query fragment stays in registers; the active K/V rows are gathered straight
// from global memory into rings of LDS tiles with per-lane-address LDS-DMA loads (the
// gather-load of Sec. 4.1, re-designed for CDNA4), one or two tiles ahead of their use
// (Sec. 4.1 "Overlapped indirect key/value load latency"); bf16 MFMA computes
// S^T = K_rel Q^T and O^T = V_rel^T P^T with fp32 online-softmax state in registers (Sec. 2
// "Efficient dense attention").  A gather instruction holds the wave that issues it until the
// vector-memory path has taken it (~170 clocks under load); MFMAs issued before it keep
// executing meanwhile, so each tile's key loop interleaves them with the MFMAs of both contractions and the previous
// tile's exponentials.  Work items are fetched from per-XCD device-side queues in the
// order a pre-pass wrote (Sec. 4.2 "Load balancing", Appendix B).
//
// Transposed formulation: scores are produced as S^T (keys x queries) so that, in the MFMA
// accumulator layout, one lane owns one query column.  Row statistics (max, sum) are then
// per-lane scalars plus one exchange between lanes l and l^32, and the probabilities are
// already laid out as the B operand of the second MFMA: P never moves between lanes.
//
// Every wave owns a 32-query x 32-key piece of each tile.  A workgroup of WV waves covers MT = 32, 64 or
// 128 query rows with RW = MT/32 waves along the rows and KW = WV/RW waves along the keys of a
// tile (NT = 32*KW keys); waves that split the keys keep private (max, sum, O) and merge once
// per work item.  WV is 4 except for the 32-row tile, which runs as single-wave workgroups: a wave's K and V
// slots take 32 KB at d = 128, of which LDS holds four per compute unit, and independent waves need no merge of their key
// halves at the end of an item and never wait for each other.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "fgattn_args.hpp"

namespace fg {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

#define FG_LDS __attribute__((address_space(3)))
#define FG_CONST __attribute__((address_space(4)))

__device__ __forceinline__ void wait_vmem_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

// Gather-load primitive: every lane names its own 16-byte global source (base + 32-bit byte
// offset); the wave's 64 chunks land lane-linearly in LDS at lds_base + 16*lane (LDS-DMA, no
// VGPR staging).  Written as inline assembly so that the compiler does not track the transfer:
// the kernel orders these loads against LDS reads itself (vmcnt(0) + workgroup barrier once per
// tile), which lets the gathers of later tiles stay in flight during all of a tile's matrix work.
// A run of up to four 1 KiB loads lands back to back in LDS: M0 is written once
// (gather16_first) and the following loads (gather16_next<K>) add K KiB through the instruction offset.  That
// offset also enters the global address, so `base_m4k` is the true base minus 4096 and the byte offset carries
// +4096 - 1024*K (kept non-negative: the 32-bit offset is zero-extended).
// gather16_next relies on M0 still holding what the preceding gather16_first wrote.  The statements in between are
// MFMAs, LDS reads and vector arithmetic, none of which the compiler implements through M0 on gfx950; the build
// enforces it: it scans the generated assembly of every kernel and fails if any instruction other than the
// `s_mov_b32 m0` lines marked fg_m0 above writes M0.
__device__ __forceinline__ const void* pin_scalar(const void* p) {
  // wave-uniform by construction; readfirstlane pins it to scalar registers (it folds away when already there)
  const uint64_t b64 = (uint64_t)(uintptr_t)p;
  return (const void*)(uintptr_t)(((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(b64 >> 32)) << 32) |
                                  (unsigned)__builtin_amdgcn_readfirstlane((int)(b64 & 0xffffffffu)));
}
__device__ __forceinline__ void gather16_first(const void* base_m4k, unsigned byte_off, unsigned lds_base) {
  base_m4k = pin_scalar(base_m4k);
  lds_base = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_base);
  asm volatile(
      "s_mov_b32 m0, %2 ; fg_m0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(byte_off), "s"(base_m4k), "s"(lds_base)
      : "memory", "m0");
}
template <int K>
__device__ __forceinline__ void gather16_next(const void* base_m4k, unsigned byte_off) {
  static_assert(K >= 1 && K <= 3, "the instruction offset is 13-bit signed");
  base_m4k = pin_scalar(base_m4k);
  if (K == 1) asm volatile("global_load_lds_dwordx4 %0, %1 offset:1024" : : "v"(byte_off), "s"(base_m4k) : "memory");
  if (K == 2) asm volatile("global_load_lds_dwordx4 %0, %1 offset:2048" : : "v"(byte_off), "s"(base_m4k) : "memory");
  if (K == 3) asm volatile("global_load_lds_dwordx4 %0, %1 offset:3072" : : "v"(byte_off), "s"(base_m4k) : "memory");
}
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(uintptr_t)((FG_LDS const unsigned char*)p);
}

// (three-input maximum, written so that the compiler selects v_max3_f32.  Not inline assembly: the compiler does not
// insert the wait states an MFMA result needs before a vector instruction reads it when that instruction is hidden
// in an asm statement)
__device__ __forceinline__ float max3(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }
__device__ __forceinline__ float lane_pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// maximum over the same two lanes
__device__ __forceinline__ float lane_pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

constexpr int cmin(int a, int b) { return a < b ? a : b; }
constexpr int cgcd(int a, int b) { return b == 0 ? a : cgcd(b, a % b); }
constexpr int clcm(int a, int b) { return a / cgcd(a, b) * b; }

// Tiling and LDS ring of one workgroup.  KS / VS = slots of the K ring / V ring (tiles of NT keys): in iteration t the
// workgroup reads K(t+1) and V(t-1) and gathers K(t+KS) and V(t+VS-2) into the slots that the previous iteration
// released, so KS-1 K tiles and VS-1 V tiles can be in flight.  The forward pass is instantiated with two slots each
// (deeper rings make the gather half alone faster -- a third K slot by 8% -- but not the whole kernel); the
// measurement aid also builds the gather half with a K ring of three.  WV = waves of a workgroup.
template <int MT, int D, int KS = 2, int VS = 2, int WV = 4>
struct FwdCfg {
  static constexpr int RW = MT / 32;            // waves along query rows (32 rows each)
  static constexpr int KW = WV / RW;            // waves along keys within a tile (32 keys each)
  static constexpr int NT = 32 * KW;            // keys per LDS tile
  static constexpr int CH = D / 8;              // 16-byte chunks per row
  static constexpr int ROWB = D * 2;            // bytes per K or V row
  static constexpr int RPI = 64 / CH;           // rows fetched by one wave-wide 16 B/lane load
  static constexpr int RPW = NT / WV;           // rows of a tile each wave fetches
  static constexpr int IPW = RPW / RPI;         // load instructions per wave, per tile, per tensor
  static constexpr int SSTEPS = D / 16;         // MFMA steps along d for S^T
  static constexpr int DBLK = D / 32;           // 32-row blocks of O^T
  static constexpr int TENSOR_BYTES = NT * ROWB;
  static constexpr int K_OFF = 0;
  static constexpr int V_OFF = KS * TENSOR_BYTES;
  static constexpr int RING_BYTES = (KS + VS) * TENSOR_BYTES;
  static constexpr int EXTRA_OFF = RING_BYTES;  // membership words or dropped-key words (variants that have them)
  static constexpr int MERGE_REGS = DBLK * 16 + 2;
  static constexpr int MERGE_BYTES = (KW - 1) * RW * MERGE_REGS * 256;
  static constexpr int ITEM_OFF = RING_BYTES - 16;   // the work-item id is handed to the waves through the ring's last bytes
  static constexpr int MEMBER_BYTES = 2 * NT * 4;           // grouped query tiles: a membership word per key and K slot
  static constexpr int DROP_BYTES = 2 * (2 * WV + 2) * 4;   // short last group: per K slot a tag, and a tag and a word of each wave
  static constexpr int NKEYS = KS - VS + 3;     // tiles whose keys a wave keeps: t+VS-2 (V gather) .. t+KS (K gather)
  static_assert(MT == 32 || MT == 64 || MT == 128, "query tile");
  static_assert(WV >= RW && WV % RW == 0 && (WV == 1 || WV == 2 || WV == 4), "waves of a workgroup");
  static_assert(D == 64 || D == 128, "head dim");
  static_assert(KS >= 2 && VS >= 2 && KS >= VS, "ring depths");
  static_assert(IPW >= 1 && RPW % RPI == 0 && (RPW & (RPW - 1)) == 0, "loader shape");
  static_assert(MERGE_BYTES <= ITEM_OFF, "merge scratch must fit in the tile buffers, below the work-item word");
};

// Online softmax of one 32-key x 32-query score block held as an MFMA accumulator: one query per
// lane (registers 8c..8c+7 of the accumulator are the keys 16c + 8*(e/4) + 4*(lane/32) + e%4).
// Masks (a key that does not count gets the score -inf):
// mask_members (grouped query tiles): a row in LDS holds, per key, the bit mask of the group members that selected it; a
//   query of member `member` keeps only the keys whose bit is set.
// mask_drop: bit 8*r4 + e of `drop` says that the key in accumulator register 4*r4 + e of this lane does not count.
// A score that does not count is replaced by bits (a mask of all ones or none and a bit-field insert) and not by a
// conditional move: one that reads its condition from vcc takes four times an ordinary instruction's time, and between
// it and the compare there are wait states.  Grouping and forward pass, 12 heads x 32760 tokens in tiles of 16 rows 7.57 ->
// 7.42 ms; 8 heads x 9360 tokens of d = 64 603 -> 577 us, 2 heads x 4096 in tiles of 64 rows 138 -> 129 us.
__device__ __forceinline__ float keep_if(float s, int all_ones) {
  return __uint_as_float((__float_as_uint(s) & (unsigned)all_ones) | (~(unsigned)all_ones & 0xFF800000u));
}
__device__ __forceinline__ void mask_members(f32x16& S, const int* members, int g, int member) {
#pragma unroll
  for (int r4 = 0; r4 < 4; r4++) {
    i32x4 bv = *reinterpret_cast<const i32x4*>(members + 8 * r4 + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; e++) S[4 * r4 + e] = keep_if(S[4 * r4 + e], __builtin_amdgcn_sbfe(bv[e], member, 1));
  }
}
__device__ __forceinline__ void mask_drop(f32x16& S, unsigned drop) {
#pragma unroll
  for (int r4 = 0; r4 < 4; r4++)
#pragma unroll
    for (int e = 0; e < 4; e++) S[4 * r4 + e] = (drop >> (8 * r4 + e)) & 1 ? -INFINITY : S[4 * r4 + e];
}
// largest score of this lane's query
__device__ __forceinline__ float row_max(const f32x16& S) {
  const float t0 = max3(S[0], S[1], S[2]), t1 = max3(S[3], S[4], S[5]), t2 = max3(S[6], S[7], S[8]);
  const float t3 = max3(S[9], S[10], S[11]), t4 = max3(S[12], S[13], S[14]);
  return lane_pair_max(fmaxf(max3(t0, t1, t2), max3(t3, t4, S[15])));
}

// NMODE selects how a compacted key position maps to a key row:
//   NMODE_DENSE   position == key (0% sparsity, no index list);
//   NMODE_N1      one key per group: key = indices[position];
//   NMODE_GROUPS  N >= 1 keys per group: key = indices[position / N] * N + position % N, L a multiple of N;
//   NMODE_GROUPS_SHORT  the same with a short last group (L not a multiple of N): any tile may then hold
//                 positions past the end of the sequence, which are masked out.
enum { NMODE_DENSE = 0, NMODE_N1 = 1, NMODE_GROUPS = 2, NMODE_GROUPS_SHORT = 3 };

// PART selects what is executed: PART_ALL is the forward pass; PART_GATHER keeps only the index translation and
// the row gathers, PART_COMPUTE everything but the row gathers (both leave meaningless results and exist so that
// the two halves of the kernel can be timed apart on the same launch shape).
enum { PART_ALL = 0, PART_GATHER = 1, PART_COMPUTE = 2 };

// LDS beyond the tile rings: grouped query tiles keep membership words there; with a short last key group the waves of a
// workgroup tell each other which keys of a tile lie past the end of the sequence (a single wave knows by itself).
// The ragged end of a list is masked by position and needs none.
template <int MT, int D, int NMODE, bool GROUPED = false, int KS = 2, int VS = 2, int WV = 4>
constexpr int fwd_lds_bytes() {
  using C = FwdCfg<MT, D, KS, VS, WV>;
  return C::RING_BYTES + (GROUPED ? C::MEMBER_BYTES : NMODE == NMODE_GROUPS_SHORT && WV > 1 ? C::DROP_BYTES : 0);
}

// id loads: plain per-lane loads written as inline assembly so that the compiler does not track them.  (A tracked load
// makes the compiler wait with vmcnt(0) before the first use, which would also wait for every gather in flight: the
// counter is shared and the compiler cannot see the gathers.)  The kernel waits with the s_waitcnt that precedes each
// tile's barrier (wait_vmem_le(loaded) ties the register to that wait for the compiler), and with a wait that ties all of
// them where the key loop ends.  In between, the compiler must neither copy nor reuse such a register: the build follows
// every path of the generated code from each marked load (fg_id) to its wait and fails if one is touched.  Consumers clamp
// what they read to [0, L), so even a register read too early could never address out of bounds.
__device__ __forceinline__ void load_id_untracked(int& dst, const int32_t* base, unsigned byte_off) {
  // (scalar base + 32-bit per-lane offset: no 64-bit address arithmetic on the vector ALU)
  base = static_cast<const int32_t*>(pin_scalar(base));
  asm volatile("global_load_dword %0, %1, %2 ; fg_id" : "=v"(dst) : "v"(byte_off), "s"(base) : "memory");
}
__device__ __forceinline__ void load_byte_untracked(int& dst, const uint8_t* base, unsigned byte_off) {
  base = static_cast<const uint8_t*>(pin_scalar(base));
  asm volatile("global_load_ubyte %0, %1, %2 ; fg_id" : "=v"(dst) : "v"(byte_off), "s"(base) : "memory");
}
// `loaded` (an untracked load's target) is valid from here on, by a wait just made
__device__ __forceinline__ void arrived(int& loaded) { asm volatile("" : "+v"(loaded)); }
template <int N>
__device__ __forceinline__ void wait_vmem_le() {   // s_waitcnt vmcnt(N): at most N vector-memory loads still in flight
  static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}
template <int N>
__device__ __forceinline__ void wait_vmem_le(int& loaded) {   // the same, and `loaded` (an untracked load's target) is valid after it
  static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%1)" : "+v"(loaded) : "n"(N) : "memory");
}

// GROUPED (paper Sec. 4.2): a work item is a GROUP of query tiles (a.tile_rows rows each, R = MT / tile_rows of
// them, listed in a.group_tiles) that shares one gathered key list -- the union of the members' lists -- while
// every member attends only to its own key blocks: a.memb holds, per entry of the union list, the bit mask of the
// members that selected it, and scores of the others are set to -inf before the softmax.
// DENSE_PRIO: the dense kernel raises the wave priority in its gather phase (the others always or never do).
template <int MT, int D, int NMODE, int OCC, int PART = PART_ALL, bool GROUPED = false, int KS = 2, int VS = 2, int WV = 4,
          bool DENSE_PRIO = false>
__global__ void __launch_bounds__(WV * 64, OCC) fgattn_fwd_kernel(const FwdArgs a) {
  using C = FwdCfg<MT, D, KS, VS, WV>;
  constexpr bool DENSE = NMODE == NMODE_DENSE;
  constexpr bool WAVE_PRIO = DENSE ? DENSE_PRIO : NMODE == NMODE_N1 || MT > 32;
  constexpr bool SHORT_GROUP = NMODE == NMODE_GROUPS_SHORT;   // (the host picks the variant from L % N)
  // the cross-lane permute of the ids is issued before the barrier that precedes its use (measured with one key per group:
  // 2.4% faster at 128 query rows, 2.5% slower at 64)
  constexpr bool EARLY_PERMUTE = NMODE == NMODE_N1 && !GROUPED && MT == 128;
  static_assert(!GROUPED || (MT == 128 && (NMODE == NMODE_N1 || NMODE == NMODE_GROUPS_SHORT)),
                "groups are 128 query rows with a sparse list (any L: the variant that masks positions past the end)");
  // vector-memory operations per iteration and wave, in program order: V gathers, K gathers, ids of a later tile (and their
  // membership bytes)
  constexpr int NIDS = DENSE ? 0 : GROUPED ? 2 : 1;
  constexpr int PER = 2 * C::IPW + NIDS;
  // What may still be in flight at the barrier that opens iteration t+1: everything issued after V(t) (gathered in
  // iteration t+2-VS, first in its iteration) and after K(t+2) (gathered in iteration t+2-KS).  With two slots each
  // that is the id load at the end of iteration t alone: the list streams from device memory, and its latency passes
  // under the whole of iteration t+1 instead of holding the barrier.
  constexpr int WAITN = cmin(C::IPW + NIDS + (VS - 2) * PER, NIDS + (KS - 2) * PER);
  // ids of tile t+KS+IDL are requested at the end of iteration t and turned into key rows at the start of iteration t+IDL
  constexpr int IDL = 2;
  constexpr int AFTER_IDS = (IDL - 1) * PER;   // operations issued after an id load by the end of the iteration before its use
  static_assert(AFTER_IDS >= WAITN && AFTER_IDS <= 63, "id wait");
  constexpr int U = clcm(clcm(KS, VS), 2);   // iterations per unrolled loop body: every slot is an immediate
  static_assert(U <= 12 && U % IDL == 0, "unroll");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int tid = threadIdx.x;
  // without a pre-pass, what it leaves in the workspace is written here: cleared control words and an order
  if (a.schedule == SCHED_DIRECT) {
    if (blockIdx.x == 0 && tid < 64) a.counter[tid] = 0;
    if (a.leave_order && tid == 0) a.order[blockIdx.x] = blockIdx.x;
  }
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int rw = wv / C::KW, kw = wv % C::KW;
  const int g = lane >> 5, ln = lane & 31;
  // loader role: this lane fetches 16-byte chunk `pc` of row `lrow` of each 1 KiB load
  const int lrow = lane / C::CH, pc = lane % C::CH;
  // transposed-read role for V: 16-lane group (g,u); lane n = 4*kq + q addresses key kq, d offset 4q
  const int u = (lane >> 4) & 1, kq = (lane & 15) >> 2, qq = lane & 3;

  int* const members = reinterpret_cast<int*>(smem + C::EXTRA_OFF);   // GROUPED: [tile % 2][key of the tile]
  // SHORT_GROUP: per tile % 2, the tag of the last tile with keys past the end of the sequence, then for each wave the
  // tag of the last tile in which its rows had some, and which
  int* const drops = reinterpret_cast<int*>(smem + C::EXTRA_OFF);
  constexpr int DROP_SLOT = 2 * WV + 2;
  volatile int* s_item = reinterpret_cast<volatile int*>(smem + C::ITEM_OFF);
  const unsigned lds0 = lds_address(smem);

  // ---- LDS layout: rows of ROWB bytes, 16-byte chunks XOR-swizzled so that reads are bank-conflict free ----
  // The LDS of gfx950 serves 256 bytes per clock (64 banks): 16 lanes of a 16-byte read or 32 lanes of an
  // 8-byte read.  K (read as the A operand of S^T: lane -> row ln, chunk 2s+g) stores logical chunk c of row
  // r at chunk c ^ kswz(r), which spreads any 16 consecutive rows over 16 distinct 16-byte bank groups.
  // V (read through the transposing 8-byte read: 4 consecutive keys x 64 bytes per 32 lanes) stores chunk c
  // at c ^ vswz(r), which puts 4 consecutive rows into 4 distinct 64-byte bank groups.
  //   d = 128 (256-byte rows): kswz(r) = r & 15,       vswz(r) = (r & 3) << 2
  //   d =  64 (128-byte rows): kswz(r) = (r >> 1) & 7, vswz(r) = ((r >> 1) & 1) << 2
  // The gather writes LDS lane-linearly, so the swizzle is applied to the global source address: the lane
  // that lands on (row r, chunk pc) fetches logical chunk pc ^ swz(r).
  // reader, K: byte offset of step s is kor ^ (32*s): the row base has its low 8 bits clear and the swizzle term
  // ((g ^ kswz) << 4) only touches bits 4..7, so the sum folds into one XOR with the step constant
  const int kor = ((kw * 32 + ln) * C::ROWB) | ((g ^ (D == 128 ? (ln & 15) : ((ln >> 1) & 7))) << 4);
  // reader, V: lane n = 4*kq + qq of 16-lane group (g,u) addresses key row 4g+kq, d offset 16u + 4qq
  const int vrow = (kw * 32 + 4 * g + kq) * C::ROWB + ((qq & 1) << 3);
  const int vlp = 2 * u + (qq >> 1);                                    // chunk within the 4-chunk d block
  const int vsw = D == 128 ? (kq << 2) : (((kq >> 1) & 1) << 2);        // vswz of this lane's rows
  int voff[C::DBLK];                                                    // per-lane byte offset of d block db
#pragma unroll
  for (int db = 0; db < C::DBLK; db++) voff[db] = vrow + ((((4 * db) ^ vsw) + vlp) << 4);
  // loader: rows r0 + lrow with r0 a multiple of RPI; the lane-dependent part of the swizzled source chunk
  const unsigned kx = (unsigned)((pc ^ (D == 128 ? lrow : (lrow >> 1))) << 4);
  const unsigned vx = (unsigned)((pc ^ (D == 128 ? (lrow << 2) : (((lrow >> 1) & 1) << 2))) << 4);

  const unsigned k_rowb = (unsigned)(a.k_sl * 2), v_rowb = (unsigned)(a.v_sl * 2);
  const int N = DENSE ? 1 : a.N;
  // tags of tiles, unique over the items of this workgroup: a word left by an earlier tile never looks current
  constexpr bool TELL_DROPS = SHORT_GROUP && !GROUPED && WV > 1;
  int tag0 = 1;
  if (TELL_DROPS && tid < 2 * DROP_SLOT) drops[tid] = 0;   // (published by the barriers around the work-item word)
  // place of this lane's row of tile 0 inside the list: group and key of the group (the same for every item)
  const int lrow_id = wv * C::RPW + (lane & (C::RPW - 1));
  const int gq0 = NMODE >= NMODE_GROUPS ? lrow_id / N : lrow_id, gr0 = NMODE >= NMODE_GROUPS ? lrow_id % N : 0;
  int iter = 0;
  // the XCD this workgroup runs on (hardware register XCC_ID, bits 3:0) picks its home queue
  const int my_xcd = __builtin_amdgcn_s_getreg((4 - 1) << 11 | 0 << 6 | 20) & 7;
  // Queue q holds the work of a contiguous eighth of the (batch, head) slices, in the order the pre-pass wrote, so that a
  // head's K/V streams through one L2 instead of eight.  Its first blocks_of(q) items belong to the workgroups with
  // blockIdx % 8 == q (where the hardware places them), one each, without asking; only the items after those are
  // popped from the counter.  Atomics on one 128-byte line are served one per 12 ns whichever word they name (2048
  // workgroups with eight each on a line: 183 us; a plain load each: 0), so a workgroup whose queue has run dry reads
  // all counters with loads and pops only where something is left; a queue once dry stays dry.
  auto queue_begin = [&](int q) { return ((q * (a.n_items / a.QB)) >> 3) * a.QB; };
  auto blocks_of = [&](int q) { return ((int)gridDim.x - q + 7) >> 3; };
  auto pop = [&](int q) -> int {   // one item of queue q, or -1
    const int j = queue_begin(q) + blocks_of(q) + atomicAdd(a.counter + queue_word(q), 1);
    return j < queue_begin(q + 1) ? a.order[j] : -1;
  };
  bool home_dry = false;
  for (;;) {
    // ---------------- fetch the next work item ----------------
    if (tid == 0) {
      int item = -1;
      if (a.schedule == SCHED_DIRECT) {   // at most one item per workgroup; a contiguous eighth of the items per XCD
        const int r = blockIdx.x & 7, per = a.n_items >> 3, rem = a.n_items & 7;
        if (iter == 0) item = r * per + min(r, rem) + (blockIdx.x >> 3);
      } else if (a.schedule == SCHED_STATIC) {
        const int j = blockIdx.x + iter * gridDim.x;
        item = j < a.n_items ? a.order[j] : -1;
      } else {
        const int mine = queue_begin(blockIdx.x & 7) + (blockIdx.x >> 3);
        if (iter == 0 && mine < queue_begin((blockIdx.x & 7) + 1)) item = a.order[mine];
        if (item < 0 && !home_dry) {
          item = pop(my_xcd);
          home_dry = item < 0;
        }
        while (item < 0) {
          int popped[8];
#pragma unroll
          for (int q = 0; q < 8; q++) popped[q] = __hip_atomic_load(a.counter + queue_word(q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          int from = -1;   // the next queue after the home queue with something left
#pragma unroll
          for (int q = 0; q < 8; q++) {
            const bool left = queue_begin(q) + blocks_of(q) + popped[q] < queue_begin(q + 1);
            if (left && (from < 0 || ((q - my_xcd) & 7) < ((from - my_xcd) & 7))) from = q;
          }
          if (from < 0) break;
          item = pop(from);
        }
      }
      *s_item = item;
    }
    iter++;
    __syncthreads();
    const int w = __builtin_amdgcn_readfirstlane(*s_item);
    __syncthreads();   // the word lies inside the tile ring: every wave has read it before any gather may land there
    if (w < 0) break;

    const int slice = w / a.QB, qi = w - slice * a.QB;
    const int b = slice / a.H, h = slice - b * a.H;
    const int row0 = qi * a.M;
    const int row_end = min(row0 + a.M, a.L);
    // this lane's query row; in a group the 32 rows of a wave come from the member tiles' own positions
    int my_row = row0 + rw * 32 + ln;
    bool my_row_valid = my_row < row_end;
    int my_member = 0;   // which member of the group this lane's query belongs to
    if constexpr (GROUPED) {
      const int qg = rw * 32 + ln;
      my_member = qg / a.tile_rows;
      const int tile = a.group_tiles[(int64_t)w * a.R + my_member];
      my_row = tile * a.tile_rows + (qg - my_member * a.tile_rows);
      my_row_valid = tile >= 0 && my_row < a.L;
    }
    int64_t beg = 0;
    int cnt;  // active key groups of this item
    if (DENSE) {
      cnt = a.L;
    } else {
      beg = a.indptr[w];
      cnt = (int)(a.indptr[w + 1] - beg);
    }
    const int total = cnt * N;  // compacted key positions (a short last group leaves invalid ones)
    const int ntiles = (total + C::NT - 1) / C::NT;
    // (wave-uniform; pinned to scalar registers here, an item's set-up ahead of the first id load that uses it as its base)
    const int32_t* idx = DENSE ? nullptr : static_cast<const int32_t*>(pin_scalar(a.indices + beg));
    const uint16_t* kbase = a.k + b * a.k_sb + h * a.k_sh;
    const uint16_t* vbase = a.v + b * a.v_sb + h * a.v_sh;

    // ---------------- Q fragment (B operand of S^T), once per item ----------------
    bf16x8 qf[C::SSTEPS];
    {
      int qrow = GROUPED ? (my_row_valid ? my_row : 0) : min(my_row, a.L - 1);
      const char* qp = reinterpret_cast<const char*>(a.q + b * a.q_sb + h * a.q_sh + (int64_t)qrow * a.q_sl);
#pragma unroll
      for (int s = 0; s < C::SSTEPS; s++) {
        i32x4 raw = *reinterpret_cast<const i32x4*>(qp + (2 * s + g) * 16);
        raw ^= (int)a.q_sign;
        qf[s] = __builtin_bit_cast(bf16x8, raw);
      }
    }

    // ---------------- loader ----------------
    // Position p = T*NT + wv*RPW + i*RPI + lrow of the compacted list is fetched by this lane with load
    // instruction i of tile T.  Pipeline per tile T (one iteration per tile, one barrier each):
    //   iteration T-KS-2  : group ids requested     iteration T-KS : ids -> key rows, K(T) gathered
    //   iteration T-1     : S(T) = K(T) Q^T          iteration T-VS+2: V(T) gathered
    //   iteration T       : P(T) = exp(S(T) - m)     iteration T+1  : O += V(T)^T P(T)^T
    // Past the end of the list the pipeline keeps running on clamped positions: a few redundant, in-bounds gathers of
    // active rows per work item instead of existence checks in every iteration.
    //
    // ids -> key rows: lane j of a wave turns the id of row j % RPW of the wave's part of the tile into a key row (one
    // load and a handful of vector instructions per tile, whatever N is); a cross-lane permute then hands every lane
    // the key of the row it fetches with each load instruction.  (With N keys per group every load instruction used to
    // fetch and convert its own ids, in tracked loads that drained the gathers: 12 heads x 32760 tokens at 32x32 4.62 ms,
    // now 3.81; 40 uneven heads at 64x8 7.14 ms, now 6.54.)
    const int lpos = wv * C::RPW + lrow;
    int gi[IDL];                   // the id of this lane's row: tile T in gi[T % IDL]
    int gm[IDL];                   // GROUPED: its membership byte
    int gr[IDL];                   // NMODE_GROUPS: the key's place inside its group
    // Key rows of tiles t+VS-2 .. t+KS in iteration t (set 0 feeds the V gathers, the last set the K gathers): with up to
    // four load instructions per tile as the permute handed them out; with eight (32 query rows) one key per lane,
    // permuted once for K and again for V, which saves 14 registers and the moves between the sets (the other way
    // round, a second permute at 64 query rows costs 3.5%).
    constexpr bool KEEP_SPREAD = C::IPW <= 4;
    constexpr int KNEW = C::NKEYS - 1;
    int keys[C::NKEYS][KEEP_SPREAD ? C::IPW : 1];
    int kk[C::IPW], vk[C::IPW];    // key rows of the next K and V gathers
    int nq = gq0, nr = gr0;        // NMODE_GROUPS: place of the next tile to request, advanced without divisions
    const uint8_t* memb = GROUPED ? static_cast<const uint8_t*>(pin_scalar(a.memb + beg)) : nullptr;
    unsigned lone_drop[2] = {0u, 0u};   // SHORT_GROUP, one wave: keys past the end of the sequence, by tile % 2
    auto fetch_ids = [&](int T, int& id, int& mb, int& off) {
      if constexpr (DENSE) return;
      if constexpr (NMODE == NMODE_N1) {
        const unsigned at = min((unsigned)(T * C::NT + lrow_id), (unsigned)(cnt - 1));
        load_id_untracked(id, idx, at * 4u);
        if constexpr (GROUPED) load_byte_untracked(mb, memb, at);
      } else {
        const unsigned at = (unsigned)min(nq, cnt - 1);
        off = nr;
        load_id_untracked(id, idx, at * 4u);
        if constexpr (GROUPED) load_byte_untracked(mb, memb, at);
        nq += a.nt_div_n;
        nr += a.nt_mod_n;
        const bool wrap = nr >= N;
        nr -= wrap ? N : 0;
        nq += wrap ? 1 : 0;
      }
    };
    // id -> this lane's key row (T = the tile, par = T % 2), clamped to [0, L): whatever the register held, the gather
    // stays inside the K/V slice; a position past the end of the list or of the sequence reads an active row, so that
    // only active rows are ever multiplied, even by zero (0 x Inf would be NaN), and its score is masked out
    auto to_key = [&](int T, int par, int id, int mb, int off) {
      const unsigned raw = NMODE >= NMODE_GROUPS ? __umul24((unsigned)id, (unsigned)N) + (unsigned)off : (unsigned)id;
      if constexpr (GROUPED) {
        // the membership word of this key; no member where there is no key
        if (lane < C::RPW) members[par * C::NT + lrow_id] = T * C::NT + lrow_id < total && raw < (unsigned)a.L ? mb : 0;
      } else if constexpr (SHORT_GROUP) {
        const uint64_t past = __builtin_amdgcn_ballot_w64(raw >= (unsigned)a.L);
        if constexpr (WV == 1) {
          lone_drop[par] = (unsigned)past;
        } else if (__builtin_expect(past != 0, 0)) {
          if (lane == 0) {
            drops[par * DROP_SLOT] = tag0 + T;
            drops[par * DROP_SLOT + 2 + wv] = tag0 + T;
            drops[par * DROP_SLOT + 2 + WV + wv] = (int)((unsigned)past & (0xFFFFFFFFu >> (32 - C::RPW)));
          }
        }
      }
      return (int)min(raw, (unsigned)(a.L - 1));
    };
    // key rows of tile T for this lane's load instructions
    auto spread = [&](int T, int key, int (&dst)[C::IPW]) {
#pragma unroll
      for (int i = 0; i < C::IPW; i++) {
        if constexpr (DENSE) dst[i] = min(T * C::NT + lpos + i * C::RPI, a.L - 1);
        else dst[i] = __builtin_amdgcn_ds_bpermute((i * C::RPI + lrow) << 2, key);
      }
    };
    // tile T enters the pipeline as its newest key set / the V gathers' set leaves it
    auto take_keys = [&](int T, int par, int id, int mb, int off) {
      const int key = DENSE ? 0 : to_key(T, par, id, mb, off);
      spread(T, key, kk);
      if constexpr (KEEP_SPREAD) {
#pragma unroll
        for (int i = 0; i < C::IPW; i++) keys[KNEW][i] = kk[i];
      } else {
        keys[KNEW][0] = key;
      }
    };
    auto v_keys = [&](int T) {
      if constexpr (KEEP_SPREAD) {
#pragma unroll
        for (int i = 0; i < C::IPW; i++) vk[i] = keys[0][i];
      } else {
        spread(T, keys[0][0], vk);
      }
    };
    auto rotate_keys = [&]() {
#pragma unroll
      for (int s = 0; s + 1 < C::NKEYS; s++)
#pragma unroll
        for (int i = 0; i < (KEEP_SPREAD ? C::IPW : 1); i++) keys[s][i] = keys[s + 1][i];
    };
    // keys of tile Tm that do not count, as bits of this lane's accumulator registers (see mask_drop)
    auto dropped = [&](int Tm, int par) -> unsigned {
      const int limit = total - Tm * C::NT - kw * 32;   // keys of this wave's part that lie inside the list
      unsigned d = limit >= 32 ? 0u : limit <= 0 ? ~0u : ~0u << limit;
      if constexpr (SHORT_GROUP && WV == 1) d |= lone_drop[par];
      if constexpr (TELL_DROPS) {
        const int* slot = drops + par * DROP_SLOT;
#pragma unroll
        for (int w2 = 0; w2 < WV; w2++) {   // (rows w2 * RPW .. of the tile are wave w2's)
          const int at = w2 * C::RPW - kw * 32;
          if (at >= 0 && at < 32 && slot[2 + w2] == tag0 + Tm) d |= (unsigned)slot[2 + WV + w2] << at;
        }
      }
      // (the lane's number formed anew: kept through the key loop for this rare path, it is spilled, and a reload waits for
      // the gathers in flight as well)
      int zero = 0;
      asm volatile("" : "+v"(zero));
      return d >> (4 * (__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero)) >> 5));
    };
    // LDS: K ring slots 0..KS-1 then V ring slots 0..VS-1, TENSOR_BYTES each.  A run of up to four gathers of one
    // wave lands back to back, so only the first writes M0 and the others use the instruction offset (which also
    // enters the global address: base - 4096 and a per-lane constant + 4096 - 1024*(i%4) compensate).
    unsigned kcon[C::IPW], vcon[C::IPW];
#pragma unroll
    for (int i = 0; i < C::IPW; i++) {
      const int r0 = wv * C::RPW + i * C::RPI;
      // uniform part of kswz(r0 + lrow): (r0 & 12) for d = 128, (r0 >> 1) & 4 for d = 64; vswz has none
      const unsigned ku = (unsigned)((D == 128 ? (r0 & 12) : ((r0 >> 1) & 4)) << 4);
      kcon[i] = (kx ^ ku) + 4096u - 1024u * (i & 3);
      vcon[i] = vx + 4096u - 1024u * (i & 3);
    }
    const char* kbase_m4k = reinterpret_cast<const char*>(kbase) - 4096;
    const char* vbase_m4k = reinterpret_cast<const char*>(vbase) - 4096;
    auto gather_k = [&](auto ic, int slot, const int (&kk)[C::IPW]) {
      constexpr int i = decltype(ic)::value;
      if constexpr (PART == PART_COMPUTE) return;
      const unsigned off = __umul24((unsigned)kk[i], k_rowb) + kcon[i];
      if constexpr ((i & 3) == 0)
        gather16_first(kbase_m4k, off, lds0 + C::K_OFF + slot * C::TENSOR_BYTES + (wv * C::RPW + i * C::RPI) * C::ROWB);
      else
        gather16_next<(i & 3)>(kbase_m4k, off);
    };
    auto gather_v = [&](auto ic, int slot, const int (&kk)[C::IPW]) {
      constexpr int i = decltype(ic)::value;
      if constexpr (PART == PART_COMPUTE) return;
      const unsigned off = __umul24((unsigned)kk[i], v_rowb) + vcon[i];
      if constexpr ((i & 3) == 0)
        gather16_first(vbase_m4k, off, lds0 + C::V_OFF + slot * C::TENSOR_BYTES + (wv * C::RPW + i * C::RPI) * C::ROWB);
      else
        gather16_next<(i & 3)>(vbase_m4k, off);
    };
    // all of one tile's K (or V) gathers of this wave, back to back (prologue)
    auto burst_k = [&](int slot, const int (&kk)[C::IPW]) {
      gather_k(std::integral_constant<int, 0>(), slot, kk);
      if constexpr (C::IPW > 1) gather_k(std::integral_constant<int, 1>(), slot, kk);
      if constexpr (C::IPW > 2) { gather_k(std::integral_constant<int, 2>(), slot, kk); gather_k(std::integral_constant<int, 3>(), slot, kk); }
      if constexpr (C::IPW > 4) {
        gather_k(std::integral_constant<int, 4>(), slot, kk); gather_k(std::integral_constant<int, 5>(), slot, kk);
        gather_k(std::integral_constant<int, 6>(), slot, kk); gather_k(std::integral_constant<int, 7>(), slot, kk);
      }
    };
    auto burst_v = [&](int slot, const int (&kk)[C::IPW]) {
      gather_v(std::integral_constant<int, 0>(), slot, kk);
      if constexpr (C::IPW > 1) gather_v(std::integral_constant<int, 1>(), slot, kk);
      if constexpr (C::IPW > 2) { gather_v(std::integral_constant<int, 2>(), slot, kk); gather_v(std::integral_constant<int, 3>(), slot, kk); }
      if constexpr (C::IPW > 4) {
        gather_v(std::integral_constant<int, 4>(), slot, kk); gather_v(std::integral_constant<int, 5>(), slot, kk);
        gather_v(std::integral_constant<int, 6>(), slot, kk); gather_v(std::integral_constant<int, 7>(), slot, kk);
      }
    };

    // ---------------- accumulators ----------------
    f32x16 O[C::DBLK];
#pragma unroll
    for (int db = 0; db < C::DBLK; db++)
#pragma unroll
      for (int r = 0; r < 16; r++) O[db][r] = 0.0f;
    f32x16 SA, SB;             // S^T of even / odd tiles (one is turned into P while the other accumulates)
    i32x4 PA[2], PB[2];        // P^T (packed bf16 pairs) of even / odd tiles: B operands of the second MFMA
    float m_run = -INFINITY;   // exponent base (raw score units) of this lane's query: a score maximum it has seen
    float l_run = 0.0f, l_run2 = 0.0f;   // this lane's partial sum of exponentials, in two chains (even / odd scores)
    float m_pend = -INFINITY;  // running max of this lane's query, over the tiles whose exponentials have been formed
    float neg_mc = 0.0f;       // -m_run * c_log2, 0 while m_run is -inf: the additive term of the exponent
    auto set_base = [&](float m) {
      m_run = m;
      neg_mc = m == -INFINITY ? 0.0f : -m * a.c_log2;
    };

    constexpr int NE = C::SSTEPS;          // MFMA slots per phase: PV slot e = (d block e/2, key half e%2); QK slot e = d chunk e
    constexpr int AHEAD = 3;               // LDS fragment reads run this many slots ahead of their MFMA
    constexpr int VPS = 16 / NE;           // score values handled per slot
    // Gathers per iteration and wave: IPW of V then IPW of K, DMA_PER in each of the first slots of phase X.  The later
    // they go, the less of the iteration is left for them to land; the more at once, the longer they wait for each other
    // and keep this wave from issuing.  In the first four slots of eight: 12 heads x 32760 tokens at 64x1 2.06 ms (one
    // per slot 2.12, in two slots 2.13, all at the start 2.19), 24 heads x 118800 tokens at 128x1 31.1 (every other
    // slot 32.1).  A 32-row tile has one wave per workgroup and nobody to wait for at the barrier but its own gathers:
    // all 16 at the start, at 32x32 3.53 ms (in four slots 3.59, in eight 3.96).
    constexpr int NDMA = 2 * C::IPW;
    constexpr int DMA_PER = MT == 32 ? NDMA : (NDMA + 3) / 4;
    static_assert(DMA_PER * NE >= NDMA, "every gather has a slot");
    auto read_vf = [&](const unsigned char* vst, int e) {
      const int db = e >> 1, c = e & 1;
      const unsigned char* p0 = vst + voff[db] + (16 * c) * C::ROWB;
      s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FG_LDS s16x4*)(p0));
      s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((FG_LDS s16x4*)(p0 + 8 * C::ROWB));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // Phase X.  O^T += V^T P^T with V in slot `vrd` of the V ring and, with QK, Sn = K Q^T with K in slot `krd` of the K
    // ring: one MFMA of each per slot.  With EXP, every slot also takes its share of the exponentials of the previous
    // tile's scores So: P = exp2(c*(So - m)) packed to bf16 into Pout, the row sum, and this lane's part m_lane of the row
    // max; they issue while the two matrix instructions just issued execute.  With GATHER, the first slots then issue this
    // iteration's gathers: V rows (keys in vk) -> V slot `vwr`, then K rows (keys in kk) -> K slot `kwr`, both released by
    // the previous iteration.  The gather holds the wave; the matrix instructions execute underneath it.
    auto x_phase = [&](auto vrd_c, auto krd_c, auto vwr_c, auto kwr_c, const i32x4 (&Pin)[2], auto with_gather,
                       auto with_qk, f32x16& Sn, auto with_exp, const f32x16& So, i32x4 (&Pout)[2], float& l_new,
                       float& l_new2, float& m_lane) {
      constexpr int vrd = decltype(vrd_c)::value, krd = decltype(krd_c)::value;
      constexpr int vwr = decltype(vwr_c)::value, kwr = decltype(kwr_c)::value;
      constexpr bool GATHER = decltype(with_gather)::value;
      constexpr bool QK = decltype(with_qk)::value && PART != PART_GATHER;   // also Sn = K(slot krd) Q^T
      constexpr bool EXP = decltype(with_exp)::value && PART != PART_GATHER;  // also P = exp2(c*(So - m)) -> Pout, row sum
      const unsigned char* vst = smem + C::V_OFF + vrd * C::TENSOR_BYTES;
      const unsigned char* kst = smem + C::K_OFF + krd * C::TENSOR_BYTES;
      auto read_kf = [&](int s) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(kst + (kor ^ (32 * s))));
      };
      bf16x8 kf[NE];
      if constexpr (QK) {
#pragma unroll
        for (int e = 0; e < AHEAD; e++) kf[e] = read_kf(e);
#pragma unroll
        for (int r = 0; r < 16; r++) Sn[r] = 0.0f;
      }
      const bf16x8 pin[2] = {__builtin_bit_cast(bf16x8, Pin[0]), __builtin_bit_cast(bf16x8, Pin[1])};
      bf16x8 vf[NE];
#pragma unroll
      for (int e = 0; e < AHEAD; e++)
        if constexpr (PART != PART_GATHER) vf[e] = read_vf(vst, e);
      auto slot = [&](auto ec) {
        constexpr int e = decltype(ec)::value;
        if constexpr (PART != PART_GATHER) {
          if constexpr (e + AHEAD < NE) vf[e + AHEAD] = read_vf(vst, e + AHEAD);
          O[e >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[e], pin[e & 1], O[e >> 1], 0, 0, 0);
        }
        if constexpr (QK) {
          if constexpr (e + AHEAD < NE) kf[e + AHEAD] = read_kf(e + AHEAD);
          Sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[e], qf[e], Sn, 0, 0, 0);
        }
        if constexpr (EXP) {
#pragma unroll
          for (int x = 0; x < VPS; x += 2) {
            const int r = e * VPS + x;
            // masked keys hold S = -inf and c_log2 > 0 (the host substitutes a tiny positive value for
            // scale = 0), so their p is exactly 0 without a select
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(So[r], a.c_log2, neg_mc));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(So[r + 1], a.c_log2, neg_mc));
            l_new = (r == 0 ? l_run : l_new) + p0;   // (l_run stays, for the case that the base has to move: new_base)
            l_new2 = (r == 0 ? l_run2 : l_new2) + p1;
            m_lane = max3(r == 0 ? m_pend : m_lane, So[r], So[r + 1]);
            f32x2 pp = {p0, p1};
            int pk = __builtin_bit_cast(int, __builtin_convertvector(pp, bf16x2));
            asm volatile("" : "+v"(pk));   // keeps the compiler from sinking the conversion out of the slot
            Pout[r >> 3][(r & 7) >> 1] = pk;
          }
        }
        if constexpr (GATHER) {
          [&]<int... I>(std::integer_sequence<int, I...>) {
            auto one = [&](auto jc) {
              constexpr int j = decltype(jc)::value;
              if constexpr (j < C::IPW) gather_v(std::integral_constant<int, j>(), vwr, vk);
              else if constexpr (j < NDMA) gather_k(std::integral_constant<int, j - C::IPW>(), kwr, kk);
            };
            (one(std::integral_constant<int, e * DMA_PER + I>()), ...);
          }(std::make_integer_sequence<int, DMA_PER>());
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      slot(std::integral_constant<int, 0>());
      slot(std::integral_constant<int, 1>());
      slot(std::integral_constant<int, 2>());
      slot(std::integral_constant<int, 3>());
      if constexpr (NE > 4) {
        slot(std::integral_constant<int, 4>());
        slot(std::integral_constant<int, 5>());
        slot(std::integral_constant<int, 6>());
        slot(std::integral_constant<int, 7>());
      }
    };
    // Masks the new scores Sn (tile Tm, par = Tm % 2) where keys of the tile do not count.  With MFMA (prologue only) it
    // first computes Sn = K Q^T with K in slot `kslot` of the K ring.
    auto y_phase = [&](auto kslot, int Tm, int par, f32x16& Sn, auto with_mfma) {
      constexpr bool MFMA = decltype(with_mfma)::value;
      // written before the barrier that precedes this phase; consumed at its end
      const int drop_tag = TELL_DROPS ? drops[par * DROP_SLOT] : 0;
      if constexpr (PART == PART_GATHER) return;
      if constexpr (MFMA) {
        const unsigned char* kst = smem + C::K_OFF + kslot * C::TENSOR_BYTES;
        auto read_kf = [&](int s) {
          return __builtin_bit_cast(bf16x8, *reinterpret_cast<const i32x4*>(kst + (kor ^ (32 * s))));
        };
        bf16x8 kf[NE];
#pragma unroll
        for (int e = 0; e < AHEAD; e++) kf[e] = read_kf(e);
#pragma unroll
        for (int r = 0; r < 16; r++) Sn[r] = 0.0f;
#pragma unroll
        for (int e = 0; e < NE; e++) {
          if (e + AHEAD < NE) kf[e + AHEAD] = read_kf(e + AHEAD);
          Sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[e], qf[e], Sn, 0, 0, 0);
        }
      }
      bool masked = (Tm + 1) * C::NT > total;   // (the same in every wave of the workgroup)
      if constexpr (SHORT_GROUP && !GROUPED && WV == 1) masked |= lone_drop[par] != 0;
      if constexpr (TELL_DROPS) masked |= __builtin_amdgcn_readfirstlane(drop_tag) == tag0 + Tm;
      if constexpr (GROUPED)
        mask_members(Sn, members + par * C::NT + kw * 32, g, my_member);
      else if (__builtin_expect(masked, 0))
        mask_drop(Sn, dropped(Tm, par));
    };
    // The exponent base of every lane moves to the running max, which includes the scores So: their exponentials Pout and
    // sums were formed with the old base (some may be +inf) and are formed again; O does not hold that tile yet.
    auto new_base = [&](const f32x16& So, i32x4 (&Pout)[2], float& l_new, float& l_new2) {
#pragma clang fp contract(off)   // (l * alpha is rounded before the tile's sums are added to it)
      const float alpha = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_run - m_pend) * a.c_log2);
      set_base(m_pend);
      l_new = l_run * alpha;
      l_new2 = l_run2 * alpha;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(So[r], a.c_log2, neg_mc));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(So[r + 1], a.c_log2, neg_mc));
        l_new += p0;
        l_new2 += p1;
        f32x2 pp = {p0, p1};
        Pout[r >> 3][(r & 7) >> 1] = __builtin_bit_cast(int, __builtin_convertvector(pp, bf16x2));
      }
#pragma unroll
      for (int db = 0; db < C::DBLK; db++)
#pragma unroll
        for (int r = 0; r < 16; r++) O[db][r] *= alpha;
    };
    // at most N operations in flight, and the ids in register set e have arrived
    auto wait_ids = [&](auto n, int e) {
      if constexpr (DENSE) {
        wait_vmem_le<decltype(n)::value>();
      } else {
        wait_vmem_le<decltype(n)::value>(gi[e]);
        if constexpr (GROUPED) arrived(gm[e]);
      }
    };
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;
    // Iteration t, J = t mod U (a constant, so every LDS slot and register set is an immediate):
    //   X: O += V(t-1)^T P(t-1)^T  ||  S(t+1) = K(t+1) Q^T  ||  P(t) = exp(S(t) - m)  ||  gathers V(t+VS-2) and K(t+KS)
    //      into the slots that iteration t-1 read last
    // then, rarely: the exponent base moves, S(t+1) is masked.  The row max of S(t) belongs in X too: all of S(t) is there, so
    // its maxima issue under the matrix instructions.  After X, over S(t+1), they wait for the last of its products: 12
    // heads x 32760 tokens at 32x32 3.66 ms in X, 3.82 after it, at 64x1 2.11 and 2.13, 16 x 2635 at 32x8 24.4 and 25.1 us.
    // (Formed with the base that held until then, a tile's exponentials are formed again when it moves.)
    // A gathered tile has at least the barrier's wait to arrive before it is published, and whole
    // iterations more where the rings are deeper than two tiles.
    auto iteration = [&](auto jc, int t) {
      constexpr int J = decltype(jc)::value;
      constexpr int PAR = J & 1;
      i32x4 (&Pin)[2] = PAR ? PA : PB;
      i32x4 (&Pout)[2] = PAR ? PB : PA;
      f32x16& Sn = PAR ? SA : SB;
      const f32x16& So = PAR ? SB : SA;
      // K(t+1) and V(t-1) become visible to every wave: all but the WAITN most recent vector-memory operations of this
      // wave have completed (they complete in order), which covers its share of both tiles and the ids converted
      // below; every wave is done reading K(t) and V(t-2), whose slots this iteration refills
      constexpr int E = (J + KS) % IDL;
      wait_ids(std::integral_constant<int, WAITN>(), E);
      __syncthreads();
      if constexpr (!EARLY_PERMUTE) {   // ids requested IDL iterations ago -> key rows
        take_keys(t + KS, (J + KS) & 1, gi[E], gm[E], gr[E]);
        v_keys(t + VS - 2);
      }
      // wave priority: the gather phase above the vector-ALU phase above everything outside the key loop, so that
      // the waves that feed the memory pipe are issued first and a neighbour's prologue or epilogue never delays them
      // (measured: 1% faster at 64 and 128 rows, 3% with grouped tiles, 6% at 16x1; 4% slower at 32x32 in single-wave
      // workgroups: not used there.  For the dense kernels see where they are launched)
      if constexpr (WAVE_PRIO) __builtin_amdgcn_s_setprio(3);
      float l_new = l_run, l_new2 = l_run2, m_lane = m_pend;
      x_phase(std::integral_constant<int, (J + U - 1) % VS>(), std::integral_constant<int, (J + 1) % KS>(),
              std::integral_constant<int, (J + U - 2) % VS>(), std::integral_constant<int, J % KS>(), Pin, yes(), yes(), Sn,
              yes(), So, Pout, l_new, l_new2, m_lane);
      if constexpr (WAVE_PRIO) __builtin_amdgcn_s_setprio(1);
      if constexpr (PART != PART_GATHER) {
        m_pend = lane_pair_max(m_lane);
        // (the same in all lanes; the first valid key of a lane also moves it: m_run = -inf until then)
        const bool moves = __builtin_amdgcn_ballot_w64(m_pend > m_run + a.lazy_raw) != 0;
        if (__builtin_expect(moves, 0)) new_base(So, Pout, l_new, l_new2);
      }
      l_run = l_new;
      l_run2 = l_new2;
      fetch_ids(t + KS + IDL, gi[E], gm[E], gr[E]);
      y_phase(std::integral_constant<int, 0>(), t + 1, (J + 1) & 1, Sn, no());
      rotate_keys();
      if constexpr (EARLY_PERMUTE) {
        // the ids of the tile whose K rows the next iteration gathers have arrived (their load was followed by
        // AFTER_IDS operations): hand them to the lanes now, so that the permute's latency passes in the barrier
        constexpr int E1 = (J + 1 + KS) % IDL;
        wait_ids(std::integral_constant<int, AFTER_IDS>(), E1);
        take_keys(t + 1 + KS, (J + 1 + KS) & 1, gi[E1], gm[E1], gr[E1]);
        v_keys(t + 1 + VS - 2);
      }
    };

    if (ntiles > 0) {
      // prologue: K(0) .. K(KS-1) -> their K slots; V(0) .. V(VS-3) -> their V slots; V(0) also -> the V slot that the
      // first iteration reads as "V(-1)", only so that its O += V^T P^T (with P = 0) multiplies finite numbers; then
      // S(0) = K(0) Q^T
#pragma unroll
      for (int c = 0; c < 2; c++)
#pragma unroll
        for (int e = 0; e < 4; e++) PB[c][e] = 0;
      int pid[KS], pmb[KS], poff[KS];   // ids of tiles 0 .. KS-1, requested together with those of the first iterations
#pragma unroll
      for (int T = 0; T < KS; T++) fetch_ids(T, pid[T], pmb[T], poff[T]);
#pragma unroll
      for (int T = KS; T < KS + IDL; T++) fetch_ids(T, gi[T % IDL], gm[T % IDL], gr[T % IDL]);
      if constexpr (!DENSE) {
#pragma unroll
        for (int T = 0; T < KS; T++) {
          wait_vmem_le<0>(pid[T]);
          if constexpr (GROUPED) arrived(pmb[T]);
        }
#pragma unroll
        for (int e = 0; e < IDL; e++) wait_ids(std::integral_constant<int, 0>(), e);
      }
#pragma unroll
      for (int T = 0; T < KS; T++) {
        if (T > 0) rotate_keys();
        take_keys(T, T & 1, pid[T], pmb[T], poff[T]);
        burst_k(T, kk);
        if (T == 0) burst_v(VS - 1, kk);
        if (T <= VS - 3) burst_v(T, kk);
      }
      rotate_keys();   // (tiles VS-2 .. KS-1 are in sets 0 ..)
      if constexpr (EARLY_PERMUTE) {
        take_keys(KS, KS & 1, gi[KS % IDL], gm[KS % IDL], gr[KS % IDL]);
        v_keys(VS - 2);
      }
      wait_vmem_all();
      __syncthreads();
      // S(0) from K slot 0
      y_phase(std::integral_constant<int, 0>(), 0, 0, SA, yes());
      m_pend = row_max(SA);
      set_base(m_pend);   // O = 0 and l = 0 so far: the first exponent base needs no rescale
      int t = 0;
      for (;;) {
#define FG_STEP(J)                                             \
        if constexpr (U > J) {                                 \
          if (t >= ntiles) break;                              \
          iteration(std::integral_constant<int, J>(), t);      \
          t++;                                                 \
        }
        FG_STEP(0) FG_STEP(1) FG_STEP(2) FG_STEP(3) FG_STEP(4) FG_STEP(5)
        FG_STEP(6) FG_STEP(7) FG_STEP(8) FG_STEP(9) FG_STEP(10) FG_STEP(11)
#undef FG_STEP
      }
      if constexpr (WAVE_PRIO) __builtin_amdgcn_s_setprio(0);
      wait_vmem_all();
      if constexpr (!DENSE) {   // (the ids of tiles past the end, which nobody reads)
#pragma unroll
        for (int e = 0; e < IDL; e++) {
          arrived(gi[e]);
          if constexpr (GROUPED) arrived(gm[e]);
        }
      }
      __syncthreads();
      // O += V(ntiles-1)^T P(ntiles-1)^T: the slot and the register set depend on ntiles - 1 modulo lcm(VS, 2)
      constexpr int UD = clcm(VS, 2);
      const int jd = (ntiles - 1) % UD;
#define FG_DRAIN(J)                                                                                                   \
      if constexpr (UD > J) {                                                                                          \
        if (jd == J)                                                                                                   \
          x_phase(std::integral_constant<int, J % VS>(), std::integral_constant<int, 0>(), std::integral_constant<int, 0>(), \
                  std::integral_constant<int, 0>(), (J & 1) ? PB : PA, no(), no(), SA, no(), SA, PA, l_run, l_run2, m_pend);         \
      }
      FG_DRAIN(0) FG_DRAIN(1) FG_DRAIN(2) FG_DRAIN(3) FG_DRAIN(4) FG_DRAIN(5) FG_DRAIN(6) FG_DRAIN(7)
#undef FG_DRAIN
    }

    // ---------------- epilogue ----------------
    float l_tot = lane_pair_sum(l_run + l_run2);
    if (C::KW > 1) {
      __syncthreads();   // every wave is done with the tile buffers
      float* scratch = reinterpret_cast<float*>(smem);
      if (kw > 0) {
        float* dst = scratch + ((rw * (C::KW - 1) + kw - 1) * C::MERGE_REGS) * 64 + lane;
#pragma unroll
        for (int db = 0; db < C::DBLK; db++)
#pragma unroll
          for (int r = 0; r < 16; r++) dst[(db * 16 + r) * 64] = O[db][r];
        dst[(C::DBLK * 16) * 64] = m_run;
        dst[(C::DBLK * 16 + 1) * 64] = l_tot;
      }
      __syncthreads();
      if (kw == 0) {
#pragma unroll
        for (int pw = 0; pw < C::KW - 1; pw++) {
          const float* src = scratch + ((rw * (C::KW - 1) + pw) * C::MERGE_REGS) * 64 + lane;
          const float m_o = src[(C::DBLK * 16) * 64];
          const float l_o = src[(C::DBLK * 16 + 1) * 64];
          const float m_new = fmaxf(m_run, m_o);
          const float a_me = (m_run == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f((m_run - m_new) * a.c_log2);
          const float a_ot = (m_o == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f((m_o - m_new) * a.c_log2);
#pragma unroll
          for (int db = 0; db < C::DBLK; db++)
#pragma unroll
            for (int r = 0; r < 16; r++) O[db][r] = O[db][r] * a_me + src[(db * 16 + r) * 64] * a_ot;
          l_tot = l_tot * a_me + l_o * a_ot;
          m_run = m_new;
        }
      }
    }
    if (kw == 0) {
      const int row = my_row;
      if (my_row_valid) {
        const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
        uint16_t* op = a.out + b * a.o_sb + h * a.o_sh + (int64_t)row * a.o_sl;
#pragma unroll
        for (int db = 0; db < C::DBLK; db++)
#pragma unroll
          for (int r4 = 0; r4 < 4; r4++) {
            f32x4 f;
#pragma unroll
            for (int e = 0; e < 4; e++) f[e] = O[db][4 * r4 + e] * inv;
            bf16x4 o4 = __builtin_convertvector(f, bf16x4);
            *reinterpret_cast<i32x2*>(op + 32 * db + 8 * r4 + 4 * g) = __builtin_bit_cast(i32x2, o4);
          }
        if (g == 0) {
          const float lse = l_tot > 0.0f ? a.scale_abs * m_run + __logf(l_tot) : -INFINITY;
          a.lse[(int64_t)slice * a.L + row] = lse;
        }
      }
    }
    tag0 += ntiles + KS + IDL + 1;
    // this item's LDS use (tile rings, merge scratch) ends here; the next item's begins with the work-item word
    __syncthreads();
  }
}

}  // namespace fg
