// Matrix-core fused int4 decode attention for gfx950 (phase 1 of Sec. 3.2: per-chunk partials; up to 32 chunks
// to a row also phase 2, the chunk merge of Eq. 6, done by the wave that has the row last).
//
// Why matrix cores: with a GQA group of G query heads every stored element is used by G heads;
// at G=8 and d=128 that is 25.6 flop per HBM byte, above the vector-ALU ridge of the chip, so the
// two contractions (the score step and the accumulator update of Alg. 1) run on v_mfma_f32_16x16x32_f16 and the vector ALU only
// unpacks nibbles, applies the per-group scale/zero-point of K and does the softmax.
//
// Data path: the packed stream never passes through vector registers on its way in.  Each wave owns
// a ring of LDS stages and fills them with direct global->LDS loads (global_load_lds_dwordx4: 64
// lanes x 16 B = 1 KB per instruction, tracked by vmcnt), one 32-token supertile ahead of the one
// being consumed, with no register cost; the per-lane source address of such a load is free, so K
// codes and the fp16 scale / zero-point arrays are gathered into the order the lanes read them back
// in.  What a supertile needs from LDS is copied into registers ahead of use (its V part at the start
// of its K phase, the next supertile's K part during the current softmax / P V phase).  The ring is
// only two stages deep on purpose: once the last byte has landed every wave still has `ring depth`
// supertiles to compute, and at 16 supertiles per wave that drain outweighs a deeper prefetch.
// The stream is read once, and its loads say so (non-temporal cache policy, template parameter NT).
//
// Exactness: codes 0..15 enter the MFMA as fp16 SUBNORMALS (the nibble sits in the low mantissa
// bits, value c*2^-24, or c*2^-20 for a nibble at bit 4) so unpacking is one AND per pair of
// elements; products and sums are exact in the fp32 accumulator.  Scale and zero-point are applied
// outside the contraction:  q.k^ = sum_g s_g (q_g.c_g - z_g sum(q_g))  in fp32 on the vector ALU, and
// sum_t p_t v^_t = sum_t (p_t s_t) c_t - sum_t (p_t s_t) z_t, where the product p_t s_t is rounded
// to fp16 once and the SAME rounded operand multiplies the codes and (in a small extra MFMA whose
// B operand is the stored fp16 zero-point itself) the zero-points.
// The matrix core aligns the 32 products of an MFMA to its fp32 accumulator and TRUNCATES each of
// them, so an accumulator that grows (a sum of positive terms, ~200x larger than the result it is
// later differenced into) costs accuracy in proportion to the tokens it has taken in.  Both sums are
// therefore kept balanced around zero, at no cost in matrix instructions: a supertile is two 16-token
// tiles, and the weights of the SECOND tile enter the A operand negated.  For the codes the second
// tile's nibbles are complemented (15 - c, one NOT per packed word):
//   sum_t0 w c - sum_t1 w (15 - c)  =  sum_t w c  - 15 sum_t1 w ,
// for the zero-points the second tile's B entries get their sign flipped and a constant B operand
// (0 on first-tile slots, 15 on second-tile slots) follows:
//   sum_t w z - 15 sum_t1 w .
// The two 15 sum_t1 w terms cancel in the difference, exactly (same A operand), and each running sum
// stays at the size of the result.
//
// Mapping (one 64-lane wave; lane = 16*kq + c):
//   QK^T is computed transposed, S^T = K Q^T: A = codes (row = token, 8 k-slots per lane = one packed
//   word), B = query.  The 16 B-columns hold G (padded to GP) heads x 16/GP group replicas: column
//   (h, r) only has non-zero query entries on the k-slots of "its" groups, so one accumulator holds
//   the per-group partial dot products of several groups side by side and the per-group scale is
//   applied to NA = (d/32)/(16/GP) accumulators instead of d/32.  Replicas are summed with DPP
//   row rotations.  The S^T accumulator layout (lane = head column, 4 token rows per lane block) is
//   the A-operand layout of P V when P V is computed as rows (h, r) x columns (dims): lane (h, r) of
//   block kq already holds the probabilities of its 8 tokens, so they never move between lanes.
//   For P V the contraction runs over tokens, so each lane needs 8 tokens of one dim in its k-slots:
//   it reads the same packed word of 8 tokens and regroups it with one v_perm_b32 per (token pair, byte);
//   a byte's two nibbles go through the matrix core mixed (n_even + 16 n_odd, still an exact subnormal)
//   next to n_even alone, and the odd dim is recovered from the two sums at the end (see `pv`).
//
// Work split: grid (n_splits, H_kv * kv_share, B), 8 waves per block, one block per compute unit; the
// waves of a block share the chunk's 32-token supertiles in a fixed pattern (17:15 or 9:7 between the older
// and the younger wave of a SIMD, see the kernel), keep private online-softmax state, and are merged through
// LDS so that the block writes one partial (o_c, m_c, l_c) per query row.  Where there are more rows, or slots of a
// device-planned chunk list, than the chip holds blocks, 2, 4 or 8 of them share a block; many rows of their own
// lengths get blocks of 8, 4, 2 or 1 waves, one per row, longest first (`ranked` in the kernel); and where that does not
// pay, the waves of one round of blocks are dealt to the sequences in proportion to their lengths (LISTED).
//
// Query rows: the tile's GP columns take the G heads of the GQA group (Sec. 3.1), or, with several query
// tokens per sequence (the sequence's last n_queries tokens, causal among themselves), the n_queries * G
// rows (token, head) of one KV head; rows beyond one tile go to further blocks on the same KV head
// (kv_share of them).  Per-row limits (causal end, window start) only exist in the masked path that the
// ragged last supertile takes anyway.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <unordered_map>

#include "tq_internal.h"

namespace tq {
namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

constexpr float kNegBig = -1.0e30f;
constexpr int kMaxDevices = 64;

// Arrival counters of the in-kernel chunk merge: one per output row, in kCounterSlots independent sets.  A set
// belongs to ONE WORKSPACE (the host keeps the table, see merge_slot_of): calls that may be in flight at the same
// time have different workspaces by the contract of the decode calls (they would overwrite each other's partials
// otherwise), hence different sets, whether they are issued eagerly or replayed from a captured graph, which
// keeps the set it was captured with.  Zero when the module is loaded; the block that arrives last wraps its
// counter back to zero, so every launch leaves them zero again.  A workspace that finds all sets taken gets the
// merge kernel instead (two launches: always correct).
constexpr int kCounterSlots = 256;
constexpr int kCountersPerSlot = 16384;
// Within a set, the counters of neighbouring rows lie 128 bytes apart (row r at (r % 512) * 32 + r / 512):
// the blocks of a launch finish at about the same time, and their atomics on counters that share a cache line
// queue up behind one another at that line's channel (8 KV heads x 32 chunks on one line: 1.4 us of a 13 us call).
__device__ __attribute__((aligned(256))) unsigned int g_arrivals[kCounterSlots * kCountersPerSlot];
static_assert(kCountersPerSlot == 512 * 32, "the spreading below");
__device__ __forceinline__ int arrival_counter(int row) { return (row & 511) * 32 + (row >> 9); }
constexpr float kSlack = 2.0f;              // log2 units: exp2(score - reference) <= 4
constexpr uint32_t kMaskLo = 0x000F000Fu;   // nibbles 0 and 4 of a word -> fp16 subnormals c * 2^-24
constexpr uint32_t kMaskHi = 0x00F000F0u;   // nibbles 1 and 5           -> c * 2^-20
constexpr uint32_t kPos15Odd = 0x4B800000u; // fp16 pair (0, 15): k-slots alternate first tile, second tile

template <int D, int GP, int NW, int GS = 0>
struct Cfg {
  static constexpr int NG = D / kGroup;          // quantisation groups per token
  static constexpr int GR = 16 / GP;             // group replicas among the 16 columns / rows
  static constexpr int NA = NG / GR;             // groups handled per lane (accumulators per K tile)
  static constexpr int NJ = NG;                  // K MFMAs per 16-token tile (= packed words per lane)
  static constexpr int NCS = D / 128;            // V column sets (16 packed words each)
  static constexpr bool SWAP = (D == 128 && GP == 8);
  // WIDE: every column of the tile is a query row of its own (no group replicas), so each of the four groups of
  // a token has its own score accumulator, and the P V columns are regrouped so that the 16 columns of one
  // matrix instruction lie in ONE group (see `pv`): its A operand p * s_v is then right for all of them.
  static constexpr bool WIDE = (GR == 1);
  static constexpr int NDW = (NA + 1) / 2;       // dwords of fp16 scales (or zero-points) a lane needs per token
  static_assert(NG % GR == 0 && NA >= 1 && (NA <= 2 || (WIDE && D == 128)), "unsupported (head_dim, padded GQA) pair");
  // K MFMA j takes, from lane block kq, packed word a_word(j,kq) of group a_group(j,kq) and adds
  // into accumulator acc(j); column replica r of that accumulator stands for group r*NA + acc(j).
  static __device__ constexpr int a_group(int j, int kq) {
    return WIDE ? j : SWAP ? 2 * (kq >> 1) + (j & 1) : (D == 128 ? kq : 2 * kq + (j >> 2));
  }
  static __device__ constexpr int a_word(int j, int kq) {
    return WIDE ? kq : SWAP ? 2 * (j >> 1) + (kq & 1) : (D == 128 ? j : (j & 3));
  }
  static __device__ constexpr int acc(int j) {
    return WIDE ? j : SWAP ? (j & 1) : (D == 128 ? 0 : (NA == 2 ? (j >> 2) : 0));
  }

  // LDS stage of one 32-token supertile, in the order the stream is laid out in HBM
  static constexpr int TB = D / 2;               // bytes of codes per token
  static constexpr int KT = 16 * TB;             // one 16-token K tile
  static constexpr int VB = 32 * TB;             // V codes of the supertile
  // one fp16 scale (or zero-point) array of the supertile.  Where it lies token by token in LDS (d = 256), larger
  // groups keep it compact, NGM values per token; the gathered layouts (PERM, WIDE below) always fill NG places.
  static constexpr int NGM = D == 256 ? NG >> GS : NG;
  static constexpr int SZ = 32 * NGM * 2 > 256 ? 32 * NGM * 2 : 256;
  static constexpr int OFF_V = 2 * KT, OFF_KS = OFF_V + VB, OFF_KZ = OFF_KS + SZ, OFF_VS = OFF_KZ + SZ,
                       OFF_VZ = OFF_VS + SZ, STAGE = OFF_VZ + SZ;
  static constexpr int NS = 2;                  // ring depth per wave (LDS: 160 KB per CU)
  // The two waves of a SIMD split its supertiles (PER / 2 + 1) : (PER / 2 - 1), the older wave the larger share:
  // 17 : 15 where the loop is leanest (measured: the older wave of the d = 128, 8-row kernel takes 1.32 us per
  // supertile, the younger 1.45 us), 9 : 7 elsewhere
  static constexpr int PER = (D == 128 && GP == 8) ? 32 : 16;
  static constexpr int LPS = 2 * (KT / 1024) + VB / 1024 + 4 * (SZ / 256);   // load instructions per stage
  static constexpr int RING = NW * NS * STAGE;
  static constexpr int NEWTOK = D + GP;          // floats of a unit's new token: its dequantised V, its scores
  static constexpr int MERGE = (NW * GP * D + 2 * NW * GP + NW * NEWTOK) * 4;  // o, m, l, and the units' new tokens
  // the block-merge area sits behind the rings where both fit into the 160 KB of a compute unit, else on top of them
  static constexpr bool ALIAS = RING + MERGE > 160 * 1024;
  // Where the query block of a wave lands before it is turned into operands: in an area of its own if
  // there is room, so that the whole ring can be filled at once; else in the last ring slot.
  // (1 KB behind it: the new token's K and V rows of a step, see `takes`)
  static constexpr int QBLK = GP * D * 2, QAREA = QBLK + 1024;
  static_assert(QAREA <= STAGE, "the query block borrows one ring slot");
  static constexpr bool QSEP = !ALIAS && RING + MERGE + NW * QAREA <= 160 * 1024;
  static constexpr int SMEM = ALIAS ? (RING > MERGE ? RING : MERGE) : RING + MERGE + (QSEP ? NW * QAREA : 0);
  // The fp16 scale and zero-point arrays are fetched dword by dword (two groups of one token), and the
  // direct loads may gather: with NA == 2 a lane needs exactly one dword per token, so the dwords are
  // laid out in LDS as [kq][replica][tile][i] and a lane reads its eight tokens with two 16-byte reads; with
  // NA == 4 (WIDE) it needs both dwords of a token: [kq][dword][tile][i], four 16-byte reads.
  static constexpr bool PERM = (NA == 2);
  // Whether the K part of the next supertile is fetched into registers during the current one (it is
  // not where the accumulators alone take half of the register file).
  static constexpr bool PFK = !(D == 256 && NA == 2);
  static __device__ constexpr int sz_token(int P) {       // token (0..31) whose dword sits at stage dword P
    return WIDE ? 16 * ((P >> 2) & 1) + 4 * (P & 3) + (P >> 4)
                : PERM ? 16 * ((P >> 2) & 1) + 4 * (P & 3) + (P >> 3) / GR : (P / (NGM / 2)) & 31;
  }
  static __device__ constexpr int sz_column(int P) {      // which dword of that token's NG/2
    return WIDE ? (P >> 3) & 1 : PERM ? (P >> 3) % GR : P % (NGM / 2);
  }
};

// token held by row r of a 16-token K tile (and by the matching k-slots of the P V contraction):
// lane block kq then owns tokens kq, kq+4, kq+8, kq+12 of each tile, which keeps the four blocks'
// LDS reads of the V codes on different banks
__device__ __forceinline__ constexpr int tok_of_row(int r) { return 4 * (r & 3) + (r >> 2); }

__device__ __forceinline__ half8v as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_bit_cast(half8v, uint4v{a, b, c, d});
}
__device__ __forceinline__ half8v unpack_word(uint32_t w) {   // 8 nibbles -> 8 fp16 subnormals
  const uint32_t s = w >> 8;
  return as_half8(w & kMaskLo, w & kMaskHi, s & kMaskLo, s & kMaskHi);
}
__device__ __forceinline__ float4v mfma16(half8v a, half8v b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
template <int ROT>
__device__ __forceinline__ float row_ror_add(float x) {      // x + (x rotated by ROT inside its 16-lane row)
  const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + ROT, 0xF, 0xF, false);
  return x + __builtin_bit_cast(float, y);
}

// ---- direct global -> LDS loads.  Written as asm so that the compiler does not serialise them
// against later LDS reads: each wave tracks its own ring with explicit vmcnt waits instead.
// Lane l's bytes land at lds_base + l * (16 | 4).  M0 carries the LDS base of the instruction.
// (M0 cannot be named as a clobber: the compiler reserves it and rejects that.  It keeps no value live in M0
// across other instructions either: each of its own uses, such as an indexed register move, writes M0 right
// before.  The kernels in this file and in tq_decode_wide.hip contain no such use at all: in their assembly M0
// appears inside these blocks only.)
// NT = the non-temporal cache policy: the packed stream is read once, and telling the caches so is worth
// 6-9 % of the kernel's time (plain loads of the same 168 MB: 28 us per launch, non-temporal: 25 us).
// Where several blocks stream the same KV head the later readers live on what the first left in the
// caches, and the loads stay plain.
#define TQ_LDS_LOAD(NT_, TEXT_PLAIN, TEXT_NT, ...)                     \
  do {                                                                 \
    if constexpr (NT_) asm volatile(TEXT_NT :: __VA_ARGS__ : "memory"); \
    else asm volatile(TEXT_PLAIN :: __VA_ARGS__ : "memory");           \
  } while (0)
template <bool NT>
__device__ __forceinline__ void dma4(const void* sbase, uint32_t voff, uint32_t lds_base) {
  TQ_LDS_LOAD(NT, "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1",
              "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1 nt",
              "v"(voff), "s"(sbase), "s"(lds_base));
}
__device__ __forceinline__ void dma16_lane(const void* addr, uint32_t lds_base) {   // per-lane 64-bit address
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(addr), "s"(lds_base) : "memory");
}
__device__ __forceinline__ void dma4_lane(const void* addr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
               :: "v"(addr), "s"(lds_base) : "memory");
}
// Several loads of one array behind a single M0: the instruction's immediate offset moves the global
// and the LDS address alike, so pieces that are equally far apart on both sides share the base.
template <bool NT, int O1>
__device__ __forceinline__ void dma16_x2(const void* sbase, uint32_t voff, uint32_t lds_base) {
  TQ_LDS_LOAD(NT, "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
                  "global_load_lds_dwordx4 %0, %1 offset:%3",
              "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\t"
              "global_load_lds_dwordx4 %0, %1 offset:%3 nt",
              "v"(voff), "s"(sbase), "s"(lds_base), "n"(O1));
}
template <bool NT, int O0, int O1>
__device__ __forceinline__ void dma16_x2o(const void* sbase, uint32_t voff, uint32_t lds_base) {
  TQ_LDS_LOAD(NT, "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3\n\t"
                  "global_load_lds_dwordx4 %0, %1 offset:%4",
              "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3 nt\n\t"
              "global_load_lds_dwordx4 %0, %1 offset:%4 nt",
              "v"(voff), "s"(sbase), "s"(lds_base), "n"(O0), "n"(O1));
}
template <bool NT>
__device__ __forceinline__ void dma16_x4(const void* sbase, uint32_t voff, uint32_t lds_base) {
  TQ_LDS_LOAD(NT, "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\t"
                  "global_load_lds_dwordx4 %0, %1 offset:1024\n\tglobal_load_lds_dwordx4 %0, %1 offset:2048\n\t"
                  "global_load_lds_dwordx4 %0, %1 offset:3072",
              "s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\t"
              "global_load_lds_dwordx4 %0, %1 offset:1024 nt\n\tglobal_load_lds_dwordx4 %0, %1 offset:2048 nt\n\t"
              "global_load_lds_dwordx4 %0, %1 offset:3072 nt",
              "v"(voff), "s"(sbase), "s"(lds_base));
}
// device-scope (all compute dies) store and load of two floats, without any cache-wide maintenance
__device__ __forceinline__ void st_dev2(float* p, float a, float b) {      // two floats, 8-byte aligned
  const uint64_t bits = (uint64_t)__builtin_bit_cast(uint32_t, a) | ((uint64_t)__builtin_bit_cast(uint32_t, b) << 32);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_dev2(const float* p) {                 // two floats, 8-byte aligned
  const uint64_t bits = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return {__builtin_bit_cast(float, (uint32_t)bits), __builtin_bit_cast(float, (uint32_t)(bits >> 32))};
}
template <int N>
__device__ __forceinline__ void wait_loads() {               // until at most N loads are outstanding
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// PLAIN = the launch has none of the per-sequence machinery: one common length, a contiguous cache, one query
// token, one block per (chunk, KV head, sequence).  Everything below that serves the other shapes then folds
// away at compile time; what is left is a short prologue (the first loads leave sooner) and a loop without the
// scalar bookkeeping of pages and packed rows.
//
// GS = log2(group size / 32).  Groups of 64 or 128 elements (Sec. 2.1) change what the stored scales and zero-points
// MEAN, not what the kernel does with them: the direct loads fetch, for every 32-dim block of a token, the dword
// that holds its group's value (one dword of two groups per token at 64, one dword of two TOKENS at 128), and the
// lane copies the half it needs into both halves of the register, after which everything is as with groups of 32.
// That is for the layouts whose metadata is gathered dword by dword (d = 128 with 8 or 16 rows).  At d = 256 a lane
// reads one halfword per token and array anyway: the stage holds the arrays as they are, and only the halfword's
// address changes with the group.
//
// SPLIT (d = 256 with larger groups): the weights p s_v go through the matrix core as TWO fp16 operands, their
// leading part and the rest: 22 bits, where the generic kernel that served these shapes before has fp32's 24; queries
// enter whole (see q_up), and sums are the matrix core's.  Error of the output against 64 bits next to the generic
// kernel's (fp16 rounding of the output is nearly all of both): 1.00002 of it over ten shapes of 600 .. 32K tokens and
// three seeds, at most 1.0001.  The reference of the exponentials then also carries an offset that keeps the largest weight
// near 2^10 whatever the size of the scales (see `softmax`), or small scales would push the rest below fp16's range.
// The matrix cores have the room (52 instructions per supertile instead of 34, a quarter of its time), and the kernel
// is bound by the stream like its groups-of-32 instance: 32 heads on 16 KV heads, one sequence of 32K tokens, groups of
// 64 (151 MB), the whole step 305.5 us on the generic kernel, 31.4 us here.
//
// PAGED = a pool of pages (with PLAIN: never).  An instance of its own keeps the page look-ups out of the others'
// scalar registers, of which the general instance has none to spare.
//
// LISTED: sequences with lengths of their own, one query token, no window (DecodeParams::listed), in a contiguous cache or in pages.
// With a wave to a slot a short sequence has one or two waves where it had eight, and as many references of the exponentials, each of
// which makes the weight of its largest score exact in fp16.  So the weights of sequences of fewer than kTwoBelow slots go in two parts
// (TWO, d = 128; a loop of its own, the other waves' is as it was), and at d = 256 all of them do (SPLIT).  Error against 64 bits, 64 sequences
// of 128 .. 4096 tokens: before 2.33e-4, one operand 2.60e-4, this 2.19e-4, two for all 2.08e-4 (but 0.2 us per tile: the 24
// paged sequences 38.5 -> 42.4 us per step); 2048 .. 4096 2.56e-4 / - / 2.56e-4; d = 256 2.87e-4 / 2.89e-4 / 2.07e-4 at 2 - 4 % of the time.
// Sequences of three slots and more, each by itself (six mixes, three seeds): 2.36e-4 .. 2.67e-4 before, 2.31e-4 .. 2.62e-4 now, by the number of their slots
// 0.96 .. 1.03 of what they had, three to seven slots 0.98 .. 1.015, on the whole the same.
enum Mode { kPlain, kPlainStep, kGeneral, kPaged, kListed, kListedPaged };   // kPlainStep: see LEAN
// LEAN: the 16-row tile's instances for plain launches and for blocks that share a KV head take no new token and come to
// the masked last supertile at the end.  Two stretches of code that few waves run, between the prologue and the loop, cost
// these launches, which are short, half a microsecond (why is open: the instruction cache is warm from launch to launch): 128 heads over 8, 8K tokens,
// decode 13.54 us with both, 13.5 with either, 13.02 with neither; 3.3K 12.87 / 12.40; 4 query tokens, 64 heads over 8,
// 32K, 26.5 / 26.1 per step.  (With up to eight rows the steps gain more by both than this costs.)  The step of one short
// sequence, whose only launch takes the token in, keeps a plain instance with both: 128 heads over 8, 300 tokens, 11.3 us,
// 12.3 with an append launch or the general instance.
template <int GP, bool NT, Mode MODE, int GS>
constexpr bool lean_tile() { return GP == 16 && GS == 0 && (MODE == kPlain || !NT); }
template <int D, int GP, int NW, bool NT, Mode MODE, int GS = 0>
__global__ __launch_bounds__(NW * 64, (NW + 3) / 4) void decode_partial_mfma_kernel(DecodeParams p) {
  constexpr bool PLAIN = MODE == kPlain || MODE == kPlainStep, LISTED = MODE == kListed || MODE == kListedPaged;
  constexpr bool paged = MODE == kPaged || MODE == kListedPaged;
  using C = Cfg<D, GP, NW, GS>;
  static_assert(GS == 0 || D == 256 || ((C::PERM || C::WIDE) && !PLAIN), "larger groups at d = 128: the gathered layouts");
  constexpr bool SPLIT = D == 256 && (GS > 0 || LISTED), MAY_TWO = D == 128 && LISTED;
  constexpr bool LEAN = lean_tile<GP, NT, MODE, GS>();
  constexpr int NGM = C::NGM;
  constexpr int SZB = (D / kGroup * 2) >> GS;     // bytes of one metadata array per token
  constexpr int NG = C::NG, NA = C::NA, NJ = C::NJ, NCS = C::NCS, TB = C::TB, NS = C::NS, LPS = C::LPS, GR = C::GR;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  if constexpr (PLAIN) {
    // every kernel argument the prologue needs, asked for at once: one round trip to the scalar cache before the
    // first stream loads leave instead of two (the compiler otherwise fetches q and start behind a branch)
    asm volatile("" :: "s"(p.q), "s"(p.start), "s"(p.k_codes), "s"(p.v_codes), "s"(p.k_scale), "s"(p.k_zero),
                 "s"(p.v_scale), "s"(p.v_zero), "s"(p.seq_len), "s"(p.tokens_per_split), "s"(p.row_stride),
                 "s"(p.n_kv_heads), "s"(p.n_q_heads), "s"(p.gqa), "s"(p.k_new));
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, kq = lane >> 4;
  const int hl = c % GP, rep = c / GP;            // head and group replica of this lane's column / row
  int split = blockIdx.x, b = blockIdx.z, tokens_per_split = p.tokens_per_split, part_stride = p.n_splits;
  int kvv = blockIdx.y;                           // KV head x part of its query group (see kv_share)
  // Many short sequences (more units of work than the chip holds blocks): a block takes NW / W of them, W waves
  // each, instead of one.  With a common length a unit is a (sequence, KV head) row of a single chunk, and
  // blockIdx.y counts groups of rows of the list [batch][KV head x part]; with per-sequence lengths a unit is a
  // slot of the chunk list, and blockIdx.x counts groups of slots.  A wave past the end of its list has no tokens
  // and only keeps the barriers company.
  int W = PLAIN ? NW : p.waves_per_row;           // NW: the whole block on one unit
  int tokens_chunk = 0;                           // (LISTED: tokens of the block's part of the sequence)
  bool row_valid = true;
  // Rows of their own lengths, the longest first (`ranked`), a block of n_waves waves each: the launch holds about two
  // rounds of blocks, and what evens out the mix is the machine itself: a compute unit that is done with a row takes
  // the next longest one.  Where the lengths are too even for that to pay (the second round costs a row's fixed time
  // once more), a block takes two rows that follow each other, half its waves each, in one round, and the other half
  // of the blocks ends at once.  blockIdx.z: the place in the order of lengths (of a row, or of a pair).
  const bool ranked = !PLAIN && !LISTED && p.ranked;
  const int n_waves = ranked ? W : NW, n_units = ranked ? 2 : NW;
  if (ranked) {
    int rank = blockIdx.z;
    auto place = [&](const auto& rows) {          // false: a block with nothing to do
      if (rows.even) {
        W = n_waves >> 1;
        rank = 2 * rank + wave / W;
        if (2 * blockIdx.z >= (unsigned)p.batch) return false;
        row_valid = rank < p.batch;
        rank = min(rank, p.batch - 1);
      }
      b = __builtin_amdgcn_readfirstlane(rows.sequence(p, rank));
      return true;
    };
    // (lists of up to 256 sequences keep a form of their own: the eight registers of the longer one cost them 1.7 us, and
    // its code on their way 0.2.
    // 300 sequences of 64 .. 2048 tokens, 32 heads over 4, taken in the given order and two to a block 77.9 us per step,
    // ordered 39.7; 512 of 64 .. 1024, 64 heads over 8, 76.8 / 66.0; 512 of 64 .. 4096, 8 heads over 1, 41.1 / 33.1)
    if (!(__builtin_expect(p.batch <= 256, 1) ? place(RankedRows<4>(p)) : place(RankedRows<kRankMaxBatch / 64>(p)))) return;
  }
  int planned_len = -1;                           // (known from the plan: the lengths need not be fetched again)
  // (LISTED) the waves of this block that hold the same sequence as this one: they share the block's part of it like the waves of a
  // block share a chunk; that sequence's partials (one per block that holds any of it), and which of them this block's is
  int first_mate = 0, n_parts = 1, part_at = 0;
  bool two = false;
  if constexpr (LISTED) {
    kvv = blockIdx.x;
    VarPlan vp;
    vp.b = 0;
    vp.chunk = 0;
    vp.len = 0;
    row_valid = var_plan<true, MAY_TWO>(p, (int)blockIdx.y * NW + wave, vp);
    const int lg = vp.waves == NW ? 3 : 0, per = NW >> lg, slot0 = (int)blockIdx.y * per, slot = slot0 + (wave >> lg);
    if (!row_valid && slot0 >= vp.chunks) return;  // (the whole block lies past the end of the list)
    planned_len = __builtin_amdgcn_readfirstlane(vp.len);
    b = __builtin_amdgcn_readfirstlane(vp.b);
    tokens_per_split = __builtin_amdgcn_readfirstlane(vp.chunk_tokens);
    part_stride = kMaxSplits;
    split = __builtin_amdgcn_readfirstlane(vp.chunk);
    if (row_valid) {
      const int first = slot - split, end = first + __builtin_amdgcn_readfirstlane(vp.chunks);      // the sequence's slots
      const int from = max(first, slot0), to = min(end, slot0 + per);                               // those of them in this block
      part_at = (int)blockIdx.y - (first >> (3 - lg));
      n_parts = ((end - 1) >> (3 - lg)) - (first >> (3 - lg)) + 1;
      first_mate = (from - slot0) << lg;
      W = (to - from) << lg;
      split = from - first;
      two = __builtin_amdgcn_readfirstlane(vp.two ? 1 : 0) != 0;
      tokens_chunk = (to - from) * tokens_per_split;
    } else {
      first_mate = wave;
      W = 1;
    }
    static_assert(NW == 8, "a slot is one wave or a block");
  }
  const bool whole = W == NW;
  const int sub = LISTED ? wave - first_mate : wave % W;       // (several rows per block: the W waves of a row take its supertiles in turn)
  if (!PLAIN && !LISTED && !whole && !ranked && p.var_chunks == 0) {
    const int rows_y = p.n_kv_heads * p.kv_share, total = p.batch * rows_y;
    const int row = blockIdx.y * (NW / W) + wave / W;
    row_valid = row < total;
    const int r = min(row, total - 1);
    b = __builtin_amdgcn_readfirstlane(r / rows_y);
    kvv = __builtin_amdgcn_readfirstlane(r - (r / rows_y) * rows_y);
  }
  const int kv_share = PLAIN || LISTED ? 1 : p.kv_share;
  const int kv = PLAIN || LISTED ? kvv : kvv / kv_share;       // the KV head whose rows are read
  if (!PLAIN && !LISTED && p.var_chunks > 0) {    // per-sequence lengths: which (sequence, chunk) is this block's
    VarPlan vp;
    vp.b = 0;
    vp.chunk = 0;
    vp.len = 0;
    const bool listed = var_plan(p, whole ? blockIdx.x : blockIdx.x * (NW / W) + wave / W, vp);
    if (whole && !listed) return;                 // (with several units per block nobody leaves before the barriers)
    row_valid = listed;
    planned_len = __builtin_amdgcn_readfirstlane(vp.len);
    split = __builtin_amdgcn_readfirstlane(vp.chunk);     // (wave-uniform by construction: tell the compiler)
    b = __builtin_amdgcn_readfirstlane(vp.b);
    tokens_per_split = __builtin_amdgcn_readfirstlane(vp.chunk_tokens);
    part_stride = kMaxSplits;
  }
  const int G = p.gqa;
  // Several query tokens per sequence (they are the sequence's last NQ tokens and causal among themselves):
  // a KV head then has NQ * GF query rows, row r = t * GF + g for query token t and head g of the group,
  // cut into kv_share parts of G rows; this block holds rows part * G .. part * G + G - 1.
  const int NQ = PLAIN || LISTED ? 1 : p.n_queries, GF = PLAIN || LISTED ? G : p.gqa_full;
  const int part = kvv - kv * kv_share;
  auto query_token = [&](int h) { return NQ > 1 ? min(part * G + h, NQ * GF - 1) / GF : 0; };
  auto query_row = [&](int h) -> int64_t {        // row of q / out / the partials that tile row h stands for
    const int r = part * G + h, t = query_token(h);
    return (int64_t)(b * NQ + t) * p.n_q_heads + kv * GF + (r - t * GF);
  };

  char* const ring = smem + wave * (NS * C::STAGE);
  const uint32_t ring_lds =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + wave * (NS * C::STAGE);

  // ---- addressing: wave-uniform bases (scalar registers) + per-lane 32-bit byte offsets
  // tokens this sequence attends: the common length, or its own (a chunk past its end is empty); with a
  // sliding window the row simply starts `start` tokens later
  const bool var_lens = LISTED || (!PLAIN && p.seq_lens != nullptr);
  // a decode step (p.k_new set): the step's new token is not among the tokens the chunks cover; the block of the
  // sequence's first chunk takes it in (see `takes`).  A sequence may hold nothing but its new token.
  const bool new_here = !LEAN && p.k_new != nullptr && split == 0 && row_valid;
  const int new_pos = !var_lens ? p.append_pos : p.k_new == nullptr ? -1 : max(1, min(p.seq_lens[b], p.seq_len)) - 1;
  const int seq = !row_valid || (var_lens && new_pos == 0) ? 0 : !var_lens ? p.seq_len : planned_len >= 0 ? planned_len : var_len(p, b);
  const int start = LISTED ? 0 : !var_lens ? p.start : p.window > 0 ? var_start(p, b) : 0;
  // first row of the six arrays this block reads from: the sequence's own row (contiguous cache), or the
  // pool's row 0 (paged cache: the page's rows are added supertile by supertile)
  // paged cache: token indices below count from `start` as well, but the rows are found page by page; the
  // window's first token may lie up to 31 tokens after `start` (see var_start)
  const int lead = (paged && !LISTED && var_lens && p.window > 0) ? var_first(p, b) - start : 0;
  const int pstart = paged ? start : 0;           // added to a token index where a page is looked up
  const int64_t row0 = paged ? 0 : (int64_t)(b * p.n_kv_heads + kv) * p.row_stride + start;
  const int begin0 = split * tokens_per_split;    // first token of the chunk
  // A chunk past the end of its sequence has nothing to emit: the merge kernel works out from the same
  // lengths which chunks exist.  (With the in-kernel merge the block still has to be counted in, so it
  // goes through and publishes an empty partial.)
  if (!PLAIN && !LISTED && whole && begin0 >= seq && p.merge_slot < 0 && !new_here) return;
  const int end = max(begin0, min(seq, begin0 + (LISTED ? tokens_chunk : tokens_per_split)));
  // Several query tokens under a sliding window: the rows start at different tokens (row t one token after
  // row t - 1); the supertile that holds those starts takes the masked path too (wave 0, after its other work)
  // and the fast path starts behind it.  The same goes for a paged cache under a window, whose first supertile
  // holds `lead` tokens before the window.  With both, the rows start at tokens lead .. lead + NQ - 1, which may
  // straddle the sequence's first two supertiles: then the second is masked as well, in whichever chunk it lies.
  const bool rows_windowed = !PLAIN && NQ > 1 && p.row_window > 0;
  const bool straddle = rows_windowed && lead + NQ - 1 >= 32;
  const bool head = (rows_windowed || lead > 0) && end > begin0 && (begin0 == 0 || (begin0 == 32 && straddle));
  const bool head2 = head && begin0 == 0 && straddle && end > 32;
  const int begin = begin0 + (head2 ? 64 : head ? 32 : 0);   // origin of the supertile indices below
  // `seq` is what the last query token attends; query token t attends NQ - 1 - t tokens fewer.  Supertiles
  // that every row attends in full take the fast path; the sequence's last one or two (ragged, or holding
  // tokens some rows must not see) take the masked path.
  const int n_full = max(0, min(end, seq - (NQ - 1)) - begin) >> 5;
  const int n_tail = ((end - begin + 31) >> 5) - n_full;   // 0, 1 or 2 (NQ <= 8)
  const int last_tok = pstart + seq - 1;
  const int end_col = min(end, seq - (NQ - 1 - query_token(hl)));   // first token this lane's column must not see
  // ... and, under a window, the first one it sees: its own length less the window, relative to the row start
  const int lo_col = !head ? 0 : rows_windowed
                                     ? max(0, start + seq - (NQ - 1 - query_token(hl)) - p.row_window) - start : lead;
  const char* kc_row = reinterpret_cast<const char*>(p.k_codes) + row0 * TB;
  const char* vc_row = reinterpret_cast<const char*>(p.v_codes) + row0 * TB;
  const char* sz_row[4] = {reinterpret_cast<const char*>(p.k_scale) + row0 * SZB,
                           reinterpret_cast<const char*>(p.k_zero) + row0 * SZB,
                           reinterpret_cast<const char*>(p.v_scale) + row0 * SZB,
                           reinterpret_cast<const char*>(p.v_zero) + row0 * SZB};
  // Where a supertile starts: in a contiguous cache, `tok0` tokens into the sequence's own row; in a paged
  // one, in the page the block table names, at the token's offset inside the page (supertiles never
  // straddle pages: a page is a multiple of 32 tokens and paged sequences start at token 0).
  struct Bases { const char* k; const char* v; const char* s[4]; };
  const Bases row_bases = {kc_row, vc_row, {sz_row[0], sz_row[1], sz_row[2], sz_row[3]}};
  const int32_t* const tbl = paged ? p.block_table + (int64_t)b * p.max_blocks : nullptr;
  const int page_mask = (1 << p.page_shift) - 1;
  // The page numbers of the chunk's first 64 pages sit in a register, one per lane, fetched before anything else (a
  // table entry looked up in the loop would stall a supertile); entries past those are fetched by a scalar load
  // that is waited for on the spot.  (32 heads over 32, one sequence of 32K tokens, 4096 to a chunk: 35.3 us per step in
  // pages of 64, 36.5 in pages of 32; 4 of 16K 61.5.  The next 64 fetched by the loop itself: 35.8 and 61.6, but
  // the registers for it cost the calls whose chunks have fewer pages more: 64 sequences of 128 .. 4096 tokens, 64 heads
  // over 8, 33.8 -> 36.9, one of 128K 37.2 -> 38.8.)
  const int page0 = paged ? (pstart + begin0) >> p.page_shift : 0;
  const int page_v = paged ? tbl[min(page0 + lane, p.max_blocks - 1)] : 0;
  auto page_of = [&](int tok0) {
    const int e = min(tok0 >> p.page_shift, p.max_blocks - 1);
    if ((uint32_t)(e - page0) < 64u) return __builtin_amdgcn_readlane(page_v, e - page0);
    int page;
    const uint32_t byte = (uint32_t)e * 4;
    asm volatile("s_load_dword %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&s"(page) : "s"(tbl), "s"(byte) : "memory");
    return page;
  };
  auto bases_of_page = [&](int page) -> Bases {   // row 0 of `page` for this KV head (a page is 2^page_shift rows)
    const int64_t r = (int64_t)(page * p.n_kv_heads + kv) << p.page_shift;
    const int64_t rc = r * TB, rs = r * SZB;
    return {row_bases.k + rc, row_bases.v + rc, {row_bases.s[0] + rs, row_bases.s[1] + rs, row_bases.s[2] + rs,
                                                 row_bases.s[3] + rs}};
  };
  const uint32_t koff = tok_of_row(c) * TB + kq * (D / 8);   // this lane's 16 B (x D/128) of a K tile
  // scale / zero-point arrays: destination dword u*64+lane of the stage comes from (token, dword) of the supertile
  uint32_t sz_tok[C::SZ / 256], sz_col[C::SZ / 256];
#pragma unroll
  for (int u = 0; u < C::SZ / 256; ++u) {
    sz_tok[u] = C::sz_token(u * 64 + lane);
    sz_col[u] = C::sz_column(u * 64 + lane);
  }

  // Fills the ring slot at LDS address l with the supertile whose codes start off_c bytes into the row:
  // LPS load instructions, all 64 lanes each.  vk, vv, vs are the per-lane byte offsets inside the
  // supertile (K tile, V block, scale array).
  const uint32_t lane16 = lane * 16;
  uint32_t szoff[C::SZ / 256];
#pragma unroll
  for (int u = 0; u < C::SZ / 256; ++u)           // (larger groups: the token's only dword, or the dword it shares)
    szoff[u] = GS == 0 || D == 256 ? (sz_tok[u] * (NGM / 2) + sz_col[u]) * 4 : GS == 1 ? sz_tok[u] * 4 : (sz_tok[u] >> 1) * 4;
  auto issue_at = [&](uint32_t l, const Bases& B, uint32_t off_c, uint32_t vk, uint32_t vv,
                      const uint32_t (&vs)[C::SZ / 256]) {
    const uint32_t off_s = off_c >> (3 + GS);     // SZB / TB: metadata bytes per code byte
    // the supertile's offset goes into the (scalar) base, not into the per-lane offsets: scalar adds are free
    // next to a vector ALU that is the kernel's bottleneck
    const char* const bk = B.k + off_c;
    const char* const bv = B.v + off_c;
    if constexpr (D == 128) {
      dma16_x2<NT, 1024>(bk, vk, l);                                   // two K tiles: 1 KB apart on both sides
      dma16_x2<NT, 1024>(bv, vv, l + C::OFF_V);
    } else {
      dma16_x2<NT, 2048>(bk, vk, l);                                   // first 16 B of each lane, tiles 0 and 1
      dma16_x2o<NT, 16, 2064>(bk, vk, l + 1024 - 16);                  // second 16 B: +16 in HBM, +1024 in LDS
      dma16_x4<NT>(bv, vv, l + C::OFF_V);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int u = 0; u < C::SZ / 256; ++u) dma4<NT>(B.s[a] + off_s, vs[u], l + C::OFF_KS + a * C::SZ + u * 256);
  };
  // supertile starting tok0 tokens into the sequence (page known in the paged case) -> ring slot at l
  auto issue_tok = [&](uint32_t l, int tok0, int page, uint32_t vk, uint32_t vv, const uint32_t (&vs)[C::SZ / 256]) {
    if (paged) issue_at(l, bases_of_page(page), (uint32_t)(tok0 & page_mask) * TB, vk, vv, vs);
    else issue_at(l, row_bases, (uint32_t)tok0 * TB, vk, vv, vs);
  };
  auto issue_tail = [&](int slot, int sidx) {     // ragged last supertile: clamp every token to the last valid one
    const int base = pstart + begin + sidx * 32;
    const uint32_t l = ring_lds + slot * C::STAGE;
    // token index -> row of the arrays below: the sequence's row, or the page that holds this supertile
    const Bases B = paged ? bases_of_page(page_of(base)) : row_bases;
    const int row_first = paged ? (base & ~page_mask) : 0;
    const char* const kc_row = B.k - (int64_t)row_first * TB;
    const char* const vc_row = B.v - (int64_t)row_first * TB;
    const char* const sz_row[4] = {B.s[0] - (int64_t)row_first * SZB, B.s[1] - (int64_t)row_first * SZB,
                                   B.s[2] - (int64_t)row_first * SZB, B.s[3] - (int64_t)row_first * SZB};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int tok = min(base + 16 * t + tok_of_row(c), last_tok);
#pragma unroll
      for (int ch = 0; ch < D / 128; ++ch)
        dma16_lane(kc_row + (int64_t)tok * TB + kq * (D / 8) + ch * 16, l + t * C::KT + ch * 1024);
    }
#pragma unroll
    for (int u = 0; u < C::VB / 1024; ++u) {
      const int chunk = u * 64 + lane;            // 16-byte chunk of the supertile's V codes
      const int tok = min(base + chunk / (TB / 16), last_tok);
      dma16_lane(vc_row + (int64_t)tok * TB + (chunk % (TB / 16)) * 16, l + C::OFF_V + u * 1024);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int u = 0; u < C::SZ / 256; ++u) {
        const int tok = min(base + (int)sz_tok[u], last_tok);
        const int64_t src = GS == 0 || D == 256 ? (int64_t)tok * (NGM * 2) + sz_col[u] * 4 : GS == 1 ? (int64_t)tok * 4 : (int64_t)(tok >> 1) * 4;
        dma4_lane(sz_row[a] + src, l + C::OFF_KS + a * C::SZ + u * 256);
      }
  };
  auto tok_of = [&](int sidx) { return pstart + begin + sidx * 32; };
  auto issue = [&](int slot, int sidx) {
    const int tok0 = tok_of(sidx);
    issue_tok(ring_lds + slot * C::STAGE, tok0, paged ? page_of(tok0) : 0, koff, lane16, szoff);
  };
  // ---- work distribution.  The block's 8 waves sit two to a SIMD (waves w and w+4), and the SIMD
  //      issues from its older wave first, so wave w gets through a supertile in less time than wave w+4
  //      (about 7/9 of it in the heavier instances, 10/11 in the leanest).  The chunk's supertiles are
  //      therefore dealt round-robin to the four SIMDs, and of every PERIOD that a SIMD gets, its older wave
  //      takes PERIOD/2 + 1 and the younger PERIOD/2 - 1, in a fixed pattern.
  //      The split is static: the summation order, and with it every output bit, is the same on every
  //      launch.  The ragged last supertile, if any, goes to the wave whose turn it would be and takes
  //      the clamped path.
  static_assert(NW == 8, "the work split assumes two waves per SIMD");
  const int simd = wave & 3, young = wave >> 2;
  constexpr int PERIOD = C::PER, OLD = PERIOD / 2 + 1, YNG = PERIOD / 2 - 1;   // of every PER supertiles of a SIMD: older wave, younger wave
  auto sidx_of = [&](int i) {                     // i-th supertile of this wave -> supertile of the chunk
    if (!whole) return W * i + sub;
    const int blk = young ? i / YNG : i / OLD, j = i - blk * (young ? YNG : OLD);
    const int k = PERIOD * blk + (young ? 2 * j + 1 : (j < PERIOD / 2 ? 2 * j : PERIOD - 1));
    return 4 * k + simd;
  };
  auto count_of = [&](int n) {                    // how many of the chunk's first n supertiles are this wave's
    if (!whole) return n > sub ? (n - sub + W - 1) / W : 0;
    const int K = n > simd ? (n - simd + 3) >> 2 : 0, r = K % PERIOD;
    return young ? YNG * (K / PERIOD) + (r >> 1) : OLD * (K / PERIOD) + ((r + 1) >> 1);
  };
  const int n_mine = count_of(n_full);
  // ---- prologue: the query rows of this KV head's group come in by direct load as well (so that every
  //      vector-memory operation of the kernel is one of the counted loads), then the ring is filled.
  //      Where the query block has to borrow the last ring slot, that slot is filled once the query
  //      operands sit in registers.
  // One stage is issued before the query operands are built.  The second follows once those operands sit in
  // registers (d = 256) or, at d = 128, only when the first has landed and its K part has been read: with every
  // wave's first stage requested alone, the first stages arrive within a short span of each other instead of
  // queueing behind other waves' second stages, and the waves start (and end) closer together (0.1 - 0.3 us of
  // the 128K launch; at d = 256 the later point costs 0.3 us).
  constexpr int NPRE = NS - 1;
  const bool kSecondAfterFirstLanded = D == 128 && whole;   // (rows packed several to a block: 256 x 512 tokens 39.2 -> 40.0 us with it)
  // (a borrowed slot: behind its K tiles where the block fits there, else from the slot's start)
  constexpr int Q_IN_SLOT = C::QAREA <= C::STAGE - C::OFF_V ? C::OFF_V : 0;
  // (a block of fewer waves, see `ranked`: the areas behind the rings move up)
  const int off_merge = C::ALIAS ? 0 : n_waves * NS * C::STAGE;
  const int off_qblk = off_merge + (n_waves * GP * D + 2 * NW * GP + n_units * C::NEWTOK) * 4;
  char* const q_area = C::QSEP ? smem + off_qblk + wave * C::QAREA : ring + (NS - 1) * C::STAGE + Q_IN_SLOT;
  // A decode step's new token (one query token; its K and V rows in p.k_new / p.v_new): one wave of the block that
  // holds its sequence's first chunk quantises it while the first stage of the stream is on its way, stores it, works
  // out its scores against the block's query rows, and brings it to the block merge as one more wave would: m = the
  // score, l = 1, o = the dequantised V.  The step needs no launch of its own for the append, and a merge kernel only
  // where the decode does.  (Steps with the merge kernel as the appender, or the append kernel in front of packed
  // rows, and like this: one sequence of 1024 tokens, 8 heads on 1, 12.5 -> 11.3 us per call; a window of 1024, d = 256,
  // 13.1 -> 10.9; 32K tokens, d = 256, 35.3 -> 33.9; 128 sequences of 512 .. 1024 tokens 35.3 -> 32.6.)
  // What the token costs is the chain of instructions of the wave that takes it: the block waits for that wave.  So its K
  // and its V go to two waves (or the two halves of one, see `one_takes`), of the older ones of their SIMDs, which are
  // 0.6 us ahead of the younger at this point, and a wave's lanes hold the row several times over, eight elements a lane, so
  // that the copies of K share the query rows' scores between them.  (One younger wave for all of it, half of its lanes idle:
  // that wave 2.0 us behind the others; us per step 8 heads over 1, 1024 tokens 8.62 -> 7.94, 64 over 8, 8K 10.77 -> 10.02,
  // 32 over 16, d = 256, a window of 1024 9.31 -> 8.78; the decode alone 7.83, 10.01, 8.80.)
  // (A chunk of few supertiles leaves the younger waves idle: then they.)
  // The choice stands in front of the first loads, like all up to here, and every instruction delays them: nothing that can wait
  // (which waves are idle, whose the last supertile is) is worked out here.  (50 - 80 more: us per decode 32 heads over 32, 8 sequences of 200
  // tokens 5.3 -> 5.7, 64 over 8, groups of 64, 200 7.35 -> 7.6.)
  const int taker = PLAIN && n_full + n_tail <= NW / 2 ? NW - 1 : NW / 2 - 1;
  // One wave takes both where a row has no other, and at d = 256 wherever a block holds several rows: all its waves have work of their own
  // then, so what counts is the sum of the instructions, and two waves quantise in twice as many as one does both rows in, for the scores
  // of only two query rows.  (us per step, two waves / one, 16 heads over 8: 79 sequences of 146 .. 214 tokens in pages 17.71 / 17.09,
  // contiguous 17.07 / 16.38, 64 of 600 21.67 / 21.38; 32 over 16, 79 of 146 .. 900 in pages 40.0 / 39.4.  At d = 128 it is the other way
  // round or even, 64 over 8: 64 of 64 .. 2000 22.53 / 22.79, 96 of 64 .. 1500 25.4 / 25.3.)
  const bool one_takes = !PLAIN && (D == 256 ? !whole : W == 1);
  const int new_part = whole ? taker - wave : sub;             // 0: K, 1: V
  const bool takes = new_here && (uint32_t)new_part < (one_takes ? 1u : 2u);
  const bool takes_k = takes && new_part == 0, takes_v = takes && (one_takes || new_part == 1);
  constexpr int PIECES = D / 8, COPIES = 64 / PIECES;
  const int new_piece = lane % PIECES, new_v = one_takes ? lane >> 5 : new_part;
  const uint32_t q_lds = C::QSEP ? (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + off_qblk + wave * C::QAREA
                                 : ring_lds + (NS - 1) * C::STAGE + Q_IN_SLOT;
#pragma unroll
  for (int u = 0; u < GP * D * 2 / 1024; ++u) {
    const int chunk = u * 64 + lane;              // 16-byte chunk of the [GP][D] fp16 query block
    const int h = min(chunk / (D / 8), G - 1);
    dma16_lane(p.q + query_row(h) * D + (chunk % (D / 8)) * 8, q_lds + u * 1024);
  }
  if (takes)                                      // the new token's K row, or its V row (one wave for both: half the lanes each)
    dma16_lane((new_v ? p.v_new : p.k_new) + (int64_t)(b * p.n_kv_heads + kv) * D + new_piece * 8, q_lds + C::QBLK);
  // A wave has up to NS stages out before its loop and issues one per supertile while it has supertiles left.
  // (Stand-in loads that kept the count of outstanding loads the same to the end were taken out: the one issued in
  // a wave's last iteration made it wait a whole memory round trip for bytes nobody reads, 0.3 us per launch at
  // llama128k and 0.8 us at gemma32k; the waits below count what is really out instead.)
  // A wave whose share includes the ragged (or partly masked) last supertile takes that one FIRST: its loads then leave
  // with the prologue's and its masked path runs while the wave's first full supertile is on its way.  (At the end it
  // was a memory round trip of its own for one wave of the launch, 2 - 3 us of a short sequence's time.)
  const bool tail_last = n_tail > 0 && count_of(n_full + 1) != count_of(n_full);
  const bool tail0 = !LEAN && tail_last;
  if (tail0) issue_tail(0, n_full);
  else if (n_mine > 0) issue(0, sidx_of(0));
  // (the first loads are on their way: whatever they do not need is worked out behind them)
  __builtin_amdgcn_sched_barrier(0);
  // A short chunk has no supertile for every wave: its first ones are its first waves', one each, and the others only keep
  // the barriers company (and take their rows of the merges).
  const bool busy = (!PLAIN && !LISTED) || n_mine > 0 || tail_last;
  bool tail_mine[4];                              // [2], [3]: the masked FIRST supertile(s) (see `head`), the one just
                                                  // before `begin` and the one before that
  tail_mine[0] = tail_last;
  tail_mine[1] = n_tail > 1 && count_of(n_full + 2) != count_of(n_full + 1);
  tail_mine[2] = head && (whole ? wave == 0 : sub == 0);
  tail_mine[3] = head2 && (whole ? wave == 0 : sub == 0);
  static_assert(NPRE == 1, "one stage follows the query block");
  if (tail0 || n_mine > 0) wait_loads<LPS>();                // (the stage issued after the query block may still be out)
  else wait_loads<0>();

  // ---- query operands (the query pre-scaling of Alg. 1 is folded into the exp2 argument instead of the query)
  half8v qb[NJ];
  float qsum[NA];                                 // 2^-24 * sum of the operand's q over each of this lane's groups
  float q_up = 1.0f;
  if (busy) {
    const _Float16* qh = reinterpret_cast<const _Float16*>(q_area) + hl * D;
    half8v qraw[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      qraw[j] = *reinterpret_cast<const half8v*>(qh + C::a_group(j, kq) * kGroup + C::a_word(j, kq) * 8);
    half8v qgrp[NA][4];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int i = 0; i < 4; ++i) qgrp[a][i] = *reinterpret_cast<const half8v*>(qh + (rep * NA + a) * kGroup + i * 8);

    // (SPLIT) Half of the operand's elements are q over 16 (below), and those of a small query would lose bits in fp16's
    // subnormals, which the fp32 queries of the generic kernel do not.  So a row with no element of 2 or more is taken 16
    // times (every fp16 is a whole number of 2^-24: q and 16 q are exact), and in the others what is lost lies 2^-22
    // below the row's largest element.  (A power of two that brings the largest element near 2^14 costs a short step 0.9 us.)
    if constexpr (SPLIT) {
      uint32_t any = 0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint4v w = __builtin_bit_cast(uint4v, qraw[j]);
        any |= (w[0] | w[1]) | (w[2] | w[3]);
      }
      // (bit 14 of an fp16: 2 or more; a row's elements are spread over the four 16-lane rows)
      q_up = blocks_max((any & 0x40004000u) != 0 ? 1.0f : 0.0f) > 0.0f ? 1.0f : 16.0f;
    }
    const _Float16 q_lo = (_Float16)q_up, q_hi = (_Float16)(q_up * 0.0625f);

#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const bool mine = (C::a_group(j, kq) == rep * NA + C::acc(j)) && hl < G;
      const half8v x = qraw[j];
      // k-slot order of unpack_word: nibbles 0,4,1,5,2,6,3,7; the "hi" slots carry c*2^-20, so pre-divide by 16
      half8v y = {x[0], x[4], x[1] * (_Float16)0.0625f, x[5] * (_Float16)0.0625f,
                  x[2], x[6], x[3] * (_Float16)0.0625f, x[7] * (_Float16)0.0625f};
      if constexpr (SPLIT)
        y = half8v{x[0] * q_lo, x[4] * q_lo, x[1] * q_hi, x[5] * q_hi, x[2] * q_lo, x[6] * q_lo, x[3] * q_hi, x[7] * q_hi};
      if (!mine) y = half8v{0, 0, 0, 0, 0, 0, 0, 0};
      qb[j] = y;
    }
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      float s = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (float)qgrp[a][i][e];
      qsum[a] = (hl < G) ? s * (SPLIT ? 0x1p-24f * q_up : 0x1p-24f) : 0.0f;
    }
  }

  uint32_t new_w = 0;                             // the new token: this lane's packed word, its group's scale and
  half2v new_sz = {0, 0};                         // zero-point, and (lane h of the first 16) its score against row h
  float new_score = 0.0f;
  if (takes) {
    const half8v x16 = *reinterpret_cast<const half8v*>(q_area + C::QBLK + lane * 16);
    half_t xh[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) xh[e] = x16[e];
    // the group's smallest and largest element: (min, -max) as a pair of fp16, exact in any order
    const auto pk_min = [](half2v a, half2v b) { return __builtin_elementwise_min(a, b); };
    const half2v x01 = {xh[0], xh[1]}, x23 = {xh[2], xh[3]}, x45 = {xh[4], xh[5]}, x67 = {xh[6], xh[7]};
    const half2v lo = pk_min(pk_min(x01, x23), pk_min(x45, x67)), hi = pk_min(pk_min(-x01, -x23), pk_min(-x45, -x67));
    half2v range = pk_min(half2v{lo[0], hi[0]}, half2v{lo[1], hi[1]});
    auto over_lanes = [&](auto ctrl_tag) {
      const int other = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, range), decltype(ctrl_tag)::value, 0xF, 0xF, false);
      range = pk_min(range, __builtin_bit_cast(half2v, other));
    };
    over_lanes(std::integral_constant<int, 0xB1>{});                       // quad_perm: the lanes 1, then 2, away
    over_lanes(std::integral_constant<int, 0x4E>{});
    if constexpr (GS >= 1) over_lanes(std::integral_constant<int, 0x141>{});   // row_half_mirror: the other four of eight
    if constexpr (GS >= 2) over_lanes(std::integral_constant<int, 0x140>{});   // row_mirror: the other eight of sixteen
    const float mn = (float)range[0], mx = -(float)range[1];
    half_t s16, z16;
    quantize_scale_zero(mn, mx, s16, z16);
    const float sf = (float)s16, zf = (float)z16;
    const QuantFast fast = quantize_fast_setup(sf, zf, fmaxf(fabsf(mn), fabsf(mx)));
    float far = 0.0f;
    new_w = quantize_word_fast(xh, fast, far);
    if (quantize_fast_in_doubt(far, fast)) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = (float)xh[e];
      new_w = quantize_word(x, sf, zf);
    }
    new_sz = half2v{s16, z16};
    if (takes_k) {
      const int copies = takes_v ? COPIES / 2 : COPIES, copy = lane / PIECES;
      float k_hat[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) k_hat[e] = ((float)((new_w >> (4 * e)) & 0xFu) - zf) * sf;   // Eq. 3
      for (int i = 0, h = copy; i * copies < GP; ++i, h += copies) {       // copy k: rows k, k + copies, ...
        const half8v qv = *reinterpret_cast<const half8v*>(q_area + min(h, GP - 1) * D * 2 + new_piece * 16);
        float dot = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) dot = __builtin_fmaf((float)qv[e], k_hat[e], dot);
        dot = row_ror_add<8>(dot);
        dot = row_ror_add<4>(dot);
        dot = row_ror_add<2>(dot);
        dot = row_ror_add<1>(dot);
        if constexpr (D == 256) {
          float a, b2;
          swap16(dot, a, b2);
          dot = a + b2;
        }
        new_score = new_piece == i ? dot : new_score;
      }
    }
    if (part == 0 && (takes_k && takes_v ? (lane & 31) < PIECES : lane < PIECES)) {   // (several blocks per KV head: the first stores)
      int64_t row = (int64_t)(b * p.n_kv_heads + kv) * p.row_stride + new_pos;
      if (paged) {
        const int page = p.block_table[(int64_t)b * p.max_blocks + (new_pos >> p.page_shift)];
        row = ((int64_t)page * p.n_kv_heads + kv) * p.row_stride + (new_pos & page_mask);
      }
      uint8_t* codes = const_cast<uint8_t*>(new_v ? p.v_codes : p.k_codes) + row * TB;
      reinterpret_cast<uint32_t*>(codes)[new_piece] = new_w;
      constexpr int GROUP = kGroup << GS;
      const int64_t g = row * (D / GROUP) + new_piece * 8 / GROUP;
      const int first = new_piece * 8 % GROUP;    // (the group's first two lanes store its scale and zero-point)
      if (first == 0) const_cast<half_t*>(new_v ? p.v_scale : p.k_scale)[g] = s16;
      if (first == 8) const_cast<half_t*>(new_v ? p.v_zero : p.k_zero)[g] = z16;
    }
  }
  const float kappa = p.scale_log2 * 0x1p24f * (SPLIT ? 1.0f / q_up : 1.0f);   // raw accumulator units -> log2 units
  const float slack = kSlack / kappa;             // the rescale slack in raw units
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the query block has been read: its slot may be refilled
  if (tail0) {
    if (n_mine > 0) issue(1, sidx_of(0));
  } else if (!kSecondAfterFirstLanded && n_mine > 1) issue(1, sidx_of(1));
  // supertile NS, the first one issued inside the loop, and how to step from one supertile to the next:
  // position j in the wave's pattern of 9 (or 7) out of 16
  int nx_j = young ? NS % YNG : NS % OLD;
  int nx_tok = tok_of(sidx_of(NS));

  // ---- running state
  float m_run = kNegBig;                          // per-head reference for exp2 (raw units)
  float l_run = 0.0f;                             // this lane's share of sum(exp)
  float4v zacc[NA];                               // sum_t w z - 15 sum_t1 w (w = p s_v), rows (head, replica), col = group
  // rows (head, replica), col = packed word; [2j]: sum_t w c - 15 sum_t1 w for dim 2j of the word, [2j+1]: the same
  // for c(2j) + 16 c(2j+1), less 255 sum_t1 w.  WIDE: [2g], [2g+1] are the even and the mixed sum of group g, whose
  // column c stands for byte c / 4 of the group's word c % 4; one accumulator each.
  constexpr int NAO = C::WIDE ? 1 : NA;
  static_assert(!SPLIT || NA == 1, "one group per lane");
  constexpr int NPA = SPLIT ? 2 : MAY_TWO ? 2 * NA : NA;   // A operands of P V: one per group of the lane, or the two parts of one, of each
  float4v oacc[NCS][8][NAO];
#pragma unroll
  for (int a = 0; a < NA; ++a) zacc[a] = float4v{0, 0, 0, 0};
#pragma unroll
  for (int cs = 0; cs < NCS; ++cs)
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int a = 0; a < NAO; ++a) oacc[cs][m][a] = float4v{0, 0, 0, 0};

  const half8v pos15_odd = as_half8(kPos15Odd, kPos15Odd, kPos15Odd, kPos15Odd);

  // per-lane LDS byte offsets inside a stage
  // K codes: the 16 B this lane asked for; where the query operand is block-diagonal over pairs of
  // groups (SWAP), words w and w+2 of groups 2(kq/2) and 2(kq/2)+1 of token row c instead
  // (WIDE: word kq of every group of token row c, one dword each, 256 B apart)
  const uint32_t k_rd = C::WIDE ? c * 16 + 4 * kq : C::SWAP ? (32 * (kq >> 1) + c) * 16 + 4 * (kq & 1) : lane * 16;
  // packed word(s) c of token kq (+4i); WIDE: word c % 4 of every group, 16 B apart
  const uint32_t v_rd = C::WIDE ? kq * TB + (c & 3) * 4 : kq * TB + c * 4 * NCS;
  const uint32_t v_sel = 0x0C000C00u | ((4u + (c >> 2)) << 16) | (uint32_t)(c >> 2);   // WIDE: this column's byte of a word
  // scales of this lane's groups / zero-point of the group this lane's P V column (packed word c) lies in,
  // tokens kq (+4i): eight consecutive dwords in the permuted layout, else one halfword per token at the
  // array's own stride
  // (WIDE: the zero-point operand's column c stands for group c % 4)
  const int gz = C::WIDE ? (c & 3) : (c * NCS) >> 2;
  const uint32_t sz_rd = C::WIDE ? kq * 64 : C::PERM ? (kq * GR + rep) * 32 : (kq * NGM + ((rep * NA) >> GS)) * 2;
  const uint32_t zb_rd = C::WIDE ? kq * 64 + (gz >> 1) * 32 : C::PERM ? (kq * GR + (gz >> 1)) * 32 : (kq * NGM + (gz >> GS)) * 2;
  // which half of a zero-point dword: the group's place in its pair; with larger groups the pair's place among the
  // token's two groups, or the token's place in its pair of tokens (this lane's tokens are kq, kq + 4, ...)
  const bool zb_hi = GS == 0 ? (gz & 1) : GS == 1 ? ((gz >> 1) & 1) : (kq & 1);
  const uint32_t zb_sel = zb_hi ? 0x07060302u : 0x05040100u;
  // larger groups: the half of a fetched scale / zero-point dword that this lane's 32-dim blocks share.  With 8 rows
  // the lane's two blocks are 2 rep and 2 rep + 1 (group rep of the token's two); with 16 rows register dw holds
  // blocks 2 dw and 2 dw + 1 (group dw); with groups of 128 it is the token's parity either way.
  const uint32_t dup_lo = 0x01000100u, dup_hi = 0x03020302u;
  const uint32_t dup_lane = (GS == 2 ? (kq & 1) : rep) ? dup_hi : dup_lo;

  // Everything a supertile needs from LDS is fetched into registers well before it is used: the K part
  // while the previous supertile is still in its P V phase, the V part at the start of the K phase.
  constexpr int NDW = C::NDW, NVW = C::WIDE ? NG : NCS;
  struct KRegs { uint32_t kw[2][NJ]; uint32_t ks[NDW][2][4], kz[NDW][2][4]; };   // kw[t][j]: A operand of K MFMA j, tile t
  struct VRegs { uint32_t v[NVW][8]; uint32_t vs[NDW][2][4]; uint32_t zb[8]; };
  auto load_sz1 = [&](const char* arr, uint32_t rd, uint32_t (&dst)[2][4]) {
    if constexpr (C::PERM || C::WIDE) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint4v x = *reinterpret_cast<const uint4v*>(arr + rd + t * 16);
        dst[t][0] = x[0]; dst[t][1] = x[1]; dst[t][2] = x[2]; dst[t][3] = x[3];
      }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          dst[t][i] = *reinterpret_cast<const uint16_t*>(arr + (t * 16 + i * 4) * NGM * 2 + rd);
    }
  };
  auto load_sz = [&](const char* arr, uint32_t rd, uint32_t (&dst)[NDW][2][4]) {
#pragma unroll
    for (int dw = 0; dw < NDW; ++dw) {
      load_sz1(arr + dw * 32, rd, dst[dw]);
      if constexpr (GS > 0 && D == 128) {
        const uint32_t sel = (GS == 1 && C::WIDE) ? (dw ? dup_hi : dup_lo) : dup_lane;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) dst[dw][t][i] = __builtin_amdgcn_perm(dst[dw][t][i], dst[dw][t][i], sel);
      }
    }
  };
  auto load_k = [&](int slot, KRegs& r) {
    const char* st = ring + slot * C::STAGE;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if constexpr (C::WIDE) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) r.kw[t][j] = *reinterpret_cast<const uint32_t*>(st + t * C::KT + j * 256 + k_rd);
      } else if constexpr (C::SWAP) {
        // the lane wants words w, w+2 of two neighbouring groups, 256 B apart in the tile: two 2-dword reads
        const uint32_t* g0 = reinterpret_cast<const uint32_t*>(st + t * C::KT + k_rd);
        r.kw[t][0] = g0[0]; r.kw[t][2] = g0[2]; r.kw[t][1] = g0[64]; r.kw[t][3] = g0[66];
      } else {
#pragma unroll
        for (int ch = 0; ch < D / 128; ++ch) {
          const uint4v x = *reinterpret_cast<const uint4v*>(st + t * C::KT + ch * 1024 + k_rd);
          r.kw[t][ch * 4 + 0] = x[0]; r.kw[t][ch * 4 + 1] = x[1]; r.kw[t][ch * 4 + 2] = x[2]; r.kw[t][ch * 4 + 3] = x[3];
        }
      }
    }
    load_sz(st + C::OFF_KS, sz_rd, r.ks);
    load_sz(st + C::OFF_KZ, sz_rd, r.kz);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_v = [&](int slot, VRegs& r) {
    const char* st = ring + slot * C::STAGE;
#pragma unroll
    for (int cs = 0; cs < NVW; ++cs)
#pragma unroll
      for (int i = 0; i < 8; ++i)                 // token slot i: token 16*(i/4) + 4*(i%4) + kq
        r.v[cs][i] = *reinterpret_cast<const uint32_t*>(st + C::OFF_V + (16 * (i >> 2) + 4 * (i & 3)) * TB + v_rd +
                                                        cs * (C::WIDE ? 16 : 4));
    load_sz(st + C::OFF_VS, sz_rd, r.vs);
    uint32_t zr[2][4];
    load_sz1(st + C::OFF_VZ, zb_rd, zr);
#pragma unroll
    for (int i = 0; i < 8; ++i) r.zb[i] = zr[i >> 2][i & 3];
    __builtin_amdgcn_sched_barrier(0);
  };
  // fp16 scale / zero-point number a (of this lane's NA) out of a fetched register
  auto sz_half = [&](uint32_t w, int a) -> _Float16 {
    const uint16_t h = (uint16_t)(a == 0 ? w : w >> 16);
    return __builtin_bit_cast(_Float16, h);
  };

  // -- scores, S^T = K Q^T, per-group scale and zero-point applied in fp32 (raw units: 2^-24)
  auto scores = [&](const KRegs& r, int sidx, auto tail_tag, float (&sc)[2][4]) {
    constexpr bool TAIL = decltype(tail_tag)::value;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float4v acc[NA];
#pragma unroll
      for (int a = 0; a < NA; ++a) acc[a] = float4v{0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[C::acc(j)] = mfma16(unpack_word(r.kw[t][j]), qb[j], acc[C::acc(j)]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {               // token 16t + 4i + kq
        float x = 0.0f;
#pragma unroll
        for (int a = 0; a < NA; ++a)
          x = __builtin_fmaf((float)sz_half(r.ks[a >> 1][t][i], a & 1),
                             __builtin_fmaf(-(float)sz_half(r.kz[a >> 1][t][i], a & 1), qsum[a], acc[a][i]), x);
        if constexpr (GR >= 2) x = row_ror_add<8>(x);
        if constexpr (GR >= 4) x = row_ror_add<4>(x);
        if constexpr (GR >= 8) x = row_ror_add<2>(x);
        if constexpr (TAIL) {
          const int tok = begin + sidx * 32 + 16 * t + tok_of_row(4 * kq + i);
          x = (tok >= lo_col && tok < end_col) ? x : -INFINITY;
        }
        sc[t][i] = x;
      }
    }
  };

  // -- online softmax over the 32 tokens (Alg. 1: the maximum, the weights and the running sum), block-wise.  m_run is a per-head
  //    REFERENCE, not the exact running max: it only moves when some score exceeds it by more than
  //    kSlack (log2 units), so exp2(score - m_run) <= 2^kSlack = 4 and p * s_v stays inside fp16 for
  //    every representable scale, while the accumulator rescale (Alg. 1, the correction factor) becomes rare.
  //    When it moves it is set kSlack ABOVE the new maximum, so the next move needs a score 2*kSlack
  //    higher than any seen so far; the weights then start at 2^-kSlack, far inside fp16's normal range.
  //    Any reference gives the same o / l, and the chunk merge (Eq. 6) accepts any m_c.
  //    Then A = fp16(+-p * s_v) (minus on the second tile's k-slots), rows (head, replica), one operand
  //    per group of the lane; the zero-point term goes through the matrix core with the stored fp16
  //    zero-points (sign flipped on the second tile's k-slots) as B operand.
  //    SPLIT: the weights are 2^off p s_v with a wave-wide off, lowered when a larger scale turns up, that keeps
  //    them below 2^12; off is part of the reference the partial is published with.  A = leading fp16 part, then
  //    the rest (both rounded towards zero: what the first leaves out the second takes).
  //    SPLIT also turns the sign of everything half way through the wave's supertiles: the matrix core's truncation
  //    pulls an accumulator the same way at every step, and what it takes from the first half it gives back in the
  //    second (32K tokens, flat softmax: 1.4 % of the output's error against 64 bits, most of it fp16 rounding).
  //    Odd waves start with the other sign, for those that have a supertile or two.
  uint32_t sv_top = 0;                            // (SPLIT) bits of the power of two no scale so far reaches
  const float sgn0 = SPLIT && (wave & 1) ? -1.0f : 1.0f;
  float off = 0.0f, sgn = sgn0;
  auto negate_sums = [&] {
    sgn = -sgn;
#pragma unroll
    for (int a = 0; a < NA; ++a) zacc[a] = -zacc[a];
#pragma unroll
    for (int cs = 0; cs < NCS; ++cs)
#pragma unroll
      for (int m = 0; m < 8; ++m)
#pragma unroll
        for (int a = 0; a < NAO; ++a) oacc[cs][m][a] = -oacc[cs][m][a];
  };
  auto softmax = [&](const float (&sc)[2][4], const VRegs& r, half8v (&pa)[NPA], auto two_tag) {
    constexpr bool TWO = decltype(two_tag)::value;
    const float mx = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                           fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
    bool move = mx > m_run + slack;
    uint32_t sv = 0;                              // (SPLIT) the largest of this lane's scales by size (positive fp16: ordered as integers)
    if constexpr (SPLIT) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) sv = max(sv, r.vs[0][t][i] & 0x7FFFu);
      move = move || sv >= sv_top;
    }
    if (__builtin_amdgcn_ballot_w64(move) != 0) {   // wave-uniform, rare
      // Every head's reference becomes at least its own current maximum plus kSlack (for the heads that outgrew
      // theirs the next move is then 2*kSlack away; the others get their headroom back while the rescale is being
      // paid for anyway).  A reference is thus never more than kSlack above its head's running maximum: one that
      // followed every move of a neighbour instead would creep up and push the head's own weights p * s_v down
      // into fp16's subnormals on a sharp softmax.
      const float m_new = fmaxf(m_run, blocks_max(mx) + slack);
      float df = (m_run - m_new) * kappa;
      if constexpr (SPLIT) {
        if (__builtin_amdgcn_ballot_w64(sv >= sv_top) != 0) {
#pragma unroll
          for (int o = 32; o >= 1; o >>= 1) sv = max(sv, (uint32_t)__shfl_xor((int)sv, o));
          const int e = __builtin_amdgcn_readfirstlane((int)(sv >> 10));   // biased exponent: every scale so far < 2^(e - 14)
          sv_top = (uint32_t)(e + 1) << 10;
          const float off_new = (float)(24 - e);                           // p <= 4: weights below 2^12
          df += off_new - off;
          off = off_new;
        }
      }
      const float f = __builtin_amdgcn_exp2f(df);
      m_run = m_new;
      l_run *= f;
      float fr[4];                                           // accumulator row 4kq+i belongs to head (4kq+i) % GP
#pragma unroll
      for (int i = 0; i < 4; ++i) fr[i] = __shfl(f, (4 * kq + i) % GP);
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) zacc[a][i] *= fr[i];
#pragma unroll
      for (int cs = 0; cs < NCS; ++cs)
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
          for (int a = 0; a < NAO; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) oacc[cs][m][a][i] *= fr[i];
    }
    const float mk = fmaxf(m_run * kappa, -3.0e38f) - off;   // (finite also for a column that has seen no token yet)
    float pr[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pr[t][i] = __builtin_amdgcn_exp2f(fmaf(sc[t][i], kappa, -mk));
        l_run += pr[t][i];
      }
    half8v zb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {                 // k-slots 2i, 2i+1: tokens 4i + kq of tile 0 and of tile 1
      if constexpr (SPLIT) {
        const float w0 = sgn * pr[0][i] * (float)sz_half(r.vs[0][0][i], 0);
        const float w1 = -(sgn * pr[1][i] * (float)sz_half(r.vs[0][1][i], 0));
        const auto hi = __builtin_amdgcn_cvt_pkrtz(w0, w1);
        const auto lo = __builtin_amdgcn_cvt_pkrtz(w0 - (float)hi[0], w1 - (float)hi[1]);
        pa[0][2 * i] = hi[0]; pa[0][2 * i + 1] = hi[1];
        pa[NPA - 1][2 * i] = lo[0]; pa[NPA - 1][2 * i + 1] = lo[1];
        continue;
      }
      if constexpr (TWO) {                        // (both rounded towards zero: what the first leaves out the second takes)
#pragma unroll
        for (int a = 0; a < NA; ++a) {
          const float w0 = pr[0][i] * (float)sz_half(r.vs[a >> 1][0][i], a & 1), w1 = -pr[1][i] * (float)sz_half(r.vs[a >> 1][1][i], a & 1);
          const auto hi = __builtin_amdgcn_cvt_pkrtz(w0, w1);
          const auto lo = __builtin_amdgcn_cvt_pkrtz(__builtin_fmaf((float)hi[0], -1.0f, w0), __builtin_fmaf((float)hi[1], -1.0f, w1));
          pa[a][2 * i] = hi[0]; pa[a][2 * i + 1] = hi[1];
          pa[NPA / 2 + a][2 * i] = lo[0]; pa[NPA / 2 + a][2 * i + 1] = lo[1];
        }
        continue;
      }
#pragma unroll
      for (int a = 0; a < NA; ++a) {
        pa[a][2 * i] = (_Float16)__builtin_fmaf(pr[0][i], (float)sz_half(r.vs[a >> 1][0][i], a & 1), 0.0f);
        pa[a][2 * i + 1] = (_Float16)__builtin_fmaf(-pr[1][i], (float)sz_half(r.vs[a >> 1][1][i], a & 1), 0.0f);
      }
    }
    if constexpr (C::PERM || C::WIDE) {
      uint32_t zw[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) zw[i] = __builtin_amdgcn_perm(r.zb[4 + i], r.zb[i], zb_sel) ^ 0x80000000u;
      zb = as_half8(zw[0], zw[1], zw[2], zw[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        zb[2 * i] = sz_half(r.zb[i], 0);
        zb[2 * i + 1] = -sz_half(r.zb[4 + i], 0);
      }
    }
    constexpr int NPZ = SPLIT ? NPA : NA;         // (TWO: the rest goes with zb15 below)
    static_assert(SPLIT || NPZ <= NA, "a zero-point sum for every operand");
#pragma unroll
    for (int a = 0; a < NPZ; ++a) zacc[SPLIT ? 0 : a] = mfma16(pa[a], zb, zacc[SPLIT ? 0 : a]);
#pragma unroll
    for (int a = 0; a < NPZ; ++a) zacc[SPLIT ? 0 : a] = mfma16(pa[a], pos15_odd, zacc[SPLIT ? 0 : a]);
    if constexpr (TWO) {
      const half8v zb15 = zb + pos15_odd;         // (one operand is enough for the rest, 2^-11 of the whole)
#pragma unroll
      for (int a = 0; a < NA; ++a) zacc[a] = mfma16(pa[NPA / 2 + a], zb15, zacc[a]);
    }
  };

  // -- V codes: each lane holds the same packed word (8 dims) of 8 tokens and needs, per dim, the 8 tokens in
  //    the k-slots of a B operand.  One byte-permute per (token pair, byte of the word) puts the pair's bytes
  //    into the low byte of the two halves of a register: as fp16 subnormals that is n_even + 16 n_odd of the
  //    byte's two nibbles, and one AND leaves n_even alone.  P V is linear in V, so the MIXED operand goes
  //    through the matrix core as it is (its accumulator holds  sum w (n_even + 16 n_odd) ) and the odd dim is
  //    recovered at the very end as (mixed - even) / 16: two vector instructions per pair of B registers instead
  //    of the four that separating every nibble takes.  (The mixed sum is 17 times larger and is divided by 16
  //    again: the odd dims carry about 1.5 times the accumulation noise of the even ones, a small part of the
  //    error budget.)  The complement of the second tile (15 - n in every nibble, i.e. 255 - byte) keeps both
  //    accumulators balanced around zero as before:  even: -15 sum_t1 w,  mixed: -255 sum_t1 w,  so that
  //    (mixed - even) / 16 carries the same -15 sum_t1 w that the zero-point sum cancels.
  //    WIDE: the 16 columns of a matrix instruction are the 4 words x 4 bytes of ONE group (column c = byte c / 4
  //    of word c % 4), so the lane holds that word of every group and picks its byte with a selector of its own.
  auto pv = [&](const VRegs& r, const half8v (&pa)[NPA], auto two_tag) {
    constexpr bool TWO = decltype(two_tag)::value;
    if constexpr (C::WIDE) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        uint32_t mix[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mix[i] = __builtin_amdgcn_perm(~r.v[g][i + 4], r.v[g][i], v_sel);
        const half8v v_mixed = as_half8(mix[0], mix[1], mix[2], mix[3]);
        const half8v v_even = as_half8(mix[0] & kMaskLo, mix[1] & kMaskLo, mix[2] & kMaskLo, mix[3] & kMaskLo);
        oacc[0][2 * g][0] = mfma16(pa[g], v_even, oacc[0][2 * g][0]);
        oacc[0][2 * g + 1][0] = mfma16(pa[g], v_mixed, oacc[0][2 * g + 1][0]);
      }
      return;
    }
#pragma unroll
    for (int cs = 0; cs < NCS; ++cs) {
      uint32_t v1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v1[i] = ~r.v[cs][i + 4];   // second tile: 15 - code in every nibble
#pragma unroll
      for (int j = 0; j < 4; ++j) {               // byte j of the word: dims 2j and 2j + 1
        const uint32_t sel = 0x0C000C00u | ((4u + j) << 16) | (uint32_t)j;   // [tile 0 byte j, 0, tile 1 byte j, 0]
        uint32_t mix[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mix[i] = __builtin_amdgcn_perm(v1[i], r.v[cs][i], sel);
        const half8v v_mixed = as_half8(mix[0], mix[1], mix[2], mix[3]);
        const half8v v_even = as_half8(mix[0] & kMaskLo, mix[1] & kMaskLo, mix[2] & kMaskLo, mix[3] & kMaskLo);
#pragma unroll
        for (int a = 0; a < NAO; ++a) {
          oacc[cs][2 * j][a] = mfma16(pa[a], v_even, oacc[cs][2 * j][a]);
          oacc[cs][2 * j + 1][a] = mfma16(pa[a], v_mixed, oacc[cs][2 * j + 1][a]);
        }
        if constexpr (TWO) {
#pragma unroll
          for (int a = 0; a < NA; ++a) {
            oacc[cs][2 * j][a] = mfma16(pa[NPA / 2 + a], v_even, oacc[cs][2 * j][a]);
            oacc[cs][2 * j + 1][a] = mfma16(pa[NPA / 2 + a], v_mixed, oacc[cs][2 * j + 1][a]);
          }
        }
        if constexpr (SPLIT) {
          oacc[cs][2 * j][0] = mfma16(pa[NPA - 1], v_even, oacc[cs][2 * j][0]);
          oacc[cs][2 * j + 1][0] = mfma16(pa[NPA - 1], v_mixed, oacc[cs][2 * j + 1][0]);
        }
      }
    }
  };

  // ---- main loop.  Supertile i: its K part already sits in registers; fetch its V part, compute the
  //      scores, fetch the K part of supertile i+1 (whose stage has to have landed by then), softmax,
  //      refill the ring slot of supertile i with supertile i+NS, P V.
  KRegs kr;
  VRegs vr;
  static_assert(C::PFK && NS == 2, "the waits below count one or two stages");
  auto masked = [&](int sidx, auto two_tag) {     // supertile sidx, whose stage sits in slot 0, by the masked path
    load_k(0, kr);
    load_v(0, vr);
    if constexpr (GS == 2 && D == 128) {
      // a token pair's dword may reach one token past the sequence's last: whatever lies there must not meet the
      // (zero) weights of the masked tokens as an Inf or NaN (the scores of such tokens are replaced, not scaled)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (begin + sidx * 32 + 16 * t + 4 * i + kq >= seq) {
#pragma unroll
            for (int dw = 0; dw < NDW; ++dw) vr.vs[dw][t][i] = 0;
            vr.zb[4 * t + i] = 0;
          }
    }
    float sc[2][4];
    scores(kr, sidx, std::true_type{}, sc);
    half8v pa[NPA];
    softmax(sc, vr, pa, two_tag);
    pv(vr, pa, two_tag);
  };
  auto supertiles = [&](auto two_tag) {
    int slot = 0;
    if (tail0) {
      if (n_mine > 0) wait_loads<LPS>();            // (loads land in order: the tail is in, the first full supertile may be out)
      else wait_loads<0>();
      masked(n_full, two_tag);
      if (n_mine > 1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // slot 0 has been read
        issue(0, sidx_of(1));
      }
      slot = 1;
    }
    if (n_mine > 0) {
      if ((tail0 || !kSecondAfterFirstLanded) && n_mine > 1) wait_loads<LPS>();   // (the first full supertile is in)
      else wait_loads<0>();
      load_k(slot, kr);
      if (!tail0 && kSecondAfterFirstLanded && n_mine > 1) issue(1, sidx_of(1));
    }
    for (int i = 0; i < n_mine; ++i) {
      const int next = (slot + 1 == NS) ? 0 : slot + 1;
      if constexpr (SPLIT) {
        if (2 * i >= n_mine && sgn == sgn0) negate_sums();
      }
      load_v(slot, vr);
      // The slot's bytes all sit in registers from here on; its refill with supertile i + NS is issued after the
      // softmax all the same.  (Measured at 128K / at the d = 256 instance: issued here, +0.4 / +0.6 us; issued after
      // the P V phase, +0.4 / +0.3 us; a ring of three stages, +1.0 us: the memory system is at its limit, and
      // requests queued earlier than needed only delay the ones a wave is waiting for.  Issued here AND waited for
      // stage by stage, so that two stages are in flight: the kernel alone unchanged, the decode call 1 us slower.)
      auto refill = [&] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // every LDS read of this slot has returned
        if (i + NS < n_mine) {
          issue_tok(ring_lds + slot * C::STAGE, nx_tok, paged ? page_of(nx_tok) : 0, koff, lane16, szoff);
          // next supertile of the pattern: of every PERIOD the older wave holds k = 0, 2, .., PERIOD-2 and PERIOD-1,
          // the younger k = 1, 3, .., PERIOD-3
          const int step = young ? (nx_j < YNG - 1 ? 2 : 4) : (nx_j < PERIOD / 2 - 1 ? 2 : 1);
          nx_j = (nx_j == (young ? YNG - 1 : OLD - 1)) ? 0 : nx_j + 1;
          nx_tok += whole ? step * (4 * 32) : W * 32;
        }
      };
      float sc[2][4];
      // (the wave asks for issue priority while it unpacks K, feeds the matrix cores and scales the scores: the two
      //  waves of a SIMD then take turns phase by phase rather than instruction by instruction, 0 - 1 % faster at
      //  128K from box to box, 0.4 % at the d = 256 instance)
      __builtin_amdgcn_s_setprio(1);
      scores(kr, 0, std::false_type{}, sc);
      __builtin_amdgcn_s_setprio(0);
      // The only stage out is the next supertile's.  Past the last supertile there is nothing to wait for and the
      // fetch reads unused bytes; skipping it there takes a branch in the loop, which the d = 128 instances pay for in
      // registers and schedule (16-row tile 33.3 -> 35.4 us, 8-row 28.7 -> 28.95) and the d = 256 instance gains by.
      if (D == 128 || i + 1 < n_mine) {
        wait_loads<0>();
        load_k(next, kr);
      }
      half8v pa[NPA];
      softmax(sc, vr, pa, two_tag);
      refill();
      pv(vr, pa, two_tag);
      slot = next;
    }
  };
  if constexpr (MAY_TWO) {
    if (two) supertiles(std::true_type{});
    else supertiles(std::false_type{});
  } else {
    supertiles(std::false_type{});
  }
  wait_loads<0>();                                           // (nothing is out any more: the rings are quiet)
  if constexpr ((!PLAIN && !LISTED) || LEAN) {
#pragma unroll 1
    for (int u = LEAN ? 0 : 1; u < (PLAIN ? 1 : 4); ++u) {   // further masked supertiles: the last but one with several
      if (!tail_mine[u]) continue;                           // query tokens, under a window the first (or first two)
      const int sidx = u < 2 ? n_full + u : 1 - u;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue_tail(0, sidx);
      wait_loads<0>();
      masked(sidx, std::false_type{});
    }
  }

  if constexpr (SPLIT) {
    if (sgn < 0.0f) negate_sums();
  }
  // ---- wave result -> LDS.  Of a lane's NA accumulators per row only the one whose group the lane's packed
  //      word belongs to is meaningful (and, the zero-point operand being laid out to match, the same one of its
  //      NA zero-point sums): it is selected, brought to common units (the 2^24 / 2^20 of the two nibble
  //      positions), the zero-point sum is taken off, and the eight dims of the word leave as two 16-byte writes.
  float* const lds_o = reinterpret_cast<float*>(smem + off_merge);     // [n_waves][GP][D]   sum_t p_t v^_t
  float* const lds_m = lds_o + n_waves * GP * D;                       // [GP][NW]
  float* const lds_l = lds_m + NW * GP;                                // [GP][NW]
  float* const lds_new = lds_l + NW * GP + (LISTED ? first_mate : whole ? 0 : wave / W) * C::NEWTOK;   // [D] V of this unit's new token, [GP] scores
  if constexpr (C::ALIAS) __syncthreads();                   // everybody is done reading the rings
  const bool active = n_mine > 0 || tail_mine[0] || tail_mine[1] || tail_mine[2] || tail_mine[3];
  const float l_tot = blocks_sum(l_run);
  if (kq == 0 && rep == 0) {
    // (a row whose tokens were all masked still has the initial reference: it counts as empty)
    lds_m[hl * NW + wave] = (active && m_run > kNegBig) ? m_run * kappa - off : kNegBig;
    lds_l[hl * NW + wave] = active ? l_tot : 0.0f;
  }
  if (takes) {
    if (new_v && (lane & 31) < PIECES) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        lds_new[new_piece * 8 + e] = ((float)((new_w >> (4 * e)) & 0xFu) - (float)new_sz[1]) * (float)new_sz[0];
    }
    const int copies = takes_v ? COPIES / 2 : COPIES, row_of = lane / PIECES + new_piece * copies;   // the row this lane's score is of
    if (takes_k && lane / PIECES < copies && row_of < GP) lds_new[D + row_of] = new_score * p.scale_log2;
  }
  if (busy) {
    if constexpr (C::WIDE) {
      // row 4 kq + i = head; group g's zero-point sum of that head sits in column g (any column c with c % 4 == g)
      // of zacc[g]; this lane's column is byte c / 4 of word c % 4 of every group: two neighbouring dims per group
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const float zc = __shfl(zacc[g][i], (lane & 48) | g);
          const float even = oacc[0][2 * g][0][i], mixed = oacc[0][2 * g + 1][0][i];
          float2 o2;
          o2.x = fmaf(even, 0x1p24f, -zc);
          o2.y = fmaf(mixed - even, 0x1p20f, -zc);
          *reinterpret_cast<float2*>(lds_o + (wave * GP + 4 * kq + i) * D + (4 * g + (c & 3)) * 8 + 2 * (c >> 2)) = o2;
        }
    }
#pragma unroll
    for (int i = 0; i < (C::WIDE ? 0 : 4); ++i) {
      const int r = 4 * kq + i, h = r % GP, rp = r / GP;       // accumulator row -> (head, replica)
#pragma unroll
      for (int cs = 0; cs < NCS; ++cs) {
        const int word = c * NCS + cs;              // packed word (8 dims) this lane's column stands for
        const int a_mine = (word >> 2) - rp * NA;
        const bool second = NA == 2 && a_mine == 1;
        const float zc = second ? zacc[NA - 1][i] : zacc[0][i];
        float4v lo, hi;
        float acc[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) acc[m] = second ? oacc[cs][m][NAO - 1][i] : oacc[cs][m][0][i];
#pragma unroll
        for (int m = 0; m < 4; ++m) {               // dim m: the even sum, or (mixed - even) / 16, in units of 2^-24
          lo[m] = fmaf((m & 1) ? acc[m] - acc[m - (m & 1)] : acc[m], (m & 1) ? 0x1p20f : 0x1p24f, -zc);
          hi[m] = fmaf((m & 1) ? acc[m + 4] - acc[m + 4 - (m & 1)] : acc[m + 4], (m & 1) ? 0x1p20f : 0x1p24f, -zc);
        }
        if (a_mine >= 0 && a_mine < NA) {
          float4v* dst = reinterpret_cast<float4v*>(lds_o + (wave * GP + h) * D + word * 8);
          dst[0] = lo;
          dst[1] = hi;
        }
      }
    }
  } else {                                        // (its sums carry no weight in the merge, but what lies there might be Inf or NaN)
#pragma unroll
    for (int u = 0; u < GP * D / 256; ++u) *reinterpret_cast<float4v*>(lds_o + wave * GP * D + (u * 64 + lane) * 4) = float4v{0, 0, 0, 0};
  }
  // 512 bytes for every wave, where its ring was (d = 256: behind the block-merge area): chunk weights, then (LISTED) what the
  // whole block has to know to share the rows of all its sequences: of the first of a sequence's waves, how many they are, the
  // sequence, its partial's place and their number (0 waves: not the first)
  static_assert(!C::ALIAS || (C::MERGE + 255) / 256 * 256 + NW * 512 <= C::RING, "behind the block-merge area");
  auto wave_area = [&](int w) { return smem + (C::ALIAS ? (C::MERGE + 255) / 256 * 256 + w * 512 : w * (NS * C::STAGE)); };
  typedef int int4v __attribute__((ext_vector_type(4)));
  if constexpr (LISTED) {
    if (lane == 0) *reinterpret_cast<int4v*>(wave_area(wave) + 256) = int4v{row_valid && sub == 0 ? W : 0, b, part_at, n_parts};
  }
  __syncthreads();

  // ---- merge the waves, write one partial per query row (Sec. 3.2); where the sequence is a single
  //      chunk and the kernel is to produce the output, that partial, normalised, IS the output.
  //      A wave takes a row, a lane two neighbouring dims of it (d = 256: four, or half a row and two): the waves' maxima and
  //      sums of that row arrive as 16-byte reads, the same for the whole wave.
  // row h of the waves first .. first + count - 1, its dims from j0 on, DPL of them a lane; output row `row`; written as the output
  // (direct), or as partial `part` of it
  auto merge_row = [&](auto dpl_tag, int h, int j0, int first, int count, int64_t row, bool direct, int part, bool with_new, const float* new_at) {
    constexpr int DPL = decltype(dpl_tag)::value;
    typedef float float_dims __attribute__((ext_vector_type(DPL)));
    const int j = j0 + lane * DPL;
    float_dims ow[NW];                            // (asked for first: their latency hides behind the weights' arithmetic)
#pragma unroll
    for (int w = 0; w < NW; ++w) ow[w] = *reinterpret_cast<const float_dims*>(lds_o + (min(w, n_waves - 1) * GP + h) * D + j);
    float mw[NW], lw[NW];
#pragma unroll
    for (int w4 = 0; w4 < NW; w4 += 4) {
      const float4v a = *reinterpret_cast<const float4v*>(lds_m + h * NW + w4);
      const float4v bb = *reinterpret_cast<const float4v*>(lds_l + h * NW + w4);
#pragma unroll
      for (int u = 0; u < 4; ++u) { mw[w4 + u] = a[u]; lw[w4 + u] = bb[u]; }
    }
    float mg = kNegBig;
#pragma unroll
    for (int w = 0; w < NW; ++w) mg = (w >= first && w < first + count) ? fmaxf(mg, mw[w]) : mg;
    float_dims num = 0.0f;
    float den = 0.0f;
    if (with_new) {
      const float sn = new_at[D + h];
      mg = fmaxf(mg, sn);
      den = __builtin_amdgcn_exp2f(sn - mg);
#pragma unroll
      for (int e2 = 0; e2 < DPL; e2 += 2) {       // (8-byte reads: a later unit's token is no better aligned)
        const float2 vn = *reinterpret_cast<const float2*>(new_at + j + e2);
        num[e2] = vn.x * den;
        num[e2 + 1] = vn.y * den;
      }
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < first || w >= first + count) continue;         // (wave-uniform)
      const float e = __builtin_amdgcn_exp2f(mw[w] - mg);
#pragma unroll
      for (int e4 = 0; e4 < DPL; ++e4) num[e4] = fmaf(ow[w][e4], e, num[e4]);
      den = fmaf(lw[w], e, den);
    }
    if (direct) {
#pragma unroll
      for (int e2 = 0; e2 < DPL; e2 += 2) {
        half2v r;
        r[0] = (_Float16)(num[e2] / den);
        r[1] = (_Float16)(num[e2 + 1] / den);
        *reinterpret_cast<half2v*>(p.out + row * D + j + e2) = r;
      }
    } else {
      // device-scope stores: they go through to where every compute die sees them (the L2 caches of
      // different dies are not coherent with each other), so no cache-wide write-back is needed later
      const int64_t ph = row * part_stride + part;
#pragma unroll
      for (int e2 = 0; e2 < DPL; e2 += 2) st_dev2(p.part_o + ph * D + j + e2, num[e2], num[e2 + 1]);
      if (j == 0) st_dev2(p.part_ml + ph * 2, mg, den);
    }
  };
  int my_row = 0, my_n = 0, n_mine_rows = 0;      // lane i: the i-th row this wave has a partial of, and how many partials it has
  if constexpr (LISTED) {
    // the rows of all the block's sequences, dealt to all its waves
    const int4v entry = *reinterpret_cast<const int4v*>(wave_area(lane & (NW - 1)) + 256);
    int u = wave;                                 // this wave's next row, counted from the sequence's first
    for (uint64_t leads = __builtin_amdgcn_ballot_w64(lane < NW && entry[0] > 0); leads != 0; leads &= leads - 1, u -= G) {
      const int lead = __builtin_ctzll(leads);
      const int count = __builtin_amdgcn_readlane(entry[0], lead), bb = __builtin_amdgcn_readlane(entry[1], lead);
      const int part = __builtin_amdgcn_readlane(entry[2], lead), parts = __builtin_amdgcn_readlane(entry[3], lead);
      for (; u < G; u += NW) {
        const int row = bb * p.n_q_heads + kv * G + u;
        merge_row(std::integral_constant<int, D / 64>{}, u, 0, lead, count, row, parts == 1, part, p.k_new != nullptr && part == 0, lds_l + NW * GP + lead * C::NEWTOK);
        if (parts == 1) continue;
        if (lane == n_mine_rows) {
          my_row = row;
          my_n = parts;
        }
        ++n_mine_rows;
      }
    }
    if (n_mine_rows == 0) return;
  } else {
    const bool direct = p.merge_slot >= 0 && p.n_splits == 1;
    const int first = whole ? 0 : wave - sub, count = whole ? NW : W;
    if (!whole) {                                 // several units per block: the W waves of one merge among themselves
      // (a single-chunk row: the output; a slot of the chunk list: its partial)
      // (halves of rows at d = 256, where the rows are as few as the waves)
      if (row_valid)
        for (int u = sub; u < G * (D / 128); u += W) {
          const int h = u / (D / 128);
          merge_row(std::integral_constant<int, 2>{}, h, u % (D / 128) * 128, first, count, query_row(h), direct, split, new_here, lds_new);
        }
      return;
    }
    if (D == 256 && (direct || p.merge_slot < 0)) {      // (no row to count in: a wave to half a row, where the rows are as few as two)
      for (int u = wave; u < G * (D / 128); u += NW) {
        const int h = u / (D / 128);
        merge_row(std::integral_constant<int, 2>{}, h, u % (D / 128) * 128, 0, NW, query_row(h), direct, split, new_here, lds_new);
      }
      return;
    }
    for (int h = wave; h < G; h += NW)
      merge_row(std::integral_constant<int, D / 64>{}, h, 0, 0, NW, query_row(h), direct, split, new_here, lds_new);
    if (p.merge_slot < 0 || direct || wave >= G) return;
  }

  // ---- chunk merge (Eq. 6), row by row, by whichever wave that has this row finishes last.  A wave publishes
  //      its row's partial (device-scope stores, waited for), then counts itself in; the one that sees all
  //      others counted re-reads the row's partials, with device-scope loads and in chunk order, so the
  //      result does not depend on which wave that is.  No barrier: a row is one wave's in every block, and the rows of
  //      a KV head may be merged by different blocks.  What bounds it is the chain store, count, fetch, and for 32 chunks
  //      the fetch through one compute unit.  (Counted block by block, two barriers, 8-byte loads with an address
  //      each: us per step 8 heads over 1, 1024 tokens, 4 chunks, 7.94 -> 7.68; 64 over 8, 8K, 32 chunks, 10.02 -> 9.35, 32K
  //      14.4 -> 14.05; d = 256, 4 chunks, 8.78 -> 8.56.)
  // What orders the partials before their readers is the machine's memory model for device-scope accesses,
  // not a pair of fences: every partial is written with device-scope atomic stores (write-through: complete, as
  // counted by vmcnt, once the data sits where every compute die reads it), the wave waits for vmcnt(0)
  // before it counts itself in with a device-scope atomic, and the last wave
  // issues its device-scope loads (which do not hit lines a die cached earlier) only after that atomic has
  // returned.  A release fence before the count and an acquire fence after it (agent scope) were measured instead:
  // each block then writes its die's whole L2 back and invalidates it, and a decode of 256 blocks over 8K tokens
  // goes from 11.0 to 13.5 us (release alone +1.2 us, acquire alone +0.9 us), more than the separate merge kernel
  // costs (13.1 us), for no access that the atomics do not already cover.
  if constexpr (GP <= 8) {                        // (a 16-row tile's chunks go to the merge kernel)
    static_assert(GP <= NW && kMergeMaxChunks <= 64, "a wave per row, a lane per chunk");
    wait_loads<0>();                              // vmcnt counts stores too: this wave's partials have landed
    // Everything is asked for at once: the row's (m, l), a chunk per lane, and the chunks' outputs, sixteen bytes a lane (D / 4
    // lanes to a chunk, PARTS chunks to an instruction).  The row's partials are addressed as a buffer of n chunks: what lies
    // past the last one reads as zero, and its weight is zero.  (The whole offset goes in per lane: it is what a raw buffer's bound is
    // promised to be checked against, the scalar offset is not.)
    auto merge_chunks = [&](int64_t row, int n) {
      constexpr int PARTS = 256 / D;
      float* const c_w = reinterpret_cast<float*>(wave_area(wave));          // [kMergeMaxChunks]
      const int cpart = PARTS == 2 ? lane >> 5 : 0, j = (lane % (D / 4)) * 4;
      float2 ml = {kNegBig, 0.0f};
      if (lane < n) ml = ld_dev2(p.part_ml + (row * part_stride + lane) * 2);
      const auto rows = __builtin_amdgcn_make_buffer_rsrc(p.part_o + row * part_stride * D, 0, n * D * 4, 0x00020000);
      auto fetch = [&](auto count_tag, int c0, float4v* o) {   // chunks c0 + cpart * U ..
        constexpr int U = decltype(count_tag)::value;
#pragma unroll
        for (int u = 0; u < U; ++u)
          o[u] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rows, ((c0 + cpart * U + u) * D + j) * 4, 0, 16));   // 16: device scope
      };
      float4v num = {0, 0, 0, 0};
      auto add = [&](auto count_tag, int c0, const float4v* o) {
        constexpr int U = decltype(count_tag)::value;
        const float* const w = c_w + c0 + cpart * U;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float e = w[u];
#pragma unroll
          for (int k = 0; k < 4; ++k) num[k] = fmaf(o[u][k], e, num[k]);
        }
      };
      float den = 0.0f;
      auto all = [&](auto count_tag) {
        constexpr int U = decltype(count_tag)::value;
        float4v o[U];
        fetch(count_tag, 0, o);
        const float top = wave_fmax(ml.x);          // (every lane takes part)
        const float w = lane < n ? __builtin_amdgcn_exp2f(ml.x - top) : 0.0f;
        c_w[lane] = w;
        den = wave_fsum(ml.y * w);
        add(count_tag, 0, o);
        for (int c0 = U * PARTS; c0 < n; c0 += U * PARTS) {
          fetch(count_tag, c0, o);
          add(count_tag, c0, o);
        }
      };
      if (n <= 4 * PARTS) all(std::integral_constant<int, 4>{});
      else if (n <= 8 * PARTS) all(std::integral_constant<int, 8>{});
      else all(std::integral_constant<int, 16>{});
      if constexpr (PARTS == 2) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float a, b2;
          swap32(num[k], a, b2);
          num[k] = a + b2;
        }
      }
      if (cpart == 0) {
        typedef _Float16 half4v __attribute__((ext_vector_type(4)));
        half4v r;
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = (_Float16)(num[k] / den);
        *reinterpret_cast<half4v*>(p.out + row * D + j) = r;
      }
    };
    auto arrived = [&](int row, int n) {          // whether all other partials of the row have been counted in (wraps to 0 on the last)
      return atomicInc(&g_arrivals[p.merge_slot * kCountersPerSlot + arrival_counter(row)], (unsigned int)(n - 1)) == (unsigned int)(n - 1);
    };
    if constexpr (LISTED) {                       // all of the wave's rows at once
      bool last = false;
      if (lane < n_mine_rows) last = arrived(my_row, my_n);
      uint64_t rows_last = __builtin_amdgcn_ballot_w64(last);
      asm volatile("" ::: "memory");              // (no load may move above the count)
      for (; rows_last != 0; rows_last &= rows_last - 1) {
        const int i = __builtin_ctzll(rows_last);
        merge_chunks(__builtin_amdgcn_readlane(my_row, i), __builtin_amdgcn_readlane(my_n, i));
      }
    } else {
      const int64_t row = query_row(wave);
      int last = 0;
      if (lane == 0) last = arrived((int)row, p.n_splits);
      if (__builtin_amdgcn_readfirstlane(last) == 0) return;
      asm volatile("" ::: "memory");
      merge_chunks(row, p.n_splits);
    }
  }
}

int padded_gqa(int head_dim, int gqa) {           // columns a group of `gqa` heads takes in the tile; 0 = too many
  if (head_dim == 128) return gqa <= 4 ? 4 : (gqa <= 8 ? 8 : (gqa <= 16 ? 16 : 0));
  return gqa <= 2 ? 2 : 0;
}
// At d = 128 a tile holds up to 16 query rows (at about 1.25 times the 8-row tile's time per token), at d = 256 two.
// A group with more rows is cut into the fewest equal parts that fit, one block each on the same KV head.
// (16 heads per KV head, one sequence, one 16-row block against two 8-row blocks: 8K tokens 14.4 against 15.5 us,
// 32K 18.8 against 19.7, 128K 39.8 against 52.1; 8 sequences of 32K 64.3 against 102.8 us.)
int kv_share_of(int head_dim, int gqa) {
  if (gqa < 1 || (head_dim != 128 && head_dim != 256)) return 0;
  // d=256: a tile of 4 rows needs more registers than a lane has (its loop spills), and two blocks of 2 rows
  // that stream the same KV head are faster than one of 4 (measured: 52.9 us against 69.0 us at 64/16 heads, 32K)
  const int cap = head_dim == 128 ? 16 : 2;
  for (int share = (gqa + cap - 1) / cap; share <= gqa; ++share)
    if (gqa % share == 0) return share;
  return 0;
}

template <int D, int GP, bool NT, Mode MODE, int GS = 0>
hipError_t launch_as(const DecodeParams& p, dim3 grid, hipStream_t s) {
  // one block of 8 waves per compute unit: 8 rings of 2 x 5 KB (d=128) or 2 x 10 KB (d=256, all 160 KB of LDS)
  constexpr int NW = 8;
  using C = Cfg<D, GP, NW, GS>;
  constexpr int smem = C::SMEM;
  // a block of W < 8 waves for one row (`ranked`): its share of the LDS, so that as many fit a compute unit as its
  // eight wave slots take (two per SIMD)
  const int waves = p.ranked ? p.waves_per_row : NW;
  const int rings = waves * C::NS * C::STAGE, merge = (waves * GP * D + 2 * NW * GP + (p.ranked ? 2 : NW) * C::NEWTOK) * 4;
  const int smem_used = C::ALIAS ? std::max(rings, merge) : rings + merge + (C::QSEP ? waves * C::QAREA : 0);
  if (smem_used > smem) return hipErrorInvalidValue;
  static_assert(smem <= 160 * 1024, "LDS budget of one compute unit");
  // dynamic LDS above 64 KB has to be opted into, once per device and kernel instance (any thread may get here first)
  static std::once_flag configured[kMaxDevices];
  static hipError_t outcome[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::call_once(configured[dev], [&] {
    outcome[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_partial_mfma_kernel<D, GP, NW, NT, MODE, GS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (outcome[dev] != hipSuccess) return outcome[dev];
  hipLaunchKernelGGL((decode_partial_mfma_kernel<D, GP, NW, NT, MODE, GS>), grid, dim3(waves * 64), smem_used, s, p);
  return hipGetLastError();
}
// the stream is read once (non-temporal loads) unless several blocks share a KV head
template <int D, int GP, Mode MODE, int GS>
hipError_t launch_nt(const DecodeParams& p, dim3 grid, hipStream_t s) {
  return p.kv_share == 1 ? launch_as<D, GP, true, MODE, GS>(p, grid, s) : launch_as<D, GP, false, MODE, GS>(p, grid, s);
}
template <int D, int GP, int GS>
hipError_t launch_mode(const DecodeParams& p, dim3 grid, hipStream_t s) {
  if constexpr (GP <= 8) {
    if (p.listed) return p.block_table ? launch_as<D, GP, true, kListedPaged, GS>(p, grid, s) : launch_as<D, GP, true, kListed, GS>(p, grid, s);
  }
  if (p.block_table != nullptr) return launch_nt<D, GP, kPaged, GS>(p, grid, s);
  const bool plain = p.kv_share == 1 && p.n_queries == 1 && p.waves_per_row == 8 && p.var_chunks == 0 && p.seq_lens == nullptr;
  if constexpr (GS == 0 || D == 256) {            // (no plain instances of the larger groups at d = 128)
    if constexpr (lean_tile<GP, true, kPlain, GS>()) {
      if (plain && p.k_new != nullptr) return launch_as<D, GP, true, kPlainStep, GS>(p, grid, s);
    }
    if (plain) return launch_as<D, GP, true, kPlain, GS>(p, grid, s);
  }
  return launch_nt<D, GP, kGeneral, GS>(p, grid, s);
}
template <int D, int GP>
hipError_t launch(const DecodeParams& p, dim3 grid, hipStream_t s) {
  if constexpr (D == 256 || GP >= 8) {            // groups of 64 / 128 elements
    if (p.group == 2 * kGroup) return launch_mode<D, GP, 1>(p, grid, s);
    if (p.group == 4 * kGroup) return launch_mode<D, GP, 2>(p, grid, s);
  }
  return p.group == kGroup ? launch_mode<D, GP, 0>(p, grid, s) : hipErrorNotSupported;
}

}  // namespace

int mfma_kv_share(int head_dim, int gqa) { return kv_share_of(head_dim, gqa); }

bool mfma_supported(int head_dim, int gqa) { return kv_share_of(head_dim, gqa) > 0; }

// Groups of 64 or 128 elements: at head_dim 256 always (a token's values fill whole dwords); at head_dim 128 two
// tokens share a dword of every metadata array where groups are 128 elements, and that dword has to be aligned and
// must not straddle two (sequence, KV head) rows: an even number of tokens per row.
bool mfma_supports_group(int head_dim, int group, int capacity) {
  if (group == kGroup || head_dim == 256) return true;
  return head_dim == 128 && (group == 2 * kGroup || (group == 4 * kGroup && capacity % 2 == 0));
}

// A 16-row tile that shares its KV head with others does not (LEAN).
bool mfma_takes_token(int head_dim, int group, int rows) {
  const int share = kv_share_of(head_dim, rows);
  return share > 0 && !(share > 1 && group == kGroup && padded_gqa(head_dim, rows / share) == 16);
}

bool mfma_can_merge(int64_t out_rows) { return out_rows <= kCountersPerSlot; }

namespace {
struct MergeSlots {
  std::mutex guard;
  std::unordered_map<const void*, int> of;        // workspace -> set
};
MergeSlots& merge_slots() {
  static MergeSlots slots;
  return slots;
}
}  // namespace

int mfma_merge_slot_of(const void* workspace) {
  MergeSlots& slots = merge_slots();
  std::lock_guard<std::mutex> lock(slots.guard);
  const auto it = slots.of.find(workspace);
  if (it != slots.of.end()) return it->second;
  if ((int)slots.of.size() >= kCounterSlots) return -1;
  const int slot = (int)slots.of.size();
  slots.of.emplace(workspace, slot);
  return slot;
}

int mfma_merge_slots_left() {
  MergeSlots& slots = merge_slots();
  std::lock_guard<std::mutex> lock(slots.guard);
  return kCounterSlots - (int)slots.of.size();
}

hipError_t launch_partial_mfma(const DecodeParams& p_in, int batch, int head_dim, int merge_slot, hipStream_t s) {
  DecodeParams p = p_in;
  if (p.n_queries < 1) p.n_queries = 1;
  if (p.n_queries > kMaxQueries) return hipErrorNotSupported;
  p.gqa_full = p.gqa;
  // blocks per KV head: the caller's choice (it sized the chunk plan by it), checked against the tiles there are
  const int rows = p.gqa * p.n_queries;
  if (p.kv_share < 1 || rows % p.kv_share != 0 || padded_gqa(head_dim, rows / p.kv_share) == 0) return hipErrorNotSupported;
  p.gqa = rows / p.kv_share;
  const int rows_y = p.n_kv_heads * p.kv_share;
  p.merge_slot = -1;
  if (merge_slot >= 0) {
    if ((p.n_splits > 1 && !mfma_can_merge((int64_t)batch * p.n_queries * p.n_q_heads)) || p.out == nullptr || merge_slot >= kCounterSlots)
      return hipErrorInvalidValue;
    p.merge_slot = merge_slot;
  }
  if (p.waves_per_row != 1 && p.waves_per_row != 2 && p.waves_per_row != 4) p.waves_per_row = 8;
  if (p.ranked && (p.seq_lens == nullptr || p.merge_slot < 0 || p.n_splits != 1 || p.var_chunks > 0)) return hipErrorInvalidValue;
  if (p.ranked && p.waves_per_row == 1 && p.rank_spread >= 0) return hipErrorInvalidValue;   // (a wave is not shared by two rows)
  if (p.listed && (p.seq_lens == nullptr || p.merge_slot < 0 || p.ranked || p.n_queries > 1 || p.window > 0 || p.kv_share != 1 ||
                   batch > kListMaxBatch || (int64_t)batch * p.seq_len >= (1ll << 31) || p.var_chunks % 8 != 0 || p.var_chunks <= batch ||
                   !mfma_can_merge((int64_t)batch * p.n_q_heads) || padded_gqa(head_dim, p.gqa) > 8))
    return hipErrorInvalidValue;
  // several units per block: single-chunk rows whose output the kernel writes itself, or the slots of a chunk list
  if (p.waves_per_row != 8 && !p.ranked && p.var_chunks == 0 && (p.merge_slot < 0 || p.n_splits != 1 || p.block_table))
    return hipErrorInvalidValue;
  const int per_block = p.ranked ? 1 : 8 / p.waves_per_row;
  const dim3 grid = p.listed ? dim3(rows_y, p.var_chunks / 8, 1)
                    : p.var_chunks > 0 ? dim3((p.var_chunks + per_block - 1) / per_block, rows_y, 1)
                    : per_block > 1  ? dim3(1, (batch * rows_y + per_block - 1) / per_block, 1)
                                     : dim3(p.n_splits, rows_y, batch);
  int gp = padded_gqa(head_dim, p.gqa);
  // (a 16-row tile has no chunk merge of its own: `out` would stay unwritten)
  if (gp == 16 && p.merge_slot >= 0 && p.n_splits > 1) return hipErrorInvalidValue;
  if (p.merge_slot >= 0 && !p.listed && p.n_splits > kMergeMaxChunks) return hipErrorInvalidValue;
  if (p.k_new != nullptr && !mfma_takes_token(head_dim, p.group, rows)) return hipErrorInvalidValue;
  if (p.group != kGroup && gp == 4) gp = 8;       // (larger groups at d = 128: the 8- and 16-row layouts only)
  if (head_dim == 128 && gp == 16) return launch<128, 16>(p, grid, s);
  if (head_dim == 128 && gp == 8) return launch<128, 8>(p, grid, s);
  if (head_dim == 128 && gp == 4) return launch<128, 4>(p, grid, s);
  if (head_dim == 256 && gp == 2) return launch<256, 2>(p, grid, s);
  return hipErrorNotSupported;
}

}  // namespace tq
