// Matrix-core fused int4 decode attention for many query rows per KV head: head_dim 512 (the global-attention column of the
// kernel configuration table, Appendix A: 32 query heads on one KV head) and head_dim 256 and 128 where the kernel with
// few rows to a block would unpack the stream again and again; phase 1 of Sec. 3.2.
//
// A KV head's query rows form tiles of 16 (every column of a matrix instruction is a row of its own), every fetched
// byte is used by all of them, and the work is arithmetic, not traffic: the vector ALU prepares the operands of the
// matrix instructions, and how often it does so per stored element is what the kernel's time goes by.
//
// One block of eight waves = one chunk of one KV head x one tile of 16 * RT query rows.  Both contractions of Alg. 1 run
// in rounds, and the waves split each along the dimension that nothing has to be summed over:
//   scores  by TOKENS: a wave takes WT tokens of the round whole, S^T = K Q^T (rows = 16 tokens, columns = 16 query rows), one
//           MFMA per group: lane (kq, c) feeds packed word kq of the group of token c, its codes as fp16 SUBNORMALS (value
//           c 2^-24, or c 2^-20 for a nibble at bit 4: two ANDs per word pair, and the products and their sum are exact in
//           the fp32 accumulator).  Scale and zero-point are applied to the accumulator in fp32,
//             q.k^ = sum_g s_g (q_g.c_g - z_g sum(q_g)).
//           The wave's weights (32 bits) go to LDS, with the reference of its exponentials: the round's one barrier.
//   P V     by DIMS: a wave takes two groups (64 dims) of all the round's tokens (d = 256 / 128: of every
//           second / fourth supertile, two / four waves to the groups).  The accumulator layout of S^T (lane =
//           query row, four tokens per lane and 16-token tile) IS the A-operand layout of P, so a lane reads back what the same
//           lane of the scoring wave wrote.  The 16 columns of one instruction lie in ONE group (column c = byte c / 4
//           of word c % 4), so that A = fp16(p s_v) (d = 128: in two parts, see SPLIT) is right for all of them and the codes enter exactly: a
//           byte's two nibbles mixed (n_even + 16 n_odd, an exact subnormal) next to n_even alone, the odd dim
//           recovered from the two sums at the end.  The zero-points go through one more instruction per group with the
//           same A.  The second 16-token tile enters with its weights negated and its codes complemented, which keeps all
//           sums at the size of the result (the matrix core truncates what it aligns to a large accumulator).
// So the operands of either contraction are prepared once per block, the scores need no exchange, a wave's sums take 24
// registers (192, if a wave kept all of a row's dims for the tokens it scored) and no sums are merged at the end.
// Measured against four waves that split the head dimension for both contractions, exchanged partial scores (a barrier per
// 32 tokens) and multiplied V out into fp16 (us per step): 32 heads on one KV head, 32K tokens 28.0 -> 18.7, 128K 71.5 ->
// 40.1, 8 sequences of 32K 74.9 -> 69; 16 heads on two 27.4 -> 19.3; 32 heads over 8 49.2 -> 40.4; the error against 64
// bits 3.6e-4 -> 2.9e-4.  (Eight waves in lock step with the dims split likewise: 25.1; a wave that keeps whole tokens and all
// dims: the compiler moves the 192 accumulator registers about.)  A round of 128 tokens takes about 3.5 us, 72 - 78 % of it
// the vector port's: some 660 instructions a wave, two waves to a SIMD.
//
// Data path: the packed stream goes from global memory straight into LDS (global_load_lds_dwordx4, no registers in
// between).  K is private to the wave that scores it: a slot of 256 dims is refilled with the next round's as soon as it sits in
// registers; V is brought in by all waves, one round ahead.  The source address of such a load is free per lane while its
// LDS destination is linear, so the 16-byte pieces of a token (one per group) are permuted by the token's number on the way
// in: both the K reads (16 tokens at once, one word of the same group) and the V reads (four tokens at once) then fall
// into different banks, and the scales and zero-points of V come to lie token by token for each pair of groups.
//
// Query rows: n_queries * G rows (t, g) per KV head (several query tokens: the sequence's last n_queries
// tokens, causal among themselves), cut into tiles of 16 * RT rows; each row has its own [first, end) of
// visible tokens, applied to the scores of the supertiles that not every row sees in full.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "tq_internal.h"

namespace tq {
namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint16_t ushort2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

constexpr int kMaxDevices = 64;
constexpr float kNegBig = -1.0e30f;         // "no token seen yet" (finite: no inf - inf)
constexpr float kSlack = 2.0f;              // log2 units: exp2(score - reference) <= 4
// The weights p carry 2^kLift, so that p s_v is a normal fp16 number from 2^-26 on (2^-14 without) and below 2^15 for scales of V below 2.
// Without the lift the weights of small scales were subnormals of one fixed spacing (relative error against 64 bits, scores of spread 2
// (nats), V of spread 1 / 1e-2 / 1e-3, without -> with: d = 512, 32K tokens 2.5e-4 / 3.8e-4 / 2.6e-3 -> 2.5e-4 / 2.5e-4 / 5.2e-4;
// d = 128, 4 query tokens, 8K 2.1e-4 / 7.0e-4 / 5.3e-3 -> 2.1e-4 / 2.1e-4 / 2.7e-4; the output's own rounding is 2.1e-4 / 2.1e-4 / 2.7e-4 ..
// 5.0e-4).  What remains of the spacing, 2^-24 of a lifted weight, moves a result by less than the spacing of fp16 outputs.  For scales from
// 2 on see sv_lim.  The lift is part of the reference that the partial is published with.  us per step, without -> with: 18.55 -> 18.65 (d = 512,
// 32K), 39.6 -> 40.1 (128K), 14.13 -> 14.2 (d = 128, 4 query tokens, 8K), 40.7 -> 41.1 (d = 256, 32 heads over 4, 128K).  (A power of two
// common to the block, from the largest scale it has met, exchanged at the round's barrier: 19.0, 14.45, 41.6.)
constexpr float kLift = 12.0f;
constexpr uint32_t scale_limit(uint32_t e) { return (e << 10 | 0x3FFu) * 0x10001u; }   // the largest scale of biased fp16 exponent e, twice
constexpr uint32_t kPlainScales = scale_limit(15);
constexpr uint32_t kMaskLo = 0x000F000Fu;   // nibbles 0 and 4 of a word -> fp16 subnormals c * 2^-24
constexpr uint32_t kMaskHi = 0x00F000F0u;   // nibbles 1 and 5           -> c * 2^-20
constexpr uint32_t kPos15Odd = 0x4B800000u; // fp16 pair (0, 15): k-slots alternate first tile, second tile

__device__ __forceinline__ half8v as_half8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  return __builtin_bit_cast(half8v, uint4v{a, b, c, d});
}
__device__ __forceinline__ half8v unpack_word(uint32_t w) {   // 8 nibbles -> 8 fp16 subnormals, dims 0,4,1,5,2,6,3,7
  const uint32_t s = w >> 8;
  return as_half8(w & kMaskLo, w & kMaskHi, s & kMaskLo, s & kMaskHi);
}
__device__ __forceinline__ float4v mfma16(half8v a, half8v b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float half_of(uint32_t w, int hi) {
  return (float)__builtin_bit_cast(half_t, (uint16_t)(hi ? w >> 16 : w));
}
// D: head dimension.  RT: 16-row tiles of query rows.  TT: 16-token tiles a wave scores per round.
template <int D, int RT, int TT>
struct Tile {
  static constexpr int NW = 8;                      // waves: two to a SIMD
  static constexpr int NG = D / kGroup;             // groups, and 16-byte pieces of codes, per token
  static constexpr int LG = D == 512 ? 4 : D == 256 ? 3 : 2;
  static constexpr int SL = D / 128;                // slices of four groups
  static constexpr int TB = D / 2;                  // bytes of codes per token
  static constexpr int SZB = NG * 2;                // bytes of one scale / zero-point array per token
  static constexpr int WT = 16 * TT, R = NW * WT;   // tokens of a wave, and of the block, per round
  // K, private to the wave: slots of SG slices: codes [token][piece], k_scale and k_zero as [slice][token][group]
  static constexpr int SG = TT == 1 ? 2 : 1, SP = SL / SG;
  static constexpr int K_SC = WT * SG * 64, K_SLOT = K_SC + 2 * WT * SG * 8;
  static constexpr int NK = SP > 1 ? SP : 2;        // slots: a round's (at one: two rounds')
  static constexpr int KOPS = 4;                    // load instructions per slot
  // V, read by all waves: one block per wave that brings it in: codes, and v_scale, v_zero as [pair of groups][token], of its
  // WT tokens; two rounds
  static constexpr int V_SC = WT * TB, V_Z = V_SC + WT * SZB, V_BLK = V_Z + WT * SZB;
  static constexpr int VC = V_SC / 1024, VM = WT * SZB / 256, VOPS = VC + 2 * VM;
  // weights p of a round, [wave's tile][row tile][lane] x 4, and the reference of each wave, [row][wave]; two rounds
  static constexpr int P_M = NW * TT * RT * 1024, P_BLK = P_M + 16 * RT * NW * 4;
  static constexpr int OFF_V = NW * NK * K_SLOT, OFF_P = OFF_V + 2 * NW * V_BLK;
  static constexpr int OFF_Q = OFF_P + 2 * P_BLK;     // sums of q over the groups, [row][group]
  // a step's new tokens, quantised: [token][K | V]: codes, (scale, zero-point) of each group
  static constexpr int N_ROW = TB + NG * 4, OFF_N = OFF_Q + 16 * RT * NG * 4, SMEM = OFF_N + kMaxQueries * 2 * N_ROW;
  static constexpr int NOPS = D == 512 ? 2 : 1;     // load instructions for a new token's K and V
  // query rows, brought in by the first QW waves, RPW each (into the second V round)
  static constexpr int ROWS = 16 * RT, QW = ROWS * D * 2 / 1024 < NW ? ROWS * D * 2 / 1024 : NW, RPW = ROWS / QW, QOPS = RPW * D * 2 / 1024;
  // The weights p s_v enter the matrix core as two fp16 operands, the leading part and the rest.  At d = 128 the kernels this one
  // takes over from have a reference per wave, which makes the weight of every wave's largest score exact in fp16; with one
  // reference to the block one operand has 3 - 10 % more error against 64 bits than they (2.25e-4 .. 2.45e-4, 2.2e-4 .. 2.35e-4), two
  // have less (2.07e-4, nearly all of it the output's own rounding).  It costs 16 vector and 3 matrix instructions per 32 tokens
  // and group (64 heads over 8, 4 query tokens, 32K tokens 22.4 -> 25.0 us per step; the rest by one fma_mixlo an element 26.4).
  // At d = 256 the kernel before has a reference per wave too (error of this one over its: scores of spread 0.16 0.997 .. 1.011, of 1
  // 0.97 .. 1.04, of 2 1.01 .. 1.05, 2.14e-4 -> 2.24e-4 of which the output's rounding is 2.07e-4; 0.1 .. 0.9 for V of spread 1e-2 and less), but
  // two operands cost 10 - 13 % of the time there (32 heads over 4, 128K 41 -> 47): one.
  static constexpr bool SPLIT = D == 128;
  static constexpr int GPW = 2, TH = NW * GPW / NG; // groups of V a wave takes; waves that share them (each every TH-th supertile)
  static_assert(SMEM <= 160 * 1024 && QOPS * 1024 == RPW * D * 2 && ROWS * D * 2 + NW * NOPS * 1024 <= NW * V_BLK && kMaxQueries <= NW && VC * 1024 == V_SC, "LDS");
  static_assert(TT * SG == 2, "a slot is 2 KB of codes and 2 x 256 B of scales and zero-points");
  static __device__ constexpr int place(int tok, int piece) { return piece ^ ((tok & 15) >> (4 - LG)); }   // V: place of a token's piece
};

// Direct global -> LDS loads of 16 (4) bytes per lane: lane l's bytes land at lds_base + l * 16 (4); M0 carries the base.
// NT: the non-temporal cache policy, where no other block reads the same bytes.
template <bool NT>
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_base) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" :: "v"(voff), "s"(sbase), "s"(lds_base) : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(voff), "s"(sbase), "s"(lds_base) : "memory");
}
template <bool NT>
__device__ __forceinline__ void dma4(const void* sbase, uint32_t voff, uint32_t lds_base) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1 nt" :: "v"(voff), "s"(sbase), "s"(lds_base) : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" :: "v"(voff), "s"(sbase), "s"(lds_base) : "memory");
}
__device__ __forceinline__ void dma16_lane(const void* addr, uint32_t lds_base) {   // per-lane 64-bit address
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(addr), "s"(lds_base) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {    // until at most N vector-memory loads of this wave are outstanding
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// device-scope store of two floats: it goes through to where every compute die sees it, so nothing is left to be written
// back at the end of the kernel, before the merge kernel may start
__device__ __forceinline__ void st_dev2(float* p, float a, float b) {      // (8-byte aligned)
  const uint64_t bits = (uint64_t)__builtin_bit_cast(uint32_t, a) | ((uint64_t)__builtin_bit_cast(uint32_t, b) << 32);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A wave-uniform value that was fetched by a vector load, in a scalar register (what it goes into is scalar asm operands).
__device__ __forceinline__ int scalar(int x) {
  asm volatile("" : "+v"(x));
  return __builtin_amdgcn_readfirstlane(x);
}
// every LDS access of this wave done, then the block's barrier (loads into LDS may stay out)
__device__ __forceinline__ void block_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// LDS by its 32-bit address: what is constant of it goes into the instruction's offset
template <typename T>
__device__ __forceinline__ T lds_get(uint32_t at) { return *(const __attribute__((address_space(3))) T*)(uintptr_t)at; }
template <typename T>
__device__ __forceinline__ void lds_put(uint32_t at, T x) { *(__attribute__((address_space(3))) T*)(uintptr_t)at = x; }

// PLAIN: one common length in a contiguous cache (what serves the other launches folds away: the first loads leave sooner).
template <int D, int RT, int TT, bool NT, bool PLAIN>
__global__ __launch_bounds__(512, 2) void decode_partial_wide_kernel(DecodeParams p) {
  using C = Tile<D, RT, TT>;
  constexpr int NW = C::NW, NG = C::NG, SL = C::SL, TB = C::TB, SZB = C::SZB, WT = C::WT, R = C::R, KOPS = C::KOPS, VOPS = C::VOPS,
                GPW = C::GPW, TH = C::TH;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  if constexpr (PLAIN) {
    // every kernel argument the prologue needs, asked for at once: one round trip to the scalar cache
    asm volatile("" :: "s"(p.q), "s"(p.start), "s"(p.k_codes), "s"(p.v_codes), "s"(p.k_scale), "s"(p.k_zero), "s"(p.v_scale),
                 "s"(p.v_zero), "s"(p.seq_len), "s"(p.tokens_per_split), "s"(p.row_stride), "s"(p.n_kv_heads), "s"(p.n_q_heads),
                 "s"(p.gqa), "s"(p.n_queries), "s"(p.kv_share));
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, kq = lane >> 4;

  int split = blockIdx.x, b = blockIdx.z, tokens_per_split = p.tokens_per_split, part_stride = p.n_splits;
  if (!PLAIN && p.var_chunks > 0) {               // per-sequence lengths: which (sequence, chunk) is this block's
    VarPlan vp;
    if (!var_plan(p, blockIdx.x, vp)) return;
    split = __builtin_amdgcn_readfirstlane(vp.chunk);           // (wave-uniform by construction: tell the compiler)
    b = __builtin_amdgcn_readfirstlane(vp.b);
    tokens_per_split = __builtin_amdgcn_readfirstlane(vp.chunk_tokens);
    part_stride = kMaxSplits;
  }
  const int tiles = NT ? 1 : p.kv_share;          // row tiles per KV head
  const int kv = tiles == 1 ? blockIdx.y : blockIdx.y / tiles, tile = blockIdx.y - kv * tiles;
  const int NQ = p.n_queries, GF = p.gqa, rows_total = NQ * GF;

  const int seq = PLAIN ? p.seq_len : scalar(p.seq_lens ? var_len(p, b) : p.seq_len);       // tokens the LAST query token attends, from `start`
  const int start = PLAIN ? p.start : scalar(p.seq_lens ? var_start(p, b) : p.start);
  const bool paged = !PLAIN && p.block_table != nullptr;
  // paged cache under a window: the chunks count from a 32-token boundary up to 31 tokens before the window
  const int lead = PLAIN ? 0 : scalar((paged && p.seq_lens) ? var_first(p, b) - start : 0);
  const int begin = split * tokens_per_split;
  if (begin >= seq) return;                       // chunk past the end of its sequence: nothing to emit
  const int end = min(seq, begin + tokens_per_split);
  const int64_t row0 = (int64_t)(b * p.n_kv_heads + kv) * p.row_stride + start;

  auto row_of = [&](int r, int& t_q) -> int64_t {               // tile row -> row of q / out / the partials
    t_q = NQ > 1 ? r / GF : 0;
    return (int64_t)(b * NQ + t_q) * p.n_q_heads + kv * GF + (r - t_q * GF);
  };

  // ---- rounds of R tokens: wave w scores the WT tokens from begin + R r + WT w on, and brings in their V
  const int n_rounds = (end - begin + R - 1) / R;
  auto first_of = [&](int r) { return begin + R * r + WT * wave; };
  // The cache row that holds that token.  Paged cache: start + the token is a multiple of 16 and a page a multiple of 32
  // tokens, so the wave's tokens lie in one page.
  const int page_mask = paged ? (1 << p.page_shift) - 1 : 0;
  const int32_t* const tbl = paged ? p.block_table + (int64_t)b * p.max_blocks : nullptr;
  auto row_at = [&](int tok) -> int64_t {
    if (!paged) return row0 + tok;
    // (a scalar load: a vector load here would make the compiler wait for every load of the stream that is out)
    const int ta = start + tok;
    const uint32_t byte = (uint32_t)min(ta >> p.page_shift, p.max_blocks - 1) * 4;
    int page;
    asm volatile("s_load_dword %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&s"(page) : "s"(tbl), "s"(byte) : "memory");
    return ((int64_t)page * p.n_kv_heads + kv) * p.row_stride + (ta & page_mask);
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const uint32_t k_lds = lds0 + wave * (C::NK * C::K_SLOT);
  // K codes of 1 KB: SG = 1: 16 tokens of 64 B, pieces permuted by token / 4; SG = 2: 8 tokens of 128 B, by token / 2
  auto k_codes_at = [&](int ln, int tok) {
    return tok * TB + (C::SG == 1 ? (ln & 3) ^ ((tok >> 2) & 3) : (ln & 7) ^ ((tok >> 1) & 7)) * 16;
  };
  constexpr int KT1 = C::SG == 1 ? 16 : 8;        // tokens of a load
  const uint32_t k_off = k_codes_at(lane, C::SG == 1 ? lane >> 2 : lane >> 3);
  const uint32_t ks_off = ((lane >> 1) & (WT - 1)) * SZB + (C::SG == 2 ? lane >> 5 : 0) * 8 + (lane & 1) * 4;   // K scales: (slice, token, dword)
  const uint32_t v_off = lane / NG * TB + C::place(lane / NG, lane % NG) * 16;   // V codes of the first 1 KB (place(t + t', g) = place(t, g) ^ place(t', 0))
  const uint32_t m_off = lane % WT * SZB + lane / WT * 4;        // V scales: token lane % WT, pair of groups lane / WT
  // K slot s of the wave's tokens (cache rows `row` on, the last valid one `last`; later ones are clamped to it): KOPS loads
  auto issue_k = [&](int slot, int s, int64_t row, int last) {
    const uint32_t l = k_lds + slot * C::K_SLOT;
    const char* const kc = reinterpret_cast<const char*>(p.k_codes) + row * TB + s * (C::SG * 64);
    const char* const sc = reinterpret_cast<const char*>(p.k_scale) + row * SZB + s * (C::SG * 8);
    const char* const zc = reinterpret_cast<const char*>(p.k_zero) + row * SZB + s * (C::SG * 8);
    if (last >= WT - 1) {
      dma16<NT>(kc, k_off, l);
      dma16<NT>(kc + KT1 * TB, C::SG == 1 ? k_off : k_off ^ 64, l + 1024);
      dma4<NT>(sc, ks_off, l + C::K_SC);
      dma4<NT>(zc, ks_off, l + C::K_SC + 256);
    } else {
      int ln = lane;
      asm volatile("" : "+v"(ln));                // (worked out where it is needed: not kept in registers throughout the loop)
      const int t0 = C::SG == 1 ? ln >> 2 : ln >> 3;
#pragma unroll
      for (int u = 0; u < 2; ++u)
        dma16<false>(kc, k_codes_at(ln, t0 + u * KT1) + (min(t0 + u * KT1, last) - (t0 + u * KT1)) * TB, l + u * 1024);
      const int t = (ln >> 1) & (WT - 1);
      const uint32_t off = min(t, last) * SZB + (C::SG == 2 ? ln >> 5 : 0) * 8 + (ln & 1) * 4;
      dma4<false>(sc, off, l + C::K_SC);
      dma4<false>(zc, off, l + C::K_SC + 256);
    }
  };
  auto issue_v = [&](int r, int64_t row, int last) {            // the wave's V block of round r: VOPS loads
    const uint32_t l = lds0 + C::OFF_V + ((r & 1) * NW + wave) * C::V_BLK;
    const char* const vc = reinterpret_cast<const char*>(p.v_codes) + row * TB;
    const char* const sc = reinterpret_cast<const char*>(p.v_scale) + row * SZB;
    const char* const zc = reinterpret_cast<const char*>(p.v_zero) + row * SZB;
    if (last >= WT - 1) {
#pragma unroll
      for (int u = 0; u < C::VC; ++u) dma16<NT>(vc + u * 1024, v_off ^ (C::place(u * (64 / NG), 0) * 16), l + u * 1024);
#pragma unroll
      for (int u = 0; u < C::VM; ++u) {           // pairs of groups u * (64 / WT) ..: 64 / WT of them, WT tokens each
        dma4<NT>(sc + u * (64 / WT) * 4, m_off, l + C::V_SC + u * 256);
        dma4<NT>(zc + u * (64 / WT) * 4, m_off, l + C::V_Z + u * 256);
      }
    } else {
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll
      for (int u = 0; u < C::VC; ++u) {
        const int tok = (u * 64 + ln) / NG;
        dma16<false>(vc, min(tok, last) * TB + C::place(tok, ln % NG) * 16, l + u * 1024);
      }
      const uint32_t off = min(ln % WT, last) * SZB + ln / WT * 4;
#pragma unroll
      for (int u = 0; u < C::VM; ++u) {
        dma4<false>(sc + u * (64 / WT) * 4, off, l + C::V_SC + u * 256);
        dma4<false>(zc + u * (64 / WT) * 4, off, l + C::V_Z + u * 256);
      }
    }
  };

  // ---- prologue: the query rows (a part of them by each wave, into the second round's V area: 16-byte pieces permuted by the
  //      row's number, so that the 16 rows read at once lie on different banks), then the first round
  {
    constexpr int PIECES = D / 8;
#pragma unroll
    for (int u = 0; u < C::QOPS; ++u) {
      if (C::QW < NW && wave >= C::QW) break;
      const int idx = u * 64 + lane, r = wave * C::RPW + idx / PIECES;
      int t_q;
      const int64_t qr = row_of(min(tile * C::ROWS + r, rows_total - 1), t_q);
      dma16_lane(p.q + qr * D + ((idx % PIECES) ^ (r & 15)) * 8, lds0 + C::OFF_V + NW * C::V_BLK + (wave * C::QOPS + u) * 1024);
    }
  }
  // A decode step (p.k_new set; common length): the sequence's last NQ tokens are not in the cache yet.  The blocks whose
  // chunk holds one quantise it, a token a wave, and put it where the loads of the round they lie in have left what
  // the cache holds there; the first row tile's block stores them.
  const int new_first = seq - NQ;
  const bool new_block = p.k_new != nullptr && end > new_first;
  const bool new_mine = new_block && wave < NQ && new_first + wave >= begin && new_first + wave < end;
  const uint32_t new_raw = lds0 + C::OFF_V + NW * C::V_BLK + C::ROWS * D * 2 + wave * (C::NOPS * 1024);
  if (new_mine) {
    const int64_t at = ((int64_t)(b * p.n_kv_heads + kv) * NQ + wave) * D;
    if constexpr (D == 512) {
      dma16_lane(p.k_new + at + lane * 8, new_raw);
      dma16_lane(p.v_new + at + lane * 8, new_raw + 1024);
    } else {
      const int l = lane & (D / 4 - 1);           // D / 8 lanes K, D / 8 lanes V (d = 128: and once more)
      dma16_lane((l < D / 8 ? p.k_new : p.v_new) + at + (l & (D / 8 - 1)) * 8, new_raw);
    }
  }
  const bool any = first_of(0) < end;             // (a wave may have no tokens at all)
  if (any) {
    const int64_t row = row_at(first_of(0));
    const int last = end - 1 - first_of(0);
#pragma unroll
    for (int s = 0; s < C::SP; ++s) issue_k(s, s, row, last);
    issue_v(0, row, last);
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- this lane's column of each row tile: which (query token, head) it is and which tokens it sees
  bool rvalid[RT];
  int lo_col[RT], end_col[RT];
  int lo_all = 0, end_all = end;                  // the tokens that every row of the tile sees
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int r = (tile * RT + rt) * 16 + c;
    rvalid[rt] = r < rows_total;
    const int t_q = NQ > 1 ? min(r, rows_total - 1) / GF : 0;
    // query token t attends NQ - 1 - t tokens fewer than the last one; under a window its own last `row_window`
    const int own_end = seq - (NQ - 1 - t_q);
    end_col[rt] = rvalid[rt] ? min(end, own_end) : begin;
    lo_col[rt] = (NQ > 1 && p.row_window > 0) ? max(0, start + own_end - p.row_window) - start : lead;
    lo_all = max(lo_all, rvalid[rt] ? lo_col[rt] : 0);
    end_all = min(end_all, rvalid[rt] ? end_col[rt] : end);
  }
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    lo_all = max(lo_all, __shfl_xor(lo_all, off));
    end_all = min(end_all, __shfl_xor(end_all, off));
  }
  lo_all = __builtin_amdgcn_readfirstlane(lo_all);
  end_all = __builtin_amdgcn_readfirstlane(end_all);

  // ---- query operands: B of S^T = K Q^T, MFMA of group g: this lane's k-slots = its dims 8kq .. 8kq+7, in the slot order of
  //      unpack_word; the nibbles at bit 4 carry c 2^-20, so their entries are pre-divided by 16.  attn_scale may have any
  //      sign: the sign goes into the query, its size into the exponent.  Every wave turns the rows it has brought in into
  //      operands, in place, and works out 2^-24 sum of q over each group.
  if (any) wait_loads<C::SP * KOPS + VOPS>();
  else wait_loads<0>();
  {
    const float sign = p.scale_log2 > 0.0f ? 1.0f : p.scale_log2 < 0.0f ? -1.0f : 0.0f;
    constexpr int PIECES = D / 8;
#pragma unroll
    for (int u = 0; u < C::QOPS; ++u) {
      if (C::QW < NW && wave >= C::QW) break;
      const int idx = u * 64 + lane, r = wave * C::RPW + idx / PIECES;
      const uint32_t at = lds0 + C::OFF_V + NW * C::V_BLK + (wave * C::QOPS + u) * 1024 + lane * 16;
      const half8v x = lds_get<half8v>(at);
      const half_t one = (half_t)(tile * C::ROWS + r < rows_total ? sign : 0.0f), sixteenth = one * (half_t)0.0625f;
      lds_put(at, half8v{x[0] * one, x[4] * one, x[1] * sixteenth, x[5] * sixteenth,
                         x[2] * one, x[6] * one, x[3] * sixteenth, x[7] * sixteenth});
      float sum = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += (float)x[e];
      sum += __shfl_xor(sum, 1);                  // the four pieces of a group lie in four neighbouring lanes, in some order
      sum += __shfl_xor(sum, 2);
      const int g = ((idx % PIECES) ^ (r & 15)) >> 2;
      if ((lane & 3) == 0) lds_put(lds0 + C::OFF_Q + (r * NG + g) * 4, sum * (0x1p-24f * (float)one));
    }
  }
  if (new_mine) {
#pragma unroll
    for (int u = 0; u < C::NOPS; ++u) {
      const int piece = lane & (D / 8 - 1);
      const bool is_v = D == 512 ? u == 1 : (lane & (D / 8)) != 0;
      const half8v x16 = lds_get<half8v>(new_raw + u * 1024 + lane * 16);
      float x[8];
      half_t xh[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) { xh[e] = x16[e]; x[e] = (float)x16[e]; }
      float mn = x[0], mx = x[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) { mn = fminf(mn, x[e]); mx = fmaxf(mx, x[e]); }
#pragma unroll
      for (int o = 1; o < 4; o <<= 1) {           // over the four lanes of the group (exact in any order)
        mn = fminf(mn, __shfl_xor(mn, o));
        mx = fmaxf(mx, __shfl_xor(mx, o));
      }
      half_t s16, z16;
      quantize_scale_zero(mn, mx, s16, z16);
      const float sf = (float)s16, zf = (float)z16;
      const QuantFast fast = quantize_fast_setup(sf, zf, fmaxf(fabsf(mn), fabsf(mx)));
      float far = 0.0f;
      uint32_t word = quantize_word_fast(xh, fast, far);
      if (quantize_fast_in_doubt(far, fast)) word = quantize_word(x, sf, zf);
      const half2v sz = {s16, z16};
      const uint32_t to = lds0 + C::OFF_N + (wave * 2 + (is_v ? 1 : 0)) * C::N_ROW;
      lds_put(to + piece * 4, word);
      if ((piece & 3) == 0) lds_put(to + TB + piece, __builtin_bit_cast(uint32_t, sz));
      if (tile == 0 && (D == 512 || lane < D / 4)) {
        const int64_t row = row_at(new_first + wave);
        reinterpret_cast<uint32_t*>(const_cast<uint8_t*>(is_v ? p.v_codes : p.k_codes) + row * TB)[piece] = word;
        if ((piece & 3) == 0) const_cast<half_t*>(is_v ? p.v_scale : p.k_scale)[row * NG + piece / 4] = s16;
        if ((piece & 3) == 1) const_cast<half_t*>(is_v ? p.v_zero : p.k_zero)[row * NG + piece / 4] = z16;
      }
    }
  }
  block_barrier();
  half8v qb[RT][NG];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int g = 0; g < NG; ++g)
      qb[rt][g] = lds_get<half8v>(lds0 + C::OFF_V + NW * C::V_BLK + (rt * 16 + c) * (D * 2) + ((4 * g + kq) ^ c) * 16);
  const float kappa = (p.scale_log2 == 0.0f ? 1.0f : fabsf(p.scale_log2)) * 0x1p24f;   // raw accumulator units -> log2 units
  const float slack = kSlack / kappa;

  // ---- running state (Alg. 1, the initialisation), per column (query row)
  float m_all[RT], m_run[RT], l_run[RT];          // references of exp2 (raw units): the sums', this wave's weights'; this lane's share of the sum
  // sv_lim: the largest size a scale of this wave's groups may have as it stands.  From 2 on its sums carry 2^lower, lower < 0, so that
  // p s_v stays below 2^15 (its two groups together).  A wave looks at its scales once per round, with the references: one branch for both;
  // scales below 2 cost it nothing more.
  uint32_t sv_lim = kPlainScales;
  auto lower_of = [](uint32_t lim) { return (float)(int)(kPlainScales >> 26) - (float)(int)(lim >> 26); };
  float4v oacc[RT][GPW][2], zacc[RT][GPW];        // rows 4kq+i; [0]: sum w c - 15 sum_t1 w of the even dim, [1]: of even + 16 odd; zero-points
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_all[rt] = m_run[rt] = kNegBig;
    l_run[rt] = 0.0f;
#pragma unroll
    for (int m = 0; m < GPW; ++m) oacc[rt][m][0] = oacc[rt][m][1] = zacc[rt][m] = float4v{0, 0, 0, 0};
  }
  const half8v pos15_odd = as_half8(kPos15Odd, kPos15Odd, kPos15Odd, kPos15Odd);

  // ---- per-lane LDS byte offsets
  uint32_t k_rd[4];                               // word kq of piece m of token c (of a slot's second slice: ^ 64)
#pragma unroll
  for (int m = 0; m < 4; ++m) k_rd[m] = k_lds + (C::SG == 1 ? c * 64 + (m ^ (c >> 2)) * 16 + 4 * kq : c * 128 + (m ^ (c >> 1)) * 16 + 4 * kq);
  uint32_t q_rd = lds0 + C::OFF_Q + c * NG * 4;
  uint32_t ks_rd = k_lds + C::K_SC + 4 * kq * 8;
  const int g0 = wave % (NW / TH) * GPW;          // this wave's first group of V
  // word c % 4 of the group at place x of token 4 kq + i (place(4 kq + i, g) = place(4 kq, g) ^ place(i, 0))
  constexpr int NX = D == 512 ? 4 : 2;
  uint32_t v_rd[NX];
#pragma unroll
  for (int x = 0; x < NX; ++x) v_rd[x] = lds0 + C::OFF_V + 4 * kq * TB + (C::place(4 * kq, g0) ^ x) * 16 + 4 * (c & 3);
  uint32_t vs_rd = lds0 + C::OFF_V + C::V_SC + (g0 / 2 * WT + 4 * kq) * 4;
  uint32_t sv_rd = lds0 + C::OFF_V + C::V_SC + g0 / 2 * (WT * 4) + lane / WT * (TH * C::V_BLK) + lane % WT * 4;   // lane: a token of the wave's supertiles
  const uint32_t v_sel = 0x0C000C00u | ((4u + (c >> 2)) << 16) | (uint32_t)(c >> 2);   // this column's byte of a word
  const uint32_t z_sel = (c & 1) ? 0x07060302u : 0x05040100u;    // the zero-point operand's column c: group c % 2 of the pair

  struct KCodes { uint32_t w[TT][4]; };
  struct KScales { uint4v s[TT][2], z[TT][2]; };
  struct VCodes { uint32_t w[GPW][8]; };
  struct VScales { uint4v s[2], z[2]; float4v p[RT][2]; };
  auto load_kw = [&](int slot, int h, KCodes& k) {   // slice h of the slot
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int m = 0; m < 4; ++m) k.w[t][m] = lds_get<uint32_t>((h ? k_rd[m] ^ 64 : k_rd[m]) + slot * C::K_SLOT + t * 1024);
  };
  auto load_ks = [&](int slot, int h, KScales& k) {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t at = ks_rd + slot * C::K_SLOT + h * (WT * 8) + t * 128 + u * 16;
        k.s[t][u] = lds_get<uint4v>(at);
        k.z[t][u] = lds_get<uint4v>(at + 256);
      }
  };
  struct VBase { uint32_t w[NX], sz, p; };       // a round's: the addresses above in that round's V area, and its weights of this lane
  auto load_vw = [&](const VBase& at, int st, VCodes& v) {  // supertile st
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < GPW; ++m)
          v.w[m][4 * t + i] = lds_get<uint32_t>(at.w[C::place(i, 0) ^ m] + (2 * st + t) / TT * C::V_BLK + ((2 * st + t) % TT * 16 + i) * TB);
  };
  auto load_vs = [&](const VBase& at, int st, VScales& v) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint32_t off = (2 * st + t) / TT * C::V_BLK + (2 * st + t) % TT * 64;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) v.p[rt][t] = lds_get<float4v>(at.p + ((2 * st + t) * RT + rt) * 1024);
      v.s[t] = lds_get<uint4v>(at.sz + off);
      v.z[t] = lds_get<uint4v>(at.sz + WT * SZB + off);
    }
  };

  for (int r = 0; r < n_rounds; ++r) {
    // (the LDS addresses made from these are worked out where they are needed: not kept in registers throughout the loop)
    asm volatile("" : "+v"(k_rd[0]), "+v"(k_rd[1]), "+v"(k_rd[2]), "+v"(k_rd[3]), "+v"(ks_rd), "+v"(q_rd), "+v"(sv_rd));
    const int tok0 = first_of(r);
    const bool mine = tok0 < end, more = first_of(r + 1) < end;  // (wave-uniform)
    float sc[RT][TT][4];                          // then the weights
    int64_t row_n = 0;
    int last_n = 0;
    if (more) {
      row_n = row_at(first_of(r + 1));
      last_n = end - 1 - first_of(r + 1);
    }
    const uint32_t pb = lds0 + C::OFF_P + (r & 1) * C::P_BLK;
    if (mine) {
      // -- scores (Alg. 1) of this wave's tokens over all head dimensions, raw units: 2^-24.  A slice's slot is refilled with the
      //    next round's as soon as it sits in registers, so the waits below always leave the same loads out.
      constexpr int OUT = (C::SP - 1) * KOPS + VOPS, SG = C::SG;
      const int slot0 = C::SP > 1 ? 0 : (r & 1);
      if (new_block && tok0 + WT > new_first) {   // (the chunk's last round: nothing else is on its way)
        wait_loads<0>();
        const int t0 = max(0, new_first - tok0), n = min(WT, end - tok0) - t0;
        const uint32_t vb = lds0 + C::OFF_V + ((r & 1) * NW + wave) * C::V_BLK;
        for (int i = lane; i < WT * NG; i += 64)  // (what else lies there must not meet the zero weights of later tokens as Inf or NaN)
          if (i % WT >= t0) lds_put(vb + C::V_SC + i * 4, 0u);
        asm volatile("" ::: "memory");            // (16-bit stores to the same places follow: not to be moved across these by their type)
        constexpr int W = D / 8;                  // words of a row, four to a group
        for (int i = lane; i < n * 2 * W; i += 64) {
          const int row = i / W, w = i % W, g = w >> 2, t = t0 + (row >> 1);
          const uint32_t from = lds0 + C::OFF_N + ((tok0 + t - new_first) * 2 + (row & 1)) * C::N_ROW;
          const uint32_t word = lds_get<uint32_t>(from + w * 4), sz = lds_get<uint32_t>(from + TB + g * 4);
          if (row & 1) {
            lds_put(vb + t * TB + C::place(t, g) * 16 + (w & 3) * 4, word);
            if ((w & 3) == 0) {
              lds_put(vb + C::V_SC + (g >> 1) * (WT * 4) + t * 4 + (g & 1) * 2, (uint16_t)sz);
              lds_put(vb + C::V_Z + (g >> 1) * (WT * 4) + t * 4 + (g & 1) * 2, (uint16_t)(sz >> 16));
            }
          } else {
            const int gs = g % (4 * SG), h = gs >> 2;            // group of the slot, slice of the slot
            const uint32_t kb = k_lds + (slot0 + g / (4 * SG)) * C::K_SLOT;
            lds_put(kb + t * (SG * 64) + (SG == 1 ? gs ^ ((t >> 2) & 3) : gs ^ ((t >> 1) & 7)) * 16 + (w & 3) * 4, word);
            if ((w & 3) == 0) {
              lds_put(kb + C::K_SC + h * (WT * 8) + t * 8 + (gs & 3) * 2, (uint16_t)sz);
              lds_put(kb + C::K_SC + 256 + h * (WT * 8) + t * 8 + (gs & 3) * 2, (uint16_t)(sz >> 16));
            }
          }
        }
      }
      KCodes kw;
      wait_loads<OUT>();
      load_kw(slot0, 0, kw);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[rt][t][i] = 0.0f;
      auto slice = [&](auto s_tag) {
        constexpr int s = decltype(s_tag)::value;
        KScales ks;
        float4v qs[RT], acc[RT][TT][4];
        load_ks(C::SP > 1 ? s / SG : slot0, s % SG, ks);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) qs[rt] = lds_get<float4v>(q_rd + rt * 16 * NG * 4 + s * 16);
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const half8v a = unpack_word(kw.w[t][m]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt][t][m] = mfma16(a, qb[rt][4 * s + m], float4v{0, 0, 0, 0});
          }
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr ((s + 1) % SG == 0) {        // the slot is in registers
          if (more) {
            issue_k(C::SP > 1 ? s / SG : slot0 ^ 1, s / SG, row_n, last_n);
            if constexpr (s + 1 < SL) wait_loads<OUT>();
          } else if constexpr (s + 1 < SL) {
            wait_loads<(C::SP - 1 - (s + 1) / SG) * KOPS + VOPS>();
          }
        }
        if constexpr (s + 1 < SL) load_kw((s + 1) / SG, (s + 1) % SG, kw);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
          for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t sw = ks.s[t][i >> 1][(i & 1) * 2 + (m >> 1)], zw = ks.z[t][i >> 1][(i & 1) * 2 + (m >> 1)];
#pragma unroll
              for (int rt = 0; rt < RT; ++rt)
                sc[rt][t][i] = __builtin_fmaf(half_of(sw, m & 1), __builtin_fmaf(-half_of(zw, m & 1), qs[rt][m], acc[rt][t][m][i]),
                                              sc[rt][t][i]);
            }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)           // (here, not where the scores are read: that keeps every slice's operands alive)
#pragma unroll
          for (int t = 0; t < TT; ++t) asm volatile("" : "+v"(sc[rt][t][0]), "+v"(sc[rt][t][1]), "+v"(sc[rt][t][2]), "+v"(sc[rt][t][3]));
      };
      slice(std::integral_constant<int, 0>{});
      if constexpr (SL > 1) slice(std::integral_constant<int, 1>{});
      if constexpr (SL > 2) slice(std::integral_constant<int, 2>{});
      if constexpr (SL > 3) slice(std::integral_constant<int, 3>{});
      if (tok0 < lo_all || tok0 + WT > end_all) { // (wave-uniform: the tokens that not every row sees)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int tok = tok0 + 16 * t + 4 * kq + i;
              sc[rt][t][i] = (tok >= lo_col[rt] && tok < end_col[rt]) ? sc[rt][t][i] : -INFINITY;
            }
      }
      // -- online softmax (Alg. 1: the maximum, the weights and the running sum).  m_run is a REFERENCE per row: it moves when
      //    a score exceeds it by more than kSlack (log2 units), and then to kSlack above the new maximum, so that exp2(score -
      //    m_run) <= 4.  Any reference gives the same o / l, and the chunk merge (Eq. 6) accepts any m_c.
      float mx[RT];
      bool move = false;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        mx[rt] = fmaxf(fmaxf(sc[rt][0][0], sc[rt][0][1]), fmaxf(sc[rt][0][2], sc[rt][0][3]));
        if constexpr (TT == 2) mx[rt] = fmaxf(mx[rt], fmaxf(fmaxf(sc[rt][1][0], sc[rt][1][1]), fmaxf(sc[rt][1][2], sc[rt][1][3])));
        move = move || mx[rt] > m_run[rt] + slack;
      }
      if (__builtin_amdgcn_ballot_w64(move) != 0) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const float m_new = fmaxf(m_run[rt], blocks_max(mx[rt]) + slack);
          l_run[rt] *= __builtin_amdgcn_exp2f((m_run[rt] - m_new) * kappa);
          m_run[rt] = m_new;
        }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float mk = fmaxf(__builtin_fmaf(m_run[rt], kappa, -kLift), -3.0e38f);    // (finite also for a column that has seen no token yet)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          float4v pr;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            pr[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[rt][t][i], kappa, -mk));
            l_run[rt] += pr[i];
          }
          lds_put(pb + (((wave * TT + t) * RT + rt) * 64 + lane) * 16, pr);
        }
      }
    } else {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < TT; ++t)
          lds_put(pb + (((wave * TT + t) * RT + rt) * 64 + lane) * 16, float4v{0, 0, 0, 0});
      // (its half of a supertile may be attended all the same: what lies there must not meet the zero weights as Inf or NaN)
      if constexpr (TT == 1) {
        static_assert(TT != 1 || 2 * WT * SZB == 1024, "16 bytes a lane");
        lds_put(lds0 + C::OFF_V + ((r & 1) * NW + wave) * C::V_BLK + C::V_SC + lane * 16, uint4v{0, 0, 0, 0});
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      if (kq == 0) lds_put(pb + C::P_M + ((rt * 16 + c) * NW + wave) * 4, m_run[rt]);
    if (more) wait_loads<C::SP * KOPS>();            // this wave's part of the round's V has landed
    else wait_loads<0>();
    // The round's one barrier: behind it everybody's weights and V are there, and everybody is done with the round before,
    // whose V area is filled again (and whose weights the next round overwrites).
    block_barrier();
    if (more) issue_v(r + 1, row_n, last_n);
    constexpr int STEPS = R / 32 / TH;
    const int st0 = wave / (NW / TH);             // (this wave's supertiles: st0, st0 + TH, ..)
    const uint32_t sv_at = sv_rd + (r & 1) * (NW * C::V_BLK) + st0 * (2 / TT * C::V_BLK);
    // -- everybody's references.  They differ from the sums' only where a row's maximum has moved: then the sums are
    //    rescaled (Alg. 1, the correction factor) and the weights brought to the common reference as they are read.
    uint32_t sv[STEPS / 2];                       // the scales of this wave's groups, 64 tokens a word
#pragma unroll
    for (int u = 0; u < STEPS / 2; ++u) sv[u] = lds_get<uint32_t>(sv_at + u * (64 / WT * TH * C::V_BLK));
    bool differ = false;
    float top[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float4v a = lds_get<float4v>(pb + C::P_M + (rt * 16 + c) * NW * 4);
      const float4v d = lds_get<float4v>(pb + C::P_M + (rt * 16 + c) * NW * 4 + 16);
      const float hi = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(d[0], d[1]), fmaxf(d[2], d[3])));
      top[rt] = fmaxf(m_all[rt], hi);
      const float lo = fminf(fminf(fminf(a[0], a[1]), fminf(a[2], a[3])), fminf(fminf(d[0], d[1]), fminf(d[2], d[3])));
      differ = differ || lo != m_all[rt] || hi != m_all[rt];
    }
    const ushort2v lim = __builtin_bit_cast(ushort2v, sv_lim);   // (fp16 bits are ordered by size)
    const uint32_t sv_a = sv[0], sv_b = sv[STEPS / 2 - 1];
    const ushort2v big = __builtin_elementwise_max(__builtin_bit_cast(ushort2v, sv_a), __builtin_bit_cast(ushort2v, sv_b));
    const bool exceed = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(big, lim)) != sv_lim;
    const bool rescale = __builtin_amdgcn_ballot_w64(differ || exceed) != 0;
    if (rescale) {
      if (__builtin_amdgcn_ballot_w64(exceed) != 0) {
        uint32_t most = 0;                        // (a negative scale comes here every time: its size counts; behind the chunk's end lies anything)
#pragma unroll
        for (int u = 0; u < STEPS / 2; ++u) {
          const int st = st0 + TH * (2 * u + (lane >> 5));
          if (32 * st + (lane & 31) < end - begin - R * r) most = max(most, max(sv[u] & 0x7FFFu, (sv[u] >> 16) & 0x7FFFu));
        }
        const uint32_t e = min(wave_max((int)most) >> 10, 30);
        if (e > sv_lim >> 26) {
          const float f = __builtin_amdgcn_exp2f(lower_of(scale_limit(e)) - lower_of(sv_lim));
          sv_lim = scale_limit(e);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int m = 0; m < GPW; ++m) {
              oacc[rt][m][0] *= f;
              oacc[rt][m][1] *= f;
              zacc[rt][m] *= f;
            }
        }
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float f = __builtin_amdgcn_exp2f((m_all[rt] - top[rt]) * kappa);
        l_run[rt] *= __builtin_amdgcn_exp2f((m_run[rt] - top[rt]) * kappa);
        m_all[rt] = m_run[rt] = top[rt];
#pragma unroll
        for (int i = 0; i < 4; ++i) {                            // accumulator row 4kq+i is the column of lane 4kq+i
          const float fr = __shfl(f, 4 * kq + i);
#pragma unroll
          for (int m = 0; m < GPW; ++m) {
            oacc[rt][m][0][i] *= fr;
            oacc[rt][m][1][i] *= fr;
            zacc[rt][m][i] *= fr;
          }
        }
      }
    }
    // -- P V (Alg. 1, the accumulator update): this wave's groups of V, all the round's tokens
    const int n_st = min(R / 32, (end - begin - R * r + 31) >> 5);
    VBase at;
    {
      const uint32_t blk = (r & 1) * (NW * C::V_BLK) + st0 * (2 / TT * C::V_BLK);
#pragma unroll
      for (int x = 0; x < NX; ++x) {
        at.w[x] = v_rd[x] + blk;
        asm volatile("" : "+v"(at.w[x]));         // (the rest of an address is a constant, in the instruction)
      }
      at.sz = vs_rd + blk;
      at.p = pb + st0 * (2 * RT * 1024) + lane * 16;
      asm volatile("" : "+v"(at.sz), "+v"(at.p));
    }
    VCodes vw;
    load_vw(at, 0, vw);
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
      if (st0 + k * TH >= n_st) break;
      VScales v;
      load_vs(at, k * TH, v);
      half8v v_mixed[GPW], v_even[GPW];
#pragma unroll
      for (int m = 0; m < GPW; ++m) {
        uint32_t mix[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mix[i] = __builtin_amdgcn_perm(~vw.w[m][i + 4], vw.w[m][i], v_sel);
        v_mixed[m] = as_half8(mix[0], mix[1], mix[2], mix[3]);
        v_even[m] = as_half8(mix[0] & kMaskLo, mix[1] & kMaskLo, mix[2] & kMaskLo, mix[3] & kMaskLo);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (k + 1 < STEPS) load_vw(at, (k + 1) * TH, vw);
      if (rescale || sv_lim != kPlainScales) {
        const float lower = lower_of(sv_lim);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const float mw = lds_get<float>(pb + C::P_M + ((rt * 16 + c) * NW + (2 * (st0 + k * TH) + t) / TT) * 4);
            const float f = __builtin_amdgcn_exp2f(__builtin_fmaf(mw - m_all[rt], kappa, lower));
#pragma unroll
            for (int i = 0; i < 4; ++i) v.p[rt][t][i] *= f;
          }
      }
      uint32_t zw[4];                             // k-slots 2i, 2i+1: tokens 4kq+i of tile 0 and of tile 1
#pragma unroll
      for (int i = 0; i < 4; ++i) zw[i] = __builtin_amdgcn_perm(v.z[1][i], v.z[0][i], z_sel) ^ 0x80000000u;
      const half8v zb = as_half8(zw[0], zw[1], zw[2], zw[3]);
      const half8v zb15 = zb + pos15_odd;         // (one operand is enough for the rest, 2^-11 of the whole)
#pragma unroll
      for (int m = 0; m < GPW; ++m)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          half8v pa, rest;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (C::SPLIT) {             // (both rounded towards zero: what the first leaves out the second takes, down to 2^-24)
              const float w0 = v.p[rt][0][i] * half_of(v.s[0][i], m), w1 = -v.p[rt][1][i] * half_of(v.s[1][i], m);
              const auto hi = __builtin_amdgcn_cvt_pkrtz(w0, w1);
              const auto lo = __builtin_amdgcn_cvt_pkrtz(__builtin_fmaf((float)hi[0], -1.0f, w0), __builtin_fmaf((float)hi[1], -1.0f, w1));
              pa[2 * i] = hi[0]; pa[2 * i + 1] = hi[1];
              rest[2 * i] = lo[0]; rest[2 * i + 1] = lo[1];
            } else {
              pa[2 * i] = (half_t)__builtin_fmaf(v.p[rt][0][i], half_of(v.s[0][i], m), 0.0f);
              pa[2 * i + 1] = (half_t)__builtin_fmaf(-v.p[rt][1][i], half_of(v.s[1][i], m), 0.0f);
            }
          }
          oacc[rt][m][0] = mfma16(pa, v_even[m], oacc[rt][m][0]);
          oacc[rt][m][1] = mfma16(pa, v_mixed[m], oacc[rt][m][1]);
          zacc[rt][m] = mfma16(pa, zb, zacc[rt][m]);
          zacc[rt][m] = mfma16(pa, pos15_odd, zacc[rt][m]);
          if constexpr (C::SPLIT) {
            oacc[rt][m][0] = mfma16(rest, v_even[m], oacc[rt][m][0]);
            oacc[rt][m][1] = mfma16(rest, v_mixed[m], oacc[rt][m][1]);
            zacc[rt][m] = mfma16(rest, zb15, zacc[rt][m]);
          }
        }
    }
  }

  // ---- the chunk's partial (o_c, m_c, l_c) per query row (Sec. 3.2), un-normalised, in final units: even sums carry 2^-24,
  //      (mixed - even) / 16 the odd dim
  block_barrier();                                // everybody is done with the weights
  float* const lds_l = reinterpret_cast<float*>(smem);          // [ROWS][NW]
  float2* const lds_o = reinterpret_cast<float2*>(smem + C::ROWS * NW * 4);   // TH > 1: the later waves' sums, [wave][rt][i][m][lane]
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const float l = blocks_sum(l_run[rt]);
    if (kq == 0) lds_l[(rt * 16 + c) * NW + wave] = l;
  }
  float2 o2[RT][GPW][4];
  const float raise = __builtin_amdgcn_exp2f(-lower_of(sv_lim));
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int m = 0; m < GPW; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float zc = __shfl(zacc[rt][m][i], (lane & ~1) | m);
        const float even = oacc[rt][m][0][i], mixed = oacc[rt][m][1][i];
        o2[rt][m][i] = float2{__builtin_fmaf(even, 0x1p24f, -zc), __builtin_fmaf(mixed - even, 0x1p20f, -zc)};
        if (__builtin_expect(sv_lim != kPlainScales, 0)) {
          o2[rt][m][i].x *= raise;
          o2[rt][m][i].y *= raise;
        }
        if constexpr (TH > 1) lds_o[(((wave * RT + rt) * 4 + i) * GPW + m) * 64 + lane] = o2[rt][m][i];
      }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < RT * 4 / TH; ++k) {         // the waves that share the groups take every TH-th row each
    const int ri = TH > 1 ? k * TH + wave / (NW / TH) : k, rt = ri >> 2, i = ri & 3;
    const int r = (tile * RT + rt) * 16 + 4 * kq + i;
    int t_q;
    const int64_t ph = row_of(min(r, rows_total - 1), t_q) * part_stride + split;
#pragma unroll
    for (int m = 0; m < GPW; ++m) {
      float2 o = {0.0f, 0.0f};
      if constexpr (TH == 1) {
        o = o2[k >> 2][m][k & 3];
      } else {
#pragma unroll
        for (int w = 0; w < TH; ++w) {
          const float2 x = lds_o[((((w * (NW / TH) + wave % (NW / TH)) * RT + rt) * 4 + i) * GPW + m) * 64 + lane];
          o.x += x.x;
          o.y += x.y;
        }
      }
      if (r < rows_total) st_dev2(p.part_o + ph * D + 32 * (g0 + m) + 8 * (c & 3) + 2 * (c >> 2), o.x, o.y);
    }
  }
  if (wave == 0 && kq == 0) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      if (!rvalid[rt]) continue;
      float l = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) l += lds_l[(rt * 16 + c) * NW + w];
      int t_q;
      const int64_t ph = row_of((tile * RT + rt) * 16 + c, t_q) * part_stride + split;
      const bool seen = m_all[rt] > kNegBig;      // (a row whose tokens were all masked counts as empty)
      st_dev2(p.part_ml + ph * 2, seen ? m_all[rt] * kappa - kLift : kNegBig, seen ? l : 0.0f);
    }
  }
}

template <int D, int RT, int TT, bool NT, bool PLAIN>
hipError_t launch_as(const DecodeParams& p, dim3 grid, hipStream_t s) {
  constexpr int smem = Tile<D, RT, TT>::SMEM;
  // dynamic LDS above 64 KB has to be opted into, once per device and kernel instance (any thread may get here first)
  static std::once_flag configured[kMaxDevices];
  static hipError_t outcome[kMaxDevices];
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::call_once(configured[dev], [&] {
    outcome[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(&decode_partial_wide_kernel<D, RT, TT, NT, PLAIN>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (outcome[dev] != hipSuccess) return outcome[dev];
  hipLaunchKernelGGL((decode_partial_wide_kernel<D, RT, TT, NT, PLAIN>), grid, dim3(512), smem, s, p);
  return hipGetLastError();
}
template <int D, int RT, int TT>
hipError_t launch(const DecodeParams& p, dim3 grid, hipStream_t s) {
  const bool plain = p.seq_lens == nullptr && p.block_table == nullptr;
  if (p.kv_share == 1) return plain ? launch_as<D, RT, TT, true, true>(p, grid, s) : launch_as<D, RT, TT, true, false>(p, grid, s);
  if constexpr (D == 128 && RT == 1) return hipErrorInvalidValue;   // (at most 16 rows: one tile per KV head)
  else return plain ? launch_as<D, RT, TT, false, true>(p, grid, s) : launch_as<D, RT, TT, false, false>(p, grid, s);
}

}  // namespace

int wide_row_tiles(int head_dim, int rows) { return head_dim == 128 ? (rows + 31) / 32 : (rows + 15) / 16; }

// Chunks of a sequence of `tiles` 32-token tiles, at most.  A block scores 128 tokens in a round (d = 256: 256); with fewer, and up
// to 64 of them, each still shortens the launch; beyond, the merge kernel pays for what the shorter chunks save (us per step at
// chunks of 32 / 64 / 128 tokens: 32 heads on one KV head, 1500 tokens 11.4 / 12.3 / 14.1; 4096 14.2 / 12.7 / 13.4; 8192
// 15.3 / 15.3 / 14.8; 16 heads on two, 700 tokens 10.4 / 11.1 / 14.2; 5000 12.0 (64) / 12.9 / 14.9).
int wide_max_chunks(int head_dim, int tiles) {
  const int m = head_dim < 512 ? (tiles <= 48 ? 2 : 4) : tiles <= 64 ? 1 : tiles < 224 ? 2 : 4;
  return (tiles + m - 1) / m;
}

hipError_t launch_partial_wide(const DecodeParams& p_in, int batch, int head_dim, hipStream_t s) {
  DecodeParams p = p_in;
  if (p.n_queries < 1) p.n_queries = 1;
  if ((head_dim != 512 && head_dim != 256 && head_dim != 128) || p.group != kGroup || p.gqa < 1 || p.kv_share < 1) return hipErrorInvalidValue;
  if (p.n_queries > kMaxQueries) return hipErrorInvalidValue;
  if (p.kv_share != wide_row_tiles(head_dim, p.n_queries * p.gqa)) return hipErrorInvalidValue;
  if (p.k_new && (p.seq_lens || p.block_table)) return hipErrorInvalidValue;
  if (p.block_table && (p.page_shift < 5 || !p.seq_lens)) return hipErrorInvalidValue;   // a supertile must not straddle pages
  const dim3 grid = p.var_chunks > 0 ? dim3(p.var_chunks, p.n_kv_heads * p.kv_share, 1)
                                     : dim3(p.n_splits, p.n_kv_heads * p.kv_share, batch);
  if (head_dim == 128) return p.n_queries * p.gqa <= 16 ? launch<128, 1, 2>(p, grid, s) : launch<128, 2, 2>(p, grid, s);
  return head_dim == 256 ? launch<256, 1, 2>(p, grid, s) : launch<512, 1, 1>(p, grid, s);
}

}  // namespace tq
