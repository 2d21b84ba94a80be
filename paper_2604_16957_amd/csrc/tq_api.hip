// C ABI of the library: host-side validation, chunk planning and kernel dispatch.
// Every argument check happens here, on the host, before any HIP call, so a rejected call
// launches nothing (and the checks themselves can be exercised on a machine without a GPU).
#include <algorithm>
#include <cmath>
#include <mutex>

#include "tq_internal.h"

namespace {

using tq::DecodeParams;
using tq::half_t;

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// head dimensions the kernels are built for
inline bool head_dim_ok(int d) { return d == 128 || d == 256 || d == 512; }

int check_cache(const tq_kv_cache* c) {
  if (!c) return TQ_ERR_NULL;
  if (!c->k_codes || !c->v_codes || !c->k_scale || !c->k_zero || !c->v_scale || !c->v_zero) return TQ_ERR_NULL;
  if (!head_dim_ok(c->head_dim)) return TQ_ERR_SHAPE;
  if (c->group_size != 32 && c->group_size != 64 && c->group_size != 128) return TQ_ERR_SHAPE;
  if (c->head_dim % c->group_size != 0) return TQ_ERR_SHAPE;
  if (c->batch < 1 || c->n_kv_heads < 1 || c->capacity < 1) return TQ_ERR_SHAPE;
  if (c->layout != TQ_LAYOUT_CANONICAL) return TQ_ERR_SHAPE;
  const void* ptrs[] = {c->k_codes, c->v_codes, c->k_scale, c->k_zero, c->v_scale, c->v_zero};
  for (const void* p : ptrs)
    if (!aligned(p, 16)) return TQ_ERR_ALIGN;
  return TQ_OK;
}

struct Plan { int n_splits, tokens_per_split; };

constexpr int kBlocksMfma = 256;   // matrix-core kernel: 8-wave blocks, one per compute unit
constexpr int kBlocksValu = 512;   // generic kernel: 4-wave blocks, two per compute unit
constexpr int kBlocksWide = 256;   // matrix-core kernel for wide rows: 8-wave blocks, one per compute unit

// A chunk is never longer than this many tokens under the heuristic, which bounds the rounding that the fp32 accumulators of one
// wave pick up however long the sequence is: at most 64 tiles in the matrix-core kernel; in the kernel for wide rows, whose waves take
// their dims of every tile, every second, every fourth (head_dim 512, 256, 128), 512, 256, 128 tiles.  Relative error against 64 bits of 16384
// tokens, planned / as one chunk: 2.90e-4 / 2.91e-4, 2.88e-4 / 2.91e-4, 2.06e-4 / 2.07e-4.  (Sequences with lengths of their own have no such bound: the
// device cuts them by the total, and a wave may hold a whole one.  5 sequences of 16000 .. 20000 tokens, 128 heads over 128, dealt to waves, some 210
// tiles each: 2.61e-4, by the chunk list 2.65e-4.)
constexpr int kMaxChunkTokens = 16384;

// Chunks of whole 32-token tiles, never an empty chunk.  The blocks of a launch run in rounds of
// `target_blocks` (what the chip holds at once): as many chunks as fill one round without spilling into a
// second (a 257th block would wait for a whole block's time), or, where that makes chunks longer than
// kMaxChunkTokens, as many as fill the fewest rounds that do not.  With `tiles_per_block_min` > 1 short
// sequences get fewer, fuller blocks (one tile per wave at least).
Plan plan_splits(int batch, int n_kv_heads, int seq_len, int requested, int target_blocks, int tiles_per_block_min) {
  const int tiles = (seq_len + tq::kTile - 1) / tq::kTile;
  int n = requested;
  if (n <= 0) {
    const int64_t rows = (int64_t)batch * n_kv_heads;
    const int64_t need = (seq_len + kMaxChunkTokens - 1) / kMaxChunkTokens;
    const int64_t rounds = std::max<int64_t>(1, (need * rows + target_blocks - 1) / target_blocks);
    n = (int)std::max<int64_t>({1, need, rounds * target_blocks / rows});
    n = std::min(n, std::max(1, tiles / tiles_per_block_min));
    n = (int)std::max<int64_t>(n, need);
  }
  n = std::max(1, std::min({n, tiles, tq::kMaxSplits}));
  const int tiles_per = (tiles + n - 1) / n;
  Plan p;
  p.tokens_per_split = tiles_per * tq::kTile;
  p.n_splits = (seq_len + p.tokens_per_split - 1) / p.tokens_per_split;
  return p;
}

// Chunks of a short sequence (1: as plan_splits has it) where up to eight rows share a block and the decode kernel merges the chunks
// in place.  A call that leaves compute units without a block is as long as its longest chain: with four tiles to a chunk or fewer a
// block has one wave to a SIMD, which is done about 0.7 us sooner than two that share it, and with two tiles the block merge has
// as good as no spread to wait for; against that a chunk more is 4 KB more for the waves that merge.  So two or three tiles
// to a chunk up to 16 chunks, then four and more up to 32; a sequence of up to eight tiles stays one chunk (no merge at all), and one of up to
// 15, which would be, is cut only where there are compute units for two tiles a chunk.  us per step, eight tiles and more to a chunk / this:
// 8 heads over 1, 300 tokens 6.3 / 6.05, 1024 7.7 / 6.3, 4096 8.0 / 7.5; 64 over 8, 600 tokens 8.0 / 6.5, 2048 8.0 / 7.0, 4096 8.4 / 7.9,
// 4 sequences of 600 8.1 / 6.7, 8 of 600 8.2 / 7.8; 32 over 32, 600 6.7 / 5.7; d = 256: 32 over 16, 300 8.1 / 6.6, 600 9.2 / 6.9, a window of 1024
// 8.6 / 7.0, 16 over 8, 3000 10.1 / 8.5.  (64 over 8, 200 tokens in four chunks 6.7, in one 6.4; 2048 tokens in 32 chunks 7.5, in 16 7.2;
// 16 sequences of 300 in two chunks each 8.0, in one 7.3.)
// `light`: at d = 128 the second tile of a wave costs less than the merge where a block has up to four rows or the launch is not a plain one
// (groups of 64 and 128, several query tokens): up to twelve tiles stay one chunk.  us per step | decode, one chunk / two tiles each:
// 32 heads over 8, 300 tokens 5.2 / 5.7 | 4.9 / 5.65, 384 5.7 / 5.7 | 5.1 / 5.6, 416 5.8 / 5.7 | 5.6 / 5.6, 480 6.0 / 5.6 | 5.8 / 5.6;
// 64 over 8, groups of 64, 288 7.9 / 8.0 | 7.6 / 8.0, 416 8.55 / 8.15 | 8.25 / 7.95; decode of 2 query tokens, 32 over 8, 384 8.0 / 8.15, 416 8.5 / 8.1.
int fine_splits(int batch, int n_kv_heads, int seq_len, int target_blocks, bool light) {
  const int tiles = (seq_len + tq::kTile - 1) / tq::kTile;
  const int64_t most = (int64_t)target_blocks / ((int64_t)batch * n_kv_heads);
  if (tiles <= (light ? 12 : 8)) return 1;
  for (int t = 2; t <= (tiles < 16 ? 2 : 8); ++t) {
    const int n = (tiles + t - 1) / t;
    if (n <= most && n <= (t < 4 ? 16 : 32)) return n;
  }
  return 1;
}

// query tokens per sequence the options ask for
int queries_of(const tq_decode_opts* opts) { return (opts && opts->n_queries > 1) ? opts->n_queries : 1; }
// query rows that share one KV head
int rows_of(const tq_kv_cache* c, int n_q_heads, const tq_decode_opts* opts) {
  return n_q_heads / c->n_kv_heads * queries_of(opts);
}
// fine_splits of a call over `tokens` tokens (up to eight rows to a block, rows_per_batch blocks to a chunk of every sequence)
int fine_splits_of(const tq_kv_cache* c, int n_q_heads, const tq_decode_opts* opts, int rows_per_batch, int tokens) {
  const bool light = c->head_dim == 128 && (rows_of(c, n_q_heads, opts) <= 4 || c->group_size != tq::kGroup || queries_of(opts) > 1);
  return fine_splits(c->batch, rows_per_batch, tokens, kBlocksMfma, light);
}

// `room`: tokens a sequence can hold (the cache's capacity, or max_blocks pages of a paged pool)
int check_decode(const tq_kv_cache* c, const void* q, int n_q_heads, int seq_len, const void* out,
                 const void* workspace, size_t workspace_bytes, const tq_decode_opts* opts, bool need_out,
                 int64_t room = -1) {
  int rc = check_cache(c);
  if (rc == TQ_ERR_NULL) return rc;
  if (!q || (need_out && !out) || !workspace) return TQ_ERR_NULL;
  if (rc != TQ_OK && rc != TQ_ERR_ALIGN) return rc;
  if (n_q_heads < 1 || n_q_heads % c->n_kv_heads != 0) return TQ_ERR_SHAPE;
  if (seq_len < queries_of(opts)) return TQ_ERR_EMPTY;   // (every query token is one of the sequence's tokens)
  if (seq_len > (room >= 0 ? room : (int64_t)c->capacity)) return TQ_ERR_CAPACITY;
  if (rc == TQ_ERR_ALIGN) return rc;
  if (!aligned(q, 16) || (need_out && !aligned(out, 16)) || !aligned(workspace, 256)) return TQ_ERR_ALIGN;
  if (opts) {
    if (opts->variant < 0 || opts->variant > 2 || opts->n_splits < 0 || opts->window < 0) return TQ_ERR_UNSUPPORTED;
    if (opts->n_queries < 0 || opts->n_queries > tq::kMaxQueries) return TQ_ERR_UNSUPPORTED;
    if (opts->n_queries > 1 && opts->variant == 1) return TQ_ERR_UNSUPPORTED;   // matrix-core kernels only
    if (opts->variant == 2 && c->head_dim != 512 &&
        !tq::mfma_supported(c->head_dim, rows_of(c, n_q_heads, opts)))
      return TQ_ERR_UNSUPPORTED;
  }
  if (workspace_bytes < tq_workspace_bytes(c->batch * queries_of(opts), n_q_heads, c->head_dim)) return TQ_ERR_WORKSPACE;
  return TQ_OK;
}

DecodeParams make_params(const tq_kv_cache* c, const void* q, int n_q_heads, int seq_len, float attn_scale,
                         void* out, void* workspace, const Plan& plan, int n_queries = 1) {
  DecodeParams p{};
  p.k_codes = static_cast<const uint8_t*>(c->k_codes);
  p.v_codes = static_cast<const uint8_t*>(c->v_codes);
  p.k_scale = static_cast<const half_t*>(c->k_scale);
  p.k_zero = static_cast<const half_t*>(c->k_zero);
  p.v_scale = static_cast<const half_t*>(c->v_scale);
  p.v_zero = static_cast<const half_t*>(c->v_zero);
  p.q = static_cast<const half_t*>(q);
  p.out = static_cast<half_t*>(out);
  p.part_o = static_cast<float*>(workspace);
  p.part_ml = p.part_o + tq::workspace_o_floats(c->batch * n_queries, n_q_heads, c->head_dim);
  p.plan = reinterpret_cast<int32_t*>(p.part_ml + tq::workspace_ml_floats(c->batch * n_queries, n_q_heads));
  p.n_q_heads = n_q_heads;
  p.n_queries = n_queries;
  p.n_kv_heads = c->n_kv_heads;
  p.gqa = n_q_heads / c->n_kv_heads;
  p.group = c->group_size;
  p.row_stride = c->capacity;
  p.seq_len = seq_len;
  p.n_splits = plan.n_splits;
  p.tokens_per_split = plan.tokens_per_split;
  p.scale_log2 = attn_scale * 1.4426950408889634f;
  // (below this every weight is 1 to the last bit of 32, |q.k| being under 2^43, and the kernels' slack in raw units, 2 / scale, would
  // pass their mark of a row that has seen no token)
  if (p.scale_log2 != 0.0f && std::fabs(p.scale_log2) < 1.0e-30f) p.scale_log2 = std::copysign(1.0e-30f, p.scale_log2);
  return p;
}

int hip_rc(hipError_t e) { return e == hipSuccess ? TQ_OK : TQ_ERR_HIP; }

// Which kernel a decode call takes, and whether that kernel can also do the chunk merge.
// merge, merge_step: whether a decode, a decode step's launch also does the chunk merge (or has none to do: one chunk).
// wide: the matrix-core kernel for many query rows (head_dim 512; 256 and 128 by wide_rows); small_tile: at most eight query rows to a block.
struct Route { bool ok, use_mfma, merge, merge_step, wide, small_tile; };
// The in-kernel merge ends the kernel with a chain of device-wide round trips (publish the partial, count in, read
// the row's partials) that one wave per row walks: about 1.3 us for 4 chunks and 2.5 us for 32, against about 3.3 us for the
// separate merge kernel plus its launch; with 64 and 128 chunks to a row that one compute unit pulls in for too long
// (one KV head, 8 heads, us per step, in place / merge kernel: 14K tokens, 55 chunks, 9.4 / 9.0; 16K,
// 64 chunks, 9.7 / 9.1).  A decode step merges in place wherever that holds (128K tokens, 64 heads over 8, 33.3 -> 32.6 us;
// 8 sequences of 8K 21.9 -> 20.6; 32 heads over 32, 32K, 31.4 -> 29.9); the decode alone up to this many packed bytes per
// call.  Above, and at head_dim 256 with larger groups, it keeps two launches, although one would be the faster there too
// (32 heads over 16, d = 256, 32K tokens: the step's one launch 33.0 us, the decode's two 33.9): callers that ask tq_decode_launches, and the
// benchmark, which times phase 1 by itself, go by them.
constexpr int64_t kMergeInKernelMaxBytes = 48ll << 20;
constexpr int kMergeInKernelMaxChunks = 32;

// tokens a sequence of length seq_len attends under the options' sliding window
// (several query tokens: the span all rows together attend, the earliest row's window start to the end)
int windowed(int seq_len, const tq_decode_opts* opts) {
  return (opts && opts->window > 0) ? std::min(seq_len, opts->window + queries_of(opts) - 1) : seq_len;
}
// blocks of the matrix-core kernel that stream one KV head
int mfma_share_of(const tq_kv_cache* cache, int n_q_heads, const tq_decode_opts* opts) {
  return tq::mfma_kv_share(cache->head_dim, rows_of(cache, n_q_heads, opts));
}

// whether the matrix-core kernel can take a step's new token in
bool takes_token(const tq_kv_cache* cache, int n_q_heads, const tq_decode_opts* opts) {
  return tq::mfma_takes_token(cache->head_dim, cache->group_size, rows_of(cache, n_q_heads, opts));
}

// What a call is: a decode, or a decode step, of one common length; either of per-sequence lengths (seq_len: their bound).
enum class Call { kDecode, kStep, kLengths };

// Where the kernel for wide rows is taken (head_dim 512: always, any finite scale; else groups of 32 and a positive one).
// head_dim 256 with more than two query rows per KV head: it takes 16 rows to a block, the other one two,
// and unpacks the stream again for every two.  It always merges in a launch of its own, so what it loses by shows where blocks of many
// rows have little to do each: with one query token it is taken from five rows on (16 heads over 4, one sequence of 32K tokens
// 17.1 / 18.7 us per step, other / this) and from 12K (token, KV head) pairs (32 heads over 4, 4 sequences of 512, 10.3 / 9.9, one of
// 3072 as long on either), and with more than 128 (sequence, KV head) rows only for sequences of 512 tokens and more (1024 where they have
// lengths of their own, which the other kernel orders).  us per step, other / this: 32 heads over 4, 6000 tokens
// 12.1 / 11.3, 20K 17.9 / 15.5, 128K 66.9 / 40.1; 8 sequences of 1000 14.4 / 11.6, of 8192 54.0 / 26.2; 64 of 200 14.4 / 15.4,
// of 600 25.2 / 22.8; 128 of 150 18.0 / 25.4, of 2000 117 / 81.1; own lengths: 8 of 400 .. 6000 22.1 / 19.0, 32 of 100 .. 1000 19.1 / 17.5,
// 64 of 60 .. 600 23.7 / 28.5, of 100 .. 2000 41.4 / 39.0, 128 of 60 .. 600 36.5 / 52.6.  Several query tokens: 32 heads over 16, 2 of
// them, 600 tokens 14.0 / 10.4, 32K 46.5 / 40.5; 8, 32K 125 / 42.4; 16 over 8, 8 of them, 4 sequences of 2000 32.7 / 16.3.
bool wide_rows_at_256(int rows, int64_t kv_rows, int tokens, int n_queries, Call call) {
  if (rows <= (n_queries > 1 ? 2 : 4) || (n_queries == 1 && kv_rows * tokens < 12288)) return false;
  return kv_rows <= 128 || tokens >= (call == Call::kLengths ? 1024 : 512);
}
// head_dim 128: up to 128 (sequence, KV head) rows (with more the other kernel's blocks are full, and it orders and packs them), and
// up to some tokens L per compute unit (and 32-row block, where a KV head's rows take several).  It starts and merges sooner and takes
// several new tokens in, where the other launches the append kernel (2.6 us); the 16-row tile takes less time per token:
//   9 .. 16 rows   a step 8.8 us (several query tokens 9.2) + 9.2 ns L here, 12.9 us (16.3) + 5.6 ns L on the 16-row tile
//   17 .. 32 rows         10.8 us                            + 13.9 ns L here, 17.0 us      + 10.4 ns L there, two tiles
// and a decode is 0.3 us shorter here, 1.3 (several query tokens 2.8 .. 4) there.  The lines lie before these meet (step 1190, several
// 1950, 17 rows and more 1790; decode 910, 1410, 870), further before where lengths next to each other go either way.  Up to eight rows only the append
// launch is saved (a launch of one new token has none to save: 64 heads over 8, 8191 tokens 10.8 / 10.5 us per step, 32 heads over 8, 4000,
// 8.4 / 9.1).  us per step, other / this (d: per decode):
// 17 rows and more: 64 heads over 8, 4 query tokens, 600 tokens 16.8 / 11.5, 8000 18.9 / 14.1 (d 16.1 / 14.0), 16K 22.4 / 17.9
// (d 18.7 / 17.6), 24K 23.9 / 21.5 (d 21.2 / 21.2), 32K 25.8 / 25.0 (d 23.1 / 24.8), 48K 32.0 / 32.2, 128K 59.5 / 67.9; 16 sequences of
// 1000 19.8 / 18.5 (d 15.9 / 18.0); 8 query tokens, 16K 25.9 / 25.6 (d 23.2 / 24.3), 24K 30.9 / 32.7; 128 heads over 8, 4, 16K 26.8 / 25.1.
// 9 .. 16 rows: 128 heads over 8, 600 tokens 13.9 / 9.4, 8192 14.3 / 10.9, 24K 17.3 / 15.7 (d 16.0 / 15.5), 32K 18.7 / 18.4 (d 17.3 / 17.8),
// 48K 21.8 / 22.8, 128K 36.7 / 46.6; 16 sequences of 1500 17.2 / 15.7 (d 15.7 / 14.9); 64 over 8, 2 query tokens, 16K 19.1 / 13.9, 32K
// 21.9 / 18.8 (d 19.3 / 18.1), 48K 24.7 / 23.3 (d 22.1 / 22.7), 64K 27.3 / 28.0, 128K 38.9 / 47.0; own lengths, 4 of 400 .. 6000
// 17.7 / 15.1, 8 of them 20.4 / 18.3, 16 of 300 .. 4000 21.6 / 21.0, 8 of 2000 .. 8000 24.0 / 24.4.
// Up to 8 rows: 32 over 8, 2, 8000 14.4 / 10.6, 24K 16.9 / 16.1, 30K 18.1 / 17.5; 32 over 32, 2, 2000 11.0 / 10.7, 4000 13.7 / 13.3.
bool wide_rows_at_128(int rows, int64_t kv_rows, int tokens, int n_queries, Call call) {
  if (kv_rows > 128) return false;
  const bool step = call == Call::kStep;
  const int64_t load = kv_rows * tokens / kBlocksWide * std::max(1, (rows + 31) / 32);   // tokens per compute unit and block
  if (call == Call::kLengths) return rows > 8 && load <= 1600;   // (tokens: the longest, the others may be any)
  if (rows > 16) return step ? load <= 1250 : load <= 600 && kv_rows <= 64;
  if (rows > 8) return load <= (n_queries > 1 ? (step ? 1800 : 1200) : (step ? 1100 : 900));
  return n_queries > 1 && step && load <= (rows > 4 ? 960 : 500);
}
bool wide_rows(const tq_kv_cache* cache, int n_q_heads, int seq_len, float attn_scale, const tq_decode_opts* opts, Call call) {
  if (cache->head_dim == 512) return std::isfinite(attn_scale);
  if (cache->group_size != tq::kGroup || !(attn_scale > 0.0f && std::isfinite(attn_scale))) return false;
  const auto rule = cache->head_dim == 256 ? wide_rows_at_256 : wide_rows_at_128;
  return rule(rows_of(cache, n_q_heads, opts), (int64_t)cache->batch * cache->n_kv_heads, windowed(seq_len, opts), queries_of(opts), call);
}

Route route_of(const tq_kv_cache* cache, int n_q_heads, int seq_len, float attn_scale, const tq_decode_opts* opts, Call call) {
  const int variant = opts ? opts->variant : 0;
  // groups of 64 or 128 elements: the matrix-core kernel at head_dim 128 and 256 (see mfma_supports_group), else the
  // generic vector-ALU kernel with one query token per sequence
  // (groups of 128 at head_dim 128 under a sliding window: a window may start at an odd token, in the middle of a
  // pair; head_dim 256 has no pairs, and takes the matrix-core kernel only by default: variant 2 and several query
  // tokens are not offered there)
  const bool larger = cache->group_size != tq::kGroup;
  const bool pairs_split = cache->head_dim == 128 && cache->group_size == 4 * tq::kGroup && opts && opts->window > 0;
  if (!tq::mfma_supports_group(cache->head_dim, cache->group_size, cache->capacity) || pairs_split ||
      (larger && cache->head_dim == 256 && (variant == 2 || queries_of(opts) > 1))) {
    const bool ok = variant != 2 && queries_of(opts) == 1;
    return {ok, false, false, false, false, false};
  }
  // the matrix-core kernel folds attn_scale into its exp2 argument and needs it positive and finite
  const bool scale_ok = attn_scale > 0.0f && std::isfinite(attn_scale);
  if (variant == 2 && !scale_ok) return {false, false, false, false, false, false};
  // the kernel for wide rows, partials merged by the merge kernel
  if (variant != 1 && wide_rows(cache, n_q_heads, seq_len, attn_scale, opts, call))
    return {true, false, false, false, true, false};
  // the matrix-core kernel addresses a (batch, KV head) row of codes with 32-bit byte offsets
  const bool offsets_ok = (int64_t)seq_len * (cache->head_dim / 2) < (1ll << 31);
  if (variant == 2 && !offsets_ok) return {false, false, false, false, false, false};
  const int rows = rows_of(cache, n_q_heads, opts);
  const bool use_mfma = variant == 2 || (variant == 0 && scale_ok && offsets_ok &&
                                         tq::mfma_supported(cache->head_dim, rows));
  if (!use_mfma && queries_of(opts) > 1) return {false, false, false, false, false, false};
  // (more query rows than the kernel's tile holds: several blocks stream each KV head, counted as rows of their own)
  const int rows_per_batch = cache->n_kv_heads * std::max(1, use_mfma ? mfma_share_of(cache, n_q_heads, opts) : 1);
  const int64_t bytes = (int64_t)tq_kv_bytes(cache->batch, rows_per_batch, windowed(seq_len, opts), cache->head_dim);
  // a sequence that is one chunk needs no merge at all: the kernel writes the output itself, whatever the size
  const int chunks = plan_splits(cache->batch, rows_per_batch, windowed(seq_len, opts), opts ? opts->n_splits : 0,
                                 kBlocksMfma, 8).n_splits;
  const bool single = use_mfma && chunks == 1;
  // (a 16-row tile leaves the last block twice the partials to fetch: there the merge kernel is the faster end,
  //  measured 21.8 against 24.1 us with 16 heads per KV head at 32K tokens)
  const bool small_tile = rows_per_batch == 0 || rows * cache->n_kv_heads / rows_per_batch <= 8;
  const bool in_place = small_tile && chunks <= kMergeInKernelMaxChunks && tq::mfma_can_merge((int64_t)cache->batch * queries_of(opts) * n_q_heads);
  // (larger groups at head_dim 256, decode alone: two launches as well)
  const bool merge = use_mfma && (single || (in_place && bytes <= kMergeInKernelMaxBytes && !(larger && cache->head_dim == 256)));
  return {true, use_mfma, merge, use_mfma && (single || in_place), false, small_tile};
}

// waves that share one (sequence, KV head) row where single-chunk rows are packed several to a block
int waves_per_packed_row(int64_t total_rows, int target) {
  return total_rows > 4 * target ? 1 : total_rows > 2 * target ? 2 : total_rows > target ? 4 : 8;
}

// Many sequences with their own lengths: from two rounds of eight-wave blocks on (512 (sequence, KV head) rows), every
// row can be ONE chunk of its own length in a block of its own (DecodeParams::ranked), with as many waves (8, 4, 2, 1)
// as make one or two rounds of what the chip holds; the decode kernel writes the output itself, and neither the
// device-side chunk plan nor the merge kernel is needed.  But such a row is never cut: the launch lasts at least as long
// as the longest row (about 1.05 us per 32 tokens of a wave, and 8 us), whatever the others are, where the plan's lasts
// as long as the sum.  The host knows only the bound, so the lines below lie where ONE sequence at the bound among very
// short ones costs about what the plan takes for it.  us per step, ranked / planned, 64 heads over 8, d = 128, for
// lengths spread over the logarithm up to the bound | one at the bound, the others 96 | all at the bound:
//   64 sequences (512 rows)   1024, 4 waves 16.0 / 21.5 | 15.3 / 18.3 | 21.3 / 30.5    2048, 4 waves 23.1 / 26.2 | 21.9 / 19.1 | 33.3 / 43.5
//                             4096, 8 waves 31.8 / 32.4 | 26.1 / 21.5 | 58.9 / 76.3    8192, 8 waves 45.2 / 44.0 | 42.7 / 21.6 | 113 / 121
//   56 (448 rows, planned)    2048, 4 waves 22.8 / 24.5 | 21.9 / 19.0 | 31.2 / 40.0    4096, 8 waves 28.1 / 29.9 | 26.0 / 19.1 | 54.4 / 62.4
//   72                        3072, 4 waves 30.8 / 38.1 | 28.8 / 28.0 | 66.2 / 75.8    4096, 8 waves 36.3 / 43.9 | 26.2 / 29.2 | 88.0 / 97.0
//   128                       3072, 4 waves 40.0 / 44.8 | 29.5 / 28.5 | 86.7 / 100     4096, 4 waves 44.4 / 51.1 | 36.0 / 30.0 | 113 / 129
//   160                       1500, 2 waves 33.1 / 57.5 | 29.6 / 33.2 | 72.3 / 97.7    2048, 4 waves 41.2 / 63.3 | 28.9 / 33.0 | 92.1 / 123
//   256                       2048, 2 waves 51.7 / 71.4 | 36.7 / 47.5 | 117 / 146      300: 1024, 1 wave 44.3 / 80.0 | 38.4 / 46.1 | 97.4 / 130
// and at d = 256, 32 heads over 16: 32 sequences, 2048, 8 waves 32.6 / 33.3 | 25.8 / 22.2 | 58.0 / 69.3, 3072 39.0 / 41.1 |
// 35.2 / 22.4 | 83.4 / 90.6; 64, 2048, 4 waves 47.0 / 55.3 | 29.2 / 31.2 | 110 / 130; 80, 2048, 4 waves 57.5 / 87.6 |
// 29.7 / 36.6 | 136 / 207.
// (One query token and no window: listed_lengths first; what is past its lines comes here, and from there to the chunk list.)
// Sequences past what a launch can order come in the given order: half the tokens per wave (600 sequences, 8 heads over 1,
// 2048, 4 waves 32.8 / 41.8 | 21.8 / 26.9 | 49.1 / 66.3).
int ranked_waves(int64_t rows, int batch, int tokens, bool d256) {
  constexpr int C = kBlocksMfma;
  if (rows < 2 * C) return 0;
  int waves = 0;
  if (rows <= 4 * C) {
    if (tokens <= (rows <= 9 * C / 4 ? (d256 ? 1024 : 2048) : (d256 ? 2048 : 3072))) waves = 4;
    else if (rows <= 11 * C / 4 && tokens <= (d256 ? 2048 : 4096)) waves = 8;
  } else if (rows <= 8 * C) {
    if (tokens <= 2048) waves = rows <= 6 * C && tokens > (d256 ? 1024 : 1536) ? 4 : 2;
  } else if (tokens <= 1024) {
    waves = 1;
  }
  return batch > tq::kRankMaxBatch && waves > 1 && tokens > 512 * waves ? 0 : waves;
}
struct Ranked { int waves, spread; };             // waves of a row's block, 0 = not this way; DecodeParams::rank_spread
Ranked ranked_rows(const tq_kv_cache* cache, int n_q_heads, int seq_len, float attn_scale, const tq_decode_opts* opts) {
  if (queries_of(opts) > 1 || (opts && opts->n_splits > 0)) return {0, -1};
  const Route r = route_of(cache, n_q_heads, seq_len, attn_scale, opts, Call::kLengths);
  if (!r.ok || !r.use_mfma) return {0, -1};
  const int64_t rows = (int64_t)cache->batch * cache->n_kv_heads * mfma_share_of(cache, n_q_heads, opts);
  const bool d256 = cache->head_dim == 256;
  const int waves = ranked_waves(rows, cache->batch, windowed(seq_len, opts), d256);
  // Two rows to a block where the longest is at most 16 tiles (d = 256: 8) per wave of its half block over the average; 5
  // where the rows fill that one round badly (us per step, two rounds / one, 64 heads over 8: 64 sequences of 128 .. 4096
  // tokens 31.5 / 37.0, all of 4096 63.9 / 58.9; 256 of 64 .. 2048 75.9 / 80.8, of 64 .. 1024 51.5 / 46.9, all of 1024
  // 86.6 / 65.6; badly filled: 34 of 33 .. 340, 32 heads over 32, 12.1 / 15.3).  Not where the rows fit one round as they
  // are (64 of 1024, 4 waves, 21.3 / 24.3), nor where the pairs don't (72 of 4096, 8 waves, 88.0 / 98.4).
  const int64_t chip = 8 * kBlocksMfma, paired = rows * (waves / 2);
  int spread = -1;
  if (cache->batch <= tq::kRankMaxBatch && waves > 1 && rows * waves > chip && paired <= chip)
    spread = (paired >= chip - kBlocksMfma ? 16 : 5) * (waves / 2) / (d256 ? 2 : 1);
  return {waves, spread};
}

// Sequences with their own lengths, up to eight query rows to a block, one query token, no window: the device deals the waves of one
// round of blocks to the sequences in proportion to their lengths (DecodeParams::listed), a sequence's waves in a block merge among themselves and
// its blocks in place.  Every wave has the same share to a tile, where the chunk list has one chunk length for all and a block or half of one
// per chunk (so that half a chunk per sequence is idle time), and there is no merge launch.  0: not this way; else slots (waves) to a KV head.
// us per step, chunk list / this, 64 heads over 8, d = 128: 24 sequences of 1000 .. 16384 in pages 42.5 / 38.3, 8 of 4386 .. 32768 40.6 / 39.2,
// 16 of 300 .. 3000 18.4 / 13.8, 48 of 300 .. 6000 42.1 / 30.8, 32 of 1000 19.2 / 14.3; 32 over 32: 8 of 500 .. 6000 27.1 / 22.0; 32 over 8:
// 32 of 100 .. 8000 26.1 / 20.3; 32 over 16, d = 256: 16 of 500 .. 8000 57.2 / 48.1, 20 of 1500 49.2 / 36.4.
// Where every row can have a block of its own (ranked_waves: 512 rows and more) no sequence is cut and the plan is shorter; and a sequence is
// one wave's at least, so with few slots to a sequence the waves' shares are uneven again: three sequences of one length on eight slots are two
// waves each and two idle.  So the lines go by slots per sequence, each drawn by the mean over three mixes, all lengths at the bound | uniform from half of it |
// spread over the logarithm from a 32nd.  us per step, a block per row or (where that has no line) chunk list / this, 64 heads over 8, d = 128:
//   64 sequences (4 slots each; in pairs they fill the chip as blocks of their own, which 65 no longer do)
//       2048  34.4 / 34.8 | 27.9 / 31.0 | 23.0 / 22.6     3072  48.3 / 49.0 | 41.1 / 42.3 | 29.6 / 24.6
//       4096  58.1 / 59.1 | 50.8 / 51.7 | 32.2 / 28.3     6000  87.8 / 84.5 | 78.6 / 73.0 | 40.5 / 37.0
//   80 (3.2)    1024  30.3 / 31.3 | 28.7 / 27.1 | 21.7 / 19.2
//   85 (3.01)   2048  48.5 / 48.6 | 47.2 / 41.8 | 24.4 / 25.1     4096  88.4 / 81.6 | 75.2 / 73.0 | 40.0 / 36.4
//   88 (2.9)    3000  71.0 / 80.1 | 62.4 / 57.9 | 32.9 / 32.7     4096  89.9 / 107  | 75.3 / 74.7 | 41.3 / 37.3     5000  119 / 130 | 106 / 90.3 | 57.4 / 43.9
//       (the older way up to 4096 a block per row, beyond the chunk list)
//   96 (2.7)    4096  104 / 112   | 99.8 / 81.9 | 51.0 / 38.4    16384  356 / 411   | 312 / 282   | 138 / 111
//   128 (2)     2048  60.5 / 74.0 | 54.2 / 66.7 | 33.8 / 31.5     8192  230 / 255   | 193 / 215   | 85.9 / 81.4
//   (more: the chunk list's waves are as short of work)
//   130 (1.97)  2200  115 / 109   | 105 / 72.7  | 60.7 / 37.1     8192  339 / 358   | 293 / 217   | 132 / 84.8
//   192 (1.33)  3500  184 / 182   | 170 / 149   | 87.8 / 72.4     8192  394 / 418   | 337 / 328   | 156 / 155
//   200 (1.28)  3000  173 / 171   | 148 / 139   | 80.3 / 75.2     8192  399 / 431   | 330 / 343   | 153 / 170
//   212 (1.21)  2200  139 / 136   | 118 / 114   | 69.6 / 64.6     3500  199 / 202   | 169 / 169   | 87.7 / 92.5
// With up to four query rows to a KV head (`light`: a wave's tile is cheaper against the rest) the dealt waves gain for longer:
//   32 over 32  22 (2.9)   1100  28.1 / 29.9 | 25.1 / 23.6 | 18.1 / 15.3     4096  81.6 / 83.2 | 66.2 / 65.5 | 37.3 / 32.9
//               54 (1.19)  4096   202 / 182  | 173 / 163   | 83.5 / 90.8     8000   358 / 350  | 299 / 314   | 140 / 168       56 (1.14)  4096  198 / 183 | 166 / 162 | 77.8 / 95.3
//   64 over 16  44 (2.9)   3000  63.5 / 64.9 | 55.0 / 51.1 | 30.7 / 26.6     105 (1.22)  4096  202 / 186 | 165 / 162 | 87.1 / 89.0     8000  363 / 354 | 301 / 311 | 141 / 160
//   32 over 8   88 (2.9)   2048  44.1 / 50.5 | 41.9 / 38.4 | 22.6 / 22.2     200 (1.28)  2200  122 / 109 | 105 / 93.0 | 58.6 / 48.5     8000  359 / 344 | 302 / 303 | 134 / 139
// and at d = 256, 32 heads over 16: 32 (4) 2048 60.6 / 63.8 | 52.3 / 52.5 | 35.5 / 29.3, 2500 81.4 / 76.8 | 70.2 / 61.9 | 40.4 / 36.0; 33 (3.9) 200 15.0 / 17.3 |
// 13.5 / 15.8 | 11.7 / 13.0, 400 21.5 / 23.1 | 18.1 / 19.6 | 15.5 / 14.5, 700 32.4 / 32.8 | 26.6 / 26.2 | 16.7 / 17.3 (the one batch that has little of it up to 768);
// 37 (3.5) 256 18.7 / 19.9 | 16.9 / 17.9 | 14.7 / 13.9, 300 21.0 / 20.8 | 19.1 / 19.0 | 15.8 / 14.3, 700 39.0 / 33.8 | 32.2 / 28.5 | 18.6 / 18.3; 42 (3) 256 19.0 / 20.6 |
// 17.4 / 18.8 | 15.3 / 14.9, 300 21.4 / 21.7 | 19.7 / 19.5 | 17.2 / 15.8, 700 39.9 / 36.4 | 33.5 / 30.6 | 20.7 / 19.3; 44 (2.9) 500 31.8 / 32.0 | 27.7 / 25.6 | 19.6 / 18.2,
// 2048 99.0 / 98.9 | 71.8 / 71.4 | 36.7 / 36.3; 64 (2) 3000 170 / 164 | 144 / 135; 109 (1.17) 4096 416 / 393 | 343 / 313 | 163 / 170, 6000 581 / 580 | 501 / 483 | 232 / 247.
// More than 128 KV heads have a block each and leave up to half the chip without one: 129 heads over 129, 4 sequences, 4000 77.7 / 78.8 | 58.4 / 81.4 | 30.9 / 37.4
// (3, where the chunk list leaves as much: 74.9 / 75.3 | 73.8 / 53.3 | 40.5 / 32.3).
// One sequence at the bound among short ones gains everywhere (64 sequences, one of 4096, the others 96: 25.3 / 14.4).
bool listed_lengths(const tq_kv_cache* cache, int n_q_heads, int slots, int tokens) {
  constexpr int C = kBlocksMfma;
  const int batch = cache->batch;
  const int64_t rows = (int64_t)batch * cache->n_kv_heads;
  const bool d256 = cache->head_dim == 256;
  const bool light = !d256 && cache->group_size == tq::kGroup && n_q_heads / cache->n_kv_heads <= 4;
  if (rows < 2 * C) return true;
  if (cache->n_kv_heads > C / 2) return false;
  if (rows == 2 * C) return tokens > (d256 ? 2048 : 3072);
  // (2.9 slots to a sequence and more)
  if (11 * slots >= 32 * batch) return tokens > (d256 ? 256 : light || slots >= 3 * batch ? 1024 : 4096);
  if (rows <= 4 * C) return d256 && tokens > 2048;
  // slots to a sequence, in sixtieths
  const int least = d256 ? 70 : light ? (tokens <= 4096 ? 70 : 75) : tokens <= 3072 ? 72 : 80;
  return tokens > 2048 && 60 * slots >= least * batch;
}
int listed_slots(const tq_kv_cache* cache, int n_q_heads, int seq_len, float attn_scale, const tq_decode_opts* opts) {
  if (opts && (opts->n_splits > 0 || opts->window > 0 || opts->n_queries > 1)) return 0;
  const Route r = route_of(cache, n_q_heads, seq_len, attn_scale, opts, Call::kLengths);
  if (!r.ok || !r.use_mfma || !r.small_tile || mfma_share_of(cache, n_q_heads, opts) != 1 || cache->n_kv_heads > kBlocksMfma) return 0;
  const int slots = kBlocksMfma / cache->n_kv_heads * 8;
  // (a slot for every sequence and one more; what the device's plan keeps in registers, and sums in 32 bits)
  if (slots <= cache->batch || cache->batch > tq::kListMaxBatch || (int64_t)cache->batch * seq_len >= (1ll << 31)) return 0;
  if (!tq::mfma_can_merge((int64_t)cache->batch * n_q_heads)) return 0;
  return listed_lengths(cache, n_q_heads, slots, seq_len) ? slots : 0;
}

// The device-planned chunk list of sequences with their own lengths, per KV head: r rounds of target / rows_per_batch slots, r the smallest count
// that leaves at least half of them once every sequence has been granted its partial last chunk.  Many sequences: the slots of several
// rounds share blocks (2, 4 or 8 to a block, `waves` each; matrix-core kernel) and run in one.
struct ChunkList { int slots, waves; };
ChunkList chunk_list(int batch, int rows_per_batch, int target) {
  const int per_round = std::max(1, target / rows_per_batch);            // (one round never spills into a second)
  const int rounds = std::max(1, (2 * batch + per_round - 1) / per_round);
  return {rounds * per_round, rounds > 4 ? 1 : rounds > 2 ? 2 : rounds > 1 ? 4 : 8};
}

// One launch of phase 1: what to attend, and what came of it.
struct PartialRequest {
  const tq_kv_cache* cache;            // validated; for a paged pool: the view with batch = sequences
  const void* q;
  int32_t n_q_heads, seq_len;          // seq_len: the common length, or the bound of seq_lens
  const int32_t* seq_lens = nullptr;   // device, per-sequence lengths
  float attn_scale = 0.0f;
  void* out = nullptr;                 // non-null: the kernel may merge the chunks itself and write it
  void* workspace = nullptr;
  const tq_decode_opts* opts = nullptr;
  const void* k_new = nullptr;         // append-and-attend: the step's new token (then seq_len includes it), taken in
  const void* v_new = nullptr;         // by the matrix-core kernel, or by the merge kernel behind the others
  bool new_in_chunks = false;          // k_new / v_new hold the last n_queries of the attended tokens: the kernel for wide rows
                                       // takes them in as tokens of the chunks (common length)
  bool step = false;                   // a decode step (the new token(s) may be in the cache already)
  const tq::PagedView* paged = nullptr;
  void* stream = nullptr;
  // results
  int32_t n_splits = 0;
  bool merged = false;                 // `out` has been written
  DecodeParams params{};               // what the kernel was given (the merge kernel takes the same)
};

// Phase 1 (and, with `out`, the whole decode where the matrix-core kernel can merge in place).
int run_partial(PartialRequest& rq) {
  const tq_kv_cache* cache = rq.cache;
  const tq_decode_opts* opts = rq.opts;
  const int32_t* seq_lens = rq.seq_lens;
  const int n_q_heads = rq.n_q_heads, seq_len = rq.seq_len;
  const Route r = route_of(cache, n_q_heads, seq_len, rq.attn_scale, opts,
                           seq_lens ? Call::kLengths : rq.step ? Call::kStep : Call::kDecode);
  if (!r.ok) return TQ_ERR_UNSUPPORTED;
  const bool use_mfma = r.use_mfma;
  const int target = use_mfma ? kBlocksMfma : r.wide ? kBlocksWide : kBlocksValu;
  int attended = windowed(seq_len, opts);         // chunks cover the attended tokens only
  // (paged cache: counted from the supertile boundary before the window, see var_start)
  if (rq.paged && attended < seq_len) attended = std::min(seq_len, attended + tq::kTile - 1);
  // append-and-attend: the new token (the last attended one) does not come from the cache
  const bool append = rq.k_new != nullptr && !rq.new_in_chunks;
  const int first = seq_len - attended;           // first attended token
  if (append) --attended;
  const int row_tiles = r.wide ? tq::wide_row_tiles(cache->head_dim, rows_of(cache, n_q_heads, opts)) : 1;
  const int mfma_share = use_mfma ? mfma_share_of(cache, n_q_heads, opts) : 1;
  const int rows_per_batch = cache->n_kv_heads * (use_mfma ? mfma_share : row_tiles);
  int merge_slot = -1;
  int slots = seq_lens && rq.out != nullptr ? listed_slots(cache, n_q_heads, seq_len, rq.attn_scale, opts) : 0;
  if (slots > 0 && (merge_slot = tq::mfma_merge_slot_of(rq.workspace)) < 0) slots = 0;     // (no arrival counters left: the other ways)
  const Ranked rank = seq_lens && rq.out != nullptr && slots == 0 ? ranked_rows(cache, n_q_heads, seq_len, rq.attn_scale, opts)
                                                                  : Ranked{0, -1};
  const bool ranked = rank.waves > 0;
  const int asked = ranked ? 1 : opts ? opts->n_splits : 0;
  Plan plan = plan_splits(cache->batch, rows_per_batch, attended, asked, target, use_mfma ? 8 : 1);
  if (r.wide && asked <= 0)
    plan = plan_splits(cache->batch, rows_per_batch, attended,
                       std::min(plan.n_splits, tq::wide_max_chunks(cache->head_dim, (attended + tq::kTile - 1) / tq::kTile)), target, 1);
  // (the chunks of one token fewer may be shorter, and then up to twice as many as the route counted)
  rq.merged = ranked || (rq.out != nullptr && (rq.step ? r.merge_step : r.merge) && !seq_lens && plan.n_splits <= tq::kMergeMaxChunks);
  if (rq.merged) {
    const int fine = ranked || asked > 0 || !r.small_tile ? 1 : fine_splits_of(cache, n_q_heads, opts, rows_per_batch, attended);
    // several chunks: the arrival counters of this workspace (none left: the merge kernel does it); rows that are
    // single chunks count nothing
    merge_slot = std::max(plan.n_splits, fine) > 1 ? tq::mfma_merge_slot_of(rq.workspace) : 0;
    if (merge_slot < 0 && plan.n_splits == 1) merge_slot = 0;
    else if (merge_slot < 0) rq.merged = false;
    else if (fine > plan.n_splits) plan = plan_splits(cache->batch, rows_per_batch, attended, fine, target, 1);
  }
  DecodeParams p = make_params(cache, rq.q, n_q_heads, seq_len, rq.attn_scale, rq.out, rq.workspace, plan,
                               queries_of(opts));
  p.seq_lens = seq_lens;
  p.batch = cache->batch;
  if (seq_lens) {
    // the kernels window every sequence's own length (append-and-attend: the lengths count the new token, the
    // chunks and the window over them do not)
    p.len_bias = append ? -1 : 0;
    p.window = (opts && opts->window > 0) ? opts->window + queries_of(opts) - 1 + p.len_bias : 0;
  } else {
    p.seq_len = attended;
    p.start = first;
  }
  p.row_window = (opts && queries_of(opts) > 1) ? opts->window : 0;
  if (rq.paged) {
    p.block_table = rq.paged->block_table;
    p.max_blocks = rq.paged->max_blocks;
    p.page_shift = rq.paged->page_shift;
  }
  if (slots > 0) {
    p.listed = 1;
    p.var_chunks = slots;
    p.n_splits = tq::kMaxSplits;
    p.waves_per_row = 8;
    rq.merged = true;
  } else if (seq_lens && !(opts && opts->n_splits > 0) && !ranked) {
    // per-sequence lengths, no chunk count asked for: the kernels plan the chunks themselves from the lengths (a requested n_splits
    // keeps the fixed chunking)
    const ChunkList list = chunk_list(cache->batch, rows_per_batch, target);
    p.var_chunks = list.slots;
    p.var_min_chunk = use_mfma ? 8 * tq::kTile : r.wide ? 2 * tq::kTile : tq::kTile;
    p.n_splits = tq::kMaxSplits;
    if (use_mfma) p.waves_per_row = list.waves;
  }
  rq.n_splits = plan.n_splits;
  hipStream_t s = static_cast<hipStream_t>(rq.stream);
  rq.params = p;
  if (append) {
    // One of the two kernels takes the token in: the decode kernel where it writes the output (there is no other) and
    // with up to eight rows to a block; with sixteen its sixteen scores are on the way of a short chunk and the merge
    // kernel, which there always is, is the cheaper place (128 heads over 8, 8K tokens, 15.3 / 14.5 us per step).
    const bool here = use_mfma && takes_token(cache, n_q_heads, opts) && (rq.merged || r.small_tile || cache->group_size != tq::kGroup);
    DecodeParams& taker = here ? p : rq.params;
    taker.k_new = static_cast<const half_t*>(rq.k_new);
    taker.v_new = static_cast<const half_t*>(rq.v_new);
    taker.append_pos = seq_len - 1;
  }
  if (ranked) {
    p.ranked = 1;
    p.waves_per_row = rank.waves;
    p.rank_spread = rank.spread;
  } else if (rq.merged && use_mfma && plan.n_splits == 1 && !rq.paged && slots == 0) {
    // more single-chunk rows than the chip holds blocks: pack 2, 4 or 8 of them into a block
    p.waves_per_row = waves_per_packed_row((int64_t)cache->batch * rows_per_batch, target);
  }
  if (use_mfma) {
    p.kv_share = mfma_share;
    return hip_rc(tq::launch_partial_mfma(p, cache->batch, cache->head_dim, merge_slot, s));
  }
  if (r.wide) {
    if (rq.new_in_chunks) {
      p.k_new = static_cast<const half_t*>(rq.k_new);
      p.v_new = static_cast<const half_t*>(rq.v_new);
    }
    p.kv_share = row_tiles;
    return hip_rc(tq::launch_partial_wide(p, cache->batch, cache->head_dim, s));
  }
  return hip_rc(tq::launch_partial_valu(p, cache->batch, cache->head_dim, false, s));
}

// Phase 2 after run_partial, unless the kernel has merged already.
int finish_decode(const PartialRequest& rq, int rc) {
  if (rc != TQ_OK || rq.merged) return rc;
  return hip_rc(tq::launch_reduce(rq.params, rq.cache->batch, rq.cache->head_dim, static_cast<hipStream_t>(rq.stream)));
}

// A pool of pages seen as a cache: `batch` sequences whose rows are pages of pool->capacity tokens.
int paged_view(const tq_kv_cache* pool, const int32_t* block_table, int32_t max_blocks, int32_t batch,
                      tq_kv_cache* view, tq::PagedView* pv) {
  const int rc = check_cache(pool);
  if (rc == TQ_ERR_NULL || !block_table) return TQ_ERR_NULL;
  if (rc != TQ_OK && rc != TQ_ERR_ALIGN) return rc;
  const int pt = pool->capacity;
  if (pt < tq::kTile || (pt & (pt - 1)) != 0 || batch < 1 || max_blocks < 1) return TQ_ERR_SHAPE;
  if (rc == TQ_ERR_ALIGN || !aligned(block_table, 4)) return TQ_ERR_ALIGN;
  *view = *pool;
  view->batch = batch;
  int shift = 0;
  while ((1 << shift) < pt) ++shift;
  *pv = tq::PagedView{block_table, max_blocks, shift, batch};
  return TQ_OK;
}

// ---- tq_sdpa_int4_decode_static: the workspace of callers that cannot allocate.
// One array per GPU the library runs on, held until the process ends.  In host code the array's name is only a
// stand-in for the symbol: the memory's address on a device is what hipGetSymbolAddress returns with that
// device current, and that pointer is what the kernels get.
constexpr size_t kScratchBytes = TQ_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void* scratch_ptr[kMaxDevices];                   // per device: where that device's copy of `scratch` lives

// The current device's copy of `scratch` (resolved once per device, on the first call with that device current).
int scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TQ_ERR_HIP;
  std::lock_guard<std::mutex> guard(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return TQ_ERR_HIP;
    scratch_ptr[dev] = ptr;
  }
  *out = scratch_ptr[dev];
  return TQ_OK;
}

}  // namespace

extern "C" {

size_t tq_workspace_bytes(int32_t batch, int32_t n_q_heads, int32_t head_dim) {
  if (batch < 1 || n_q_heads < 1 || !head_dim_ok(head_dim)) return 0;
  // partial outputs, their (m, l), and one cache line for the device-side chunk plan
  return (tq::workspace_o_floats(batch, n_q_heads, head_dim) + tq::workspace_ml_floats(batch, n_q_heads)) *
             sizeof(float) + 256;
}

size_t tq_dense_scratch_bytes(int32_t batch, int32_t n_kv_heads, int32_t seq_len, int32_t head_dim) {
  if (batch < 1 || n_kv_heads < 1 || seq_len < 1 || !head_dim_ok(head_dim)) return 0;
  return (size_t)2 * batch * n_kv_heads * seq_len * head_dim * sizeof(half_t);
}

size_t tq_kv_bytes_grouped(int32_t batch, int32_t n_kv_heads, int32_t capacity, int32_t head_dim, int32_t group_size) {
  if (group_size != 32 && group_size != 64 && group_size != 128) return 0;
  if (batch < 1 || n_kv_heads < 1 || capacity < 1 || head_dim < group_size || head_dim % group_size != 0) return 0;
  const size_t per_token = (size_t)head_dim / 2 + 2 * sizeof(half_t) * (head_dim / group_size);
  return (size_t)2 * batch * n_kv_heads * capacity * per_token;
}

size_t tq_kv_bytes(int32_t batch, int32_t n_kv_heads, int32_t capacity, int32_t head_dim) {
  return tq_kv_bytes_grouped(batch, n_kv_heads, capacity, head_dim, tq::kGroup);
}

int32_t tq_plan_splits(int32_t batch, int32_t n_kv_heads, int32_t seq_len) {
  if (batch < 1 || n_kv_heads < 1 || seq_len < 1) return 0;
  return plan_splits(batch, n_kv_heads, seq_len, 0, kBlocksMfma, 8).n_splits;
}

int32_t tq_decode_launches(const tq_kv_cache* cache, int32_t n_q_heads, int32_t seq_len, float attn_scale,
                           const tq_decode_opts* opts) {
  const int rc = check_cache(cache);
  if (rc != TQ_OK && rc != TQ_ERR_ALIGN) return 0;
  if (n_q_heads < 1 || n_q_heads % cache->n_kv_heads != 0 || seq_len < 1 || seq_len > cache->capacity) return 0;
  if (opts && (opts->variant < 0 || opts->variant > 2)) return 0;
  if (opts && (opts->n_queries < 0 || opts->n_queries > tq::kMaxQueries || seq_len < queries_of(opts))) return 0;
  if (opts && opts->variant == 2 && cache->head_dim != 512 &&
      !tq::mfma_supported(cache->head_dim, rows_of(cache, n_q_heads, opts)))
    return 0;
  const Route r = route_of(cache, n_q_heads, seq_len, attn_scale, opts, Call::kDecode);
  if (!r.ok) return 0;
  return r.merge ? 1 : 2;
}

int32_t tq_internal_decode_kernel(const tq_kv_cache* cache, int32_t n_q_heads, int32_t seq_len, float attn_scale,
                                  const tq_decode_opts* opts, int32_t call) {
  const Route r = route_of(cache, n_q_heads, seq_len, attn_scale, opts, call == 0 ? Call::kDecode : call == 1 ? Call::kStep : Call::kLengths);
  return !r.ok ? 0 : r.wide ? 4 : !r.use_mfma ? 1 : r.small_tile ? 2 : 3;
}

int32_t tq_internal_fine_chunks(const tq_kv_cache* cache, int32_t n_q_heads, int32_t tokens, const tq_decode_opts* opts) {
  return fine_splits_of(cache, n_q_heads, opts, cache->n_kv_heads * mfma_share_of(cache, n_q_heads, opts), tokens);
}

int32_t tq_internal_listed_slots(const tq_kv_cache* cache, int32_t n_q_heads, int32_t max_seq_len, float attn_scale, const tq_decode_opts* opts) {
  return listed_slots(cache, n_q_heads, max_seq_len, attn_scale, opts);
}

int32_t tq_internal_lengths_waves(const tq_kv_cache* cache, int32_t n_q_heads, int32_t max_seq_len, float attn_scale, const tq_decode_opts* opts) {
  const Route r = route_of(cache, n_q_heads, max_seq_len, attn_scale, opts, Call::kLengths);
  if (!r.ok || !r.use_mfma || (opts && opts->n_splits > 0)) return 0;
  const int waves = ranked_rows(cache, n_q_heads, max_seq_len, attn_scale, opts).waves;
  return waves > 0 ? waves : -chunk_list(cache->batch, cache->n_kv_heads * mfma_share_of(cache, n_q_heads, opts), kBlocksMfma).waves;
}

int32_t tq_internal_counter_sets_left() { return tq::mfma_merge_slots_left(); }

const char* tq_status_string(int status) {
  switch (status) {
    case TQ_OK: return "ok";
    case TQ_ERR_NULL: return "a required pointer is NULL";
    case TQ_ERR_SHAPE: return "unsupported or inconsistent shape";
    case TQ_ERR_EMPTY: return "empty request (seq_len < 1 or n_new < 1)";
    case TQ_ERR_CAPACITY: return "position or sequence length exceeds the cache capacity";
    case TQ_ERR_WORKSPACE: return "workspace or dense scratch too small";
    case TQ_ERR_UNSUPPORTED: return "shape or option not covered by the kernels";
    case TQ_ERR_HIP: return "HIP runtime error at launch";
    case TQ_ERR_ALIGN: return "pointer not sufficiently aligned";
    default: return "unknown status";
  }
}

int tq_quantize_kv(const tq_kv_cache* cache, const void* k_new, const void* v_new, int32_t pos, int32_t n_new,
                   void* stream) {
  int rc = check_cache(cache);
  if (rc == TQ_ERR_NULL) return rc;
  if (!k_new || !v_new) return TQ_ERR_NULL;
  if (rc != TQ_OK && rc != TQ_ERR_ALIGN) return rc;
  if (n_new < 1) return TQ_ERR_EMPTY;
  if (pos < 0 || (int64_t)pos + n_new > cache->capacity) return TQ_ERR_CAPACITY;
  if (rc == TQ_ERR_ALIGN || !aligned(k_new, 16) || !aligned(v_new, 16)) return TQ_ERR_ALIGN;
  return hip_rc(tq::launch_quantize(*cache, k_new, v_new, pos, nullptr, n_new, static_cast<hipStream_t>(stream)));
}

int tq_quantize_kv_varlen(const tq_kv_cache* cache, const void* k_new, const void* v_new, const int32_t* positions,
                          int32_t n_new, void* stream) {
  int rc = check_cache(cache);
  if (rc == TQ_ERR_NULL) return rc;
  if (!k_new || !v_new || !positions) return TQ_ERR_NULL;
  if (rc != TQ_OK && rc != TQ_ERR_ALIGN) return rc;
  if (n_new < 1) return TQ_ERR_EMPTY;
  if (n_new > cache->capacity) return TQ_ERR_CAPACITY;
  if (rc == TQ_ERR_ALIGN || !aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(positions, 4)) return TQ_ERR_ALIGN;
  return hip_rc(tq::launch_quantize(*cache, k_new, v_new, 0, positions, n_new, static_cast<hipStream_t>(stream)));
}

int tq_sdpa_int4_partial(const tq_kv_cache* cache, const void* q, int32_t n_q_heads, int32_t seq_len,
                         float attn_scale, void* workspace, size_t workspace_bytes, const tq_decode_opts* opts,
                         int32_t* n_splits_out, void* stream) {
  const int rc = check_decode(cache, q, n_q_heads, seq_len, nullptr, workspace, workspace_bytes, opts, false);
  if (rc != TQ_OK) return rc;
  PartialRequest rq{cache, q, n_q_heads, seq_len};
  rq.attn_scale = attn_scale;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.stream = stream;
  const int out_rc = run_partial(rq);
  if (n_splits_out) *n_splits_out = rq.n_splits;
  return out_rc;
}

int tq_sdpa_int4_reduce(int32_t batch, int32_t n_q_heads, int32_t head_dim, int32_t n_splits, const void* workspace,
                        size_t workspace_bytes, void* out, void* stream) {
  if (!workspace || !out) return TQ_ERR_NULL;
  if (batch < 1 || n_q_heads < 1 || !head_dim_ok(head_dim)) return TQ_ERR_SHAPE;
  if (n_splits < 1) return TQ_ERR_EMPTY;
  if (n_splits > tq::kMaxSplits) return TQ_ERR_UNSUPPORTED;
  if (!aligned(workspace, 256) || !aligned(out, 16)) return TQ_ERR_ALIGN;
  if (workspace_bytes < tq_workspace_bytes(batch, n_q_heads, head_dim)) return TQ_ERR_WORKSPACE;
  DecodeParams p{};
  p.part_o = const_cast<float*>(static_cast<const float*>(workspace));
  p.part_ml = p.part_o + tq::workspace_o_floats(batch, n_q_heads, head_dim);
  p.out = static_cast<half_t*>(out);
  p.n_q_heads = n_q_heads;
  p.n_splits = n_splits;
  return hip_rc(tq::launch_reduce(p, batch, head_dim, static_cast<hipStream_t>(stream)));
}

int tq_sdpa_int4_decode(const tq_kv_cache* cache, const void* q, int32_t n_q_heads, int32_t seq_len, float attn_scale,
                        void* out, void* workspace, size_t workspace_bytes, const tq_decode_opts* opts, void* stream) {
  int rc = check_decode(cache, q, n_q_heads, seq_len, out, workspace, workspace_bytes, opts, true);
  if (rc != TQ_OK) return rc;
  PartialRequest rq{cache, q, n_q_heads, seq_len};
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.stream = stream;
  return finish_decode(rq, run_partial(rq));
}

int tq_sdpa_int4_decode_static(const tq_kv_cache* cache, const void* q, int32_t n_q_heads, int32_t seq_len,
                               float attn_scale, void* out, const tq_decode_opts* opts, void* stream) {
  // everything that can be told without the workspace first (a fake, aligned address stands in for it), so that a
  // rejected call touches neither the device nor the runtime
  void* const fake = reinterpret_cast<void*>(uintptr_t{256});
  int rc = check_decode(cache, q, n_q_heads, seq_len, out, fake, ~size_t{0}, opts, true);
  if (rc != TQ_OK) return rc;
  if (tq_workspace_bytes(cache->batch * queries_of(opts), n_q_heads, cache->head_dim) > kScratchBytes)
    return TQ_ERR_WORKSPACE;
  void* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc != TQ_OK) return rc;
  // Nothing in the array has to start at zero: every partial the merge reads has been written by the same call's
  // first phase, and the arrival counters of the one-launch route live elsewhere and reset themselves.
  PartialRequest rq{cache, q, n_q_heads, seq_len};
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = ws;
  rq.opts = opts;
  rq.stream = stream;
  return finish_decode(rq, run_partial(rq));
}

int tq_sdpa_int4_append_decode(const tq_kv_cache* cache, const void* k_new, const void* v_new, const void* q,
                               int32_t n_q_heads, int32_t seq_len, float attn_scale, void* out, void* workspace,
                               size_t workspace_bytes, const tq_decode_opts* opts, void* stream) {
  int rc = check_decode(cache, q, n_q_heads, seq_len, out, workspace, workspace_bytes, opts, true);
  if (rc != TQ_OK) return rc;
  if (!k_new || !v_new) return TQ_ERR_NULL;
  if (!aligned(k_new, 16) || !aligned(v_new, 16)) return TQ_ERR_ALIGN;
  const Route r = route_of(cache, n_q_heads, seq_len, attn_scale, opts, Call::kStep);
  if (!r.ok) return TQ_ERR_UNSUPPORTED;
  PartialRequest rq{cache, q, n_q_heads, seq_len};
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.stream = stream;
  rq.step = true;
  // The matrix-core kernel takes the token in, or the merge kernel behind it or the others (there with groups of 32
  // only); one query token, at least one cached token to attend: no append launch, nothing read back.  Else the
  // append kernel runs first (also for a tile that takes no token and writes the output itself).
  const bool taken_in = r.use_mfma ? !r.merge_step || takes_token(cache, n_q_heads, opts) : cache->group_size == tq::kGroup;
  if (r.wide) {                                   // (any number of query tokens, the sequence's first token too)
    rq.k_new = k_new;
    rq.v_new = v_new;
    rq.new_in_chunks = true;
  } else if (queries_of(opts) == 1 && windowed(seq_len, opts) >= 2 && taken_in) {
    rq.k_new = k_new;
    rq.v_new = v_new;
  } else {                                        // the append kernel first, then the plain decode
    const int n_new = queries_of(opts);
    rc = hip_rc(tq::launch_quantize(*cache, k_new, v_new, seq_len - n_new, nullptr, n_new,
                                    static_cast<hipStream_t>(stream)));
    if (rc != TQ_OK) return rc;
  }
  return finish_decode(rq, run_partial(rq));
}

int tq_quantize_kv_paged(const tq_kv_cache* pool, const int32_t* block_table, int32_t max_blocks, int32_t batch,
                         const void* k_new, const void* v_new, const int32_t* positions, int32_t n_new, void* stream) {
  tq_kv_cache view;
  tq::PagedView pv;
  const int rc = paged_view(pool, block_table, max_blocks, batch, &view, &pv);
  if (rc != TQ_OK) return rc;
  if (!k_new || !v_new || !positions) return TQ_ERR_NULL;
  if (n_new < 1) return TQ_ERR_EMPTY;
  if ((int64_t)n_new > (int64_t)max_blocks * pool->capacity) return TQ_ERR_CAPACITY;
  if (!aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(positions, 4)) return TQ_ERR_ALIGN;
  return hip_rc(tq::launch_quantize(view, k_new, v_new, 0, positions, n_new, static_cast<hipStream_t>(stream), &pv));
}

int tq_sdpa_int4_decode_paged(const tq_kv_cache* pool, const int32_t* block_table, int32_t max_blocks, int32_t batch,
                              const void* q, int32_t n_q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                              float attn_scale, void* out, void* workspace, size_t workspace_bytes,
                              const tq_decode_opts* opts, void* stream) {
  tq_kv_cache view;
  tq::PagedView pv;
  int rc = paged_view(pool, block_table, max_blocks, batch, &view, &pv);
  if (rc != TQ_OK) return rc;
  rc = check_decode(&view, q, n_q_heads, max_seq_len, out, workspace, workspace_bytes, opts, true,
                    (int64_t)max_blocks * pool->capacity);
  if (rc != TQ_OK) return rc;
  if (!seq_lens) return TQ_ERR_NULL;
  if (!aligned(seq_lens, 4)) return TQ_ERR_ALIGN;
  PartialRequest rq{&view, q, n_q_heads, max_seq_len};
  rq.seq_lens = seq_lens;
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.paged = &pv;
  rq.stream = stream;
  return finish_decode(rq, run_partial(rq));
}

namespace {
// One decode step with per-sequence lengths that count the step's new token: the matrix-core kernel (or the merge
// kernel behind the others) takes the token in where it can (one query token; a window, if any, of at least two
// tokens), else the append kernel runs first.
int append_decode_with_lengths(PartialRequest& rq, const void* k_new, const void* v_new) {
  const tq_decode_opts* opts = rq.opts;
  const bool taken_in = route_of(rq.cache, rq.n_q_heads, rq.seq_len, rq.attn_scale, opts, Call::kLengths).use_mfma
                            ? takes_token(rq.cache, rq.n_q_heads, opts) ||
                                  ranked_rows(rq.cache, rq.n_q_heads, rq.seq_len, rq.attn_scale, opts).waves == 0
                            : rq.cache->group_size == tq::kGroup;
  if (queries_of(opts) == 1 && !(opts && opts->window == 1) && rq.seq_len >= 2 && taken_in) {
    rq.k_new = k_new;
    rq.v_new = v_new;
  } else {
    const int n_new = queries_of(opts);
    const int rc = hip_rc(tq::launch_quantize(*rq.cache, k_new, v_new, -n_new, rq.seq_lens, n_new,
                                              static_cast<hipStream_t>(rq.stream), rq.paged));
    if (rc != TQ_OK) return rc;
  }
  return finish_decode(rq, run_partial(rq));
}
}  // namespace

int tq_sdpa_int4_append_decode_varlen(const tq_kv_cache* cache, const void* k_new, const void* v_new, const void* q,
                                      int32_t n_q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                                      float attn_scale, void* out, void* workspace, size_t workspace_bytes,
                                      const tq_decode_opts* opts, void* stream) {
  int rc = check_decode(cache, q, n_q_heads, max_seq_len, out, workspace, workspace_bytes, opts, true);
  if (rc != TQ_OK) return rc;
  if (!seq_lens || !k_new || !v_new) return TQ_ERR_NULL;
  if (!aligned(seq_lens, 4) || !aligned(k_new, 16) || !aligned(v_new, 16)) return TQ_ERR_ALIGN;
  if (!route_of(cache, n_q_heads, max_seq_len, attn_scale, opts, Call::kLengths).ok) return TQ_ERR_UNSUPPORTED;
  PartialRequest rq{cache, q, n_q_heads, max_seq_len};
  rq.seq_lens = seq_lens;
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.stream = stream;
  return append_decode_with_lengths(rq, k_new, v_new);
}

int tq_sdpa_int4_append_decode_paged(const tq_kv_cache* pool, const int32_t* block_table, int32_t max_blocks,
                                     int32_t batch, const void* k_new, const void* v_new, const void* q,
                                     int32_t n_q_heads, const int32_t* seq_lens, int32_t max_seq_len,
                                     float attn_scale, void* out, void* workspace, size_t workspace_bytes,
                                     const tq_decode_opts* opts, void* stream) {
  tq_kv_cache view;
  tq::PagedView pv;
  int rc = paged_view(pool, block_table, max_blocks, batch, &view, &pv);
  if (rc != TQ_OK) return rc;
  rc = check_decode(&view, q, n_q_heads, max_seq_len, out, workspace, workspace_bytes, opts, true,
                    (int64_t)max_blocks * pool->capacity);
  if (rc != TQ_OK) return rc;
  if (!seq_lens || !k_new || !v_new) return TQ_ERR_NULL;
  if (!aligned(seq_lens, 4) || !aligned(k_new, 16) || !aligned(v_new, 16)) return TQ_ERR_ALIGN;
  if (!route_of(&view, n_q_heads, max_seq_len, attn_scale, opts, Call::kLengths).ok) return TQ_ERR_UNSUPPORTED;
  PartialRequest rq{&view, q, n_q_heads, max_seq_len};
  rq.seq_lens = seq_lens;
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.paged = &pv;
  rq.stream = stream;
  return append_decode_with_lengths(rq, k_new, v_new);
}

int tq_sdpa_int4_decode_varlen(const tq_kv_cache* cache, const void* q, int32_t n_q_heads, const int32_t* seq_lens,
                               int32_t max_seq_len, float attn_scale, void* out, void* workspace,
                               size_t workspace_bytes, const tq_decode_opts* opts, void* stream) {
  int rc = check_decode(cache, q, n_q_heads, max_seq_len, out, workspace, workspace_bytes, opts, true);
  if (rc != TQ_OK) return rc;
  if (!seq_lens) return TQ_ERR_NULL;
  if (!aligned(seq_lens, 4)) return TQ_ERR_ALIGN;
  PartialRequest rq{cache, q, n_q_heads, max_seq_len};
  rq.seq_lens = seq_lens;
  rq.attn_scale = attn_scale;
  rq.out = out;
  rq.workspace = workspace;
  rq.opts = opts;
  rq.stream = stream;
  return finish_decode(rq, run_partial(rq));       // the merge works out from the same lengths which chunks exist
}

int tq_dequant_then_attend(const tq_kv_cache* cache, const void* q, int32_t n_q_heads, int32_t seq_len,
                           float attn_scale, void* out, void* workspace, size_t workspace_bytes, void* dense_scratch,
                           size_t dense_scratch_bytes, const tq_decode_opts* opts, void* stream) {
  int rc = check_decode(cache, q, n_q_heads, seq_len, out, workspace, workspace_bytes, opts, true);
  if (rc != TQ_OK) return rc;
  if (!dense_scratch) return TQ_ERR_NULL;
  if (!aligned(dense_scratch, 16)) return TQ_ERR_ALIGN;
  const size_t need = tq_dense_scratch_bytes(cache->batch, cache->n_kv_heads, seq_len, cache->head_dim);
  if (dense_scratch_bytes < need) return TQ_ERR_WORKSPACE;
  if (opts && (opts->window > 0 || opts->n_queries > 1)) return TQ_ERR_UNSUPPORTED;
  hipStream_t s = static_cast<hipStream_t>(stream);
  half_t* k_dense = static_cast<half_t*>(dense_scratch);
  half_t* v_dense = k_dense + need / sizeof(half_t) / 2;
  rc = hip_rc(tq::launch_dequant_dense(*cache, seq_len, k_dense, v_dense, s));
  if (rc != TQ_OK) return rc;
  // attention over the dense tensors: on the matrix cores where that kernel covers the shape (variant 1 asks for
  // the generic vector-ALU kernel), one block per compute unit and at least a supertile per wave
  const bool on_mfma = !(opts && opts->variant == 1) && attn_scale > 0.0f && std::isfinite(attn_scale) &&
                       tq::dense_mfma_supported(cache->head_dim, n_q_heads / cache->n_kv_heads);
  const Plan plan = on_mfma ? plan_splits(cache->batch, cache->n_kv_heads, seq_len, opts ? opts->n_splits : 0,
                                          kBlocksMfma, tq::dense_mfma_waves(cache->head_dim))
                            : plan_splits(cache->batch, cache->n_kv_heads, seq_len, opts ? opts->n_splits : 0,
                                          kBlocksValu, 1);
  DecodeParams p = make_params(cache, q, n_q_heads, seq_len, attn_scale, out, workspace, plan);
  p.k_dense = k_dense;
  p.v_dense = v_dense;
  p.row_stride = seq_len;                  // the dense buffers are packed to seq_len rows
  rc = hip_rc(on_mfma ? tq::launch_partial_dense_mfma(p, cache->batch, cache->head_dim, s)
                      : tq::launch_partial_valu(p, cache->batch, cache->head_dim, true, s));
  if (rc != TQ_OK) return rc;
  return hip_rc(tq::launch_reduce(p, cache->batch, cache->head_dim, s));
}

}  // extern "C"
