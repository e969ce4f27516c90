// C ABI of the LazyAttention hot path: argument checks, launch configuration and dispatch to the HIP kernels.
// The library never allocates device memory and never synchronises; every launch goes to the caller's stream.
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "lazy_attn.h"
#include "lazy_attn_internal.h"

namespace {

constexpr int kNumCUs = 256;              // MI355X compute units

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int check_params(const lazy_attn_params_t* p) {
  if (!p) return LAZY_EINVAL;
  if (p->num_q_heads <= 0 || p->num_kv_heads <= 0 || p->num_q_heads % p->num_kv_heads != 0) return LAZY_EINVAL;
  if (p->causal != 0 && p->causal != 1) return LAZY_EINVAL;
  if (!isfinite(p->softmax_scale) || p->softmax_scale < 0.f) return LAZY_EINVAL;
  if (p->rope_style != LAZY_ALIBI && !p->inv_freq && !(isfinite(p->rope_base) && p->rope_base > 0.f)) return LAZY_EINVAL;
  if (p->num_splits < 0) return LAZY_EINVAL;
  if (p->key_positions != LAZY_KEYS_NOPE && p->key_positions != LAZY_KEYS_LOCAL) return LAZY_EINVAL;
  if (p->rope_style != LAZY_ROPE_HALF && p->rope_style != LAZY_ROPE_INTERLEAVED && p->rope_style != LAZY_ALIBI)
    return LAZY_EINVAL;
  if (p->rope_style == LAZY_ALIBI && p->key_positions != LAZY_KEYS_NOPE) return LAZY_EINVAL;
  if (p->q_prerotated != 0 && p->q_prerotated != 1) return LAZY_EINVAL;
  if (p->cache_hint != LAZY_CACHE_DEFAULT && p->cache_hint != LAZY_CACHE_STREAM) return LAZY_EINVAL;
  if (p->head_dim != 64 && p->head_dim != 128) return LAZY_EUNSUPPORTED;
  return LAZY_OK;
}

float scale_log2(const lazy_attn_params_t* p) {
  const float s = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->head_dim);
  return s * 1.4426950408889634f;
}

// 256 packed rows per workgroup (eight waves, one workgroup per CU; head_dim 128 only) once a request has enough
// rows; otherwise 128 rows (four waves, two workgroups per CU).  Must match the kernel chosen in launch_prefill.
int prefill_row_blocks(const lazy_attn_params_t* p, int32_t max_q_len) {
  const int64_t g = p->num_q_heads / p->num_kv_heads;
  return p->head_dim == 128 && (int64_t)max_q_len * g >= 2 * lazy::kPrefillRowsPerBlock ? 2 : 1;
}

int prefill_q_tiles(const lazy_attn_params_t* p, int32_t max_q_len) {
  const int64_t g = p->num_q_heads / p->num_kv_heads;
  return (int)ceil_div((int64_t)max_q_len * g, (int64_t)lazy::kPrefillRowsPerBlock * prefill_row_blocks(p, max_q_len));
}

// A batch is ragged when its mean query length is below 3/4 of the maximum.
bool prefill_ragged(int32_t batch, int32_t total_q, int32_t max_q_len) {
  return 4 * (int64_t)total_q < 3 * (int64_t)batch * max_q_len;
}

// Split-KV workspace: bf16 normalised partial outputs [splits][rows][d], then fp32 partial lse [splits][rows]
// (16-byte aligned because d is a multiple of 8).
size_t split_workspace(int splits, int64_t rows, int d) {
  if (splits <= 1) return 0;
  return (size_t)splits * (size_t)rows * ((size_t)d * sizeof(uint16_t) + sizeof(float));
}

// Workgroups per KV split that have rows to work on.  Row tiles of the batch: exact where all requests are as long as
// the longest, else the rows' tiles and on average half a tile per request for its last one, and at least one each.
int64_t prefill_busy(const lazy_attn_params_t* p, int32_t batch, int32_t total_q, int32_t max_q_len) {
  const int64_t g = p->num_q_heads / p->num_kv_heads;
  const int64_t rows_per_tile = (int64_t)lazy::kPrefillRowsPerBlock * prefill_row_blocks(p, max_q_len);
  const int64_t most = (int64_t)batch * prefill_q_tiles(p, max_q_len);
  const int64_t row_tiles =
      (int64_t)total_q >= (int64_t)batch * max_q_len
          ? most
          : std::min(most, std::max<int64_t>(batch, ceil_div((int64_t)total_q * g, rows_per_tile) + batch / 2));
  return row_tiles * p->num_kv_heads;
}

// KV splits per request.  Workgroups are (query tile, KV head, request, split); those of a query tile past the end of a
// shorter request exit at once, which leaves `busy` per split in a ragged batch.  Where the lengths are nearly equal
// all that are launched count, with rows or without, since a launch of more than a round's workgroups begins a second
// round on some XCDs (two requests of 102 queries and 27K keys, 40 / 8 heads, 32 workgroups of which 24 have rows:
// eight splits 155 us, nine 262).  A CU holds `per_cu` of them: one of 256 rows (LDS), two of 128 rows, three with
// head_dim 64.  The count is the one with the least estimated time, in key tiles:
//     sharing * rounds * (tiles per split + prologue) + merge,    rounds = ceil(busy * splits / (256 per_cu)).
// Until its first tile is done and at its end a workgroup spends about as long as on kPrologueTiles tiles; two or three
// workgroups on a CU take 1.2 or 1.35 times as long each as one alone; a split batch is merged by a second launch.  A
// count just past a full round runs the last one nearly empty.  Tiles: max_kv_len / 64, with 15% more for records that
// end in a partial tile.
//
// Ragged query lengths (mean below 3/4 of the maximum) usually come with ragged key lengths, which the call does not
// tell.  A launch of no more than one round, empty workgroups among them, takes as long as its longest one: 1.4 per +
// 4, per = max_kv_len / (64 splits).  A larger one takes 0.6 per + 7 for the average workgroup, times the rounds that
// the busy ones make with 1.3 to a slot (shorter ones make room early), and 0.85 per + 4 for the longest at the end.
// Just past one round the time jumps by up to half (three requests of up to 41 queries and 2.6K keys, 28 / 4 heads, 24
// workgroups: ten splits 36 us, eleven 54).
//
// The constants are a fit over split sweeps of 5983 batches (128 and 256 rows, head_dim 64 and 128, all key modes,
// contiguous and paged, 8 to 6775 tiles), checked on 4476 others: the chosen count is 3.7% off each batch's best of 1
// to 64 on average, 1.9% if equal or nearly so and 5.8% if ragged.  One round for equal and three for ragged query
// lengths, with at least four tiles a split, is 18% off: one request of 22 tiles, busy 8, five splits 23.5 us, twenty
// 19.3; 8 requests of 95 tiles at head_dim 64, busy 256, one to four splits 178 / 126 / 107 / 123 us; ragged, busy 176,
// 81 tiles, fifteen and five splits 153 / 127 us.  4% of the batches are more than 5% faster that way.  Close estimates
// are worth following: the least count within 3% of the least estimate would be 1.7% slower over the equal batches and
// 0.3% over the ragged ones, and nine requests of 2340 tiles at head_dim 64 get seventeen splits on 1.7% less than for
// two, and take 3.01 ms instead of 3.44.  Longer batches than the fitted ones, eight of equal requests with 1030 to
// 2340 tiles: within 2% of the best of one to seventeen splits, on one 9% off.  Still missed: how the keys are spread
// over a ragged batch's requests, and records much shorter than a tile.
constexpr double kPrologueTiles = 8, kMergeTiles = 3, kMergeTilesPerSplit = 0.05;
constexpr double kSharing[4] = {1, 1, 1.2, 1.35};
constexpr int64_t kMaxSplits = 64;
// A split batch's outputs pass through bf16 partials, an unsplit one's are rounded once (one request of 8 tiles, seven
// splits: error against 64 bits 0.0035 instead of 0.0032).  A batch with fewer than kSplitTiles tiles, or whose rows alone
// fill the chip (three times over if ragged), is therefore never split, also where it would be faster so (40 requests of
// 83 tiles, busy 320: 342 us, two splits 296).
constexpr int64_t kSplitTiles = 8;
// Past the fitted lengths every further split of a ragged batch looks a little cheaper, and the partials would reach
// 1 GB; they are held to LAZY_PREFILL_WORKSPACE_MAX.  The rows of a batch that may be split (above) are less than 768
// tiles of 256 or 1536 of 128, 51 MB a split at most, so at least five splits fit.  Four requests of 96-143K keys, six
// splits under it and sixteen without: 10.3 and 10.1 ms; 32 requests of 94-147K keys, seven and eleven: 14.0 and 14.0 ms.

int prefill_splits(const lazy_attn_params_t* p, int32_t batch, int32_t total_q, int32_t max_q_len,
                   int32_t max_kv_len) {
  if (p->num_splits > 0) return p->num_splits;
  const int per_cu = prefill_row_blocks(p, max_q_len) == 2 ? 1 : p->head_dim == 64 ? 3 : 2;
  const int64_t tiles = std::max<int64_t>(1, ceil_div(max_kv_len, lazy::kPrefillTileKeys));
  const bool ragged = prefill_ragged(batch, total_q, max_q_len);
  const double launched = (double)batch * prefill_q_tiles(p, max_q_len) * p->num_kv_heads;
  const double busy = ragged ? (double)prefill_busy(p, batch, total_q, max_q_len) : launched;
  const double slots = (double)(kNumCUs * per_cu);
  const int64_t rows = (int64_t)total_q * (p->num_q_heads / p->num_kv_heads);
  const int64_t per_tile = (int64_t)lazy::kPrefillRowsPerBlock * prefill_row_blocks(p, max_q_len);
  const int64_t full = (int64_t)kNumCUs * (per_cu == 1 ? 1 : 2) * (ragged ? 3 : 1);
  if (tiles < kSplitTiles || p->num_kv_heads * ceil_div(rows, per_tile) >= full) return 1;
  const int64_t per_split = (int64_t)split_workspace(2, (int64_t)total_q * p->num_q_heads, p->head_dim) / 2;
  const int64_t most =
      std::min({tiles, kMaxSplits, (int64_t)LAZY_PREFILL_WORKSPACE_MAX / std::max<int64_t>(1, per_split)});
  int64_t best = 1;
  double least = 0;
  for (int64_t s = 1; s <= most; ++s) {
    const double groups = busy * (double)s, per = (double)tiles / (double)s;
    const double sharing = kSharing[(int)std::min((double)per_cu, std::ceil(groups / kNumCUs))];
    const double merge = s > 1 ? kMergeTiles + kMergeTilesPerSplit * (double)s : 0;
    double cost;
    if (!ragged)
      cost = std::ceil(groups / slots) * ((1.15 * (double)tiles + 1) / (double)s + kPrologueTiles);
    else if (launched * (double)s <= slots)
      cost = 1.4 * per + 4;
    else
      cost = std::max(1.0, groups / (1.3 * slots)) * (0.6 * per + 7) + 0.85 * per + 4;
    cost = sharing * cost + merge;
    if (s == 1 || cost < least) {
      best = s;
      least = cost;
    }
  }
  // A ragged batch is not left in one piece otherwise (busy 240, 9 tiles: 127 us with one split, 121 with two; busy 239,
  // 13 tiles: 83 and 90 us).
  if (ragged && best == 1) best = 2;
  // The grid's z axis holds batch x splits.
  return (int)std::max<int64_t>(1, std::min<int64_t>(best, batch > 0 ? 65535 / batch : best));
}

// Which workgroups of a ragged prefill stay together on an XCD.  One unit per KV head evens out the XCDs, one per request
// and split reads its table once: the former from kUnitHeadsTiles tiles a split.  Four requests of 96-143K keys, two to
// eight splits: 14.3 / 11.8 / 14.4 / 11.1 / 12.2 / 11.0 / 9.8 ms by request, 10.8 / 11.1 / 10.4 / 10.2 / 10.3 / 10.2 /
// 10.1 by head (eight splits put a part of each request on every XCD); 16 requests of up to 27.6K keys in five, eight and
// nine splits (86, 54 and 48 tiles) 899 / 807 / 832 us by request, 822 / 794 / 811 by head.  Over 13148 ragged batches and
// split counts by head is 0.3% slower under 2 tiles a split, 0.4% faster at 2 to 4, 0.9% at 4 to 8, 1.4% at 8 to 16, 1.5%
// at 16 to 48 (a quarter of the batches gain more than 2%, one in thirty loses that) and 2.2% beyond; the line is not at
// the crossing because short splits gain little and some lose (16 requests of 4.7K keys in seven, 10 tiles: 122.6 -> 123.5
// us).
constexpr int64_t kUnitHeadsTiles = 16;

int prefill_units(int32_t batch, int32_t total_q, int32_t max_q_len, int32_t max_kv_len, int splits) {
  if (!prefill_ragged(batch, total_q, max_q_len)) return lazy::kUnitNone;
  return max_kv_len / lazy::kPrefillTileKeys >= kUnitHeadsTiles * splits ? lazy::kUnitHeads : lazy::kUnitRequests;
}

int decode_head_groups(const lazy_attn_params_t* p) {
  const int g = p->num_q_heads / p->num_kv_heads;
  return (g + lazy::kDecodeHeadsPerGroup - 1) / lazy::kDecodeHeadsPerGroup;
}

int decode_splits(const lazy_attn_params_t* p, int32_t batch, int32_t max_kv_len) {
  if (p->num_splits > 0) return p->num_splits;
  // Two streaming workgroups per CU; split only when the batch alone cannot fill the chip.
  const int64_t base = (int64_t)batch * p->num_kv_heads * decode_head_groups(p);
  const int64_t tiles = ceil_div(max_kv_len, lazy::kDecodeTileKeys);
  int64_t s = base > 0 ? ceil_div(2 * kNumCUs, base) : 1;
  const int64_t cap = tiles / 2 > 1 ? tiles / 2 : 1;
  if (s > cap) s = cap;
  if (s > 64) s = 64;
  return s < 1 ? 1 : (int)s;
}

// Requests that share chunks list them in orders of their own, so each reads them at another time and the caches hold
// little for the next.  The decode therefore walks a request's records in the order their values are stored (outputs
// change only in the order of the sums): four requests over one pool of 128 exemplars, 33K keys each, 84.1 -> 63.2 us a
// step; 64 requests with sixteen of 256 chunks of 1024 keys, 583 -> 526 us; with the stream hint 88.6 -> 80.7 and 622
// -> 608.  Sorting takes a workgroup 1-2 us and finding that there is nothing to sort, or that the request has its
// chunks for itself, 0.3-0.9 us (four private contexts of 33K keys in order 102.2 -> 103.0 us, shuffled 99.5 -> 100.2,
// with the stream hint 92.4 -> 92.7 and 90.8 -> 91.1; at head_dim 64 54.8 -> 55.2 and 55.6 -> 56.0; 64 of 4K 185.9 ->
// 186.6; tables of 560 and 620 blocks of 32 keys 147.5 -> 148.6 and 127.6 -> 129.2), so it is left out where that shows:
// one request, or under 1536 keys per split (10K keys in 16 splits: 20.8 -> 21.3 us; 52 requests of 6.4K keys in 5 splits,
// in order: 36.8 -> 38.1 us; two requests of 2.6K keys in 13 splits: 16.9 -> 17.3 us).  The cache hint has no say: it must
// not change a result.
bool decode_sorted(int32_t batch, int splits, int32_t max_kv_len) {
  return batch > 1 && max_kv_len / splits >= 1536;
}

int status(hipError_t e) { return e == hipSuccess ? LAZY_OK : LAZY_EHIP; }

int run_prefill(bool rotate_k, const lazy_attn_params_t* p, const void* q, const int32_t* q_start,
                const int32_t* q_pos0, const void* k_pool, const void* v_pool, const lazy_chunk_t* chunks,
                const int32_t* chunk_start, int32_t batch, int32_t total_q, int32_t max_q_len, int32_t max_kv_len,
                void* out, float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  int e = check_params(p);
  if (e != LAZY_OK) return e;
  if (!rotate_k && p->rope_style == LAZY_ALIBI) return LAZY_EUNSUPPORTED;  // no materialised copy for ALiBi
  if (batch < 0 || total_q < 0 || max_q_len < 0 || max_kv_len < 0) return LAZY_EINVAL;
  if (batch == 0 || total_q == 0) return LAZY_OK;
  if (max_q_len == 0) return LAZY_EINVAL;
  if (!q || !q_start || !q_pos0 || !k_pool || !v_pool || !chunks || !chunk_start || !out) return LAZY_EINVAL;
  const int splits = prefill_splits(p, batch, total_q, max_q_len, max_kv_len);
  const int q_tiles = prefill_q_tiles(p, max_q_len);
  if ((int64_t)batch * splits > 65535 || p->num_kv_heads > 65535) return LAZY_EUNSUPPORTED;
  const int64_t rows = (int64_t)total_q * p->num_q_heads;
  const size_t need = split_workspace(splits, rows, p->head_dim);
  if (need > 0 && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 15u))) return LAZY_EWORKSPACE;

  lazy::AttnArgs a = {};
  a.q = static_cast<const uint16_t*>(q);
  a.q_start = q_start;
  a.q_pos0 = q_pos0;
  a.k_pool = static_cast<const uint16_t*>(k_pool);
  a.v_pool = static_cast<const uint16_t*>(v_pool);
  a.chunks = chunks;
  a.chunk_start = chunk_start;
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.ws_o = need ? static_cast<uint16_t*>(workspace) : nullptr;
  a.ws_lse = need ? reinterpret_cast<float*>(static_cast<uint16_t*>(workspace) + (size_t)splits * rows * p->head_dim)
                  : nullptr;
  a.inv_freq = p->inv_freq;
  a.batch = batch;
  a.total_q = total_q;
  a.hq = p->num_q_heads;
  a.hkv = p->num_kv_heads;
  a.group = p->num_q_heads / p->num_kv_heads;
  a.causal = p->causal;
  a.splits = splits;
  a.q_tiles = q_tiles;
  a.row_blocks = prefill_row_blocks(p, max_q_len);
  // Three workgroups a CU (head_dim 64) where the launch has more than two for each; below that the third wave's tighter
  // register allotment (a few spills) only costs (39 requests of up to 5 tiles, 320 workgroups: 23.3 against 21.5 us).
  a.crowded = prefill_busy(p, batch, total_q, max_q_len) * splits > 2 * kNumCUs;
  // Ragged batches spread units over the XCDs; alike requests keep whole requests per XCD.
  a.xcd_interleave = prefill_units(batch, total_q, max_q_len, max_kv_len, splits);
  a.head_groups = 1;
  a.rope_log2_base = p->inv_freq || p->rope_style == LAZY_ALIBI ? 0.0 : log2((double)p->rope_base);
  a.scale_log2 = scale_log2(p);
  a.local_keys = p->key_positions == LAZY_KEYS_LOCAL;
  a.interleaved = p->rope_style == LAZY_ROPE_INTERLEAVED;
  a.alibi = p->rope_style == LAZY_ALIBI;
  a.q_prerot = p->q_prerotated && p->rope_style != LAZY_ALIBI;
  return status(lazy::launch_prefill(a, p->head_dim, rotate_k, static_cast<hipStream_t>(stream)));
}

int run_decode(bool rotate_k, const lazy_attn_params_t* p, const void* q, const int32_t* q_pos, const void* k_pool,
               const void* v_pool, const lazy_chunk_t* chunks, const int32_t* chunk_start, int32_t batch,
               int32_t max_kv_len, void* out, float* lse, void* workspace, size_t workspace_bytes, void* stream) {
  int e = check_params(p);
  if (e != LAZY_OK) return e;
  if (!rotate_k && p->rope_style == LAZY_ALIBI) return LAZY_EUNSUPPORTED;
  if (batch < 0 || max_kv_len < 0) return LAZY_EINVAL;
  if (batch == 0) return LAZY_OK;
  if (!q || !q_pos || !k_pool || !v_pool || !chunks || !chunk_start || !out) return LAZY_EINVAL;
  const int splits = decode_splits(p, batch, max_kv_len);
  const int hg = decode_head_groups(p);
  if (batch > 65535 || (int64_t)p->num_kv_heads * hg > 65535) return LAZY_EUNSUPPORTED;
  const int64_t rows = (int64_t)batch * p->num_q_heads;
  const size_t need = split_workspace(splits, rows, p->head_dim);
  if (need > 0 && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 15u))) return LAZY_EWORKSPACE;

  lazy::AttnArgs a = {};
  a.q = static_cast<const uint16_t*>(q);
  a.q_start = nullptr;
  a.q_pos0 = q_pos;
  a.k_pool = static_cast<const uint16_t*>(k_pool);
  a.v_pool = static_cast<const uint16_t*>(v_pool);
  a.chunks = chunks;
  a.chunk_start = chunk_start;
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.ws_o = need ? static_cast<uint16_t*>(workspace) : nullptr;
  a.ws_lse = need ? reinterpret_cast<float*>(static_cast<uint16_t*>(workspace) + (size_t)splits * rows * p->head_dim)
                  : nullptr;
  a.inv_freq = p->inv_freq;
  a.batch = batch;
  a.total_q = batch;
  a.hq = p->num_q_heads;
  a.hkv = p->num_kv_heads;
  a.group = p->num_q_heads / p->num_kv_heads;
  a.causal = p->causal;
  a.splits = splits;
  a.q_tiles = 1;
  a.row_blocks = 1;
  a.head_groups = hg;
  a.rope_log2_base = p->inv_freq || p->rope_style == LAZY_ALIBI ? 0.0 : log2((double)p->rope_base);
  a.scale_log2 = scale_log2(p);
  a.local_keys = p->key_positions == LAZY_KEYS_LOCAL;
  a.interleaved = p->rope_style == LAZY_ROPE_INTERLEAVED;
  a.alibi = p->rope_style == LAZY_ALIBI;
  a.q_prerot = p->q_prerotated && p->rope_style != LAZY_ALIBI;
  a.stream_kv = p->cache_hint == LAZY_CACHE_STREAM;
  a.sort_records = decode_sorted(batch, splits, max_kv_len);
  return status(lazy::launch_decode(a, p->head_dim, rotate_k, static_cast<hipStream_t>(stream)));
}

}  // namespace

extern "C" {

size_t lazy_attn_prefill_workspace_size(const lazy_attn_params_t* params, int32_t batch, int32_t total_q,
                                        int32_t max_q_len, int32_t max_kv_len) {
  if (check_params(params) != LAZY_OK || batch <= 0 || total_q <= 0 || max_q_len <= 0 || max_kv_len < 0) return 0;
  const int splits = prefill_splits(params, batch, total_q, max_q_len, max_kv_len);
  return split_workspace(splits, (int64_t)total_q * params->num_q_heads, params->head_dim);
}

size_t lazy_attn_decode_workspace_size(const lazy_attn_params_t* params, int32_t batch, int32_t max_kv_len) {
  if (check_params(params) != LAZY_OK || batch <= 0 || max_kv_len < 0) return 0;
  const int splits = decode_splits(params, batch, max_kv_len);
  return split_workspace(splits, (int64_t)batch * params->num_q_heads, params->head_dim);
}

int lazy_attn_prefill(const lazy_attn_params_t* params, const void* q, const int32_t* q_start,
                      const int32_t* q_pos0, const void* k_pool, const void* v_pool, const lazy_chunk_t* chunks,
                      const int32_t* chunk_start, int32_t batch, int32_t total_q, int32_t max_q_len,
                      int32_t max_kv_len, void* out, float* lse, void* workspace, size_t workspace_bytes,
                      void* stream) {
  return run_prefill(true, params, q, q_start, q_pos0, k_pool, v_pool, chunks, chunk_start, batch, total_q,
                     max_q_len, max_kv_len, out, lse, workspace, workspace_bytes, stream);
}

int lazy_plain_attn_prefill(const lazy_attn_params_t* params, const void* q, const int32_t* q_start,
                            const int32_t* q_pos0, const void* k_pool, const void* v_pool,
                            const lazy_chunk_t* chunks, const int32_t* chunk_start, int32_t batch, int32_t total_q,
                            int32_t max_q_len, int32_t max_kv_len, void* out, float* lse, void* workspace,
                            size_t workspace_bytes, void* stream) {
  return run_prefill(false, params, q, q_start, q_pos0, k_pool, v_pool, chunks, chunk_start, batch, total_q,
                     max_q_len, max_kv_len, out, lse, workspace, workspace_bytes, stream);
}

int lazy_attn_decode(const lazy_attn_params_t* params, const void* q, const int32_t* q_pos, const void* k_pool,
                     const void* v_pool, const lazy_chunk_t* chunks, const int32_t* chunk_start, int32_t batch,
                     int32_t max_kv_len, void* out, float* lse, void* workspace, size_t workspace_bytes,
                     void* stream) {
  return run_decode(true, params, q, q_pos, k_pool, v_pool, chunks, chunk_start, batch, max_kv_len, out, lse,
                    workspace, workspace_bytes, stream);
}

int lazy_plain_attn_decode(const lazy_attn_params_t* params, const void* q, const int32_t* q_pos,
                           const void* k_pool, const void* v_pool, const lazy_chunk_t* chunks,
                           const int32_t* chunk_start, int32_t batch, int32_t max_kv_len, void* out, float* lse,
                           void* workspace, size_t workspace_bytes, void* stream) {
  return run_decode(false, params, q, q_pos, k_pool, v_pool, chunks, chunk_start, batch, max_kv_len, out, lse,
                    workspace, workspace_bytes, stream);
}

int lazy_attn_decode_noalloc(const lazy_attn_params_t* params, const void* q, const int32_t* q_pos,
                             const void* k_pool, const void* v_pool, const lazy_chunk_t* chunks,
                             const int32_t* chunk_start, int32_t batch, int32_t max_kv_len, void* out, float* lse,
                             void* stream) {
  const int e = check_params(params);
  if (e != LAZY_OK) return e;
  if (batch < 0 || max_kv_len < 0) return LAZY_EINVAL;
  if (batch == 0) return LAZY_OK;
  const size_t need = lazy_attn_decode_workspace_size(params, batch, max_kv_len);
  if (need > (size_t)LAZY_NOALLOC_SCRATCH_BYTES) return LAZY_EWORKSPACE;
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess) return LAZY_EHIP;
  if (stream) {
    hipDevice_t sd = -1;
    if (hipStreamGetDevice(static_cast<hipStream_t>(stream), &sd) != hipSuccess) return LAZY_EHIP;
    if (sd != device) return LAZY_EINVAL;
  }
  void* ws = nullptr;
  if (lazy::noalloc_scratch(device, &ws) != hipSuccess) return LAZY_EHIP;
  return run_decode(true, params, q, q_pos, k_pool, v_pool, chunks, chunk_start, batch, max_kv_len, out, lse, ws,
                    (size_t)LAZY_NOALLOC_SCRATCH_BYTES, stream);
}

int lazy_attn_combine(const void* part_o, const float* part_lse, int32_t splits, int32_t rows, int32_t head_dim,
                      void* out, float* lse, void* stream) {
  if (head_dim != 64 && head_dim != 128) return LAZY_EUNSUPPORTED;
  if (splits <= 0 || rows < 0) return LAZY_EINVAL;
  if (rows == 0) return LAZY_OK;
  if (!part_o || !part_lse || !out || ((uintptr_t)part_o & 15u)) return LAZY_EINVAL;
  return status(lazy::launch_combine(static_cast<const uint16_t*>(part_o), part_lse, splits, rows, head_dim,
                                     static_cast<uint16_t*>(out), lse, static_cast<hipStream_t>(stream)));
}

int lazy_materialize_k(const lazy_attn_params_t* params, const void* k_pool, const lazy_chunk_t* chunks,
                       int32_t num_records, int32_t max_chunk_len, int64_t total_kv, void* k_out,
                       lazy_chunk_t* chunks_out, void* stream) {
  int e = check_params(params);
  if (e != LAZY_OK) return e;
  if (params->rope_style == LAZY_ALIBI) return LAZY_EUNSUPPORTED;
  if (num_records < 0 || max_chunk_len < 0 || total_kv < 0) return LAZY_EINVAL;
  if (num_records == 0) return LAZY_OK;
  if (!k_pool || !chunks || !chunks_out || (total_kv > 0 && !k_out)) return LAZY_EINVAL;
  if (num_records > 65535 || params->num_kv_heads > 65535) return LAZY_EUNSUPPORTED;
  return status(lazy::launch_materialize(static_cast<const uint16_t*>(k_pool), chunks, num_records, max_chunk_len,
                                         params->num_kv_heads, params->head_dim,
                                         params->inv_freq ? 0.0 : log2((double)params->rope_base),
                                         params->inv_freq, params->key_positions == LAZY_KEYS_LOCAL,
                                         params->rope_style == LAZY_ROPE_INTERLEAVED,
                                         static_cast<uint16_t*>(k_out), chunks_out,
                                         static_cast<hipStream_t>(stream)));
}

size_t lazy_attn_decode_shared_workspace_size(const lazy_attn_params_t* params, int32_t batch, int32_t max_slots) {
  if (check_params(params) != LAZY_OK || batch <= 0 || max_slots <= 0) return 0;
  return (size_t)max_slots * (size_t)batch * params->num_q_heads *
         ((size_t)params->head_dim * sizeof(uint16_t) + sizeof(float));
}

int lazy_attn_decode_shared(const lazy_attn_params_t* p, const void* q, const int32_t* q_pos, const void* k_pool,
                            const void* v_pool, const lazy_shared_item_t* items, int32_t num_items,
                            const lazy_shared_range_t* ranges, const lazy_shared_user_t* users,
                            const int32_t* slot_start, int32_t batch, int32_t max_slots, void* out, float* lse,
                            void* workspace, size_t workspace_bytes, void* stream) {
  int e = check_params(p);
  if (e != LAZY_OK) return e;
  if (p->num_q_heads / p->num_kv_heads > 16) return LAZY_EUNSUPPORTED;
  if (batch < 0 || num_items < 0 || max_slots < 0 || (num_items > 0 && max_slots == 0)) return LAZY_EINVAL;
  if (batch == 0) return LAZY_OK;
  if (!q || !q_pos || !k_pool || !v_pool || !slot_start || !out || (num_items > 0 && (!items || !ranges || !users)))
    return LAZY_EINVAL;
  if (p->num_kv_heads > 65535) return LAZY_EUNSUPPORTED;
  const size_t need = lazy_attn_decode_shared_workspace_size(p, batch, max_slots);
  if (need > 0 && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 15u))) return LAZY_EWORKSPACE;
  lazy::SharedArgs a = {};
  a.q = static_cast<const uint16_t*>(q);
  a.q_pos = q_pos;
  a.k_pool = static_cast<const uint16_t*>(k_pool);
  a.v_pool = static_cast<const uint16_t*>(v_pool);
  a.items = items;
  a.ranges = ranges;
  a.users = users;
  const int64_t rows = (int64_t)batch * p->num_q_heads;
  a.ws_o = need ? static_cast<uint16_t*>(workspace) : nullptr;
  a.ws_lse = need ? reinterpret_cast<float*>(static_cast<uint16_t*>(workspace) + (size_t)max_slots * rows * p->head_dim)
                  : nullptr;
  a.inv_freq = p->inv_freq;
  a.batch = batch;
  a.hq = p->num_q_heads;
  a.hkv = p->num_kv_heads;
  a.group = p->num_q_heads / p->num_kv_heads;
  a.causal = p->causal;
  a.local_keys = p->key_positions == LAZY_KEYS_LOCAL;
  a.interleaved = p->rope_style == LAZY_ROPE_INTERLEAVED;
  a.alibi = p->rope_style == LAZY_ALIBI;
  a.q_prerot = p->q_prerotated && p->rope_style != LAZY_ALIBI;
  a.stream_kv = p->cache_hint == LAZY_CACHE_STREAM;
  a.rope_log2_base = p->inv_freq || p->rope_style == LAZY_ALIBI ? 0.0 : log2((double)p->rope_base);
  a.scale_log2 = scale_log2(p);
  return status(lazy::launch_decode_shared(a, num_items, max_slots, slot_start, p->head_dim,
                                           static_cast<uint16_t*>(out), lse, static_cast<hipStream_t>(stream)));
}

const char* lazy_attn_strerror(int code) {
  switch (code) {
    case LAZY_OK: return "success";
    case LAZY_EINVAL: return "invalid argument";
    case LAZY_EUNSUPPORTED: return "unsupported configuration";
    case LAZY_EWORKSPACE: return "workspace missing, too small or misaligned";
    case LAZY_EHIP: return "HIP runtime error at launch";
    case LAZY_EDATA: return "chunk or query table violates the layout contract";
    default: return "unknown error";
  }
}

int lazy_attn_version(void) { return 100; }

}  // extern "C"
