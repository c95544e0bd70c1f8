// C ABI of the CaliDrop hot path: argument validation, workspace carving and kernel launches.
// Everything here runs on the host; validation never touches HIP, so it can be exercised on a
// machine without a GPU.
#include "../../include/calidrop.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <limits>

#include "cd_attend.h"
#include "cd_common.h"
#include "cd_given.h"
#include "cd_h2o.h"
#include "cd_score.h"
#include "cd_select.h"

// Fixed device memory for calidrop_decode_static, the decode entry point for callers that cannot
// bring a workspace: every GPU the library runs on holds its own copy of this array until the
// process ends.  Host code never uses the array's name as an address: the per-device address comes
// from hipGetSymbolAddress (static_scratch_ptr below).
constexpr size_t kStaticScratchBytes = static_cast<size_t>(CALIDROP_STATIC_SCRATCH_BYTES);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
// floats per vote plane: a multiple of 64, so that every plane starts 256-byte aligned
inline int64_t vote_plane(int64_t total_tokens, int n_kv_heads) { return (total_tokens * n_kv_heads + 63) / 64 * 64; }

constexpr uint32_t kParamsSizeV1 = 48;      // layout up to theta2, without calib_size and flags
constexpr uint32_t kParamsSizeV2 = 52;      // layout up to calib_size, without flags

// Copies the caller's struct (either known layout) into `q` with every field defined.
int load_params(const calidrop_params* in, calidrop_params* q) {
  if (!in) return fail(CALIDROP_EINVAL, "params is NULL");
  if (in->struct_size != sizeof(calidrop_params) && in->struct_size != kParamsSizeV1 &&
      in->struct_size != kParamsSizeV2)
    return fail(CALIDROP_EINVAL, "params.struct_size is %u, this library expects %zu (or %u, %u)", in->struct_size,
                sizeof(calidrop_params), kParamsSizeV2, kParamsSizeV1);
  std::memset(q, 0, sizeof(*q));
  std::memcpy(q, in, in->struct_size);
  q->struct_size = sizeof(calidrop_params);
  return CALIDROP_OK;
}

int check_params(const calidrop_params* p) {
  if (p->dtype != CALIDROP_BF16 && p->dtype != CALIDROP_FP32)
    return fail(CALIDROP_EUNSUPPORTED, "dtype %d is not CALIDROP_BF16 or CALIDROP_FP32", p->dtype);
  if (p->batch < 1) return fail(CALIDROP_EINVAL, "batch must be >= 1 (got %d)", p->batch);
  if (p->n_q_heads < 1 || p->n_kv_heads < 1)
    return fail(CALIDROP_EINVAL, "head counts must be >= 1 (got %d query, %d KV)", p->n_q_heads, p->n_kv_heads);
  if (p->n_q_heads % p->n_kv_heads != 0)
    return fail(CALIDROP_ESHAPE, "n_q_heads %d is not a multiple of n_kv_heads %d", p->n_q_heads, p->n_kv_heads);
  if (p->n_q_heads / p->n_kv_heads > 16)
    return fail(CALIDROP_EUNSUPPORTED, "GQA group size %d exceeds 16", p->n_q_heads / p->n_kv_heads);
  if (p->head_dim != 64 && p->head_dim != 128)
    return fail(CALIDROP_EUNSUPPORTED, "head_dim %d is not 64 or 128", p->head_dim);
  if (p->window < 1) return fail(CALIDROP_EINVAL, "window must be >= 1 (got %d)", p->window);
  if (p->budget <= p->window)
    return fail(CALIDROP_EINVAL, "budget %d must exceed window %d (the window counts toward the budget)", p->budget,
                p->window);
  if (p->budget > (1 << 24))
    return fail(CALIDROP_EUNSUPPORTED, "budget %d exceeds %d", p->budget, 1 << 24);
  if (p->pool_kernel < 1 || p->pool_kernel % 2 == 0)
    return fail(CALIDROP_EINVAL, "pool_kernel must be odd and >= 1 (got %d)", p->pool_kernel);
  if (!(p->scale >= 0.f) || std::isinf(p->scale))
    return fail(CALIDROP_EINVAL, "scale must be finite and >= 0 (0 selects 1/sqrt(head_dim))");
  if (std::isnan(p->theta1) || std::isnan(p->theta2) || p->theta1 > p->theta2)
    return fail(CALIDROP_EINVAL, "thresholds must satisfy theta1 <= theta2 and not be NaN");
  if (p->calib_size < 0) return fail(CALIDROP_EINVAL, "calib_size must be >= 0 (got %d)", p->calib_size);
  if (p->flags & ~(CALIDROP_OPT_WRITE_SCORES | CALIDROP_OPT_WIDE_SELECTION))
    return fail(CALIDROP_EINVAL, "flags 0x%x holds bits that are no CALIDROP_OPT_* option", p->flags);
  {  // launch grids put (sequence, KV head, row block) on one grid axis of at most 65535
    const int64_t nrb = (static_cast<int64_t>(p->n_q_heads / p->n_kv_heads) * p->window + cd::kRowBlock - 1) / cd::kRowBlock;
    if (static_cast<int64_t>(p->batch) * p->n_kv_heads * nrb > 65535 || p->n_q_heads > 65535)
      return fail(CALIDROP_EUNSUPPORTED, "batch * n_kv_heads * ceil(G*window/128) exceeds 65535");
  }
  return CALIDROP_OK;
}

float logit_scale(const calidrop_params* p) {
  return p->scale > 0.f ? p->scale : 1.0f / std::sqrt(static_cast<float>(p->head_dim));
}

int live_rows(const calidrop_params* p, int max_cache_len) { return std::min(p->budget, max_cache_len); }

// Waves of a decode workgroup that has a whole (sequence, KV head).  8, so that its compute unit has more rows in flight, but 4
//   - for caches of at most 4 tiles (one tile a wave);
//   - in fp32, where a lane has two pieces of every row in flight (8 pairs of 1002 rows, D = 128 29.6 us with 4 waves, 33.4
//     with 8, 512 pairs of 308 31.0 / 35.3, D = 64 15.6 / 16.6, 16.8 / 18.7);
//   - in bf16 with D = 128 where the pairs fill the chip (12.8 / 13.0 at 512 rows; 40.5 / 42.0 at 2048, where three such
//     workgroups share a compute unit and one's merge overlaps the others' streaming; with D = 64, 256 pairs of 500 rows,
//     9.5 / 8.5);
//   - where the partial outputs of 8 do not fit what a launch may use of LDS without raising the limit.
// Where the pairs fill the chip it is the rows that live which count: 1024 pairs of 64 rows, D = 64, with room for 512, 8.6
// with 4 waves, 9.7 with 8.
size_t decode_wave_lds(const calidrop_params* p) {
  return static_cast<size_t>(p->n_q_heads / p->n_kv_heads) * (p->head_dim + 2) * sizeof(float);
}
int decode_waves(const calidrop_params* p, int max_cache_len) {
  const int64_t pairs = static_cast<int64_t>(p->batch) * p->n_kv_heads;
  const int tiles = ceil_div(pairs < 192 ? max_cache_len : live_rows(p, max_cache_len), cd::kTileRows);
  return tiles <= 4 || p->dtype == CALIDROP_FP32 || (pairs >= 192 && p->head_dim == 128) || 8 * decode_wave_lds(p) > 48 * 1024 ? 4 : 8;
}

// Decode runs as one workgroup per (sequence, KV head) - one launch, no workspace - or with the rows of a pair split over
// workgroups and a second launch that merges them.  The form that is expected to take less time is taken.
//
// One workgroup: a start, its rows, the tiles of its fullest wave (a step every 32 x waves rows: fp32, D = 64, 8 pairs of
// 384 rows 7.8 us, of 400 8.9) and a share of the traffic of all.  Where the fullest of the 256 compute units has two, rows and
// tiles cost nearly twice that; where every XCD has at most one (8 pairs), its L2 still has rows of the call before if that
// read the same caches, and they cost less (bf16, D = 128, 512 rows: 8 pairs 7.5 us, 16 pairs 8.8; all from memory 9.8, 9.9).
// Split: the two launches, which the host does not issue faster than in `host` us, the traffic of all, and workgroups whose
// rows hold nothing yet.
//
// us per call, one workgroup / split, from the host: bf16, D = 128, 8 pairs of 512 rows 7.5 / 7.7, of 520 7.8 / 7.7, of 1016
// 12.2 / 7.7, of 2044 28.3 / 8.1; 64 pairs of 384 8.2 / 7.9, of 1016 17.4 / 9.9; 184 pairs of 1016 20.4 / 21.7; 320 pairs of
// 776 28.6 / 25.6; D = 64, 8 pairs of 768 7.3 / 7.4, of 900 9.0 / 7.4; fp32, D = 64, 64 pairs of 384 9.4 / 8.2; D = 128, 8
// pairs of 200 9.7 / 10.3, of 1016 30.4 / 10.6.
// Fitted to 3500 calls (2 to 512 pairs, 48 to 4090 rows, both types and head dimensions), caches that were just read and, from
// 9 pairs on, caches that were not, those in which the forms are close counting most: the form taken is 0.1 to 0.4 % (fp32,
// D = 128: 0.8 %) slower on average than the better one, 27 % at most (8 pairs of 512 rows from memory, 9.8 / 7.9).
//
// Both follow the rows that live, which only the device knows, and max_cache_len may be far above them: with room for 2048
// rows, 64 pairs of 200 live ones take 6.0 in one workgroup and 10.5 split, 184 pairs in fp32 12.0 and 25.8.  The longest cache
// is therefore taken to hold `budget` rows, what a compressed prompt starts with; from there on the split form gains on the
// other with every row.  Few pairs with room for more than 2048 rows are priced full: one workgroup would take 25 to 70 us for
// what the split form does in 8 to 30, and loses up to 4 while it is empty.
struct DecodeCost {
  float start, row, tile, pair_row, near, crowded;      // one workgroup; near, crowded: factors of row and tile
  float host, split, split_pair_row, split_room;        // us; the latter two per (pair, row)
};
bool decode_splits(const calidrop_params* p, int max_cache_len) {
  const int64_t pairs = static_cast<int64_t>(p->batch) * p->n_kv_heads;
  if (pairs > 512) return false;
  constexpr DecodeCost kCost[2][2] = {{{3.57f, .00512f, .286f, 1.24e-5f, .805f, 1.87f, 7.7f, 6.48f, 3.91e-5f, 2.98e-6f},
                                       {3.21f, .01159f, .12f, 2.34e-5f, .689f, 1.87f, 7.7f, 6.98f, 7.68e-5f, 3.95e-6f}},
                                      {{3.56f, .00569f, 1.02f, 1.88e-5f, .855f, 1.87f, 8.2f, 7.34f, 7.59e-5f, 4.58e-6f},
                                       {5.14f, .02457f, 0.f, 6.77e-5f, 1.f, 1.82f, 9.4f, 9.1f, 1.78e-4f, 1.15e-5f}}};
  const DecodeCost& c = kCost[p->dtype == CALIDROP_FP32][p->head_dim == 128];
  const bool priced_full = pairs < 192 && max_cache_len > 2048;
  const int rows = priced_full ? max_cache_len : live_rows(p, max_cache_len);
  const float all = static_cast<float>(rows) * static_cast<float>(pairs), room = static_cast<float>(max_cache_len) * static_cast<float>(pairs) - all;
  const int tiles = ceil_div(rows, cd::kTileRows * decode_waves(p, max_cache_len));
  const float factor = pairs <= 8 ? c.near : pairs > 256 ? c.crowded : 1.f;
  const float one = c.start + (c.row * static_cast<float>(rows) + c.tile * static_cast<float>(tiles)) * factor + c.pair_row * all;
  return std::max(c.host, c.split + c.split_pair_row * all + c.split_room * room) < one;
}

// How the rows of a streaming-attention pass are split over workgroups.
struct SplitPlan { int rows_per_split, NS; };
// `few`: a pass over prompt rows whose splits, where there are no more than `few` of them with a few tiles per wave each,
// are halved down to one tile per wave.  In 288 calls (2 to 64 (sequence, KV head) pairs, 2048 to 16384 rows) that is up to
// 28 % faster while it ends below two workgroups per compute unit - where V is streamed alone, and in fp32, whose products
// keep a wave busy longer (8 heads of 8192 rows, V alone 7.9 -> 6.3 us) - and up to 21 % slower where it goes on to more
// (16 heads of 8192 rows, K and V in bf16: 17.9 us a call at 256 rows, 20.3 at 128), in bf16 with K and V streamed from
// one per unit on.  Longer splits stay at 32 (131072 rows: 44 us at 4096 rows, 45 us at 1024).
SplitPlan plan_splits(int heads_kv_total, int max_rows, int few = 0) {
  const int kTargetGroups = 4096;                      // ~16 workgroups per compute unit
  const int kMaxSplits = 32;
  const int kMinRows = cd::kTileRows * cd::kAttWaves;  // one tile per wave
  if (max_rows < 1) max_rows = 1;
  int want = ceil_div(kTargetGroups, heads_kv_total);
  if (want < 1) want = 1;
  if (want > kMaxSplits) want = kMaxSplits;
  int rps = ceil_div(ceil_div(max_rows, want), kMinRows) * kMinRows;
  if (rps < kMinRows) rps = kMinRows;
  if (rps <= 4 * kMinRows)
    while (rps > kMinRows && static_cast<int64_t>(heads_kv_total) * ceil_div(max_rows, rps) <= few) rps = ceil_div(rps / 2, kMinRows) * kMinRows;
  return SplitPlan{rps, ceil_div(max_rows, rps)};
}

// The most splits any prompt or cache of up to max_rows plans: a number that does not fall as they grow, unlike a plan's own, so
// that a workspace sized for a long one serves the shorter ones.  (A plan starts from at most `want` splits and halves only
// prompts of up to 32 * 512 rows, to at most twice the splits that `few` allows.)
int most_splits(int heads_kv_total, int max_rows, int few) {
  const int want = std::min(std::max(ceil_div(4096, heads_kv_total), 1), 32);
  return std::min(ceil_div(std::max(max_rows, 1), cd::kTileRows * cd::kAttWaves), std::max(want, std::min(2 * (few / heads_kv_total), 128)));
}

constexpr int kFewV = 256;                             // V alone streamed (the logits come from the scoring pass)
int few_kv(const calidrop_params* p) { return p->dtype == CALIDROP_FP32 ? 256 : 128; }      // K and V streamed

// Keys per scoring workgroup, in units of 64.  The 256 compute units share the workgroups of a launch, so a plan costs the
// workgroups of the fullest unit times the key units of one, plus half a unit for its start (query fragments, first
// stage).  A unit holds `fit` 128-row workgroups at a time; fewer than three of them (bf16, D = 128: two) save nothing, the
// matrix pipe or the memory waits, and one left over when the others are through takes the time of two (fp32, 4
// prompts of 20000 tokens, 8 KV heads, 64 window rows: four of 640 keys 455 us a call, five of 512 keys 406).
// The chunk of least cost is taken, all chunks of the longest prompt alike, at most 16 units (256-row blocks start
// slower: 32).  Prompts of different lengths: the host knows their sum and the longest only.  What the short last
// chunks take is estimated (half a workgroup per prompt at 128 rows and, in fp32, while a prompt has fewer than four chunks;
// else nothing: with 256 rows they mostly fill gaps), and since the last round is not full everywhere, the rounded count
// weighs one part and the plain one, half a round later, three; at 128 rows chunks stay at 8 units.
// Measured over 635 calls (350 to 131072 tokens, 1 to 64 prompts, both types, D 64 and 128, 16 to 256 window rows per KV
// head), each at 21 chunk lengths: the chunk taken is on average 1 % (prompts of one length) to 3.5 % (256 rows, several
// lengths) slower than the best of them.  Examples, us a call at 256-512 keys and many rounds / at one workgroup for each
// of 512 places / now: fp32, 256 rows, 6 prompts of 9000-17000 tokens 798 / 958 / 730; one of 16384 230 / 209 / 192; bf16,
// 131072 tokens, 256 rows 281 / 239 / 239.
// `most_chunks`: what the workspace has room for.
int plan_chunk(const calidrop_params* p, int64_t total_tokens, int32_t max_seq_len, int RB, int NRB, int64_t most_chunks) {
  const bool even = total_tokens == static_cast<int64_t>(p->batch) * max_seq_len;
  const bool narrow = RB == cd::kRowBlock;
  const int64_t rows = static_cast<int64_t>(p->n_kv_heads) * NRB;          // grid rows of one prompt
  const bool bf16 = p->dtype == CALIDROP_BF16;
  const int fit = bf16 ? 4 : p->head_dim == 128 ? 3 : 5, least = !narrow ? 1 : even && !(bf16 && p->head_dim == 128) ? 3 : 2;
  int best = 0;
  int64_t best_cost = std::numeric_limits<int64_t>::max();
  for (int most = narrow ? (even ? 16 : 8) : 32; most >= 1; --most) {
    const int nch = ceil_div(max_seq_len, most * cd::kChunkUnit);
    if (best && nch > most_chunks) break;
    const int units = ceil_div(ceil_div(max_seq_len, nch), cd::kChunkUnit);      // the chunks of the longest prompt alike
    const int64_t keys = static_cast<int64_t>(units) * cd::kChunkUnit;
    const bool last = narrow || (!bf16 && total_tokens < 4 * keys * p->batch);
    const int64_t groups = even ? rows * p->batch * ((max_seq_len + keys - 1) / keys) : total_tokens * rows / keys + (last ? rows * p->batch / 2 : 0);
    const int64_t full = (groups + 255) / 256;
    int64_t load = even ? 1024 * full : 256 * full + 3 * (groups + 128);         // 1024 = one workgroup on every unit
    if (narrow && even && full % fit == 1) load += 1024;
    load = std::max<int64_t>(load, 1024 * least);
    const int64_t cost = load * (2 * units + 1);
    if (cost < best_cost) { best_cost = cost; best = static_cast<int>(keys); }
  }
  return best;
}

// Heads whose pooled scores fit in LDS are pooled and selected by one workgroup each; longer ones (and wider pooling)
// go through the multi-workgroup chain.  `window` = trailing positions always kept.
bool uses_lds_selection(const calidrop_params* p, int window, int pool_k, int max_seq_len) {
  return max_seq_len - window <= cd::kSelMaxLdsKeys && p->budget <= cd::kSelMaxLdsKeys && pool_k <= cd::kSelMaxPool &&
         !(p->flags & CALIDROP_OPT_WIDE_SELECTION);
}
// Words a kernel ahead of the selection has to clear for it.
int64_t wide_words(const calidrop_params* p) { return static_cast<int64_t>(p->batch) * p->n_kv_heads * cd::kWideHistWords; }
// What the multi-workgroup selection keeps in the workspace: nothing where it is not used.
struct WideRegions { size_t hist = 0, seg = 0; };      // bytes
WideRegions wide_regions(const calidrop_params* p, int window, int pool_k, int max_seq_len, int nseg) {
  if (uses_lds_selection(p, window, pool_k, max_seq_len)) return {};
  const size_t heads = static_cast<size_t>(p->batch) * p->n_kv_heads;
  return {round256(heads * cd::kWideHistWords * sizeof(uint32_t)), round256(heads * nseg * cd::kWideSegWords * sizeof(uint32_t))};
}

// Most chunk partials per row that the workgroups of pass 2 merge for themselves, and most bytes of partials that all of them
// read for it: every workgroup reads the partials of all its rows, from its L2, before its first stage is done.  236 calls (1 to
// 12 prompts of 600 to 90000 tokens, both types, 16 to 64 window rows): without the launch that merges them 0.8 to 2.4 us
// less up to 24 MiB, from there on 0.5 less to 9 us more (131072 tokens, 256 rows, 64 MiB: 244 -> 246).
constexpr int kMergeInVotes = 64;
constexpr int64_t kMergeInVotesBytes = 24 << 20;

struct CompressLayout {
  size_t rowpart, row_lse, vote, score, bitmap, cal_logit, part_o, part_ml, sel_hist, sel_cnt, total;
  int RB, NRB, NCH, W32, chunk_keys, zstride, NSEG;
  bool merge_in_votes;
  SplitPlan sp;
};

CompressLayout compress_layout(const calidrop_params* p, int64_t total_tokens, int32_t max_seq_len) {
  CompressLayout L{};
  const int G = p->n_q_heads / p->n_kv_heads;
  L.RB = G * p->window > cd::kRowBlock ? 2 * cd::kRowBlock : cd::kRowBlock;     // 256-row blocks: such heads stream K once
  L.NRB = ceil_div(G * p->window, L.RB);
  L.W32 = ceil_div(max_seq_len, 64) * 2;
  L.zstride = ceil_div(max_seq_len, 32) * 32;
  L.NSEG = ceil_div(std::max(max_seq_len - p->window, 1), cd::kWideSeg);
  const int heads = p->batch * p->n_kv_heads;
  L.sp = plan_splits(heads, max_seq_len, kFewV);
  const size_t rows = static_cast<size_t>(heads) * L.NRB * L.RB;
  const size_t toks = static_cast<size_t>(total_tokens) * p->n_kv_heads;
  size_t off = 0;
  L.row_lse = off; off += round256(rows * sizeof(float));
  // multi-workgroup selection (prefixes beyond the single-workgroup variant): histograms and counts
  const WideRegions wide = wide_regions(p, p->window, p->pool_kernel, max_seq_len, L.NSEG);
  L.sel_hist = off; off += wide.hist;
  L.sel_cnt = off;  off += wide.seg;
  // Few partials per row are merged by the workgroups of pass 2, next to their writing votes: a region of their own.  Many are
  // merged into row_lse before anything is written to the regions from the votes on: they lie under them.  No plan takes
  // more room than those regions, or than chunks of 8 units need where that is more, so that the size of the workspace does not
  // fall as prompts grow.
  const size_t chunk_bytes = rows * sizeof(float2);
  L.rowpart = off; off += round256(chunk_bytes * std::min(kMergeInVotes, ceil_div(max_seq_len, cd::kChunkUnit)));
  L.vote = off;    off += round256(static_cast<size_t>(vote_plane(total_tokens, p->n_kv_heads)) * L.NRB * sizeof(float));
  L.score = off;   off += round256(toks * sizeof(float));
  L.bitmap = off;  off += round256(static_cast<size_t>(heads) * L.W32 * sizeof(uint32_t));
  L.cal_logit = off; off += round256(static_cast<size_t>(p->batch) * p->n_q_heads * L.zstride * sizeof(float));
  const size_t slots = static_cast<size_t>(p->batch) * p->n_q_heads * most_splits(heads, max_seq_len, kFewV);
  L.part_o = off;  off += round256(slots * p->head_dim * sizeof(float));
  L.part_ml = off; off += round256(slots * sizeof(float2));
  const size_t room = std::max(off - L.vote, round256(chunk_bytes * ceil_div(max_seq_len, 8 * cd::kChunkUnit)));
  L.chunk_keys = plan_chunk(p, total_tokens, max_seq_len, L.RB, L.NRB, static_cast<int64_t>(room / chunk_bytes));
  L.NCH = ceil_div(max_seq_len, L.chunk_keys);
  L.merge_in_votes = L.NCH <= kMergeInVotes && static_cast<int64_t>(chunk_bytes) * L.NCH * L.NCH <= kMergeInVotesBytes;
  if (L.NCH > kMergeInVotes) L.rowpart = L.vote;
  L.total = L.vote + room;
  return L;
}

// `total`: what a workspace for caches of up to these rows holds, the most splits of any of them (4096 rows are cut into 32,
// 4097 into 17); `used`: what this call writes of it.
struct DecodeLayout { size_t part_o, part_ml, used, total; SplitPlan sp; };

DecodeLayout decode_layout(const calidrop_params* p, int32_t max_cache_len) {
  DecodeLayout L{};
  const int pairs = p->batch * p->n_kv_heads;
  L.sp = plan_splits(pairs, max_cache_len);
  const size_t heads = static_cast<size_t>(p->batch) * p->n_q_heads;
  const auto out_bytes = [&](int splits) { return round256(heads * splits * p->head_dim * sizeof(float)); };
  const auto ml_bytes = [&](int splits) { return round256(heads * splits * sizeof(float2)); };
  const int most = most_splits(pairs, max_cache_len, 0);
  L.part_o = 0;
  L.part_ml = out_bytes(L.sp.NS);
  L.used = L.part_ml + ml_bytes(L.sp.NS);
  L.total = out_bytes(most) + ml_bytes(most);
  return L;
}

int check_sizes(const calidrop_params* p, int64_t total_tokens, int32_t max_seq_len) {
  if (total_tokens < 1 || max_seq_len < 1 || max_seq_len > total_tokens)
    return fail(CALIDROP_ESHAPE, "need 1 <= max_seq_len <= total_tokens (got %d, %lld)", max_seq_len,
                static_cast<long long>(total_tokens));
  if (total_tokens > (static_cast<int64_t>(1) << 31) - 1)
    return fail(CALIDROP_EUNSUPPORTED, "total_tokens exceeds int32 offsets");
  if (static_cast<int64_t>(p->batch) * max_seq_len < total_tokens)
    return fail(CALIDROP_ESHAPE, "batch * max_seq_len < total_tokens");
  return CALIDROP_OK;
}

int launch_status(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CALIDROP_EHIP, "%s: %s", what, hipGetErrorString(e));
  return CALIDROP_OK;
}

// The skip bitmap of a sequence fits LDS up to 48 KiB (393216 positions): built there, stored once.
void launch_bitmap(const cd::BitmapArgs& ba, int pairs, hipStream_t st) {
  const size_t lds = static_cast<size_t>(ba.W32) * sizeof(uint32_t);
  if (lds <= 48 * 1024) hipLaunchKernelGGL(cd::bitmap_from_indices_lds_kernel, dim3(pairs), dim3(256), lds, st, ba);
  else hipLaunchKernelGGL(cd::bitmap_from_indices_kernel, dim3(pairs), dim3(256), 0, st, ba);
}

// The single-workgroup selection kernels stage up to kSelMaxLdsKeys votes in dynamic LDS, more
// than the 48 KiB a kernel may use without asking.  The limit is raised to the largest size any call
// can need of a variant, once per (kernel variant, device) at that variant's first use on the device - a host-side
// setting that enqueues nothing - and never again, so that calls on the enqueue path (also under
// stream capture) only launch.
constexpr size_t kSelMaxListBytes = 64 * 1024;            // the retained list, where the selection gathers too
constexpr size_t select_max_lds(int per) { return std::max(cd::select_row_bytes(cd::kSelThreads * per, per), kSelMaxListBytes); }
constexpr int kMaxDevices = 64;
constexpr int kLdsSlots = 8;                              // kernels that ask for more than 48 KiB of dynamic LDS
enum { kLdsSelect = 0 };                                  // four variants of the selection kernel
std::atomic<uint8_t> g_lds_ready[kLdsSlots][kMaxDevices]; // zero-initialised: nothing raised yet

// `bytes` is the largest size any call can ask of this kernel, so one setting per (slot, device) is enough.
int ensure_kernel_lds(int slot, const void* fn, size_t bytes, const char* what) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(CALIDROP_EHIP, "hipGetDevice failed or device index %d is beyond %d", dev, kMaxDevices - 1);
  if (g_lds_ready[slot][dev].load(std::memory_order_acquire)) return CALIDROP_OK;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
  if (e != hipSuccess) return fail(CALIDROP_EHIP, "hipFuncSetAttribute(%s): %s", what, hipGetErrorString(e));
  g_lds_ready[slot][dev].store(1, std::memory_order_release);
  return CALIDROP_OK;
}

// Device address of `scratch` on the current device, looked up once per device.
std::atomic<void*> g_scratch_ptr[kMaxDevices];            // zero-initialised: not looked up yet

int static_scratch_ptr(char** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(CALIDROP_EHIP, "hipGetDevice failed or device index %d is beyond %d", dev, kMaxDevices - 1);
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!ptr) {
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(CALIDROP_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);
  }
  *out = static_cast<char*>(ptr);
  return CALIDROP_OK;
}

// Where the gather of the retained rows runs.  It costs no launch as further workgroups of the streaming pass, where they
// take the places of streaming ones (LDS and registers are the pass's), or of the launch that merges the pass's partials,
// where they wait for the pass.  134 calls (2 to 80 (sequence, KV head) pairs, budgets 128 to 2500, 512 to 60000 rows), in the
// merge / in the pass, us a call: the pass is 1-2 % faster while its splits are short (2 heads of 3000 rows, fp32 30.0 / 29.4, 8
// heads 28.6 / 28.1), the merge 1-3 % from some 600 rows on (8 heads of 20000 rows 56.7 / 58.5); against a launch of its own the
// merge saves 3-4 us (131072 rows, budget 4096: 12.1 us in two launches, 8.4 in one).  The pass was measured up to some 8000
// gathering workgroups; 512 heads of 1024 rows, 32768 of them, held it up for 160 us.  With more heads than the merge takes
// four groups of threads for, its workgroups are small and the gather is a launch of its own.
// With many heads the selection kernel does it: while one workgroup selects, others copy (140 us for both, against
// 36 + 100 in two launches).
enum class GatherIn { kPass, kDone, kAfter };
GatherIn gather_place(const calidrop_params* p, const cd::GatherArgs& ga, int rows_per_split, bool lds_selection) {
  const int64_t pairs = static_cast<int64_t>(p->batch) * p->n_kv_heads;
  const bool fits = p->budget * sizeof(int32_t) <= kSelMaxListBytes;           // the list in LDS
  if (lds_selection && fits && pairs >= 128 && pairs * ga.blocks > 256) return GatherIn::kDone;
  return rows_per_split < 512 && pairs * ga.blocks <= 4096 ? GatherIn::kPass : GatherIn::kAfter;
}

cd::GatherArgs gather_args(const calidrop_params* p, const int32_t* indices, const int32_t* cache_offsets, const void* k, const void* v,
                           void* k_c, void* v_c) {
  const int row_bytes = p->head_dim * (p->dtype == CALIDROP_BF16 ? 2 : 4);
  const int64_t vecs = static_cast<int64_t>(p->budget) * (row_bytes / 16);
  return cd::GatherArgs{indices, cache_offsets, k, v, k_c, v_c, row_bytes, static_cast<int>((vecs + cd::kGatherVecs - 1) / cd::kGatherVecs)};
}

// Pooling + selection of the votes in se.vote.  For the multi-workgroup chain `sel_hist` has been cleared.
int run_selection(const calidrop_params* p, int max_seq_len, cd::SelectArgs& se, uint32_t* sel_hist, uint32_t* sel_seg, int NSEG,
                  int rows_per_split, GatherIn& place, hipStream_t st) {
  int rc;
  const int bg = p->batch * p->n_kv_heads;
  const int max_prefix = max_seq_len - se.w;
  se.write_scores = (p->flags & CALIDROP_OPT_WRITE_SCORES) ? 1 : 0;
  const bool lds_selection = uses_lds_selection(p, se.w, se.pool_k, max_seq_len);
  place = gather_place(p, se.gather, rows_per_split, lds_selection);
  se.gather_here = place == GatherIn::kDone;
  if (lds_selection) {
    // 1024 threads, and positions per thread: the smallest of 2 / 8 / 16 / 32 that covers the longest prefix.
    const dim3 grid(bg);
    auto launch = [&](auto per) {
      constexpr int PER = decltype(per)::value;
      const auto fn = &cd::select_lds_kernel<cd::kSelThreads, PER>;
      const int slot = kLdsSelect + (PER == 2 ? 3 : PER == 8 ? 0 : PER == 16 ? 1 : 2);
      // dynamic LDS: staged votes, later reused for the retained indices
      size_t lds = max_seq_len > p->budget ? cd::select_row_bytes(max_prefix, PER) : 0;
      if (se.gather_here) lds = std::max(lds, static_cast<size_t>(p->budget) * sizeof(int32_t));
      if (int e = ensure_kernel_lds(slot, reinterpret_cast<const void*>(fn), select_max_lds(PER), "select")) return e;
      hipLaunchKernelGGL(fn, grid, dim3(cd::kSelThreads), lds, st, se);
      return static_cast<int>(CALIDROP_OK);
    };
    using std::integral_constant;
    if (max_prefix <= cd::kSelThreads * 2) rc = launch(integral_constant<int, 2>{});
    else if (max_prefix <= cd::kSelThreads * 8) rc = launch(integral_constant<int, 8>{});
    else if (max_prefix <= cd::kSelThreads * 16) rc = launch(integral_constant<int, 16>{});
    else rc = launch(integral_constant<int, 32>{});
    if (rc) return rc;
  } else {
    cd::WideArgs wa{};
    wa.s = se; wa.NSEG = NSEG; wa.hist = sel_hist; wa.seg = sel_seg;
    const dim3 grid_w(NSEG, bg), block_w(cd::kWideThreads);
    if (max_seq_len > p->budget) {
      hipLaunchKernelGGL(cd::wide_pool_kernel, grid_w, block_w, 0, st, wa);
      if ((rc = launch_status("wide_pool"))) return rc;
      hipLaunchKernelGGL(cd::wide_hist_kernel, grid_w, block_w, 0, st, wa);
      if ((rc = launch_status("wide_hist"))) return rc;
      hipLaunchKernelGGL(cd::wide_last_kernel, grid_w, block_w, 0, st, wa);
      if ((rc = launch_status("wide_last"))) return rc;
    }
    hipLaunchKernelGGL(cd::wide_emit_kernel, grid_w, block_w, 0, st, wa);
  }
  return launch_status("select");
}

// The merge of the split partials.  Four groups of threads per head shorten the chain of loads while the heads leave the chip
// room (32 heads, 64 splits 6.7 -> 4.0 us; 96 heads 4.6 -> 3.7 us; 256 to 640 heads the same); with a thousand heads and more
// their workgroups no longer fit it at once (1024 heads 5.5 -> 6.5 us, 1920 heads 5.0 -> 7.3 us): one group then.
constexpr int64_t kFourGroupHeads = 768;
// `gather`: the rows this launch gathers as well, or NULL (more than kFourGroupHeads heads: always NULL).
template <typename T, int D>
int launch_finalize(const calidrop_params* p, cd::FinalArgs& fa, hipStream_t st, const char* what, const cd::GatherArgs* gather = nullptr) {
  dim3 grid(p->n_q_heads, p->batch);
  const bool four = static_cast<int64_t>(p->batch) * p->n_q_heads <= kFourGroupHeads;
  if (gather) {
    fa.gather = *gather;
    grid.x += p->n_kv_heads * ceil_div(gather->blocks * cd::kGatherVecs, 4 * D);
    hipLaunchKernelGGL((cd::attend_finalize_kernel<T, D, 4, true>), grid, dim3(4 * D), 0, st, fa);
  } else if (four) {
    hipLaunchKernelGGL((cd::attend_finalize_kernel<T, D, 4>), grid, dim3(4 * D), 0, st, fa);
  } else {
    hipLaunchKernelGGL((cd::attend_finalize_kernel<T, D, 1>), grid, dim3(D), 0, st, fa);
  }
  return launch_status(what);
}

// A pass over K and V of `rows` cached or prompt rows.  The first tile of a wave - all of K while a split is one tile per wave -
// goes through the caches while the K and V of the call are at most three times the last-level cache, and around it beyond:
// decode calls and given sets that are repeated find it there (120 calls, us with / without: 44 caches of 3026 rows, 68 MB,
// 16.4 / 18.2; one cache of 4100 rows 9.7 / 9.9; 216 prompts of 462, 51 MB, 20.1 / 21.1; 104 prompts of 3660, 195 MB,
// 36.2 / 39.7); from 0.6 to 1.2 GB both are alike, above that it is up to 12 % slower (1.5 GB: 303 / 269).
template <typename T, int D, bool kGather = false>
void launch_kv_pass(const cd::AttendArgs& aa, dim3 grid, int64_t rows, hipStream_t st) {
  const bool keep = 2 * rows * aa.Hkv * D * static_cast<int64_t>(sizeof(T)) <= (768ll << 20);
  if (keep) hipLaunchKernelGGL((cd::attend_partial_kernel<T, D, false, false, kGather, false, true>), grid, dim3(256), 0, st, aa);
  else hipLaunchKernelGGL((cd::attend_partial_kernel<T, D, false, false, kGather>), grid, dim3(256), 0, st, aa);
}

// The streaming pass over KV_evict, and the gather unless the selection has done it.  `left` is set where the gather is left
// to the launch that merges the partials.
template <typename T, int D>
int launch_calibration(const calidrop_params* p, cd::AttendArgs& aa, const cd::GatherArgs& ga, GatherIn place, hipStream_t st,
                       const cd::GatherArgs** left) {
  const bool evicts = aa.max_len > p->budget;          // otherwise no sequence can have anything to evict
  *left = nullptr;
  if (place == GatherIn::kAfter || (place == GatherIn::kPass && !evicts)) {
    if (static_cast<int64_t>(p->batch) * p->n_q_heads <= kFourGroupHeads) {
      *left = &ga;
    } else {
      cd::GatherOnlyArgs go{ga, aa.row_off, aa.total_tokens, p->n_kv_heads, p->budget, aa.max_len};
      hipLaunchKernelGGL(cd::gather_kv_kernel, dim3(ga.blocks, p->batch * p->n_kv_heads), dim3(256), 0, st, go);
      if (int rc = launch_status("gather_kv")) return rc;
    }
  }
  if (!evicts) return CALIDROP_OK;
  aa.gather = ga;
  const bool carry = place == GatherIn::kPass;
  // the gathering workgroups fill whole planes of NS x Hkv behind the last sequence's
  const dim3 grid(aa.NS, p->n_kv_heads, p->batch + (carry ? ceil_div(p->batch * ga.blocks, aa.NS) : 0));
  if (aa.cal_logit && carry) hipLaunchKernelGGL((cd::attend_partial_kernel<T, D, true, false, true>), grid, dim3(256), 0, st, aa);
  else if (aa.cal_logit) hipLaunchKernelGGL((cd::attend_partial_kernel<T, D, true>), grid, dim3(256), 0, st, aa);
  else if (carry) launch_kv_pass<T, D, true>(aa, grid, aa.total_tokens, st);
  else launch_kv_pass<T, D>(aa, grid, aa.total_tokens, st);
  return launch_status("attend_partial(calibration)");
}

template <typename T, int D>
int compress_impl(const calidrop_params* p, const void* q_win, const void* k, const void* v,
                  const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len, const float* win_lse,
                  const void* q_cal, void* k_c, void* v_c, const int32_t* cache_offsets, int32_t* cache_lens,
                  int32_t* indices, int32_t* cal_indices, float* c_q, float* c_out, float* c_lse, char* ws,
                  const CompressLayout& L, hipStream_t st) {
  const int G = p->n_q_heads / p->n_kv_heads;
  const float sl2 = logit_scale(p) * cd::kLog2e;
  int rc;

  cd::ScoreArgs sa{};
  sa.q_win = q_win; sa.k = k; sa.seq_off = seq_offsets; sa.total_tokens = total_tokens;
  sa.batch = p->batch; sa.Hq = p->n_q_heads; sa.Hkv = p->n_kv_heads; sa.G = G; sa.w = p->window;
  sa.B = p->budget; sa.R = G * p->window; sa.RB = L.RB; sa.row_stride = L.NRB * L.RB; sa.NRB = L.NRB; sa.NCH = L.NCH; sa.max_seq_len = max_seq_len;
  sa.sl2 = sl2; sa.chunk_keys = L.chunk_keys;
  // K of the whole call well inside the 256 MB last-level cache: pass 1 reads it with cached loads so
  // that pass 2 finds it there; larger calls stream it both times
  sa.keep_k = static_cast<int64_t>(total_tokens) * p->n_kv_heads * D * static_cast<int64_t>(sizeof(T)) <= (160ll << 20);
  sa.rowpart = reinterpret_cast<float2*>(ws + L.rowpart);
  sa.row_lse = reinterpret_cast<float*>(ws + L.row_lse);
  sa.vote = reinterpret_cast<float*>(ws + L.vote);
  sa.plane = vote_plane(total_tokens, p->n_kv_heads);
  if (!uses_lds_selection(p, p->window, p->pool_kernel, max_seq_len)) {
    sa.zero_words = reinterpret_cast<uint32_t*>(ws + L.sel_hist); sa.zero_count = wide_words(p);
  }
  // default calibration query = last window query: the vote pass exports its logits
  sa.cal_logit = (q_cal || G > cd::kMaxCalHeads || p->window % 4 != 0)
                     ? nullptr : reinterpret_cast<float*>(ws + L.cal_logit);
  sa.zstride = L.zstride;

  const int bg = p->batch * p->n_kv_heads;
  if (max_seq_len > p->budget) {       // otherwise no sequence can need eviction
    dim3 grid_s(L.NCH, bg * L.NRB);
    const int64_t rows = static_cast<int64_t>(bg) * L.NRB * L.RB;
    sa.win_lse = win_lse;                // pass 1 is the caller's
    if (!win_lse) {
      if (L.RB == 256) hipLaunchKernelGGL((cd::score_rowstats_kernel<T, D, 8>), grid_s, dim3(512), 0, st, sa);
      else hipLaunchKernelGGL((cd::score_rowstats_kernel<T, D, 4>), grid_s, dim3(256), 0, st, sa);
      if ((rc = launch_status("score_rowstats"))) return rc;
      sa.rows_merged = !L.merge_in_votes;
      if (sa.rows_merged) {
        hipLaunchKernelGGL(cd::rowstats_merge_kernel, dim3(static_cast<unsigned>(rows / cd::kMergeRows)), dim3(256), 0, st, sa);
        if ((rc = launch_status("rowstats_merge"))) return rc;
      }
    }
    if (L.RB == 256) hipLaunchKernelGGL((cd::score_votes_kernel<T, D, 8>), grid_s, dim3(512), 0, st, sa);
    else hipLaunchKernelGGL((cd::score_votes_kernel<T, D, 4>), grid_s, dim3(256), 0, st, sa);
    if ((rc = launch_status("score_votes"))) return rc;
  }

  // Pooling + selection.  Heads whose pooled scores fit in LDS are pooled inside the
  // selection kernel; longer ones go through the pooled-score buffer in the workspace.
  const cd::GatherArgs ga = gather_args(p, indices, cache_offsets, k, v, k_c, v_c);
  GatherIn place;
  cd::SelectArgs se{};
  se.gather = ga;
  se.seq_off = seq_offsets; se.total_tokens = total_tokens; se.batch = p->batch;
  se.Hkv = p->n_kv_heads; se.w = p->window; se.B = p->budget; se.max_seq_len = max_seq_len; se.W32 = L.W32;
  se.NRB = L.NRB; se.pool_k = p->pool_kernel;
  se.vote = sa.vote; se.plane = sa.plane; se.score = reinterpret_cast<float*>(ws + L.score); se.indices = indices; se.cache_lens = cache_lens;
  se.calib = p->calib_size; se.cal_indices = cal_indices;
  se.bitmap = reinterpret_cast<uint32_t*>(ws + L.bitmap);
  if ((rc = run_selection(p, max_seq_len, se, reinterpret_cast<uint32_t*>(ws + L.sel_hist),
                          reinterpret_cast<uint32_t*>(ws + L.sel_cnt), L.NSEG, L.sp.rows_per_split, place, st)))
    return rc;

  cd::AttendArgs aa{};
  aa.q = q_cal ? q_cal : q_win; aa.q_is_window = q_cal ? 0 : 1;
  aa.k = k; aa.v = v; aa.row_off = seq_offsets; aa.row_len = nullptr; aa.bitmap = se.bitmap;
  aa.total_tokens = total_tokens; aa.batch = p->batch; aa.Hq = p->n_q_heads; aa.Hkv = p->n_kv_heads; aa.G = G;
  aa.w = p->window; aa.B = p->budget; aa.max_len = max_seq_len; aa.W32 = L.W32;
  aa.rows_per_split = L.sp.rows_per_split; aa.NS = L.sp.NS; aa.sl2 = sl2;
  aa.cal_logit = sa.cal_logit; aa.zstride = L.zstride;
  aa.part_o = reinterpret_cast<float*>(ws + L.part_o);
  aa.part_ml = reinterpret_cast<float2*>(ws + L.part_ml);
  const cd::GatherArgs* left;
  if ((rc = launch_calibration<T, D>(p, aa, ga, place, st, &left))) return rc;
  cd::FinalArgs fa{};
  fa.part_o = aa.part_o; fa.part_ml = aa.part_ml; fa.row_off = seq_offsets; fa.row_len = nullptr;
  fa.total_tokens = total_tokens; fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G;
  fa.w = p->window; fa.B = p->budget; fa.max_len = max_seq_len; fa.rows_per_split = L.sp.rows_per_split;
  fa.NS = L.sp.NS; fa.calib_mode = 1; fa.q_is_window = aa.q_is_window; fa.q = aa.q;
  fa.c_q = c_q; fa.c_out = c_out; fa.c_lse = c_lse;
  return launch_finalize<T, D>(p, fa, st, "attend_finalize(calibration)", left);
}

template <typename T, int D>
int decode_impl(const calidrop_params* p, const void* q_t, const void* k_c, const void* v_c,
                const int32_t* cache_offsets, const int32_t* cache_lens, int32_t max_cache_len, const float* c_q,
                const float* c_out, const float* c_lse, void* out, float* a_lse, uint8_t* flags, char* ws,
                const DecodeLayout& L, hipStream_t st) {
  const int G = p->n_q_heads / p->n_kv_heads;
  int rc;
  if (!decode_splits(p, max_cache_len)) {
    cd::DecodeFusedArgs fa{};
    fa.q = q_t; fa.k = k_c; fa.v = v_c; fa.row_off = cache_offsets; fa.row_len = cache_lens;
    fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G; fa.max_len = max_cache_len;
    fa.sl2 = logit_scale(p) * cd::kLog2e; fa.theta1 = p->theta1; fa.theta2 = p->theta2;
    fa.c_q = c_q; fa.c_out = c_out; fa.c_lse = c_lse; fa.out = out; fa.a_lse = a_lse; fa.flags = flags;
    const int tiles = ceil_div(max_cache_len, cd::kTileRows);
    const int nw = decode_waves(p, max_cache_len);
    fa.xcd_blocks = (tiles >= 32 && p->batch % 8 == 0) ? 1 : 0;
    const dim3 grid(p->n_kv_heads, p->batch);
    const size_t lds = nw * decode_wave_lds(p);
    if constexpr (sizeof(T) == 2) {
      if (nw == 8) {
        hipLaunchKernelGGL((cd::decode_fused_kernel<T, D, 8>), grid, dim3(512), lds, st, fa);
        return launch_status("decode_fused");
      }
    }
    hipLaunchKernelGGL((cd::decode_fused_kernel<T, D, 4>), grid, dim3(256), lds, st, fa);
    return launch_status("decode_fused");
  }
  cd::AttendArgs aa{};
  aa.q = q_t; aa.q_is_window = 0; aa.k = k_c; aa.v = v_c; aa.row_off = cache_offsets; aa.row_len = cache_lens;
  aa.bitmap = nullptr; aa.total_tokens = 0; aa.batch = p->batch; aa.Hq = p->n_q_heads; aa.Hkv = p->n_kv_heads;
  aa.G = G; aa.w = p->window; aa.B = p->budget; aa.max_len = max_cache_len; aa.W32 = 0;
  aa.rows_per_split = L.sp.rows_per_split; aa.NS = L.sp.NS; aa.sl2 = logit_scale(p) * cd::kLog2e;
  aa.cal_logit = nullptr; aa.zstride = 0;
  aa.part_o = reinterpret_cast<float*>(ws + L.part_o);
  aa.part_ml = reinterpret_cast<float2*>(ws + L.part_ml);
  launch_kv_pass<T, D>(aa, dim3(L.sp.NS, p->n_kv_heads, p->batch), static_cast<int64_t>(p->batch) * max_cache_len, st);
  if ((rc = launch_status("attend_partial(decode)"))) return rc;
  cd::FinalArgs fa{};
  fa.part_o = aa.part_o; fa.part_ml = aa.part_ml; fa.row_off = cache_offsets; fa.row_len = cache_lens;
  fa.total_tokens = 0; fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G;
  fa.w = p->window; fa.B = p->budget; fa.max_len = max_cache_len; fa.rows_per_split = L.sp.rows_per_split;
  fa.NS = L.sp.NS; fa.calib_mode = 0; fa.q_is_window = 0; fa.q = q_t; fa.theta1 = p->theta1; fa.theta2 = p->theta2;
  fa.c_q = const_cast<float*>(c_q); fa.c_out = const_cast<float*>(c_out); fa.c_lse = const_cast<float*>(c_lse);
  fa.out = out; fa.a_lse = a_lse; fa.flags = flags;
  return launch_finalize<T, D>(p, fa, st, "attend_finalize(decode)");
}

struct RecalLayout { size_t bitmap, part_o, part_ml, total; int W32; SplitPlan sp; };

RecalLayout recal_layout(const calidrop_params* p, int32_t max_seq_len) {
  RecalLayout L{};
  L.W32 = ceil_div(max_seq_len, 64) * 2;
  L.sp = plan_splits(p->batch * p->n_kv_heads, max_seq_len, few_kv(p));
  const size_t slots = static_cast<size_t>(p->batch) * p->n_q_heads * most_splits(p->batch * p->n_kv_heads, max_seq_len, few_kv(p));
  size_t off = 0;
  L.bitmap = off;  off += round256(static_cast<size_t>(p->batch) * p->n_kv_heads * L.W32 * sizeof(uint32_t));
  L.part_o = off;  off += round256(slots * p->head_dim * sizeof(float));
  L.part_ml = off; off += round256(slots * sizeof(float2));
  L.total = off;
  return L;
}

template <typename T, int D>
int recal_impl(const calidrop_params* p, const void* q_t, const void* k, const void* v, const int32_t* seq_offsets,
               int64_t total_tokens, int32_t max_seq_len, const int32_t* indices, const int32_t* cal_indices,
               uint8_t* flags, const float* a_lse, void* out, float* c_q, float* c_out, float* c_lse, char* ws,
               const RecalLayout& L, hipStream_t st) {
  const int G = p->n_q_heads / p->n_kv_heads;
  int rc;
  // the skip bits: made by each workgroup of the pass from the position list while that list is short beside the rows it
  // streams, otherwise by a launch ahead
  const bool from_cal = p->calib_size > 0;
  const int list_len = from_cal ? p->calib_size : p->budget;
  const bool in_pass = L.sp.rows_per_split <= cd::kListMaxRows && list_len <= 2 * L.sp.rows_per_split;
  if (!in_pass) {
    cd::BitmapArgs ba{};
    ba.seq_off = seq_offsets; ba.indices = indices; ba.cal_indices = cal_indices;
    ba.bitmap = reinterpret_cast<uint32_t*>(ws + L.bitmap); ba.calib = p->calib_size;
    ba.total_tokens = total_tokens; ba.batch = p->batch; ba.Hkv = p->n_kv_heads; ba.B = p->budget;
    ba.max_seq_len = max_seq_len; ba.W32 = L.W32;
    ba.only_flagged = flags; ba.Hq = p->n_q_heads; ba.G = G;
    launch_bitmap(ba, p->batch * p->n_kv_heads, st);
    if ((rc = launch_status("bitmap_from_indices"))) return rc;
  }

  cd::AttendArgs aa{};
  aa.q = q_t; aa.q_is_window = 0; aa.k = k; aa.v = v; aa.row_off = seq_offsets; aa.row_len = nullptr;
  aa.bitmap = reinterpret_cast<uint32_t*>(ws + L.bitmap); aa.total_tokens = total_tokens; aa.batch = p->batch; aa.Hq = p->n_q_heads;
  // w = 0: the pass covers every position; the bitmap masks the retained ones, window included
  aa.Hkv = p->n_kv_heads; aa.G = G; aa.w = 0; aa.B = p->budget; aa.max_len = max_seq_len; aa.W32 = L.W32;
  aa.rows_per_split = L.sp.rows_per_split; aa.NS = L.sp.NS; aa.sl2 = logit_scale(p) * cd::kLog2e;
  aa.cal_logit = nullptr; aa.zstride = 0; aa.only_flagged = flags;
  aa.part_o = reinterpret_cast<float*>(ws + L.part_o);
  aa.part_ml = reinterpret_cast<float2*>(ws + L.part_ml);
  aa.list = from_cal ? cal_indices : indices; aa.list_len = list_len; aa.list_is_calib = from_cal;
  const dim3 grid(L.sp.NS, p->n_kv_heads, p->batch);
  if (in_pass) hipLaunchKernelGGL((cd::attend_partial_kernel<T, D, false, false, false, true>), grid, dim3(256), 0, st, aa);
  else launch_kv_pass<T, D>(aa, grid, total_tokens, st);
  if ((rc = launch_status("attend_partial(recalibrate)"))) return rc;

  cd::FinalArgs fa{};
  fa.part_o = aa.part_o; fa.part_ml = aa.part_ml; fa.row_off = seq_offsets; fa.row_len = nullptr;
  fa.total_tokens = total_tokens; fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G;
  fa.w = 0; fa.B = p->budget; fa.max_len = max_seq_len; fa.rows_per_split = L.sp.rows_per_split;
  fa.NS = L.sp.NS; fa.calib_mode = 2; fa.q_is_window = 0; fa.q = q_t;
  fa.c_q = c_q; fa.c_out = c_out; fa.c_lse = c_lse; fa.out = out; fa.a_lse = const_cast<float*>(a_lse); fa.flags = flags;
  return launch_finalize<T, D>(p, fa, st, "attend_finalize(recalibrate)");
}

// Skip bitmap of a sequence in LDS (131072 positions) for the given-set preparation; the gather blocks that share its
// launch then still fit eight to a compute unit.
constexpr size_t kGivenLdsBytes = 16 * 1024;

// Alg. 1 steps 4-8 for a retained set that is already known (caller's strategy, or the
// StreamingLLM list): bitmap + cache_lens, gather, calibration pass over everything else.
template <typename T, int D>
int compress_given_impl(const calidrop_params* p, const void* q_cal, const void* k, const void* v,
                        const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len, int32_t* indices,
                        void* k_c, void* v_c, const int32_t* cache_offsets, int32_t* cache_lens, float* c_q,
                        float* c_out, float* c_lse, char* ws, const RecalLayout& L, hipStream_t st) {
  const int G = p->n_q_heads / p->n_kv_heads;
  const int bg = p->batch * p->n_kv_heads;
  int rc;
  cd::GivenArgs ga{};
  ga.seq_off = seq_offsets; ga.total_tokens = total_tokens; ga.batch = p->batch; ga.Hkv = p->n_kv_heads;
  ga.B = p->budget; ga.max_seq_len = max_seq_len; ga.W32 = L.W32; ga.indices = indices; ga.cache_lens = cache_lens;
  ga.bitmap = reinterpret_cast<uint32_t*>(ws + L.bitmap);
  // the gather needs nothing the preparation produces: both in one launch, the bitmaps first
  const cd::GatherArgs gather = gather_args(p, indices, cache_offsets, k, v, k_c, v_c);
  const size_t lds = static_cast<size_t>(L.W32) * sizeof(uint32_t);
  const bool in_lds = lds <= kGivenLdsBytes;
  ga.gather = gather;
  const dim3 grid_p(in_lds ? 1 + gather.blocks : 1, bg);
  if (in_lds) hipLaunchKernelGGL(cd::given_prepare_kernel<true>, grid_p, dim3(256), lds, st, ga);
  else hipLaunchKernelGGL(cd::given_prepare_kernel<false>, grid_p, dim3(256), 0, st, ga);
  if ((rc = launch_status("given_prepare"))) return rc;

  cd::AttendArgs aa{};
  aa.q = q_cal; aa.q_is_window = 0; aa.k = k; aa.v = v; aa.row_off = seq_offsets; aa.row_len = nullptr;
  aa.bitmap = ga.bitmap; aa.total_tokens = total_tokens; aa.batch = p->batch; aa.Hq = p->n_q_heads;
  aa.Hkv = p->n_kv_heads; aa.G = G; aa.w = 0; aa.B = p->budget; aa.max_len = max_seq_len; aa.W32 = L.W32;
  aa.rows_per_split = L.sp.rows_per_split; aa.NS = L.sp.NS; aa.sl2 = logit_scale(p) * cd::kLog2e;
  aa.part_o = reinterpret_cast<float*>(ws + L.part_o);
  aa.part_ml = reinterpret_cast<float2*>(ws + L.part_ml);
  const cd::GatherArgs* left;
  if ((rc = launch_calibration<T, D>(p, aa, gather, in_lds ? GatherIn::kDone : GatherIn::kAfter, st, &left))) return rc;
  cd::FinalArgs fa{};
  fa.part_o = aa.part_o; fa.part_ml = aa.part_ml; fa.row_off = seq_offsets; fa.row_len = nullptr;
  fa.total_tokens = total_tokens; fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G;
  fa.w = 0; fa.B = p->budget; fa.max_len = max_seq_len; fa.rows_per_split = L.sp.rows_per_split;
  fa.NS = L.sp.NS; fa.calib_mode = 1; fa.q_is_window = 0; fa.q = q_cal;
  fa.c_q = c_q; fa.c_out = c_out; fa.c_lse = c_lse;
  return launch_finalize<T, D>(p, fa, st, "attend_finalize(given)", left);
}

int packed_rows_host(const calidrop_params* p, int n) {
  if (n <= p->budget) return 0;
  return p->calib_size > 0 ? std::min(p->calib_size, n - p->budget) : n - p->budget;
}

struct PackLayout { size_t bitmap, total; int W32; };
PackLayout pack_layout(const calidrop_params* p, int32_t max_seq_len) {
  PackLayout L{};
  L.W32 = ceil_div(max_seq_len, 64) * 2;
  L.bitmap = 0;
  L.total = round256(static_cast<size_t>(p->batch) * p->n_kv_heads * L.W32 * sizeof(uint32_t));
  return L;
}

// KV_evict (or the calibration set) of every head as contiguous rows, ready to be moved elsewhere.
int pack_impl(const calidrop_params* p, const void* k, const void* v, const int32_t* seq_offsets, int64_t total_tokens,
              int32_t max_seq_len, const int32_t* indices, const int32_t* cal_indices, void* k_e, void* v_e,
              const int32_t* evict_offsets, int32_t* evict_lens, int32_t* evict_indices, char* ws,
              const PackLayout& L, hipStream_t st) {
  int rc;
  const int bg = p->batch * p->n_kv_heads;
  cd::BitmapArgs ba{};
  ba.seq_off = seq_offsets; ba.indices = indices; ba.cal_indices = cal_indices;
  ba.bitmap = reinterpret_cast<uint32_t*>(ws + L.bitmap); ba.calib = p->calib_size;
  ba.total_tokens = total_tokens; ba.batch = p->batch; ba.Hkv = p->n_kv_heads; ba.B = p->budget;
  ba.max_seq_len = max_seq_len; ba.W32 = L.W32;
  ba.only_flagged = nullptr; ba.Hq = p->n_q_heads; ba.G = p->n_q_heads / p->n_kv_heads;
  launch_bitmap(ba, bg, st);
  if ((rc = launch_status("bitmap_from_indices"))) return rc;
  cd::PackArgs pa{};
  pa.seq_off = seq_offsets; pa.evict_off = evict_offsets; pa.total_tokens = total_tokens; pa.batch = p->batch;
  pa.Hkv = p->n_kv_heads; pa.B = p->budget; pa.calib = p->calib_size; pa.max_seq_len = max_seq_len; pa.W32 = L.W32;
  pa.row_bytes = p->head_dim * (p->dtype == CALIDROP_BF16 ? 2 : 4);
  pa.bitmap = ba.bitmap; pa.evict_lens = evict_lens; pa.evict_indices = evict_indices;
  pa.k = k; pa.v = v; pa.k_e = k_e; pa.v_e = v_e;
  hipLaunchKernelGGL(cd::evict_list_kernel, dim3(bg), dim3(256), 0, st, pa);
  if ((rc = launch_status("evict_list"))) return rc;
  const int max_rows = packed_rows_host(p, max_seq_len);
  if (max_rows > 0) {
    const int64_t vecs = static_cast<int64_t>(max_rows) * (pa.row_bytes / 16);
    hipLaunchKernelGGL(cd::pack_gather_kernel, dim3(static_cast<unsigned>((vecs + 255) / 256), bg), dim3(256), 0, st, pa);
    if ((rc = launch_status("pack_gather"))) return rc;
  }
  return CALIDROP_OK;
}

// Recomputation branch over the packed rows: the same streaming pass and tail as calidrop_recalibrate,
// with the geometry of a packed buffer (offsets + live rows) instead of a prompt and its skip bitmap.
bool is_host_memory(const void* ptr) {
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, ptr) != hipSuccess) {
    (void)hipGetLastError();                     // a pointer the runtime does not know: treat as device memory
    return false;
  }
  return attr.type == hipMemoryTypeHost;
}

template <typename T, int D>
int recal_packed_impl(const calidrop_params* p, const void* q_t, const void* k_e, const void* v_e,
                      const int32_t* evict_offsets, const int32_t* evict_lens, int32_t max_evict_len, uint8_t* flags,
                      const float* a_lse, void* out, float* c_q, float* c_out, float* c_lse, char* ws,
                      const DecodeLayout& L, hipStream_t st) {
  const int G = p->n_q_heads / p->n_kv_heads;
  int rc;
  cd::AttendArgs aa{};
  aa.q = q_t; aa.q_is_window = 0; aa.k = k_e; aa.v = v_e; aa.row_off = evict_offsets; aa.row_len = evict_lens;
  aa.bitmap = nullptr; aa.total_tokens = 0; aa.batch = p->batch; aa.Hq = p->n_q_heads; aa.Hkv = p->n_kv_heads;
  aa.G = G; aa.w = 0; aa.B = p->budget; aa.max_len = max_evict_len; aa.W32 = 0;
  aa.rows_per_split = L.sp.rows_per_split; aa.NS = L.sp.NS; aa.sl2 = logit_scale(p) * cd::kLog2e;
  aa.only_flagged = flags;
  aa.part_o = reinterpret_cast<float*>(ws + L.part_o);
  aa.part_ml = reinterpret_cast<float2*>(ws + L.part_ml);
  // rows in host memory (the offloaded form) are requested as whole rows: the host link moves the
  // 64-byte pieces of the operand layout a quarter slower
  const dim3 grid(L.sp.NS, p->n_kv_heads, p->batch);
  if (is_host_memory(k_e)) hipLaunchKernelGGL((cd::attend_partial_kernel<T, D, false, true>), grid, dim3(256), 0, st, aa);
  else launch_kv_pass<T, D>(aa, grid, static_cast<int64_t>(p->batch) * max_evict_len, st);
  if ((rc = launch_status("attend_partial(recalibrate, packed)"))) return rc;
  cd::FinalArgs fa{};
  fa.part_o = aa.part_o; fa.part_ml = aa.part_ml; fa.row_off = evict_offsets; fa.row_len = evict_lens;
  fa.total_tokens = 0; fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G;
  fa.w = 0; fa.B = p->budget; fa.max_len = max_evict_len; fa.rows_per_split = L.sp.rows_per_split;
  fa.NS = L.sp.NS; fa.calib_mode = 2; fa.q_is_window = 0; fa.q = q_t;
  fa.c_q = c_q; fa.c_out = c_out; fa.c_lse = c_lse; fa.out = out; fa.a_lse = const_cast<float*>(a_lse); fa.flags = flags;
  return launch_finalize<T, D>(p, fa, st, "attend_finalize(recalibrate, packed)");
}

// Shares into which the streams of a call of few workgroups are cut (blocks: 128-row blocks of all heads of the longest
// prompt).  us for one layer in 1 -> 2 -> 4 shares: bf16, D = 128, 8 heads x 1793 rows (120 blocks) 74 -> 54 -> 45, 8 x 5000
// (320) 169 -> 115 -> 100, 8 x 10000 (632) 364 -> 286 -> 261; 32 heads x 700 (192) 43 -> 40 -> 40, 32 x 2600 (672) 126 -> 103
// -> 107, 32 x 10000 (2528) 964 -> 900 -> 888; 64 x 700 (384) 45 -> 45 -> 48, 64 x 1793 (960) 108 -> 104 -> 110, 64 x 5000
// (2560) 525 -> 494 -> 494, 64 x 10000 (5056) 1774 -> 1728 -> 1732.  fp32, 8 x 1100, D = 128 (72) 196 -> 117 -> 78, 32 x 1100,
// D = 64 (288) 136 -> 115 -> 98, 64 x 3000 (1536) 777 -> 731 -> 701.  So four shares of fp32 streams (long ones, for the
// matrix cores run at an eighth) and of few heads, two otherwise; beyond 2560 blocks 2 to 3 % are left and the planes grow.
constexpr int64_t kH2oSplitBlocks = 2560;
int64_t h2o_blocks(const calidrop_params* p, int32_t max_seq_len) {
  return static_cast<int64_t>(ceil_div(max_seq_len, cd::h2o_block(2))) * p->batch * p->n_q_heads;
}
// What the calls of these heads are cut into whatever their prompts: the room a workspace has for shares.
int h2o_most_splits(const calidrop_params* p) {
  if (h2o_blocks(p, 1) > kH2oSplitBlocks) return 1;
  return p->dtype == CALIDROP_FP32 || p->batch * p->n_q_heads < 32 ? 4 : 2;
}
int h2o_splits(const calidrop_params* p, int32_t max_seq_len) {
  return h2o_blocks(p, max_seq_len) > kH2oSplitBlocks ? 1 : h2o_most_splits(p);
}

struct H2oLayout {
  size_t row_part, row_lse, vote, score, bitmap, q_last, part_o, part_ml, sel_hist, sel_cnt, total;
  int lse_stride, W32, NSEG, splits;
  SplitPlan sp;
};

H2oLayout h2o_layout(const calidrop_params* p, int64_t total_tokens, int32_t max_seq_len, int n_local) {
  H2oLayout L{};
  L.lse_stride = ceil_div(max_seq_len, 256) * 256;
  L.W32 = ceil_div(max_seq_len, 64) * 2;
  L.sp = plan_splits(p->batch * p->n_kv_heads, max_seq_len, few_kv(p));
  L.NSEG = ceil_div(std::max(max_seq_len - n_local, 1), cd::kWideSeg);
  const size_t toks = static_cast<size_t>(total_tokens) * p->n_kv_heads;
  const size_t slots = static_cast<size_t>(p->batch) * p->n_q_heads * most_splits(p->batch * p->n_kv_heads, max_seq_len, few_kv(p));
  size_t off = 0;
  L.row_lse = off; off += round256(static_cast<size_t>(p->batch) * p->n_q_heads * L.lse_stride * sizeof(float));
  L.splits = h2o_splits(p, max_seq_len);
  L.vote = off;    // one plane per head of a group and share
  {
    // What splits needs, for this and any shorter prompts, so that sizes do not fall as prompts grow: a call with more than one
    // share has at most kH2oSplitBlocks blocks, so no more than `few` tokens.
    const int most = h2o_most_splits(p);
    const int64_t few = std::min<int64_t>(total_tokens, kH2oSplitBlocks * cd::h2o_block(2) / p->n_q_heads + 1);
    const int64_t plane = std::max(vote_plane(total_tokens, p->n_kv_heads), most * vote_plane(few, p->n_kv_heads));
    off += round256(static_cast<size_t>(plane) * (p->n_q_heads / p->n_kv_heads) * sizeof(float));
    L.row_part = off;
    if (most > 1) {
      const int64_t heads = static_cast<int64_t>(p->batch) * p->n_q_heads;
      const int64_t rows = std::min(heads * L.lse_stride, kH2oSplitBlocks * cd::h2o_block(2) + heads * 256);
      off += round256(static_cast<size_t>(rows) * most * sizeof(float2));
    }
  }
  L.score = off;   off += round256(toks * sizeof(float));
  L.bitmap = off;  off += round256(static_cast<size_t>(p->batch) * p->n_kv_heads * L.W32 * sizeof(uint32_t));
  L.q_last = off;  off += round256(static_cast<size_t>(p->batch) * p->n_q_heads * p->head_dim * sizeof(float));
  L.part_o = off;  off += round256(slots * p->head_dim * sizeof(float));
  L.part_ml = off; off += round256(slots * sizeof(float2));
  const WideRegions wide = wide_regions(p, n_local, 1, max_seq_len, L.NSEG);
  L.sel_hist = off; off += wide.hist;
  L.sel_cnt = off;  off += wide.seg;
  L.total = off;
  return L;
}

// Alg. 1 steps 3-8 with H2O as f: accumulated attention of every prompt query (two dense passes),
// top-(B - n_local) among the positions outside the local window, gather, calibration state.
// Blocks of 256 stationary rows from which a call of H2O uses them (bf16): five and a half rounds of two workgroups on
// each of the 256 compute units.  Below that 128-row blocks, twice as many workgroups, win or are within 3 %: one prompt,
// 32 heads, 2573 tokens 130 us against 174, 8192 tokens 605 / 640, 12000 tokens (1504 blocks) 1209 / 1272, 16384 2235 /
// 2170, 20000 (2528 blocks) 3270 / 3330; above it 24000 (3008) 4596 / 4368, 28000 6226 / 6250, 32768 8.2 / 7.9 ms.
constexpr int64_t kH2oWideBlocks = 2816;
template <typename T, int D>
int h2o_impl(const calidrop_params* p, int n_local, const void* q_full, const void* k, const void* v,
             const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len, void* k_c, void* v_c,
             const int32_t* cache_offsets, int32_t* cache_lens, int32_t* indices, int32_t* cal_indices, float* c_q,
             float* c_out, float* c_lse, char* ws, const H2oLayout& L, hipStream_t st) {
  const int G = p->n_q_heads / p->n_kv_heads;
  const int bg = p->batch * p->n_kv_heads;
  const float sl2 = logit_scale(p) * cd::kLog2e;
  int rc;
  cd::H2oArgs ha{};
  ha.q_full = q_full; ha.k = k; ha.seq_off = seq_offsets; ha.total_tokens = total_tokens; ha.batch = p->batch;
  ha.Hq = p->n_q_heads; ha.Hkv = p->n_kv_heads; ha.G = G; ha.B = p->budget; ha.max_seq_len = max_seq_len;
  ha.lse_stride = L.lse_stride; ha.sl2 = sl2;
  ha.row_lse = reinterpret_cast<float*>(ws + L.row_lse);
  ha.splits = L.splits; ha.row_part = reinterpret_cast<float2*>(ws + L.row_part);
  ha.vote = reinterpret_cast<float*>(ws + L.vote);
  ha.plane = vote_plane(total_tokens, p->n_kv_heads);
  ha.q_last = ws + L.q_last;
  if (!uses_lds_selection(p, n_local, 1, max_seq_len)) {
    ha.zero_words = reinterpret_cast<uint32_t*>(ws + L.sel_hist); ha.zero_count = wide_words(p);
  }
  auto passes = [&](auto tiles, auto split) {
    constexpr int RT = decltype(tiles)::value;
    constexpr bool kSplit = decltype(split)::value;
    const int nblk = ceil_div(max_seq_len, cd::h2o_block(RT));     // blocks of stationary rows (or keys)
    // always launched: it also extracts Q_{-1}, which prompts within the budget need as C_q
    hipLaunchKernelGGL((cd::h2o_rowlse_kernel<T, D, RT, kSplit>), dim3(nblk * L.splits, p->batch * p->n_q_heads), dim3(256), 0, st, ha);
    if (int e = launch_status("h2o_rowlse")) return e;
    if (max_seq_len <= p->budget) return static_cast<int>(CALIDROP_OK);
    if constexpr (kSplit) {
      hipLaunchKernelGGL(cd::h2o_rowmerge_kernel, dim3(ceil_div(L.lse_stride, 256), p->batch * p->n_q_heads), dim3(256), 0, st, ha, cd::h2o_block(RT));
      if (int e = launch_status("h2o_rowmerge")) return e;
    }
    const dim3 pairs((nblk + 1) / 2, bg, G * L.splits);
    if constexpr (kSplit) hipLaunchKernelGGL((cd::h2o_shared_votes_kernel<T, D, RT>), pairs, dim3(256), 0, st, ha);
    else hipLaunchKernelGGL((cd::h2o_votes_kernel<T, D, RT>), pairs, dim3(256), 0, st, ha);
    return launch_status("h2o_votes");
  };
  using std::integral_constant;
  const int64_t blocks = static_cast<int64_t>(ceil_div(max_seq_len, cd::h2o_block(4))) * p->batch * p->n_q_heads;
  if (L.splits > 1) rc = passes(integral_constant<int, 2>{}, std::true_type{});
  else if constexpr (sizeof(T) == 2) rc = blocks >= kH2oWideBlocks ? passes(integral_constant<int, 4>{}, std::false_type{}) : passes(integral_constant<int, 2>{}, std::false_type{});
  else rc = passes(integral_constant<int, 2>{}, std::false_type{});
  if (rc) return rc;
  // selection: the votes are the scores (no pooling); the local window plays the part of the
  // observation window (always kept, not a candidate)
  const cd::GatherArgs ga = gather_args(p, indices, cache_offsets, k, v, k_c, v_c);
  GatherIn place;
  cd::SelectArgs se{};
  se.gather = ga;
  se.seq_off = seq_offsets; se.total_tokens = total_tokens; se.batch = p->batch;
  se.Hkv = p->n_kv_heads; se.w = n_local; se.B = p->budget; se.max_seq_len = max_seq_len; se.W32 = L.W32;
  se.NRB = G * L.splits; se.pool_k = 1;
  se.vote = ha.vote; se.plane = ha.plane; se.score = reinterpret_cast<float*>(ws + L.score); se.indices = indices; se.cache_lens = cache_lens;
  se.calib = p->calib_size; se.cal_indices = cal_indices;
  se.bitmap = reinterpret_cast<uint32_t*>(ws + L.bitmap);
  if ((rc = run_selection(p, max_seq_len, se, reinterpret_cast<uint32_t*>(ws + L.sel_hist),
                          reinterpret_cast<uint32_t*>(ws + L.sel_cnt), L.NSEG, L.sp.rows_per_split, place, st)))
    return rc;

  cd::AttendArgs aa{};
  aa.q = ha.q_last; aa.q_is_window = 0; aa.k = k; aa.v = v; aa.row_off = seq_offsets; aa.row_len = nullptr;
  aa.bitmap = se.bitmap; aa.total_tokens = total_tokens; aa.batch = p->batch; aa.Hq = p->n_q_heads;
  aa.Hkv = p->n_kv_heads; aa.G = G; aa.w = n_local; aa.B = p->budget; aa.max_len = max_seq_len; aa.W32 = L.W32;
  aa.rows_per_split = L.sp.rows_per_split; aa.NS = L.sp.NS; aa.sl2 = sl2;
  aa.part_o = reinterpret_cast<float*>(ws + L.part_o);
  aa.part_ml = reinterpret_cast<float2*>(ws + L.part_ml);
  const cd::GatherArgs* left;
  if ((rc = launch_calibration<T, D>(p, aa, ga, place, st, &left))) return rc;
  cd::FinalArgs fa{};
  fa.part_o = aa.part_o; fa.part_ml = aa.part_ml; fa.row_off = seq_offsets; fa.row_len = nullptr;
  fa.total_tokens = total_tokens; fa.batch = p->batch; fa.Hq = p->n_q_heads; fa.Hkv = p->n_kv_heads; fa.G = G;
  fa.w = n_local; fa.B = p->budget; fa.max_len = max_seq_len; fa.rows_per_split = L.sp.rows_per_split;
  fa.NS = L.sp.NS; fa.calib_mode = 1; fa.q_is_window = 0; fa.q = ha.q_last;
  fa.c_q = c_q; fa.c_out = c_out; fa.c_lse = c_lse;
  return launch_finalize<T, D>(p, fa, st, "attend_finalize(h2o)", left);
}

}  // namespace

extern "C" {

const char* calidrop_last_error(void) { return g_err; }
int calidrop_version(void) { return 200; }

size_t calidrop_compress_workspace_bytes(const calidrop_params* p_in, int64_t total_tokens, int32_t max_seq_len) {
  calidrop_params pp; const calidrop_params* p = &pp;
  if (load_params(p_in, &pp) != CALIDROP_OK) return 0;
  if (check_params(p) != CALIDROP_OK || check_sizes(p, total_tokens, max_seq_len) != CALIDROP_OK) return 0;
  return compress_layout(p, total_tokens, max_seq_len).total;
}

size_t calidrop_decode_workspace_bytes(const calidrop_params* p_in, int32_t max_cache_len) {
  calidrop_params pp; const calidrop_params* p = &pp;
  if (load_params(p_in, &pp) != CALIDROP_OK) return 0;
  if (check_params(p) != CALIDROP_OK) return 0;
  if (max_cache_len < 1) { fail(CALIDROP_ESHAPE, "max_cache_len must be >= 1"); return 0; }
  return decode_layout(p, max_cache_len).total;
}

int calidrop_compress_workspace_region(const calidrop_params* p_in, int64_t total_tokens, int32_t max_seq_len,
                                       int32_t region, size_t* offset, size_t* bytes) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  if (!offset || !bytes) return fail(CALIDROP_EINVAL, "offset/bytes is NULL");
  const CompressLayout L = compress_layout(p, total_tokens, max_seq_len);
  if (region == CALIDROP_REGION_ROW_LSE) {
    *offset = L.row_lse;
    *bytes = static_cast<size_t>(p->batch) * p->n_kv_heads * L.NRB * L.RB * sizeof(float);
  } else if (region == CALIDROP_REGION_SCORE) {
    *offset = L.score;
    *bytes = static_cast<size_t>(total_tokens) * p->n_kv_heads * sizeof(float);
  } else if (region == CALIDROP_REGION_ROW_PARTS) {
    *offset = L.rowpart;
    *bytes = static_cast<size_t>(p->batch) * p->n_kv_heads * L.NRB * L.RB * L.NCH * sizeof(float2);
  } else {
    return fail(CALIDROP_EINVAL, "unknown workspace region %d", region);
  }
  return CALIDROP_OK;
}

int calidrop_compress(const calidrop_params* p_in, const void* q_win, const void* k, const void* v,
                      const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len, const void* q_cal,
                      void* k_c, void* v_c, const int32_t* cache_offsets, int32_t* cache_lens, int32_t* indices,
                      int32_t* cal_indices, float* c_q, float* c_out, float* c_lse, void* workspace,
                      size_t workspace_bytes, void* stream) {
  return calidrop_compress_with_lse(p_in, q_win, k, v, seq_offsets, total_tokens, max_seq_len, nullptr, q_cal, k_c, v_c,
                                    cache_offsets, cache_lens, indices, cal_indices, c_q, c_out, c_lse, workspace,
                                    workspace_bytes, stream);
}

int calidrop_compress_with_lse(const calidrop_params* p_in, const void* q_win, const void* k, const void* v,
                               const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len,
                               const float* win_lse, const void* q_cal, void* k_c, void* v_c,
                               const int32_t* cache_offsets, int32_t* cache_lens, int32_t* indices,
                               int32_t* cal_indices, float* c_q, float* c_out, float* c_lse, void* workspace,
                               size_t workspace_bytes, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  const struct { const void* ptr; const char* name; } req[] = {
      {q_win, "q_win"}, {k, "k"}, {v, "v"}, {seq_offsets, "seq_offsets"}, {k_c, "k_c"}, {v_c, "v_c"},
      {cache_offsets, "cache_offsets"}, {cache_lens, "cache_lens"}, {indices, "indices"}, {c_q, "c_q"},
      {c_out, "c_out"}, {c_lse, "c_lse"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (!aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  if (q_cal && !aligned16(q_cal)) return fail(CALIDROP_EALIGN, "q_cal is not 16-byte aligned");
  if (win_lse && !aligned16(win_lse)) return fail(CALIDROP_EALIGN, "win_lse is not 16-byte aligned");
  if (p->calib_size > 0) {
    if (!cal_indices) return fail(CALIDROP_EINVAL, "cal_indices is NULL although calib_size is %d", p->calib_size);
    if (!aligned16(cal_indices)) return fail(CALIDROP_EALIGN, "cal_indices is not 16-byte aligned");
  } else {
    cal_indices = nullptr;
  }
  const CompressLayout L = compress_layout(p, total_tokens, max_seq_len);
  if (!workspace || workspace_bytes < L.total)
    return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                L.total);
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
#define CD_DISPATCH(T, D)                                                                                       \
  return compress_impl<T, D>(p, q_win, k, v, seq_offsets, total_tokens, max_seq_len, win_lse, q_cal, k_c, v_c,  \
                             cache_offsets, cache_lens, indices, cal_indices, c_q, c_out, c_lse, ws, L, st)
  if (p->dtype == CALIDROP_BF16) {
    if (p->head_dim == 128) CD_DISPATCH(cd::bf16_t, 128);
    CD_DISPATCH(cd::bf16_t, 64);
  }
  if (p->head_dim == 128) CD_DISPATCH(float, 128);
  CD_DISPATCH(float, 64);
#undef CD_DISPATCH
}

namespace {
// calidrop_decode and calidrop_decode_static: the same validation and launches; they differ in where
// the scratch for the split partials comes from (the caller's workspace, or the fixed per-GPU array).
int decode_entry(const calidrop_params* p_in, const void* q_t, const void* k_c, const void* v_c,
                 const int32_t* cache_offsets, const int32_t* cache_lens, int32_t max_cache_len, const float* c_q,
                 const float* c_out, const float* c_lse, void* out, float* a_lse, uint8_t* flags, void* workspace,
                 size_t workspace_bytes, bool fixed_scratch, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if (max_cache_len < 1) return fail(CALIDROP_ESHAPE, "max_cache_len must be >= 1 (got %d)", max_cache_len);
  const struct { const void* ptr; const char* name; } req[] = {
      {q_t, "q_t"}, {k_c, "k_c"}, {v_c, "v_c"}, {cache_lens, "cache_lens"},
      {c_q, "c_q"}, {c_out, "c_out"}, {c_lse, "c_lse"}, {out, "out"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (!aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  if (cache_offsets) {
    if (!aligned16(cache_offsets)) return fail(CALIDROP_EALIGN, "cache_offsets is not 16-byte aligned");
  } else if (static_cast<int64_t>(p->batch) * max_cache_len > (static_cast<int64_t>(1) << 31) - 1) {
    return fail(CALIDROP_EUNSUPPORTED, "batch * max_cache_len exceeds int32 offsets (uniform layout)");
  }
  const DecodeLayout L = decode_layout(p, max_cache_len);
  char* ws = static_cast<char*>(workspace);
  if (fixed_scratch) {
    if (L.used > kStaticScratchBytes)
      return fail(CALIDROP_EWORKSPACE, "this call needs %zu bytes of scratch and the fixed array holds %zu: use "
                  "calidrop_decode with a workspace", L.used, kStaticScratchBytes);
    if ((rc = static_scratch_ptr(&ws))) return rc;       // the first HIP call, after all validation
  } else {
    if (!workspace || workspace_bytes < L.total)
      return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                  L.total);
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
#define CD_DISPATCH(T, D)                                                                                      \
  return decode_impl<T, D>(p, q_t, k_c, v_c, cache_offsets, cache_lens, max_cache_len, c_q, c_out, c_lse, out, \
                           a_lse, flags, ws, L, st)
  if (p->dtype == CALIDROP_BF16) {
    if (p->head_dim == 128) CD_DISPATCH(cd::bf16_t, 128);
    CD_DISPATCH(cd::bf16_t, 64);
  }
  if (p->head_dim == 128) CD_DISPATCH(float, 128);
  CD_DISPATCH(float, 64);
#undef CD_DISPATCH
}
}  // namespace

int calidrop_decode(const calidrop_params* p_in, const void* q_t, const void* k_c, const void* v_c,
                    const int32_t* cache_offsets, const int32_t* cache_lens, int32_t max_cache_len,
                    const float* c_q, const float* c_out, const float* c_lse, void* out, float* a_lse,
                    uint8_t* flags, void* workspace, size_t workspace_bytes, void* stream) {
  return decode_entry(p_in, q_t, k_c, v_c, cache_offsets, cache_lens, max_cache_len, c_q, c_out, c_lse, out, a_lse,
                      flags, workspace, workspace_bytes, false, stream);
}

int calidrop_decode_static(const calidrop_params* p_in, const void* q_t, const void* k_c, const void* v_c,
                           const int32_t* cache_offsets, const int32_t* cache_lens, int32_t max_cache_len,
                           const float* c_q, const float* c_out, const float* c_lse, void* out, float* a_lse,
                           uint8_t* flags, void* stream) {
  return decode_entry(p_in, q_t, k_c, v_c, cache_offsets, cache_lens, max_cache_len, c_q, c_out, c_lse, out, a_lse,
                      flags, nullptr, 0, true, stream);
}

size_t calidrop_recalibrate_workspace_bytes(const calidrop_params* p_in, int32_t max_seq_len) {
  calidrop_params pp; const calidrop_params* p = &pp;
  if (load_params(p_in, &pp) != CALIDROP_OK) return 0;
  if (check_params(p) != CALIDROP_OK) return 0;
  if (max_seq_len < 1) { fail(CALIDROP_ESHAPE, "max_seq_len must be >= 1"); return 0; }
  return recal_layout(p, max_seq_len).total;
}

int calidrop_recalibrate(const calidrop_params* p_in, const void* q_t, const void* k, const void* v,
                         const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len,
                         const int32_t* indices, const int32_t* cal_indices, uint8_t* flags, const float* a_lse,
                         void* out, float* c_q, float* c_out, float* c_lse, void* workspace, size_t workspace_bytes,
                         void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  const struct { const void* ptr; const char* name; } req[] = {
      {q_t, "q_t"}, {k, "k"}, {v, "v"}, {seq_offsets, "seq_offsets"}, {indices, "indices"}, {flags, "flags"},
      {a_lse, "a_lse"}, {out, "out"}, {c_q, "c_q"}, {c_out, "c_out"}, {c_lse, "c_lse"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (r.ptr != flags && !aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  if (p->calib_size > 0) {
    if (!cal_indices) return fail(CALIDROP_EINVAL, "cal_indices is NULL although calib_size is %d", p->calib_size);
    if (!aligned16(cal_indices)) return fail(CALIDROP_EALIGN, "cal_indices is not 16-byte aligned");
  } else {
    cal_indices = nullptr;
  }
  const RecalLayout L = recal_layout(p, max_seq_len);
  if (!workspace || workspace_bytes < L.total)
    return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                L.total);
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
#define CD_DISPATCH(T, D)                                                                                        \
  return recal_impl<T, D>(p, q_t, k, v, seq_offsets, total_tokens, max_seq_len, indices, cal_indices, flags, a_lse, \
                          out, c_q, c_out, c_lse, ws, L, st)
  if (p->dtype == CALIDROP_BF16) {
    if (p->head_dim == 128) CD_DISPATCH(cd::bf16_t, 128);
    CD_DISPATCH(cd::bf16_t, 64);
  }
  if (p->head_dim == 128) CD_DISPATCH(float, 128);
  CD_DISPATCH(float, 64);
#undef CD_DISPATCH
}

size_t calidrop_compress_given_workspace_bytes(const calidrop_params* p_in, int32_t max_seq_len) {
  return calidrop_recalibrate_workspace_bytes(p_in, max_seq_len);   // same regions: bitmap + split partials
}

int calidrop_streaming_indices(const calidrop_params* p_in, int32_t n_sink, const int32_t* seq_offsets,
                               int64_t total_tokens, int32_t max_seq_len, int32_t* indices, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  if (n_sink < 0 || n_sink > p->budget)
    return fail(CALIDROP_EINVAL, "n_sink must lie in [0, budget] (got %d, budget %d)", n_sink, p->budget);
  if (!seq_offsets) return fail(CALIDROP_EINVAL, "seq_offsets is NULL");
  if (!indices) return fail(CALIDROP_EINVAL, "indices is NULL");
  if (!aligned16(seq_offsets) || !aligned16(indices))
    return fail(CALIDROP_EALIGN, "seq_offsets / indices is not 16-byte aligned");
  cd::StreamingArgs sa{};
  sa.seq_off = seq_offsets; sa.total_tokens = total_tokens; sa.batch = p->batch; sa.Hkv = p->n_kv_heads;
  sa.B = p->budget; sa.n_sink = n_sink; sa.max_seq_len = max_seq_len; sa.indices = indices;
  hipLaunchKernelGGL(cd::streaming_indices_kernel, dim3(ceil_div(p->budget, 256), p->batch * p->n_kv_heads), dim3(256),
                     0, static_cast<hipStream_t>(stream), sa);
  return launch_status("streaming_indices");
}

int calidrop_compress_given(const calidrop_params* p_in, const void* q_cal, const void* k, const void* v,
                            const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len, int32_t* indices,
                            void* k_c, void* v_c, const int32_t* cache_offsets, int32_t* cache_lens, float* c_q,
                            float* c_out, float* c_lse, void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  const struct { const void* ptr; const char* name; } req[] = {
      {q_cal, "q_cal"}, {k, "k"}, {v, "v"}, {seq_offsets, "seq_offsets"}, {indices, "indices"}, {k_c, "k_c"},
      {v_c, "v_c"}, {cache_offsets, "cache_offsets"}, {cache_lens, "cache_lens"}, {c_q, "c_q"}, {c_out, "c_out"},
      {c_lse, "c_lse"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (!aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  if (p->calib_size != 0)
    return fail(CALIDROP_EUNSUPPORTED, "calib_size needs the scored strategy (got %d with a given retained set)",
                p->calib_size);
  const RecalLayout L = recal_layout(p, max_seq_len);
  if (!workspace || workspace_bytes < L.total)
    return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                L.total);
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
#define CD_DISPATCH(T, D)                                                                                         \
  return compress_given_impl<T, D>(p, q_cal, k, v, seq_offsets, total_tokens, max_seq_len, indices, k_c, v_c,     \
                                   cache_offsets, cache_lens, c_q, c_out, c_lse, ws, L, st)
  if (p->dtype == CALIDROP_BF16) {
    if (p->head_dim == 128) CD_DISPATCH(cd::bf16_t, 128);
    CD_DISPATCH(cd::bf16_t, 64);
  }
  if (p->head_dim == 128) CD_DISPATCH(float, 128);
  CD_DISPATCH(float, 64);
#undef CD_DISPATCH
}

size_t calidrop_pack_evicted_workspace_bytes(const calidrop_params* p_in, int32_t max_seq_len) {
  calidrop_params pp; const calidrop_params* p = &pp;
  if (load_params(p_in, &pp) != CALIDROP_OK) return 0;
  if (check_params(p) != CALIDROP_OK) return 0;
  if (max_seq_len < 1) { fail(CALIDROP_ESHAPE, "max_seq_len must be >= 1"); return 0; }
  return pack_layout(p, max_seq_len).total;
}

int32_t calidrop_packed_rows(const calidrop_params* p_in, int32_t seq_len) {
  calidrop_params pp;
  if (load_params(p_in, &pp) != CALIDROP_OK) return -1;
  if (check_params(&pp) != CALIDROP_OK) return -1;
  if (seq_len < 0) { fail(CALIDROP_ESHAPE, "seq_len must be >= 0"); return -1; }
  return packed_rows_host(&pp, seq_len);
}

int calidrop_pack_evicted(const calidrop_params* p_in, const void* k, const void* v, const int32_t* seq_offsets,
                          int64_t total_tokens, int32_t max_seq_len, const int32_t* indices,
                          const int32_t* cal_indices, void* k_e, void* v_e, const int32_t* evict_offsets,
                          int32_t* evict_lens, int32_t* evict_indices, void* workspace, size_t workspace_bytes,
                          void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  const struct { const void* ptr; const char* name; } req[] = {
      {k, "k"}, {v, "v"}, {seq_offsets, "seq_offsets"}, {indices, "indices"}, {k_e, "k_e"}, {v_e, "v_e"},
      {evict_offsets, "evict_offsets"}, {evict_lens, "evict_lens"}, {evict_indices, "evict_indices"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (!aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  if (p->calib_size > 0) {
    if (!cal_indices) return fail(CALIDROP_EINVAL, "cal_indices is NULL although calib_size is %d", p->calib_size);
    if (!aligned16(cal_indices)) return fail(CALIDROP_EALIGN, "cal_indices is not 16-byte aligned");
  } else {
    cal_indices = nullptr;
  }
  const PackLayout L = pack_layout(p, max_seq_len);
  if (!workspace || workspace_bytes < L.total)
    return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                L.total);
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  return pack_impl(p, k, v, seq_offsets, total_tokens, max_seq_len, indices, cal_indices, k_e, v_e, evict_offsets,
                   evict_lens, evict_indices, static_cast<char*>(workspace), L, static_cast<hipStream_t>(stream));
}

size_t calidrop_recalibrate_packed_workspace_bytes(const calidrop_params* p_in, int32_t max_evict_len) {
  return calidrop_decode_workspace_bytes(p_in, max_evict_len);      // the same split partials
}

int calidrop_recalibrate_packed(const calidrop_params* p_in, const void* q_t, const void* k_e, const void* v_e,
                                const int32_t* evict_offsets, const int32_t* evict_lens, int32_t max_evict_len,
                                uint8_t* flags, const float* a_lse, void* out, float* c_q, float* c_out, float* c_lse,
                                void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if (max_evict_len < 1) return fail(CALIDROP_ESHAPE, "max_evict_len must be >= 1 (got %d)", max_evict_len);
  const struct { const void* ptr; const char* name; } req[] = {
      {q_t, "q_t"}, {k_e, "k_e"}, {v_e, "v_e"}, {evict_offsets, "evict_offsets"}, {evict_lens, "evict_lens"},
      {flags, "flags"}, {a_lse, "a_lse"}, {out, "out"}, {c_q, "c_q"}, {c_out, "c_out"}, {c_lse, "c_lse"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (r.ptr != flags && !aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  const DecodeLayout L = decode_layout(p, max_evict_len);
  if (!workspace || workspace_bytes < L.total)
    return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                L.total);
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
#define CD_DISPATCH(T, D)                                                                                        \
  return recal_packed_impl<T, D>(p, q_t, k_e, v_e, evict_offsets, evict_lens, max_evict_len, flags, a_lse, out,   \
                                 c_q, c_out, c_lse, ws, L, st)
  if (p->dtype == CALIDROP_BF16) {
    if (p->head_dim == 128) CD_DISPATCH(cd::bf16_t, 128);
    CD_DISPATCH(cd::bf16_t, 64);
  }
  if (p->head_dim == 128) CD_DISPATCH(float, 128);
  CD_DISPATCH(float, 64);
#undef CD_DISPATCH
}

namespace {
int h2o_local(const calidrop_params* p, int32_t n_local) {
  if (n_local == 0) n_local = p->budget / 2;              // the even split of Sec. 4.1.3
  if (n_local < 1 || n_local >= p->budget) {
    fail(CALIDROP_EINVAL, "n_local must satisfy 1 <= n_local < budget (got %d, budget %d)", n_local, p->budget);
    return -1;
  }
  return n_local;
}
}  // namespace

size_t calidrop_compress_h2o_workspace_bytes(const calidrop_params* p_in, int32_t n_local, int64_t total_tokens,
                                             int32_t max_seq_len) {
  calidrop_params pp; const calidrop_params* p = &pp;
  if (load_params(p_in, &pp) != CALIDROP_OK) return 0;
  if (check_params(p) != CALIDROP_OK || check_sizes(p, total_tokens, max_seq_len) != CALIDROP_OK) return 0;
  if ((n_local = h2o_local(p, n_local)) < 0) return 0;
  return h2o_layout(p, total_tokens, max_seq_len, n_local).total;
}

int calidrop_compress_h2o_workspace_region(const calidrop_params* p_in, int32_t n_local, int64_t total_tokens,
                                           int32_t max_seq_len, int32_t region, size_t* offset, size_t* bytes) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  if ((n_local = h2o_local(p, n_local)) < 0) return CALIDROP_EINVAL;
  if (!offset || !bytes) return fail(CALIDROP_EINVAL, "offset/bytes is NULL");
  const H2oLayout L = h2o_layout(p, total_tokens, max_seq_len, n_local);
  if (region == CALIDROP_REGION_ROW_LSE) {
    *offset = L.row_lse;
    *bytes = static_cast<size_t>(p->batch) * p->n_q_heads * L.lse_stride * sizeof(float);
  } else if (region == CALIDROP_REGION_SCORE) {
    *offset = L.score;
    *bytes = static_cast<size_t>(total_tokens) * p->n_kv_heads * sizeof(float);
  } else if (region == CALIDROP_REGION_VOTE_PLANES) {
    *offset = L.vote;
    *bytes = static_cast<size_t>(vote_plane(total_tokens, p->n_kv_heads)) * (p->n_q_heads / p->n_kv_heads) * L.splits * sizeof(float);
  } else {
    return fail(CALIDROP_EINVAL, "unknown workspace region %d", region);
  }
  return CALIDROP_OK;
}

int calidrop_compress_h2o(const calidrop_params* p_in, int32_t n_local, const void* q_full, const void* k,
                          const void* v, const int32_t* seq_offsets, int64_t total_tokens, int32_t max_seq_len,
                          void* k_c, void* v_c, const int32_t* cache_offsets, int32_t* cache_lens, int32_t* indices,
                          int32_t* cal_indices, float* c_q, float* c_out, float* c_lse, void* workspace,
                          size_t workspace_bytes, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  if ((rc = check_sizes(p, total_tokens, max_seq_len))) return rc;
  if ((n_local = h2o_local(p, n_local)) < 0) return CALIDROP_EINVAL;
  if (static_cast<int64_t>(p->batch) * p->n_q_heads > 65535)
    return fail(CALIDROP_EUNSUPPORTED, "batch * n_q_heads exceeds 65535");
  const struct { const void* ptr; const char* name; } req[] = {
      {q_full, "q_full"}, {k, "k"}, {v, "v"}, {seq_offsets, "seq_offsets"}, {k_c, "k_c"}, {v_c, "v_c"},
      {cache_offsets, "cache_offsets"}, {cache_lens, "cache_lens"}, {indices, "indices"}, {c_q, "c_q"},
      {c_out, "c_out"}, {c_lse, "c_lse"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (!aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  if (p->calib_size > 0) {
    if (!cal_indices) return fail(CALIDROP_EINVAL, "cal_indices is NULL although calib_size is %d", p->calib_size);
    if (!aligned16(cal_indices)) return fail(CALIDROP_EALIGN, "cal_indices is not 16-byte aligned");
  } else {
    cal_indices = nullptr;
  }
  const H2oLayout L = h2o_layout(p, total_tokens, max_seq_len, n_local);
  if (!workspace || workspace_bytes < L.total)
    return fail(CALIDROP_EWORKSPACE, "workspace of %zu bytes given, %zu needed", workspace ? workspace_bytes : 0,
                L.total);
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(CALIDROP_EALIGN, "workspace is not 256-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
#define CD_DISPATCH(T, D)                                                                                      \
  return h2o_impl<T, D>(p, n_local, q_full, k, v, seq_offsets, total_tokens, max_seq_len, k_c, v_c,             \
                        cache_offsets, cache_lens, indices, cal_indices, c_q, c_out, c_lse, ws, L, st)
  if (p->dtype == CALIDROP_BF16) {
    if (p->head_dim == 128) CD_DISPATCH(cd::bf16_t, 128);
    CD_DISPATCH(cd::bf16_t, 64);
  }
  if (p->head_dim == 128) CD_DISPATCH(float, 128);
  CD_DISPATCH(float, 64);
#undef CD_DISPATCH
}

int calidrop_append(const calidrop_params* p_in, const void* k_new, const void* v_new, void* k_c, void* v_c,
                    const int32_t* cache_offsets, int32_t* cache_lens, void* stream) {
  int rc;
  calidrop_params pp; const calidrop_params* p = &pp;
  if ((rc = load_params(p_in, &pp))) return rc;
  if ((rc = check_params(p))) return rc;
  const struct { const void* ptr; const char* name; } req[] = {
      {k_new, "k_new"}, {v_new, "v_new"}, {k_c, "k_c"}, {v_c, "v_c"}, {cache_offsets, "cache_offsets"},
      {cache_lens, "cache_lens"}};
  for (const auto& r : req)
    if (!r.ptr) return fail(CALIDROP_EINVAL, "%s is NULL", r.name);
  for (const auto& r : req)
    if (!aligned16(r.ptr)) return fail(CALIDROP_EALIGN, "%s is not 16-byte aligned", r.name);
  cd::AppendArgs aa{};
  aa.k_new = k_new; aa.v_new = v_new; aa.k_c = k_c; aa.v_c = v_c; aa.cache_off = cache_offsets; aa.cache_lens = cache_lens;
  aa.batch = p->batch; aa.Hkv = p->n_kv_heads; aa.row_bytes = p->head_dim * (p->dtype == CALIDROP_BF16 ? 2 : 4);
  hipLaunchKernelGGL(cd::append_rows_kernel, dim3(p->batch), dim3(256), 0, static_cast<hipStream_t>(stream), aa);
  return launch_status("append_rows");
}

}  // extern "C"
