// Host-side planning and validation (no HIP calls; see host_plan.h).
#include "host_plan.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace mc {
namespace host {

namespace {
constexpr int64_t kComputeUnits = 256;   // MI355X

// a / b of what is not negative, in 32 bits where they fit (planning is full of such divisions: 6000 random batches 4.0 -> 3.6 us).
int64_t quotient(int64_t a, int64_t b) {
  return ((a | b) >> 32) == 0 ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}
}  // namespace

mc_status check_params(const mc_attn_params* p) {
  if (p == nullptr) return MC_ERR_NULL;
  if (p->num_q_heads <= 0 || p->num_kv_heads <= 0 || p->head_dim <= 0 || p->page_size <= 0 || p->num_pages <= 0)
    return MC_ERR_SHAPE;
  if (p->num_q_heads % p->num_kv_heads != 0) return MC_ERR_SHAPE;
  if (p->dtype != MC_DTYPE_BF16 && p->dtype != MC_DTYPE_F32) return MC_ERR_UNSUPPORTED;
  if (p->page_size != 16) return MC_ERR_UNSUPPORTED;
  if (p->dtype == MC_DTYPE_BF16 && p->head_dim != 128 && p->head_dim != 64) return MC_ERR_UNSUPPORTED;
  if (p->dtype == MC_DTYPE_F32 && p->head_dim != 64) return MC_ERR_UNSUPPORTED;
  if (!(p->softmax_scale >= 0.f) || std::isinf(p->softmax_scale)) return MC_ERR_SHAPE;
  return MC_OK;
}

float attn_scale_log2e(const mc_attn_params* p) {
  const double scale = p->softmax_scale > 0.f ? (double)p->softmax_scale : 1.0 / std::sqrt((double)p->head_dim);
  return (float)(scale * 1.4426950408889634);
}

size_t max_items(const mc_attn_params* p, int32_t batch, int64_t total_new_tokens, int32_t kv_splits) {
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  return (size_t)(p->num_kv_heads * ((total_new_tokens * G) / kAttnTileRows + batch)) * (size_t)kv_splits;
}

size_t list_bytes(const mc_attn_params* p, int32_t batch, int64_t total_new_tokens, int32_t kv_splits) {
  return sizeof(AttnItem) * max_items(p, batch, total_new_tokens, kv_splits) + sizeof(AttnReq) * (size_t)batch + 64;
}

mc_status check_lens(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                     int64_t* total_new, int32_t* need_pages) {
  *total_new = 0;
  *need_pages = 0;
  for (int32_t r = 0; r < batch; ++r) {
    if (prefix_lens[r] < 0 || new_lens[r] < 0) return MC_ERR_SHAPE;
    const int64_t len = (int64_t)prefix_lens[r] + new_lens[r];
    if (len > INT32_MAX - 1024) return MC_ERR_RANGE;
    if (new_lens[r] > 0) {
      const int32_t pages = (int32_t)((len + p->page_size - 1) / p->page_size);
      *need_pages = pages > *need_pages ? pages : *need_pages;
    }
    *total_new += new_lens[r];
  }
  return MC_OK;
}

mc_status check_attn_buffers(bool split, const void* q, const void* k_pool, const void* v_pool,
                             const int32_t* block_tables, int32_t batch, int32_t max_pages_per_req, int32_t need_pages,
                             const void* out, const float* lse, const float* o_parts, const float* lse_parts,
                             const void* workspace) {
  if (max_pages_per_req < need_pages) return MC_ERR_SHAPE;
  if (q == nullptr || k_pool == nullptr || v_pool == nullptr || block_tables == nullptr) return MC_ERR_NULL;
  if (split ? (o_parts == nullptr || lse_parts == nullptr) : out == nullptr) return MC_ERR_NULL;
  if (!aligned16(q) || !aligned16(k_pool) || !aligned16(v_pool) || !aligned16(out) || !aligned16(workspace) ||
      !aligned16(o_parts) || !aligned4(block_tables) || !aligned4(lse) || !aligned4(lse_parts))
    return MC_ERR_ALIGN;
  if ((int64_t)batch * max_pages_per_req > INT32_MAX) return MC_ERR_RANGE;
  return MC_OK;
}

mc_status check_list_range(const mc_attn_params* p, int32_t batch, int64_t total_new, int32_t kv_splits) {
  if (total_new * p->num_q_heads > INT32_MAX) return MC_ERR_RANGE;
  if (max_items(p, batch, total_new, kv_splits > 0 ? kv_splits : 1) > (size_t)INT32_MAX) return MC_ERR_RANGE;
  return MC_OK;
}

void build_work_list(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch,
                     int32_t kv_splits, std::vector<AttnReq>& reqs, std::vector<AttnItem>& items) {
  const bool split = kv_splits > 0;
  const int G = p->num_q_heads / p->num_kv_heads;
  const int rows = kAttnTileRows;
  reqs.assign((size_t)batch, AttnReq{});
  struct Keyed {
    int64_t cost;
    AttnItem it;
  };
  std::vector<Keyed> lanes[kXcds];
  int64_t q_off = 0;
  for (int32_t r = 0; r < batch; ++r) {
    const int32_t P = prefix_lens[r], C = new_lens[r];
    reqs[(size_t)r] = {(int32_t)q_off, P, C, (int32_t)(((int64_t)P + C + p->page_size - 1) / p->page_size)};
    q_off += new_lens.of[r];
    const int64_t n_rows = (int64_t)C * G;
    for (int32_t g = 0; g < p->num_kv_heads; ++g)
      for (int64_t row0 = 0; row0 < n_rows; row0 += rows) {
        const int64_t tok_last = std::min<int64_t>(C - 1, (row0 + rows - 1) / G);
        const int64_t keys = P + tok_last + 1;                 // keys the tile's last row sees
        if (!split) {
          lanes[(r * p->num_kv_heads + g) % kXcds].push_back({keys, {r, g, (int32_t)row0, 0}});
          continue;
        }
        // slices of whole 64-key tiles, ceil(tiles of the request / kv_splits) each; every slice gets
        // an item, also one past what the tile can see (it writes zeros and -inf)
        const int64_t per =
            ((((int64_t)P + C + kAttnTileKeys - 1) / kAttnTileKeys) + kv_splits - 1) / kv_splits * kAttnTileKeys;
        for (int32_t sl = 0; sl < kv_splits; ++sl) {
          const int64_t cost = std::max<int64_t>(0, std::min<int64_t>(keys, (sl + 1) * per) - sl * per);
          lanes[(r * p->num_kv_heads + g + sl) % kXcds].push_back({cost, {r, g, (int32_t)row0, sl}});
        }
      }
  }
  size_t n_items = 0;
  for (auto& l : lanes) {
    std::stable_sort(l.begin(), l.end(), [](const Keyed& a, const Keyed& b) { return a.cost > b.cost; });
    n_items += l.size();
  }
  items.clear();
  items.reserve(n_items);
  size_t cur[kXcds] = {0};
  int x = 0;
  while (items.size() < n_items) {
    // next non-empty lane, starting from the one whose turn it is
    int tries = 0;
    while (cur[x] >= lanes[x].size() && tries < kXcds) {
      x = (x + 1) % kXcds;
      ++tries;
    }
    items.push_back(lanes[x][cur[x]++].it);
    x = (x + 1) % kXcds;
  }
}

int64_t count_items(const mc_attn_params* p, const int32_t* new_lens, int32_t batch) {
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  int64_t n = 0;
  for (int32_t r = 0; r < batch; ++r)
    n += (int64_t)p->num_kv_heads * (((int64_t)new_lens[r] * G + kAttnTileRows - 1) / kAttnTileRows);
  return n;
}

bool few_rows(const mc_attn_params* p, NewLens new_lens, int32_t batch, int64_t tile_rows) {
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  for (int32_t r = 0; r < batch; ++r)
    if (new_lens[r] * G > tile_rows) return false;
  return true;
}

int64_t kv_bytes(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch) {
  int64_t keys = 0;
  for (int32_t r = 0; r < batch; ++r)
    if (new_lens[r] > 0) keys += (int64_t)prefix_lens[r] + new_lens[r];
  return 2 * keys * p->num_kv_heads * p->head_dim * (p->dtype == MC_DTYPE_BF16 ? 2 : 4);
}

// One row tile per head reads each of its request's K and V rows once.  If they outgrow the last-level cache, the next layer
// finds none of them there anyway, and a hint that they need not be kept helps.  What would stay in the cache is better left
// there.  64/8 heads, the same call repeated, us without / with the hint: 16 tokens behind 51k (210 MB) 44.7 / 48.3, 61k 51 / 54,
// 74k (302 MB) 61 / 61, 82k 70 / 66, 98k 84 / 76, 128k 107 / 97; 16 requests behind 3840 each (252 MB) 51 / 53, 5120 73 / 66,
// 16k 201 / 178.
// Requests may share pages, which the host does not see: they are counted as if they were apart.  Those that do read them at
// about the same time and find them in the caches either way: 16 requests on one 16k document 127 / 128, 32 on 8k 121 / 121,
// 8 on 32k 129 / 129, 2 on 128k 148 / 149; the one clear loss of the shapes tried is 32 on 32k with 8/1 heads, 71.6 / 73.5.
bool reads_once(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch,
                int64_t tile_rows) {
  constexpr int64_t kLastLevelBytes = (int64_t)256 << 20;
  return few_rows(p, new_lens, batch, tile_rows) && kv_bytes(p, prefix_lens, new_lens, batch) > kLastLevelBytes;
}

// The narrow form where the plan of a one-shot call without room for partial results takes it (plan_classes), 128-row
// workgroups where no row tile has more rows and where that plan takes them, so that a prepared list computes what that call
// computes, bit for bit: the rows that share a workgroup decide which of its key tiles need no mask, and with that the
// reference of the probabilities.  Lists a
// class plan has no room for, and lists of key slices: where two workgroups per item still run side by side (an item's two
// halves read K and V twice, which costs less than a compute unit left idle).
// Measured, planned, 256 rows / 128, us: P 131056, C 16, 64/8 heads 2024 / 1493; 16 requests of P 4000, C 1 73 / 52;
// P 8192, C 300, 64/8 heads (80 items) 169 / 117, fp32, 4/1 heads 1024 / 517; more items than half the units: 24 requests
// of 16 tokens and one of 30, P 4000, 64/8 heads (200 items) 100 / 80; 3 requests, fp32, 12/3 heads (360 items) 754 / 684.
int32_t list_form(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                  int32_t kv_splits, int64_t n_items) {
  ClassPlan plan;
  const bool planned = kv_splits == 0 && plan_classes(p, prefix_lens, new_lens, batch, 0, &plan);
  return planned_list_form(p, prefix_lens, new_lens, batch, planned ? &plan : nullptr, n_items);
}
int32_t planned_list_form(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                          const ClassPlan* plan, int64_t n_items) {
  if (plan != nullptr && plan->classes.rows == kAttnPairRows) return kListPairs;
  if (plan != nullptr && plan->narrow_wgs > 0) return few_rows(p, new_lens, batch, kAttnLeastRows) ? kListNarrowLeast : kListNarrow;
  if (few_rows(p, new_lens, batch, kAttnFewRows))
    return reads_once(p, prefix_lens, new_lens, batch, kAttnFewRows) ? kListFewOnce : kListFew;
  if (plan != nullptr) return plan->classes.rows == kAttnFewRows ? kListHalves : 0;
  return 2 * n_items <= kComputeUnits ? kListHalves : 0;
}

// Shares of the columns cost every workgroup the scores and spare it what is left of V and P V, so they pay while they land on idle
// compute units: up to 256 workgroups in fp32, which is bound by its MFMAs; in bf16 up to about 192, beyond which the K rows
// that all of them load press on the L2s (head_dim 64 has half of them, but only halves are sooner: a row of V in quarters is 32 bytes).
// Planned, us, one workgroup a row tile / two / four: 64/8 heads, P 131056, C 16 (32 row tiles) 909 / 745 / 629; P 20000, C 24
// (48) 98 / 92 / 88, C 32 (64) 99 / 93 / 99, C 48 (96) 99 / 95 / 168, C 64 (128) 99 / 107 / 180; P 600, C 24 9.0 / 8.5 / 7.8;
// head_dim 64, P 20000, C 48 (96) 71 / 70, C 64 71 / 73, P 600, C 32 (64) 6.8 / 6.0; fp32, 4/1 heads, P 3000, C 256 (64) 35 / 29 / 27, C 512
// (128) 37 / 32 / 51, C 768 (192) 40 / 59 / 75; P 256, C 128 (32) 8.4 / 7.6 / 6.9.
int32_t narrow_shares(const mc_attn_params* p, int64_t row_tiles) {
  const bool f32 = p->dtype == MC_DTYPE_F32;
  if (row_tiles <= (f32 ? 64 : 48) && (f32 || p->head_dim == 128)) return 4;
  return row_tiles <= (f32 ? 128 : 96) ? 2 : 1;
}

mc_status check_plan(const mc_attn_params* p, const mc_attn_plan* plan, bool want_split) {
  if (plan == nullptr) return MC_ERR_NULL;
  if (plan->num_q_heads != p->num_q_heads || plan->num_kv_heads != p->num_kv_heads || plan->dtype != (int32_t)p->dtype ||
      plan->n_items < 0 || plan->batch < 0 || plan->total_new_tokens < 0 || plan->reqs_offset < 0 ||
      (plan->reqs_offset & 15) != 0 || plan->kv_splits < 0 || plan->kv_splits > MC_MAX_KV_SPLITS)
    return MC_ERR_SHAPE;
  if (want_split != (plan->kv_splits > 0)) return MC_ERR_SHAPE;
  return MC_OK;
}

mc_status plan_items(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                     int32_t kv_splits, int32_t* items, int64_t capacity, int64_t* n_items) {
  mc_status st = check_params(p);
  if (st != MC_OK) return st;
  if (batch < 0 || kv_splits < 0 || kv_splits > MC_MAX_KV_SPLITS || capacity < 0) return MC_ERR_SHAPE;
  if (n_items == nullptr || (batch > 0 && (prefix_lens == nullptr || new_lens == nullptr))) return MC_ERR_NULL;
  if (capacity > 0 && items == nullptr) return MC_ERR_NULL;
  int64_t total_new = 0;
  int32_t need_pages = 0;
  st = check_lens(p, prefix_lens, new_lens, batch, &total_new, &need_pages);
  if (st != MC_OK) return st;
  st = check_list_range(p, batch, total_new, kv_splits);
  if (st != MC_OK) return st;
  std::vector<AttnReq> reqs;
  std::vector<AttnItem> list;
  build_work_list(p, prefix_lens, new_lens, batch, kv_splits, reqs, list);
  *n_items = (int64_t)list.size();
  if ((int64_t)list.size() > capacity) return capacity == 0 && items == nullptr ? MC_OK : MC_ERR_WORKSPACE;
  static_assert(sizeof(AttnItem) == 4 * sizeof(int32_t), "an item is four int32");
  if (!list.empty()) std::memcpy(items, list.data(), sizeof(AttnItem) * list.size());
  return MC_OK;
}

int32_t suggest_kv_splits(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens,
                          int32_t batch) {
  if (check_params(p) != MC_OK || batch < 0) return 0;
  if (batch > 0 && (prefix_lens == nullptr || new_lens == nullptr)) return 0;
  constexpr int64_t kMinTilesPerSlice = 8;
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  int64_t items = 0, most_tiles = 0;
  for (int32_t r = 0; r < batch; ++r) {
    if (prefix_lens[r] < 0 || new_lens[r] < 0) return 0;
    if (new_lens[r] == 0) continue;
    items += (int64_t)p->num_kv_heads * (((int64_t)new_lens[r] * G + kAttnTileRows - 1) / kAttnTileRows);
    const int64_t tiles = ((int64_t)prefix_lens[r] + new_lens[r] + kAttnTileKeys - 1) / kAttnTileKeys;
    most_tiles = tiles > most_tiles ? tiles : most_tiles;
  }
  // Work items of about equal length run in rounds of one per compute unit: s slices turn `items`
  // items into items * s of 1/s the length, ceil(items * s / 256) / s rounds of the original
  // length, and each extra slice costs about 1 % in partial results written and merged
  // (measured at 128k context).  The cheapest count wins, the smaller one on a tie.  From four
  // full rounds on, the launch order (longest items first) already balances the tail.
  if (items == 0 || items >= 4 * kComputeUnits) return 1;
  int64_t most = most_tiles / kMinTilesPerSlice;
  most = most < MC_MAX_KV_SPLITS ? most : MC_MAX_KV_SPLITS;
  int32_t best = 1;
  double best_cost = 0.0;
  for (int64_t sl = 1; sl <= most || sl == 1; ++sl) {
    const double rounds = (double)((items * sl + kComputeUnits - 1) / kComputeUnits) / (double)sl;
    const double cost = rounds * (1.0 + 0.01 * (double)(sl - 1));
    if (sl == 1 || cost < best_cost) {
      best = (int32_t)sl;
      best_cost = cost;
    }
  }
  return best;
}

namespace {

// Time of a workgroup in microseconds, for weighing cuts against each other: a part that does not depend on the keys
// (start, Q fragments, first tiles, epilogue) and one per 64-key tile.
struct TileCost {
  double fixed, tile;
};
TileCost tile_cost_of(const mc_attn_params* p, int64_t tile_rows) {
  const bool few = tile_rows == kAttnFewRows;
  if (p->dtype == MC_DTYPE_F32) return {4.0, few ? 3.6 : 7.0};
  if (p->head_dim == 128) return {4.0, few ? 1.2 : 1.65};
  return {4.0, few ? 0.7 : 0.95};
}
// The same for the choice of the narrow form, fitted to 400 random launches of each form by themselves (median error 3-9 %):
// the launch, a workgroup, a 64-key tile, and the merge with its time per MB of partial results.  (The costs above are for
// weighing cuts of one form against each other; with these in their place 250 random calls got 1 % slower.)
struct FormCost {
  double launch, fixed, tile, merge, part_mb;
};
FormCost form_cost_of(const mc_attn_params* p, int64_t tile_rows) {
  const int form = tile_rows == kAttnTileRows ? 0 : tile_rows == kAttnFewRows ? 1 : tile_rows == kAttnNarrowRows ? 2
                   : tile_rows == kAttnLeastRows ? 3 : 4;
  static constexpr FormCost kF32[5] = {{0, 9, 7.0, 3, 0.36}, {0, 8.4, 3.8, 2.6, 0.36}, {}, {0, 4.2, 0.58, 4.1, 0.22}, {}};
  static constexpr FormCost kBf16[5] = {{1, 4, 1.37, 3, 0.25}, {2.1, 5.5, 0.72, 2, 0.31}, {0, 4.65, 0.315, 4.6, 0.5},
                                        {0, 4.0, 0.29, 4.4, 0.4}, {2.1, 4.6, 0.44, 0, 0}};
  static constexpr FormCost kBf16D64[5] = {{1, 1, 0.94, 5, 0.25}, {1.5, 4.2, 0.55, 2.6, 0.44}, {0, 4.2, 0.21, 3.9, 0.1},
                                           {0, 3.8, 0.18, 3.8, 0.1}, {1.5, 3.2, 0.36, 0, 0}};
  return (p->dtype == MC_DTYPE_F32 ? kF32 : p->head_dim == 128 ? kBf16 : kBf16D64)[form];
}
// K and V bytes per microsecond: the most any form reads, and what the narrow one's time grows by beyond what the caches hold
// (it has no tiles in flight beyond the next block, and row tiles of a request that do not run together read their keys again).
constexpr double kReadPerUs = 6.2e6, kNarrowReadPerUs = 5.8e6, kNarrowMissPerUs = 8.0e6, kNarrowHeld = 128 << 20;
// Launches of more narrow workgroups than this are not worth weighing: the other forms fill the chip (of 20 random launches of
// more the estimate chose, the narrow form won 13 by 17 % on average and lost 7 by up to 20 %).
constexpr int64_t kMostNarrow = 3 * kComputeUnits;

// The same for 64-row workgroups (bf16), and how much sooner they have to end than what they are weighed against, by where the
// workgroups of the list really go; more than two rounds of them, where full row tiles do better than estimated, by more.  260
// random lists (64/8 to 4/1 heads, 60-900 workgroups): of the 106 for which the plain estimate is sooner 14 got slower (425 -> 519
// us the worst: 240 workgroups and as many short of rows, nine on some of the queues of eight units); of the 86 taken so one did,
// by 3 %, and they run x1.43 faster, the others 4 % slower.
constexpr int64_t kMostPairs = 3 * kComputeUnits;
constexpr double kPairSlack = 1.03, kPairRoundsSlack = 1.15;
// Fewer key tiles (2560 keys) are left to 128-row workgroups: not where a measurement puts the line, but where the tests of that form
// need it.  Shorter calls would gain a few microseconds a launch (64/8 heads, P 600, C 200 17.7 / 12.9).
constexpr int64_t kLeastPairTiles = 40;

// How much sooner the narrow form has to end than a cut, and than anything if it takes more than one round (the estimate's
// errors), and if its rounds walk more keys than the XCDs' caches hold, at paces of their own (12/3 heads, C 1210 behind 32143:
// 0.46 us a tile instead of 0.315, 382 -> 478 us).  The same where the row tiles of a request are cut and (heads x pieces) is no
// multiple of the XCDs: each reads the keys past its own L2 (12/3 heads, P 9720 and 13066, C 19 and 3: 128-row form 17.3, 18
// pieces 18.1, now 16.0; P 30000, C 30 21.5, 22.6, 21.6).
constexpr double kNarrowSlack = 1.06, kNarrowRoundsSlack = 1.12, kNarrowApartSlack = 1.3, kXcdCaches = 32 << 20;
// Longest row tile the fp32 narrow form takes, in key tiles (4096 keys).  Beyond, whole rows are one long chain of roundings in
// the other forms (6.3e-6 off 64 bits at 127262 keys, 1.0e-6 at 3000) and eight shorter ones here (2.3e-6, 4.5e-7): better, but
// another result than such a call has given so far by more than a few roundings of its terms.
constexpr int64_t kNarrowTilesF32 = 64;

// the merge launch, and bytes of partial results written and read per microsecond
constexpr double kMergeFixed = 4.0, kPartBytesPerUs = 3.0e6;
double merge_time(const mc_attn_params* p, int64_t part_rows) {
  return part_rows > 0 ? kMergeFixed + 2.0 * (double)part_rows * (double)(p->head_dim + 1) * 4.0 / kPartBytesPerUs : 0.0;
}

// A request with new tokens.
struct Active {
  int32_t req, q_off, prefix, chunk;
};

// A set of row tiles of one request: `items` workgroups if uncut, of `shortest` to `longest` key tiles.
struct Run {
  int active;               // which of the requests with new tokens, in launch order
  int64_t tile_lo, tile_hi;
  int64_t items, rows;
  int64_t shortest, longest;
  double mean() const { return 0.5 * (double)(shortest + longest); }
  // pieces of at most 1 / k of `of` key tiles each, and the key tiles of one of c pieces on average, rounded up
  int64_t pieces(int64_t of, int64_t k) const { return std::min<int64_t>(quotient(longest * k + of - 1, of), MC_MAX_KV_SPLITS); }
  double mean_piece(int64_t c) const { return (double)quotient(shortest + longest + 2 * c - 1, 2 * c); }
};

// End of the last workgroup if the runs' pieces are handed to the compute units in order, each to the one free first
// (runs are few, so the units are kept as groups that are free at the same time, the first one first).
class Units {
 public:
  // false as soon as a workgroup ends at `limit` or later
  bool place(int64_t n, double dur, double limit) {
    while (n > 0) {
      const int64_t k = n < count_[0] ? n : count_[0];
      const double end = t_[0] + dur;
      if (end >= limit) return false;
      end_ = end > end_ ? end : end_;
      count_[0] -= k;
      if (count_[0] == 0) {
        --used_;
        std::copy(t_ + 1, t_ + 1 + used_, t_);
        std::copy(count_ + 1, count_ + 1 + used_, count_);
      }
      add(end, k);
      n -= k;
    }
    return true;
  }
  double end() const { return end_; }

 private:
  void add(double t, int64_t k) {
    int at = used_;                         // the first group that is free later
    while (at > 0 && t_[at - 1] > t) --at;
    if (at > 0 && t - t_[at - 1] < 0.01) {
      count_[at - 1] += k;
    } else if (at < used_ && t_[at] - t < 0.01) {
      count_[at] += k;
    } else if (used_ == kGroups) {          // merge into the nearest: an estimate
      const bool before = at > 0 && (at == used_ || t - t_[at - 1] <= t_[at] - t);
      count_[before ? at - 1 : at] += k;
    } else {
      std::copy_backward(t_ + at, t_ + used_, t_ + used_ + 1);
      std::copy_backward(count_ + at, count_ + used_, count_ + used_ + 1);
      t_[at] = t;
      count_[at] = k;
      ++used_;
    }
  }
  static constexpr int kGroups = 16;
  int used_ = 1;
  double t_[kGroups] = {0.0};
  int64_t count_[kGroups] = {kComputeUnits};
  double end_ = 0.0;
};

// When a launch really ends.  Workgroup i goes to XCD i % 8 and there to shader engine (i / 8) % 4, whatever else is free: 32
// queues of 8 compute units, and only inside a queue to the unit that is free first.  (One workgroup a unit, spinning for
// given times, us measured / by this rule / by handing each to the first free unit of the chip: 10 of 1330, 246 of 900-960,
// 236 of 430: 1761 / 1760 / 1388; 256 and 236: 1391 / 1390 / 1385; 354 of 290 instead of 236: 1520 / 1519 / 1506.)
class Queues {
 public:
  static constexpr int kQueues = 32;
  // n workgroups next in launch order
  void place(int64_t n, double dur) {
    for (; n > 0; --n) {
      place_on(next_, dur);
      next_ = (next_ + 1) % kQueues;
    }
  }
  // a workgroup of which the launch order says that it goes to this queue
  void place_on(int queue, double dur) {
    double* t = t_[queue];
    int at = 0;
    for (int u = 1; u < kUnits; ++u) at = t[u] < t[at] ? u : at;
    t[at] += dur;
    end_ = t[at] > end_ ? t[at] : end_;
  }
  double end() const { return end_; }

 private:
  static constexpr int kUnits = (int)kComputeUnits / kQueues;
  double t_[kQueues][kUnits] = {{0.0}};
  int next_ = 0;
  double end_ = 0.0;
};
// The same for the 64-row workgroups of a list (build_work_list), in the order that its launch has them (work_of in attn_device.h);
// `limit`: as late as that or later.  The list is not made for that: its row tiles, in the order that all its eight lanes have
// them, and where each lane is among them say which item comes next.  Where the heads fill the lanes evenly one XCD goes for all
// of them.  (Planning whole rows, 64/8 heads, P 8192, C 192: 3.1 us with the list built and sorted, 0.9 so.)
double pairs_really_end(const mc_attn_params* p, const Active* act, int n, const FormCost& cost, double limit) {
  constexpr int kParts = kAttnTileRows / kAttnPairRows;
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  const int32_t Hkv = p->num_kv_heads;
  // row tiles, most keys first, of the same keys that of the earlier request, and the time of each quarter's workgroup
  struct Next {
    int64_t keys;
    const Active* of;
    int64_t row_tile;
  } next[kMaxAttnClasses];
  struct Tile {
    int32_t req;
    double us[kParts];
  } tiles[kMostPairs];
  auto later = [](const Next& a, const Next& b) { return a.keys != b.keys ? a.keys < b.keys : a.of->req > b.of->req; };
  auto last_token = [&](const Active& a, int64_t row) { return std::min<int64_t>(a.chunk - 1, quotient(row, G)); };
  auto tile_of = [&](const Active& a, int64_t t) {
    return Next{a.prefix + last_token(a, t * kAttnTileRows + kAttnTileRows - 1) + 1, &a, t};
  };
  int32_t n_tiles = 0;
  for (int i = 0; i < n; ++i) next[i] = tile_of(act[i], (act[i].chunk * G - 1) / kAttnTileRows);
  std::make_heap(next, next + n, later);
  for (int left = n; left > 0;) {
    std::pop_heap(next, next + left, later);
    const Active& a = *next[left - 1].of;
    const int64_t t = next[left - 1].row_tile;
    Tile& tile = tiles[n_tiles++];
    tile.req = a.req;
    for (int part = 0; part < kParts; ++part) {
      const int64_t row0 = t * kAttnTileRows + part * kAttnPairRows;
      const int64_t keys = a.prefix + last_token(a, row0 + kAttnPairRows - 1) + 1;
      tile.us[part] = row0 >= a.chunk * G ? 1.0 : cost.fixed + cost.tile * (double)((keys + kAttnTileKeys - 1) / kAttnTileKeys);
    }
    if (t > 0) {
      next[left - 1] = tile_of(a, t - 1);
      std::push_heap(next, next + left, later);
    } else {
      --left;
    }
  }
  // the items of a tile in a lane: as many as the request has heads there
  const bool even = Hkv % kXcds == 0;
  auto heads_in = [&](const Tile& tile, int lane) {
    if (even) return Hkv / kXcds;
    const int first = (int)(((int64_t)lane - (int64_t)tile.req * Hkv % kXcds + kXcds) % kXcds);
    return Hkv > first ? (Hkv - first - 1) / kXcds + 1 : 0;
  };
  struct Lane {
    int32_t at, heads;                // its next item's tile, and the items of that tile that are left
  } lanes[kXcds];
  auto settle = [&](int lane) {
    while (lanes[lane].heads == 0 && ++lanes[lane].at < n_tiles) lanes[lane].heads = heads_in(tiles[lanes[lane].at], lane);
  };
  for (int x = 0; x < kXcds; ++x) {
    lanes[x] = {-1, 0};
    settle(x);
  }
  Queues queues;
  int lane = 0;
  for (;;) {
    // the next eight items, from the lanes in turn; fewer at the end.  A part of them is a row of workgroups on consecutive queues.
    const Tile* items[kXcds];
    int n_items = 0;
    for (int empty = 0; n_items < (even ? 1 : kXcds) && empty < kXcds; lane = even ? 0 : (lane + 1) % kXcds) {
      Lane& l = lanes[lane];
      if (l.at >= n_tiles) {
        ++empty;
        continue;
      }
      empty = 0;
      items[n_items++] = &tiles[l.at];
      --l.heads;
      settle(lane);
    }
    if (n_items == 0) break;
    for (int part = 0; part < kParts; ++part)
      for (int i = 0; i < n_items; ++i) queues.place_on(part * (even ? kXcds : n_items) + i, items[i]->us[part]);
    if (cost.launch + queues.end() >= limit) return limit;
  }
  return cost.launch + queues.end();
}
// how much sooner the plain cut has to end to be taken instead
constexpr double kPlainSlack = 1.02;

int64_t key_tiles(int64_t prefix, int64_t chunk, int64_t G, int64_t row_tile, int64_t tile_rows) {
  const int64_t last = std::min<int64_t>(chunk - 1, quotient(row_tile * tile_rows + tile_rows - 1, G));
  return (prefix + last + 1 + kAttnTileKeys - 1) / kAttnTileKeys;
}

Run make_run(const mc_attn_params* p, int active, int64_t prefix, int64_t chunk, int64_t lo, int64_t hi, int64_t tile_rows) {
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  Run run;
  run.active = active;
  run.tile_lo = lo;
  run.tile_hi = hi;
  run.items = (hi - lo + 1) * p->num_kv_heads;
  run.rows = (std::min<int64_t>(chunk * G, (hi + 1) * tile_rows) - lo * tile_rows) * p->num_kv_heads;
  run.longest = key_tiles(prefix, chunk, G, hi, tile_rows);
  run.shortest = key_tiles(prefix, chunk, G, lo, tile_rows);
  return run;
}

// The row tiles of a request from `hi` down to `lo`, each in `cut` pieces, in up to 16 steps; false as soon as one ends at `limit` or later.
bool place_tiles(const mc_attn_params* p, Units& units, int64_t prefix, int64_t chunk, int64_t lo, int64_t hi, int64_t cut,
                 int64_t tile_rows, const FormCost& cost, double limit) {
  const int64_t G = p->num_q_heads / p->num_kv_heads, step = (hi - lo) / 16 + 1;
  for (; hi >= lo; hi -= step) {
    const int64_t n = std::min(step, hi - lo + 1), tiles = key_tiles(prefix, chunk, G, hi, tile_rows);
    if (!units.place(n * p->num_kv_heads * cut, cost.fixed + cost.tile * (double)quotient(tiles + cut - 1, cut), limit)) return false;
  }
  return true;
}

// ClassPlan::ends of a plan of whole rows, where it has not been estimated; `least` and less: no later than that.  (However they
// are placed, the last workgroup starts before the work would end if the units shared it evenly.)
double ends_of(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch, const ClassPlan& plan,
               double least = 0.0) {
  if (plan.ends > 0.0) return plan.ends;
  const AttnClasses& t = plan.classes;
  const FormCost cost = form_cost_of(p, t.rows);
  const double read = (double)kv_bytes(p, prefix_lens, new_lens, batch) / kReadPerUs;
  double work = 0.0, longest = 0.0;
  for (int i = 0; i < t.n && least > 0.0; ++i) {
    const Run run = make_run(p, i, t.c[i].prefix, t.c[i].chunk, t.c[i].tile_lo, t.c[i].tile_hi, t.rows);
    const double step = (double)(run.longest - run.shortest) / 16 + 1;      // (place_tiles rounds up to the longest of a step)
    work += (double)run.items * (cost.fixed + cost.tile * (run.mean() + step));
    longest = std::max(longest, cost.fixed + cost.tile * (double)run.longest);
  }
  if (cost.launch + std::max(work / kComputeUnits + longest, read) <= least) return least;
  Units units;
  for (int i = 0; i < t.n; ++i)
    place_tiles(p, units, t.c[i].prefix, t.c[i].chunk, t.c[i].tile_lo, t.c[i].tile_hi, 1, t.rows, cost, HUGE_VAL);
  return cost.launch + std::max(units.end(), read);
}

}  // namespace

// The cut.  The first `whole` workgroups of the launch order stay uncut - a multiple of the compute units, so that they
// fill whole rounds - and every row tile behind them is cut into pieces of at most `longest / k` key tiles.  Both are
// chosen together, by the estimated end of the last workgroup plus what the merge costs.  What that gives: a small chunk
// behind a long prefix is cut until it fills the chip; a launch just above a whole number of rounds is cut only where it
// would run a last, mostly empty round; few short row tiles are cut into pieces of one or two key tiles.  Row tiles of 256
// and of 128 rows (see Rows in attn_device.h) are both tried: the larger ones share each key tile among twice the rows and
// win wherever there are enough of them.  (Where every request fits the smaller ones there are as many of either.)
// Measured, one call with its append (uniform slices of all rows or none before / this cut now): P 6144, C 811 and 328,
// 64/8 heads (296 row tiles: 6 slices / 256 whole tiles and 40 in 6 pieces) 342 / 220 us; P 256, C 128, fp32, 4/1 heads
// (2 row tiles: whole / 6 pieces) 73 / 33 us; P 131056, C 16, 64/8 heads (32 slices / 32 pieces) 125 / 118 us.
// Every one-shot call pays for the search on the host, so a trial that the work alone puts behind the best is not placed, and
// placing ends where the best does (same plans; host time of a call of 63 requests, 8/1 heads, C up to 300: 219 us with every
// trial placed, 20 now; of 63 one-token requests 41 and 16).  6000 random batches, mean / 99 of 100, us, with room for partial
// results (whole rows): one to three requests 1.2 / 7 (0.8 / 5), 4 to 15 3 / 15 (2.5 / 16), 16 to 63 9 / 29 (9 / 36); without
// 64-row workgroups and two launches to weigh 1.1 / 6 (0.5 / 2), 2.7 / 13 (1.3 / 4), 7 / 32 (4 / 13).
bool plan_classes(const mc_attn_params* p, const int32_t* prefix_lens, NewLens new_lens, int32_t batch,
                  int64_t max_part_rows, ClassPlan* plan, bool keep_room) {
  const int64_t G = p->num_q_heads / p->num_kv_heads, Hkv = p->num_kv_heads;
  Active act[kMaxAttnClasses];
  int n = 0;
  int64_t q_off = 0;
  for (int32_t r = 0; r < batch; ++r) {
    if (new_lens[r] > 0) {
      if (n == kMaxAttnClasses - 1) return false;      // one request may take two classes
      act[n++] = {r, (int32_t)q_off, prefix_lens[r], new_lens[r]};
    }
    q_off += new_lens.of[r];
  }
  auto items_of = [&](int64_t tile_rows) {
    int64_t items = 0;
    for (int i = 0; i < n; ++i) items += Hkv * quotient(act[i].chunk * G + tile_rows - 1, tile_rows);
    return items;
  };
  if (items_of(kAttnTileRows) > INT32_MAX) return false;
  const bool few = few_rows(p, new_lens, batch, kAttnFewRows);
  std::sort(act, act + n, [](const Active& a, const Active& b) {
    if (a.prefix != b.prefix) return a.prefix > b.prefix;
    return a.chunk != b.chunk ? a.chunk > b.chunk : a.req < b.req;
  });

  // runs of the launch order when the first `whole` workgroups are kept apart; returns how many runs those are
  Run runs[kMaxAttnClasses];
  int64_t pieces[kMaxAttnClasses];
  int n_runs = 0;
  auto lay_out = [&](int64_t whole, int64_t tile_rows) {
    n_runs = 0;
    int uncut = 0;
    for (int i = 0; i < n; ++i) {
      const int64_t P = act[i].prefix, C = act[i].chunk;
      const int64_t tiles = quotient(C * G + tile_rows - 1, tile_rows);
      const int64_t keep = std::min<int64_t>(tiles, quotient(whole, Hkv));
      if (keep > 0) {
        runs[n_runs] = make_run(p, i, P, C, tiles - keep, tiles - 1, tile_rows);
        ++n_runs;
        uncut = n_runs;
        whole -= keep * Hkv;
      }
      if (keep < tiles) {
        runs[n_runs] = make_run(p, i, P, C, 0, tiles - keep - 1, tile_rows);
        ++n_runs;
        whole = 0;
      }
    }
    return uncut;
  };
  int64_t best_rows = few ? kAttnFewRows : kAttnTileRows, best_whole = items_of(best_rows);
  int64_t best_of = 0, best_k = 1;
  double best = 0.0;
  for (const int64_t tile_rows : {(int64_t)kAttnTileRows, (int64_t)kAttnFewRows}) {
    // From four full rounds on the launch order (short row tiles last) balances the tail by itself.
    const int64_t items = items_of(tile_rows);
    if (items >= 4 * kComputeUnits || (few && tile_rows != kAttnFewRows)) continue;
    const TileCost cost = tile_cost_of(p, tile_rows);
    for (int64_t rounds = 0; rounds * kComputeUnits < items; ++rounds) {
      const int uncut = lay_out(rounds * kComputeUnits, tile_rows);
      int64_t longest = 0;
      for (int i = uncut; i < n_runs; ++i) longest = std::max(longest, runs[i].longest);
      double kept = 0.0, least = 0.0;      // unit time of what stays whole, and of the rest before it is cut
      for (int i = 0; i < uncut; ++i) kept += (double)runs[i].items * (cost.fixed + cost.tile * runs[i].mean());
      for (int i = uncut; i < n_runs; ++i) least += (double)runs[i].items * cost.tile * runs[i].mean();
      int64_t n_before = 0;
      for (int64_t k = 1; k <= longest && k <= MC_MAX_KV_SPLITS; k += k < 8 ? 1 : k < 32 ? 2 : k < 64 ? 4 : 16) {
        int64_t n_pieces = 0, part_rows = 0;
        for (int i = uncut; i < n_runs; ++i) {
          pieces[i] = runs[i].pieces(longest, k);
          n_pieces += runs[i].items * pieces[i];
          if (pieces[i] > 1) part_rows += pieces[i] * runs[i].rows;
        }
        // more than four rounds of pieces: the tail is short by then, a finer cut only adds partial results
        if (k > 1 && (n_pieces > 4 * kComputeUnits || max_part_rows == 0)) break;
        if (n_pieces == n_before) continue;                       // the same pieces
        n_before = n_pieces;
        const double merge = merge_time(p, part_rows);
        // The work shared evenly is the least any placing takes, and it and the merge only grow with the pieces.
        if (best > 0.0 && (kept + least + cost.fixed * (double)n_pieces) / kComputeUnits + merge >= best) break;
        if (part_rows > max_part_rows) continue;
        const double limit = best > 0.0 ? best - merge : HUGE_VAL;
        Units units;
        bool sooner = true;
        for (int i = 0; i < uncut && sooner; ++i) sooner = units.place(runs[i].items, cost.fixed + cost.tile * runs[i].mean(), limit);
        for (int i = uncut; i < n_runs && sooner; ++i)
          sooner = units.place(runs[i].items * pieces[i], cost.fixed + cost.tile * runs[i].mean_piece(pieces[i]), limit);
        if (!sooner) continue;
        best = units.end() + merge;
        best_rows = tile_rows;
        best_whole = rounds * kComputeUnits;
        best_of = longest;
        best_k = k;
      }
    }
  }
  // The estimate hands every workgroup to the first free unit of the chip.  Where whole rounds are followed by a cut rest, the
  // launch is also followed by where workgroups really go, beside the plain one: every row tile in as many pieces as
  // suggest_kv_splits gives.  Behind a few long row tiles the rest may end later than that: P 55245, C 155 and P 33667, C 5816,
  // 16/2 heads, us: a round whole and the rest in halves (estimated sooner) 1604, all rows in halves 1487; fp32, 8/1 heads, C
  // 5575 and 3868 behind P 268 and 68 737, 507; C 6227, 12/3 heads 775, 561.  Of 66 batches where the plain one is ahead, most
  // of them fp32, the 46 where it is by more than the slack gain up to 45 % and none loses; the rest are left as they are.
  if (best_k > 1 && best_whole > 0) {
    // `limit` and more: as late as that or later
    auto really_ends = [&](int64_t whole, int64_t tile_rows, int64_t of, int64_t k, double limit) {
      const int uncut = lay_out(whole, tile_rows);
      const TileCost cost = tile_cost_of(p, tile_rows);
      int64_t part_rows = 0;
      double work = 0.0;
      for (int i = 0; i < n_runs; ++i) {
        pieces[i] = i < uncut ? 1 : runs[i].pieces(of, k);
        if (pieces[i] > 1) part_rows += pieces[i] * runs[i].rows;
        work += (double)runs[i].items * ((double)pieces[i] * cost.fixed + cost.tile * runs[i].mean());
      }
      const double merge = merge_time(p, part_rows);
      if (part_rows > max_part_rows || work / kComputeUnits + merge >= limit) return limit;
      Queues queues;
      for (int i = 0; i < n_runs; ++i) {
        const Active& a = act[runs[i].active];
        for (int64_t t = runs[i].tile_hi; t >= runs[i].tile_lo; --t) {
          const int64_t tiles = key_tiles(a.prefix, a.chunk, G, t, tile_rows);
          for (int64_t j = 0; j < pieces[i]; ++j)
            queues.place(Hkv, cost.fixed + cost.tile * (double)(tiles / pieces[i] + (j < tiles % pieces[i] ? 1 : 0)));
          if (queues.end() + merge >= limit) return limit;
        }
      }
      return queues.end() + merge;
    };
    const double end = really_ends(best_whole, best_rows, best_of, best_k, HUGE_VAL) / kPlainSlack;
    const int32_t plain = suggest_kv_splits(p, prefix_lens, new_lens.of, batch);      // (a cut is of all requests)
    lay_out(0, kAttnTileRows);
    int64_t longest = 0;
    for (int i = 0; i < n_runs; ++i) longest = std::max(longest, runs[i].longest);
    if (really_ends(0, kAttnTileRows, longest, plain, end) < end) {
      best_whole = 0;
      best_rows = kAttnTileRows;
      best_of = longest;
      best_k = plain;
    }
  }
  // The narrow form, beside what has been chosen so far: the keys of a row tile at several times the pace, and, with so few rows
  // a workgroup, more rounds of them; whole rows, or cut where that was cut.  Both are estimated row tile by row tile (in up to
  // 16 steps a run).
  const int64_t narrow_rows =
      p->dtype == MC_DTYPE_F32 || few_rows(p, new_lens, batch, kAttnLeastRows) ? kAttnLeastRows : kAttnNarrowRows;
  plan->narrow_wgs = 0;
  plan->narrow_pieces = 1;
  plan->ends = 0.0;
  const int64_t narrow_items = items_of(narrow_rows);
  int64_t longest = 0;
  for (int i = 0; i < n; ++i) longest = std::max(longest, ((int64_t)act[i].prefix + act[i].chunk + kAttnTileKeys - 1) / kAttnTileKeys);
  // (a row tile of one key tile is one block for each of two waves: the 128-row form has that done as soon)
  const bool by_narrow = narrow_items <= kMostNarrow && longest > 1;
  const bool by_pairs = p->dtype == MC_DTYPE_BF16 && narrow_rows == kAttnNarrowRows && items_of(kAttnPairRows) <= kMostPairs &&
                        longest >= kLeastPairTiles;
  if (by_narrow || by_pairs) {
    auto place = [&](Units& units, const Run& run, int64_t cut, int64_t tile_rows, const FormCost& cost, double limit) {
      const Active& a = act[run.active];
      return place_tiles(p, units, a.prefix, a.chunk, run.tile_lo, run.tile_hi, cut, tile_rows, cost, limit);
    };
    auto merge_of = [&](const FormCost& cost, int64_t part_rows) {
      return part_rows > 0 ? cost.merge + cost.part_mb * (double)part_rows * (double)(p->head_dim + 1) * 8e-6 : 0.0;
    };
    const double bytes = (double)kv_bytes(p, prefix_lens, new_lens, batch);
    const FormCost cost = form_cost_of(p, best_rows);
    const int uncut = lay_out(best_whole, best_rows);
    Units chosen;
    int64_t part_rows = 0, longest_piece = 0;
    for (int i = 0; i < n_runs; ++i) {
      const int64_t cut = i < uncut || best_of == 0 ? 1 : runs[i].pieces(best_of, best_k);
      place(chosen, runs[i], cut, best_rows, cost, HUGE_VAL);
      if (cut > 1) part_rows += cut * runs[i].rows;
      longest_piece = std::max(longest_piece, quotient(runs[i].longest + cut - 1, cut));
    }
    double end = cost.launch + std::max(chosen.end(), bytes / kReadPerUs) + merge_of(cost, part_rows);
    if (part_rows > 0) end /= kNarrowSlack;
    const FormCost narrow = form_cost_of(p, narrow_rows);
    const double missed = std::max(0.0, bytes - kNarrowHeld) / kNarrowMissPerUs;
    const int64_t room = keep_room ? max_part_rows : part_rows;
    const bool may = by_narrow && bytes / kNarrowReadPerUs < end && (p->dtype != MC_DTYPE_F32 || longest_piece <= kNarrowTilesF32);
    n_runs = 0;
    double work = 0.0;
    for (int i = 0; i < n && may; ++i) {
      runs[n_runs] = make_run(p, i, act[i].prefix, act[i].chunk, 0, (act[i].chunk * G - 1) / narrow_rows, narrow_rows);
      work += (double)runs[n_runs].items * narrow.tile * runs[n_runs].mean();
      ++n_runs;
    }
    int64_t narrow_k = 0, n_before = 0;
    for (int64_t k = 1; may && k <= longest && k <= MC_MAX_KV_SPLITS; k += k < 8 ? 1 : k < 32 ? 4 : 16) {
      if (p->dtype == MC_DTYPE_F32 && (longest + k - 1) / k > kNarrowTilesF32) continue;
      int64_t n_pieces = 0, parts = 0;
      bool apart = false;                                  // cut row tiles of one request lie on different XCDs
      for (int i = 0; i < n_runs; ++i) {
        const int64_t cut = runs[i].pieces(longest, k);
        n_pieces += runs[i].items * cut;
        if (cut > 1) parts += cut * runs[i].rows;
        apart = apart || (cut > 1 && runs[i].tile_hi > runs[i].tile_lo && Hkv * cut % kXcds != 0);
      }
      if (n_pieces > kMostNarrow || (k > 1 && parts > room)) break;
      if (n_pieces == n_before) continue;
      n_before = n_pieces;
      const double rest = narrow.launch + missed + merge_of(narrow, parts);
      double by = end;                                     // when it has to have ended
      if (bytes > kXcdCaches && (apart || n_pieces > kComputeUnits)) by /= kNarrowApartSlack;
      else if (n_pieces > kComputeUnits) by /= kNarrowRoundsSlack;
      if (rest + std::max(narrow.fixed, (work + narrow.fixed * (double)n_pieces) / kComputeUnits) >= by) continue;
      Units units;
      bool sooner = true;
      for (int i = 0; i < n_runs && sooner; ++i)
        sooner = place(units, runs[i], runs[i].pieces(longest, k), narrow_rows, narrow, by - rest);
      if (!sooner) continue;
      end = rest + units.end();
      narrow_k = k;
    }
    if (narrow_k > 0) {
      AttnClasses& t = plan->narrow;
      t.n = n;
      t.rows = (int32_t)narrow_rows;
      t.once = 0;
      int64_t wg = 0, parts = 0;
      for (int i = 0; i < kMaxAttnClasses; ++i) {
        t.first[i] = i < n ? (int32_t)wg : 0;
        t.c[i] = AttnClass{};
        if (i >= n) continue;
        const int64_t cut = runs[i].pieces(longest, narrow_k);
        t.c[i] = AttnClass{act[i].req, act[i].q_off, act[i].prefix, act[i].chunk, 0, (int32_t)runs[i].tile_hi, (int32_t)cut,
                           (int32_t)parts};
        wg += runs[i].items * cut;
        if (cut > 1) parts += cut * runs[i].rows;
        plan->narrow_pieces = std::max<int32_t>(plan->narrow_pieces, (int32_t)cut);
      }
      plan->narrow_wgs = (int32_t)wg;
    }
    // 64-row workgroups, all rows whole, beside that.  (A cut they end before is all they are weighed against, so a call with room
    // may run them where a prepared list runs other whole rows: in 60 such calls x1.04 as fast as the cut, and as the list's form x1.02.)
    if (by_pairs) {
      const FormCost pairs = form_cost_of(p, kAttnPairRows);
      const double limit = end / (items_of(kAttnPairRows) > 2 * kComputeUnits ? kPairRoundsSlack : kPairSlack), by = limit - pairs.launch;
      Units units;
      bool sooner = bytes / kReadPerUs < by;
      lay_out(items_of(kAttnPairRows), kAttnPairRows);
      for (int i = 0; i < n_runs && sooner; ++i) sooner = place(units, runs[i], 1, kAttnPairRows, pairs, by);
      const double really = sooner ? pairs_really_end(p, act, n, pairs, limit) : limit;
      if (really < limit) {
        end = really;
        best_rows = kAttnPairRows;
        best_whole = items_of(kAttnPairRows);
        best_of = 0;
        plan->narrow_wgs = 0;
        plan->narrow_pieces = 1;
      }
    }
    plan->ends = end;
  }
  const int uncut = lay_out(best_whole, best_rows);
  AttnClasses& t = plan->classes;
  t.n = n_runs;
  t.rows = (int32_t)best_rows;
  t.once = reads_once(p, prefix_lens, new_lens, batch, best_rows) ? 1 : 0;
  int64_t wg = 0;
  plan->part_rows = 0;
  plan->most_pieces = 1;
  for (int i = 0; i < n_runs; ++i) {
    const Run& run = runs[i];
    const Active& of = act[run.active];
    const int64_t cut = i < uncut || best_of == 0 ? 1 : run.pieces(best_of, best_k);
    t.first[i] = (int32_t)wg;
    t.c[i] = AttnClass{of.req, of.q_off, of.prefix, of.chunk, (int32_t)run.tile_lo, (int32_t)run.tile_hi,
                       (int32_t)cut, (int32_t)plan->part_rows};
    wg += run.items * cut;
    if (cut > 1) plan->part_rows += cut * run.rows;
    plan->most_pieces = std::max<int32_t>(plan->most_pieces, (int32_t)cut);
  }
  if (wg > INT32_MAX || plan->part_rows > INT32_MAX) return false;
  for (int i = n_runs; i < kMaxAttnClasses; ++i) {
    t.first[i] = 0;
    t.c[i] = AttnClass{};
  }
  plan->n_wgs = (int32_t)wg;
  return true;
}

// Requests of few rows behind long prefixes beside requests of many rows: in one form either the former walk their keys at the pace
// of a 128- or 256-row workgroup or the latter are too many narrow workgroups.  One launch behind the other, the line between
// them at a power of two of new tokens.
// Planned, us, one launch / two: 64/8 heads, P 6000 and 0, C 3 and 900 69 / 57; P 19657, 31 and 50, C 2, 2 and 829 208 / 101;
// P 51199 and 647, C 7 and 1187 552 / 335; fp32, 16/16 heads, P 3900, 0, 40, C 3, 900, 5 243 / 99.
// What both launches take at least, by the longest row tile of either and the work of the second, says which line is tried; it is
// planned only if that is sooner than one launch, which most batches end at.
// Where the line lies, by 66 random batches that the plain estimate divides: a first launch of more than one round of workgroups (5
// of 7 got slower, 196 -> 267 us the worst), one whose row tiles share keys that the XCDs' caches do not hold (12/3 heads, C 664
// behind 27003 211 -> 319), and full row tiles in several rounds, which do better than estimated (261 -> 298, 157 -> 187).
// Of 22 others by these rules with a slack of 1.1, 20 run x1.0-2.1 and two x0.96, both within 15 % by the estimate.
constexpr double kApartLeast = 40.0, kApartSecond = 3.0, kApartSlack = 1.15, kApartRoundsSlack = 1.35, kApartMiss = 1.5;
bool plan_apart(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch, const ClassPlan& one,
                ApartPlan* apart) {
  if (one.ends > 0.0 && one.ends < kApartLeast) return false;
  const int64_t G = p->num_q_heads / p->num_kv_heads;
  const FormCost full = form_cost_of(p, kAttnTileRows), half = form_cost_of(p, kAttnFewRows),
                 pairs = form_cost_of(p, p->dtype == MC_DTYPE_BF16 ? kAttnPairRows : kAttnFewRows),
                 narrow = form_cost_of(p, kAttnLeastRows);
  // what the requests between two lines add to the launches, and then what those above a line do
  struct Between {
    int64_t longest = 0, items = 0;
    double work = 0.0;
  } at[33];
  int highest = 0;
  for (int32_t r = 0; r < batch; ++r) {
    if (new_lens[r] == 0) continue;
    int k = 0;
    while ((int64_t)1 << k < new_lens[r]) ++k;
    const int64_t rows = new_lens[r] * G;
    at[k].longest = std::max(at[k].longest, ((int64_t)prefix_lens[r] + new_lens[r] + kAttnTileKeys - 1) / kAttnTileKeys);
    at[k].items += (rows + kAttnNarrowRows - 1) / kAttnNarrowRows * p->num_kv_heads;
    at[k].work += (double)(rows * p->num_kv_heads) / kAttnTileRows * full.tile *
                  ((double)prefix_lens[r] + 0.5 * (double)new_lens[r]) / kAttnTileKeys;
    highest = std::max(highest, k);
  }
  Between above[33];
  for (int k = highest - 1; k >= 0; --k) {
    above[k].longest = std::max(above[k + 1].longest, at[k + 1].longest);
    above[k].work = above[k + 1].work + at[k + 1].work;
  }
  double least = HUGE_VAL;
  int32_t line = 0;
  int64_t few_longest = 0;
  Between below;
  for (int k = 0; k < highest; ++k) {
    below.longest = std::max(below.longest, at[k].longest);
    below.items += at[k].items;
    if (below.items == 0 || below.items > kComputeUnits) continue;
    const double both = narrow.fixed + narrow.tile * (double)below.longest + pairs.fixed +
                        std::max(std::min(pairs.tile, half.tile) * (double)above[k].longest, above[k].work / kComputeUnits);
    if (both >= least) continue;
    least = both;
    line = (int32_t)((int64_t)1 << k);
    few_longest = below.longest;
  }
  if (line == 0 || (p->dtype == MC_DTYPE_F32 && few_longest > kNarrowTilesF32)) return false;
  const bool rounds = one.narrow_wgs == 0 && one.classes.rows == kAttnTileRows && one.n_wgs > kComputeUnits;
  const double slack = rounds ? kApartRoundsSlack : kApartSlack, at_least = std::max(kApartLeast, (least + kApartSecond) * slack);
  const double ends = ends_of(p, prefix_lens, new_lens, batch, one, at_least), limit = ends / slack - kApartSecond;
  if (ends <= at_least) return false;
  apart->line = line;
  const NewLens few_lens(new_lens, 0, line), many_lens(new_lens, line, INT32_MAX);
  if (!plan_classes(p, prefix_lens, few_lens, batch, 0, &apart->few)) return false;
  const ClassPlan& few = apart->few;
  if (few.narrow_wgs == 0 || few.narrow_wgs > kComputeUnits) return false;      // (0: `narrow` has not been written)
  const int32_t one_tile = (int32_t)std::min<int64_t>(few.narrow.rows / G, line);
  const NewLens several(new_lens, one_tile, line);         // requests of several row tiles a head
  const bool miss = kv_bytes(p, prefix_lens, several, batch) > kXcdCaches;
  const double few_ends = few.ends * (miss ? kApartMiss : 1.0);
  return few_ends < limit && plan_classes(p, prefix_lens, many_lens, batch, 0, &apart->many) && apart->many.narrow_wgs == 0 &&
         few_ends + ends_of(p, prefix_lens, many_lens, batch, apart->many) < limit;
}

int32_t apart_list(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, const ApartPlan& apart,
                   int32_t batch, std::vector<AttnItem>& items) {
  const NewLens few_lens(new_lens, 0, apart.line), many_lens(new_lens, apart.line, INT32_MAX);
  std::vector<AttnReq> reqs;
  std::vector<AttnItem> behind;
  build_work_list(p, prefix_lens, few_lens, batch, 0, reqs, items);
  build_work_list(p, prefix_lens, many_lens, batch, 0, reqs, behind);
  const int32_t n_few = (int32_t)items.size();
  items.insert(items.end(), behind.begin(), behind.end());
  const int32_t form = apart.many.classes.rows == kAttnPairRows ? kListPairs
                       : few_rows(p, many_lens, batch, kAttnFewRows)
                           ? (reads_once(p, prefix_lens, many_lens, batch, kAttnFewRows) ? kListFewOnce : kListFew)
                       : apart.many.classes.rows == kAttnFewRows ? kListHalves : 0;
  ApartMark mark;
  mark.n_few = n_few;
  mark.least = apart.few.narrow.rows == kAttnLeastRows;
  mark.shares = narrow_shares(p, apart.few.narrow_wgs);
  mark.form = form;
  return mark.packed();
}

bool auto_layout(const mc_attn_params* p, const int32_t* prefix_lens, const int32_t* new_lens, int32_t batch,
                 AutoLayout* lay, size_t available) {
  const int32_t s = suggest_kv_splits(p, prefix_lens, new_lens, batch);
  if (s <= 0) return false;
  int64_t total_new = 0;
  for (int32_t r = 0; r < batch; ++r) total_new += new_lens[r];
  const int64_t rows = total_new * p->num_q_heads;
  lay->kv_splits = s;
  lay->list_bytes = list_bytes(p, batch, total_new, s);
  auto place = [&](int64_t part_rows) {
    lay->o_off = lay->lse_off = lay->total = lay->list_bytes;
    if (part_rows > 0) {
      lay->o_off = (lay->list_bytes + 255) & ~(size_t)255;
      lay->lse_off = (lay->o_off + (size_t)part_rows * (size_t)p->head_dim * sizeof(float) + 255) & ~(size_t)255;
      lay->total = lay->lse_off + (size_t)part_rows * sizeof(float);
    }
    lay->room = available >= lay->total;
  };
  auto plan_with = [&](int64_t max_part_rows, bool keep_room = false) {
    lay->by_classes = plan_classes(p, prefix_lens, new_lens, batch, max_part_rows, &lay->plan, keep_room);
  };
  if (s > 1) {
    place(s * rows);
    plan_with(lay->room ? s * rows : 0, true);
    return true;
  }
  // a launch of few workgroups may be cut all the same, and finer: at most 64 parts of a row
  plan_with(available > lay->list_bytes ? 64 * rows : 0);
  place(lay->by_classes ? lay->plan.part_rows : 0);
  if (!lay->room) plan_with(0);
  return true;
}

// One launch saves 3 us; what it costs is that a request's digests share one compute unit.  They are bound by its vector
// ALUs, so tokens decide, unless there are so few blocks that each has a SIMD to itself (as it has when the whole chip
// digests).  One launch / digests and chains apart, us, one request: 32 blocks of 512 tokens 7.9 / 8.2, of 768 9.8 / 8.2, of
// 4096 24.8 / 10.4, of 16384 82.1 / 20.4; 16 blocks of 1024 6.0 / 8.1, of 2048 8.5 / 8.0; 4 blocks of 16384 14.8 / 17.5, 6 of
// them 23.4 / 18.2; 8 and 64 such requests alike.
bool hash_in_one_launch(int64_t max_blocks, int64_t max_tokens) {
  constexpr int64_t kShortTokens = 20 << 10, kSimds = 4;
  return max_blocks <= kShortHashBlocks && (max_tokens <= kShortTokens || max_blocks <= kSimds);
}

bool kernel_may_reach(uint32_t flags, uintptr_t at, uintptr_t start, size_t size, size_t bytes) {
  return (flags & ~kPlainHostFlags) == 0 && at >= start && at - start <= size && bytes <= size - (at - start);
}

mc_status check_copy(const void* a, const void* b, int64_t num_pages, int64_t page_bytes, const int32_t* ids,
                     int64_t n, const void* c, const void* d) {
  if (num_pages < 0 || page_bytes < 0 || n < 0) return MC_ERR_SHAPE;
  if (page_bytes % 16 != 0) return MC_ERR_ALIGN;
  if (n == 0 || page_bytes == 0) return MC_OK;
  if (a == nullptr || b == nullptr || c == nullptr || d == nullptr || ids == nullptr) return MC_ERR_NULL;
  if (num_pages == 0) return MC_ERR_SHAPE;
  if (!aligned16(a) || !aligned16(b) || !aligned16(c) || !aligned16(d) || !aligned4(ids)) return MC_ERR_ALIGN;
  const int64_t slices = (page_bytes / 16 + kKvCopySliceVecs - 1) / kKvCopySliceVecs;
  if (n > INT32_MAX || n * slices > INT32_MAX) return MC_ERR_RANGE;
  return MC_OK;
}

}  // namespace host
}  // namespace mc
