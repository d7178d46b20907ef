// Host-side planning (see ba_plan.h) and the schedule queries of the C boundary.  No device code
// and no device calls in this file.
#include "ba_plan.h"

#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>

namespace ba {

namespace {
thread_local char g_err[512] = "";
}

int32_t fail(int32_t status, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return status;
}

const char *last_error() { return g_err; }

int32_t check_heads(const ba_heads *h, bool attention) {
  if (!h) return fail(BA_ERR_INVALID_ARG, "heads: null");
  if (h->head_dim != 64 && h->head_dim != 128)
    return fail(BA_ERR_UNSUPPORTED, "head_dim %d: only 64 and 128 are built", h->head_dim);
  if (h->n_kv_heads <= 0) return fail(BA_ERR_INVALID_ARG, "n_kv_heads must be positive");
  if (h->rope_layout != BA_ROPE_INTERLEAVED && h->rope_layout != BA_ROPE_HALF)
    return fail(BA_ERR_INVALID_ARG, "rope_layout %d unknown", h->rope_layout);
  if (!h->inv_freq && !(h->rope_base > 0.0)) return fail(BA_ERR_INVALID_ARG, "rope_base must be positive");
  if (attention) {
    if (h->n_q_heads <= 0 || h->n_q_heads % h->n_kv_heads)
      return fail(BA_ERR_INVALID_ARG, "n_q_heads must be a positive multiple of n_kv_heads");
    const int g = h->n_q_heads / h->n_kv_heads;
    if (h->q_to_kv)
      for (int i = 0; i < h->n_q_heads; ++i)
        if (h->q_to_kv[i] != i / g)
          return fail(BA_ERR_UNSUPPORTED, "q_to_kv: only the map h -> h / group is built");
  }
  return BA_OK;
}

int32_t check_offsets(int32_t n_blocks, const int32_t *offs) {
  if (n_blocks < 0 || !offs) return fail(BA_ERR_INVALID_ARG, "block_offsets: null or negative block count");
  if (offs[0] != 0) return fail(BA_ERR_INVALID_ARG, "block_offsets[0] must be 0");
  for (int b = 0; b < n_blocks; ++b)
    if (offs[b + 1] < offs[b]) return fail(BA_ERR_INVALID_ARG, "block_offsets must not decrease (block %d)", b);
  return BA_OK;
}

int32_t check_prompt_blocks(int32_t n_prompts, const int32_t *cu_blk, const int32_t *block_offsets) {
  if (n_prompts < 0 || !cu_blk) return fail(BA_ERR_INVALID_ARG, "cu_blk: null or negative prompt count");
  if (cu_blk[0] != 0) return fail(BA_ERR_INVALID_ARG, "cu_blk[0] must be 0");
  for (int n = 0; n < n_prompts; ++n)
    if (cu_blk[n + 1] <= cu_blk[n]) return fail(BA_ERR_INVALID_ARG, "prompt %d: at least one block needed", n);
  return check_offsets(cu_blk[n_prompts], block_offsets);
}

// One workgroup runs per compute unit, so a launch takes ceil(workgroups / CUs) rounds, each as long
// as one workgroup: a fixed part (prologue, output, worth about four key tiles) plus its share of the
// key tiles; every split also adds a little to the merge.  Take the cheapest count, never fewer than four
// key tiles per split.
// Few workgroups per split and a long context want many splits, and have few rows to merge (64 KB per workgroup
// and split at D = 128): up to 64 splits, the merge priced by its rows.  32 splits at most / up to 64, us: 50
// queries, 31,950 tokens: 4 over 4 heads of 64: 24.3 / 21.0, 8 over 2 of 64: 28.9 / 23.5, 4 over 1 of 128: 30.5 / 24.9;
// 64,000: 6 over 6 of 64: 35.7 / 31.7, 7 over 7: 36.1 / 34.6, 16 over 4 of 128: 49.2 / 43.8.  At D = 128 five workgroups
// gain only where the merge at its full price leaves a gain (20 over 5, 60 queries: 24,000 tokens 30.1 with 32,
// 30.9 with 51; 64,000: 52.4 / 50.2), six and seven hardly ever (28 over 7, one query: 16,000: 24.9 / 25.6, 64,000:
// 48.1 / 49.1).  From eight on, 32 splits fill the chip: more would only grow the partials, beyond the static
// scratch for contexts of 400,000 tokens and more, and leave the shares by XCD speed (kMaxCutSplits).
int choose_splits(int64_t base_wgs, int max_tiles, int n_cu, int head_dim) {
  if (base_wgs <= 0) return 1;
  if (n_cu < 1) n_cu = 1;
  const int64_t row_bytes = base_wgs * head_dim;  // of a split's partials, in units that compare only
  const int s_max = std::min(base_wgs < 8 && row_bytes <= 5 * 128 ? kMaxSplits : kMaxCutSplits, std::max(1, max_tiles / 4));
  const double merge = row_bytes <= 4 * 128 ? 0.25 * std::min(1.0, (double)base_wgs / 8) : 0.25;
  int best = 1;
  double best_cost = 0;
  for (int s = 1; s <= s_max; ++s) {
    const double rounds = (double)((base_wgs * s + n_cu - 1) / n_cu);
    const double cost = rounds * (4.0 + (max_tiles + s - 1) / s) + merge * s;
    if (s == 1 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

int32_t plan_final(const ba_heads *h, int32_t n_prompts, const int32_t *cu_q, const int32_t *cu_ctx,
                   int32_t rope_mode, bool have_rot_out, int n_cu, FinalPlan *plan) {
  if (n_prompts < 0 || (n_prompts > 0 && (!cu_q || !cu_ctx)))
    return fail(BA_ERR_INVALID_ARG, "cu_q / cu_ctx: null or negative prompt count");
  const int G = h->n_q_heads / h->n_kv_heads;
  FinalPlan pl;
  if (n_prompts > 0 && cu_q[0] != 0) return fail(BA_ERR_INVALID_ARG, "cu_q[0] must be 0");
  if (n_prompts > 0 && cu_ctx[0] < 0) return fail(BA_ERR_INVALID_ARG, "cu_ctx[0] must not be negative");
  for (int n = 0; n < n_prompts; ++n) {
    const int64_t lq = (int64_t)cu_q[n + 1] - cu_q[n];
    const int64_t tc = (int64_t)cu_ctx[n + 1] - cu_ctx[n];
    if (lq < 1) return fail(BA_ERR_INVALID_ARG, "prompt %d: the final block needs at least one token", n);
    if (tc < 0) return fail(BA_ERR_INVALID_ARG, "prompt %d: cu_ctx decreases", n);
    if (lq * G > 0x3fffffff) return fail(BA_ERR_INVALID_ARG, "prompt %d: too many packed rows", n);
    pl.total_tiles += (lq * G + kTileRows - 1) / kTileRows;
    const int nt = (int)((tc + kTileKeys - 1) / kTileKeys + (lq + kTileKeys - 1) / kTileKeys);
    pl.max_nt = std::max(pl.max_nt, nt);
  }
  pl.lq_total = n_prompts > 0 ? cu_q[n_prompts] : 0;
  pl.n_splits = choose_splits(pl.total_tiles * h->n_kv_heads, pl.max_nt, n_cu, h->head_dim);
  if (rope_mode == BA_ROPE_APPLY) {
    if (!have_rot_out) pl.kf_bytes = (size_t)pl.lq_total * h->n_kv_heads * h->head_dim * 2;
    pl.q_bytes = (size_t)pl.lq_total * h->n_q_heads * h->head_dim * 2;  // rotated, pre-scaled queries
  }
  if (pl.n_splits > 1) {
    const size_t rows = partial_rows(pl.total_tiles, h->n_kv_heads);
    pl.part_o_bytes = (size_t)pl.n_splits * rows * h->head_dim * 2;  // fp16
    pl.part_ml_bytes = (size_t)pl.n_splits * rows * 2 * 4;
    pl.part_idx_bytes = rows * 4;
  }
  *plan = pl;
  return BA_OK;
}

namespace {
// Cut lists of one candidate order of the work items, and how long its launch is expected to take,
// in tile periods of a workgroup: an XCD is done when its longest item is, or when its compute
// units have worked through all its items, whichever is later; before that it fetches the query
// rows of the KV heads it hosts (about a megabyte per microsecond and XCD, a tile period being 1.6).
double try_kv_group(const float *speed, int64_t tiles, int n_kv_heads, int n_splits, int kv_group, unsigned runs, int max_nt,
                    int n_cu, double q_bytes_per_kv_head, uint32_t cuts[kMaxCutHeads][33]) {
  const ItemOrder order = {(int)tiles, n_kv_heads, n_splits, kv_group};
  const unsigned n_wg = (unsigned)(tiles * n_kv_heads * n_splits);
  double longest[kNumXcds] = {0}, sum[kNumXcds] = {0};
  bool hosts[kNumXcds][kMaxCutHeads] = {};
  for (int h = 0; h < n_kv_heads; ++h) {
    double w[kMaxCutSplits], total = 0.0;
    for (int s = 0; s < n_splits; ++s) {
      double acc = 0.0;
      for (int64_t t = 0; t < tiles; ++t) acc += speed[xcd_of_work_item(item_id((int)t, h, s, order), n_wg, runs)];
      w[s] = acc / (double)tiles;
      total += w[s];
    }
    double acc = 0.0;
    for (int s = 0; s < n_splits; ++s) {
      cuts[h][s] = (uint32_t)(acc / total * 65536.0 + 0.5);
      acc += w[s];
    }
    for (int s = n_splits; s <= kMaxCutSplits; ++s) cuts[h][s] = 65536;
    for (int s = 0; s < n_splits; ++s) {
      const double item_tiles = (double)max_nt * (double)(cuts[h][s + 1] - cuts[h][s]) / 65536.0;
      for (int64_t t = 0; t < tiles; ++t) {
        const int x = xcd_of_work_item(item_id((int)t, h, s, order), n_wg, runs);
        longest[x] = std::max(longest[x], item_tiles);
        sum[x] += item_tiles;
        hosts[x][h] = true;
      }
    }
  }
  const double cu_per_xcd = std::max(1.0, (double)n_cu / kNumXcds);
  double worst = 0.0;
  for (int x = 0; x < kNumXcds; ++x) {
    int hosted = 0;
    for (int h = 0; h < n_kv_heads; ++h) hosted += hosts[x][h];
    const double fetch = hosted * q_bytes_per_kv_head / 1.0e6 / 1.6;
    worst = std::max(worst, std::max(longest[x], sum[x] / cu_per_xcd) / (double)speed[x] + fetch);
  }
  return worst;
}

// Which run of work items each XCD takes (work_item_of_workgroup) under groups of kv_group KV heads:
// the runs of one group of KV heads are neighbours, and only their XCDs can be balanced against each
// other, so the XCDs are dealt to the groups in order of speed, to and fro (fastest and slowest end
// up together), which brings the groups' mean speeds as close as a greedy deal gets them.  Identity
// when the runs do not line up with the groups.
unsigned deal_xcd_runs(const float *speed, int64_t tiles, int n_kv_heads, int n_splits, int kv_group) {
  const int64_t n_wg = tiles * n_kv_heads * n_splits;
  if (n_wg % kNumXcds || (kNumXcds * kv_group) % n_kv_heads) return kIdentityXcdRuns;
  const int per_group = kNumXcds * kv_group / n_kv_heads;  // runs (= XCDs) that share one group of KV heads
  if (per_group < 2 || per_group >= kNumXcds || kNumXcds % per_group) return kIdentityXcdRuns;
  const int n_groups = kNumXcds / per_group;
  int by_speed[kNumXcds];
  for (int x = 0; x < kNumXcds; ++x) by_speed[x] = x;
  std::stable_sort(by_speed, by_speed + kNumXcds, [&](int a, int b) { return speed[a] > speed[b]; });
  int taken[kNumXcds] = {0};
  unsigned runs = 0;
  for (int i = 0; i < kNumXcds; ++i) {
    const int pass = i / n_groups, pos = i % n_groups;
    const int group = (pass & 1) ? n_groups - 1 - pos : pos;
    runs |= (unsigned)(group * per_group + taken[group]++) << (4 * by_speed[i]);
  }
  return runs;
}
}  // namespace

int32_t plan_split_cuts(const float *xcd_speed, int64_t tiles, int n_kv_heads, int n_splits, int max_nt, int n_cu,
                        double q_bytes_per_kv_head, uint32_t cuts[kMaxCutHeads][33], int32_t *use, int32_t *kv_group,
                        uint32_t *xcd_runs) {
  *use = 0;
  *kv_group = kDefaultKvGroup;
  *xcd_runs = kIdentityXcdRuns;
  for (int h = 0; h < kMaxCutHeads; ++h)
    for (int s = 0; s <= kMaxCutSplits; ++s) cuts[h][s] = 0;
  if (!xcd_speed || n_splits <= 1 || tiles <= 0) return BA_OK;
  for (int x = 0; x < kNumXcds; ++x)
    if (!(xcd_speed[x] >= 0.5f && xcd_speed[x] <= 2.0f))
      return fail(BA_ERR_INVALID_ARG, "xcd_speed[%d] = %g: relative speeds lie between 0.5 and 2", x, (double)xcd_speed[x]);
  if (n_kv_heads > kMaxCutHeads || n_splits > kMaxCutSplits || tiles * n_kv_heads * n_splits > 0x7fffffff) return BA_OK;  // equal splits
  // The speed of (KV head, split) = the mean speed of the XCDs that run its row tiles (item_id,
  // xcd_of_work_item), and a KV head's key range is shared out in proportion to its splits' speeds.
  // How far that can even out the XCDs depends on the order of the work items: with small groups of
  // KV heads an XCD fetches few query rows but shares a KV head with few other XCDs; with one group
  // of all KV heads every XCD fetches every query row and all of them can be balanced against each
  // other.  Every group size (a power of two that divides the KV heads, or all of them) is tried, with
  // the XCDs in their own order and dealt to the groups by speed (deal_xcd_runs).
  double best = 0.0;
  int best_group = 0;
  for (int g = 1; g <= n_kv_heads; g = (2 * g <= n_kv_heads || g == n_kv_heads) ? 2 * g : n_kv_heads) {
    if (n_kv_heads % g) continue;
    const unsigned dealt = deal_xcd_runs(xcd_speed, tiles, n_kv_heads, n_splits, g);
    for (int k = 0; k < (dealt == kIdentityXcdRuns ? 1 : 2); ++k) {
      const unsigned runs = k ? dealt : kIdentityXcdRuns;
      uint32_t trial[kMaxCutHeads][33];
      const double t = try_kv_group(xcd_speed, tiles, n_kv_heads, n_splits, g, runs, std::max(1, max_nt), n_cu,
                                    q_bytes_per_kv_head, trial);
      if (!best_group || t < best - 1e-9) {
        best = t;
        best_group = g;
        *xcd_runs = runs;
        memcpy(cuts, trial, sizeof(trial));
      }
    }
  }
  *kv_group = best_group;
  *use = 1;
  return BA_OK;
}

int64_t build_final_meta(const int32_t *cu_q, const int32_t *cu_ctx, int n0, int n, int G, FinalMeta *meta) {
  memset(meta, 0, sizeof(*meta));
  meta->n = n;
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    meta->cu_q[i] = cu_q[n0 + i];
    meta->cu_ctx[i] = cu_ctx[n0 + i];
    meta->tile_start[i] = (int32_t)tiles;
    tiles += ((int64_t)(cu_q[n0 + i + 1] - cu_q[n0 + i]) * G + kTileRows - 1) / kTileRows;
  }
  meta->cu_q[n] = cu_q[n0 + n];
  meta->cu_ctx[n] = cu_ctx[n0 + n];
  meta->tile_start[n] = (int32_t)tiles;
  return tiles;
}

int32_t plan_final_blocks(const ba_heads *h, int32_t n_prompts, const int32_t *cu_q, const int32_t *cu_blk,
                          const int32_t *blk_len, bool have_rot_out, int32_t gather_below, int n_cu,
                          BlocksPlan *plan) {
  if (gather_below < 0 && gather_below != BA_GATHER_DEFAULT)
    return fail(BA_ERR_INVALID_ARG, "gather_below %d: a token count, 0 or BA_GATHER_DEFAULT", gather_below);
  if (gather_below == BA_GATHER_DEFAULT) gather_below = 256;
  if (n_prompts < 0 || (n_prompts > 0 && (!cu_q || !cu_blk)))
    return fail(BA_ERR_INVALID_ARG, "cu_q / cu_blk: null or negative prompt count");
  BlocksPlan pl;
  if (n_prompts > 0 && (cu_q[0] != 0 || cu_blk[0] != 0)) return fail(BA_ERR_INVALID_ARG, "cu_q[0] and cu_blk[0] must be 0");
  const int G = h->n_q_heads / h->n_kv_heads;
  int64_t max_nb = 0;  // most non-empty blocks in one prompt
  for (int n = 0; n < n_prompts; ++n) {
    const int64_t lq = (int64_t)cu_q[n + 1] - cu_q[n];
    if (lq < 1) return fail(BA_ERR_INVALID_ARG, "prompt %d: the final block needs at least one token", n);
    if (cu_blk[n + 1] < cu_blk[n]) return fail(BA_ERR_INVALID_ARG, "prompt %d: cu_blk decreases", n);
    if (cu_blk[n + 1] > cu_blk[n] && !blk_len) return fail(BA_ERR_INVALID_ARG, "blk_len is null");
    if (lq * G > 0x3fffffff) return fail(BA_ERR_INVALID_ARG, "prompt %d: too many packed rows", n);
    int64_t tiles = (lq + kTileKeys - 1) / kTileKeys, ctx = 0, nb = 0;
    for (int b = cu_blk[n]; b < cu_blk[n + 1]; ++b) {
      if (blk_len[b] < 0) return fail(BA_ERR_INVALID_ARG, "block %d: negative length", b);
      if (blk_len[b] == 0) continue;
      tiles += (blk_len[b] + kTileKeys - 1) / kTileKeys;
      ctx += blk_len[b];
      ++nb;
    }
    if (ctx > 0x3fffffff || tiles > 0x1ffffff) return fail(BA_ERR_INVALID_ARG, "prompt %d: context too long", n);
    max_nb = std::max(max_nb, nb);
    pl.n_blocks += nb;
    pl.total_tiles += (lq * G + kTileRows - 1) / kTileRows;
    pl.max_nt = std::max(pl.max_nt, (int)tiles);
  }
  pl.lq_total = n_prompts > 0 ? cu_q[n_prompts] : 0;
  // The kernel that reads the block table pays a fixed price per block (it turns its queries at
  // every block boundary), a gathered copy a price per token: short blocks are gathered.
  int64_t ctx_total = 0;
  pl.cu_ctx.assign(n_prompts + 1, 0);
  for (int n = 0; n < n_prompts; ++n) {
    for (int b = cu_blk[n]; b < cu_blk[n + 1]; ++b) ctx_total += blk_len[b];
    if (ctx_total > 0x3fffffff) return fail(BA_ERR_INVALID_ARG, "context too long");
    pl.cu_ctx[n + 1] = (int32_t)ctx_total;
  }
  if (pl.n_blocks > 0 && ctx_total < (int64_t)gather_below * pl.n_blocks) {
    FinalPlan fp;
    int32_t rc = plan_final(h, n_prompts, cu_q, pl.cu_ctx.data(), BA_ROPE_APPLY, have_rot_out, n_cu, &fp);
    if (rc) return rc;
    pl.gather = true;
    pl.gather_kv_bytes = (size_t)ctx_total * h->n_kv_heads * h->head_dim * 2;
    pl.gather_final_bytes = fp.total();
    *plan = pl;
    return BA_OK;
  }
  if (max_nb > kBlkMaxBlocks)
    return fail(BA_ERR_UNSUPPORTED, "%lld cached blocks in one prompt, at most %d when the kernel reads the block table",
                (long long)max_nb, kBlkMaxBlocks);
  pl.n_splits = choose_splits(pl.total_tiles * h->n_kv_heads, pl.max_nt, n_cu, h->head_dim);
  if (!have_rot_out) pl.kf_bytes = (size_t)pl.lq_total * h->n_kv_heads * h->head_dim * 2;
  pl.q_bytes = (size_t)pl.lq_total * h->n_q_heads * h->head_dim * 2;
  pl.rot_bytes = (size_t)pl.n_blocks * h->head_dim * 4;  // D/2 (cos, sin) pairs per block
  if (pl.n_splits > 1) {
    const size_t rows = partial_rows(pl.total_tiles, h->n_kv_heads);
    pl.part_o_bytes = (size_t)pl.n_splits * rows * h->head_dim * 2;
    pl.part_ml_bytes = (size_t)pl.n_splits * rows * 2 * 4;
    pl.part_idx_bytes = rows * 4;
  }
  *plan = pl;
  return BA_OK;
}

// Blocks up to this length take the schedule with small workgroups, several to a compute unit; longer
// ones the main core.  (The short-block kernel addresses the rows of a block with 32-bit element
// offsets.)
// Fewer than four query heads per KV head make few row tiles of a block, and both schedules give such a call
// the same bits, so the call as a whole takes one.  The main core walks a long block faster (a tile of 64 keys
// in 1.0 us against two of 32 in 1.5, D = 128), but runs one workgroup per compute unit and spends on each
// what four tiles take: the small workgroups win where there are more of those than compute units to run
// them.  So the main core has the call if a block is long enough to tell (512 tokens) and its own work (a
// workgroup's mean walk and the fixed part, over all compute units) comes to no more than two thirds of
// its longest workgroup.  Main core / small workgroups, us: 8 over 8 heads of 128: one block of 2,048: 52 / 60,
// of 6,144: 121 / 154, two of 6,144: 222 / 204, 24 of 512: 72 / 59; 4 over 4 of 64: 8 of 2,048: 50 / 60; 3 over 1 of
// 64: 24 of 1,024: 43 / 32, 8 of 2,048: 44 / 46; 16 over 8 of 128: one of 6,000 and 160 of 200: 362 / 273, and at 2
// over 2: 134 / 159.  Of 706 calls of such groups (1 to 8,000 row tiles) the rule leaves these with the slower
// schedule by 2 % or more: 24 blocks of 384 and 512 at 4 over 4 heads of 128 (4 %), two of 6,144 at 24 over 8 (3 %).
int64_t encode_short_max(const ba_heads *h, int32_t n_blocks, const int32_t *offs, int64_t widest_stride) {
  if (((int64_t)kShortMaxLen + 1) * widest_stride >= 0x40000000) return -1;
  const int G = h->n_q_heads / h->n_kv_heads;
  if (G >= kSmallGroup) return kShortMaxLen;
  int64_t longest = 0, twice_load = 0;  // in key tiles; over the main core's workgroups
  for (int b = 0; b < n_blocks; ++b) {
    const int64_t len = (int64_t)offs[b + 1] - offs[b];
    const int64_t n_t = (len + kTileKeys - 1) / kTileKeys;
    longest = std::max(longest, len);
    twice_load += (len * G + kTileRows - 1) / kTileRows * h->n_kv_heads * (n_t + 1 + 2 * kFixedTiles);
  }
  const int64_t longest_wg = (longest + kTileKeys - 1) / kTileKeys + kFixedTiles;
  if (longest > kSmallGroupShortLen && 3 * twice_load <= 4 * kEncodeCus * longest_wg) return -1;
  return kShortMaxLen;
}

int32_t build_encode_metas(const int32_t *block_offsets, int b0, int n, int G, int64_t short_max, EncodeMeta meta[2],
                           int64_t tiles[2]) {
  tiles[0] = tiles[1] = 0;
  memset(meta, 0, 2 * sizeof(EncodeMeta));
  for (int i = 0; i < n; ++i) {
    const int64_t len = (int64_t)block_offsets[b0 + i + 1] - block_offsets[b0 + i];
    if (len * G > 0x3fffffff) return fail(BA_ERR_INVALID_ARG, "block %d: too many packed rows", b0 + i);
    const int which = len <= short_max ? 1 : 0;
    for (int m = 0; m < 2; ++m) {
      meta[m].offs[i] = block_offsets[b0 + i];
      meta[m].tile_start[i] = (int32_t)tiles[m];
    }
    const int tile_rows = which ? kShortTileRows : kTileRows;
    tiles[which] += (len * G + tile_rows - 1) / tile_rows;
    if (tiles[which] > 0x3fffffff) return fail(BA_ERR_INVALID_ARG, "too many row tiles in one call");
  }
  for (int m = 0; m < 2; ++m) {
    meta[m].n = n;
    meta[m].offs[n] = block_offsets[b0 + n];
    meta[m].tile_start[n] = (int32_t)tiles[m];
    for (int i = n + 1; i <= kEncMaxBlocks; ++i) meta[m].tile_start[i] = 0x7fffffff;
  }
  return BA_OK;
}

std::vector<PromptBlock> list_prompt_blocks(int32_t n_prompts, const int32_t *cu_blk, const int32_t *block_offsets) {
  std::vector<PromptBlock> blks;
  for (int n = 0; n < n_prompts; ++n) {
    const int last = cu_blk[n + 1] - 1;
    const int32_t fs = block_offsets[last], fl = block_offsets[last + 1] - fs;
    for (int b = cu_blk[n]; b <= last; ++b) {
      const int32_t len = block_offsets[b + 1] - block_offsets[b];
      if (len == 0) continue;
      // first key a block sees: its own first token, or for a prompt's last block the prompt's
      blks.push_back({block_offsets[b], len, b == last ? block_offsets[cu_blk[n]] : block_offsets[b], fs,
                      b == last ? 0 : fl, n, block_offsets[b] - block_offsets[cu_blk[n]]});
    }
  }
  return blks;
}

namespace {
constexpr int kPromptKeys = 32;  // keys per tile of the forward and dq kernels
int walk_tiles(int64_t keys) { return (int)((keys - 1) / kPromptKeys + 1); }
int64_t short_row_tiles(int64_t len, int64_t G) { return (len * G + kShortTileRows - 1) / kShortTileRows; }
// a last block that sees enough of its prompt for more than one workgroup per row tile
int shared_splits(int64_t ctx, int64_t len, int64_t G, int n_kv_heads, const WalkShares &ws) {
  if (ctx <= 0 || len <= 0) return 1;
  const int w = walk_tiles(ctx + len);
  const int64_t pairs = short_row_tiles(len, G) * n_kv_heads;
  if (w <= kShareAbove) return 1;
  if (pairs <= kSharePairs / 2) return shared_walk_splits(w, kShareChunk, (int)pairs, kSharePairs);
  if (ws.chunk == 0 || w <= kShareManyAbove || pairs > kShareManyPairs || n_kv_heads > kSharePairs / 2) return 1;
  return shared_walk_splits(w, w >= kShareLongWalk ? ws.long_chunk : ws.chunk, (int)pairs, kShareManyPairs);
}

// many: last blocks of many row tiles too; any_many: whether the call has any.
WalkShares plan_shares(const ba_heads *h, int32_t n_prompts, const int32_t *cu_blk, const int32_t *block_offsets, bool dq, bool many, bool *any_many) {
  WalkShares ws;
  const int64_t G = h->n_q_heads / h->n_kv_heads;
  const bool wide = h->head_dim == 128;
  if (many) {
    ws.chunk = wide ? kShareManyChunk : kShareChunk;
    ws.long_chunk = dq && wide && G >= kSmallGroup && h->n_kv_heads >= 4 ? kShareLongChunk : ws.chunk;
  }
  const double part_tiles = wide ? kSharePartTiles : 0.0;
  double load = 0.0;  // of the launch with its walks cut, in key tiles
  int longest = 0, longest_left = 0;  // of the walks that would be cut, and of the others
  *any_many = false;
  const auto add = [&](int64_t ctx, int64_t len, int s) {
    load += (double)short_row_tiles(len, G) * (((double)ctx + 0.5 * (double)len) / kPromptKeys + 0.5 + kFixedTiles + part_tiles * (s - 1));
    int &most = s > 1 ? longest : longest_left;
    if (len > 0) most = std::max(most, walk_tiles(ctx + len));
  };
  for (int n = 0; n < n_prompts; ++n) {
    const int last = cu_blk[n + 1] - 1;
    for (int b = cu_blk[n]; b < last; ++b) add(0, block_offsets[b + 1] - block_offsets[b], 1);
    const int64_t len = block_offsets[last + 1] - block_offsets[last], ctx = block_offsets[last] - block_offsets[cu_blk[n]];
    const int s = shared_splits(ctx, len, G, h->n_kv_heads, ws);
    add(ctx, len, s);
    if (s < 2) continue;
    ++ws.n_split;
    ws.items += short_row_tiles(len, G) * s;
    *any_many = *any_many || short_row_tiles(len, G) * h->n_kv_heads > kSharePairs / 2;
  }
  load *= h->n_kv_heads / (double)kShareCus;  // ... per compute unit
  const size_t slots = (size_t)ws.items * h->n_kv_heads * (kShortTileRows / 32);
  const double least = dq && *any_many ? dq_share_load(h->head_dim, G) : kShareLoad;
  if (ws.n_split == 0 || longest < least * load) return WalkShares();
  const int lead = longest_left / (*any_many ? kShareManyLead : kShareLead);
  if (longest <= longest_left + lead && longest <= (*any_many && !dq ? kShareManyAnyway : kShareAnyway) * load) return WalkShares();
  // (the tables need the first: the shared blocks are in the first launch's.  With 8 KV heads it would take over 170 prompts, whose
  // load is far beyond the line)
  if (ws.n_split > kEncMaxBlocks || slots * 32 * h->head_dim * 4 > kShareMaxBytes) return WalkShares();
  ws.part_bytes = slots * 32 * h->head_dim * 4;
  ws.ml_bytes = slots * 256;
  ws.count_bytes = (size_t)ws.items * h->n_kv_heads * 4;
  return ws;
}
}  // namespace

WalkShares plan_walk_shares(const ba_heads *h, int32_t n_prompts, const int32_t *cu_blk, const int32_t *block_offsets, bool dq) {
  bool any_many;
  const WalkShares ws = plan_shares(h, n_prompts, cu_blk, block_offsets, dq, true, &any_many);
  if (ws.n_split > 0 || !any_many) return ws;
  return plan_shares(h, n_prompts, cu_blk, block_offsets, dq, false, &any_many);
}

namespace {
// row tiles that see a block's first key
int64_t kv_walk(int64_t len, int64_t fin_len, int64_t G) {
  return (len * G + kKvTileRows - 1) / kKvTileRows + (fin_len * G + kKvTileRows - 1) / kKvTileRows;
}
int kv_splits(int64_t len, int64_t fin_len, int64_t G, int chunk) {
  const int64_t w = kv_walk(len, fin_len, G);
  return w > kKvShareAbove && w < (1 << 20) ? walk_splits((int)w, chunk) : 1;
}
int64_t key_tiles(int64_t len) { return (len + kBwdTileKeys - 1) / kBwdTileKeys; }
}  // namespace

WalkShares plan_kv_shares(const ba_heads *h, int32_t n_prompts, const int32_t *cu_blk, const int32_t *block_offsets) {
  WalkShares ws;
  const int64_t G = h->n_q_heads / h->n_kv_heads;
  double load = 0.0;
  int64_t longest = 0;
  const auto each = [&](auto &&visit) {
    for (int n = 0; n < n_prompts; ++n) {
      const int last = cu_blk[n + 1] - 1;
      const int64_t fin = block_offsets[last + 1] - block_offsets[last];
      for (int b = cu_blk[n]; b <= last; ++b) {
        const int64_t len = block_offsets[b + 1] - block_offsets[b];
        if (len > 0) visit(len, b == last ? (int64_t)0 : fin);
      }
    }
  };
  each([&](int64_t len, int64_t fin) {
    const double n_kt = (double)key_tiles(len);
    load += n_kt * ((double)kv_walk(len, fin, G) - 0.5 * (double)len * (double)G / kKvTileRows + kFixedTiles);
    longest = std::max(longest, kv_walk(len, fin, G));
  });
  load *= h->n_kv_heads / (double)kShareCus;  // ... per compute unit
  if (longest <= kKvShareAbove || (double)longest < kKvShareLoad * load) return ws;
  const int chunk = std::max(kKvShareChunk, (int)std::min(1e6, 0.5 * load));
  double left = kKvShareLoad * load;  // what the launch takes with its walks cut
  each([&](int64_t len, int64_t fin) {
    const int s = kv_splits(len, fin, G, chunk);
    left = std::max(left, (double)((kv_walk(len, fin, G) + s - 1) / s));
    if (s < 2) return;
    ++ws.n_split;
    ws.items += key_tiles(len) * s;
  });
  if (h->head_dim == 128 && G >= 4 && (double)longest < kKvShareLight * load && (double)longest < left + kKvShareLead) return WalkShares();
  const size_t slots = (size_t)ws.items * h->n_kv_heads * (kBwdTileKeys / 16);  // a pair of waves per 32 keys
  if (ws.n_split == 0 || ws.n_split > kEncMaxBlocks || slots * 32 * h->head_dim * 4 > kShareMaxBytes) return WalkShares();
  ws.chunk = chunk;
  ws.part_bytes = slots * 32 * h->head_dim * 4;
  ws.count_bytes = (size_t)ws.items * h->n_kv_heads * 4;
  return ws;
}

void sort_by_query_rows(std::vector<PromptBlock> *blks, int G, const WalkShares &shares) {
  const auto shared = [&](const PromptBlock &b) { return shares.n_split > 0 && kv_splits(b.len, b.fin_len, G, shares.chunk) > 1; };
  std::stable_sort(blks->begin(), blks->end(), [&](const PromptBlock &a, const PromptBlock &b) {
    const bool sa = shared(a), sb = shared(b);
    if (sa != sb) return sa;
    return a.len + a.fin_len > b.len + b.fin_len;
  });
}

int64_t build_kv_meta(const std::vector<PromptBlock> &blks, size_t b0, int n, int G, const WalkShares &shares, BwdKvMeta *meta) {
  memset(meta, 0, sizeof(*meta));
  meta->n = n;
  meta->n_split = b0 == 0 ? shares.n_split : 0;
  meta->chunk = shares.chunk;
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    const PromptBlock &b = blks[b0 + i];
    meta->start[i] = b.start;
    meta->len[i] = b.len;
    meta->pos0[i] = b.pos0;
    meta->fin_start[i] = b.fin_start;
    meta->fin_len[i] = b.fin_len;
    meta->tile_start[i] = (int32_t)tiles;
    tiles += key_tiles(b.len) * (i < meta->n_split ? kv_splits(b.len, b.fin_len, G, shares.chunk) : 1);
    if (tiles > 0x3fffffff) return -1;
  }
  for (int i = n; i <= kEncMaxBlocks; ++i) meta->tile_start[i] = i == n ? (int32_t)tiles : 0x7fffffff;
  return tiles;
}

void sort_by_key_range(std::vector<PromptBlock> *blks, int G, int n_kv_heads, const WalkShares &shares) {
  // (a prompt's last block walks the whole prompt, and a launch should not end on a few of those)
  const auto shared = [&](const PromptBlock &b) {
    return shares.n_split > 0 && shared_splits(b.start - b.kstart, b.len, G, n_kv_heads, shares) > 1;
  };
  std::stable_sort(blks->begin(), blks->end(), [&](const PromptBlock &a, const PromptBlock &b) {
    const bool sa = shared(a), sb = shared(b);
    if (sa != sb) return sa;
    return (int64_t)a.start + a.len - a.kstart > (int64_t)b.start + b.len - b.kstart;
  });
}

int64_t build_prompt_meta(const std::vector<PromptBlock> &blks, size_t b0, int n, int G, int n_kv_heads, const WalkShares &shares,
                          PromptMeta *meta) {
  memset(meta, 0, sizeof(*meta));
  meta->n = n;
  meta->n_split = b0 == 0 ? shares.n_split : 0;
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    const PromptBlock &b = blks[b0 + i];
    meta->start[i] = b.start;
    meta->len[i] = b.len;
    meta->kstart[i] = b.kstart;
    meta->pos0[i] = b.pos0;
    meta->tile_start[i] = (int32_t)tiles;
    tiles += short_row_tiles(b.len, G) * (i < meta->n_split ? shared_splits((int64_t)b.start - b.kstart, b.len, G, n_kv_heads, shares) : 1);
    if (tiles > 0x3fffffff) return -1;
  }
  meta->tile_start[n] = (int32_t)tiles;
  for (int i = n + 1; i <= kEncMaxBlocks; ++i) meta->tile_start[i] = 0x7fffffff;
  return tiles;
}

namespace {

// largest i < n with tile_start[i] <= tile: what the kernels look up
int segment_of(const int32_t *tile_start, int n, int tile) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (tile_start[mid] <= tile) lo = mid; else hi = mid;
  }
  return lo;
}

struct ItemSink {
  ba_work_item *out;
  int64_t max, n = 0;
  void put(const ba_work_item &w) {
    if (out && n < max) out[n] = w;
    ++n;
  }
};

}  // namespace
}  // namespace ba

extern "C" {

const char *ba_last_error(void) { return ba::last_error(); }

int64_t ba_schedule_final_block(const ba_heads *heads, int32_t n_prompts, const int32_t *cu_q, const int32_t *cu_ctx,
                                int32_t n_compute_units, ba_work_item *items, int64_t max_items) {
  int32_t rc;
  if ((rc = ba::check_heads(heads, true))) return rc;
  if (n_compute_units < 1) return ba::fail(BA_ERR_INVALID_ARG, "n_compute_units must be positive");
  ba::FinalPlan pl;
  if ((rc = ba::plan_final(heads, n_prompts, cu_q, cu_ctx, BA_ROPE_APPLY, false, n_compute_units, &pl))) return rc;
  const int G = heads->n_q_heads / heads->n_kv_heads;
  ba::ItemSink sink{items, items ? max_items : 0};
  int launch = 0;
  for (int n0 = 0; n0 < n_prompts; n0 += ba::kFinMaxPrompts, ++launch) {
    const int n = std::min(ba::kFinMaxPrompts, n_prompts - n0);
    ba::FinalMeta meta;
    const int64_t tiles = ba::build_final_meta(cu_q, cu_ctx, n0, n, G, &meta);
    uint32_t cuts[ba::kMaxCutHeads][33];
    int32_t use_cuts = 0;
    int32_t kv_group = 0;
    uint32_t xcd_runs = ba::kIdentityXcdRuns;
    if ((rc = ba::plan_split_cuts(heads->xcd_speed, tiles, heads->n_kv_heads, pl.n_splits, pl.max_nt, n_compute_units,
                                  ba::final_q_bytes_per_kv_head(heads, pl.lq_total), cuts, &use_cuts, &kv_group, &xcd_runs)))
      return rc;
    // the kernel's own walk: every (split, row tile) of the launch; the same at every KV head unless
    // the splits are sized by XCD speed, when every KV head has shares of its own
    const ba::ItemOrder order = {(int)tiles, heads->n_kv_heads, pl.n_splits, kv_group};
    const int64_t n_wg = tiles * heads->n_kv_heads * pl.n_splits;
    for (int kvh = use_cuts ? 0 : -1; kvh < (use_cuts ? heads->n_kv_heads : 0); ++kvh)
    for (int split = 0; split < pl.n_splits; ++split)
      for (int64_t tile = 0; tile < tiles; ++tile) {
        const int i = ba::segment_of(meta.tile_start, meta.n, (int)tile);
        const int lq = meta.cu_q[i + 1] - meta.cu_q[i], tctx = meta.cu_ctx[i + 1] - meta.cu_ctx[i];
        const int jt = (int)tile - meta.tile_start[i];
        const int n_rows = lq * G, row0 = jt * ba::kTileRows;
        const int last_row = std::min(n_rows, row0 + ba::kTileRows) - 1;
        const int n_ctx_tiles = (tctx + ba::kTileKeys - 1) / ba::kTileKeys;
        const int n_causal = ba::causal_key_tiles(last_row / G, ba::kTileKeys);
        const ba::TileRange tr = ba::split_tile_range(n_ctx_tiles, n_causal, pl.n_splits, split, use_cuts ? cuts[kvh] : nullptr);
        ba_work_item w;
        memset(&w, 0, sizeof(w));
        w.launch = launch;
        w.problem = n0 + i;
        w.first_token = meta.cu_q[i];
        w.tile_rows = ba::kTileRows;
        w.tile_keys = ba::kTileKeys;
        w.row_begin = row0;
        w.row_end = last_row + 1;
        w.split = split;
        w.n_splits = pl.n_splits;
        w.kv_head = kvh;
        w.xcd = kvh >= 0 && n_wg <= 0x7fffffff
                    ? ba::xcd_of_work_item(ba::item_id((int)tile, kvh, split, order), (unsigned)n_wg, xcd_runs) : -1;
        w.ctx_begin = std::min(tctx, std::min(tr.begin, n_ctx_tiles) * ba::kTileKeys);
        w.ctx_end = std::min(tctx, std::min(tr.end, n_ctx_tiles) * ba::kTileKeys);
        w.self_begin = std::min(lq, std::max(0, tr.begin - n_ctx_tiles) * ba::kTileKeys);
        w.self_end = std::min(lq, std::max(0, tr.end - n_ctx_tiles) * ba::kTileKeys);
        sink.put(w);
      }
  }
  return sink.n;
}

int64_t ba_schedule_encode_blocks(const ba_heads *heads, int32_t n_blocks, const int32_t *block_offsets,
                                  ba_work_item *items, int64_t max_items) {
  int32_t rc;
  if ((rc = ba::check_heads(heads, true))) return rc;
  if ((rc = ba::check_offsets(n_blocks, block_offsets))) return rc;
  const int G = heads->n_q_heads / heads->n_kv_heads;
  const int64_t short_max = ba::encode_short_max(heads, n_blocks, block_offsets, (int64_t)heads->n_q_heads * heads->head_dim);
  ba::ItemSink sink{items, items ? max_items : 0};
  int launch = 0;
  for (int b0 = 0; b0 < n_blocks; b0 += ba::kEncMaxBlocks) {
    const int n = std::min(ba::kEncMaxBlocks, n_blocks - b0);
    ba::EncodeMeta meta[2];
    int64_t tiles[2];
    if ((rc = ba::build_encode_metas(block_offsets, b0, n, G, short_max, meta, tiles))) return rc;
    for (int m = 1; m >= 0; --m) {
      if (tiles[m] == 0) continue;
      const int tile_rows = m ? ba::kShortTileRows : ba::kTileRows, tile_keys = m ? 32 : ba::kTileKeys;
      for (int64_t tile = 0; tile < tiles[m]; ++tile) {
        const int i = ba::segment_of(meta[m].tile_start, meta[m].n, (int)tile);
        const int lq = meta[m].offs[i + 1] - meta[m].offs[i];
        const int jt = (int)tile - meta[m].tile_start[i];
        const int n_rows = lq * G, row0 = jt * tile_rows;
        const int last_row = std::min(n_rows, row0 + tile_rows) - 1;
        ba_work_item w;
        memset(&w, 0, sizeof(w));
        w.kv_head = w.xcd = -1;
        w.launch = launch;
        w.problem = b0 + i;
        w.first_token = meta[m].offs[i];
        w.tile_rows = tile_rows;
        w.tile_keys = tile_keys;
        w.row_begin = row0;
        w.row_end = last_row + 1;
        w.n_splits = 1;
        w.self_end = std::min(lq, ba::causal_key_tiles(last_row / G, tile_keys) * tile_keys);
        sink.put(w);
      }
      ++launch;
    }
  }
  return sink.n;
}

int64_t ba_schedule_prompts(const ba_heads *heads, int32_t n_prompts, const int32_t *cu_blk,
                            const int32_t *block_offsets, ba_work_item *items, int64_t max_items) {
  int32_t rc;
  if ((rc = ba::check_heads(heads, true))) return rc;
  if ((rc = ba::check_prompt_blocks(n_prompts, cu_blk, block_offsets))) return rc;
  const int G = heads->n_q_heads / heads->n_kv_heads;
  const ba::WalkShares shares = ba::plan_walk_shares(heads, n_prompts, cu_blk, block_offsets, false);
  std::vector<ba::PromptBlock> blks = ba::list_prompt_blocks(n_prompts, cu_blk, block_offsets);
  ba::sort_by_key_range(&blks, G, heads->n_kv_heads, shares);
  ba::ItemSink sink{items, items ? max_items : 0};
  int launch = 0;
  for (size_t b0 = 0; b0 < blks.size(); b0 += ba::kEncMaxBlocks, ++launch) {
    const int n = (int)std::min<size_t>(ba::kEncMaxBlocks, blks.size() - b0);
    ba::PromptMeta meta;
    const int64_t tiles = ba::build_prompt_meta(blks, b0, n, G, heads->n_kv_heads, shares, &meta);
    if (tiles < 0) return ba::fail(BA_ERR_INVALID_ARG, "too many row tiles in one call");
    for (int64_t tile = 0; tile < tiles; ++tile) {
      const int i = ba::segment_of(meta.tile_start, meta.n, (int)tile);
      const int lq = meta.len[i], dq = meta.start[i] - meta.kstart[i];  // dq: earlier tokens of the prompt it sees
      int jt = (int)tile - meta.tile_start[i], split = 0, n_splits = 1;
      const int n_rows = lq * G;
      if (i < meta.n_split) {
        const int n_rt = (n_rows + ba::kShortTileRows - 1) / ba::kShortTileRows;
        n_splits = ba::shared_splits(dq, lq, G, heads->n_kv_heads, shares);
        split = jt / n_rt;
        jt -= split * n_rt;
      }
      const int row0 = jt * ba::kShortTileRows;
      const int last_row = std::min(n_rows, row0 + ba::kShortTileRows) - 1;
      // keys counted from the first visible one: tiles up to the one that holds the last row's own token
      const ba::TileRange walk = ba::walk_split_range((dq + last_row / G) / 32 + 1, n_splits, split);
      const int k_begin = walk.begin * 32, k_end = walk.end * 32;
      ba_work_item w;
      memset(&w, 0, sizeof(w));
      w.kv_head = w.xcd = -1;
      w.launch = launch;
      w.problem = blks[b0 + i].prompt;
      w.first_token = meta.start[i];
      w.tile_rows = ba::kShortTileRows;
      w.tile_keys = 32;
      w.row_begin = row0;
      w.row_end = last_row + 1;
      w.split = split;
      w.n_splits = n_splits;
      w.ctx_begin = std::min(dq, k_begin);
      w.ctx_end = std::min(dq, k_end);
      w.self_begin = std::min(lq, std::max(0, k_begin - dq));
      w.self_end = std::min(lq, std::max(0, k_end - dq));
      sink.put(w);
    }
  }
  return sink.n;
}

}  // extern "C"
