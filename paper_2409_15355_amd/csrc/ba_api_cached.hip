// C boundary, the final block straight from a table of cached blocks (Section 2.3 Eq. 2-3 folded into
// Section 2.5): the block-table launches, and the gathered route for short blocks.
#include <string.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "ba_api_common.h"

namespace {
using ba::align256;
using ba::check_heads;
using ba::check_offsets;
using ba::check_prompt_blocks;
using ba::fail;
using ba::FinalPlan;
using ba::BlocksPlan;
using ba::device_fail;
using ba::num_cus;
using namespace ba::api;
}  // namespace
// ------------------------------------------------------------------------------------------
namespace {

struct BlocksCall {
  const ba_heads *heads;
  const ba::RopeTable *rt;
  const ba_tensor *q_f;
  uint16_t *q_ws;
  const ba_tensor *k_f;
  const ba_tensor *kf_use;
  float *rot_ws;
  int32_t n_prompts;
  const int32_t *cu_q, *cu_blk, *blk_tok_off, *blk_len, *blk_old_pos0, *blk_new_pos0, *q_pos0;
  hipStream_t stream;
  int max_nt;  // longest walk of the call, key tiles
};

// Launches of at most MetaT::kPrompts prompts and MetaT::kBlocks non-empty blocks each: the RoPE
// pre-pass (fresh q and k of the chunk, rotations of its blocks), then the attention core.
template <typename MetaT, typename RotsT>
int32_t run_final_blocks(const BlocksCall &c, ba::AttnParams ap) {
  const int D = c.heads->head_dim, G = c.heads->n_q_heads / c.heads->n_kv_heads;
  std::vector<MetaT> metas(1);
  std::vector<RotsT> rots(1);
  int n0 = 0;
  int64_t rot_base = 0, tile_base = 0;
  while (n0 < c.n_prompts) {
    MetaT &meta = metas[0];
    RotsT &rr = rots[0];
    memset(&meta, 0, sizeof(meta));
    memset(&rr, 0, sizeof(rr));
    int np = 0, nb = 0;
    int64_t tiles = 0;
    std::vector<int32_t> pos0;
    while (n0 + np < c.n_prompts && np < MetaT::kPrompts) {
      const int n = n0 + np;
      int cnt = 0;
      for (int b = c.cu_blk[n]; b < c.cu_blk[n + 1]; ++b) cnt += c.blk_len[b] > 0;
      if (nb + cnt > MetaT::kBlocks) break;  // (a single prompt always fits: checked by the plan)
      meta.cu_q[np] = c.cu_q[n];
      meta.cu_blk[np] = nb;
      meta.tile_start[np] = (int32_t)tiles;
      int32_t ctx_tiles = 0;
      int64_t run = 0;  // the prompt's context so far = default position of the next block
      for (int b = c.cu_blk[n]; b < c.cu_blk[n + 1]; ++b) {
        const int32_t new0 = c.blk_new_pos0 ? c.blk_new_pos0[b] : (int32_t)run;
        run += c.blk_len[b];
        if (c.blk_len[b] == 0) continue;
        meta.blk_off[nb] = c.blk_tok_off[b];
        meta.blk_len[nb] = c.blk_len[b];
        meta.blk_tile0[nb] = ctx_tiles;
        ctx_tiles += (c.blk_len[b] + ba::kTileKeys - 1) / ba::kTileKeys;
        // the queries are turned back by the block's shift: angle = -(new - old) positions
        rr.angle[nb] = -(new0 - (c.blk_old_pos0 ? c.blk_old_pos0[b] : 0));
        ++nb;
      }
      meta.ctx_tiles[np] = ctx_tiles;
      pos0.push_back(c.q_pos0 ? c.q_pos0[n] : (int32_t)run);
      tiles += ((int64_t)(c.cu_q[n + 1] - c.cu_q[n]) * G + ba::kTileRows - 1) / ba::kTileRows;
      ++np;
    }
    meta.n = np;
    meta.cu_q[np] = c.cu_q[n0 + np];
    meta.cu_blk[np] = nb;
    meta.tile_start[np] = (int32_t)tiles;
    meta.rot_base = (int32_t)rot_base;
    ap.total_tiles = (int32_t)tiles;
    ap.tile_base = (int32_t)tile_base;
    tile_base += tiles;
    {
      int32_t rc_cuts = ba::plan_split_cuts(c.heads->xcd_speed, tiles, c.heads->n_kv_heads, ap.n_splits, c.max_nt, num_cus(),
                                            ba::final_q_bytes_per_kv_head(c.heads, c.cu_q[c.n_prompts]), ap.split_cut,
                                            &ap.use_cuts, &ap.kv_group, &ap.xcd_runs);
      if (rc_cuts) return rc_cuts;
    }
    const ba::RopeRots *big = nullptr;
    const ba::RopeRotsSmall *small = nullptr;
    if constexpr (std::is_same<RotsT, ba::RopeRots>::value) big = &rr; else small = &rr;
    int32_t rc = run_rope_prepass(c.heads, *c.rt, c.q_f, c.q_ws, c.k_f, c.kf_use, np, meta.cu_q, pos0.data(), c.stream,
                                  big, small, c.rot_ws + rot_base * D, nb);
    if (rc) return rc;
    hipError_t e;
    {
      ProfileScope ps(BA_PROFILE_ATTENTION, c.stream);
      e = ba::launch_attn_final_blocks(ap, meta, c.stream);
    }
    if (e != hipSuccess) return device_fail(e, "final-block (cached) attention launch");
    rot_base += nb;
    n0 += np;
  }
  return BA_OK;
}

// Whether the attention kernel turns a context's keys itself: where that pays (turn_pays) and a split's part of the tables of FinalTurnMeta
// fits in LDS, and where it lies there: the longest split's tiles (tables are fetched sixteen tiles at a time), the rotations of the
// blocks that the most mixed one meets.
bool turn_layout(const ba_heads *h, int32_t n_prompts, const int32_t *cu_q, const int32_t *cu_ctx, const int32_t *ctx0,
                 const std::vector<int32_t> &first_row, int n_splits, uint32_t *blk_at, uint32_t *rot_at) {
  const int G = h->n_q_heads / h->n_kv_heads;
  int most_tiles = 1, most_blocks = 1;
  double turned = 0.0, walked = 0.0;  // tokens whose keys a row tile turns, tiles in the walks of all row tiles
  const auto block_of = [&](int64_t row) { return (int)(std::upper_bound(first_row.begin(), first_row.end(), (int32_t)row) - first_row.begin()) - 1; };
  for (int n = 0; n < n_prompts; ++n) {
    const int ctx_tiles = (cu_ctx[n + 1] - cu_ctx[n] + ba::kTileKeys - 1) / ba::kTileKeys;
    const int64_t n_rows = (int64_t)(cu_q[n + 1] - cu_q[n]) * G;
    const double row_tiles = (double)((n_rows + ba::kTileRows - 1) / ba::kTileRows);
    turned += row_tiles * (double)(cu_ctx[n + 1] - cu_ctx[n]);
    walked += row_tiles * (double)ctx_tiles;
    for (int64_t row0 = 0; row0 < n_rows; row0 += ba::kTileRows) {
      const int causal = ba::causal_key_tiles((int)((std::min(n_rows, row0 + ba::kTileRows) - 1) / G), ba::kTileKeys);
      for (int s = 0; s < n_splits; ++s) {
        const ba::TileRange r = ba::split_tile_range(ctx_tiles, causal, n_splits, s);
        const int end = std::min(r.end, ctx_tiles);
        if (end <= r.begin) continue;
        most_tiles = std::max(most_tiles, end - r.begin);
        most_blocks = std::max(most_blocks, block_of((int64_t)ctx0[n] + (int64_t)end * ba::kTileKeys - 1) -
                                                block_of((int64_t)ctx0[n] + (int64_t)r.begin * ba::kTileKeys) + 1);
      }
    }
  }
  const double tokens = cu_ctx[n_prompts];
  const double mean = std::ceil(walked * h->n_kv_heads / num_cus());
  if (!ba::turn_pays(tokens * h->n_kv_heads * h->head_dim * 2.0, turned / tokens, most_tiles, mean)) return false;
  const int64_t table = (int64_t)(most_tiles + 15) / 16 * 16 * ba::kTileKeys * 4;  // of either table
  const int64_t rots = ((int64_t)most_blocks * h->head_dim * 4 + 1023) / 1024 * 1024;
  if (2 * table + rots > (int64_t)ba::kTurnLds) return false;
  *blk_at = (uint32_t)table;
  *rot_at = (uint32_t)(2 * table);
  return true;
}

}  // namespace

extern "C" {

size_t ba_final_block_attention_cached_workspace_bytes(const ba_heads *heads, int32_t n_prompts,
                                                       const int32_t *cu_q, const int32_t *cu_blk,
                                                       const int32_t *blk_len, int32_t have_k_f_rot_out,
                                                       int32_t gather_below) {
  if (check_heads(heads, true) != BA_OK) return 0;
  BlocksPlan pl;
  if (ba::plan_final_blocks(heads, n_prompts, cu_q, cu_blk, blk_len, have_k_f_rot_out != 0, gather_below, num_cus(), &pl) != BA_OK)
    return 0;
  return pl.total();
}

int32_t ba_final_block_attention_cached(const ba_heads *heads, const ba_tensor *q_f, const ba_tensor *k_cache,
                                        const ba_tensor *v_cache, const ba_tensor *k_f, const ba_tensor *v_f,
                                        const ba_tensor *o_out, const ba_tensor *k_f_rot_out, int32_t n_prompts,
                                        const int32_t *cu_q, const int32_t *cu_blk, const int32_t *blk_tok_off,
                                        const int32_t *blk_len, const int32_t *blk_old_pos0,
                                        const int32_t *blk_new_pos0, const int32_t *q_pos0,
                                        int32_t gather_below, void *ws, size_t ws_bytes, void *stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  int32_t rc;
  if ((rc = check_heads(heads, true))) return rc;
  const int D = heads->head_dim;
  BlocksPlan pl;
  if ((rc = ba::plan_final_blocks(heads, n_prompts, cu_q, cu_blk, blk_len, k_f_rot_out != nullptr, gather_below, num_cus(), &pl)))
    return rc;
  if (n_prompts == 0) return BA_OK;
  if ((rc = check_tensor(q_f, "q_f", false, D, heads->n_q_heads))) return rc;
  if ((rc = check_tensor(k_f, "k_f", false, D, heads->n_kv_heads))) return rc;
  if ((rc = check_tensor(v_f, "v_f", false, D, heads->n_kv_heads))) return rc;
  if ((rc = check_tensor(o_out, "o_out", false, D, heads->n_q_heads))) return rc;
  if (pl.n_blocks > 0) {
    if (!blk_tok_off) return fail(BA_ERR_INVALID_ARG, "blk_tok_off is null");
    for (int b = 0; b < cu_blk[n_prompts]; ++b)
      if (blk_len[b] > 0 && blk_tok_off[b] < 0) return fail(BA_ERR_INVALID_ARG, "block %d: negative cache offset", b);
    if ((rc = check_tensor(k_cache, "k_cache", false, D, heads->n_kv_heads))) return rc;
    if ((rc = check_tensor(v_cache, "v_cache", false, D, heads->n_kv_heads))) return rc;
  }
  if (k_f_rot_out && (rc = check_tensor(k_f_rot_out, "k_f_rot_out", false, D, heads->n_kv_heads))) return rc;
  if (!ws || ws_bytes < pl.total() || ((uintptr_t)ws & 255))
    return fail(BA_ERR_WORKSPACE, "final block (cached): 256-byte aligned workspace of %zu bytes needed, %zu given",
                pl.total(), ws_bytes);

  if (pl.gather) {
    // non-empty blocks in prompt order: where they lie in the cache, where they go, and their positions
    std::vector<int32_t> src, dst, len, oldp, newp, zero;
    for (int n = 0; n < n_prompts; ++n) {
      int32_t at = pl.cu_ctx[n], pos = 0;
      for (int b = cu_blk[n]; b < cu_blk[n + 1]; ++b) {
        if (blk_len[b] == 0) continue;
        src.push_back(blk_tok_off[b]);
        dst.push_back(at);
        len.push_back(blk_len[b]);
        oldp.push_back(blk_old_pos0 ? blk_old_pos0[b] : 0);
        newp.push_back(blk_new_pos0 ? blk_new_pos0[b] : pos);
        at += blk_len[b];
        pos += blk_len[b];
      }
    }
    zero.assign(src.size(), 0);
    ba_tensor kg, vg;
    kg.ptr = ws;
    kg.stride_head = D;
    kg.stride_tok = (int64_t)heads->n_kv_heads * D;
    kg.dtype = BA_DTYPE_BF16;
    vg = kg;
    vg.ptr = (char *)ws + align256(pl.gather_kv_bytes);
    const int nb = (int)src.size();
    // Values need no rotation: where there are enough of them, 32 bits reach every row of the cache and a split's share of
    // the table fits in LDS, only the keys are gathered, next to a table of where each context token's value row lies.  512 blocks of
    // 20 to 60 tokens at 32 over 8 heads of 128: 80 us with the values gathered as well (172 MB through memory, 42 us
    // of it), 62 so; how many are enough: kRowTableBytes.
    FinalPlan fp;
    if ((rc = ba::plan_final(heads, n_prompts, cu_q, pl.cu_ctx.data(), BA_ROPE_APPLY, k_f_rot_out != nullptr, num_cus(), &fp))) return rc;
    const size_t row_b = (size_t)heads->n_kv_heads * D * 2;
    std::vector<int32_t> ctx0(n_prompts);
    int64_t padded = 0, reach = 0;
    for (int n = 0; n < n_prompts; ++n) {
      ctx0[n] = (int32_t)padded;
      padded += (pl.cu_ctx[n + 1] - pl.cu_ctx[n] + ba::kTileKeys - 1) / ba::kTileKeys * ba::kTileKeys;
    }
    for (int b = 0; b < nb; ++b) reach = std::max<int64_t>(reach, (int64_t)src[b] + len[b]);
    const size_t table_at = align256((size_t)padded * row_b);
    const bool rows32 = n_prompts <= ba::kFinMaxPrompts && !heads->xcd_speed && reach * v_cache->stride_tok * 2 < ((int64_t)1 << 32) - 65536;
    const size_t ctx_bytes = (size_t)pl.cu_ctx[n_prompts] * row_b;
    void *const ws_final = (char *)ws + 2 * align256(pl.gather_kv_bytes);
    Gather g;
    memset(&g, 0, sizeof(g));
    g.p.src = k_cache->ptr;
    g.p.dst = kg.ptr;
    g.p.src_st = k_cache->stride_tok;
    g.p.src_sh = k_cache->stride_head;
    g.p.dst_st = kg.stride_tok;
    g.p.dst_sh = kg.stride_head;
    g.p.n_kv_heads = heads->n_kv_heads;
    g.p.head_dim = D;
    g.p.dtype = BA_DTYPE_BF16;
    g.p.layout = heads->rope_layout;
    g.p.mode = BA_REENC_SHIFT;
    g.p.n_layers = 1;
    g.p.row_bytes = (uint32_t)(v_cache->stride_tok * 2);
    g.p.table_end = (int32_t)padded;
    g.ctx0 = ctx0.data();
    const auto padded_rows = [&]() {  // the blocks' places with every prompt on a whole tile
      int at = 0;
      for (int n = 0; n < n_prompts; ++n)
        for (; at < nb && dst[at] < pl.cu_ctx[n + 1]; ++at) dst[at] += ctx0[n] - pl.cu_ctx[n];
    };
    const bool table = rows32 && nb <= ba::kRowTableBlocks && ctx_bytes >= ba::kRowTableBytes && (fp.max_nt + fp.max_nt / (2 * fp.n_splits)) / fp.n_splits + 2 <= ba::kRowTableTiles &&
        table_at + (size_t)padded * 4 <= 2 * align256(pl.gather_kv_bytes);
    // Nothing is copied at all where, with values through the table, the attention kernel can turn the keys as they arrive: one stride for keys and values, so that
    // one table serves both, tables and rotations of a split's blocks in LDS, and nothing written that the walk still reads.
    if (table && nb <= ba::kReencMaxBlocksLarge && (double)ctx_bytes >= ba::kTurnBytes &&
        k_cache->stride_tok == v_cache->stride_tok &&
        2 * align256((size_t)padded * 4) + (size_t)nb * D * 4 + 1024 <= 2 * align256(pl.gather_kv_bytes)) {
      const std::vector<int32_t> close = dst;
      padded_rows();
      g.n_blocks = nb;
      g.src_off = src.data(), g.dst_off = dst.data(), g.len = len.data(), g.pos_old = oldp.data(), g.pos_new = newp.data();
      if (turn_layout(heads, n_prompts, cu_q, pl.cu_ctx.data(), ctx0.data(), dst, fp.n_splits, &g.blk_at, &g.rot_at) &&
          !writes_gathered_rows(g, o_out, heads->n_q_heads, cu_q[0], cu_q[n_prompts]) &&
          !(k_f_rot_out && writes_gathered_rows(g, k_f_rot_out, heads->n_kv_heads, cu_q[0], cu_q[n_prompts]))) {
        g.turn = true;
        g.turned.rows = (uint32_t *)ws;
        g.turned.blk = (uint32_t *)((char *)ws + align256((size_t)padded * 4));
        g.turned.rot = (float *)((char *)ws + 2 * align256((size_t)padded * 4));
        g.turned.row_bytes = g.p.row_bytes;
        g.turned.table_end = (int32_t)padded;
        return final_block(heads, q_f, k_cache, v_cache, k_f, v_f, o_out, k_f_rot_out, n_prompts, cu_q, pl.cu_ctx.data(),
                           q_pos0, BA_ROPE_APPLY, ws_final, pl.gather_final_bytes, stream_, &g);
      }
      dst = close;
    }
    if (!table && (k_cache->stride_tok != v_cache->stride_tok || k_cache->stride_head != v_cache->stride_head)) {
      if ((rc = ba_reencode_positions(heads, k_cache, &kg, 1, 0, 0, nb, src.data(), dst.data(), len.data(), oldp.data(),
                                      newp.data(), BA_REENC_SHIFT, stream_)))
        return rc;
      // (a shift of zero positions is a plain copy)
      if ((rc = ba_reencode_positions(heads, v_cache, &vg, 1, 0, 0, nb, src.data(), dst.data(), len.data(), zero.data(),
                                      zero.data(), BA_REENC_SHIFT, stream_)))
        return rc;
      return ba_final_block_attention(heads, q_f, &kg, &vg, k_f, v_f, o_out, k_f_rot_out, n_prompts, cu_q, pl.cu_ctx.data(), q_pos0,
                                      BA_ROPE_APPLY, ws_final, pl.gather_final_bytes, stream_);
    }
    if (table) {
      padded_rows();
      g.p.copy_from_layer = 0x7fffffff;
      g.p.row_table = (uint32_t *)((char *)ws + table_at);
    } else {
      // One launch for both: the values ride along as a second "layer" of the key cache (the layer
      // strides are the distances between the two tensors) that is copied, not rotated.
      g.p.src_sl = ((const char *)v_cache->ptr - (const char *)k_cache->ptr) / 2;  // in elements
      g.p.dst_sl = (int64_t)(align256(pl.gather_kv_bytes) / 2);
      g.p.n_layers = 2;
      g.p.copy_from_layer = 1;
    }
    // all but the last table-full of blocks in launches ahead of the final block's
    const int ahead = nb > 0 ? (nb - 1) / ba::kReencMaxBlocksLarge * ba::kReencMaxBlocksLarge : 0;
    if (ahead > 0) {
      ba::RopeTable rt;
      build_rope_table(heads, &rt);
      ba::ReencRowsParams p = g.p;
      p.table_end = dst[ahead];
      const ba::ReencParams &plain = p;
      rc = table ? run_reencode(p, rt, ahead, src.data(), dst.data(), len.data(), oldp.data(), newp.data(), stream)
                 : run_reencode(plain, rt, ahead, src.data(), dst.data(), len.data(), oldp.data(), newp.data(), stream);
      if (rc) return rc;
    }
    g.n_blocks = nb - ahead;
    g.src_off = src.data() + ahead, g.dst_off = dst.data() + ahead, g.len = len.data() + ahead;
    g.pos_old = oldp.data() + ahead, g.pos_new = newp.data() + ahead;
    return final_block(heads, q_f, &kg, table ? v_cache : &vg, k_f, v_f, o_out, k_f_rot_out, n_prompts, cu_q, pl.cu_ctx.data(),
                       q_pos0, BA_ROPE_APPLY, ws_final, pl.gather_final_bytes, stream_, &g);
  }

  char *wsp = (char *)ws;
  void *kf_ws = wsp;
  wsp += align256(pl.kf_bytes);
  uint16_t *q_ws = (uint16_t *)wsp;
  wsp += align256(pl.q_bytes);
  float *rot_ws = (float *)wsp;
  wsp += align256(pl.rot_bytes);
  uint16_t *part_o = (uint16_t *)wsp;
  wsp += align256(pl.part_o_bytes);
  float *part_ml = (float *)wsp;
  wsp += align256(pl.part_ml_bytes);
  int32_t *part_idx = (int32_t *)wsp;

  ba::RopeTable rt;
  build_rope_table(heads, &rt);

  ba_tensor kf_use = *k_f;
  if (k_f_rot_out) {
    kf_use = *k_f_rot_out;
  } else {
    kf_use.ptr = kf_ws;
    kf_use.stride_head = D;
    kf_use.stride_tok = (int64_t)heads->n_kv_heads * D;
  }

  const int G = heads->n_q_heads / heads->n_kv_heads;
  ba::AttnParams ap;
  memset(&ap, 0, sizeof(ap));
  ap.q = q_ws;
  ap.q_st = (int64_t)heads->n_q_heads * D;
  ap.q_sh = D;
  ap.kf = (const uint16_t *)kf_use.ptr;
  ap.kf_st = kf_use.stride_tok;
  ap.kf_sh = kf_use.stride_head;
  ap.vf = (const uint16_t *)v_f->ptr;
  ap.vf_st = v_f->stride_tok;
  ap.vf_sh = v_f->stride_head;
  if (pl.n_blocks > 0) {
    ap.kc = (const uint16_t *)k_cache->ptr;
    ap.kc_st = k_cache->stride_tok;
    ap.kc_sh = k_cache->stride_head;
    ap.vc = (const uint16_t *)v_cache->ptr;
    ap.vc_st = v_cache->stride_tok;
    ap.vc_sh = v_cache->stride_head;
  } else {
    ap.kc = ap.kf;
    ap.kc_st = ap.kf_st;
    ap.kc_sh = ap.kf_sh;
    ap.vc = ap.vf;
    ap.vc_st = ap.vf_st;
    ap.vc_sh = ap.vf_sh;
  }
  ap.o = (uint16_t *)o_out->ptr;
  ap.o_st = o_out->stride_tok;
  ap.o_sh = o_out->stride_head;
  ap.part_o = part_o;
  ap.part_ml = part_ml;
  ap.part_idx = part_idx;
  ap.part_units = pl.total_tiles * heads->n_kv_heads * (ba::kTileRows / 32);
  ap.n_q_heads = heads->n_q_heads;
  ap.n_kv_heads = heads->n_kv_heads;
  ap.group = G;
  set_merge_rows(&ap, n_prompts, cu_q, G);
  ap.group_div = ba::make_fast_div((uint32_t)G);
  ap.head_dim = D;
  ap.scale_log2e = scale_log2e(heads);
  ap.q_ready = 1;
  ap.rope_layout = heads->rope_layout;
  ap.blk_rot = rot_ws;
  ap.n_splits = pl.n_splits;

  BlocksCall call{heads, &rt, q_f, q_ws, k_f, &kf_use, rot_ws, n_prompts, cu_q, cu_blk, blk_tok_off, blk_len,
                  blk_old_pos0, blk_new_pos0, q_pos0, stream, pl.max_nt};
  if (n_prompts <= ba::kBlkSmallPrompts && pl.n_blocks <= ba::kBlkSmallBlocks)
    rc = run_final_blocks<ba::FinalBlocksMetaSmall, ba::RopeRotsSmall>(call, ap);
  else
    rc = run_final_blocks<ba::FinalBlocksMeta, ba::RopeRots>(call, ap);
  if (rc) return rc;
  if (pl.n_splits > 1) {
    hipError_t e;
    {
      ProfileScope ps(BA_PROFILE_COMBINE, stream);
      e = ba::launch_combine(ap, stream);
    }
    if (e != hipSuccess) return device_fail(e, "split combine launch");
  }
  return BA_OK;
}

}  // extern "C"

