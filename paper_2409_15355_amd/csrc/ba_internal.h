// Internal interface between the C boundary (ba_api.hip) and the gfx950 kernels.
// Small per-call metadata travels BY VALUE in the kernel-argument segment, so no call
// ever copies host memory to the device or needs device-side scratch for schedules;
// long block lists are cut into several launches by the host code.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ba_schedule.h"

namespace ba {

constexpr int kMaxFreq = 64;  // head_dim / 2 <= 64

// theta_j / (2*pi) as an unsigned Q0.64 fraction of a turn.  position * turns[j]
// (mod 2^64) is then the exact phase of the RoPE angle position * theta_j (Eq. 1).
struct RopeTable {
  uint64_t turns[kMaxFreq];
};

// ---------------------------------------------------------------- re-encode ----------
// Two capacities (the table travels by value in the kernel arguments): retrieval-sized block lists,
// and the long lists of small blocks that a gathered context is made of.
constexpr int kReencMaxBlocks = 96, kReencMaxBlocksLarge = 1024;

template <int NB>
struct ReencBlocksT {
  static constexpr int kBlocks = NB;
  int32_t n;
  int32_t src_off[NB];
  int32_t dst_off[NB];
  int32_t len[NB];
  int32_t pos_old[NB];
  int32_t pos_new[NB];
};
using ReencBlocks = ReencBlocksT<kReencMaxBlocks>;
using ReencBlocksLarge = ReencBlocksT<kReencMaxBlocksLarge>;

struct ReencParams {
  const void *src;
  void *dst;
  int64_t src_st, src_sh, dst_st, dst_sh;  // token / head strides, elements
  int64_t src_sl, dst_sl;                  // layer strides, elements
  int32_t n_layers, n_kv_heads, head_dim;
  int32_t dtype, layout, mode;
  int32_t max_len;  // longest block in this launch
  int32_t heads_per_thread, n_head_groups;  // how the KV heads are split over workgroups
  int32_t copy_from_layer;  // layers from this one on are copied as they are (a gathered V rides along as a layer)
};

// The keys of a gathered context whose values stay where they are (bf16, uniform shift): row_table[destination token] =
// where its value row lies, in bytes (source token * row_bytes); destination tokens between a block's end and the next
// block's start (table_end behind the launch's last block) get the block's last row.
// Kernels of their own: in the others the code for it, never entered, took up to 0.2 us of a launch of 4 to 12 (one layer of
// 40 x 40 tokens, 8 heads of 128, absolute: 4.5 us with it, 4.3 without; 160 x 200, 4 heads of 64, half pairs: 12.5, 12.4).
struct ReencRowsParams : ReencParams {
  uint32_t *row_table;
  uint32_t row_bytes;
  int32_t table_end;
};

// Params = ReencParams or ReencRowsParams, Blocks = ReencBlocks or ReencBlocksLarge
template <typename Params, typename Blocks>
hipError_t launch_reencode(const Params &p, const Blocks &blocks, const RopeTable &rt, hipStream_t stream);

// Final block over a block table: prompts and cached blocks per launch.  Two capacities, because
// the tables travel by value in the kernel arguments and many large argument blocks in flight
// throttle the launch queue: the small one covers retrieval-sized prompts.
constexpr int kBlkMaxPrompts = 64, kBlkMaxBlocks = 1024;
constexpr int kBlkSmallPrompts = 16, kBlkSmallBlocks = 64;

// ---------------------------------------------------------------- RoPE pre-pass ------
// Fresh (un-rotated) Q and K rows of a run of consecutive segments: segment s covers tokens
// [start[s], start[s+1]) and its first token has position pos0[s].
constexpr int kRopeMaxSegs = 320;

// (two capacities: the table travels by value in the kernel arguments, and a final-block call of a
// few prompts should not carry 2.5 KB of it through every launch)
template <int N>
struct RopeSegsT {
  static constexpr int kSegs = N;
  int32_t n;
  int32_t start[N + 1];
  int32_t pos0[N];
};
using RopeSegs = RopeSegsT<kRopeMaxSegs>;
constexpr int kRopeSmallSegs = 8;
using RopeSegsSmall = RopeSegsT<kRopeSmallSegs>;

struct RopePrepassParams {
  const uint16_t *q_src;
  uint16_t *q_dst;
  int64_t q_st, q_sh, qd_st, qd_sh;  // token / head strides, elements
  const uint16_t *k_src;
  uint16_t *k_dst;
  int64_t k_st, k_sh, kd_st, kd_sh;
  float q_scale;  // Q is multiplied by this before its one rounding
  int32_t n_q_heads, n_kv_heads, head_dim, layout;
  int32_t heads_per_thread;
  int32_t do_q, do_k;
  float *rot_dst;    // [n_rot][D/2][2]: (cos, sin) of rot_angle[b] * theta_j, or null
  int32_t n_rot;
  float *q_table;    // do_q == 2: instead of rotating Q rows, write q_scale * (cos, sin) by position: [table_rows][D/2][2]
                     // (for calls all of whose segments start at position 0)
  int32_t table_rows;
  int32_t *zero;     // n_zero words cleared on the way (counters of the attention launch behind this one)
  int32_t n_zero;
};

// positions (in tokens) by which the rows of the rotation table turn
template <int NB>
struct RopeRotsT {
  int32_t angle[NB];
};
using RopeRots = RopeRotsT<kBlkMaxBlocks>;
using RopeRotsSmall = RopeRotsT<kBlkSmallBlocks>;

// A gathered context's re-encoding (bf16, uniform shift, one or two layers) and the pre-pass of the query block's rows
// (rotated q and k; no table of rotations, nothing to clear) in one launch.  Params = ReencParams or ReencRowsParams.
using RopeSegsGather = RopeSegsT<64>;
// ... where one launch takes both; else the caller launches the two passes one after the other
template <typename Params, typename Blocks>
bool gather_takes_prepass(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs);
template <typename Params, typename Blocks>
hipError_t launch_gather_prepass(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                                 const RopeTable &rt, hipStream_t stream);

// rots / rots_small: at most one non-null, and only with p.rot_dst
hipError_t launch_rope_prepass(const RopePrepassParams &p, const RopeSegs &segs, const RopeRots *rots,
                               const RopeRotsSmall *rots_small, const RopeTable &rt, hipStream_t stream);
hipError_t launch_rope_prepass(const RopePrepassParams &p, const RopeSegsSmall &segs, const RopeRots *rots,
                               const RopeRotsSmall *rots_small, const RopeTable &rt, hipStream_t stream);

// ---------------------------------------------------------------- shared by the files of the boundary ----
int32_t device_fail(hipError_t e, const char *what);  // BA_ERR_DEVICE with the runtime's text
int num_cus();                                        // compute units of the current device
unsigned long long *&probe_clock();                   // this thread's AttnParams::wg_clock for the next final-block launches

// ---------------------------------------------------------------- attention ----------

constexpr int kProbeRecord = 16;
constexpr int kTileRows = 256;  // packed (token, head-in-group) query rows per workgroup
constexpr int kTileKeys = 64;   // keys per K/V tile
constexpr int kShortTileRows = 128;  // packed query rows per workgroup of the short-block schedule
constexpr int kBwdTileKeys = 64;     // keys per workgroup of the dk/dv kernel
constexpr int kKvTileRows = 32;      // packed query rows per tile of its walk
// Per-block encoding sends blocks up to this length through the short-block schedule (measured
// crossover: beyond about 6,000 to 8,000 tokens the deep pipeline of the main core wins).
constexpr int kShortMaxLen = 6144;
// The cache in front of HBM.  Query-side rows pass once, between K/V tiles that are read again; where a call's rows
// exceed this cache, they carry the non-temporal hint.  Below, the hint sends them past a cache that would
// have held them (from the kernel before, and for the one behind).  Without / with it, us, and MB of rows:
// per-block encoding, blocks of 200, 32 over 8 heads of 128: 6,000 tokens (123) 39.0 / 43.0, 12,000 (246) 67.6 / 69.4,
// 16,000 (328) 95.2 / 88.6; 16 over 8: 16,000 (197) 61.4 / 64.5, 24,000 (295) 94.4 / 87.7; 8 over 2 of 64: 66,000 (169)
// 61.9 / 65.0.  Forward and backward, prompts of 20 x 200 + 64 tokens, MB in the dq kernel: 16 over 8 of 128: two
// (200) 287 / 289, three (300) 334 / 328; 32 over 8: two (366) 337 / 332; 8 over 2 of 64: eight (183) 239 / 245.
constexpr int64_t kCacheBytes = 256 << 20;
// Per-block encoding with fewer query heads per KV head than this gives the same bits on either schedule, and
// a call takes one by its amount of work (encode_short_max).
constexpr int kSmallGroup = 4;
constexpr int kSmallGroupShortLen = 512;  // no block longer than this: small workgroups
constexpr int kFixedTiles = 4;            // what a workgroup of the main core spends besides its walk, in key tiles
constexpr int kEncodeCus = 256;           // compute units the rule reckons with

// Whole prompts: last blocks that walk more than kShareAbove key tiles have the walk shared by workgroups of
// kShareChunk tiles or more, as many as come to kSharePairs workgroups for the block.  Forward and backward, us,
// unshared / 24 workgroups / 32 / 48: 4 over 4 heads of 64, one prompt of 20 x 161-477 tokens and 41-124 219 / 83 / 78 /
// 76, eight of 20 x 100-300 and 32-128 224 / 141 / 144 / 150; 8 over 2, two of 6 x 370-1105 215 / 155 / 132 / 128; 32 over
// 8 of 128, three of 11 x 117-351 and 13-40 252 / 241 / 223 / 225, two of 21 x 134-396 and 31-94 465 / 465 / 368 / 358.  But
// eight of 20 x 100-300 and 32-128 there, which fill the chip by themselves, 967 / 967 / 972 / 974: hence 24.
// (Sharing does not stop to pay at kShareAbove either: 48 calls of one and two prompts with walks of 18 to 36 tiles take
// 0.74 to 0.94 of the time when theirs are shared too.  It lies above the 35 tiles up to which ba_schedule_prompts
// has always listed one item per row tile.)
// Into how many parts a walk is cut follows from the block's own sizes; whether any is cut, from the call: only if
// the longest of them is kShareLoad or more of what each compute unit has to do.  A launch that fills the chip hides a long walk
// and pays for cutting it (each part loads and turns its query rows again, and K and V are read in a burst): 64
// prompts of 6 x 200 + 20 tokens, 32 over 8 heads of 128, forward kernel 280 -> 316 us, of that 20 without any exchange
// of partial results.  110 calls of 2 to 50 prompts, walk / load and time shared / unshared: 0.26-0.57 0.95-1.05, in the
// mean 1.00; 0.62 1.007, 0.63 0.996 and 0.95, 0.66 1.005, 0.69 0.99, 0.70 1.00 and 1.03, 0.71 0.99, 0.72 0.86, 0.73 0.87,
// 0.74 0.83, 0.75 0.92 and 0.86; beyond, 0.80 in the mean of 69, two of them slower (1.01, 1.07).
// (At head_dim 128 every part beyond a walk's first counts as kSharePartTiles in that: 64 KB of partial results out and in,
// and the forward and dq kernels' times in the call of 64 prompts above, 25 and 12 tiles a part.  Without it 13 prompts
// of 16 x 111 + 124 or 19 x 83 + 97 tokens, 8 over 8 heads, and 24 of 13 x 101 + 45, 8 over 1, were 3, 4 and 6 % slower shared; six
// other calls that it leaves alone, 0.99 to 1.01.  At 64 calls down to 0.65 of the load with as many parts take 0.76 to 0.97 shared.)
// ... and only if the longest of them is longer by 1 / kShareLead than every walk that stays: a last block of
// too many row tiles or a passage as long leaves the launch no shorter.  Thirteen calls where one was as long, 1 to 11
// prompts: 1.02 in the mean, 0.94 to 1.08 (8 over 1 of 128, eight prompts of 650-1520 tokens and 120-260, forward kernel 52 us
// unshared and 59 shared, dq 76 and 91); with a lead of one tile of 37 to 86 0.97 to 1.02, of two to five 0.92 to
// 1.01.  (Calls of hardly any work, a load of less than a quarter of the walk, either way: 1.00 to 1.02.)
// Last blocks of more than kSharePairs / 2 row tiles times KV heads (a query block of 64 tokens at 32 over 8 heads has 16): their
// walks were never cut, and a call of one or two such prompts took as long as one workgroup walks, 0.77 us a tile in the forward
// kernel and 0.85 in the dq kernel (one prompt of 4,400 tokens at 32 over 8 heads of 128: 101 and 111 us, as long as two prompts).  From
// kShareManyAbove + 1 tiles on they are cut into parts of kShareManyChunk tiles (kShareChunk at head_dim 64), at most
// kShareManyPairs workgroups a block, in calls that the rules below let share.  Forward and backward, us, unshared / shared, prompts
// of 20 x 100-300 and 32-128: one 280 / 168, two 336 / 282, at 16 over 8 heads 255 / 120 and 294 / 194; one of 6 x 300-800 and 200-256
// 238 / 183; 8 over 2 of 64, one of 20 x 100-300 and 200-256 191 / 79.  Parts of 16, 20 and 32 tiles: 170, 169 and 170, 285, 281 and 282;
// at 64 79 with 16, 85 with 24, 90 with 32.  At most 96, 128 and 256 workgroups: 238, 186 and 182 where 192 take 183.  60 drawn calls of 1 to 6
// prompts whose walks are as long: 0.48 to 1.01 of the time, 0.85 in the mean.
// Next to a walk that stays and is nearly as long they are not: the launch gets no shorter, and its parts, many and all early, hold up the
// long ones.  Forward kernel, unshared / shared, us, a passage and a query block: 8 over 1 of 128, 5,000 and 900 tokens (longest walk 1.18 of
// the longest that stays) 170 / 238, 6,750 and 250 (1.04) 197 / 258; 14 over 2 of 64, 5,700 and 270 (1.04) 149 / 167; 16 over 8
// of 128, 3,450 and 105 (1.03) 95 / 98.  From 1.23 on 0.55 to 1.01, below 0.79 to 1.40, 1.02 in the mean of 52.  So only if the longest is longer
// by 1 / kShareManyLead, or more than kShareManyAnyway times the load: beyond that 0.86 to 1.00 with any lead.  (The dq kernel, whose
// parts cost more, has kShareAnyway there: 410 us unshared and 426 at 2.1 of the load, 3 over 3 of 128.)
// With more than kSharePairs / 2 KV heads no walk is cut, whatever the block: one row tile of it is too many pairs for the first rule, and
// the second goes no further.  So with 13 KV heads and more a prompt's output, log-sum-exps and dq are the same bits in every
// batch (ba.h says so).  What that costs, prompts of 20 x 200 + 64 tokens, forward and backward, us, as they are / cut: 64 over 16 heads of 64 one
// 89 and 141 / 42 and 104, two 113 and 207 / 71 and 188; 64 over 16 of 128 121 and 226 / 72 and 187, 154 and 349 / 117 and 346; 32 over 32 of
// 128 124 and 205 / 74 and 155, 172 and 333 / 120 and 295; four of any of these nothing.  Up to twelve: 48 over 12 of 128 117 and 215 / 65 and
// 160, 151 and 311 / 100 and 274, four 200 and 529 / 201 and 528.
// The dq kernel pays more for a cut (each part reads its q, dO and o rows again) and gains later: where the longest walk is 0.64 to 1.1 of
// the load, its call took up to 1.15 of the time (8 over 8 heads of 64, ten prompts of 28 x 115 + 268), the forward pass 0.6 to
// 1.0.  So in calls with such blocks it shares from dq_share_load of the load on, and walks of kShareLongWalk tiles and more are cut into parts of
// kShareLongChunk (head_dim 128, groups of four and more, four KV heads and more: the fewer parts are as fast in a prompt alone and
// half the loss among four; 8 over 2 of 128 0.79 -> 0.84, 16 over 8 0.59 -> 0.65).  Backward, shared / unshared, by walk / load (without the parts' own):
// groups of one and two at 128 0.93 1.04, 1.06 1.01, 1.18 1.02, 1.27 0.96, 1.43 0.99, at 64 0.64 1.08, 0.76 1.15, 0.95 1.00, 1.05 1.04, 1.22 0.95;
// of four at 128 0.75 to 1.2 0.99 to 1.04 in parts of 24 and 0.99 to 1.02 in parts of 48, 1.28 0.97, at 64 0.71 1.07, 0.77 1.05, 0.79 0.99, 0.81 1.04,
// 0.85 0.98, 0.90 0.93; of eight 0.45 to 1.0 0.92 to 1.02.  (Four at 128 could begin higher, but a prompt of 20 x 200 + 64 tokens, 0.70 of it
// alone, has the same bits in dq among four, 0.77 of the load.)
constexpr int kShareAbove = 36, kShareChunk = 16, kSharePairs = 24;
constexpr int kShareManyAbove = 55, kShareManyChunk = 24, kShareManyPairs = 192;
constexpr int kShareLongWalk = 96, kShareLongChunk = 48;
constexpr double kShareLoad = 0.64;
constexpr double dq_share_load(int head_dim, int64_t group) {
  if (group >= 8) return kShareLoad;
  if (group >= kSmallGroup) return head_dim == 64 ? 0.8 : 0.7;
  return head_dim == 64 ? 1.1 : 0.86;
}
constexpr double kSharePartTiles = 24.0;  // head_dim 128
constexpr int kShareLead = 100, kShareManyLead = 4;
constexpr double kShareAnyway = 4.0, kShareManyAnyway = 1.5;
constexpr size_t kShareMaxBytes = (size_t)256 << 20;
// ... and the same for the walks of the dk/dv kernel (0.73 us a tile; a key tile's rows are its block's and the last
// block's).  Forward and backward, us, dk/dv unshared / shared: 8 over 2 heads of 64, five prompts of 4 x 700 tokens and a last
// block of 200 244 / 221, two of 16 x 135 + 64 70 / 64; 32 over 8 of 128, two of 4 x 52 + 150 73 / 69, two of 3 x 268 + 144
// 133 / 120, one of 3 x 164 + 4 72 / 65; three of 11 x 234 + 26 256 / 256.  Sharing does not stop to pay at kKvShareAbove:
// 80 calls of one and two prompts with walks of 14 to 21 tiles take 0.88 to 1.00 of the time when theirs are shared too.
// It lies where calls of short passages (100 tokens, a last block of 64) ask for no more workspace than without.
// In calls whose longest such walk is more than kKvShareLoad of what every one of kShareCus compute units has to do
// (a call that fills the chip adds up in one order, whatever else is in the batch), in chunks of half of that.
// Four query heads and more per KV head of 128, where that walk is less than kKvShareLight of that load: only if it is
// kKvShareLead tiles longer than what is left when it is cut (the longest part, the longest walk that stays,
// kKvShareLoad of the load).  The 64 KB of every part, out past the caches and in again, take the time of some ten
// tiles.  52 calls of 1 to 15 prompts, tiles gained and time shared / unshared of forward and backward: below 9 0.96 to
// 1.09, a third of them slower (64 over 8, ten prompts of 4 x 45-135 + 5 tokens 176 / 160 us; 32 over 8, three of 5 x 140-195
// + 12, the dk/dv kernel 37 / 34); from 9 on 0.71 to 0.99, one 1.02.  Smaller groups and head_dim 64 gain below 9 too: 24
// calls, 0.88 to 1.00.
constexpr int kKvShareAbove = 21, kKvShareChunk = 12, kShareCus = 256, kKvShareLead = 9;
constexpr double kKvShareLoad = 0.75, kKvShareLight = 1.5;

struct AttnParams {
  const uint16_t *q;
  int64_t q_st, q_sh;
  const uint16_t *kc;  // context keys / values (final block only; used as given)
  int64_t kc_st, kc_sh;
  const uint16_t *vc;
  int64_t vc_st, vc_sh;
  const uint16_t *kf;  // causal-segment keys / values (already rotated)
  int64_t kf_st, kf_sh;
  const uint16_t *vf;
  int64_t vf_st, vf_sh;
  uint16_t *o;
  int64_t o_st, o_sh;
  // Split partials, per "unit" = the 32 packed rows one wave owns: unit = ((tile_base + row tile) *
  // n_kv_heads + KV head) * 8 + wave.  A split's normalised output stays in the layout the MFMA
  // accumulators have (no transposition on the way out; every wave instruction stores 1 KB of
  // consecutive memory); the merge kernel reads that layout back and writes the rows where they belong.
  uint16_t *part_o;   // [n_splits][part_units][D / 16][64 lanes][8] fp16
  float *part_ml;     // [n_splits][part_units][32][2]  (reference in log2 units, sum of exponentials)
  int32_t *part_idx;  // [part_units][32]  output row (token * n_q_heads + head) of each packed row, -1: none
  // (whole prompts, shared walks: part_o holds the accumulators in 32 bits, part_ml (reference, sum), per wave of
  // (row tile of the launch, KV head); part_idx counts, per the same of a block's first split, who is done)
  int64_t part_units;
  int32_t tile_base;  // row tiles of the call's earlier launches
  int32_t merge_rows;    // merge of the partials: packed rows of the call's only prompt, 0 if it has several
  FastDiv merge_div;     // ... division by a row tile's units
  int32_t merge_sparse;  // ... most units have no rows
  int32_t n_q_heads, n_kv_heads, group, head_dim;
  FastDiv group_div;  // division by `group`
  float scale_log2e;  // softmax scale * log2(e)
  int32_t q_ready;    // q is already rotated and multiplied by scale_log2e (the RoPE pre-pass ran)
  int32_t q_rows_fit32;  // main core, filled at the launch: 32 tokens and a group of heads of q span less than 2^32 bytes
  // else, if non-null: [positions][D/2][2] = scale_log2e * (cos, sin) of the position times theta_j; the kernel rotates q with
  // it.  A row per position, not per token, so that blocks (per-block encoding, where all start at 0) and prompts share
  // them: every XCD reads the rows for its own KV heads, and 2 MB by position stay in its L2 where 17 MB by token (eight prompts,
  // 33,746 tokens, head_dim 128) did not: forward and backward 967 -> 957 us, of that 6 in the two pre-passes that write it.
  const float *q_table;
  int32_t rope_layout;
  const float *blk_rot;  // block table only: [blocks][D/2][2] (cos, sin) of minus each block's shift
  int32_t n_splits;
  int32_t use_cuts;            // split_cut holds unequal shares (see split_tile_range)
  uint32_t split_cut[kMaxCutHeads][33];  // per KV head: cumulative shares of its splits, 1 / 65536 units
  unsigned long long *wg_clock;  // probe only, else null: kProbeRecord numbers per workgroup:
                                 // [0] XCC id, [1] shader cycles and [2] 100 MHz ticks at entry, [4] and [5] the same
                                 // behind the walk, ticks [3] first tile copies issued, [6] first tiles and query
                                 // fragments landed, [7] loop entered, [8] partials' stores issued, [9] complete
  int32_t total_tiles;  // row tiles over all problems of this launch
  FastDiv tiles_div;    // division by total_tiles
  int32_t kv_group;     // main core, filled at the launch: KV heads per group in the order of the work items
  uint32_t xcd_runs;    // main core: which run of work items each XCD takes (work_item_of_workgroup); 0 = in order
  ItemDivs item_divs;   // ... and the divisors of item_coords
  SplitDivs split_divs; // divisions by n_splits and 2 n_splits (main core; filled at the launch)
  float *lse;           // short-block schedule: [tokens][n_q_heads] log-sum-exp of the scaled scores, or null
  int32_t rows_past_cache;  // short-block schedule, dq kernel: the call's rows exceed kCacheBytes
};

constexpr int kEncMaxBlocks = 320;
struct EncodeMeta {
  int32_t n;
  int32_t offs[kEncMaxBlocks + 1];        // token offsets of the blocks
  int32_t tile_start[kEncMaxBlocks + 1];  // first row tile of each block; [n] = all tiles, INT_MAX beyond
};

// Whole prompts (Section 2.4): blocks in any order (the host lists the ones with the longest key
// ranges first), each with its first token, its length and the first key it sees.
struct PromptMeta {
  int32_t n;
  int32_t start[kEncMaxBlocks];
  int32_t len[kEncMaxBlocks];
  int32_t tile_start[kEncMaxBlocks + 1];  // in row tiles of kShortTileRows rows; INT_MAX beyond [n]
  int32_t kstart[kEncMaxBlocks];          // token offset of the first visible key
  int32_t pos0[kEncMaxBlocks];            // position of the first token inside its prompt
  // The first n_split blocks' walks are shared out, each by as many workgroups per row tile and KV head as it has
  // times its row tiles in tile_start (all row tiles of split 0 first, then of split 1 ...)
  int32_t n_split;
};

// ---------------------------------------------------------------- backward of whole prompts ----
struct BwdParams {
  const uint16_t *dout;  // gradient of the output, [T][n_q_heads][D] with these strides
  int64_t do_st, do_sh;
  const uint16_t *o;     // the forward output, [T][n_q_heads][D] with these strides
  int64_t o_st, o_sh;
  const float *lse;      // [T][n_q_heads]: the forward pass's log-sum-exps
  uint16_t *q_rot;       // [T][n_q_heads][D]: q rotated and times scale * log2 e, written by the dq kernel, read by the dk/dv kernel
  float *ld;             // -log-sum-exp / ln 2 and -delta per packed row, written by the dq kernel, read by the dk/dv
                         // kernel: per KV head and block, from 2 * (kvh * T + first token) * ld_group floats on, four
                         // rows of the one and four rows of the other in turn
  int32_t ld_group;      // the group rounded up to a multiple of four (keeps every block's start 16-byte aligned)
  int64_t T;
  uint16_t *dq, *dk, *dv;  // the gradients, with these strides
  int64_t dq_st, dq_sh, dk_st, dk_sh, dv_st, dv_sh;
};

// Owners of keys: blocks in any order, and for a passage the last block of its prompt (whose rows
// see the passage's keys as well).
struct BwdKvMeta {
  int32_t n;
  int32_t start[kEncMaxBlocks];
  int32_t len[kEncMaxBlocks];
  int32_t pos0[kEncMaxBlocks];            // position of the first token inside its prompt
  int32_t tile_start[kEncMaxBlocks + 1];  // in key tiles of kBwdTileKeys keys; INT_MAX beyond [n]
  int32_t fin_start[kEncMaxBlocks];
  int32_t fin_len[kEncMaxBlocks];          // 0: the block is its prompt's last
  // The first n_split blocks' walks are shared out: a block whose first key is seen by w tiles of kKvTileRows packed rows
  // has walk_splits(w, chunk) entries per key tile (all key tiles of split 0 first, then of split 1 ...), of which a key
  // tile takes as many as its own walk wants
  int32_t n_split, chunk;
};

hipError_t launch_bwd_dq(const AttnParams &p, const PromptMeta &meta, const BwdParams &bp, hipStream_t stream);
hipError_t launch_bwd_dkv(const AttnParams &p, const BwdKvMeta &meta, const BwdParams &bp, hipStream_t stream);

constexpr int kFinMaxPrompts = 64;
static_assert(RopeSegsGather::kSegs >= kFinMaxPrompts, "a launch's prompts are segments of its pre-pass");
struct FinalMeta {
  int32_t n;
  int32_t cu_q[kFinMaxPrompts + 1];
  int32_t cu_ctx[kFinMaxPrompts + 1];
  int32_t tile_start[kFinMaxPrompts + 1];
};

// Final block over a context whose keys have been gathered into one place (prompt n's from key row ctx0[n] on, a multiple
// of kTileKeys) and whose value rows are fetched from the cache through a table: byte offset of context token
// t's row at rows[ctx0[n] + t], entries up to the next multiple of kTileKeys holding some row that exists.
constexpr int kRowTableTiles = 112;  // context tiles of one split at most: 16 rows of each per copying wave lie in LDS
// ... for contexts of this many bytes of values at least: a workgroup waits for its part of the table before it asks for
// the first values, 1 to 2 us of a call, and copying a few MB takes less.  200 drawn calls of 1 to 20 prompts, time with
// the table / with copied values: below 1 MB 0.99 to 1.10, in the mean 1.05; 1 to 2.5 MB 1.02; 2.5 to 5 MB 1.01; 5 to 10 0.97; beyond 0.91.
// And of this many blocks at most, eight launches of the gather: beyond, 0.89, 0.96, 1.05 and 1.21 (26,514 blocks).
constexpr size_t kRowTableBytes = (size_t)4 << 20;
constexpr int kRowTableBlocks = 8 * kReencMaxBlocksLarge;
struct FinalGatherMeta : FinalMeta {
  int32_t ctx0[kFinMaxPrompts];
  const uint32_t *rows;
};

// Final block over short cached blocks none of which is copied: keys and values are fetched through the table of rows (one
// stride for both), and the attention kernel turns a tile's keys in LDS by the shift of the block they belong to: blk[] names it
// for every entry of rows[], a row of rot = (cos, sin) of the shift per frequency.  LDS behind the tile buffers: a split's
// part of rows[], from blk_at on its part of blk[], from rot_at on the rotations of its blocks.
// Saved: the keys' way out to memory and back (84 of 168 MB for 20,000 tokens of 8 heads of 128; the gather took 16 us of 54).
// Paid: 2 to 3 us of start-up (table, then first tile and rotations, then the turning of it, one behind the other) and some 0.3 us a key
// tile that a workgroup walks, by every row tile anew.  So only
//   - where a key is turned by kTurnRowTiles row tiles at most, in the mean over the context (each prompt by its share of the tokens);
//   - for contexts of kTurnBytes of keys and kTurnBytesTile more for each of those row tiles;
//   - of kTurnBytesWalk of keys or more for every tile of the longest walk, and of what a compute unit walks in the mean, which is more
//     in several rounds of workgroups.  (With all compute units at work it is head_dim / 32 MiB over the row tiles: at head_dim
//     64 one row tile only, at 128 two where the walks are nearly as long as each other);
//   - where the longest walk is no more than kTurnUneven times the mean (else it ends the launch alone, some 0.55 us a tile longer).
// Copied / turned, us.  32 over 8 heads of 128, blocks of 130, one row tile: 16 MiB 31.0 / 30.8, 22 MiB 35.0 / 33.6, 44 MiB 50.9 / 46.7, 90 MiB
// 91.1 / 74.7; two, 16 MiB 37.0 / 37.7, 22 MiB 43.5 / 43.4, 32 MiB 54.8 / 54.5, 44 MiB 68.2 / 67.2; blocks of 60 to 180 and more, three, 23 MiB 57.7 / 56.9,
// 32 MiB 74.1 / 75.9, 44 MiB 91.2 / 94.4; four, 23 MiB 65.3 / 67.0, 38 MiB 102.9 / 109.2; six, 15 MiB 62.6 / 70.0.  32 over 32 of 64: one, 22 MiB
// 35.9 / 35.4, 90 MiB 98.2 / 87.7; two, 22 MiB 49.8 / 53.6, 44 MiB 82.1 / 87.4.
// Few KV heads, whose splits are 64 at most: 8 over 1 of 128, 22 tiles of 22 MiB, 5.5 in the mean, 50.9 / 58.4; 8 over 2 of 64 46.4 / 50.2; 8 over 2
// of 128, 17 tiles and 8 of 32 MiB, 47.5 / 49.5 and 52.3 / 49.3.  Several prompts: 180 query tokens over 3,000 and 30 over 16,000 (37
// MiB, 32 tiles, 12 in the mean) 65.5 / 74.9; over 4,000 and 16,000 (32 and 14) 66.8 / 75.8; over 6,000 and 16,000 (43 MiB, 32 and 17) 69.7 /
// 75.4; 180 over 7,000 and two of 30 over 9,000 (49 MiB, 24 and 19) 66.4 / 63.1; 60 over 16,000 and 60 over 3,000 (37 MiB, 16 and 9) 57.8 / 52.3; 8 over 1
// of 128, three of 17,000 and two row tiles (49 MiB, 34 and 25) 72.8 / 80.5; 32 over 32 of 64, three of 2,600 and two (31 MiB, 13 and 31: three
// rounds) 84.7 / 90.1.  1,387 drawn calls of 20 to 90 MiB, one and two row tiles: 984 are turned, 0.90 of a copy's time in the mean, 0.63 to 1.06
// (up to 1.05 where both sides copy).  One block of 3,000 among 500 of 30: 59.1 / 34.0.
constexpr double kTurnRowTiles = 2.0, kTurnUneven = 1.8;
constexpr double kTurnBytes = 12 << 20, kTurnBytesTile = 9 << 20, kTurnBytesWalk = 1.5 * (1 << 20);
inline bool turn_pays(double key_bytes, double row_tiles, double longest_walk, double mean_walk) {
  return row_tiles <= kTurnRowTiles && key_bytes >= kTurnBytes + kTurnBytesTile * row_tiles && longest_walk <= kTurnUneven * mean_walk &&
         key_bytes >= kTurnBytesWalk * (longest_walk > mean_walk ? longest_walk : mean_walk);
}
constexpr uint32_t kTurnLds = 32 * 1024;
constexpr uint32_t kTurnPlain = 0x80000000u;  // in blk[]: a shift of zero, the key stays as it is
struct FinalTurnMeta : FinalGatherMeta {
  const uint32_t *blk;
  const float *rot;
  uint32_t blk_at, rot_at;
};
// What the tables are written from: shift of block b = blocks.pos_new[b] - blocks.pos_old[b].
struct TurnTables {
  uint32_t *rows, *blk;
  float *rot;          // [blocks.n][head_dim / 2][2]
  uint32_t row_bytes;  // of the caches
  int32_t table_end;   // as in ReencRowsParams
};

// Final block whose query rows and keys are as the caller gave them: no RoPE pre-pass has run, the kernel turns them itself
// (see attn_kernel).  Every prompt has one row tile and one key tile of its own.
constexpr int kFreshTokens = kTileKeys;
struct FinalFreshMeta : FinalMeta {
  int32_t pos0[kFinMaxPrompts];  // position of a row tile's first token
  RopeTable rt;
};

// Final block over a table of cached blocks (each at the positions it was encoded at).
template <int NP, int NB>
struct FinalBlocksMetaT {
  static constexpr int kPrompts = NP, kBlocks = NB;
  int32_t n;
  int32_t rot_base;            // row of AttnParams::blk_rot that belongs to block 0 of this launch
  int32_t cu_q[NP + 1];
  int32_t cu_blk[NP + 1];      // blocks of prompt n: [cu_blk[n], cu_blk[n+1])
  int32_t ctx_tiles[NP];       // key tiles of prompt n's context
  int32_t tile_start[NP + 1];  // first row tile of each prompt
  int32_t blk_off[NB];         // first cache row of the block
  int32_t blk_len[NB];         // rows (>= 1)
  int32_t blk_tile0[NB];       // first key tile of the block inside its prompt
};
using FinalBlocksMeta = FinalBlocksMetaT<kBlkMaxPrompts, kBlkMaxBlocks>;
using FinalBlocksMetaSmall = FinalBlocksMetaT<kBlkSmallPrompts, kBlkSmallBlocks>;

// Rows of [tokens][heads][chunks * 16 bytes] tensors moved between a caller's tensor with `group`
// query heads per KV head and a packed one with `group_padded` (phantom heads are zero).
struct HeadPadParams {
  void *real;          // [tokens][n_kv_heads * group] rows, strides in elements of `elt` bytes
  int64_t real_st, real_sh;
  void *padded;        // [tokens][n_kv_heads * group_padded] rows
  int64_t padded_st, padded_sh;
  int64_t tokens;
  int32_t n_kv_heads, group, group_padded;
  int32_t chunks;      // 16-byte pieces per row
  int32_t elt;         // bytes per element (strides are in elements)
};
// to_padded: real -> padded (phantoms zeroed); else padded -> real (real heads only)
hipError_t launch_pad_heads(const HeadPadParams &p, bool to_padded, hipStream_t stream);
// the same for [tokens][heads] floats (real: packed [tokens][n_kv_heads * group])
hipError_t launch_pad_lse(float *real, float *padded, int64_t tokens, int n_kv_heads, int group, int group_padded,
                          bool to_padded, hipStream_t stream);

// MFMA rate diagnostic (diag.hip): n_wg workgroups of 8 waves, `iters` x 16 MFMAs each, with
// reads_per_two (0, 1, 2) LDS fragment reads per two MFMAs; per wave (shader cycles, 100 MHz ticks) into ws
size_t diag_mfma_workspace_bytes(int n_wg);
hipError_t launch_mfma_ceiling(int reads_per_two, int n_wg, int iters, void *ws, uint32_t seed, hipStream_t stream);

// n pseudo-random bf16 values (synthetic operands of the XCD speed probe)
hipError_t launch_fill_random_bf16(uint16_t *dst, int64_t n, uint32_t seed, hipStream_t stream);

// Per-block encoding whose query rows and keys are as the caller gave them: no RoPE pre-pass has run, the kernel turns them itself
// and leaves the turned keys in k_out, if that is given.  One round of workgroups at most; the table of a block's positions
// in LDS.  Working it out grows with the block, the pre-pass and its launch, some 4 us of latency, do not: pre-pass / here, 4
// over 4 heads of 64, blocks of 96 tokens 12.4 / 8.8 us, 128 12.5 / 10.0, 160 13.5 / 10.6, 200 12.6 / 11.7, 250 14.2 / 14.6; 32 over 8 of 128,
// 64 12.0 / 9.3, 80 12.4 / 10.6, 100 12.6 / 11.3, 128 12.9 / 12.7.  Blocks of 104 tokens of 128 dimensions, 208 of 64.
constexpr int kEncFreshLds = 52 * 1024;
// Workgroups that a compute unit holds at once, by registers and LDS; none if the table is too large.  Beyond one round every further one
// works its factors out again.  Pre-pass / here, one round and more than one: 32 over 8 of 128, 20 and 40 blocks of 64 15.5 / 13.5 and
// 19.8 / 20.7 us, 8 and 12 of 100 13.8 / 12.3 and 15.6 / 20.1; 4 over 4 of 64, 200 of 32 13.2 / 8.4, 80 of 128 16.1 / 13.3, 80 of 200 19.0 / 25.9.
constexpr int encode_fresh_by_registers(int head_dim) { return head_dim == 128 ? 2 : 4; }  // (a wave a SIMD each; the kernel's launch bounds)
constexpr int encode_fresh_per_cu(int head_dim, int64_t longest) {
  const int64_t table = longest * head_dim * 4, tiles = 6 * 32 * head_dim * 2;  // (three tiles of 32 keys and values)
  if (table > kEncFreshLds) return 0;
  const int64_t by_lds = (160 * 1024) / (tiles + table), by_registers = encode_fresh_by_registers(head_dim);
  return (int)(by_lds < by_registers ? by_lds : by_registers);
}
struct EncodeFreshMeta : EncodeMeta {
  RopeTable rt;
  int32_t table_rows;  // positions of the longest block
  uint16_t *k_out;
  int64_t k_out_st, k_out_sh;
};

hipError_t launch_attn_encode(const AttnParams &p, const EncodeMeta &meta, hipStream_t stream);
// the same for short blocks: meta.tile_start counts row tiles of kShortTileRows rows
hipError_t launch_attn_encode_short(const AttnParams &p, const EncodeMeta &meta, hipStream_t stream);
hipError_t launch_attn_encode_fresh(const AttnParams &p, const EncodeFreshMeta &meta, hipStream_t stream);
hipError_t launch_attn_prompt_short(const AttnParams &p, const PromptMeta &meta, hipStream_t stream);
hipError_t launch_attn_final_blocks(const AttnParams &p, const FinalBlocksMeta &meta, hipStream_t stream);
hipError_t launch_attn_final_blocks(const AttnParams &p, const FinalBlocksMetaSmall &meta, hipStream_t stream);
hipError_t launch_attn_final(const AttnParams &p, const FinalMeta &meta, hipStream_t stream);
hipError_t launch_attn_final_fresh(const AttnParams &p, const FinalFreshMeta &meta, hipStream_t stream);
hipError_t launch_attn_final_gathered(const AttnParams &p, const FinalGatherMeta &meta, hipStream_t stream);
hipError_t launch_attn_final_turned(const AttnParams &p, const FinalTurnMeta &meta, hipStream_t stream);
// the tables of FinalTurnMeta, and the pre-pass of the query block's rows as in launch_gather_prepass
template <typename Blocks>
hipError_t launch_turn_tables(const TurnTables &t, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                              const RopeTable &rt, hipStream_t stream);
// Merge the split-KV partials of all p.part_units units into the bf16 output.
hipError_t launch_combine(const AttnParams &p, hipStream_t stream);

}  // namespace ba
