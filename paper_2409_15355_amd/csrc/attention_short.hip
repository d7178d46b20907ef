// Per-block encoding of SHORT blocks (arXiv 2409.15355, Section 2.1): the same causal attention
// inside every passage block as the main attention core computes, scheduled for key ranges of a
// few hundred tokens, where a work item is over before a deep software pipeline has filled.
//
// Mapping onto the hardware
//   - A workgroup of 4 wavefronts owns 128 packed query rows (row = token * G + head in group) of
//     one KV head of one block; a wave owns 32 of them.  Workgroups are small (48 KB of LDS at
//     head_dim 128) so that three of them share a compute unit: the latencies of one (its query
//     load, its first tiles, its output) are covered by the arithmetic of the others, not by a
//     pipeline inside the workgroup.
//   - K/V tiles of 32 keys go from memory straight into LDS (LDS-direct loads), two tiles ahead.
//     Per tile a wave computes S^T = K Q^T, the exponentials, and O^T += V^T P^T, in that order,
//     with one workgroup barrier per tile.  A wave whose rows all lie before a tile's first key
//     skips that tile's arithmetic.
//   - Rows of q and o pass once, 32 KB per workgroup, between K/V tiles that the block's other row tiles
//     read again: in calls larger than the cache they carry the non-temporal hint (kPast; 160 passages of 100
//     to 300 tokens, 681 MB: 157 -> 151 us; 101 of it remain with no key tiles walked at all).  A tenth fewer
//     vector instructions changed nothing: the stream bounds it, not the issue.
//   - Any group size: a row tile is 32 packed rows to a wave whatever tokens and heads they are.
//   - Arithmetic, operand layouts and rounding are those of the main core; the softmax takes its reference
//     from the first tile and moves it only to avoid overflow.  The main core's tiles are of 64 keys, so
//     its reference and the order of its sums differ and with them the last bits of an output.  Per-block
//     encoding of fewer than four query heads per KV head takes either schedule by the whole call, and a
//     passage's output must not change with its neighbours there: kAsCore gives the main core's numbers,
//     bit for bit as long as no reference has to move.  (Larger groups take the schedule by a block's own
//     length, whole prompts have this one only: they keep the cheaper order.)
#include <atomic>
#include <type_traits>

#include "ba_device.h"
#include "ba_lds.h"

namespace ba {
namespace {

constexpr int kSWaves = kShortTileRows / 32;  // 4
constexpr int kSThreads = kSWaves * 64;
constexpr int kSKeys = 32;   // keys per tile
constexpr int kSBuf = 3;     // tile buffers of each kind
constexpr float kRebaseAbove = 1099511627776.0f;  // 2^40: a tile sum beyond this moves the reference

template <int D>
struct SGeo {
  static constexpr int KCH = D / 16;          // k-steps of the QK contraction
  static constexpr int DT = D / 32;           // 32-row slabs of O^T
  static constexpr int CPR = D / 8;           // 16-byte chunks per row
  static constexpr int ROWB = D * 2;          // bytes per K/V row in LDS
  static constexpr int LPR = 256 / ROWB;      // rows per 256-byte LDS line (1 or 2)
  static constexpr int GPR = ROWB / 64;       // 64-byte granules per row
  static constexpr int TILEB = kSKeys * ROWB;
  static constexpr int RPI = 1024 / ROWB;     // rows filled by one LDS-direct wave instruction
  static constexpr int IPW = kSKeys / RPI / kSWaves;  // such instructions per wave, tile and kind
  static constexpr size_t LDS = (size_t)2 * kSBuf * TILEB;
  static_assert(IPW >= 1, "every wave takes part in a tile copy");
  static_assert(LDS == (size_t)6 * 32 * D * 2 && kSWaves == 4, "as encode_fresh_per_cu has it");
  static_assert((size_t)kSWaves * 32 * ROWB + 16 <= LDS, "the output staging must fit the tile buffers, and a word behind it");
};

// A table with shared walks.  A kernel of its own: the code for them, never entered, was 3.5 us of 202 in a launch of
// 1,134 row tiles of 32 heads of 128, and 0.8 of the 58 us of a small call's two passes.
struct SharedPromptMeta : PromptMeta {
  explicit SharedPromptMeta(const PromptMeta &m) : PromptMeta(m) {}
};

// Meta = EncodeMeta: a block sees its own tokens only (Section 2.1).  Meta = PromptMeta: a block's keys
// start wherever the table says -- at the block itself for a passage, at the first token of the
// prompt for its last block (Section 2.4: the lower-triangular mask with only the last block seeing
// the others); keys and queries then carry positions inside the prompt.
// kAsCore: the numbers of the main core (the reference from the first 64 keys, sums by 64 keys).
// kPast: rows of q and o go past the caches (see kCacheBytes).
template <int D, typename Meta, bool kAsCore, bool kPast>
__global__ __launch_bounds__(kSThreads, (std::is_same<Meta, EncodeFreshMeta>::value ? encode_fresh_by_registers(D) : 3)) void encode_short_kernel(AttnParams p, Meta meta) {
  using G = SGeo<D>;
  constexpr bool kPrompt = std::is_base_of<PromptMeta, Meta>::value, kShared = std::is_same<Meta, SharedPromptMeta>::value;
  constexpr bool kFresh = std::is_same<Meta, EncodeFreshMeta>::value;  // query rows and keys as the caller gave them
  extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
  lds_char *smem = (lds_char *)smem_generic;
  // LDS map: buffer b = bytes [2 b TB, 2 (b + 1) TB): its K tile, then its V tile
  constexpr uint32_t TB = G::TILEB;

  // ---- which work item: consecutive items are the row tiles of one block at one KV head, and
  //      they share its K/V rows.  Workgroup ids are dealt round-robin to the 8 XCDs, so regroup
  //      them such that each XCD (and its L2) gets a contiguous run of items ---------------------
  uint32_t id = blockIdx.x;
  {
    constexpr uint32_t kXcds = 8;
    const uint32_t n_wg = gridDim.x, q = n_wg / kXcds, r = n_wg % kXcds, x = id % kXcds;
    id = x * q + min(x, r) + id / kXcds;
  }
  const uint32_t n_rowtiles = (uint32_t)p.total_tiles;
  const int kvh = (int)fast_div(id, p.tiles_div);
  // (per-block encoding: a block's long row tiles first; whole prompts: the host's order)
  const uint32_t id_lo = id - (uint32_t)kvh * n_rowtiles;
  const int rowtile = kPrompt ? (int)id_lo : (int)(n_rowtiles - 1 - id_lo);
  const int b = find_block(meta.tile_start, rowtile);
  int q_tok0, lq, k_tok0;  // the block's first token, its length, the first key it sees
  int pos0 = 0;            // position of the block's first token
  if constexpr (kPrompt) {
    q_tok0 = meta.start[b];
    lq = meta.len[b];
    k_tok0 = meta.kstart[b];
    pos0 = meta.pos0[b];
  } else {
    q_tok0 = meta.offs[b];
    lq = meta.offs[b + 1] - q_tok0;
    k_tok0 = q_tok0;
  }
  const int dq = q_tok0 - k_tok0;  // the block's first token, counted in keys
  const int lk = dq + lq;          // keys up to the block's end
  int jt = rowtile - meta.tile_start[b];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31;  // query column inside the 32-wide MFMA group
  const int hf = lane >> 5;   // which half of the wave
  const int Gq = p.group;
  const int n_rows = lq * Gq;
  // a block whose walk is shared: which split, of how many
  int split = 0, n_splits = 1;
  if constexpr (kShared) {
    if (b < meta.n_split) {
      const WalkSplit ws = walk_split_of(n_rows, jt, meta.tile_start[b + 1] - meta.tile_start[b]);
      split = ws.split, n_splits = ws.n_splits;
      jt -= split * ws.n_row_tiles;
    }
  }
  const int row0 = jt * kShortTileRows;

  // key tiles of the workgroup (up to its last row's token) and of this wave
  const int last_row = min(n_rows, row0 + kShortTileRows) - 1;
  TileRange walk = {0, (dq + (int)fast_div((uint32_t)last_row, p.group_div)) / kSKeys + 1};
  if (kShared && n_splits > 1) walk = walk_split_range(walk.end, n_splits, split);
  const int t0 = kPrompt ? walk.begin : 0, n_t = walk.end;
  const int wave_row0 = row0 + wave * 32;
  const int wave_last_row = min(n_rows, wave_row0 + 32) - 1;
  const int wave_n_t =
      wave_last_row >= wave_row0 ? (dq + (int)fast_div((uint32_t)wave_last_row, p.group_div)) / kSKeys + 1 : 0;
  const int first_tok_wave = (int)fast_div((uint32_t)wave_row0, p.group_div);
  const int first_key_wave = dq + first_tok_wave;  // the key that is the wave's first token

  const int my_row = wave_row0 + col;
  const int my_tok = (int)fast_div((uint32_t)my_row, p.group_div);
  const int my_key = dq + my_tok;  // the key that is this lane's token: the last one it sees

  // ---- Q rows (B operand of S^T = K Q^T) and, if they are to be rotated, the rows of the pre-pass's
  //      table of scale * log2(e) * (cos, sin) for this wave's tokens: requested first and all at
  //      once, so that the set-up below runs under their latency.  Both arrive as whole rows (a
  //      lane fetching only its own 16 bytes of a row would cost a cache line each); the Q rows are
  //      then turned into the fragment layout (lane = row) through this wave's slice of LDS ---------
  // (rows beyond the block's take its last row: finite numbers that are never stored)
  constexpr int QRPI = 64 / G::CPR;  // Q rows per load instruction
  static_assert(32 / QRPI == G::KCH, "as many row loads as fragments");
  u32x4_t ld[G::KCH];
  constexpr uint32_t TROW = D * 4;    // bytes of a table row
  constexpr int TCH = TROW / 16;      // its 16-byte chunks
  constexpr int kTabOps = 8 * TROW / 1024;  // LDS-direct loads per wave for 8 table rows
  static_assert(kSBuf == 3, "tile buffers 0 and 1 take the first tiles, 2 the waves' slices");
  static_assert(kSWaves * 8 * TROW <= 2 * TB, "the table slices fit one tile buffer");
  static_assert(kSWaves * 16 * G::ROWB <= 2 * TB, "the Q slices (16 rows at a time) fit one tile buffer");
  static_assert(16 * G::ROWB == 8 * TROW, "one slice serves both uses");
  const uint32_t tab_ofs = 2 * (2 * TB) + wave * (8 * TROW);  // first the table rows ...
  const uint32_t q_ofs = tab_ofs;                              // ... then, once those are in registers, Q rows
  int tab_tl = 0;  // this lane's row of the table slice
  // Whole rows move QRPI at a time: this lane's row in step u is wave_row0 + u * QRPI + lane / CPR and
  // its piece chunk lane % CPR.  Its element offset tok * st + g * sh (relative to the block's first
  // token and the group's first head; 32 bits by the host's check) is carried from step to step:
  // QRPI rows on is QRPI / G tokens and QRPI % G heads on, the latter perhaps past the group's last head
  // and into one more token.
  // (worked out afresh by each of the two walks, load and store: kept, the row numbers would occupy
  // registers all through the tile loop)
  auto walk_rows = [&](int ln, uint32_t st, uint32_t sh, auto &&visit) __attribute__((always_inline)) {
    const int wr_r0 = wave_row0 + ln / G::CPR;
    const int wr_tok0 = (int)fast_div((uint32_t)wr_r0, p.group_div);
    const int wr_g0 = wr_r0 - wr_tok0 * Gq;
    uint32_t off = (uint32_t)wr_tok0 * st + (uint32_t)wr_g0 * sh;
    int g = wr_g0;
    const int step_tok = (int)fast_div((uint32_t)QRPI, p.group_div), step_g = QRPI - step_tok * Gq;
    const uint32_t d_in = (uint32_t)step_tok * st + (uint32_t)step_g * sh, d_wrap = d_in + st - (uint32_t)Gq * sh;
#pragma unroll
    for (int u = 0; u < G::KCH; ++u) {
      visit(u, off, wr_r0);
      g += step_g;
      const bool wrap = g >= Gq;
      g = wrap ? g - Gq : g;
      off += wrap ? d_wrap : d_in;
    }
  };
  {
    const char *qbase = (const char *)(p.q + (int64_t)q_tok0 * p.q_st + (int64_t)(kvh * Gq) * p.q_sh);
    const uint32_t q_st = (uint32_t)p.q_st, q_sh = (uint32_t)p.q_sh;
    const uint32_t last_off = (uint32_t)(lq - 1) * q_st + (uint32_t)(Gq - 1) * q_sh;  // the block's last row
    walk_rows(lane, q_st, q_sh, [&](int u, uint32_t off, int wr_r0) __attribute__((always_inline)) {
      const uint32_t o = wr_r0 < n_rows - u * QRPI ? off : last_off;
      ld[u] = load_row_piece<kPast>(qbase + (o * 2u + (uint32_t)(lane % G::CPR) * 16u));
    });
    if (!kFresh && p.q_table && Gq >= 4) {
      // The rows of a wave span at most 8 tokens.  Chunk c of token row t sits at chunk c ^ (t & 7),
      // which keeps the reads of different tokens off each other's banks.
      const char *tbase = (const char *)(p.q_table + (int64_t)pos0 * D);
#pragma unroll
      for (int u = 0; u < kTabOps; ++u) {
        const int t = u * (1024 / TROW) + lane / TCH, pc = lane % TCH;
        const uint32_t tok = (uint32_t)min(first_tok_wave + t, lq - 1);
        lds_dma16(tbase, tok * TROW + (uint32_t)((pc ^ (t & 7)) << 4), (uint32_t)(uintptr_t)smem + tab_ofs + u * 1024);
      }
      const int ld_tok = (int)fast_div((uint32_t)min(my_row, n_rows - 1), p.group_div);
      tab_tl = max(ld_tok - first_tok_wave, 0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- per-lane LDS read offsets inside a tile buffer (same swizzles as the tile fill below) ----
  uint32_t k_rd[G::KCH];  // K fragment: row `col`, chunk 2 kk + hf
  {
    const int swz = (col / G::LPR) & (G::CPR - 1);
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk) k_rd[kk] = col * G::ROWB + (((kk * 2 + hf) ^ swz) << 4);
  }
  uint32_t v_rd[G::DT];  // V^T fragment (16-key step 0, low half)
  {
    const int vrow = hf * 4 + ((lane & 15) >> 2);
    const int vwithin = ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    const int swz = (vrow / G::LPR) & (G::GPR - 1);
#pragma unroll
    for (int dt = 0; dt < G::DT; ++dt) v_rd[dt] = vrow * G::ROWB + ((dt ^ swz) << 6) + vwithin;
  }

  // ---- tile fill: one wave instruction fills 1024 contiguous LDS bytes, lane i writing
  //      [16 i, 16 i + 16); the swizzle is applied on the global side.  Rows at or beyond a tile's
  //      valid count re-read its last valid row: their scores are masked, and a finite duplicate
  //      keeps 0 * v equal to 0 ------------------------------------------------------------------
  const char *k_base = (const char *)(p.kf + (int64_t)k_tok0 * p.kf_st + (int64_t)kvh * p.kf_sh);
  const char *v_base = (const char *)(p.vf + (int64_t)k_tok0 * p.vf_st + (int64_t)kvh * p.vf_sh);
  const uint32_t k_rb = (uint32_t)p.kf_st * 2u, v_rb = (uint32_t)p.vf_st * 2u;  // row strides, bytes
  int c_row[G::IPW];
  uint32_t c_kchunk[G::IPW], c_vchunk[G::IPW];
#pragma unroll
  for (int u = 0; u < G::IPW; ++u) {
    const int row = (wave * G::IPW + u) * G::RPI + lane / G::CPR, pos = lane % G::CPR;
    c_row[u] = row;
    c_kchunk[u] = (uint32_t)(pos ^ ((row / G::LPR) & (G::CPR - 1))) << 4;
    c_vchunk[u] = (uint32_t)((((pos >> 2) ^ ((row / G::LPR) & (G::GPR - 1))) << 2) | (pos & 3)) << 4;
  }
  const uint32_t lds_copy = (uint32_t)(uintptr_t)smem + wave * G::IPW * 1024;
  auto issue_copy = [&](int t, int buf) __attribute__((always_inline)) {
    const int valid = min(kSKeys, lk - t * kSKeys);
    const char *kp = k_base + (uint64_t)(uint32_t)(t * kSKeys) * (uint64_t)k_rb;
    const char *vp = v_base + (uint64_t)(uint32_t)(t * kSKeys) * (uint64_t)v_rb;
#pragma unroll
    for (int u = 0; u < G::IPW; ++u) {
      const uint32_t row = (uint32_t)min(c_row[u], valid - 1);
      lds_dma16(kp, row * k_rb + c_kchunk[u], lds_copy + (uint32_t)buf * (2 * TB) + u * 1024);
      lds_dma16(vp, row * v_rb + c_vchunk[u], lds_copy + (uint32_t)buf * (2 * TB) + TB + u * 1024);
    }
  };
  // ---- rows that no pre-pass has turned (small calls: one round of workgroups at most).  (cos, sin) of the block's positions are
  //      worked out into the LDS behind the tile buffers while the query rows and the first tiles are on their way; a wave turns
  //      the rows of a key tile that it has copied itself, before the barrier that publishes the tile, and in the block's last row tile, which
  //      walks all of them, leaves them in k_out as well.  The products are the pre-pass's: the same bits.  Bound by latency, the pre-pass's
  //      launch saved: two blocks of 128 tokens, 4 over 4 heads of 64, 12.5 -> 10.0 us, one of 32 12.5 -> 6.1 -------------------
  constexpr uint32_t FRESH = (uint32_t)G::LDS;
  typedef __attribute__((address_space(3))) f32x2_t lds_f32x2;
  typedef __attribute__((address_space(3))) f32x4_t lds_f32x4;
  typedef __attribute__((address_space(3))) u32x4_t lds_u32x4;
  // pairs 2 i and 2 i + 1 of position t are 16-byte piece i of its row
  auto piece = [&](int t, int i) __attribute__((always_inline)) { return FRESH + (uint32_t)t * TROW + ((uint32_t)(i ^ (t & 7)) << 4); };
  const int last_tok = (int)fast_div((uint32_t)last_row, p.group_div);  // the positions wanted: up to the last row's
  auto turn_tile = [&](int t, int buf) __attribute__((always_inline)) {
    if constexpr (kFresh) {
      constexpr int HC = G::CPR / 2, ROWS = kSKeys / kSWaves;  // a wave's rows
      static_assert(ROWS * HC <= 64, "one step of the wave");
      const bool halves = p.rope_layout != 0;
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const int c = ln % HC, row = wave * ROWS + ln / HC;
      if (ln / HC < ROWS) {
        const uint32_t at = (uint32_t)buf * (2 * TB) + (uint32_t)row * G::ROWB + (uint32_t)((c ^ ((row / G::LPR) & (G::CPR - 1))) << 4);
        const u32x4_t xa = *(const lds_u32x4 *)(smem + at), xb = *(const lds_u32x4 *)(smem + (at ^ (HC << 4)));
        const int tok = min(t * kSKeys + row, last_tok);  // (rows behind it are masked)
        f32x4_t ct[4];
#pragma unroll
        for (int h = 0; h < 4; ++h)
          ct[h] = *(const lds_f32x4 *)(smem + piece(tok, halves ? c * 4 + h : (h < 2 ? c * 2 + h : (c + HC) * 2 + h - 2)));
        u32x4_t ya, yb;
        turn_chunks(xa, xb, ct, halves, ya, yb);
        *(lds_u32x4 *)(smem + at) = ya;
        *(lds_u32x4 *)(smem + (at ^ (HC << 4))) = yb;
        if (meta.k_out && last_row == n_rows - 1 && t * kSKeys + row < lq) {
          uint16_t *out = meta.k_out + (int64_t)(q_tok0 + t * kSKeys + row) * meta.k_out_st + (int64_t)kvh * meta.k_out_sh + c * 8;
          *reinterpret_cast<u32x4_t *>(out) = ya;
          *reinterpret_cast<u32x4_t *>(out + HC * 8) = yb;
        }
      }
      lds_wait();  // (published by the next barrier)
    }
  };
  constexpr int kOpsPerTile = 2 * G::IPW;  // vector-memory operations of one wave per tile
  if (!kPrompt || t0 < n_t) issue_copy(t0, 0);  // (buffer 2 holds the waves' slices until the first barrier)
  if (t0 + 1 < n_t) issue_copy(t0 + 1, 1);
  __builtin_amdgcn_sched_barrier(0);  // the copies go out before anything waits for the Q rows
  if constexpr (kFresh) {
    static_assert(kSThreads % (D / 2) == 0, "a thread keeps its frequency");
    const int j = (int)threadIdx.x % (D / 2);
    const uint64_t turns = meta.rt.turns[j];
    for (int t = (int)threadIdx.x / (D / 2); t <= last_tok; t += kSThreads / (D / 2)) {
      float c, sn;
      sincos_phase(rope_phase(t, turns), c, sn);
      *(lds_f32x2 *)(smem + piece(t, j >> 1) + (j & 1) * 8) = f32x2_t{c, sn};
    }
  }

  // ---- rotate (or just scale) the Q rows into the fragments ---------------------------------------
  dma_wait<0>();  // the table rows and the first tile (this wave's share) have landed
  // the table first
  f32x4_t cs[2 * G::KCH];
  if constexpr (kFresh) {
    lds_wait();
    wg_barrier();  // the table is whole (and every wave's share of the first two tiles has landed)
    turn_tile(0, 0);
    if (1 < n_t) turn_tile(1, 1);
    const int tok = (int)fast_div((uint32_t)min(my_row, n_rows - 1), p.group_div);
    const int t_q = min(tok, last_tok);
#pragma unroll
    for (int j = 0; j < 2 * G::KCH; ++j) {
      cs[j] = *(const lds_f32x4 *)(smem + piece(t_q, fragment_table_piece(j, hf, p.rope_layout != 0)));
#pragma unroll
      for (int e = 0; e < 4; ++e) cs[j][e] *= p.scale_log2e;
    }
  } else if (p.q_table && Gq < 4) {
    // Fewer heads than that share a token's row of the table, down to one: hardly any of it would be read
    // twice, so every lane takes its pieces from where they lie.
    const int tok = (int)fast_div((uint32_t)min(my_row, n_rows - 1), p.group_div);
    const f32x4_t *row = reinterpret_cast<const f32x4_t *>(p.q_table + (int64_t)(pos0 + tok) * D);
#pragma unroll
    for (int j = 0; j < 2 * G::KCH; ++j) cs[j] = row[fragment_table_piece(j, hf, p.rope_layout != 0)];
  } else if (p.q_table) {
    const bool halves = p.rope_layout != 0;
#pragma unroll
    for (int j = 0; j < 2 * G::KCH; ++j) {
      const int c = fragment_table_piece(j, hf, halves);
      cs[j] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4_t *>(
          smem + tab_ofs + (uint32_t)(tab_tl * TROW + ((c ^ (tab_tl & 7)) << 4)));
    }
  }
  // whole rows -> fragments: 16 rows at a time through the slice (LDS serves a wave's accesses in
  // order, so the slice needs no barrier); every lane reads the chunks of row `col mod 16` in both
  // passes and keeps those of the pass its row was in
  u32x4_t raw[G::KCH];
  {
    u32x4_t got[2][G::KCH];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
      for (int u = 0; u < G::KCH / 2; ++u) {
        const int rp = u * QRPI + lane / G::CPR, c = lane % G::CPR;
        *reinterpret_cast<__attribute__((address_space(3))) u32x4_t *>(
            smem + q_ofs + rp * G::ROWB + ((c ^ (rp & (G::CPR - 1))) << 4)) = ld[pass * (G::KCH / 2) + u];
      }
      const int rp = col & 15;
#pragma unroll
      for (int kk = 0; kk < G::KCH; ++kk)
        got[pass][kk] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4_t *>(
            smem + q_ofs + rp * G::ROWB + (((kk * 2 + hf) ^ (rp & (G::CPR - 1))) << 4));
    }
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e) raw[kk][e] = (col >> 4) ? got[1][kk][e] : got[0][kk][e];
  }
  bf16x8_t qf[G::KCH];
  if (kFresh || p.q_table) {
    rotate_fragments<G::KCH, kAsCore>(raw, cs, p.rope_layout != 0);
  } else if (!p.q_ready) {
    const float c2 = p.scale_log2e;
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e) raw[kk][e] = pack_bf16(bf16_lo(raw[kk][e]) * c2, bf16_hi(raw[kk][e]) * c2);
  }
#pragma unroll
  for (int kk = 0; kk < G::KCH; ++kk) {
    asm volatile("" : "+v"(raw[kk]));  // the loads are waited for here, not inside the loop
    qf[kk] = __builtin_bit_cast(bf16x8_t, raw[kk]);
  }

  // ---- running state -----------------------------------------------------------------------------
  f32x16_t oacc[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[dt][v] = 0.f;
  float mb = 0.f;     // the row's reference, log2 units
  float l_run = 0.f;  // this lane's share of the running sum of exponentials
  float s0 = 0.f, s1 = 0.f;  // the tile's two partial sums

  // Fragments of a tile on their way from LDS: a rolling window of four per product (the compiler's own order is two,
  // a wait, two more), two of V^T asked for ahead of the exponentials (the variant with the main core's numbers
  // has no registers for that).  Small forward and backward calls 0.95 to 0.99 of the time, at head_dim 64 the forward kernel
  // of 300 passages of 40 to 160 tokens, 16 over 2 heads, 118 -> 110 us; six of K and none of V^T ahead gain half of
  // that.  160 passages at 128, bound by their rows, 143 us with and without.
  constexpr int kKWin = G::KCH < 4 ? G::KCH : 4, kVWin = 4, kVAhead = kAsCore ? 0 : 2;
  auto row_max = [&](const f32x16_t &s) __attribute__((always_inline)) {
    float m0 = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m0 = fmaxf(m0, s[v]);
    return fmaxf(m0, other_half(m0));
  };
  // P = 2^S' rounded to bf16 (the B operand of PV), added up in fp32 on top of s0 and s1
  auto exponentials = [&](const f32x16_t &s, bf16x8_t (&pf)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      u32x4_t w;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p0 = __builtin_amdgcn_exp2f(s[e * 8 + 2 * i]);
        const float p1 = __builtin_amdgcn_exp2f(s[e * 8 + 2 * i + 1]);
        s0 += p0;
        s1 += p1;
        w[i] = pack_bf16(p0, p1);
      }
      pf[e] = __builtin_bit_cast(bf16x8_t, w);
    }
  };
  // K Q'^T of the tile at kofs on top of `start`, keys this lane's row does not see at -infinity (diagonal
  // and ragged tiles only; all branches are wave-uniform)
  auto scores = [&](int i, uint32_t kofs, float start) __attribute__((always_inline)) {
    f32x16_t sacc;
#pragma unroll
    for (int v = 0; v < 16; ++v) sacc[v] = start;
    auto k_frag = [&](int kk) __attribute__((always_inline)) {
      return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t *>(smem + (k_rd[kk] + kofs));
    };
    bf16x8_t fr[kKWin];
#pragma unroll
    for (int kk = 0; kk < kKWin; ++kk) fr[kk] = k_frag(kk);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk) {
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk % kKWin], qf[kk], sacc, 0, 0, 0);
      if (kk + kKWin < G::KCH) fr[kk % kKWin] = k_frag(kk + kKWin);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int key0 = i * kSKeys;
    const int valid = min(kSKeys, lk - key0);
    if (key0 + kSKeys - 1 > first_key_wave || valid < kSKeys) {
      const int lim = min(my_key - key0 + 1, valid);  // visible keys in this tile
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = (v >> 2) * 8 + hf * 4 + (v & 3);
        if (key >= lim) sacc[v] = -INFINITY;
      }
    }
    return sacc;
  };

  if (kAsCore) {
    // The main core's first tile is this schedule's first two (both have been waited for above): the second
    // one's row maximum is wanted ahead of the first one's exponentials.  Its scores are worked out once more
    // when its turn comes (kept, they would not fit next to the accumulators): 16,384 tokens of 16 over 8
    // heads of 128 in blocks of 128 take 60.7 us so, 59.7 with a reference of this schedule's own, 75.8 in the
    // main core; 4 over 4 of 64, 33,000 tokens in blocks of 200: 34.1, 33.5, 49.6.
    mb = -INFINITY;
    if (n_t > 1) wg_barrier();
    if (wave_n_t > 1) mb = row_max(scores(1, 2 * TB, 0.f));
  }

  // ---- the walk over the key tiles: tile i lives in buffer i % 3.  The barrier at the head of
  //      iteration i says two things: every wave's share of tile i has landed, and every wave is
  //      done with tile i-1 (at i = 0: with its slice of buffer 2), so the copy of tile i+2 may
  //      overwrite that buffer ------------------------------------------------------------------------
  int buf = 0;
#pragma unroll 1
  for (int i = t0; i < n_t; ++i) {
    if (i + 1 < n_t) dma_wait<kOpsPerTile>(); else dma_wait<0>();  // tile i + 1 may still be on its way
    if (kFresh && i >= 2) turn_tile(i, buf);
    wg_barrier();
    if (i + 2 < n_t) issue_copy(i + 2, buf == 0 ? 2 : buf - 1);
    if (i < wave_n_t) {
      const uint32_t kofs = (uint32_t)buf * (2 * TB), vofs = kofs + TB;
      // S'^T = K Q'^T - reference: the accumulator starts at minus the row's reference, so the MFMA
      // result is directly the base-2 exponent (as the main core: from the second tile of 64 keys on)
      f32x16_t sacc = scores(i, kofs, kAsCore && i < 2 ? 0.f : -mb);
      if (i == t0) {
        // the first tile sets the reference: its row maximum whatever the sign (nothing visible:
        // stay at 0), so a row's largest exponential so far is exactly 1
        const float mx = kAsCore ? fmaxf(mb, row_max(sacc)) : row_max(sacc);
        mb = mx == -INFINITY ? 0.f : mx;
      }
      if (i < (kAsCore ? 2 : t0 + 1)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) sacc[v] -= mb;
      }
      auto v_frag = [&](int st) __attribute__((always_inline)) {
        typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;
        typedef short s16x8_t __attribute__((ext_vector_type(8)));
        const int kc = st / G::DT, dt = st % G::DT;
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(smem + (v_rd[dt] + vofs) + kc * 16 * G::ROWB));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(smem + (v_rd[dt] + vofs) + (kc * 16 + 8) * G::ROWB));
        const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8_t, both);
      };
      bf16x8_t vf[kVWin];
#pragma unroll
      for (int st = 0; st < kVAhead; ++st) vf[st] = v_frag(st);
      __builtin_amdgcn_sched_barrier(0);
      bf16x8_t pf[2];
      // what the tile's sums start at: nothing, or (as the main core) the first half of a tile of 64 keys
      const float c0 = kAsCore && (i & 1) ? s0 : 0.f, c1 = kAsCore && (i & 1) ? s1 : 0.f;
      s0 = c0;
      s1 = c1;
      exponentials(sacc, pf);
      if (__builtin_amdgcn_ballot_w64(!(s0 + s1 < kRebaseAbove)) != 0) {  // overflow guard: practically never
        asm volatile("" ::: "memory");
        const float shift = fmaxf(row_max(sacc), 0.f);  // only ever raise the reference here
        const float alpha = __builtin_amdgcn_exp2f(-shift);
        mb += shift;
#pragma unroll
        for (int v = 0; v < 16; ++v) sacc[v] -= shift;
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
        s0 = c0 * alpha;
        s1 = c1 * alpha;
        exponentials(sacc, pf);
      }
      if (!kAsCore || (i & 1) || i + 1 == wave_n_t) l_run += s0 + s1;
      // O^T += V^T P^T
#pragma unroll
      for (int st = kVAhead; st < kVWin; ++st) vf[st] = v_frag(st);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < 2 * G::DT; ++st) {
        oacc[st % G::DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[st % kVWin], pf[st / G::DT], oacc[st % G::DT], 0, 0, 0);
        if (st + kVWin < 2 * G::DT) vf[st % kVWin] = v_frag(st + kVWin);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    buf = buf == kSBuf - 1 ? 0 : buf + 1;
  }

  // ---- epilogue: normalise, round once to bf16, and transpose each wave's O^T through its own
  //      slice of LDS so that rows leave as contiguous lines.  The slices lie in the tile buffers:
  //      every wave must be done with the last tile first -----------------------------------------
  // (all of this wave's LDS reads were consumed by its MFMAs, so only the barrier is needed)
  wg_barrier();
  // (lane-dependent addresses are worked out from here on, not carried through the loop in registers)
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int ecol = ln & 31, ehf = ln >> 5;
  lds_char *stage = smem + wave * (32 * G::ROWB);
  float l_tot = l_run + other_half(l_run);
  if constexpr (kShared) {
    // The walk of this row tile is shared: a last block walks its whole prompt, 0.58 us a tile, and a call of a few
    // prompts ends with that chain.  One block of 19 tokens behind 5,000: 157 tiles, 92 us of a launch whose
    // passages take 35.  Leave (accumulators, reference, sum); the last workgroup to do so merges: rows of
    // reference m_i and sum l_i come to sum_i 2^(m_i - m) o_i over sum_i 2^(m_i - m) l_i, m = max m_i.
    int bs = b;
    asm volatile("" : "+s"(bs));  // (its split is looked up anew: held over the loop it costs the loop its scalar registers)
    if (bs < meta.n_split) {
      const int first = meta.tile_start[bs];
      const WalkSplit ws = walk_split_of(n_rows, rowtile - first, meta.tile_start[bs + 1] - first);
      const int tile0 = rowtile - ws.split * ws.n_row_tiles;                                   // of split 0
      const int64_t slot = ((int64_t)tile0 * p.n_kv_heads + kvh) * kSplitWaves + wave;         // of split 0
      const int64_t step = (int64_t)ws.n_row_tiles * p.n_kv_heads * kSplitWaves;               // to the next
      float *const part_o = (float *)p.part_o;
      char *const part_ml = (char *)p.part_ml;
      const bool live = wave_row0 < n_rows;
      if (live) {
        leave_accumulators<D>(part_o, slot + ws.split * step, ln, oacc);
        if (ehf == 0) {
          const u32x2_t ml = {__float_as_uint(l_tot > 0.f ? mb : -INFINITY), __float_as_uint(l_tot)};
          __builtin_amdgcn_raw_buffer_store_b64(ml, shared_buffer(part_ml + (slot + ws.split * step) * 256, 256), ecol * 8, 0, kAgentScope);
        }
      }
      if (!last_of_splits(p.part_idx + (int64_t)tile0 * p.n_kv_heads + kvh, ws.n_splits, smem + G::LDS - 16)) return;
      if (live) {
        mb = -INFINITY;
        l_tot = 0.f;
#pragma unroll
        for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[dt][v] = 0.f;
#pragma unroll 1
        for (int s = 0; s < ws.n_splits; ++s) {
          u32x4_t w[D / 8];
          const u32x2_t ml = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(
              shared_buffer(part_ml + (slot + s * step) * 256, 256), ecol * 8, 0, kAgentScope));
          fetch_accumulators<D>(part_o, slot + s * step, ln, w);
          const float ms = __uint_as_float(ml[0]);
          const float to = fmaxf(mb, ms);
          const float keep = mb == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mb - to);
          const float add = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - to);
          mb = to;
          l_tot = l_tot * keep + __uint_as_float(ml[1]) * add;
#pragma unroll
          for (int k = 0; k < D / 8; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float &o = *((float *)&oacc[k >> 2] + (k & 3) * 4 + e);
              o = o * keep + __uint_as_float(w[k][e]) * add;
            }
        }
      }
    }
  }
  const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      // dims dt * 32 + q4 * 8 + hf * 4 + (0..3) of query row `col`
      const int col = ecol, hf = ehf;
      const int chunk = dt * 4 + q4;
      u32x2_t w;
      w[0] = pack_bf16(oacc[dt][q4 * 4 + 0] * inv, oacc[dt][q4 * 4 + 1] * inv);
      w[1] = pack_bf16(oacc[dt][q4 * 4 + 2] * inv, oacc[dt][q4 * 4 + 3] * inv);
      *reinterpret_cast<__attribute__((address_space(3))) u32x2_t *>(
          stage + col * G::ROWB + ((chunk ^ (col & (G::CPR - 1))) << 4) + hf * 8) = w;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  {
    // (all the pieces are read back before the first store, so that the stores do not each wait
    // for their own read)
    u32x4_t w[G::KCH];
#pragma unroll
    for (int u = 0; u < G::KCH; ++u) {
      const int rr = u * QRPI + ln / G::CPR;  // row inside this wave's 32
      const int ch = ln % G::CPR;
      w[u] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4_t *>(
          stage + rr * G::ROWB + ((ch ^ (rr & (G::CPR - 1))) << 4));
    }
    char *obase = (char *)(p.o + (int64_t)q_tok0 * p.o_st + (int64_t)(kvh * Gq) * p.o_sh);
    walk_rows(ln, (uint32_t)p.o_st, (uint32_t)p.o_sh, [&](int u, uint32_t off, int wr_r0) __attribute__((always_inline)) {
      if (wr_r0 < n_rows - u * QRPI)
        store_row_piece<kPast>(obase + (off * 2u + (uint32_t)(ln % G::CPR) * 16u), w[u]);
    });
  }
  // the row's log-sum-exp of its scaled scores (natural logarithm), for a backward pass
  if (p.lse != nullptr && ehf == 0 && wave_row0 + ecol < n_rows) {
    const int r = wave_row0 + ecol;
    const int tok = (int)fast_div((uint32_t)r, p.group_div);
    p.lse[(int64_t)(q_tok0 + tok) * p.n_q_heads + kvh * Gq + (r - tok * Gq)] =
        (mb + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f;  // (v_log_f32 is the base-2 logarithm)
  }
}

template <int D, bool kAsCore>
hipError_t launch_fresh_t(const AttnParams &p, const EncodeFreshMeta &meta, hipStream_t stream) {
  const int64_t n_wg = (int64_t)p.total_tiles * p.n_kv_heads;
  if (n_wg == 0) return hipSuccess;
  if (n_wg > 0x7fffffff || p.rows_past_cache) return hipErrorInvalidValue;
  const size_t lds = SGeo<D>::LDS + (size_t)meta.table_rows * D * 4;
  if (lds > SGeo<D>::LDS + kEncFreshLds) return hipErrorInvalidValue;
  static std::atomic<bool> raised{false};  // (set twice, from two host threads at once: harmless)
  if (SGeo<D>::LDS + kEncFreshLds > 64 * 1024 && !raised.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&encode_short_kernel<D, EncodeFreshMeta, kAsCore, false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)(SGeo<D>::LDS + kEncFreshLds));
    if (e != hipSuccess) return e;
    raised.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((encode_short_kernel<D, EncodeFreshMeta, kAsCore, false>), dim3((unsigned)n_wg), dim3(kSThreads), lds, stream, p, meta);
  return hipGetLastError();
}

template <int D, bool kAsCore, typename Meta>
hipError_t launch_short_t(const AttnParams &p, const Meta &meta, hipStream_t stream) {
  const int64_t n_wg = (int64_t)p.total_tiles * p.n_kv_heads;
  if (n_wg == 0) return hipSuccess;
  if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
  static_assert(SGeo<D>::LDS <= 64 * 1024, "fits the default dynamic LDS limit");
  if (p.rows_past_cache)
    hipLaunchKernelGGL((encode_short_kernel<D, Meta, kAsCore, true>), dim3((unsigned)n_wg), dim3(kSThreads), SGeo<D>::LDS, stream, p, meta);
  else
    hipLaunchKernelGGL((encode_short_kernel<D, Meta, kAsCore, false>), dim3((unsigned)n_wg), dim3(kSThreads), SGeo<D>::LDS, stream, p, meta);
  return hipGetLastError();
}

}  // namespace


hipError_t launch_attn_encode_short(const AttnParams &p, const EncodeMeta &meta, hipStream_t stream) {
  if (p.n_splits != 1) return hipErrorInvalidValue;
  const bool as_core = p.group < kSmallGroup;
  if (p.head_dim == 128) return as_core ? launch_short_t<128, true>(p, meta, stream) : launch_short_t<128, false>(p, meta, stream);
  if (p.head_dim == 64) return as_core ? launch_short_t<64, true>(p, meta, stream) : launch_short_t<64, false>(p, meta, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_attn_encode_fresh(const AttnParams &p, const EncodeFreshMeta &meta, hipStream_t stream) {
  if (p.n_splits != 1) return hipErrorInvalidValue;
  const bool as_core = p.group < kSmallGroup;
  if (p.head_dim == 128) return as_core ? launch_fresh_t<128, true>(p, meta, stream) : launch_fresh_t<128, false>(p, meta, stream);
  if (p.head_dim == 64) return as_core ? launch_fresh_t<64, true>(p, meta, stream) : launch_fresh_t<64, false>(p, meta, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_attn_prompt_short(const AttnParams &p, const PromptMeta &meta, hipStream_t stream) {
  if (p.n_splits != 1) return hipErrorInvalidValue;
  const bool shared = meta.n_split > 0;
  const SharedPromptMeta with(meta);
  if (p.head_dim == 128) return shared ? launch_short_t<128, false>(p, with, stream) : launch_short_t<128, false>(p, meta, stream);
  if (p.head_dim == 64) return shared ? launch_short_t<64, false>(p, with, stream) : launch_short_t<64, false>(p, meta, stream);
  return hipErrorInvalidValue;
}

}  // namespace ba
