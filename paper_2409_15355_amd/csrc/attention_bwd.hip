// Backward pass of whole-prompt Block-attention (arXiv 2409.15355, Section 2.4: the mask a block
// fine-tune step trains under).  With P the masked softmax of S = scale * q^ k^T (q^, k^ rotated at
// their positions inside the prompt), O = P V and dO given:
//   delta_r = sum_d dO_rd O_rd,   dV = P^T dO,   dP = dO V^T,   dS = P o (dP - delta),
//   dq^ = scale * dS k^,          dk^ = scale * dS^T q^.
// Nothing of the forward pass is kept but O and the rows' log-sum-exps L: P is recomputed as
// exp(S - L).  Two kernels, so that every sum has one owner (or owners that leave partial sums, which the last of
// them adds up in a fixed order) and no atomics on gradients are needed:
//   - bwd_dq_kernel: a workgroup owns 128 packed query rows (as the forward kernel for short items
//     does) and walks the key tiles its rows see; it accumulates dq^.  It rotates its query rows itself and
//     leaves them in memory for the other kernel, with -L / ln 2 and -delta of every row.
//   - bwd_dkv_kernel: a workgroup owns 64 keys (16 a wave) of one block and KV head and walks the 32-row
//     query tiles that see them (the rest of its own block, and the prompt's last block if it is a
//     passage); it accumulates dk^ and dV over all query heads of the group.
// Each turns its gradient of the rotated tensor back to the un-rotated frame in its epilogue, with the
// (cos, sin) table of the RoPE pre-pass (Eq. 1 is orthogonal: the transposed map is the rotation by
// minus the angle).
//
// Operand layouts are the forward kernel's: products are computed transposed with
// v_mfma_f32_32x32x16_bf16 (dk/dv: 16x16x32), the owner's side along lanes and in registers as B operands, the
// walked side from LDS tiles as A operands (16-byte row reads for the products that contract over
// head_dim, LDS transpose reads for those that contract over the walked index), and a probability
// tile in accumulator layout is directly the B operand of the next product.
#include <type_traits>

#include "ba_device.h"
#include "ba_lds.h"

namespace ba {
namespace {

constexpr int kBWaves = 4;
constexpr int kBThreads = kBWaves * 64;
constexpr int kBKeys = 32;  // walked rows (keys, or packed query rows) per tile
constexpr int kBBuf = 3;    // tile buffers
constexpr int kKvRows = kKvTileRows;
constexpr float kLn2 = 0.6931471805599453f, kLog2e = 1.4426950408889634f;

template <int D>
struct BGeo {
  static constexpr int KCH = D / 16;
  static constexpr int DT = D / 32;
  static constexpr int CPR = D / 8;
  static constexpr int ROWB = D * 2;
  static constexpr int RPI = 1024 / ROWB;             // rows filled by one LDS-direct wave instruction
  static constexpr int GRPB = 1024 + 16 * (RPI / 4);  // bytes from one such group of rows to the next (see tile_ofs)
  static constexpr int TILEB = kBKeys / RPI * GRPB;
  static constexpr int SLICEB = 16 / RPI * GRPB;      // sixteen rows
  static constexpr int IPW = kBKeys / RPI / kBWaves;  // such instructions per wave and tile
  static constexpr int QRPI = 64 / CPR;               // whole rows per plain load instruction
  static_assert(IPW >= 1 && 32 / QRPI == KCH, "tile geometry");
};

// Where row `row` of a tile keeps its 16-byte chunk `chunk`.  Both reads of a tile have to spread over the
// LDS banks: a row read (a lane per row, the same chunk of 16 rows) by 16-byte chunk, a transpose read
// (four rows, the same 64 bytes of each) by 64-byte granule.  So a row's low bits move the granule (an
// XOR), and what is left tells the rows apart inside it: at D = 128 the 16 bytes by which the groups of
// four rows are spaced beyond their 1 KB, at D = 64 the 32 bytes between groups of eight and one more
// XOR of the chunk's low bit.  (With the XOR of the row number over all chunk bits, the four rows of a
// transpose read shared one granule's banks.  The dk/dv kernel, whose products have another shape, has a layout of its own.)
// The XORs reach a chunk's granule and lowest bit only, so the two chunk pairs of a granule, the 16-row
// steps of a transpose read and the tiles of a buffer lie at constant distances from each other: a
// kernel keeps one address per granule, and the rest are offsets inside the instructions.
template <int D>
__device__ __forceinline__ int granule_xor(int row) { return D == 128 ? row & 3 : (row >> 1) & 1; }
template <int D>
__device__ __forceinline__ int low_xor(int row) { return D == 128 ? 0 : (row >> 2) & 1; }
template <int D>
__device__ __forceinline__ uint32_t tile_ofs(int row, int chunk) {
  using G = BGeo<D>;
  return (uint32_t)((row / G::RPI) * G::GRPB + (row % G::RPI) * G::ROWB +
                    ((chunk ^ (granule_xor<D>(row) << 2) ^ low_xor<D>(row)) << 4));
}
// Row read as A operand, k-step kk: row `col`, chunk 2 kk + hf.  base[kk / 2] + row_read_ofs(kk).
template <int D>
__device__ __forceinline__ void row_read_bases(uint32_t (&base)[D / 32], int col, int hf) {
#pragma unroll
  for (int g = 0; g < D / 32; ++g) base[g] = tile_ofs<D>(col, g * 4 + hf);
}
__device__ __forceinline__ constexpr uint32_t row_read_ofs(int kk) { return (uint32_t)(kk & 1) * 32u; }
// Transposed A operand, 16-row step kc, half `h` of its 8-byte pieces: base[dt] + tr_read_ofs(kc, h).
template <int D>
__device__ __forceinline__ void tr_read_bases(uint32_t (&base)[D / 32], int lane) {
  const int trow = (lane >> 5) * 4 + ((lane & 15) >> 2);
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt) {
    const int byte = dt * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    base[dt] = tile_ofs<D>(trow, byte >> 4) + (byte & 15);
  }
}
template <int D>
__device__ __forceinline__ constexpr uint32_t tr_read_ofs(int kc, int h) {
  return (uint32_t)((kc * 16 + h * 8) / BGeo<D>::RPI * BGeo<D>::GRPB);
}
template <int D>
__device__ __forceinline__ bf16x8_t row_frag(const lds_char *at, int kk) {
  return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t *>(at + row_read_ofs(kk));
}
template <int D>
__device__ __forceinline__ bf16x8_t tr_frag(lds_char *at, int kc) {
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at + tr_read_ofs<D>(kc, 0)));
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at + tr_read_ofs<D>(kc, 1)));
  const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, both);
}

// A gradient in the rotated frame, held in accumulator layout (lane = row `col`, register v of slab dt =
// head dim 32 dt + (v >> 2) * 8 + hf * 4 + (v & 3)), turned back to the un-rotated frame: the
// transposed map of Eq. 1, [x', y'] = [c x + s y, -s x + c y] per pair, times `mul`.  tab = the row's
// entry of the pre-pass's table, (cos, sin) per pair times some factor that `mul` takes out again.
template <int D>
__device__ __forceinline__ void rotate_back(f32x16_t (&acc)[D / 32], const f32x4_t *tab, int hf, bool halves, float mul) {
  constexpr int DT = D / 32;
  if (!halves) {
    // pairs (d, d + 1): the four values of (dt, q4) are pairs 2 m and 2 m + 1 with m = dt * 8 + q4 * 2 + hf
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4_t t = tab[dt * 8 + q4 * 2 + hf];
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          const float c = t[2 * h2] * mul, sn = t[2 * h2 + 1] * mul;
          const float x = acc[dt][q4 * 4 + 2 * h2], y = acc[dt][q4 * 4 + 2 * h2 + 1];
          acc[dt][q4 * 4 + 2 * h2] = c * x + sn * y;
          acc[dt][q4 * 4 + 2 * h2 + 1] = c * y - sn * x;
        }
      }
  } else {
    // pairs (d, d + D/2): slab dt pairs with slab dt + DT/2; the four values of (dt, q4) are pairs
    // j .. j + 3 with j = dt * 32 + q4 * 8 + hf * 4
#pragma unroll
    for (int dt = 0; dt < DT / 2; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          const f32x4_t t = tab[(dt * 32 + q4 * 8 + hf * 4) / 2 + h2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float c = t[2 * e] * mul, sn = t[2 * e + 1] * mul;
            const float x = acc[dt][q4 * 4 + 2 * h2 + e], y = acc[dt + DT / 2][q4 * 4 + 2 * h2 + e];
            acc[dt][q4 * 4 + 2 * h2 + e] = c * x + sn * y;
            acc[dt + DT / 2][q4 * 4 + 2 * h2 + e] = c * y - sn * x;
          }
        }
  }
}

// ---------------------------------------------------------------------------------------------------
// dq.  Bound by memory: q, dO and O in, q^ and dq out are 1.38 GB at 33,746 tokens of 32 heads of 128 (256 us
// at the 5.4 TB/s such a mix reaches here), and 1.88 GB move with the keys and values (re-read by a block's
// row tiles where L2 has let go of them).  350 us on rows that a pre-pass of 125 us had rotated; 386 rotating
// them itself; 357 with the rows that pass once marked non-temporal (kPast, in calls larger than the cache).  287
// of it remain with one key tile each.
// kShared: the table has blocks whose walk is shared (a kernel of its own, as in the forward pass).
template <int D, bool kPast, bool kShared>
__global__ __launch_bounds__(kBThreads, 2) void bwd_dq_kernel(AttnParams p, PromptMeta meta, BwdParams bp) {
  using G = BGeo<D>;
  extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
  lds_char *smem = (lds_char *)smem_generic;
  // LDS map: buffer b = bytes [2 b TB, 2 (b + 1) TB): its K tile, then its V tile
  constexpr uint32_t TB = G::TILEB;

  uint32_t id = blockIdx.x;
  {
    constexpr uint32_t kXcds = 8;
    const uint32_t n_wg = gridDim.x, q = n_wg / kXcds, r = n_wg % kXcds, x = id % kXcds;
    id = x * q + min(x, r) + id / kXcds;
  }
  const uint32_t n_rowtiles = (uint32_t)p.total_tiles;
  const int kvh = (int)fast_div(id, p.tiles_div);
  const int rowtile = (int)(id - (uint32_t)kvh * n_rowtiles);
  const int b = find_block(meta.tile_start, rowtile);
  const int q_tok0 = meta.start[b], lq = meta.len[b], k_tok0 = meta.kstart[b];
  const int pos0 = meta.pos0[b];  // position of the block's first token
  int jt = rowtile - meta.tile_start[b];
  const int dq = q_tok0 - k_tok0;  // the block's first token, counted in keys
  const int lk = dq + lq;          // keys up to the block's end

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, hf = lane >> 5;
  const int Gq = p.group;
  const int n_rows = lq * Gq;
  // a block whose walk is shared (see the forward kernel): which split, of how many
  int split = 0, n_splits = 1;
  if constexpr (kShared) {
    if (b < meta.n_split) {
      const WalkSplit ws = walk_split_of(n_rows, jt, meta.tile_start[b + 1] - meta.tile_start[b]);
      split = ws.split, n_splits = ws.n_splits;
      jt -= split * ws.n_row_tiles;
    }
  }
  const int row0 = jt * kShortTileRows;
  const int last_row = min(n_rows, row0 + kShortTileRows) - 1;
  TileRange walk = {0, (dq + (int)fast_div((uint32_t)last_row, p.group_div)) / kBKeys + 1};
  if (kShared && n_splits > 1) walk = walk_split_range(walk.end, n_splits, split);
  const int t0 = walk.begin, n_t = walk.end;
  const int wave_row0 = row0 + wave * 32;
  const int wave_last_row = min(n_rows, wave_row0 + 32) - 1;
  const int wave_n_t =
      wave_last_row >= wave_row0 ? (dq + (int)fast_div((uint32_t)wave_last_row, p.group_div)) / kBKeys + 1 : 0;
  const int first_key_wave = dq + (int)fast_div((uint32_t)wave_row0, p.group_div);
  const int my_row = min(wave_row0 + col, n_rows - 1);  // (lanes beyond the block's rows repeat its last row)
  const int my_tok = (int)fast_div((uint32_t)my_row, p.group_div);
  const int my_key = dq + my_tok;

  // ---- whole rows of q and dO for this wave, requested first (see the forward kernel) ------------
  // (Ofs: 32 bits where the host has checked that the offsets fit, 64 for q, whose strides are anyone's)
  auto walk_rows = [&](auto st, auto sh, auto &&visit) __attribute__((always_inline)) {
    typedef decltype(st) Ofs;
    const int wr_r0 = wave_row0 + lane / G::CPR;
    const int wr_tok0 = (int)fast_div((uint32_t)wr_r0, p.group_div);
    const int wr_g0 = wr_r0 - wr_tok0 * Gq;
    Ofs off = (Ofs)wr_tok0 * st + (Ofs)wr_g0 * sh;
    int g = wr_g0;
    const int step_tok = (int)fast_div((uint32_t)G::QRPI, p.group_div), step_g = G::QRPI - step_tok * Gq;
    const Ofs d_in = (Ofs)step_tok * st + (Ofs)step_g * sh, d_wrap = d_in + st - (Ofs)Gq * sh;
#pragma unroll
    for (int u = 0; u < G::KCH; ++u) {
      visit(u, off, wr_r0);
      g += step_g;
      const bool wrap = g >= Gq;
      g = wrap ? g - Gq : g;
      off += wrap ? d_wrap : d_in;
    }
  };
  u32x4_t ld_q[G::KCH], ld_do[G::KCH];
  {
    const char *qbase = (const char *)(p.q + (int64_t)q_tok0 * p.q_st + (int64_t)(kvh * Gq) * p.q_sh);
    const int64_t st = p.q_st, sh = p.q_sh;
    const int64_t last_off = (int64_t)(lq - 1) * st + (int64_t)(Gq - 1) * sh;
    walk_rows(st, sh, [&](int u, auto off, int wr_r0) __attribute__((always_inline)) {
      const int64_t o = wr_r0 < n_rows - u * G::QRPI ? off : last_off;
      ld_q[u] = load_row_piece<kPast>(qbase + (o * 2 + (lane % G::CPR) * 16));
    });
  }
  {
    const char *dbase = (const char *)(bp.dout + (int64_t)q_tok0 * bp.do_st + (int64_t)(kvh * Gq) * bp.do_sh);
    const uint32_t st = (uint32_t)bp.do_st, sh = (uint32_t)bp.do_sh;
    const uint32_t last_off = (uint32_t)(lq - 1) * st + (uint32_t)(Gq - 1) * sh;
    walk_rows(st, sh, [&](int u, auto off, int wr_r0) __attribute__((always_inline)) {
      const uint32_t o = wr_r0 < n_rows - u * G::QRPI ? off : last_off;
      ld_do[u] = load_row_piece<kPast>(dbase + (o * 2u + (uint32_t)(lane % G::CPR) * 16u));
    });
  }
  // ... and of O, for delta = rowsum(dO o O); this lane's row's log-sum-exp (to base-2 units below)
  u32x4_t ld_o[G::KCH];
  {
    const char *obase = (const char *)(bp.o + (int64_t)q_tok0 * bp.o_st + (int64_t)(kvh * Gq) * bp.o_sh);
    const uint32_t st = (uint32_t)bp.o_st, sh = (uint32_t)bp.o_sh;
    const uint32_t last_off = (uint32_t)(lq - 1) * st + (uint32_t)(Gq - 1) * sh;
    walk_rows(st, sh, [&](int u, auto off, int wr_r0) __attribute__((always_inline)) {
      const uint32_t o = wr_r0 < n_rows - u * G::QRPI ? off : last_off;
      ld_o[u] = load_row_piece<kPast>(obase + (o * 2u + (uint32_t)(lane % G::CPR) * 16u));
    });
  }
  const float my_lse = bp.lse[(int64_t)(q_tok0 + my_tok) * p.n_q_heads + kvh * Gq + (my_row - my_tok * Gq)];
  __builtin_amdgcn_sched_barrier(0);

  // ---- per-lane LDS read offsets inside a tile ---------------------------------------------------
  uint32_t k_rd[G::DT], t_rd[G::DT];
  row_read_bases<D>(k_rd, col, hf);
  tr_read_bases<D>(t_rd, lane);

  // ---- tile fill (K and V rows of 32 keys; rows beyond the valid ones repeat the last valid row) ----
  const char *k_base = (const char *)(p.kf + (int64_t)k_tok0 * p.kf_st + (int64_t)kvh * p.kf_sh);
  const char *v_base = (const char *)(p.vf + (int64_t)k_tok0 * p.vf_st + (int64_t)kvh * p.vf_sh);
  const uint32_t k_rb = (uint32_t)p.kf_st * 2u, v_rb = (uint32_t)p.vf_st * 2u;
  const int c_row = wave * G::IPW * G::RPI + lane / G::CPR;  // this lane's row of the wave's first instruction
  // (the XORs of tile_ofs depend on the row's place in its group only)
  const uint32_t c_chunk = (uint32_t)((lane % G::CPR) ^ (granule_xor<D>(lane / G::CPR) << 2) ^ low_xor<D>(lane / G::CPR)) << 4;
  const uint32_t lds_copy = (uint32_t)(uintptr_t)smem + wave * G::IPW * G::GRPB;
  auto issue_copy = [&](int t, int buf) __attribute__((always_inline)) {
    const int valid = min(kBKeys, lk - t * kBKeys);
    const char *kp = k_base + (uint64_t)(uint32_t)(t * kBKeys) * (uint64_t)k_rb;
    const char *vp = v_base + (uint64_t)(uint32_t)(t * kBKeys) * (uint64_t)v_rb;
#pragma unroll
    for (int u = 0; u < G::IPW; ++u) {
      const uint32_t row = (uint32_t)min(c_row + u * G::RPI, valid - 1);
      lds_dma16(kp, row * k_rb + c_chunk, lds_copy + (uint32_t)buf * (2 * TB) + u * G::GRPB);
      lds_dma16(vp, row * v_rb + c_chunk, lds_copy + (uint32_t)buf * (2 * TB) + TB + u * G::GRPB);
    }
  };
  constexpr int kOpsPerTile = 2 * G::IPW;
  // the pre-pass's table rows of this wave's tokens, 16-byte piece c of row t at c ^ (t & 7), into this
  // wave's slice of buffer 2; they come in here, the rows themselves pass through the slice behind them.
  // (Groups of four or more: at most 8 rows.  Smaller groups read their pieces from memory below.)
  constexpr uint32_t TROW = D * 4;
  constexpr int TCH = TROW / 16, kTabOps = 8 * TROW / 1024;
  static_assert(kBWaves * G::SLICEB <= 2 * TB && 8 * TROW <= G::SLICEB, "the slices fit one tile buffer");
  const uint32_t s_ofs = 2 * (2 * TB) + wave * G::SLICEB;
  const int first_tok_wave = first_key_wave - dq;
  if (Gq >= 4) {
    const char *tbase = (const char *)(p.q_table + (int64_t)pos0 * D);
#pragma unroll
    for (int u = 0; u < kTabOps; ++u) {
      const int t = u * (1024 / TROW) + lane / TCH, pc = lane % TCH;
      const uint32_t tok = (uint32_t)min(first_tok_wave + t, lq - 1);
      lds_dma16(tbase, tok * TROW + (uint32_t)((pc ^ (t & 7)) << 4), (uint32_t)(uintptr_t)smem + s_ofs + u * 1024);
    }
  }
  if (t0 < n_t) issue_copy(t0, 0);
  if (t0 + 1 < n_t) issue_copy(t0 + 1, 1);
  __builtin_amdgcn_sched_barrier(0);
  dma_wait<0>();

  // ---- whole rows -> B-operand fragments (lane = row), 16 rows at a time through this wave's slice ----
  f32x4_t cs[2 * G::KCH];
  if (Gq < 4) {
    const f32x4_t *row = reinterpret_cast<const f32x4_t *>(p.q_table + (int64_t)(pos0 + my_tok) * D);
#pragma unroll
    for (int j = 0; j < 2 * G::KCH; ++j) cs[j] = row[fragment_table_piece(j, hf, p.rope_layout != 0)];
  } else {
    const int tl = max(my_tok - first_tok_wave, 0);  // this lane's row of the table slice
#pragma unroll
    for (int j = 0; j < 2 * G::KCH; ++j)
      cs[j] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4_t *>(
          smem + s_ofs + (uint32_t)tl * TROW + (uint32_t)((fragment_table_piece(j, hf, p.rope_layout != 0) ^ (tl & 7)) << 4));
  }
  auto rows_to_frags = [&](const u32x4_t (&ld)[G::KCH], u32x4_t (&out)[G::KCH]) __attribute__((always_inline)) {
    u32x4_t got[2][G::KCH];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
      for (int u = 0; u < G::KCH / 2; ++u)
        *reinterpret_cast<__attribute__((address_space(3))) u32x4_t *>(
            smem + s_ofs + tile_ofs<D>(u * G::QRPI + lane / G::CPR, lane % G::CPR)) = ld[pass * (G::KCH / 2) + u];
#pragma unroll
      for (int kk = 0; kk < G::KCH; ++kk)
        got[pass][kk] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4_t *>(
            smem + s_ofs + tile_ofs<D>(col & 15, kk * 2 + hf));
    }
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk)
#pragma unroll
      for (int e = 0; e < 4; ++e) out[kk][e] = (col >> 4) ? got[1][kk][e] : got[0][kk][e];
  };
  // delta of this wave's rows: a row's CPR lanes add up their pieces, one of them hands the sum over
  // through the slice to the lane that owns the row; -L / ln 2 and -delta also go to memory in packed-row
  // order per KV head, four rows of the one and four of the other in turn: as the dk/dv kernel's
  // lanes read them from its tile
  float2 my_ld;
  {
    float mine = 0.f;  // lane j of a run of CPR lanes takes the sum of the run's j-th row
#pragma unroll
    for (int u = 0; u < G::KCH; ++u) {
      float part = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        part += bf16_lo(ld_o[u][e]) * bf16_lo(ld_do[u][e]) + bf16_hi(ld_o[u][e]) * bf16_hi(ld_do[u][e]);
      part = sum_over_lanes<G::CPR>(part);
      mine = lane % G::CPR == u ? part : mine;
    }
    if (lane % G::CPR < G::KCH)
      *reinterpret_cast<__attribute__((address_space(3))) float *>(
          smem + s_ofs + ((lane % G::CPR) * G::QRPI + lane / G::CPR) * 4) = mine;
    const int r_in_wave = min(col, max(wave_last_row - wave_row0, 0));  // (lanes beyond the block's rows: its last row)
    my_ld.y = *reinterpret_cast<const __attribute__((address_space(3))) float *>(smem + s_ofs + r_in_wave * 4);
    my_ld.x = my_lse * kLog2e;
    if (split == 0 && wave_row0 + col < n_rows) {
      const int r = wave_row0 + col;
      float *dst = bp.ld + 2 * (((int64_t)kvh * bp.T + q_tok0) * bp.ld_group) + (r >> 2) * 8 + (r & 3);
      dst[hf * 4] = hf ? -my_ld.y : -my_ld.x;  // the two halves of the wave hold the same rows
    }
  }
  // q^ = the rows rotated and scaled, this kernel's operand and, in memory, what the dk/dv kernel walks
  bf16x8_t qf[G::KCH], dof[G::KCH];
  {
    u32x4_t raw[G::KCH];
    rows_to_frags(ld_q, raw);
    rotate_fragments<G::KCH>(raw, cs, p.rope_layout != 0);
    uint16_t *dst = bp.q_rot + ((int64_t)(q_tok0 + my_tok) * p.n_q_heads + kvh * Gq + (my_row - my_tok * Gq)) * D + hf * 8;
    const bool mine = split == 0 && wave_row0 + col < n_rows;
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk) {
      if (mine) *reinterpret_cast<u32x4_t *>(dst + kk * 16) = raw[kk];
      qf[kk] = __builtin_bit_cast(bf16x8_t, raw[kk]);
    }
    rows_to_frags(ld_do, raw);
#pragma unroll
    for (int kk = 0; kk < G::KCH; ++kk) {
      asm volatile("" : "+v"(raw[kk]));
      dof[kk] = __builtin_bit_cast(bf16x8_t, raw[kk]);
    }
  }

  f32x16_t acc[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[dt][v] = 0.f;

  // ---- the walk over the key tiles ---------------------------------------------------------------
  // (rolling windows of LDS fragments: the first four transposed ones are asked for ahead of the
  // exponentials.  Six row fragments instead of four would spill.  The same call 958 -> 953 us.  At head_dim 64, whose kernel
  // has the registers for it, no difference.)
  constexpr int kRowWin = 4, kTrWin = 4;
  int buf = 0;
#pragma unroll 1
  for (int i = t0; i < n_t; ++i) {
    // (the first two tiles have landed; waiting here would be for the stores of q^)
    if (i >= t0 + 2) {
      if (i + 1 < n_t) dma_wait<kOpsPerTile>(); else dma_wait<0>();
    }
    wg_barrier();
    if (i + 2 < n_t) issue_copy(i + 2, buf == 0 ? 2 : buf - 1);
    if (i < wave_n_t) {
      lds_char *const bk = smem + (uint32_t)buf * (2 * TB);  // this tile: K rows, then (TB on) V rows
      // S'^T - L: the base-2 exponent of P;  dP^T - delta
      // (step st is product st / 2 of the one, K, if st is even, else of the other, V; a window of fragments)
      f32x16_t sacc, dpacc;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sacc[v] = -my_ld.x;
        dpacc[v] = -my_ld.y;
      }
      auto kv_frag = [&](int st) __attribute__((always_inline)) {
        return row_frag<D>(bk + k_rd[st / 4] + (st & 1) * TB, st / 2);
      };
      bf16x8_t fr[kRowWin];
#pragma unroll
      for (int st = 0; st < kRowWin; ++st) fr[st] = kv_frag(st);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < 2 * G::KCH; ++st) {
        if (st & 1) dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[st % kRowWin], dof[st / 2], dpacc, 0, 0, 0);
        else sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[st % kRowWin], qf[st / 2], sacc, 0, 0, 0);
        if (st + kRowWin < 2 * G::KCH) fr[st % kRowWin] = kv_frag(st + kRowWin);
        __builtin_amdgcn_sched_barrier(0);
      }
      bf16x8_t tr[kTrWin];
#pragma unroll
      for (int st = 0; st < kTrWin; ++st) tr[st] = tr_frag<D>(bk + t_rd[st % G::DT], st / G::DT);
      __builtin_amdgcn_sched_barrier(0);
      const int key0 = i * kBKeys;
      const int valid = min(kBKeys, lk - key0);
      if (key0 + kBKeys - 1 > first_key_wave || valid < kBKeys) {
        const int lim = min(my_key - key0 + 1, valid);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = (v >> 2) * 8 + hf * 4 + (v & 3);
          if (key >= lim) sacc[v] = -INFINITY;
        }
      }
      // dS^T = P^T o (dP^T - delta), rounded to bf16: the B operand of dq^^T += K^T dS^T
      bf16x8_t dsf[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        u32x4_t w;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float d0 = __builtin_amdgcn_exp2f(sacc[e * 8 + 2 * j]) * dpacc[e * 8 + 2 * j];
          const float d1 = __builtin_amdgcn_exp2f(sacc[e * 8 + 2 * j + 1]) * dpacc[e * 8 + 2 * j + 1];
          w[j] = pack_bf16(d0, d1);
        }
        dsf[e] = __builtin_bit_cast(bf16x8_t, w);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < 2 * G::DT; ++st) {
        acc[st % G::DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr[st % kTrWin], dsf[st / G::DT], acc[st % G::DT], 0, 0, 0);
        if (st + kTrWin < 2 * G::DT) tr[st % kTrWin] = tr_frag<D>(bk + t_rd[(st + kTrWin) % G::DT], (st + kTrWin) / G::DT);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    buf = buf == kBBuf - 1 ? 0 : buf + 1;
  }

  // ---- epilogue: dq^ = scale * acc, turned back to dq with the row's entry of the pre-pass's table
  //      (which carries scale * log2 e: scale / (scale * log2 e) = ln 2 remains), bf16, as whole rows
  //      through each wave's slice of LDS -------------------------------------------------------------
  wg_barrier();
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int ecol = ln & 31, ehf = ln >> 5;
  if constexpr (kShared) {
    // (a shared walk: the accumulators of all splits add up in their order)
    int bs = b;
    asm volatile("" : "+s"(bs));  // (as in the forward kernel)
    if (bs < meta.n_split) {
      const int first = meta.tile_start[bs];
      const WalkSplit ws = walk_split_of(n_rows, rowtile - first, meta.tile_start[bs + 1] - first);
      const int tile0 = rowtile - ws.split * ws.n_row_tiles;                                   // of split 0
      const int64_t slot = ((int64_t)tile0 * p.n_kv_heads + kvh) * kSplitWaves + wave;         // of split 0
      const int64_t step = (int64_t)ws.n_row_tiles * p.n_kv_heads * kSplitWaves;               // to the next
      float *const part_o = (float *)p.part_o;
      const bool live = wave_row0 < n_rows;
      if (live) leave_accumulators<D>(part_o, slot + ws.split * step, ln, acc);
      static_assert(kBWaves * G::TILEB + 16 <= 2 * kBBuf * G::TILEB, "a word behind the output staging");
      if (!last_of_splits(p.part_idx + (int64_t)tile0 * p.n_kv_heads + kvh, ws.n_splits,
                          smem + 2 * kBBuf * G::TILEB - 16))
        return;
      if (live) {
#pragma unroll
        for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[dt][v] = 0.f;
#pragma unroll 1
        for (int s = 0; s < ws.n_splits; ++s) {
          u32x4_t w[D / 8];
          fetch_accumulators<D>(part_o, slot + s * step, ln, w);
#pragma unroll
          for (int k = 0; k < D / 8; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) *((float *)&acc[k >> 2] + (k & 3) * 4 + e) += __uint_as_float(w[k][e]);
        }
      }
    }
  }
  rotate_back<D>(acc, reinterpret_cast<const f32x4_t *>(p.q_table + (int64_t)(pos0 + my_tok) * D), ehf,
                 p.rope_layout != 0, kLn2);
  lds_char *stage = smem + wave * G::TILEB;
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      u32x2_t w;
      w[0] = pack_bf16(acc[dt][q4 * 4 + 0], acc[dt][q4 * 4 + 1]);
      w[1] = pack_bf16(acc[dt][q4 * 4 + 2], acc[dt][q4 * 4 + 3]);
      *reinterpret_cast<__attribute__((address_space(3))) u32x2_t *>(stage + tile_ofs<D>(ecol, dt * 4 + q4) + ehf * 8) = w;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  {
    u32x4_t w[G::KCH];
#pragma unroll
    for (int u = 0; u < G::KCH; ++u)
      w[u] = *reinterpret_cast<const __attribute__((address_space(3))) u32x4_t *>(
          stage + tile_ofs<D>(u * G::QRPI + ln / G::CPR, ln % G::CPR));
    char *obase = (char *)(bp.dq + (int64_t)q_tok0 * bp.dq_st + (int64_t)(kvh * Gq) * bp.dq_sh);
    walk_rows((uint32_t)bp.dq_st, (uint32_t)bp.dq_sh, [&](int u, auto off, int wr_r0) __attribute__((always_inline)) {
      if (wr_r0 < n_rows - u * G::QRPI)
        store_row_piece<kPast>(obase + (off * 2u + (uint32_t)(ln % G::CPR) * 16u), w[u]);
    });
  }
}

// ---------------------------------------------------------------------------------------------------
// dk and dV.  A wave owns 16 keys with both sums (dK^ and dV: 64 registers) and both operands (K^ and V: 32), which with
// 16x16x32 products leaves three waves a SIMD room for windows of fragments; per tile of 32 packed rows it forms
//   S = q^ K^^T - L,  dP = dO V^T - delta,  P = 2^S,  dS = P o dP,  dV^T += dO^T P,  dK^^T += q^^T dS
// from its own registers and the tile, with one barrier.  (Waves of 32 keys have no registers left to look ahead with, two to a SIMD:
// 370 us.  Split between a pair of waves, S and dV here, dP and dK^ there, with P handed over through LDS behind a
// second barrier: 320.)  Each fragment of a tile feeds half as many products as with 32 keys, so LDS is read twice as much, 44 %
// of the time: the price of doing without the exchange.
// Eight prompts of 20 passages of 100 to 300 tokens and a query block (33,746 tokens, 32 query heads over 8 of
// 128, 208 GFLOP in four products): 320 -> 285 us, forward and backward 940 -> 903; 32 over 8 of 64 524 -> 486; two
// prompts there 282 -> 270.  1.0 GB read (q^ and dO once are 553 MB), 138 MB written.  What is left is waiting, 38 % of the waves' time for
// memory and at barriers and 30 % to issue; a third tile buffer, which now fits three workgroups, changes nothing.
template <int D>
struct KvGeo {
  static constexpr int KK = D / 32;                   // k-steps of the products over head_dim
  static constexpr int DT = D / 16;                   // 16-row slabs of dV^T and dK^^T
  static constexpr int CPR = D / 8;                   // 16-byte chunks per row
  static constexpr uint32_t ROWB = D * 2;
  static constexpr uint32_t TB = kKvRows * ROWB;      // a tile of q^ or dO
  static constexpr uint32_t BUFB = 2 * TB + kKvRows * 8;  // ... of both, and their rows' -L and -delta
  static constexpr int RPI = 1024 / ROWB;             // rows filled by one LDS-direct wave instruction
  static constexpr int IPW = kKvRows / RPI / 2;       // such instructions of one wave per tile (one tensor's half)
  static constexpr int KEYS = kBwdTileKeys / kBWaves; // a wave's keys
  static constexpr size_t LDS = 2 * (size_t)BUFB;
  static_assert(KEYS == 16 && kKvRows == 32 && BUFB % 256 == 0, "16x16x32 products, two row halves a tile, transpose reads");
};

typedef __attribute__((address_space(3))) f32x4_t lds_f32x4;
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4;
typedef __attribute__((address_space(3))) u32x2_t lds_u32x2;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8;

// Where row `row` of a tile keeps its 16-byte chunk `chunk`: XORed with a number that depends on the row's place among
// sixteen (a row of LDS banks holds one row at D = 128, two at 64), so that both kinds of reads spread over all banks.  A row
// read (lane = row, four neighbouring chunks to the lane groups) goes through the banks in four rounds, the first of
// lanes 0-3, 12-15, 20-23 and 24-27: rows 0-3 and 12-15 of one chunk, 4-11 of the next, so either set's numbers come in
// pairs that differ in the lowest bit.  A transpose read takes two neighbouring chunks of eight rows a round, whose numbers
// differ above the lowest bit.  (Numbers that only differ over sixteen rows: a third of the LDS cycles were conflicts.)
template <int D>
__device__ __forceinline__ uint32_t kv_xor(int row) {
  const uint32_t s = (uint32_t)(D == 128 ? row : row >> 1);
  constexpr int kLow = D == 128 ? 2 : 1;  // bits that tell neighbours apart
  const uint32_t lo = s & ((1u << kLow) - 1), a = (s >> kLow) & 1u, b = (s >> (kLow + 1)) & 1u;
  return lo << 1 | (a ^ b) << (kLow + 1) | b;
}
template <int D>
__device__ __forceinline__ uint32_t kv_ofs(int row, int chunk) {
  return (uint32_t)row * KvGeo<D>::ROWB + (((uint32_t)chunk ^ kv_xor<D>(row)) << 4);
}

// 16x16x32 products.  Row read, step st of the four products over head_dim that go side by side (of tensor st >> 1 & 1, TB
// apart, rows 16 (st & 1) + lane % 16, k-step st / 4): at[k-step] + kv_row_ofs(st).
template <int D>
__device__ __forceinline__ void kv_row_bases(uint32_t (&at)[D / 32], int col, int g) {
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) at[kk] = kv_ofs<D>(col, kk * 4 + g);
}
template <int D>
__device__ __forceinline__ constexpr uint32_t kv_row_ofs(int st) {
  return (uint32_t)((st >> 1) & 1) * KvGeo<D>::TB + (uint32_t)(st & 1) * 16u * KvGeo<D>::ROWB;
}
// Transpose read of slab dt (16 head dims) of a tile: kv_tr_frag(tile + (kv_tr_base ^ 32 dt)), for tiles 256-byte aligned in
// LDS.  Its k-slots are rows 4 g + 0..3 and 16 + 4 g + 0..3: the order in which two accumulators of 16 rows hold theirs.
template <int D>
__device__ __forceinline__ uint32_t kv_tr_base(int lane) {
  return kv_ofs<D>(4 * (lane >> 4) + ((lane & 15) >> 2), (lane >> 1) & 1) + (lane & 1) * 8;
}
template <int D>
__device__ __forceinline__ bf16x8_t kv_tr_frag(lds_char *at) {
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)at);
  const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(at + 16 * KvGeo<D>::ROWB));
  const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, both);
}
// two accumulators of 16 rows each -> the B operand of the next product (see kv_tr_frag)
__device__ __forceinline__ bf16x8_t pack_rows(const f32x4_t &lo, const f32x4_t &hi) {
  const u32x4_t w = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
  return __builtin_bit_cast(bf16x8_t, w);
}

// rotate_back for sums in this kernel's layout (lane = key `col`, register v of slab dt = head dim 16 dt + 4 g + v).
template <int D>
__device__ __forceinline__ void rotate_back_keys(f32x4_t (&acc)[D / 16], const f32x4_t *tab, int g, bool halves, float mul) {
  constexpr int DT = D / 16;
  if (!halves) {
    // pairs (d, d + 1): slab dt holds pairs 8 dt + 2 g and the next
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4_t t = tab[dt * 4 + g];
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        const float c = t[2 * h2] * mul, sn = t[2 * h2 + 1] * mul;
        const float x = acc[dt][2 * h2], y = acc[dt][2 * h2 + 1];
        acc[dt][2 * h2] = c * x + sn * y;
        acc[dt][2 * h2 + 1] = c * y - sn * x;
      }
    }
  } else {
    // pairs (d, d + D/2): slab dt pairs with slab dt + DT/2, pairs 16 dt + 4 g + (0..3)
#pragma unroll
    for (int dt = 0; dt < DT / 2; ++dt)
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        const f32x4_t t = tab[dt * 8 + g * 2 + h2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float c = t[2 * e] * mul, sn = t[2 * e + 1] * mul;
          const float x = acc[dt][2 * h2 + e], y = acc[dt + DT / 2][2 * h2 + e];
          acc[dt][2 * h2 + e] = c * x + sn * y;
          acc[dt + DT / 2][2 * h2 + e] = c * y - sn * x;
        }
      }
  }
}
// A sum's 16 rows into LDS, as kv_ofs has them, to leave as whole rows.
template <int D>
__device__ __forceinline__ void stage_rows(lds_char *stage, const f32x4_t (&acc)[D / 16], int col, int g) {
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const u32x2_t w = {pack_bf16(acc[dt][0], acc[dt][1]), pack_bf16(acc[dt][2], acc[dt][3])};
    *(lds_u32x2 *)(stage + kv_ofs<D>(col, dt * 2 + (g >> 1)) + (g & 1) * 8) = w;
  }
}
// Partial sums of a shared walk: N registers of 16 bytes a lane, a kilobyte of consecutive memory each, past the L2 caches.
template <int N>
__device__ __forceinline__ void leave_sums(char *at, int lane, int first, const f32x4_t (&acc)[N]) {
  const auto to = shared_buffer(at, (first + N) * 1024);
#pragma unroll
  for (int k = 0; k < N; ++k)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[k]), to, lane * 16 + (first + k) * 1024, 0, kAgentScope);
}
template <int N>
__device__ __forceinline__ void add_sums(char *at, int lane, f32x4_t (&a)[N], f32x4_t (&b)[N]) {
  const auto from = shared_buffer(at, 2 * N * 1024);
  f32x4_t w[2 * N];
#pragma unroll
  for (int k = 0; k < 2 * N; ++k)
    w[k] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(from, lane * 16 + k * 1024, 0, kAgentScope));
#pragma unroll
  for (int k = 0; k < N; ++k) {
    a[k] += w[k];
    b[k] += w[N + k];
  }
}

template <int D, bool kShared>
__global__ __launch_bounds__(kBThreads, D == 128 ? 3 : 5) void bwd_dkv_kernel(AttnParams p, BwdKvMeta meta, BwdParams bp) {
  using KG = KvGeo<D>;
  extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
  lds_char *smem = (lds_char *)smem_generic;
  // LDS map: two buffers of BUFB: the tile of q^, of dO, -L and -delta of their rows (four of the one, four of the other in turn)
  constexpr uint32_t TB = KG::TB, BUFB = KG::BUFB, ROWB = KG::ROWB;
  constexpr int IPW = KG::IPW;

  uint32_t id = blockIdx.x;
  {
    constexpr uint32_t kXcds = 8;
    const uint32_t n_wg = gridDim.x, q = n_wg / kXcds, r = n_wg % kXcds, x = id % kXcds;
    id = x * q + min(x, r) + id / kXcds;
  }
  const uint32_t n_keytiles = (uint32_t)p.total_tiles;
  const int kvh = (int)fast_div(id, p.tiles_div);
  const int keytile = (int)(id - (uint32_t)kvh * n_keytiles);
  const int b = find_block(meta.tile_start, keytile);
  const int k_tok0 = meta.start[b], lk = meta.len[b];  // the block that owns the keys
  const int f_tok0 = meta.fin_start[b], lf = meta.fin_len[b];  // its prompt's last block, if it is a passage
  // a block whose walks are shared: which split of which key tile
  int split = 0, n_kt = 0, jt = keytile - meta.tile_start[b];
  const bool shared = kShared && b < meta.n_split;
  if (shared) {
    n_kt = (lk + kBwdTileKeys - 1) / kBwdTileKeys;
    split = jt / n_kt;
    jt -= split * n_kt;
  }
  const int k0 = jt * kBwdTileKeys;  // the workgroup's first key, inside the block

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, g = lane >> 4;
  const int Gq = p.group;
  const int kw0 = k0 + wave * KG::KEYS;  // this wave's first key
  const bool wave_has_keys = kw0 < lk;
  const int my_key = kw0 + col;    // (may lie beyond the block: such columns are never stored)

  // ---- query row tiles that see these keys: every row of the prompt's last block, then the block's own
  //      rows, both from the end to the front, down to the first key's token.  The workgroups of a block
  //      start together and so meet each tile at about the same time, in one XCD's L2; walked from the
  //      front, each starts at a row of its own and fetches its tiles alone (1692 MB per launch at 33,746
  //      tokens where q^ and dO are 553) ---------------------------------------------------------------
  const int n_rows_a = lk * Gq, n_rows_f = lf * Gq;
  const int n_f = (n_rows_f + kKvRows - 1) / kKvRows;
  TileRange walk = {0, n_f + (n_rows_a + kKvRows - 1) / kKvRows - (k0 * Gq) / kKvRows};
  int n_splits = 1;
  if (shared) {
    n_splits = walk_splits(walk.end, meta.chunk);
    if (split >= n_splits) return;  // (the key tiles behind a block's first walk less and take fewer)
    walk = walk_split_range(walk.end, n_splits, split);
  }
  const int t0 = walk.begin, n_t = walk.end;  // this workgroup's tiles
  const int own_last = ((n_rows_a - 1) / kKvRows) * kKvRows;  // first row of the block's last tile
  const int fin_last = (n_f - 1) * kKvRows;

  // ---- tile fill: kKvRows packed query rows of q^ (the even waves) and of dO (the odd ones), and the
  //      rows' -L / ln 2 and -delta.  Where the group divides 32, every tile begins with a token's first
  //      head and its rows lie at the same distances from there: the lanes' offsets are worked out once and
  //      a tile moves one pointer (the copy goes out between the barrier and the products; with the
  //      rows divided out per instruction a wave spent 180 scalar instructions on a tile).  Otherwise, and
  //      in the last tile of a block (rows beyond the block repeat its last row), every lane finds its own ----
  const bool of_do = wave & 1;
  const int half = wave >> 1;
  const uint32_t c_st = of_do ? (uint32_t)bp.do_st : (uint32_t)(p.n_q_heads * D), c_sh = of_do ? (uint32_t)bp.do_sh : (uint32_t)D;
  const uint32_t lds_copy = (uint32_t)(uintptr_t)smem + (of_do ? TB : 0u) + half * IPW * 1024;
  const uint32_t lds_ld = (uint32_t)(uintptr_t)smem + 2 * TB + wave * 64;
  auto c_row = [&](int u) __attribute__((always_inline)) { return (half * IPW + u) * KG::RPI + lane / KG::CPR; };  // this lane's row of instruction u
  auto row_ofs = [&](uint32_t r, int u) __attribute__((always_inline)) {  // packed row r, in bytes from its block's first; this lane's chunk
    const uint32_t tok = fast_div(r, p.group_div), gh = r - tok * (uint32_t)Gq;
    return (tok * c_st + gh * c_sh) * 2u + (((uint32_t)(lane % KG::CPR) ^ kv_xor<D>(c_row(u))) << 4);
  };
  const bool regular = kKvRows % Gq == 0;
  const uint32_t c_step = regular ? (uint32_t)(kKvRows / Gq) * c_st * 2u : 0u;  // bytes from tile to tile
  uint32_t c_in[IPW];
#pragma unroll
  for (int u = 0; u < IPW; ++u) c_in[u] = row_ofs((uint32_t)c_row(u), u);
  const char *c_base = nullptr, *l_base = nullptr;  // the next tile's rows (their block's first, if not regular); its -L, -delta
  int c_row0 = 0, c_rows = 0;                       // its first packed row inside its block; the block's rows
  auto enter_block = [&](int tok0, int row0, int rows) __attribute__((always_inline)) {
    c_row0 = row0;
    c_rows = rows;
    c_base = of_do ? (const char *)(bp.dout + (int64_t)tok0 * bp.do_st + (int64_t)(kvh * Gq) * bp.do_sh)
                   : (const char *)(bp.q_rot + ((int64_t)tok0 * p.n_q_heads + kvh * Gq) * D);
    c_base += (uint64_t)(uint32_t)(row0 / kKvRows) * c_step;
    l_base = (const char *)(bp.ld + 2 * (((int64_t)kvh * bp.T + tok0) * bp.ld_group)) + (uint32_t)row0 * 8u;
  };
  if (t0 < n_f) enter_block(f_tok0, fin_last - t0 * kKvRows, n_rows_f);
  else enter_block(k_tok0, own_last - (t0 - n_f) * kKvRows, n_rows_a);
  auto issue_copy = [&](int t, int buf) __attribute__((always_inline)) {
    if (t == n_f) enter_block(k_tok0, own_last, n_rows_a);
    const uint32_t lds_tile = lds_copy + (uint32_t)buf * BUFB;
    if (regular && c_row0 + kKvRows <= c_rows) {
#pragma unroll
      for (int u = 0; u < IPW; ++u) lds_dma16(c_base, c_in[u], lds_tile + u * 1024);
    } else {
      const uint32_t from = regular ? (uint32_t)c_row0 : 0u;  // the row that c_base is at
#pragma unroll
      for (int u = 0; u < IPW; ++u)
        lds_dma16(c_base, row_ofs((uint32_t)min(c_row0 + c_row(u), c_rows - 1) - from, u), lds_tile + u * 1024);
    }
    // four rows of -L and four of -delta in turn, 16 bytes each (the block's last four perhaps partly
    // unwritten; beyond them the last are read again)
    if (lane < 4)
      lds_dma16(l_base, (uint32_t)(min(wave * 2 + (lane >> 1), (c_rows - 1 - c_row0) >> 2) * 2 + (lane & 1)) * 16u, lds_ld + (uint32_t)buf * BUFB);
    c_row0 -= kKvRows;
    c_base -= c_step;
    l_base -= kKvRows * 8;
  };
  if (t0 < n_t) issue_copy(t0, 0);

  // ---- this wave's operands: fragments of its K^ and V rows (B operands: column = key, k-step kk holds chunk 4 kk + g) ----
  bf16x8_t kf[KG::KK], vf[KG::KK];
  {
    const uint64_t tok = (uint64_t)(uint32_t)min(my_key, lk - 1);
    const char *kp = (const char *)(p.kf + (int64_t)k_tok0 * p.kf_st + (int64_t)kvh * p.kf_sh) + tok * (uint64_t)p.kf_st * 2u + g * 16;
    const char *vp = (const char *)(p.vf + (int64_t)k_tok0 * p.vf_st + (int64_t)kvh * p.vf_sh) + tok * (uint64_t)p.vf_st * 2u + g * 16;
#pragma unroll
    for (int kk = 0; kk < KG::KK; ++kk) kf[kk] = *reinterpret_cast<const bf16x8_t *>(kp + kk * 64);
#pragma unroll
    for (int kk = 0; kk < KG::KK; ++kk) vf[kk] = *reinterpret_cast<const bf16x8_t *>(vp + kk * 64);
  }
  __builtin_amdgcn_sched_barrier(0);
  dma_wait<0>();
#pragma unroll
  for (int kk = 0; kk < KG::KK; ++kk) asm volatile("" : "+v"(kf[kk]), "+v"(vf[kk]));  // (waited for here, not inside the loop)

  f32x4_t dv[KG::DT], dk[KG::DT];
#pragma unroll
  for (int dt = 0; dt < KG::DT; ++dt) dv[dt] = dk[dt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

  uint32_t r_rd[KG::KK];
  kv_row_bases<D>(r_rd, col, g);
  const uint32_t t_rd = kv_tr_base<D>(lane);

  // ---- the walk over the query row tiles, two buffers in turn.  A tile's barrier says that every wave's share of it
  //      has landed and that all are done with the tile before, so the copy of the next may overwrite that buffer ----
  // Fragments come through rolling windows, as many as the registers take: three waves a SIMD at D = 128 (168), five at 64
  // (96; with four of either and four waves 219 and 502 us where two and five take 211 and 486: prompts of 30 passages of 40 to
  // 160 tokens at 16 over 2 heads, of 20 of 100 to 300 at 32 over 8).  At 128 four of either take 921 us a step where six take 919.
  constexpr int kRowWin = D == 128 ? 6 : 2, kTrWin = D == 128 ? 6 : 2, kTrAhead = D == 128 ? 2 : 0;  // (kTrAhead: ahead of the exponentials)
  const auto fence = []() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
  uint32_t cur = 0;  // this tile's buffer
#pragma unroll 1
  for (int i = t0; i < n_t; ++i, cur ^= BUFB) {
    dma_wait<0>();
    wg_barrier();
    if (i + 1 < n_t) issue_copy(i + 1, cur == 0);
    const bool own = i >= n_f;
    const int r0 = own ? own_last - (i - n_f) * kKvRows : fin_last - i * kKvRows;  // the tile's first packed row, inside its block
    const int n_rows = own ? n_rows_a : n_rows_f;
    // a tile of the block's own rows whose tokens all lie before this wave's first key sees none of them
    // (row = token * group + head: row r's token is at or behind key k exactly if r >= k * group)
    if (!wave_has_keys || (own && min(r0 + kKvRows, n_rows) <= kw0 * Gq)) continue;
    lds_char *const buf = smem + cur;
    // The accumulators start at minus the rows' log-sum-exp or delta, so that the products come out as
    // the exponent of P and as dP - delta.  Half rt, register v is row 16 rt + 4 g + v.
    f32x4_t x[4];  // S - L of both halves, then P; dP - delta of both halves, then dS
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      x[rt] = *(const lds_f32x4 *)(buf + 2 * TB + (rt * 4 + g) * 32);
      x[2 + rt] = *(const lds_f32x4 *)(buf + 2 * TB + (rt * 4 + g) * 32 + 16);
    }
    auto row_frag_of = [&](int st) __attribute__((always_inline)) {  // step st: k-step st / 4 of x[st % 4]
      return *(const lds_bf16x8 *)(buf + r_rd[st / 4] + kv_row_ofs<D>(st));
    };
    bf16x8_t fr[kRowWin];
#pragma unroll
    for (int st = 0; st < kRowWin; ++st) fr[st] = row_frag_of(st);
    fence();
#pragma unroll
    for (int st = 0; st < 4 * KG::KK; ++st) {
      x[st & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[st % kRowWin], (st & 2) ? vf[st / 4] : kf[st / 4], x[st & 3], 0, 0, 0);
      if (st + kRowWin < 4 * KG::KK) fr[st % kRowWin] = row_frag_of(st + kRowWin);
      fence();
    }
    // transposed fragments: slab st % DT of dO^T, then of q^^T; rows in the order that P and dS have (4 g + 0..3 of either half)
    auto tr_frag_of = [&](int st) __attribute__((always_inline)) {
      return kv_tr_frag<D>(smem + ((cur + t_rd) ^ (uint32_t)((st % KG::DT) * 32)) + (st < KG::DT ? TB : 0u));
    };
    bf16x8_t tr[kTrWin];
#pragma unroll
    for (int st = 0; st < kTrAhead; ++st) tr[st] = tr_frag_of(st);
    fence();
    // Rows this key may not see: rows beyond the block, and (own block) tokens before the key; their P and
    // dS become 0 whatever the products gave.  Under one branch, which most tiles do not take.
    if (r0 + kKvRows > n_rows || (own && r0 < (kw0 + KG::KEYS - 1) * Gq)) {
      const int lo = own ? max(my_key * Gq - r0, 0) : 0;
      const uint32_t span = (uint32_t)max(n_rows - r0 - lo, 0);
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const bool hidden = (uint32_t)(rt * 16 + 4 * g + v - lo) >= span;
          x[rt][v] = hidden ? -INFINITY : x[rt][v];
          x[2 + rt][v] = hidden ? 0.f : x[2 + rt][v];
        }
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
      for (int v = 0; v < 4; ++v) x[rt][v] = __builtin_amdgcn_exp2f(x[rt][v]);
      x[2 + rt] *= x[rt];
    }
    const bf16x8_t pf = pack_rows(x[0], x[1]), dsf = pack_rows(x[2], x[3]);
#pragma unroll
    for (int st = kTrAhead; st < kTrWin; ++st) tr[st] = tr_frag_of(st);
    fence();
#pragma unroll
    for (int st = 0; st < 2 * KG::DT; ++st) {
      if (st < KG::DT) dv[st % KG::DT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr[st % kTrWin], pf, dv[st % KG::DT], 0, 0, 0);
      else dk[st % KG::DT] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tr[st % kTrWin], dsf, dk[st % KG::DT], 0, 0, 0);
      if (st + kTrWin < 2 * KG::DT) tr[st % kTrWin] = tr_frag_of(st + kTrWin);
      fence();
    }
  }

  // ---- epilogue: dV as it is; dk^ = ln 2 * acc (the q^ tiles carry scale * log2 e), turned back to dk
  //      with the key's entry of the pre-pass's table (which carries scale * log2 e once more); bf16,
  //      whole rows ------------------------------------------------------------------------------------
  wg_barrier();
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int ecol = ln & 15, eg = ln >> 4;
  if (n_splits > 1) {
    // (a shared walk: every wave leaves its sums, the last workgroup adds the splits up in their order)
    const int64_t slot = ((int64_t)(keytile - split * n_kt) * p.n_kv_heads + kvh) * kBWaves + wave;  // of split 0
    const int64_t step = (int64_t)n_kt * p.n_kv_heads * kBWaves;                                     // to the next
    char *const part = (char *)p.part_o;
    constexpr int kBytes = 32 * D * 4;  // of one wave: both sums of 16 keys
    static_assert(2 * KG::DT * 64 * 16 == kBytes, "a kilobyte per slab");
    if (wave_has_keys) {
      leave_sums(part + (slot + split * step) * kBytes, ln, 0, dv);
      leave_sums(part + (slot + split * step) * kBytes, ln, KG::DT, dk);
    }
    if (!last_of_splits(p.part_idx + (int64_t)(keytile - split * n_kt) * p.n_kv_heads + kvh, n_splits, smem + KG::LDS - 16)) return;
    if (wave_has_keys) {
#pragma unroll
      for (int dt = 0; dt < KG::DT; ++dt) dv[dt] = dk[dt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int s = 0; s < n_splits; ++s) add_sums(part + (slot + s * step) * kBytes, ln, dv, dk);
    }
  }
  rotate_back_keys<D>(dk, reinterpret_cast<const f32x4_t *>(p.q_table + (int64_t)(meta.pos0[b] + min(kw0 + ecol, lk - 1)) * D), eg,
                 p.rope_layout != 0, kLn2 / p.scale_log2e);
  static_assert(kBWaves * 2 * KG::KEYS * (size_t)ROWB <= KG::LDS, "the output staging fits");
  lds_char *stage = smem + wave * (2 * KG::KEYS * ROWB);  // this wave's rows of dV, then of dk
  stage_rows<D>(stage, dv, ecol, eg);
  stage_rows<D>(stage + KG::KEYS * ROWB, dk, ecol, eg);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int QRPI = 64 / KG::CPR;  // whole rows per store instruction
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    uint16_t *dst = t ? bp.dk : bp.dv;
    const int64_t st = t ? bp.dk_st : bp.dv_st, sh = t ? bp.dk_sh : bp.dv_sh;
#pragma unroll
    for (int u = 0; u < KG::KEYS / QRPI; ++u) {
      const int rr = u * QRPI + ln / KG::CPR;
      const u32x4_t w = *(const lds_u32x4 *)(stage + t * KG::KEYS * ROWB + kv_ofs<D>(rr, ln % KG::CPR));
      if (kw0 + rr < lk)
        *reinterpret_cast<u32x4_t *>(dst + (int64_t)(k_tok0 + kw0 + rr) * st + (int64_t)kvh * sh + (ln % KG::CPR) * 8) = w;
    }
  }
}

template <int D>
hipError_t launch_dkv_t(const AttnParams &p, const BwdKvMeta &meta, const BwdParams &bp, hipStream_t stream) {
  const int64_t n_wg = (int64_t)p.total_tiles * p.n_kv_heads;
  if (n_wg == 0) return hipSuccess;
  if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
  constexpr size_t lds = KvGeo<D>::LDS;
  static_assert(lds <= 64 * 1024, "fits the default dynamic LDS limit");
  if (meta.n_split > 0)
    hipLaunchKernelGGL((bwd_dkv_kernel<D, true>), dim3((unsigned)n_wg), dim3(kBThreads), lds, stream, p, meta, bp);
  else
    hipLaunchKernelGGL((bwd_dkv_kernel<D, false>), dim3((unsigned)n_wg), dim3(kBThreads), lds, stream, p, meta, bp);
  return hipGetLastError();
}

template <int D, bool kShared>
hipError_t launch_dq_t(const AttnParams &p, const PromptMeta &meta, const BwdParams &bp, hipStream_t stream) {
  const int64_t n_wg = (int64_t)p.total_tiles * p.n_kv_heads;
  if (n_wg == 0) return hipSuccess;
  if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
  constexpr size_t lds = (size_t)2 * kBBuf * BGeo<D>::TILEB;
  static_assert(lds <= 64 * 1024, "fits the default dynamic LDS limit");
  if (p.rows_past_cache)
    hipLaunchKernelGGL((bwd_dq_kernel<D, true, kShared>), dim3((unsigned)n_wg), dim3(kBThreads), lds, stream, p, meta, bp);
  else
    hipLaunchKernelGGL((bwd_dq_kernel<D, false, kShared>), dim3((unsigned)n_wg), dim3(kBThreads), lds, stream, p, meta, bp);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_dkv(const AttnParams &p, const BwdKvMeta &meta, const BwdParams &bp, hipStream_t stream) {
  if (p.head_dim == 128) return launch_dkv_t<128>(p, meta, bp, stream);
  if (p.head_dim == 64) return launch_dkv_t<64>(p, meta, bp, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_bwd_dq(const AttnParams &p, const PromptMeta &meta, const BwdParams &bp, hipStream_t stream) {
  const bool shared = meta.n_split > 0;
  if (p.head_dim == 128) return shared ? launch_dq_t<128, true>(p, meta, bp, stream) : launch_dq_t<128, false>(p, meta, bp, stream);
  if (p.head_dim == 64) return shared ? launch_dq_t<64, true>(p, meta, bp, stream) : launch_dq_t<64, false>(p, meta, bp, stream);
  return hipErrorInvalidValue;
}

}  // namespace ba
