// Device code of the two rotation passes (re-encoding of cached keys, RoPE pre-pass of fresh rows): each has kernels of
// its own, and the gather of a cached context runs both in one launch.
#pragma once

#include <type_traits>

#include "ba_device.h"

namespace ba {
namespace {

constexpr int kRotThreads = 256;

// 16 bytes of T as floats.  kLoadPast, kStorePast: they go past the caches.
template <typename T_, bool kLoadPast, bool kStorePast>
struct Chunk {
  typedef T_ T;
  static constexpr int VEC = 16 / sizeof(T);
  float f[VEC];
  __device__ __forceinline__ void load(const T *p) {
    const u32x4_t w = load_row_piece<kLoadPast>((const char *)p);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (VEC == 8) {
        f[2 * i] = bf16_lo(w[i]);
        f[2 * i + 1] = bf16_hi(w[i]);
      } else {
        f[i] = __uint_as_float(w[i]);
      }
    }
  }
  __device__ __forceinline__ void store(T *p) const {
    u32x4_t w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (VEC == 8)
        w[i] = pack_bf16(f[2 * i], f[2 * i + 1]);
      else
        w[i] = __float_as_uint(f[i]);
    }
    store_row_piece<kStorePast>((char *)p, w);
  }
};

// A launch has as many workgroups per block and layer as its longest block needs, and those of the shorter blocks find nothing
// to do.  Where one long block lies among many short ones these are nearly all, and starting them, four to five a
// nanosecond, is what the launch takes; two pieces per thread instead of eight make four times as many.  A launch of few
// workgroups does not feel them, nor one whose memory traffic takes as long: eight idle ones for each that works, and 32,768.
// Re-encoding, one block among n of 60 tokens at 8 heads of 128, two pieces / eight: 1,920 among 90 (42,000 idle) 14.5 / 14.5 us,
// 3,840 among 90 (85,000) 20.9 / 14.9; 480 among 500 (52,000 idle, 7,600 work) 22.8 / 27.4, 960 (112,000) 30.2 / 28.8,
// 3,840 (473,000) 105 / 42; 3,200 among 31 of 200, four layers (93,000, 9,400) 26.1 / 32.3, 6,400 (191,000, 12,600) 51.8 / 40.4.
inline bool mostly_idle(int64_t launched, int64_t needed) { return launched - needed > 32768 + 8 * needed; }

// y = R(angle) x on one (x, y) pair: [[c, -s], [s, c]] (Eq. 1 / Eq. 3).  Which product is the fused one is written out: left
// to the compiler it changes with the code around it, and with it the last bit of a key now and then.  (It did: packed fp32
// keys, a third of them, came out with other last bits than the same keys with strides.)
__device__ __forceinline__ float rot_x(float x, float y, float c, float s) { return __builtin_fmaf(c, x, -(s * y)); }
__device__ __forceinline__ float rot_y(float x, float y, float c, float s) { return __builtin_fmaf(s, x, c * y); }
__device__ __forceinline__ void rotate(float &a, float &b, float c, float s) {
  const float na = rot_x(a, b, c, s);
  b = rot_y(a, b, c, s);
  a = na;
}

// The block's entries of ReencRowsParams::row_table, by one workgroup.
template <typename Blocks>
__device__ __forceinline__ void write_row_table(const ReencRowsParams &p, const Blocks &blocks, int b) {
  const int len = blocks.len[b], at = blocks.dst_off[b];
  const int next = b + 1 < blocks.n ? blocks.dst_off[b + 1] : p.table_end;
  for (int u = threadIdx.x; u < next - at; u += kRotThreads)
    p.row_table[at + u] = (uint32_t)(blocks.src_off[b] + min(u, len - 1)) * p.row_bytes;
}

// Tokens of one block (workgroup bx of block b), any strides, any pairing, either mode.
template <typename Ch, int D, int LAYOUT, int MODE, int TOK_PER_WG, typename Params, typename Blocks>
__device__ __forceinline__ void reencode_tokens(const Params &p, const Blocks &blocks, const RopeTable &rt, uint32_t bx, int b, int layer) {
  typedef typename Ch::T T;
  constexpr int VEC = Ch::VEC;
  constexpr int CH = D / VEC;           // chunks per head vector
  constexpr int TPV = CH / 2;           // threads per head vector
  constexpr int TPP = kRotThreads / TPV;   // tokens per pass
  static_assert(TOK_PER_WG % TPP == 0, "tokens per workgroup must be whole passes");

  const int len = blocks.len[b];
  // bx = token chunk * head groups + head group: small inputs spread their heads over
  // more workgroups, large ones keep all heads in one thread so that sin/cos are reused
  const int hg = bx % p.n_head_groups;
  const int tok0 = (bx / p.n_head_groups) * TOK_PER_WG;
  if (tok0 >= len) return;

  const int c = threadIdx.x % TPV;
  const int tl = threadIdx.x / TPV;

  // frequencies of this thread's VEC pairs
  uint64_t turns[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    int j;
    if (LAYOUT == 0)  // interleaved: pairs live inside each chunk
      j = (e < VEC / 2) ? c * (VEC / 2) + e : (c + CH / 2) * (VEC / 2) + (e - VEC / 2);
    else  // half: element e of chunk c pairs with element e of chunk c + CH/2
      j = c * VEC + e;
    turns[e] = rt.turns[j];
  }

  const int shift0 = layer >= p.copy_from_layer ? 0 : blocks.pos_new[b] - blocks.pos_old[b];
  const T *src = static_cast<const T *>(p.src) + (int64_t)layer * p.src_sl +
                 (int64_t)blocks.src_off[b] * p.src_st;
  T *dst = static_cast<T *>(p.dst) + (int64_t)layer * p.dst_sl + (int64_t)blocks.dst_off[b] * p.dst_st;

  float cs[VEC], sn[VEC];
  if (MODE == 0) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) sincos_phase(rope_phase(shift0, turns[e]), cs[e], sn[e]);
  }
  // zero shift, or a layer that only rides along: bit-for-bit copy
  const bool plain_copy = ((MODE == 0) && (shift0 == 0)) || layer >= p.copy_from_layer;
  const int g_begin = hg * p.heads_per_thread;
  const int g_end = min(p.n_kv_heads, g_begin + p.heads_per_thread);

#pragma unroll 1
  for (int pass = 0; pass < TOK_PER_WG / TPP; ++pass) {
    const int u = tok0 + pass * TPP + tl;
    if (u >= len) break;
    if (MODE == 1) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) sincos_phase(rope_phase(shift0 + u, turns[e]), cs[e], sn[e]);
    }
    const T *s0 = src + (int64_t)u * p.src_st + c * VEC;
    T *d0 = dst + (int64_t)u * p.dst_st + c * VEC;
#pragma unroll 4
    for (int g = g_begin; g < g_end; ++g) {
      Ch x, y;
      x.load(s0 + g * p.src_sh);
      y.load(s0 + g * p.src_sh + (CH / 2) * VEC);
      if (!plain_copy) {
        if (LAYOUT == 0) {
#pragma unroll
          for (int e = 0; e < VEC / 2; ++e) {
            rotate(x.f[2 * e], x.f[2 * e + 1], cs[e], sn[e]);
            rotate(y.f[2 * e], y.f[2 * e + 1], cs[VEC / 2 + e], sn[VEC / 2 + e]);
          }
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) rotate(x.f[e], y.f[e], cs[e], sn[e]);
        }
      }
      x.store(d0 + g * p.dst_sh);
      y.store(d0 + g * p.dst_sh + (CH / 2) * VEC);
    }
  }
  if constexpr (std::is_same<Params, ReencRowsParams>::value)
    if (layer == 0 && bx == 0) write_row_table(p, blocks, b);
}

// Fast path: uniform shift (the angle depends on the block only), interleaved pairs (every pair
// lives inside one 16-byte chunk) and packed [tokens][heads][D] storage.  A block is then one
// contiguous run of chunks, and because the workgroup size is a multiple of the chunks per head
// vector, a thread that walks the run with stride 256 always meets the same four frequencies:
// a pure streaming pass, every wave instruction moving 1 KB of consecutive memory.
template <typename Ch, int D, int UNROLL, typename Params, typename Blocks>
__device__ __forceinline__ void reencode_run(const Params &p, const Blocks &blocks, const RopeTable &rt, uint32_t bx, int b, int layer) {
  typedef typename Ch::T T;
  constexpr int VEC = Ch::VEC;
  constexpr int CH = D / VEC;
  static_assert(kRotThreads % CH == 0, "a thread must keep its chunk position inside the head vector");
  const int64_t n_chunks = (int64_t)blocks.len[b] * p.n_kv_heads * CH;
  const int64_t first = (int64_t)bx * (UNROLL * kRotThreads) + threadIdx.x;
  if ((int64_t)bx * (UNROLL * kRotThreads) >= n_chunks) return;
  const int c = threadIdx.x % CH;
  const int shift0 = layer >= p.copy_from_layer ? 0 : blocks.pos_new[b] - blocks.pos_old[b];
  float cs[VEC / 2], sn[VEC / 2];
#pragma unroll
  for (int e = 0; e < VEC / 2; ++e) sincos_phase(rope_phase(shift0, rt.turns[c * (VEC / 2) + e]), cs[e], sn[e]);
  const T *src = static_cast<const T *>(p.src) + (int64_t)layer * p.src_sl + (int64_t)blocks.src_off[b] * p.src_st;
  T *dst = static_cast<T *>(p.dst) + (int64_t)layer * p.dst_sl + (int64_t)blocks.dst_off[b] * p.dst_st;
  Ch x[UNROLL];
#pragma unroll
  for (int k = 0; k < UNROLL; ++k) {
    const int64_t L = first + (int64_t)k * kRotThreads;
    if (L < n_chunks) x[k].load(src + L * VEC);
  }
  if (shift0 != 0) {  // zero shift: bit-for-bit copy
#pragma unroll
    for (int k = 0; k < UNROLL; ++k)
#pragma unroll
      for (int e = 0; e < VEC / 2; ++e) rotate(x[k].f[2 * e], x[k].f[2 * e + 1], cs[e], sn[e]);
  }
#pragma unroll
  for (int k = 0; k < UNROLL; ++k) {
    const int64_t L = first + (int64_t)k * kRotThreads;
    if (L < n_chunks) x[k].store(dst + L * VEC);
  }
  if constexpr (std::is_same<Params, ReencRowsParams>::value)
    if (layer == 0 && bx == 0) write_row_table(p, blocks, b);
}

// ---- RoPE pre-pass -------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t rotated(float x, float y, float c, float s) {
  return pack_bf16(rot_x(x, y, c, s), rot_y(x, y, c, s));
}

// workgroup rows of the Q job: head groups, or one row when only the table of factors is written
__host__ __device__ inline int q_groups(const RopePrepassParams &p) {
  return p.do_q == 1 ? (p.n_q_heads + p.heads_per_thread - 1) / p.heads_per_thread : (p.do_q ? 1 : 0);
}

// Rows of Q head groups, then K head groups (by), kRotThreads / (D / 16) tokens each (bx).
template <int D, int LAYOUT, typename Segs>
__device__ __forceinline__ void rope_prepass_rows(const RopePrepassParams &p, const Segs &segs, const RopeTable &rt, int bx, int by) {
  constexpr int VEC = 8;
  constexpr int CH = D / VEC;
  constexpr int TPV = CH / 2;          // threads per head vector
  constexpr int TPP = kRotThreads / TPV;  // tokens per workgroup
  const int c = threadIdx.x % TPV;
  // which tensor and which heads this workgroup handles: Q head groups first, then K
  const int groups_q = q_groups(p);
  const bool is_q = by < groups_q;
  int t = segs.start[0] + bx * TPP + threadIdx.x / TPV;
  int pos;
  if (is_q && p.do_q == 2) {
    // the table of factors: this thread's row is a position, not a token
    t = bx * TPP + threadIdx.x / TPV;
    if (t >= p.table_rows) return;
    pos = t;
  } else {
    if (t >= segs.start[segs.n]) return;
    int lo = 0, hi = segs.n;  // largest s with start[s] <= t
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (segs.start[mid] <= t) lo = mid; else hi = mid;
    }
    pos = segs.pos0[lo] + (t - segs.start[lo]);
  }
  const int grp = is_q ? by : by - groups_q;
  const int n_heads = is_q ? p.n_q_heads : p.n_kv_heads;
  const int h_begin = grp * p.heads_per_thread;
  const int h_end = min(n_heads, h_begin + p.heads_per_thread);
  const uint16_t *src = (is_q ? p.q_src : p.k_src) + (int64_t)t * (is_q ? p.q_st : p.k_st) + c * VEC;
  uint16_t *dst = (is_q ? p.q_dst : p.k_dst) + (int64_t)t * (is_q ? p.qd_st : p.kd_st) + c * VEC;
  const int64_t src_sh = is_q ? p.q_sh : p.k_sh, dst_sh = is_q ? p.qd_sh : p.kd_sh;
  const float scale = is_q ? p.q_scale : 1.0f;

  float cs[VEC], sn[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    int j;
    if (LAYOUT == 0)  // interleaved: pairs live inside each chunk
      j = (e < VEC / 2) ? c * (VEC / 2) + e : (c + CH / 2) * (VEC / 2) + (e - VEC / 2);
    else  // half: element e of chunk c pairs with element e of chunk c + CH/2
      j = c * VEC + e;
    sincos_phase(rope_phase(pos, rt.turns[j]), cs[e], sn[e]);
    if (scale != 1.0f) {
      cs[e] *= scale;
      sn[e] *= scale;
    }
  }
  if (is_q && p.do_q == 2) {
    // the factors themselves, for the attention core to rotate q with: entry j at [position][j] = (cos, sin)
    float2 *row = reinterpret_cast<float2 *>(p.q_table) + (int64_t)t * (D / 2);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      int j;
      if (LAYOUT == 0)
        j = (e < VEC / 2) ? c * (VEC / 2) + e : (c + CH / 2) * (VEC / 2) + (e - VEC / 2);
      else
        j = c * VEC + e;
      row[j] = make_float2(cs[e], sn[e]);
    }
    return;
  }
#pragma unroll 4
  for (int h = h_begin; h < h_end; ++h) {
    const u32x4_t xa = *reinterpret_cast<const u32x4_t *>(src + h * src_sh);
    const u32x4_t xb = *reinterpret_cast<const u32x4_t *>(src + h * src_sh + (CH / 2) * VEC);
    u32x4_t ya, yb;
    if (LAYOUT == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a0 = bf16_lo(xa[e]), a1 = bf16_hi(xa[e]);
        ya[e] = rotated(a0, a1, cs[e], sn[e]);
        const float b0 = bf16_lo(xb[e]), b1 = bf16_hi(xb[e]);
        yb[e] = rotated(b0, b1, cs[4 + e], sn[4 + e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a0 = bf16_lo(xa[e]), a1 = bf16_hi(xa[e]), b0 = bf16_lo(xb[e]), b1 = bf16_hi(xb[e]);
        ya[e] = pack_bf16(rot_x(a0, b0, cs[2 * e], sn[2 * e]), rot_x(a1, b1, cs[2 * e + 1], sn[2 * e + 1]));
        yb[e] = pack_bf16(rot_y(a0, b0, cs[2 * e], sn[2 * e]), rot_y(a1, b1, cs[2 * e + 1], sn[2 * e + 1]));
      }
    }
    *reinterpret_cast<u32x4_t *>(dst + h * dst_sh) = ya;
    *reinterpret_cast<u32x4_t *>(dst + h * dst_sh + (CH / 2) * VEC) = yb;
  }
}

}  // namespace
}  // namespace ba
