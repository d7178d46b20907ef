// Device-side helpers shared by the attention kernels: LDS-direct tile loads and the waits and
// barriers that go with them, the half-wave exchange, and the search in a table of tile starts.
#pragma once

#include <type_traits>

#include "ba_device.h"

namespace ba {

__device__ __forceinline__ int find_segment(const int32_t *tile_start, int n, int tile) {
  int lo = 0, hi = n;  // largest i with tile_start[i] <= tile
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (tile_start[mid] <= tile) lo = mid; else hi = mid;
  }
  return lo;
}

// The same in a table of kEncMaxBlocks + 1 tile starts whose entries past the last block hold INT_MAX, so
// that no candidate needs a bounds check: the number of starts behind the first that are at or below the tile, a lane
// per start and five loads that go out together.  It is the first link of the chain that a short work item spends most of its
// time in (table, block, query rows, walk, store), and was three dependent rounds of scalar loads: forward and backward of small
// calls 0.96 to 0.98 of the time, of calls that fill the chip 0.98 to 0.99, the encode kernel of two blocks of 128 tokens 8.9 -> 8.3 us
// (its call by less than two runs of it differ).
// (In the main core's tables of prompts and blocks it changes nothing: 20 calls 1.003.)
__device__ __forceinline__ int find_block(const int32_t *tile_start, int tile) {
  static_assert(kEncMaxBlocks == 5 * 64, "a lane per start");
  const int lane = threadIdx.x & 63;
  int start[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) start[k] = tile_start[1 + k * 64 + lane];
  int b = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) b += __builtin_popcountll(__builtin_amdgcn_ballot_w64(start[k] <= tile));
  return b;
}

__device__ __forceinline__ float other_half(float x) {
  // value held by lane ^ 32, combined with ours by the caller
  uint32_t u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return (threadIdx.x & 32) ? __uint_as_float(r[0]) : __uint_as_float(r[1]);
}

typedef __attribute__((address_space(3))) char lds_char;

// LDS-direct load: every lane fetches 16 bytes from base + offset and the wave writes them to
// LDS bytes [lds_base + 16 lane, +16).  Issued through inline assembly ON PURPOSE: the compiler
// would otherwise treat the copy as a store that may alias every later LDS read and wait for
// it (vmcnt(0)) before the first fragment read of the same iteration, which exposes the whole
// HBM latency on every tile.  The price is that completion is ours to wait for: a dma_wait
// must come before the barrier that publishes the buffer.
__device__ __forceinline__ void lds_dma16(const char *base, uint32_t offset, uint32_t lds_base) {
  // base and lds_base are wave-uniform by construction; say so, or a value the compiler cannot
  // prove uniform would not fit the scalar operands
  const uint64_t b = (uint64_t)base;
  const uint64_t bu = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  base = (const char *)bu;
  lds_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_base);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(offset), "s"(base), "s"(lds_base)
               : "memory");
}
// Workgroup barrier without the memory fence of __syncthreads(): LDS reads that are still in flight
// (fragments requested ahead of their use) need not drain first.  What a barrier publishes here are
// LDS-direct copies, and the copying wave has waited for those (dma_wait) before it arrives.
// (Written as assembly so that the compiler does not drain the LDS counter in front of it.)
__device__ __forceinline__ void wg_barrier() {
  asm volatile("s_barrier" ::: "memory");
}
// Wait until this wave's LDS writes (and reads) have been done, ahead of a wg_barrier that publishes them.
__device__ __forceinline__ void lds_wait() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Query rows in fragment layout (lane = row; fragment kk holds 16-byte chunk 2 kk + hf) times the row's
// entry of the pre-pass's table of (cos, sin) times some factor, rounded once.  The table row's 16-byte
// pieces that a lane needs, in the order of `cs`: fragment_table_piece(j, ...).  Interleaved pairs: fragment kk
// holds pairs kk * 8 + hf * 4 + (0..3); half-split pairs: fragments kk and kk + KCH/2 hold dims
// kk * 16 + hf * 8 + (0..7) and their partners, i.e. pairs of those same numbers.  (Which product is the
// fused one is written out: left to the compiler it changes with the code around it, and the forward and
// the backward pass are to see the same rows.  kAsCore: the choice that the main core's rotation compiles to,
// which differs for the second member of an interleaved pair.)
__device__ __forceinline__ int fragment_table_piece(int j, int hf, bool halves) {
  return halves ? (j / 4) * 8 + (j & 3) + hf * 4 : (j / 2) * 4 + (j & 1) + hf * 2;
}
template <int KCH, bool kAsCore = false>
__device__ __forceinline__ void rotate_fragments(u32x4_t (&raw)[KCH], const f32x4_t (&cs)[2 * KCH], bool halves) {
  if (!halves) {
#pragma unroll
    for (int kk = 0; kk < KCH; ++kk) {
      const f32x4_t cs0 = cs[2 * kk], cs1 = cs[2 * kk + 1];
      const float c[4] = {cs0[0], cs0[2], cs1[0], cs1[2]}, sn[4] = {cs0[1], cs0[3], cs1[1], cs1[3]};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = bf16_lo(raw[kk][e]), y = bf16_hi(raw[kk][e]);
        raw[kk][e] = pack_bf16(__builtin_fmaf(c[e], x, -(sn[e] * y)),
                               kAsCore ? __builtin_fmaf(sn[e], x, c[e] * y) : __builtin_fmaf(c[e], y, sn[e] * x));
      }
    }
  } else {
#pragma unroll
    for (int kk = 0; kk < KCH / 2; ++kk) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const f32x4_t t = cs[4 * kk + e];  // pairs kk * 16 + hf * 8 + 2 e and the next
        const float c0 = t[0], s0 = t[1], c1 = t[2], s1 = t[3];
        const uint32_t wa = raw[kk][e], wb = raw[kk + KCH / 2][e];
        const float xa0 = bf16_lo(wa), xa1 = bf16_hi(wa), xb0 = bf16_lo(wb), xb1 = bf16_hi(wb);
        raw[kk][e] = pack_bf16(__builtin_fmaf(c0, xa0, -(s0 * xb0)), __builtin_fmaf(c1, xa1, -(s1 * xb1)));
        raw[kk + KCH / 2][e] = pack_bf16(__builtin_fmaf(s0, xa0, c0 * xb0), __builtin_fmaf(s1, xa1, c1 * xb1));
      }
    }
  }
}

// Sum over each run of N consecutive lanes (8 or 16), in every lane of the run: adds of neighbours
// through the vector unit's own lane permutations, no trip through LDS.
template <int N>
__device__ __forceinline__ float sum_over_lanes(float x) {
  static_assert(N == 8 || N == 16, "runs inside one row of sixteen lanes");
  auto add = [&](auto ctrl) __attribute__((always_inline)) {
    x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  add(std::integral_constant<int, 0xb1>{});   // lane ^ 1
  add(std::integral_constant<int, 0x4e>{});   // lane ^ 2
  add(std::integral_constant<int, 0x141>{});  // the other four of eight (mirrored: they all hold one sum)
  if constexpr (N == 16) add(std::integral_constant<int, 0x140>{});  // the other eight of sixteen
  return x;
}

// Wait until at most NEWER of this wave's vector-memory operations are still in flight
// (they complete in order), leaving the other counters alone.  gfx9 encoding of s_waitcnt.
template <int NEWER>
__device__ __forceinline__ void dma_wait() {
  static_assert(NEWER >= 0 && NEWER < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (NEWER & 15) | ((NEWER >> 4) << 14));
  asm volatile("" ::: "memory");
}

// Chunks c and c + CPR / 2 of a row of keys, turned.  t: the pieces of the row's (cos, sin) that the two need -- interleaved pairs: pairs
// 4 c .. 4 c + 3 lie in the first chunk, 4 (c + CPR / 2) .. in the other; half-split: element e of the one pairs with element e of
// the other, pairs 8 c .. 8 c + 7.
__device__ __forceinline__ void turn_chunks(const u32x4_t &a, const u32x4_t &b, const f32x4_t (&t)[4], bool halves, u32x4_t &ya, u32x4_t &yb) {
  auto x_of = [](float x, float y, float c, float s) { return __builtin_fmaf(c, x, -(s * y)); };
  auto y_of = [](float x, float y, float c, float s) { return __builtin_fmaf(s, x, c * y); };
  if (!halves) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float ca = t[e / 2][(e & 1) * 2], sa = t[e / 2][(e & 1) * 2 + 1], cb = t[2 + e / 2][(e & 1) * 2], sb = t[2 + e / 2][(e & 1) * 2 + 1];
      ya[e] = pack_bf16(x_of(bf16_lo(a[e]), bf16_hi(a[e]), ca, sa), y_of(bf16_lo(a[e]), bf16_hi(a[e]), ca, sa));
      yb[e] = pack_bf16(x_of(bf16_lo(b[e]), bf16_hi(b[e]), cb, sb), y_of(bf16_lo(b[e]), bf16_hi(b[e]), cb, sb));
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a0 = bf16_lo(a[e]), a1 = bf16_hi(a[e]), b0 = bf16_lo(b[e]), b1 = bf16_hi(b[e]);
      ya[e] = pack_bf16(x_of(a0, b0, t[e][0], t[e][1]), x_of(a1, b1, t[e][2], t[e][3]));
      yb[e] = pack_bf16(y_of(a0, b0, t[e][0], t[e][1]), y_of(a1, b1, t[e][2], t[e][3]));
    }
  }
}

// ---- row tiles whose walk several workgroups share (PromptMeta::n_split): each leaves its accumulators in
//      32 bits, in the layout they have (1 KB of consecutive memory per wave instruction), and the one that
//      is last to count itself in adds them up in the order of the splits --------------------------------
constexpr int kSplitWaves = kShortTileRows / 32;
template <int D>
__device__ __forceinline__ void leave_accumulators(float *part, int64_t slot, int lane, const f32x16_t (&acc)[D / 32]) {
  const auto to = shared_buffer((char *)part + slot * (32 * D * 4), 32 * D * 4);
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      u32x4_t w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(acc[dt][q4 * 4 + e]);
      __builtin_amdgcn_raw_buffer_store_b128(w, to, lane * 16 + (dt * 4 + q4) * 1024, 0, kAgentScope);
    }
}
template <int D>
__device__ __forceinline__ void fetch_accumulators(float *part, int64_t slot, int lane, u32x4_t (&w)[D / 8]) {
  const auto from = shared_buffer((char *)part + slot * (32 * D * 4), 32 * D * 4);
#pragma unroll
  for (int k = 0; k < D / 8; ++k)
    w[k] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(from, lane * 16 + k * 1024, 0, kAgentScope));
}
// Which split of a shared walk a row tile of the launch's list is: n_row_tiles of the block, n_splits times over.
struct WalkSplit {
  int n_row_tiles, n_splits, split;
};
__device__ __forceinline__ WalkSplit walk_split_of(int n_rows, int tile, int n_tiles) {
  WalkSplit w;
  w.n_row_tiles = (n_rows + kShortTileRows - 1) / kShortTileRows;
  w.n_splits = n_tiles / w.n_row_tiles;
  w.split = tile / w.n_row_tiles;
  return w;
}
// Counts this workgroup in; true (in every wave) if all n are in now.  told: a word of LDS nobody else uses.
__device__ __forceinline__ bool last_of_splits(int32_t *counter, int n, lds_char *told_at) {
  __attribute__((address_space(3))) volatile int *const told = (__attribute__((address_space(3))) volatile int *)told_at;
  dma_wait<0>();  // this wave's stores have left its XCD
  wg_barrier();   // every wave's have
  if (threadIdx.x == 0) {
    *told = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    lds_wait();
  }
  wg_barrier();
  return __builtin_amdgcn_readfirstlane(*told) == n;
}

}  // namespace ba
