// Gather of a context of short cached blocks and RoPE pre-pass of the query block behind it, in one launch.
//
// The two are independent of each other and the attention core waits for both.  The pre-pass is 4 us of latency for a few
// hundred kilobytes of rows; as the first workgroups of the gather's launch it is done before the gather is, and a
// dependent launch is saved: 8 blocks of 46 to 138 tokens, 16 over 8 heads of 128, 25.5 -> 19.5 us, 25 calls of 100 to 20,000
// context tokens 0.76 to 0.98 of the time.
// The gather is bound by memory and by how fast it gets going.  What it writes is read by the next kernel and what it
// reads may still be in the caches, so neither goes past them, and a thread moves two pieces, not eight (four times the
// workgroups): 512 blocks of 20 to 60 tokens, 32 over 8 heads of 128, 42 MB in and out: the call 61.7 -> 54.3 us (57.7 -> 46.6 on
// one cache over and over; contexts of that size are mostly not copied any more, see FinalTurnMeta).  (On one box, where two
// pieces took 52.1: four 56, with the hint 59; one piece 50, at twice the workgroups where block lengths differ.)
#include <string.h>

#include "ba_rotate.h"
#include "ba_schedule.h"

namespace ba {
namespace {

constexpr int kUnroll = 2;  // 16-byte pieces of a run per thread
constexpr int kWgPieces = kUnroll * kRotThreads;

struct GatherGrid {
  uint32_t n_pre, pre_x;  // workgroups of the pre-pass, and of one of its head groups
  FastDiv pre_div;        // division by pre_x
  uint32_t x;             // workgroups per block and layer of the gather
  FastDiv x_div;
};

// kRuns: packed keys of interleaved pairs, where a block is one run of 16-byte pieces
template <int D, int LAYOUT, bool kRuns, typename Params, typename Blocks>
__global__ __launch_bounds__(kRotThreads) void gather_prepass_kernel(Params gp, Blocks blocks, RopePrepassParams pp,
                                                                     RopeSegsGather segs, RopeTable rt, GatherGrid g) {
  uint32_t id = blockIdx.x;
  if (id < g.n_pre) {
    const uint32_t by = fast_div(id, g.pre_div);
    rope_prepass_rows<D, LAYOUT>(pp, segs, rt, (int)(id - by * g.pre_x), (int)by);
    return;
  }
  id -= g.n_pre;
  const uint32_t row = fast_div(id, g.x_div);
  const uint32_t bx = id - row * g.x;
  const int layer = (int)row >= blocks.n ? 1 : 0, b = (int)row - layer * blocks.n;
  if constexpr (kRuns)
    reencode_run<Chunk<uint16_t, false, false>, D, kUnroll>(gp, blocks, rt, bx, b, layer);
  else
    reencode_tokens<Chunk<uint16_t, false, false>, D, LAYOUT, 0, kRotThreads / (D / 16)>(gp, blocks, rt, bx, b, layer);
}

// packed keys of interleaved pairs
template <typename Params>
bool is_runs(const Params &gp) {
  const int64_t D = gp.head_dim, row = gp.n_kv_heads * D;
  return gp.layout == 0 && gp.src_sh == D && gp.dst_sh == D && gp.src_st == row && gp.dst_st == row;
}

// the grid, and how many workgroups it has in all
template <typename Params, typename Blocks>
int64_t make_grid(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs, GatherGrid *g) {
  const int TPP = kRotThreads / (gp.head_dim / 16);  // tokens per workgroup, of either pass
  const int64_t pre_x = ((int64_t)segs.start[segs.n] - segs.start[0] + TPP - 1) / TPP;
  const int64_t n_pre = pre_x * (q_groups(pp) + (pp.n_kv_heads + pp.heads_per_thread - 1) / pp.heads_per_thread);
  const int64_t x = is_runs(gp) ? ((int64_t)gp.max_len * gp.n_kv_heads * (gp.head_dim / 8) + kWgPieces - 1) / kWgPieces
                                : ((int64_t)gp.max_len + TPP - 1) / TPP * gp.n_head_groups;
  g->pre_x = (uint32_t)pre_x;
  g->n_pre = (uint32_t)n_pre;
  g->x = (uint32_t)x;
  return n_pre + x * blocks.n * gp.n_layers;
}

template <int D, int LAYOUT, bool kRuns, typename Params, typename Blocks>
hipError_t launch_t(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                    const RopeTable &rt, hipStream_t stream) {
  GatherGrid g;
  const int64_t n_wg = make_grid(gp, blocks, pp, segs, &g);
  if (g.pre_x == 0 || g.x == 0 || gp.n_layers > 2) return hipErrorInvalidValue;
  g.pre_div = make_fast_div(g.pre_x);
  g.x_div = make_fast_div(g.x);
  hipLaunchKernelGGL((gather_prepass_kernel<D, LAYOUT, kRuns, Params, Blocks>), dim3((unsigned)n_wg), dim3(kRotThreads), 0, stream,
                     gp, blocks, pp, segs, rt, g);
  return hipGetLastError();
}

template <int D, typename Params, typename Blocks>
hipError_t launch_d(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                    const RopeTable &rt, hipStream_t stream) {
  if (gp.layout != 0) return launch_t<D, 1, false>(gp, blocks, pp, segs, rt, stream);
  return is_runs(gp) ? launch_t<D, 0, true>(gp, blocks, pp, segs, rt, stream) : launch_t<D, 0, false>(gp, blocks, pp, segs, rt, stream);
}

// The tables with which the attention kernel fetches and turns the cached keys itself (FinalTurnMeta), a workgroup per block, next to
// the pre-pass.  A few hundred kilobytes at most: latency.
template <int D, int LAYOUT, typename Blocks>
__global__ __launch_bounds__(kRotThreads) void turn_tables_kernel(TurnTables tt, Blocks blocks, RopePrepassParams pp,
                                                                  RopeSegsGather segs, RopeTable rt, GatherGrid g) {
  if (blockIdx.x < g.n_pre) {
    const uint32_t by = fast_div(blockIdx.x, g.pre_div);
    rope_prepass_rows<D, LAYOUT>(pp, segs, rt, (int)(blockIdx.x - by * g.pre_x), (int)by);
    return;
  }
  const int b = (int)(blockIdx.x - g.n_pre);
  const int len = blocks.len[b], at = blocks.dst_off[b], src = blocks.src_off[b];
  const int next = b + 1 < blocks.n ? blocks.dst_off[b + 1] : tt.table_end;
  const int shift = blocks.pos_new[b] - blocks.pos_old[b];
  for (int u = threadIdx.x; u < next - at; u += kRotThreads) {
    tt.rows[at + u] = (uint32_t)(src + min(u, len - 1)) * tt.row_bytes;
    tt.blk[at + u] = (uint32_t)b | (shift == 0 ? kTurnPlain : 0u);
  }
  if ((int)threadIdx.x < D / 2) {
    float c, s;
    sincos_phase(rope_phase(shift, rt.turns[threadIdx.x]), c, s);
    reinterpret_cast<float2 *>(tt.rot)[b * (D / 2) + (int)threadIdx.x] = make_float2(c, s);
  }
}

template <int D, typename Blocks>
hipError_t launch_turn_d(const TurnTables &tt, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                         const RopeTable &rt, hipStream_t stream) {
  constexpr int TPP = kRotThreads / (D / 16);
  GatherGrid g;
  memset(&g, 0, sizeof(g));
  g.pre_x = (uint32_t)(((int64_t)segs.start[segs.n] - segs.start[0] + TPP - 1) / TPP);
  if (g.pre_x == 0) return hipErrorInvalidValue;
  g.n_pre = g.pre_x * (uint32_t)(q_groups(pp) + (pp.n_kv_heads + pp.heads_per_thread - 1) / pp.heads_per_thread);
  g.pre_div = make_fast_div(g.pre_x);
  const dim3 grid(g.n_pre + (unsigned)blocks.n);
  if (pp.layout == 0)
    hipLaunchKernelGGL((turn_tables_kernel<D, 0, Blocks>), grid, dim3(kRotThreads), 0, stream, tt, blocks, pp, segs, rt, g);
  else
    hipLaunchKernelGGL((turn_tables_kernel<D, 1, Blocks>), grid, dim3(kRotThreads), 0, stream, tt, blocks, pp, segs, rt, g);
  return hipGetLastError();
}

}  // namespace

template <typename Blocks>
hipError_t launch_turn_tables(const TurnTables &tt, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                              const RopeTable &rt, hipStream_t stream) {
  if (pp.head_dim == 128) return launch_turn_d<128>(tt, blocks, pp, segs, rt, stream);
  if (pp.head_dim == 64) return launch_turn_d<64>(tt, blocks, pp, segs, rt, stream);
  return hipErrorInvalidValue;
}
template hipError_t launch_turn_tables(const TurnTables &, const ReencBlocks &, const RopePrepassParams &, const RopeSegsGather &, const RopeTable &, hipStream_t);
template hipError_t launch_turn_tables(const TurnTables &, const ReencBlocksLarge &, const RopePrepassParams &, const RopeSegsGather &, const RopeTable &, hipStream_t);

// Where the two are one launch.  Not where one long block lies among many short ones and the launch would be mostly_idle (or, further
// on, beyond the 2^32 threads that the runtime launches in the one dimension used here): the re-encode kernels have the
// eight pieces a thread for that, and an idle workgroup costs less with their arguments.  One block among n of 30 tokens, 8
// heads of 128, together / apart: 700 among 255 (43,000 idle, 2,400 work) 38.6 / 43, 1,000 (62,000) 42.3 / 41.8, 3,000 (190,000) 73.7 / 49.3;
// 400 among 1,023 (93,000, 8,800) 73.9 / 73.1, 1,000 (247,000) 107 / 81; half pairs 1,000 among 255 53.8 / 55, 3,000 47.3 / 44.9.
// And not where it reads and writes more than the cache holds: plain loads and stores lose there.  1,024 blocks, together / apart, also with
// four such caches in turn: of 60 tokens (252 MB) 111 / 117, of 80 (336 MB) 148 / 146, of 130 233 / 227, of 200 350 / 336; half pairs 110 / 115,
// 147 / 150, 242 / 232, 363 / 342.
template <typename Params, typename Blocks>
bool gather_takes_prepass(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs) {
  GatherGrid g;
  const int64_t n_wg = make_grid(gp, blocks, pp, segs, &g);
  int64_t tokens = 0;
  for (int b = 0; b < blocks.n; ++b) tokens += blocks.len[b];
  const int64_t pieces = tokens * gp.n_kv_heads * (gp.head_dim / 8);  // of 16 bytes, of one layer
  const int64_t needed = (is_runs(gp) ? pieces / kWgPieces + blocks.n : (tokens / (kRotThreads / (gp.head_dim / 16)) + blocks.n) * gp.n_head_groups) * gp.n_layers;
  return n_wg * kRotThreads <= 0xffffffffll && !mostly_idle(n_wg - g.n_pre, needed) && pieces * gp.n_layers * 32 <= kCacheBytes;
}

template <typename Params, typename Blocks>
hipError_t launch_gather_prepass(const Params &gp, const Blocks &blocks, const RopePrepassParams &pp, const RopeSegsGather &segs,
                                 const RopeTable &rt, hipStream_t stream) {
  if (gp.head_dim == 128) return launch_d<128>(gp, blocks, pp, segs, rt, stream);
  if (gp.head_dim == 64) return launch_d<64>(gp, blocks, pp, segs, rt, stream);
  return hipErrorInvalidValue;
}

template bool gather_takes_prepass(const ReencParams &, const ReencBlocks &, const RopePrepassParams &, const RopeSegsGather &);
template hipError_t launch_gather_prepass(const ReencParams &, const ReencBlocks &, const RopePrepassParams &, const RopeSegsGather &, const RopeTable &, hipStream_t);
template bool gather_takes_prepass(const ReencParams &, const ReencBlocksLarge &, const RopePrepassParams &, const RopeSegsGather &);
template hipError_t launch_gather_prepass(const ReencParams &, const ReencBlocksLarge &, const RopePrepassParams &, const RopeSegsGather &, const RopeTable &, hipStream_t);
template bool gather_takes_prepass(const ReencRowsParams &, const ReencBlocks &, const RopePrepassParams &, const RopeSegsGather &);
template hipError_t launch_gather_prepass(const ReencRowsParams &, const ReencBlocks &, const RopePrepassParams &, const RopeSegsGather &, const RopeTable &, hipStream_t);
template bool gather_takes_prepass(const ReencRowsParams &, const ReencBlocksLarge &, const RopePrepassParams &, const RopeSegsGather &);
template hipError_t launch_gather_prepass(const ReencRowsParams &, const ReencBlocksLarge &, const RopePrepassParams &, const RopeSegsGather &, const RopeTable &, hipStream_t);

}  // namespace ba
