// Position re-encoding of cached keys (Section 2.3 of arXiv 2409.15355): the two
// rotations of Eq. 2 and Eq. 3 collapse into one rotation by the position difference,
// applied here as a single coalesced HBM pass: 16-byte loads, fp32 rotate, 16-byte
// stores.  Memory-bound: 2 B read + 2 B written per bf16 element.
//
// Thread mapping.  A head vector of D elements is CH = D / VEC 16-byte chunks.  A
// thread owns chunk c and chunk c + CH/2 of one token and walks over that token's KV
// heads, so its VEC (cos, sin) pairs are computed once per token (ABSOLUTE mode) or
// once per workgroup (SHIFT mode: the angle depends on the block only) and reused for
// every head.  CH/2 neighbouring lanes cover half a head vector contiguously.
#include <type_traits>

#include "ba_rotate.h"

namespace ba {
namespace {

template <typename Ch, int D, int LAYOUT, int MODE, int TOK_PER_WG, typename Params, typename Blocks>
__global__ __launch_bounds__(kRotThreads) void reencode_kernel(Params p, Blocks blocks, RopeTable rt) {
  reencode_tokens<Ch, D, LAYOUT, MODE, TOK_PER_WG>(p, blocks, rt, blockIdx.x, (int)blockIdx.y, (int)blockIdx.z);
}

template <typename Ch, int D, int UNROLL, typename Params, typename Blocks>
__global__ __launch_bounds__(kRotThreads) void reencode_shift_linear_kernel(Params p, Blocks blocks, RopeTable rt) {
  reencode_run<Ch, D, UNROLL>(p, blocks, rt, blockIdx.x, (int)blockIdx.y, (int)blockIdx.z);
}

template <typename Ch, int D, int UNROLL, typename Params, typename Blocks>
dim3 linear_grid(const Params &p, const Blocks &blocks) {
  const int64_t max_chunks = (int64_t)p.max_len * p.n_kv_heads * (D / Ch::VEC);
  return dim3((unsigned)((max_chunks + UNROLL * kRotThreads - 1) / (UNROLL * kRotThreads)), blocks.n, p.n_layers);
}
template <typename Ch, int D, int UNROLL, typename Params, typename Blocks>
hipError_t launch_linear(const Params &p, const Blocks &blocks, const RopeTable &rt, dim3 grid, hipStream_t stream) {
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return hipSuccess;
  hipLaunchKernelGGL((reencode_shift_linear_kernel<Ch, D, UNROLL, Params, Blocks>), grid, dim3(kRotThreads), 0, stream, p, blocks, rt);
  return hipGetLastError();
}

template <typename Ch, int D, int LAYOUT, int MODE, typename Params, typename Blocks>
hipError_t launch_t(const Params &p, const Blocks &blocks, const RopeTable &rt, hipStream_t stream) {
  constexpr int TPP = kRotThreads / (D / Ch::VEC / 2);
  constexpr int TOK_PER_WG = TPP;
  dim3 grid(((p.max_len + TOK_PER_WG - 1) / TOK_PER_WG) * p.n_head_groups, blocks.n, p.n_layers);
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return hipSuccess;
  hipLaunchKernelGGL((reencode_kernel<Ch, D, LAYOUT, MODE, TOK_PER_WG, Params, Blocks>), grid, dim3(kRotThreads), 0,
                     stream, p, blocks, rt);
  return hipGetLastError();
}

// Which loads and how much per thread, by the bytes of a launch (read and written).  The rotated keys go past the caches, but
// the keys as cached may still lie there.  Time with plain loads / with the hint, one cache re-encoded over and over and
// eight in turn (880 MB to 2 GB, nothing of which is found again):
//   - runs, two pieces per thread instead of eight (four times the workgroups): 157 MB 0.78 and 0.92, 128 MB 0.74 and 0.87
//     (of that the two pieces alone 0.87 and 0.90, 0.80 and 0.84); 412 MB 1.00 and 1.00.  In launches beyond the cache eight,
//     and where a launch is mostly_idle, with the hint as beyond the cache.
//   - the others: 39 MB 0.91 and 0.90, 45 MB 0.96 and 0.84; but 110 MB 0.87 and 1.02, 157 MB 0.87 and 1.03, 262 MB 0.86 and
//     1.02, and with three in turn 262 MB is 1.02 as well: plain up to a quarter of the cache.
// (By launch, not by call: eight caches in turn are what a longer list is, several launches of such a size.)
template <typename T, int D, typename Params, typename Blocks>
hipError_t launch_d(const Params &p, const Blocks &blocks, const RopeTable &rt, hipStream_t stream) {
  typedef Chunk<T, true, true> Past;
  typedef Chunk<T, false, true> Near;
  const bool packed = p.src_sh == D && p.dst_sh == D && p.src_st == (int64_t)p.n_kv_heads * D &&
                      p.dst_st == (int64_t)p.n_kv_heads * D;
  int64_t tokens = 0;
  for (int i = 0; i < blocks.n; ++i) tokens += blocks.len[i];
  const int64_t bytes = tokens * p.n_layers * p.n_kv_heads * D * (int64_t)sizeof(T) * 2;
  if (p.layout == 0 && p.mode == 0 && packed) {
    const dim3 two = linear_grid<Near, D, 2>(p, blocks);
    const int64_t needed = (tokens * p.n_kv_heads * (D / Near::VEC) / (2 * kRotThreads) + blocks.n) * p.n_layers;
    const bool idle = mostly_idle((int64_t)two.x * two.y * two.z, needed);
    if (bytes <= kCacheBytes && !idle) return launch_linear<Near, D, 2>(p, blocks, rt, two, stream);
    dim3 eight = linear_grid<Past, D, 8>(p, blocks);
    // (an odd number per block: workgroups go to the XCDs in turn, and the first few of every block, all that short blocks
    // need, went to the same ones: 1,280 among 500 of 20 tokens, four layers: 80 per block 218 us, 81 54, two pieces 140)
    if (idle) eight.x |= 1;
    return launch_linear<Past, D, 8>(p, blocks, rt, eight, stream);
  }
  const auto launch = [&](auto ch) {
    typedef decltype(ch) Ch;
    if (p.mode == 0)
      return p.layout == 0 ? launch_t<Ch, D, 0, 0>(p, blocks, rt, stream) : launch_t<Ch, D, 1, 0>(p, blocks, rt, stream);
    if constexpr (std::is_same<Params, ReencParams>::value)
      return p.layout == 0 ? launch_t<Ch, D, 0, 1>(p, blocks, rt, stream) : launch_t<Ch, D, 1, 1>(p, blocks, rt, stream);
    return hipErrorInvalidValue;
  };
  return bytes > kCacheBytes / 4 ? launch(Past{}) : launch(Near{});
}

}  // namespace

template <typename Params, typename Blocks>
hipError_t launch_reencode(const Params &p, const Blocks &blocks, const RopeTable &rt, hipStream_t stream) {
  if (p.dtype == 0) {
    if (p.head_dim == 128) return launch_d<uint16_t, 128>(p, blocks, rt, stream);
    if (p.head_dim == 64) return launch_d<uint16_t, 64>(p, blocks, rt, stream);
  } else if constexpr (std::is_same<Params, ReencParams>::value) {
    if (p.head_dim == 128) return launch_d<float, 128>(p, blocks, rt, stream);
    if (p.head_dim == 64) return launch_d<float, 64>(p, blocks, rt, stream);
  }
  return hipErrorInvalidValue;
}

template hipError_t launch_reencode(const ReencParams &, const ReencBlocks &, const RopeTable &, hipStream_t);
template hipError_t launch_reencode(const ReencParams &, const ReencBlocksLarge &, const RopeTable &, hipStream_t);
template hipError_t launch_reencode(const ReencRowsParams &, const ReencBlocks &, const RopeTable &, hipStream_t);
template hipError_t launch_reencode(const ReencRowsParams &, const ReencBlocksLarge &, const RopeTable &, hipStream_t);

}  // namespace ba
