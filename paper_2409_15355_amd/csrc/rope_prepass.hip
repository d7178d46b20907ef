// RoPE pre-pass for fresh queries and keys (Eq. 1 of arXiv 2409.15355, positions per
// Section 2.3: local to the block for per-block encoding, absolute for the final block).
//
// One launch rotates the un-rotated K rows (the result is the cacheable key, an output of the
// step anyway) and the Q rows of a run of segments; Q is also multiplied by
// softmax_scale * log2(e) before its one rounding to bf16, so that the attention core's
// score accumulators hold base-2 exponents directly.  Doing this ahead of the attention core
// keeps 32 sin/cos evaluations per lane out of every workgroup's start-up.
//
// Thread mapping as in the re-encode kernel: a thread owns 16-byte chunk c and chunk c + CH/2
// of one token and walks a group of heads, its sin/cos computed once.  Few tokens: one head
// per thread (many short threads); many tokens: several heads per thread.
#include <string.h>

#include <algorithm>

#include "ba_rotate.h"

namespace ba {
namespace {

// Table of rotations for the block-table form of the final block: row b, frequency j holds
// (cos, sin) of angle[b] * theta_j.  One thread per entry.
template <int NB>
__global__ __launch_bounds__(kRotThreads) void rope_rot_table_kernel(float *dst, int n_rot, int half_dim,
                                                                  RopeRotsT<NB> rots, RopeTable rt) {
  const int idx = blockIdx.x * kRotThreads + threadIdx.x;
  if (idx >= n_rot * half_dim) return;
  const int b = idx / half_dim, j = idx - b * half_dim;
  float c, s;
  sincos_phase(rope_phase(rots.angle[b], rt.turns[j]), c, s);
  reinterpret_cast<float2 *>(dst)[idx] = make_float2(c, s);
}

template <int D, int LAYOUT, typename Segs>
__global__ __launch_bounds__(kRotThreads) void rope_prepass_kernel(RopePrepassParams p, Segs segs, RopeTable rt,
                                                                   RopeRotsSmall rots) {
  if (blockIdx.y == 0)
    for (int i = (int)(blockIdx.x * kRotThreads + threadIdx.x); i < p.n_zero; i += (int)gridDim.x * kRotThreads) p.zero[i] = 0;
  {
    // workgroup rows beyond the head groups fill a (small) table of rotations, one thread per entry
    const int head_groups = q_groups(p) + (p.do_k ? (p.n_kv_heads + p.heads_per_thread - 1) / p.heads_per_thread : 0);
    if ((int)blockIdx.y >= head_groups) {
      const int idx = (((int)blockIdx.y - head_groups) * (int)gridDim.x + (int)blockIdx.x) * kRotThreads + (int)threadIdx.x;
      if (idx < p.n_rot * (D / 2)) {
        const int b = idx / (D / 2), j = idx - b * (D / 2);
        float c, s;
        sincos_phase(rope_phase(rots.angle[b], rt.turns[j]), c, s);
        reinterpret_cast<float2 *>(p.rot_dst)[idx] = make_float2(c, s);
      }
      return;
    }
  }
  rope_prepass_rows<D, LAYOUT>(p, segs, rt, (int)blockIdx.x, (int)blockIdx.y);
}

// rots: a small table of rotations to fill in the same launch, or null
template <int D, typename Segs>
hipError_t launch_d(RopePrepassParams p, const Segs &segs, const RopeTable &rt, const RopeRotsSmall *rots,
                    hipStream_t stream) {
  constexpr int TPP = kRotThreads / (D / 8 / 2);
  const int64_t tokens = (int64_t)segs.start[segs.n] - segs.start[0];
  const int groups = q_groups(p) + (p.do_k ? (p.n_kv_heads + p.heads_per_thread - 1) / p.heads_per_thread : 0);
  if (tokens <= 0 || groups == 0) return hipSuccess;
  // (a table has rows of its own to cover, perhaps more than this launch has tokens)
  const int64_t span = std::max<int64_t>(tokens, p.do_q == 2 ? p.table_rows : 0);
  const unsigned gx = (unsigned)((span + TPP - 1) / TPP);
  RopeRotsSmall none;
  unsigned rot_rows = 0;
  if (rots) {
    const int64_t entries = (int64_t)p.n_rot * (D / 2);
    rot_rows = (unsigned)((entries + (int64_t)gx * kRotThreads - 1) / ((int64_t)gx * kRotThreads));
  } else {
    p.n_rot = 0;
    memset(&none, 0, sizeof(none));
  }
  dim3 grid(gx, (unsigned)groups + rot_rows, 1);
  if (p.layout == 0)
    hipLaunchKernelGGL((rope_prepass_kernel<D, 0, Segs>), grid, dim3(kRotThreads), 0, stream, p, segs, rt, rots ? *rots : none);
  else
    hipLaunchKernelGGL((rope_prepass_kernel<D, 1, Segs>), grid, dim3(kRotThreads), 0, stream, p, segs, rt, rots ? *rots : none);
  return hipGetLastError();
}

template <typename Segs>
hipError_t launch_rope_prepass_t(const RopePrepassParams &p, const Segs &segs, const RopeRots *rots,
                                 const RopeRotsSmall *rots_small, const RopeTable &rt, hipStream_t stream) {
  // a large table of rotations gets a launch of its own; a small one rides along with the rows
  const bool want_rot = p.rot_dst && p.n_rot > 0;
  if (want_rot && rots) {
    const int entries = p.n_rot * (p.head_dim / 2);
    hipLaunchKernelGGL((rope_rot_table_kernel<kBlkMaxBlocks>), dim3((entries + kRotThreads - 1) / kRotThreads),
                       dim3(kRotThreads), 0, stream, p.rot_dst, p.n_rot, p.head_dim / 2, *rots, rt);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const RopeRotsSmall *ride = (want_rot && !rots) ? rots_small : nullptr;
  if (p.head_dim == 128) return launch_d<128>(p, segs, rt, ride, stream);
  if (p.head_dim == 64) return launch_d<64>(p, segs, rt, ride, stream);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_rope_prepass(const RopePrepassParams &p, const RopeSegs &segs, const RopeRots *rots,
                               const RopeRotsSmall *rots_small, const RopeTable &rt, hipStream_t stream) {
  return launch_rope_prepass_t(p, segs, rots, rots_small, rt, stream);
}
hipError_t launch_rope_prepass(const RopePrepassParams &p, const RopeSegsSmall &segs, const RopeRots *rots,
                               const RopeRotsSmall *rots_small, const RopeTable &rt, hipStream_t stream) {
  return launch_rope_prepass_t(p, segs, rots, rots_small, rt, stream);
}

}  // namespace ba
