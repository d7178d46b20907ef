// What the files of the C boundary share: the profiling hooks around a launch, the checks of a device
// tensor, the RoPE frequency table, and the two helpers that run the re-encode and RoPE pre-pass kernels
// over a list of blocks or segments.  Defined in ba_api.hip.
#pragma once

#include <mutex>
#include <vector>

#include "../../include/ba.h"
#include "ba_internal.h"
#include "ba_plan.h"

namespace ba {
namespace api {

// ---- optional per-kernel timing (ba_profile_begin / ba_profile_end) ------------------------
struct Profiler {
  std::mutex mu;
  bool on = false;
  int max_records = 0;
  std::vector<hipEvent_t> start[BA_PROFILE_CLASSES], stop[BA_PROFILE_CLASSES];
};
extern Profiler g_prof;

// Brackets one kernel launch with two events on its stream while profiling is on.
struct ProfileScope {
  hipStream_t stream;
  int cls;
  bool active = false;
  hipEvent_t stop_event = nullptr;  // this scope's own: another thread may open a scope of the class meanwhile
  ProfileScope(int cls_, hipStream_t s) : stream(s), cls(cls_) {
    std::lock_guard<std::mutex> lk(g_prof.mu);
    if (!g_prof.on || (int)g_prof.start[cls].size() >= g_prof.max_records) return;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return;
    if (hipEventCreate(&e1) != hipSuccess) {
      (void)hipEventDestroy(e0);
      return;
    }
    g_prof.start[cls].push_back(e0);
    g_prof.stop[cls].push_back(e1);
    (void)hipEventRecord(e0, stream);
    stop_event = e1;
    active = true;
  }
  ~ProfileScope() {
    if (!active) return;
    // (under the lock: ba_profile_end destroys the events, and must not do so between the
    // constructor and this record)
    std::lock_guard<std::mutex> lk(g_prof.mu);
    if (g_prof.on) (void)hipEventRecord(stop_event, stream);
  }
};


size_t elt_size(int32_t dtype);
// pointer, dtype, alignment and strides of a device tensor; BA_OK or a status with ba_last_error() set
int32_t check_tensor(const ba_tensor *t, const char *name, bool allow_f32, int32_t D, int32_t n_heads);
// theta_j / (2 pi) as a Q0.64 fraction, from extended-precision host arithmetic
void build_rope_table(const ba_heads *h, RopeTable *rt);
float scale_log2e(const ba_heads *h);  // softmax scale * log2(e)
template <typename Params>  // ReencParams or ReencRowsParams
int32_t run_reencode(Params p, const RopeTable &rt, int n_blocks, const int32_t *src_off, const int32_t *dst_off,
                     const int32_t *len, const int32_t *pos_old, const int32_t *pos_new, hipStream_t stream);
// Rotate fresh Q (into q_rot, packed, pre-scaled) and fresh K (into k_rot) for segments
// [seg0, seg0 + n) given by start offsets and first positions.
int32_t run_rope_prepass(const ba_heads *h, const RopeTable &rt, const ba_tensor *q, uint16_t *q_rot, const ba_tensor *k,
                         const ba_tensor *k_rot, int n, const int32_t *start, const int32_t *pos0, hipStream_t stream,
                         const RopeRots *rots = nullptr, const RopeRotsSmall *rots_small = nullptr, float *rot_dst = nullptr,
                         int n_rot = 0, float *q_table = nullptr, int table_rows = 0, int32_t *zero = nullptr, int n_zero = 0);

// What the merge of the split partials knows of the rows (AttnParams::merge_rows, merge_sparse).
// Sparse: the indices are waited for ahead of the other loads, to skip units without rows.  Calls of eight prompts over 2,000
// context tokens, 32 over 8 heads of 128, sparse / not, by the share of units with rows: 1/8 24.9 / 26.0 us, 3/8 26.3 / 27.2, 4/8
// 27.1 / 28.2, 5/8 29.5 / 29.9, 6/8 31.3 / 31.2, all 34.7 / 34.7; 8 over 2 of 64 1/8 16.2 / 16.0, 4/8 17.8 / 17.5, all 19.9 / 19.8.
inline void set_merge_rows(AttnParams *ap, int n_prompts, const int32_t *cu_q, int G) {
  int64_t live = 0, units = 0;  // per KV head
  for (int n = 0; n < n_prompts; ++n) {
    const int64_t rows = (int64_t)(cu_q[n + 1] - cu_q[n]) * G;
    live += (rows + 31) / 32;
    units += (rows + kTileRows - 1) / kTileRows * (kTileRows / 32);
  }
  ap->merge_rows = n_prompts == 1 ? (cu_q[1] - cu_q[0]) * G : 0;
  ap->merge_div = make_fast_div((uint32_t)(ap->n_kv_heads * (kTileRows / 32)));
  ap->merge_sparse = 2 * live < units;
}
// A context of cached blocks that a final block's first launch gathers (keys re-encoded; values copied as a second layer, or
// left where they are and fetched through a table).
struct Gather {
  ReencRowsParams p;    // (row_table null: no table)
  const int32_t *ctx0;  // with a table: prompt n's keys from row ctx0[n] of k_ctx on (FinalGatherMeta)
  int n_blocks;         // the last of them, at most kReencMaxBlocksLarge (the others: launches before)
  const int32_t *src_off, *dst_off, *len, *pos_old, *pos_new;
  // nothing is copied, the attention kernel turns the keys (p.row_table and p.dst unused)
  bool turn;
  ba::TurnTables turned;
  uint32_t blk_at, rot_at;  // of FinalTurnMeta
};
bool fresh_apart(const ba_tensor *q_f, const ba_tensor *k_f, const ba_tensor *o, int64_t t0, int64_t t1, const ba_heads *h);
bool encode_keys_apart(const ba_heads *h, const ba_tensor *q, const ba_tensor *k, const ba_tensor *v, const ba_tensor *o, const ba_tensor *k_out, int64_t T);
bool writes_gathered_rows(const Gather &g, const ba_tensor *k_rot, int n_heads, int64_t t0, int64_t t1);
// ba_final_block_attention, its context gathered first if so asked
int32_t final_block(const ba_heads *heads, const ba_tensor *q_f, const ba_tensor *k_ctx, const ba_tensor *v_ctx,
                    const ba_tensor *k_f, const ba_tensor *v_f, const ba_tensor *o_out, const ba_tensor *k_f_rot_out,
                    int32_t n_prompts, const int32_t *cu_q, const int32_t *cu_ctx, const int32_t *q_pos0,
                    int32_t rope_mode, void *ws, size_t ws_bytes, void *stream_, const Gather *gather);

}  // namespace api
}  // namespace ba
