// Internal declarations shared by the translation units of libpyr (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "../../include/pyr.h"

namespace pyr {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr float kLog2e = 1.4426950408889634f;

// Compute units and XCDs of the current device (cached per device); PYR_ERR_LAUNCH if the runtime
// cannot tell - the launchers do not guess.
struct DeviceInfo { int device, compute_units, xccs; };
int device_info(DeviceInfo* out);

// Every launcher returns PYR_OK or PYR_ERR_LAUNCH; arguments are already validated.
int launch_gather(const void* src0, void* dst0, const void* src1, void* dst1, size_t row_bytes,
                  const int32_t* kept_idx, int64_t n_kept, hipStream_t stream);

// up to three row sources (chunks of 16 bytes) and, if pos != nullptr, the position ids, in one launch
struct GatherSources {
    const u32x4* src[3];
    u32x4* dst[3];
    int32_t chunks[3];            // 16-byte chunks per row
    int32_t n;
    const int32_t* pos;
    int32_t* pos_out;
    void add(const void* from, void* to, size_t row_bytes) {
        src[n] = (const u32x4*)from;
        dst[n] = (u32x4*)to;
        chunks[n++] = (int32_t)(row_bytes / 16);
    }
};
int launch_gather_multi(const GatherSources& sources, const int32_t* kept_idx, int64_t n_kept, hipStream_t stream);

// groups > 1: parts holds `groups` rows of total_tokens partial scores, whose sums the kernel writes to `scores` and ranks;
// else `scores` is only read.
int launch_select(const float* parts, int groups, int32_t total_tokens, float* scores, const int32_t* seq_offsets_dev,
                  const int32_t* keep_len_dev, int32_t n_seqs, int32_t max_seqlen, int32_t w, int32_t* kept_idx,
                  int32_t* out_offsets_dev, hipStream_t stream);

// How the selection and the gather of what it keeps go about it (groups rows of partial sums; row_chunks: 16-byte chunks gathered per kept row).
struct SelectPlan {
    bool sums;                    // the rows of partial sums are added by a launch of their own
    int split;                    // > 0: selection and gather in one launch, so many workgroups per sequence; 0: in two
};
SelectPlan plan_select(int groups, int32_t n_seqs, int32_t max_seqlen, int32_t max_kept, int64_t row_chunks);
int launch_select_gather(const float* parts, int groups, int32_t total_tokens, float* scores, const int32_t* seq_offsets_dev,
                         const int32_t* keep_len_dev, int32_t n_seqs, int32_t max_seqlen, int32_t max_kept, int64_t n_kept, int32_t w,
                         int32_t* kept_idx, int32_t* out_offsets_dev, const GatherSources& sources, hipStream_t stream);

// kernel 0: lists of 256-row tiles (attention.hip), whose place in them moves on by `turn`; 1, 2: attention_tile.hip with so many groups.
struct AttentionChoice {
    int kernel, turn;
    double cost;                  // predicted microseconds
};
int choose_attention(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len, AttentionChoice* out);
int launch_attention(const AttentionChoice& choice, const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev,
                     const int32_t* seq_offsets_host, const pyr_shape& shape, int32_t uniform_len, float scale_log2,
                     void* out, float* lse, int32_t* item_map, hipStream_t stream);

// One 128-row query tile per workgroup, by one group of four wavefronts or by two that share its keys (attention_tile.hip).
int launch_attention_tile(const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                          const pyr_shape& shape, int32_t uniform_len, float scale_log2, void* out, float* lse, int32_t* tile_map,
                          int groups, hipStream_t stream);

// What the launchers above and below would do with a batch (pyr_diag_route, pyr_diag_launches).
void attention_route(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len, const DeviceInfo& dev, pyr_route* out);
void attention_tile_route(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len, int groups, const DeviceInfo& dev,
                          pyr_launches* out);
int64_t attention_tiles(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len);      // 128-row tiles of a query head
bool attention_tile_listed(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len);
// (returns the rows of partial sums)
int update_route(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t min_seqlen, int32_t w, const DeviceInfo& dev, pyr_launches* out);
int update_task_order(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t min_seqlen, int32_t w, const DeviceInfo& dev);      // as pyr_diag_update
int layer_groups(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len, int32_t min_seqlen, int32_t w, bool parts, const DeviceInfo& dev);
void score_route(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t min_seqlen, int32_t w, bool parts, const DeviceInfo& dev,
                 pyr_route* out);

// row_weights: device [w] or nullptr (uniform); min_seqlen: the shortest sequence (0 if not known)
int launch_score(const void* q, const void* k, const float* lse, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                 const pyr_shape& shape, int32_t min_seqlen, int32_t w, float scale_log2, const float* row_weights,
                 float* scores, hipStream_t stream);

// How a walk over K is cut up (score.hip): 32-key tiles of a range, wavefronts of a workgroup, workgroups a range's tasks are split over.
struct StripPlan {
    int range_tiles, waves, groups;
    double cost;                  // predicted microseconds
};

// A prefill step's scores.  groups > 0: in the launch of the attention tiles (launch_layer), with so many rows of partial sums; 0: by a walk of
// their own (launch_score_groups).  parts: whether the workspace has room for partial sums (score_parts_bytes()).
struct LayerPlan {
    int groups;
    StripPlan strip;
};
LayerPlan plan_layer(const pyr_shape& shape, const int32_t* seq_offsets_host, int32_t uniform_len, int32_t min_seqlen, int32_t w, bool parts,
                     const AttentionChoice& choice, const DeviceInfo& dev);

// The score pass with its small-batch extra (see score.hip): the tasks of a range split over several workgroups when the
// grid is small.  plan.groups > 1: `parts` (score_parts_bytes()) then holds that many rows of total_tokens partial
// sums and `scores` is not written yet (launch_select does it); else `scores` is complete.
constexpr int kMaxScoreGroups = 16;
size_t score_parts_bytes(const pyr_shape& shape);
int launch_score_groups(const StripPlan& plan, const void* q, const void* k, const float* lse, const int32_t* seq_offsets_dev,
                        const int32_t* seq_offsets_host, const pyr_shape& shape, int32_t min_seqlen, int32_t w, float scale_log2,
                        const float* row_weights, float* scores, float* parts, hipStream_t stream);

// Attention tiles and the scores' one walk over K in one launch (layer.hip).  groups > 1: sums [groups, total_tokens]; 1: the scores themselves.
// No row statistics are written.
constexpr int layer_max_keys(int attention_groups) { return 1024 * attention_groups; }
int launch_layer(const AttentionChoice& choice, int groups, const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev,
                 const int32_t* seq_offsets_host, const pyr_shape& shape, int32_t uniform_len, int32_t w, float scale_log2,
                 const float* row_weights, void* out, float* sums, hipStream_t stream);

// Generation phase: the same scores from the window's own query buffer q_win [B, w, Hq, d]
// (right-aligned), in one launch (launch_window) or three: row statistics per range of keys -> part, folded into lse_win
// [B, w, Hq], then the score pass.  part holds window_score_part_bytes() bytes; *groups as above, the partial sums in part.
size_t window_score_part_bytes(const pyr_shape& shape, int32_t w);
int launch_window_score(const void* q_win, const void* k, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                        const pyr_shape& shape, int32_t min_seqlen, int32_t w, float scale_log2, const float* row_weights, float* lse_win, void* part,
                        float* scores, int* groups, hipStream_t stream);

// The same in one launch, where every sequence is short enough for a workgroup to keep its logits (window.hip): workgroups of `waves`
// wavefronts, a sequence's tasks spread over `groups` of them, each with a row of partial sums.  waves == 0: not for this batch.
// tiles: 32-key tiles of the batch.  launch_window writes sums [groups, total_tokens] (the scores themselves if groups == 1).
struct WindowPlan {
    int waves, groups;
    double cost;                  // microseconds, selection included
};
WindowPlan plan_window(const pyr_shape& shape, double tiles, int32_t w, int max_groups, const DeviceInfo& dev);
int window_task_order(const pyr_shape& shape, bool equal, int32_t w, const DeviceInfo& dev);      // 1: by KV head
int launch_window(const void* q, const void* k, const int32_t* seq_offsets_dev, const pyr_shape& shape, bool equal, int32_t w,
                  int32_t q_window, float scale_log2, const float* row_weights, float* sums, const WindowPlan& plan, const DeviceInfo& dev,
                  hipStream_t stream);

// scores[t] = the sum of `groups` rows of partial sums; whether that is worth a launch in front of the selection.
inline bool sums_pay(int groups, int32_t max_seqlen) { return groups >= 48 || (groups >= 24 && groups * (int64_t)max_seqlen >= 36864); }
int launch_sum_parts(const float* parts, int groups, int32_t total_tokens, float* scores, hipStream_t stream);

int launch_gather_positions(const int32_t* pos, const int32_t* kept_idx, int64_t n_kept, int32_t* pos_out,
                            hipStream_t stream);

// Raise a kernel's dynamic LDS limit to `bytes`, once per device (done_mask: one bit per device id).
int ensure_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>* done_mask);

inline int check_launch() { return hipGetLastError() == hipSuccess ? PYR_OK : PYR_ERR_LAUNCH; }

}  // namespace pyr
