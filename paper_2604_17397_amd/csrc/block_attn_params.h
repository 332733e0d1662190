// Launch parameters shared by the attention kernels (internal to libsdvg).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "block_attn_index.h"
#include "row_map.h"

namespace sdvg {

constexpr int kMaxAttnItems = 8;  // (q, cache, block, out) sets one launch can take

struct AttnItem {
  const void *q, *k_cache, *v_cache, *k_blk, *v_blk;
  void *out;
};

struct AttnParams {
  AttnItem items[kMaxAttnItems];
  int64_t q_ts, q_hs, o_ts, o_hs, kv_ts, kv_hs, blk_ts, blk_hs;  // strides in elements
  int64_t cache_len;
  float *partials;    // partial results of query tiles whose keys are split over workgroups (or null)
  // fused commit: workgroups past the attention work copy item 0's block into these rows (or null)
  void *k_commit_dst, *v_commit_dst;
  int32_t n_blk, copy_first_block, n_copy_blocks;
  int32_t n_items, n_q, n_k, n_heads, n_qtiles;
  int32_t n_hq;       // query tiles of the launch: n_items * n_heads * n_qtiles
  int32_t n_tiles;    // key tiles: n_k / 64, rounded up (4 key groups: of 32 keys)
  attn_index::KeySplit split;  // how the keys are cut over workgroups, if they are
  int32_t total_work; // workgroups with work
  int32_t work_per_xcd;
  int32_t wt_base, wt_rem;  // 32-row wave tiles per query tile: wt_base, plus one for the first wt_rem
  FastDiv div_qtiles, div_heads;  // by n_qtiles and by n_heads
  float scale_log2e;  // scale * log2(e)
};

// fp32 check path (block_attn_f32.hip): same mathematics, fp32 inputs / P / output; item 0 only.
int launch_block_attn_f32(const AttnParams &p, hipStream_t stream);

// Kernel for few query rows (block_attn_groups.hip): `groups` (2 or 4) key groups per workgroup.
// p.n_qtiles / p.n_tiles count its own tiles (256 / groups query rows; 64 keys for 2 groups, 32 for 4).
hipError_t prepare_block_attn_groups();  // once per device: raises the dynamic-LDS limit
int launch_block_attn_groups(const AttnParams &p, int groups, hipStream_t stream);

// Kernel for the smallest launches (block_attn_rows32.hip): 32 query rows per workgroup, tiles of 32 keys.
hipError_t prepare_block_attn_rows32();  // once per device: raises the dynamic-LDS limit
// `halves`: two workgroups per 32 rows, each with half of the output dims.
int launch_block_attn_rows32(AttnParams p, bool halves, hipStream_t stream);

}  // namespace sdvg
