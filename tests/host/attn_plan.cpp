// The launch plan of csrc/block_attn_plan.h behind a C function, for the tests.
#include "block_attn_plan.h"

// out: key groups and query rows per workgroup, workgroups, query tiles, 1 if the keys are split, workspace bytes
extern "C" void attn_plan(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, int split_mode, int64_t out[6]) {
  const sdvg::Plan p = sdvg::make_plan(n_items, n_q, n_heads, n_k, n_cu, split_mode);
  out[0] = p.groups;
  out[1] = p.rows;
  out[2] = p.total_wg;
  out[3] = p.n_hq;
  out[4] = p.units != p.n_tiles;
  out[5] = p.workspace_bytes;
}

// Workspace of the call that uses the library's own array.
extern "C" int64_t attn_plan_static_workspace(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, int split_mode) {
  return sdvg::make_plan(n_items, n_q, n_heads, n_k, n_cu, split_mode, true, sdvg::kAutoIdleStatic).workspace_bytes;
}

extern "C" int attn_plan_rows(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, int split_mode, int rows32_ok) {
  return sdvg::make_plan(n_items, n_q, n_heads, n_k, n_cu, split_mode, rows32_ok != 0).rows;
}

// Whether two workgroups share 32 query rows, for a call whose q and out have these addresses and strides.
extern "C" int attn_plan_halves(int n_q, int n_heads, int64_t n_k, int n_cu, const void *q, int64_t q_ts, int64_t q_hs, const void *out,
                                int64_t o_ts, int64_t o_hs) {
  const bool in_place = sdvg::ranges_overlap(q, sdvg::rows_bytes(n_q, n_heads, q_ts, q_hs), out, sdvg::rows_bytes(n_q, n_heads, o_ts, o_hs));
  return sdvg::make_plan(1, n_q, n_heads, n_k, n_cu, 0, true, sdvg::kAutoIdle, in_place).halves;
}

// Attention and copying workgroups of a fused commit.
extern "C" void attn_plan_commit(int n_q, int n_blk, int n_heads, int64_t n_k, int n_cu, int out[2]) {
  const sdvg::Plan p = sdvg::make_plan(1, n_q, n_heads, n_k, n_cu, 0);
  out[0] = sdvg::attention_workgroups(p);
  out[1] = sdvg::copy_workgroups(p, static_cast<int64_t>(n_blk) * n_heads, n_cu);
}
