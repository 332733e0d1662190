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
