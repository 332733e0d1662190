// The cut of a launch in two (csrc/block_attn_plan.h) behind a C function, for the tests.
#include "block_attn_plan.h"

// out: heads and query rows of the first part (0, 0: one launch), estimated us of one launch and of the two
extern "C" void attn_cut(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, double out[4]) {
  const sdvg::Cut c = sdvg::choose_cut(n_items, n_q, n_heads, n_k, n_cu, true);
  auto us = [&](int heads, int rows) { return sdvg::choose_groups(n_items, rows, heads, n_k, n_cu, true).us; };
  out[0] = c.heads;
  out[1] = c.rows;
  out[2] = us(n_heads, n_q);
  out[3] = c.heads ? us(c.heads, n_q) + us(n_heads - c.heads, n_q) : c.rows ? us(n_heads, c.rows) + us(n_heads, n_q - c.rows) : 0;
}
