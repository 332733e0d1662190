// Walks every workgroup of split launches on the CPU, with the plan and the index functions that the kernel uses: each
// (query tile, key tile) pair is taken exactly once, each partial result has a slot of its own inside the workspace
// that the plan asks for, a query tile has as many pieces as its merge counts, in the slots where the merge looks.
#include <cstdio>
#include <vector>

#include "block_attn_plan.h"

namespace ix = sdvg::attn_index;

static bool check(int n_hq, int n_tiles, const sdvg::Plan &pl) {
  const ix::KeySplit &ks = pl.split;
  const int64_t slots = pl.workspace_bytes / (sdvg::kPartialFloats * 4);
  const int wgs = pl.total_wg, per_xcd = (wgs + 7) / 8;
  const int64_t rest = ix::split_rest(ks, n_tiles);
  std::vector<char> taken(static_cast<size_t>(n_hq) * n_tiles), slot_used(slots);
  std::vector<int> pieces(n_hq), seen(wgs);
  auto piece = [&](const ix::Piece &pc, int slot, int order) {
    if (pc.hq < 0 || pc.hq >= n_hq || pc.t_first < 0 || pc.t_end <= pc.t_first || pc.t_end > n_tiles) return false;
    if (slot < 0 || slot >= slots || slot_used[slot]++) return false;
    for (int t = pc.t_first; t < pc.t_end; ++t)
      if (taken[static_cast<size_t>(pc.hq) * n_tiles + t]++) return false;
    ++pieces[pc.hq];
    return ix::piece_slot(ks, pc.hq, order, n_hq, ix::first_helper_of(ks, pc.hq, n_tiles)) == slot &&
            order < ix::split_pieces(ks, pc.hq, n_tiles);
  };
  for (int b = 0; b < 8 * per_xcd; ++b) {
    const ix::SplitWork w = ix::split_work(ks, n_hq, wgs, b, per_xcd);
    if (!w.any) continue;
    if (w.helper) {
      if (w.index < 0 || w.index >= ks.n_help || seen[w.index]++) return false;
      const int64_t all = n_hq * rest, u0 = static_cast<int64_t>(w.index) * ks.run, end = u0 + ks.run < all ? u0 + ks.run : all;
      if (u0 >= end) return false;
      for (int64_t u = u0; u < end;) {
        const ix::Piece pc = ix::helper_piece(ks, u, end, n_tiles);
        const int order = ks.cols + w.index - ix::first_wg_of(pc.hq, static_cast<int>(rest), ks.run);
        if (!piece(pc, ix::helper_slot(ks, pc.hq, w.index, n_hq), order)) return false;
        u += pc.t_end - pc.t_first;
      }
    } else {
      const int hq = w.index / ks.cols, c = w.index % ks.cols;
      if (w.index < 0 || w.index >= n_hq * ks.cols || seen[ks.n_help + w.index]++) return false;
      if (!piece(ix::column_piece(ks, hq, c, n_tiles), ix::column_slot(hq, c, n_hq), c)) return false;
    }
  }
  for (int s : seen)
    if (s != 1) return false;
  for (char t : taken)
    if (t != 1) return false;
  for (int hq = 0; hq < n_hq; ++hq)
    if (pieces[hq] != ix::split_pieces(ks, hq, n_tiles)) return false;
  return true;
}

int main() {
  long n = 0;
  for (int n_cu : {256, 304, 250, 64, 7})
    for (int n_hq = 1; n_hq <= 4 * n_cu; n_hq += n_hq < 40 ? 1 : (n_hq < n_cu + 40 ? 3 : 41))
      for (int n_tiles : {32, 33, 36, 64, 97, 147, 220, 512, 1025}) {
        if (static_cast<int64_t>(n_hq) * n_tiles > 300000) continue;
        const sdvg::Plan pl = sdvg::make_plan(1, 256, n_hq, static_cast<int64_t>(n_tiles) * 64 - 3, n_cu, SDVG_SPLIT_ALWAYS);
        // split unless the query tiles fill the rounds, or almost: a workgroup's share is all tiles of one, or too few tiles
        const int64_t all = static_cast<int64_t>(n_hq) * n_tiles, slots = (n_hq + n_cu - 1) / n_cu * static_cast<int64_t>(n_cu);
        const int64_t even = (all + slots - 1) / slots;
        if (pl.split.any() != (n_hq % n_cu != 0 && even >= 16 && even < n_tiles)) {
          std::printf("FAIL cus %d query tiles %d key tiles %d: split %d\n", n_cu, n_hq, n_tiles, pl.split.any());
          return 1;
        }
        if (!pl.split.any()) continue;
        if (pl.n_hq != n_hq || pl.n_tiles != n_tiles || pl.units >= n_tiles || !check(n_hq, n_tiles, pl)) {
          std::printf("FAIL cus %d query tiles %d key tiles %d: cols %d x %d, helpers %d x %d\n", n_cu, n_hq, n_tiles,
                      pl.split.cols, pl.split.col, pl.split.n_help, pl.split.run);
          return 1;
        }
        ++n;
      }
  std::printf("ok: %ld plans\n", n);
  return 0;
}
