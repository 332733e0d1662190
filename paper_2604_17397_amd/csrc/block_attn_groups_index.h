// Index arithmetic of the grouped attention kernel (block_attn_groups.hip), on top of
// block_attn_index.h (key streams, swizzle, operand reads, work distribution); plain integer and
// pointer arithmetic, compiled into the kernel and into tests/host/attn_groups_replay.cpp.
#pragma once
#include <stddef.h>

#include <type_traits>
#include <utility>

#include "block_attn_index.h"

namespace sdvg {
namespace attn_index {

// ---- key groups (block_attn_groups.hip): the 8 waves form G groups of R = 8 / G waves. The groups
// share the same R x 32 query rows and deal the key tiles out among themselves (group g takes tiles
// g, g + G, ...); every group copies its own tiles into its own part of the LDS.
template <int G>
struct Groups {
  static constexpr int kRowWaves = kWaves / G;
  static constexpr int kKeys = G == 2 ? 64 : 32;       // keys per tile
  static constexpr int kHalves = kKeys / 32;
  static constexpr int kTile = kKeys * 256;            // bytes of one K or V tile
  static constexpr int kVSlots = 3 * kTile;            // a group's LDS: K slots 0, 1, 2, then V slots 0, 1
  static constexpr int kGroup = 5 * kTile;
  static constexpr int kCopies = kKeys / (4 * kRowWaves);  // 1 KB copies per wave, tile and tensor
  // K swizzles that occur among a lane's rows (the swizzle is a function of row % 16)
  static constexpr int kVariants = kCopies < 16 / (4 * kRowWaves) ? kCopies : 16 / (4 * kRowWaves);
};

// What a wave starts before the loop: K(0), its share of the query rows, K(1) and then K(2), V(0). The kernel goes through
// kGroupStart, and copies land in the order in which they were started. How many may still be under way at the
// barrier ahead of the first scores (which read K(0) and the query rows), and at the barrier of the common maximum:
// behind that one the first operands of K(1) are read, before the loop's first wait and barrier.
enum GroupStart { kStartK0, kStartQ, kStartK1K2, kStartV0 };
constexpr GroupStart kGroupStart[] = {kStartK0, kStartQ, kStartK1K2, kStartV0};
template <int G>
SDVG_HD constexpr int group_start_copies(GroupStart what) {
  return what == kStartQ ? Groups<G>::kRowWaves : what == kStartK1K2 ? 2 * Groups<G>::kCopies : Groups<G>::kCopies;
}
// Copies started behind `what`.
template <int G>
SDVG_HD constexpr int group_started_after(GroupStart what) {
  int n = 0;
  bool behind = false;
  for (GroupStart w : kGroupStart) {
    if (behind) n += group_start_copies<G>(w);
    behind = behind || w == what;
  }
  return n;
}
template <int G>
SDVG_HD constexpr int group_left_at_scores() {
  const int k0 = group_started_after<G>(kStartK0), q = group_started_after<G>(kStartQ);
  return k0 < q ? k0 : q;
}
template <int G>
SDVG_HD constexpr int group_left_at_maximum() {
  return group_started_after<G>(kStartK1K2) + Groups<G>::kCopies;  // (and K(2))
}
// Calls f with every step of kGroupStart as a constant, in order.
template <class F, size_t... N>
SDVG_HD void group_start_steps(F f, std::index_sequence<N...>) {
  (f(std::integral_constant<GroupStart, kGroupStart[N]>{}), ...);
}
template <class F>
SDVG_HD void group_start_steps(F f) {
  group_start_steps(f, std::make_index_sequence<sizeof(kGroupStart) / sizeof(kGroupStart[0])>{});
}

// Rows and bytes of copy u of row wave wr: lane i moves physical chunk i % 16 of tile row
// group_copy_row to group_copy_dst + 16 * i.
template <int G>
SDVG_HD int group_copy_row(int wr, int lane, int u) {
  return 4 * (wr + Groups<G>::kRowWaves * u) + (lane >> 4);
}
template <int G>
SDVG_HD uint32_t group_copy_dst(int group, int wr, int u, int slot, int is_v) {
  using C = Groups<G>;
  return static_cast<uint32_t>(group * C::kGroup + is_v * C::kVSlots + slot * C::kTile +
                               (wr + C::kRowWaves * u) * 1024);
}
// Where the query rows of row wave wr pass through the LDS, laid out like 32 rows of a K tile: in the
// groups' second V slots, which are written for the first time in matrix phase 0.
template <int G>
SDVG_HD uint32_t group_query_tile(int wr) {
  using C = Groups<G>;
  return static_cast<uint32_t>(wr / C::kHalves * C::kGroup + C::kVSlots + C::kTile + wr % C::kHalves * 8192);
}
SDVG_HD int swizzled_chunk(int row, int lane, int is_v) { return (lane & 15) ^ (is_v ? 4 * (row & 3) : (row & 15)); }

// Iteration i of a group (its i-th tile) copies V of its tile i + 1 and K of its tile i + 3. The copy
// pointers move on from iteration i - 1 by the same step as long as all tiles concerned lie in the
// cache (i < cache_end), or all in the block before the ragged end (block_first <= i < block_end).
// Elsewhere (around the seam, at the end and past it) they are computed from the rows.
struct GroupRuns {
  int cache_end, block_first, block_end;
  uint64_t step_c, step_b;  // G tiles of the cache / of the block, in bytes
};
template <int G>
SDVG_HD GroupRuns group_runs(const Streams &s, int group) {
  constexpr int n = Groups<G>::kKeys;
  auto first_at = [&](int tile) { return (tile - group + G - 1 + 8 * G) / G - 8; };  // first i with group + G i >= tile
  return GroupRuns{first_at(s.c_len / n) - 3, first_at((s.c_len + n - 1) / n), first_at(s.n_k / n) - 3,
                   static_cast<uint64_t>(G * n) * s.kv_tsb, static_cast<uint64_t>(G * n) * s.blk_tsb};
}
SDVG_HD bool group_steady(const GroupRuns &r, int i) {
  return i < r.cache_end || (i >= r.block_first && i < r.block_end);
}
SDVG_HD uint64_t group_step(const GroupRuns &r, int i) { return i < r.cache_end ? r.step_c : r.step_b; }
// Token 0 of one tensor's cache rows and the (virtual) token 0 of its block rows, were they numbered
// like the cache's, plus this lane's swizzled 16-byte chunk: key j is at cache + j * kv_tsb or at
// block + j * blk_tsb.
struct LaneBase {
  uint64_t cache, block;
};
SDVG_HD LaneBase group_lane_base(const Streams &s, int row, int lane, int is_v) {
  const uint64_t chunk = swizzled_chunk(row, lane, is_v) * 16;
  return LaneBase{reinterpret_cast<uint64_t>(is_v ? s.vc : s.kc) + chunk,
                  reinterpret_cast<uint64_t>(is_v ? s.vb : s.kb) + chunk -
                      static_cast<uint64_t>(static_cast<uint32_t>(s.c_len)) * s.blk_tsb};
}
// Address of the row of key min(j, n_k - 1).
SDVG_HD const char *group_key_ptr(const Streams &s, const LaneBase &b, int j) {
  j = j < s.n_k ? j : s.n_k - 1;
  const bool in_cache = j < s.c_len;
  return reinterpret_cast<const char *>((in_cache ? b.cache : b.block) +
                                        static_cast<uint64_t>(static_cast<uint32_t>(j)) *
                                            (in_cache ? s.kv_tsb : s.blk_tsb));
}

// Where the merge (of the 32-row kernel too) keeps O: the 16 bytes holding dims 8 c + 4 hh .. + 3 of a row, in the part of the wave
// they come from. The row is turned by c so that 16 lanes that read one row's chunks c = 0 .. 15 touch
// every bank once.
SDVG_HD int merge_offset(int c, int hh, int row) { return (c * 64 + hh * 32 + (row ^ c)) * 16; }

}  // namespace attn_index
}  // namespace sdvg
