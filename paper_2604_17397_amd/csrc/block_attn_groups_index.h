// Index arithmetic of the grouped attention kernel (block_attn_groups.hip), on top of
// block_attn_index.h (key streams, swizzle, operand reads, work distribution); plain integer and
// pointer arithmetic, compiled into the kernel and into tests/host/attn_groups_replay.cpp.
#pragma once
#include <stddef.h>
#include <stdint.h>

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
  static constexpr int kTogether = kRowWaves * 1024 < 4096 ? 2 : 1;  // copies that share one LDS address (group_copy_imm)
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

// Iteration i of a group (its i-th tile) copies V of its tile i + 1 and K of its tile i + 3. No tile holds keys of both the
// cache and the block: the cache's tiles come first, then the block's, and the last tile of each may be short. A copy
// then takes a scalar address and a 32-bit offset per lane, which only change with the source and with a short tile.
// What follows the last key of a short tile repeats that key's row and is masked; past the last tile a group
// takes the last one, masked as a whole.
SDVG_HD int source_tiles(int n_keys, int per_tile) { return (n_keys + per_tile - 1) / per_tile; }
// The first tiles that are not a whole tile of the cache, in the block, not a whole tile of the block, past the end.
struct GroupBounds {
  int cache_whole, block, block_whole, end;
};
template <int G>
SDVG_HD GroupBounds group_bounds(int c_len, int n_blk) {
  constexpr int n = Groups<G>::kKeys;
  const int block = source_tiles(c_len, n);
  return GroupBounds{c_len / n, block, block + n_blk / n, block + source_tiles(n_blk, n)};
}
// The next of them behind tile t, from which on the kind of tile may be another one.
SDVG_HD int group_next_bound(const GroupBounds &b, int t) {
  return t < b.cache_whole ? b.cache_whole : t < b.block ? b.block : t < b.block_whole ? b.block_whole
                                                           : t < b.end ? b.end : INT32_MAX;
}
// Keys of tile t, and of the last tile for those past the end (which are masked).
template <int G>
SDVG_HD int group_tile_keys(const GroupBounds &b, int c_len, int n_blk, int t) {
  constexpr int n = Groups<G>::kKeys;
  if (t < b.block) return t < b.cache_whole ? n : c_len % n;
  return t < b.block_whole || n_blk % n == 0 ? n : n_blk % n;
}
// Keys of tile t that count: all `keys` of it, none past the end.
SDVG_HD int group_counted_keys(const GroupBounds &b, int t, int keys) { return t < b.end ? keys : 0; }
// Token 0 of the block's rows, were the tiles' rows numbered through: tile t's first row is at this + t * keys * pitch.
template <int G>
SDVG_HD uint64_t group_block_base(const GroupBounds &b, uint64_t block_row0, uint32_t pitch) {
  return block_row0 - static_cast<uint64_t>(static_cast<uint32_t>(b.block * Groups<G>::kKeys)) * pitch;
}
template <int G>
SDVG_HD uint64_t group_tile_base(const GroupBounds &b, int t, uint64_t cache_row0, uint64_t block_base, uint32_t pitch) {
  t = t < b.end ? t : b.end - 1;
  return (t < b.block ? cache_row0 : block_base) + static_cast<uint64_t>(static_cast<uint32_t>(t * Groups<G>::kKeys)) * pitch;
}
// From a group's tile to its next one of the same kind.
template <int G>
SDVG_HD uint64_t group_step(const GroupBounds &b, int t, uint32_t pitch) {
  return t < b.end ? static_cast<uint64_t>(G * Groups<G>::kKeys) * pitch : 0;
}
// Pitches (bytes) for which the offsets fit 32 bits; with others a copy takes a 64-bit address per lane.
SDVG_HD bool group_takes(uint64_t pitch) { return pitch < (uint64_t{1} << 26); }
// The copy instruction adds its immediate to the LDS address as well as to the source address: of copies that share an LDS
// address each has an offset that is less by its immediate, and the scalar address is kImm below the tile's first row, so
// that no offset is negative.
template <int G>
SDVG_HD constexpr int group_copy_imm(int u) {
  return u % Groups<G>::kTogether * Groups<G>::kRowWaves * 1024;
}
template <int G>
SDVG_HD constexpr int group_max_imm() {
  return group_copy_imm<G>(Groups<G>::kTogether - 1);
}
SDVG_HD int clamped_row(int row, int keys) { return row < keys ? row : keys - 1; }
template <int G>
SDVG_HD uint32_t group_lane_offset(int wr, int lane, int u, uint32_t pitch, int keys, int is_v) {
  const int row = group_copy_row<G>(wr, lane, u);
  return static_cast<uint32_t>(clamped_row(row, keys)) * pitch + static_cast<uint32_t>(swizzled_chunk(row, lane, is_v) * 16) +
         static_cast<uint32_t>(group_max_imm<G>() - group_copy_imm<G>(u));
}

// Where the merge (of the 32-row kernel too) keeps O: the 16 bytes holding dims 8 c + 4 hh .. + 3 of a row, in the part of the wave
// they come from. The row is turned by c so that 16 lanes that read one row's chunks c = 0 .. 15 touch
// every bank once.
SDVG_HD int merge_offset(int c, int hh, int row) { return (c * 64 + hh * 32 + (row ^ c)) * 16; }

}  // namespace attn_index
}  // namespace sdvg
