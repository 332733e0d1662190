// Index arithmetic of the 32-row attention kernel (block_attn_rows32.hip), on top of
// block_attn_index.h (key streams, operand reads, work distribution) and block_attn_groups_index.h
// (swizzle, address of a key's row); plain integer and pointer arithmetic, compiled into the kernel and
// into tests/host/attn_rows32_replay.cpp.
#pragma once
#include "block_attn_groups_index.h"

namespace sdvg {
namespace attn_index {

// All 8 waves of a workgroup share 32 query rows; wave w takes the key tiles w, w + 8, ... (32 keys), one
// K and one V tile at a time in its own part of the LDS. Behind the waves' parts: the query rows, laid out
// like a K tile, and the waves' first maxima.
struct Rows32 {
  static constexpr int kKeys = 32;
  static constexpr int kTile = kKeys * 256;
  static constexpr int kWavePart = 2 * kTile;             // K at 0, V at kTile
  static constexpr int kQ = kWaves * kWavePart;
  static constexpr int kMax = kQ + kTile;
  static constexpr int kLdsBytes = kMax + kWaves * 64 * 4;
  static constexpr int kCopies = kTile / 1024;            // 1 KB copies per tile and tensor
};

// Copy u of a tile moves tile rows 4 u .. 4 u + 3: lane i the physical 16-byte chunk i % 16 of this row.
SDVG_HD int rows32_copy_row(int lane, int u) { return 4 * u + (lane >> 4); }
// Copies 4 h .. 4 h + 3 share one destination register: copy u lands 1024 * (u % 4) past rows32_copy_dst
// (+ 16 per lane), because the copy instruction adds its immediate to the LDS address as well as to the
// source address, which rows32_copy_step takes into account.
SDVG_HD uint32_t rows32_copy_dst(int wave, int is_v, int h) {
  return static_cast<uint32_t>(wave * Rows32::kWavePart + is_v * Rows32::kTile + h * 4096);
}

// Key tiles. No tile holds keys of both the cache and the block: the cache's tiles come first, then the
// block's, and the last tile of each may be short. All rows of a tile then lie at one pitch from one
// scalar address, and a lane's offset from there fits 32 bits (rows32_takes). What follows the last key of
// a short tile repeats that key's row and is masked.
SDVG_HD int rows32_tiles(int n_keys) { return (n_keys + Rows32::kKeys - 1) / Rows32::kKeys; }
struct Rows32Tile {
  int in_cache;  // else in the block
  int first;     // token of its first row, in the cache or in the block
  int keys;      // 1 .. 32
};
SDVG_HD Rows32Tile rows32_tile(int c_len, int n_blk, int t) {
  const int n_cache = rows32_tiles(c_len), in_cache = t < n_cache;
  const int first = (in_cache ? t : t - n_cache) * Rows32::kKeys, left = (in_cache ? c_len : n_blk) - first;
  return Rows32Tile{in_cache, first, left < Rows32::kKeys ? left : Rows32::kKeys};
}
// Pitches (bytes) this holds for.
SDVG_HD bool rows32_takes(uint64_t pitch) { return pitch < (uint64_t{1} << 26); }

// Whole tiles: the step from the rows of copy u to those of copy u + 1, less what the immediate moves on
// (copies 3 and 4: back), and a lane's offset from there. The swizzle repeats every 16 rows (K: u and u + 4
// agree; V: all u do).
SDVG_HD int rows32_copy_step(uint32_t pitch, int u) { return static_cast<int>(4 * pitch) - (u % 4 == 3 ? -3072 : 1024); }
SDVG_HD uint32_t rows32_lane_offset(uint32_t pitch, int lane, int u, int is_v) {
  return static_cast<uint32_t>(lane >> 4) * pitch +
         static_cast<uint32_t>(swizzled_chunk(rows32_copy_row(lane, u), lane, is_v) * 16);
}
// Short tiles: a lane's offset from the tile's first row, immediate not taken into account.
SDVG_HD uint32_t rows32_short_offset(uint32_t pitch, int keys, int lane, int u, int is_v) {
  const int row = rows32_copy_row(lane, u);
  return static_cast<uint32_t>(row < keys ? row : keys - 1) * pitch +
         static_cast<uint32_t>(swizzled_chunk(row, lane, is_v) * 16);
}

// ---- two workgroups per 32 query rows, each with half of the output dims: both need all of K, but a V tile is 128
// bytes of each row. Copy u of a V tile moves rows 8 u .. 8 u + 7: lane i the physical 16-byte chunk i % 8 of row 8 u + i / 8,
// whose 64-byte halves change places in every second pair of rows, so that the transposing read of 4 rows x 64
// bytes touches every bank once.
constexpr int kHalfRow = 128;
constexpr int kHalfCopies = Rows32::kTile / 2 / 1024;
SDVG_HD int rows32_half_copy_row(int lane, int u) { return 8 * u + (lane >> 3); }
SDVG_HD int rows32_half_chunk(int row, int lane) { return (lane & 7) ^ (2 * (row & 2)); }
SDVG_HD int rows32_half_copy_step(uint32_t pitch) { return static_cast<int>(8 * pitch) - 1024; }
SDVG_HD uint32_t rows32_half_lane_offset(uint32_t pitch, int lane) {  // (the same for all u: 8 u is a multiple of 4)
  return static_cast<uint32_t>(lane >> 3) * pitch + static_cast<uint32_t>(rows32_half_chunk(lane >> 3, lane) * 16);
}
SDVG_HD uint32_t rows32_half_short_offset(uint32_t pitch, int keys, int lane, int u) {
  const int row = rows32_half_copy_row(lane, u);
  return static_cast<uint32_t>(row < keys ? row : keys - 1) * pitch + static_cast<uint32_t>(rows32_half_chunk(row, lane) * 16);
}
// v_read_offset of such a tile (db 0 or 1).
SDVG_HD int rows32_half_read_offset(int lane, int j, int db, int hi) {
  const int i16 = lane & 15, b16 = (lane >> 4) & 1, hh = lane >> 5;
  return (16 * j + 8 * hi + 4 * hh + (i16 >> 2)) * kHalfRow + ((db ^ (i16 >> 3)) * 64) + 32 * b16 + 8 * (i16 & 3);
}
// merge_offset for 64 dims: dims 4 q .. 4 q + 3 of a row.
SDVG_HD int rows32_half_merge_offset(int q, int row) { return (q * 32 + (row ^ q)) * 16; }

// Key tiles of a wave (at least one: a wave past the last tile goes through a tile that is masked).
SDVG_HD int rows32_tiles_of(int wave, int n_tiles) { return wave < n_tiles ? (n_tiles - wave + kWaves - 1) / kWaves : 1; }

}  // namespace attn_index
}  // namespace sdvg
