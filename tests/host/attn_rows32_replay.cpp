// Host replay of the 32-row attention kernel's copies, from the index header the kernel compiles in. For
// every configuration all 8 waves x 64 lanes copy their tiles as block_attn_rows32.hip does, with fake
// base addresses; each tile must then hold the wave's keys (the last one again past the end) with the
// swizzle the operand reads undo, no copy may address a token at or past c_len in the cache or at or past n_blk in
// the block, every LDS address stays inside the wave's part, and every key is handled once. The merge's
// layout must be a permutation of a wave's part. Exit code 0 = passed.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "block_attn_rows32_index.h"

namespace ix = sdvg::attn_index;
using R = ix::Rows32;

namespace {

constexpr uint64_t kSpan = uint64_t{1} << 44;
const char *const kBase = reinterpret_cast<const char *>(uint64_t{1} << 48);

struct Replay {
  ix::Streams s;
  int n_blk = 0;
  struct Cell {
    int v, key, chunk;
  };
  std::vector<Cell> lds = std::vector<Cell>(R::kQ / 16, Cell{-1, -1, -1});
  const char *error = nullptr;

  bool put(const char *src, uint32_t dst, int wave, int is_v) {
    const uint64_t all = static_cast<uint64_t>(src - kBase);
    const int region = static_cast<int>(all / kSpan);
    if (region < 0 || region > 3 || (region & 1) != is_v) return error = "source in the wrong tensor", false;
    const bool blk = region >= 2;
    const uint32_t pitch = blk ? s.blk_tsb : s.kv_tsb;
    const uint64_t tok = all % kSpan / pitch, inner = all % kSpan % pitch;
    if (inner >= 256 || inner % 16 || tok >= static_cast<uint64_t>(blk ? n_blk : s.c_len))
      return error = "source out of bounds", false;
    if (dst % 16 || dst / R::kWavePart != static_cast<uint32_t>(wave)) return error = "destination out of bounds", false;
    lds[dst / 16] = Cell{is_v, static_cast<int>(blk ? s.c_len + tok : tok), static_cast<int>(inner / 16)};
    return true;
  }

  bool copy(int wave, int t, int is_v) {
    const ix::Rows32Tile tile = ix::rows32_tile(s.c_len, n_blk, t);
    if (tile.keys < 1 || tile.keys > R::kKeys || tile.first < 0) return error = "not a tile", false;
    const uint32_t pitch = tile.in_cache ? s.kv_tsb : s.blk_tsb;
    uint64_t base[8];
    base[0] = reinterpret_cast<uint64_t>(tile.in_cache ? (is_v ? s.vc : s.kc) : (is_v ? s.vb : s.kb)) +
              static_cast<uint64_t>(static_cast<uint32_t>(tile.first)) * pitch;
    for (int u = 0; u < 7; ++u) base[u + 1] = base[u] + static_cast<int64_t>(ix::rows32_copy_step(pitch, u));
    for (int lane = 0; lane < 64; ++lane)
      for (int u = 0; u < R::kCopies; ++u) {
        const uint32_t imm = (u & 3) * 1024;
        const uint64_t src = tile.keys == R::kKeys
                                 ? base[u] + ix::rows32_lane_offset(pitch, lane, u & 3, is_v) + imm
                                 : base[0] - imm + ix::rows32_short_offset(pitch, tile.keys, lane, u, is_v) + imm;
        if (!put(reinterpret_cast<const char *>(src), ix::rows32_copy_dst(wave, is_v, u / 4) + imm + 16 * lane, wave, is_v))
          return false;
      }
    return true;
  }

  // Reads the tile as the kernel does (every operand of every lane).
  bool check(int wave, int t, int is_v) {
    for (int lane = 0; lane < 64; ++lane) {
      const int r32 = lane & 31, hh = lane >> 5, i16 = lane & 15, b16 = (lane >> 4) & 1;
      auto want = [&](int off, int row, int byte_in_row) {
        off += wave * R::kWavePart + is_v * R::kTile;
        const ix::Rows32Tile tile = ix::rows32_tile(s.c_len, n_blk, t);
        const int j = (tile.in_cache ? 0 : s.c_len) + tile.first + (row < tile.keys ? row : tile.keys - 1);
        const Cell &c = lds[off / 16];
        if (c.v == is_v && c.key == j && c.chunk == byte_in_row / 16 && off % 16 == byte_in_row % 16) return true;
        error = is_v ? "V tile holds the wrong rows" : "K tile holds the wrong rows";
        return false;
      };
      if (!is_v) {
        for (int sd = 0; sd < 8; ++sd)
          if (!want(ix::k_read_offset(lane, sd, 0), r32, (2 * sd + hh) * 16)) return false;
      } else {
        for (int j = 0; j < 2; ++j)
          for (int db = 0; db < 4; ++db)
            for (int hi = 0; hi < 2; ++hi)
              if (!want(ix::v_read_offset(lane, 0, db, 0) + j * 16 * 256 + hi * 8 * 256,
                        16 * j + 8 * hi + 4 * hh + (i16 >> 2), 64 * db + 32 * b16 + 8 * (i16 & 3)))
                return false;
      }
    }
    return true;
  }

  bool run(int c_len, int nb, uint32_t kv_tsb, uint32_t blk_tsb) {
    s = ix::Streams{kBase, kBase + kSpan, kBase + 2 * kSpan, kBase + 3 * kSpan, kv_tsb, blk_tsb, c_len, c_len + nb};
    n_blk = nb;
    const int n_tiles = ix::rows32_tiles(c_len) + ix::rows32_tiles(nb);
    std::vector<char> seen(s.n_k, 0);
    for (int w = 0; w < ix::kWaves; ++w) {
      const int n_it = ix::rows32_tiles_of(w, n_tiles);
      for (int i = 0; i < n_it; ++i) {
        const int t = w + ix::kWaves * i, taken = t < n_tiles ? t : n_tiles - 1;
        for (int is_v = 0; is_v < 2; ++is_v)
          if (!copy(w, taken, is_v) || !check(w, taken, is_v)) return false;
        const ix::Rows32Tile tile = ix::rows32_tile(c_len, nb, taken);
        for (int r = 0; t < n_tiles && r < tile.keys; ++r) seen[(tile.in_cache ? 0 : c_len) + tile.first + r]++;
      }
    }
    for (char c : seen)
      if (c != 1) return error = "a key is not handled exactly once", false;
    return true;
  }
};

}  // namespace

int main() {
  int bad = 0;
  long n = 0;
  auto one = [&](int c, int nb, uint32_t kv, uint32_t bl) {
    Replay r;
    if (!r.run(c, nb, kv, bl) && !bad++) std::printf("FAIL c_len=%d n_blk=%d: %s\n", c, nb, r.error);
    ++n;
  };
  for (int c = 0; c < 300; c += (c < 70 ? 1 : 7))
    for (int nb : {1, 2, 31, 32, 33, 63, 64, 65, 95, 97, 128, 129, 200, 255, 257, 312}) one(c, nb, 40 * 256, 12 * 256);
  for (int k : {0, 1, 6})
    for (int nb : {312, 1031, 4680}) one(k * nb, nb, 12 * 256, 256);
  const uint32_t most = (1u << 26) - 16;  // the largest pitch the kernel takes
  if (!ix::rows32_takes(most) || ix::rows32_takes(most + 16)) return std::printf("FAIL limit of the pitch\n"), 1;
  one(128, 128, most, most);
  one(2000, 77, most, 256);
  std::vector<char> hit(R::kWavePart / 16, 0);
  for (int c = 0; c < 16; ++c)
    for (int hh = 0; hh < 2; ++hh)
      for (int row = 0; row < 32; ++row) hit[ix::merge_offset(c, hh, row) / 16]++;
  for (char h : hit) bad += h != 1;
  if (bad) return 1;
  std::printf("ok: %ld configurations\n", n);
  return 0;
}
