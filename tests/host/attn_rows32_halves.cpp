// The V tiles of the 32-row kernel's workgroups with half of the output dims, replayed on the CPU from the index header
// that the kernel compiles in: what every lane copies must be a key of the tile (the last one again past the
// end) and inside the workgroup's 64 dims, the reads must find each operand where its copy put it, a read of half
// a wave must touch every LDS bank once, and the merge's layout must be a permutation.
#include <cstdio>
#include <vector>

#include "block_attn_rows32_index.h"

namespace ix = sdvg::attn_index;
using R = ix::Rows32;

struct Cell {
  int row, chunk;
};

static bool tile(uint32_t pitch, int keys) {
  std::vector<Cell> lds(R::kTile / 2 / 16, Cell{-1, -1});
  int64_t base[4] = {0, 0, 0, 0};
  for (int u = 0; u < 3; ++u) base[u + 1] = base[u] + ix::rows32_half_copy_step(pitch);
  for (int u = 0; u < ix::kHalfCopies; ++u)
    for (int lane = 0; lane < 64; ++lane) {
      const int64_t imm = 1024 * u;
      const int64_t src = keys == R::kKeys ? base[u] + ix::rows32_half_lane_offset(pitch, lane) + imm
                                           : -imm + ix::rows32_half_short_offset(pitch, keys, lane, u) + imm;
      const int64_t row = src / pitch, inner = src % pitch;
      if (src < 0 || row >= keys || inner >= ix::kHalfRow || inner % 16) return false;
      const int own = ix::rows32_half_copy_row(lane, u);
      if (row != (own < keys ? own : keys - 1)) return false;
      lds[(imm + 16 * lane) / 16] = Cell{own, static_cast<int>(inner / 16)};
    }
  for (int j = 0; j < 2; ++j)
    for (int db = 0; db < 2; ++db)
      for (int hi = 0; hi < 2; ++hi) {
        std::vector<int> bank(64);
        for (int lane = 0; lane < 64; ++lane) {
          const int i16 = lane & 15, b16 = (lane >> 4) & 1, hh = lane >> 5;
          const int off = ix::rows32_half_read_offset(lane, 0, db, 0) + j * 16 * ix::kHalfRow + hi * 8 * ix::kHalfRow;
          if (off != ix::rows32_half_read_offset(lane, j, db, hi)) return false;
          const int row = 16 * j + 8 * hi + 4 * hh + (i16 >> 2), byte = 64 * db + 32 * b16 + 8 * (i16 & 3);
          const Cell &c = lds[off / 16];
          if (c.row != row || c.chunk != byte / 16 || off % 16 != byte % 16) return false;
          if (lane < 32)
            for (int w = 0; w < 2; ++w)
              if (bank[(off / 4 + w) % 64]++) return false;
        }
      }
  return true;
}

int main() {
  for (uint32_t pitch : {256u, 12u * 256, 40u * 256, (1u << 26) - 16})
    for (int keys = 1; keys <= R::kKeys; ++keys)
      if (!tile(pitch, keys)) return std::printf("FAIL pitch %u, %d keys\n", pitch, keys), 1;
  std::vector<char> hit(R::kTile / 16);
  for (int q = 0; q < 16; ++q)
    for (int row = 0; row < 32; ++row) hit[ix::rows32_half_merge_offset(q, row) / 16]++;
  for (char h : hit)
    if (h != 1) return std::printf("FAIL merge\n"), 1;
  std::printf("ok\n");
  return 0;
}
