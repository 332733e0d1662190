// Host replay of the grouped attention kernel's copy schedule, from the index header the kernel
// compiles in. For every configuration all 8 waves x 64 lanes perform the copies of
// block_attn_groups.hip in its order with fake base addresses; at each point of use K slot / V slot
// of every group must hold exactly the keys of that group's tile (the last one again past the end of a short tile) with the
// swizzle the reads undo, every key is handled once, no copy may address a token at or past c_len in the cache or at or past
// n_blk in the block, and every LDS address stays inside the workgroup's part. Exit code 0 = passed.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "block_attn_groups_index.h"

namespace ix = sdvg::attn_index;

namespace {

constexpr uint64_t kSpan = uint64_t{1} << 44;
const char *const kBase = reinterpret_cast<const char *>(uint64_t{1} << 48);

template <int G>
struct Replay {
  using C = ix::Groups<G>;
  ix::Streams s;
  int n_blk = 0;
  struct Cell {
    int v, key, chunk;
  };
  std::vector<Cell> lds = std::vector<Cell>(G * C::kGroup / 16, Cell{-1, -1, -1});
  const char *error = nullptr;

  bool put(const char *src, uint32_t dst, int is_v) {
    const uint64_t all = static_cast<uint64_t>(src - kBase);
    const int region = static_cast<int>(all / kSpan);
    if (region < 0 || region > 3 || (region & 1) != is_v) return error = "source in the wrong tensor", false;
    const bool blk = region >= 2;
    const uint32_t pitch = blk ? s.blk_tsb : s.kv_tsb;
    const uint64_t tok = all % kSpan / pitch, inner = all % kSpan % pitch;
    if (inner >= 256 || inner % 16 || tok >= static_cast<uint64_t>(blk ? n_blk : s.c_len))
      return error = "source out of bounds", false;
    if (dst % 16 || dst / 16 >= lds.size()) return error = "destination out of bounds", false;
    lds[dst / 16] = Cell{is_v, static_cast<int>(blk ? s.c_len + tok : tok), static_cast<int>(inner / 16)};
    return true;
  }

  // One tensor's copies as the kernel makes them: set_kind and start_copies of block_attn_groups.hip.
  struct Copies {
    uint64_t base = 0, step = 0;
    int bound = 0, keys = 0;
    uint32_t pitch = 0;
    uint32_t off[C::kRowWaves][64][C::kCopies] = {};
  };
  ix::GroupBounds bounds{};
  bool wide = false;
  void set_kind(Copies &x, int t, int is_v) {
    x.bound = ix::group_next_bound(bounds, t);
    x.keys = ix::group_tile_keys<G>(bounds, s.c_len, n_blk, t);
    x.pitch = t < bounds.block ? s.kv_tsb : s.blk_tsb;
    auto at = [&](const char *q) { return reinterpret_cast<uint64_t>(q); };
    x.step = ix::group_step<G>(bounds, t, x.pitch);
    x.base = ix::group_tile_base<G>(bounds, t, at(is_v ? s.vc : s.kc),
                                    ix::group_block_base<G>(bounds, at(is_v ? s.vb : s.kb), s.blk_tsb), x.pitch) -
             x.step - (wide ? 0 : ix::group_max_imm<G>());
    if (wide) return;
    for (int wr = 0; wr < C::kRowWaves; ++wr)
      for (int lane = 0; lane < 64; ++lane)
        for (int u = 0; u < C::kCopies; ++u)
          x.off[wr][lane][u] = ix::group_lane_offset<G>(wr, lane, u, x.pitch, x.keys, is_v);
  }
  bool copy(Copies &x, int t, int grp, int is_v, int slot) {
    if (t >= x.bound) set_kind(x, t, is_v);
    if (x.keys < 1 || x.keys > C::kKeys) return error = "not a tile", false;
    x.base += x.step;
    for (int wr = 0; wr < C::kRowWaves; ++wr)
      for (int lane = 0; lane < 64; ++lane)
        for (int u = 0; u < C::kCopies; ++u) {
          const uint32_t imm = ix::group_copy_imm<G>(u);
          const int row = ix::group_copy_row<G>(wr, lane, u);
          const uint64_t src = wide ? x.base + static_cast<uint64_t>(ix::clamped_row(row, x.keys)) * x.pitch +
                                          ix::swizzled_chunk(row, lane, is_v) * 16
                                    : x.base + x.off[wr][lane][u] + imm;
          // copies that share an LDS address: the first one's, plus the immediate
          const uint32_t dst = ix::group_copy_dst<G>(grp, wr, u - u % C::kTogether, slot, is_v) + imm;
          if (dst != ix::group_copy_dst<G>(grp, wr, u, slot, is_v)) return error = "immediate and LDS address disagree", false;
          if (!put(reinterpret_cast<const char *>(src), dst + 16 * lane, is_v)) return false;
        }
    return true;
  }
  // Keys of tile t by the definition: the cache's tiles, then the block's.
  struct Tile {
    int key0, keys;
  };
  Tile tile_at(int t) const {
    const int n_cache = (s.c_len + C::kKeys - 1) / C::kKeys, n = n_cache + (n_blk + C::kKeys - 1) / C::kKeys;
    t = t < n ? t : n - 1;
    const int first = (t < n_cache ? t : t - n_cache) * C::kKeys, left = (t < n_cache ? s.c_len : n_blk) - first;
    return Tile{(t < n_cache ? 0 : s.c_len) + first, left < C::kKeys ? left : C::kKeys};
  }

  // Reads the tile exactly as the matrix phase does (every operand of every lane).
  bool check(int grp, int is_v, int t, int slot) {
    for (int lane = 0; lane < 64; ++lane) {
      const int r32 = lane & 31, hh = lane >> 5, i16 = lane & 15, b16 = (lane >> 4) & 1;
      const int base = grp * C::kGroup + is_v * C::kVSlots + slot * C::kTile;
      auto want = [&](int off, int row, int byte_in_row) {
        const Tile tile = tile_at(t);
        const int j = tile.key0 + (row < tile.keys ? row : tile.keys - 1);
        const Cell &c = lds[(base + off) / 16];
        if (c.v == is_v && c.key == j && c.chunk == byte_in_row / 16 && (base + off) % 16 == byte_in_row % 16) return true;
        error = is_v ? "V tile holds the wrong rows" : "K tile holds the wrong rows";
        return false;
      };
      if (!is_v) {
        for (int sd = 0; sd < 8; ++sd)
          for (int kb = 0; kb < C::kHalves; ++kb)
            if (!want(ix::k_read_offset(lane, sd, 0) + kb * 32 * 256, 32 * kb + r32, (2 * sd + hh) * 16)) return false;
      } else {
        for (int j = 0; j < 2 * C::kHalves; ++j)
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
    bounds = ix::group_bounds<G>(c_len, nb);
    wide = (c_len > 0 && !ix::group_takes(kv_tsb)) || !ix::group_takes(blk_tsb);
    const int n_it = (bounds.end + G - 1) / G;
    std::vector<char> seen(s.n_k, 0);
    for (int g = 0; g < G; ++g) {
      auto tile_of = [&](int i) { return g + G * i; };
      Copies k, v;
      for (int i = 0; i < 3; ++i)
        if (!copy(k, tile_of(i), g, 0, i)) return false;
      if (!copy(v, tile_of(0), g, 1, 0) || !check(g, 0, tile_of(0), 0)) return false;
      int keys_next = ix::group_counted_keys(bounds, tile_of(0), v.keys);
      for (int i = 0; i < n_it; ++i) {
        // V(i) of a short tile is cleared past its keys: at the next change of kind, or behind the loop
        const int keys_now = keys_next;
        if (keys_now != (tile_of(i) < bounds.end ? tile_at(tile_of(i)).keys : 0)) return error = "wrong mask", false;
        if (i + 1 < n_it && keys_now < C::kKeys && tile_of(i + 3) < k.bound && tile_of(i + 1) < v.bound)
          return error = "a short tile that is not cleared", false;
        if (i + 1 < n_it && tile_of(i + 1) >= v.bound) {
          set_kind(v, tile_of(i + 1), 1);
          keys_next = ix::group_counted_keys(bounds, tile_of(i + 1), v.keys);
        }
        // matrix phase i reads K(i+1) and V(i); its copies of V(i+1) and K(i+3) land at any time in it
        for (int late = 0; late < 2; ++late) {
          if (late && i + 1 < n_it && (!copy(v, tile_of(i + 1), g, 1, (i + 1) % 2) || !copy(k, tile_of(i + 3), g, 0, i % 3)))
            return false;
          if (i + 1 < n_it && !check(g, 0, tile_of(i + 1), (i + 1) % 3)) return false;
          if (!check(g, 1, tile_of(i), i % 2)) return false;
        }
        for (int r = 0; r < keys_now; ++r) seen[tile_at(tile_of(i)).key0 + r]++;
      }
    }
    for (char c : seen)
      if (c != 1) return error = "a key is not handled exactly once", false;
    return true;
  }
};

template <int G>
long sweep(int &bad) {
  long n = 0;
  auto one = [&](int c, int nb, uint32_t kv, uint32_t bl) {
    Replay<G> r;
    if (!r.run(c, nb, kv, bl) && !bad++) std::printf("FAIL G=%d c_len=%d n_blk=%d: %s\n", G, c, nb, r.error);
    ++n;
  };
  for (int c = 0; c < 200; c += (c < 70 ? 1 : 7))
    for (int nb : {1, 2, 31, 32, 33, 63, 64, 65, 95, 97, 128, 129, 200, 312}) one(c, nb, 40 * 256, 12 * 256);
  for (int k : {0, 1, 6})
    for (int nb : {312, 1031, 4680}) one(k * nb, nb, 12 * 256, 256);
  one(100, 100, 0xfffffff0u / 16 * 8, 0x7ffffff0u);  // the largest pitches
  const uint32_t most = (1u << 26) - 16;             // the largest that 32-bit offsets take
  if (!ix::group_takes(most) || ix::group_takes(most + 16)) std::printf("FAIL limit of the pitch\n"), ++bad;
  one(130, 130, most, most);
  one(300, 77, most, 256);
  // the query rows' tiles lie in second V slots, one beside the other
  using C = ix::Groups<G>;
  std::vector<char> taken(G * C::kGroup / 8192, 0);
  for (int r = 0; r < C::kRowWaves; ++r) {
    const int at = ix::group_query_tile<G>(r), in_group = at % C::kGroup - C::kVSlots;
    if (at % 8192 || at >= G * C::kGroup || in_group < C::kTile || in_group + 8192 > 2 * C::kTile || taken[at / 8192]++)
      std::printf("FAIL G=%d query tile %d\n", G, r), ++bad;
  }
  return n;
}

}  // namespace

// The counts of the two waits ahead of the loop against the order in which the kernel starts its copies (kGroupStart):
// what has landed at a wait that leaves n under way is all but the last n. Which operands are read behind which
// barrier is the kernel's own affair; test_second_tile_has_landed_when_it_is_read looks at that on the GPU.
template <int G>
bool start_waits() {
  enum Tile { kK0, kQ, kK1, kK2, kV0 };
  std::vector<Tile> order;
  ix::group_start_steps([&](auto what) {
    const int n = ix::group_start_copies<G>(what);
    switch (what) {
      case ix::kStartK0: order.insert(order.end(), n, kK0); break;
      case ix::kStartQ: order.insert(order.end(), n, kQ); break;
      case ix::kStartK1K2: order.insert(order.end(), n / 2, kK1), order.insert(order.end(), n / 2, kK2); break;
      case ix::kStartV0: order.insert(order.end(), n, kV0); break;
    }
  });
  auto landed = [&](Tile t, int left) {
    bool started = false;
    for (size_t i = 0; i < order.size(); ++i) {
      if (order[i] != t) continue;
      if (i + left >= order.size()) return false;
      started = true;
    }
    return started;
  };
  return landed(kK0, ix::group_left_at_scores<G>()) && landed(kQ, ix::group_left_at_scores<G>()) &&
         landed(kK1, ix::group_left_at_maximum<G>());
}

int main() {
  int bad = 0;
  const long n = sweep<2>(bad) + sweep<4>(bad);
  if (!start_waits<2>() || !start_waits<4>()) return std::printf("FAIL waits ahead of the loop\n"), 1;
  if (bad) return 1;
  std::printf("ok: %ld configurations\n", n);
  return 0;
}
