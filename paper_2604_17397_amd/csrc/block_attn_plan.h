// The launch plan of the bf16 attention kernels: which kernel a call takes, and how it is cut into
// workgroups. Host arithmetic only, from sizes and the number of compute units; the tests compile it
// (tests/host/attn_plan.cpp) to tell which kernel each of their cases runs.
#pragma once
#include <stdint.h>

#include "block_attn_index.h"
#include "sdvg.h"

namespace sdvg {

// Floats one workgroup writes per partial result: 8 waves x (64 accumulators + row sum + shift) x 64 lanes.
constexpr int64_t kPartialFloats = 8 * 66 * 64;

constexpr int kPlanRows = 256;  // query rows of a workgroup without key groups

// How a launch is cut into workgroups. Plain: one workgroup per query tile (units == n_tiles).
// Key split: when the query tiles would leave a good part of the last round of workgroups idle
// (5 heads x 19 query tiles are 95 workgroups for 256 compute units), every query tile's keys are cut into equal
// columns, as many as there is room for, and the workgroups left over share what the columns leave (cut_keys); the
// pieces leave partial results that a second, small kernel merges.
struct Plan {
  int n_qtiles, n_hq, n_tiles;
  int units;     // key tiles of a workgroup; == n_tiles when nothing is split
  int total_wg;  // workgroups
  attn_index::KeySplit split;
  int64_t workspace_bytes;  // what a caller is asked for; 0 when no split was considered
  int groups;               // key groups per workgroup (1: block_attn.hip, 2 or 4: block_attn_groups.hip)
  int rows;                 // query rows per workgroup (32: block_attn_rows32.hip)
  bool halves;              // two workgroups per 32 rows, each with half of the output dims
  double us;                // estimated time without a split
};

// Key groups per workgroup, and the query rows they share. Estimated time: rounds of workgroups over the
// compute units, times a fixed part plus the key tiles each group walks.
// Measured on MI355X, us among others in a graph (1 / 2 / 4 groups; workgroups of 256 / 128 / 64 rows in brackets):
//   12 heads x 312 x 936 keys [24/36/60] 25.7 / 17.5 / 13.1; 12 x 1031 x 6186 [60/108/204] 104 / 62 / 47;
//   12 x 1560 x 4680 [84/156/300] 83 / 51 / 70; 5 x 4680 x 32760 [95/185/370] 505 / 350 / 448;
//   40 x 1031 x 3093 [200/360/680] 73 / 86 / 97; 16 x 4680 x 14040 [304/592/1184] 554 / 482 / 543;
//   12 x 4680 x 14040 [228/444/888] 314 / 337 / 450.
// A tile takes 1.0 us alone on the chip and 1.5 us on a full one (power), hence the middle value, and
// the estimate is up to 25 % off in absolute terms; what counts is the order. Over 1 to 40 heads, 156
// to 4680 rows and 193 to 32760 keys it is within 1 % of the fastest of the four in 296 of 299 launches and 4 to 9 % off in
// three, where 64 rows beat 32 (profiles/attn_plan_sweep.txt, as the other figures here). Up to 192 keys it stays with
// 1 group, where more are faster (3 heads x 250 rows x 128 keys 11.8 / 7.4 / 6.3).
// Of the launches of four groups, those whose 32-row workgroups need no more rounds than 64-row ones take the kernel
// where the two waves of a group share 32 rows and deal the group's tiles out as well (rows = 32). One round, us
// with 64 / 32 rows: 12 x 312 x 936 13.1 / 9.4; 16 x 500 x 1000 13.8 / 12.1; 8 x 1024 x 6144 41.1 / 39.3, with keys from
// HBM 61.4 / 46.1. (4 x 2000 x 14000 loses, 83.5 / 96.2, where the memory-side cache holds the layer's 29 MB; the layers of
// a model of this size come from HBM, 129 / 95.) More rounds with as many workgroups (up to 32 rows), before the copies from
// scalar addresses (block_attn_groups.hip), which gave 64 rows 1 to 2 %: 300 x 32 x 512 24.6 / 22.7; 259 x 1 x 936 34.7 / 33.2.
// In a round more than with 64 rows every workgroup walks all keys again: 12 x 1031 x 1031 14.1 / 20.1; 320 x 33 x 256 16.8 /
// 20.3; 300 x 64 x 256 17.7 / 18.5.
struct Groups {
  int groups, rows;
  double us;  // the estimate
};
inline Groups choose_groups(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, bool rows32_ok) {
  if (n_cu <= 0) return Groups{1, kPlanRows, 0};
  const struct { int groups, rows, keys, walkers; double fixed_us, tile_us; } variants[] = {
      {1, 256, 64, 1, 4.0, 1.25}, {2, 128, 64, 2, 5.5, 1.3}, {4, 64, 32, 4, 6.0, 0.9}, {4, 32, 32, 8, 3.5, 1.4}};
  Groups best{1, kPlanRows, 0};
  int64_t best_rounds = 0;
  for (const auto &v : variants) {
    if (v.rows == 32 && (best.groups != 4 || !rows32_ok)) continue;
    const int64_t wgs = static_cast<int64_t>(n_items) * n_heads * ((n_q + v.rows - 1) / v.rows);
    const int64_t tiles = (n_k + v.keys - 1) / v.keys, its = (tiles + v.walkers - 1) / v.walkers;
    const int64_t rounds = (wgs + n_cu - 1) / n_cu;
    if (v.rows == 32 && rounds > best_rounds) continue;
    const double us = static_cast<double>(rounds) * (v.fixed_us + static_cast<double>(its) * v.tile_us);
    if (v.groups == 1 || us < best.us) {
      best = Groups{v.groups, v.rows, us};
      best_rounds = rounds;
    }
  }
  return best;
}

// An unsplit launch in two, one behind the other on its stream: `heads` heads of every item, or `rows` query rows of every
// head, and then the rest; 0, 0: one launch. Where the 256-row workgroups fill some rounds and a small part of another, one
// launch takes that round for little (16 heads x 19 query tiles: 304 workgroups for 256 compute units) or takes
// smaller workgroups for all rows, which copy and read every key tile for fewer rows. In two, the whole rounds
// keep 256 rows and only the rest is cut finer. Nothing is merged, no row is computed in two parts. us, one / two launches:
//   13 + 3 heads x 4680 x 14040 498 / 445, 13 + 1 x 4680 x 23400 801 / 667, 36 + 2 x 1757 x 12299 434 / 374,
//   15 + 4 x 4112 x 24672 860 / 813, 21 + 9 x 3044 x 12176 466 / 460, 128 + 11 x 410 x 897 58 / 43, 256 + 3 x 183 x 342 36 / 28.
// With the estimate of choose_groups, of 174 drawn launches of more than a round (3 to 400 heads, 1 to 4680 rows) that it
// would rather cut, 108 are cut by this rule, 7.8 % faster on average (0.988 to 1.32 times as fast;
// profiles/attn_two_launches.txt); without the 2 % and 8 us
// (a launch's start and end, and compute units that wait for the slowest) two more are slower. A launch that
// fills less than a round of 256-row workgroups never gains, although the estimate of a finer first part would have it so:
// 18 heads x 1800 x 10800, 144 workgroups, 179 / 190, as fewer busy compute units run at a higher clock.
struct Cut {
  int heads, rows;
};
inline Cut choose_cut(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, bool rows32_ok) {
  Cut best{0, 0};
  const int64_t tiles = (n_q + kPlanRows - 1) / kPlanRows, per_head = n_items * tiles, all = n_heads * per_head;
  if (n_cu <= 0 || all <= n_cu || all % n_cu == 0) return best;
  const int64_t full = all / n_cu * n_cu;  // workgroups of the whole rounds
  auto us = [&](int heads, int rows) { return choose_groups(n_items, rows, heads, n_k, n_cu, rows32_ok).us; };
  double limit = (us(n_heads, n_q) - 8.0) / 1.02;
  const int heads = static_cast<int>(full / per_head);
  if (heads > 0) {  // (< n_heads, because full < all)
    const double t = us(heads, n_q) + us(n_heads - heads, n_q);
    if (t < limit) {
      limit = t;
      best = Cut{heads, 0};
    }
  }
  const int64_t rows = full / (static_cast<int64_t>(n_items) * n_heads) * kPlanRows;
  if (rows > 0 && rows < n_q) {
    const double t = us(n_heads, static_cast<int>(rows)) + us(n_heads, static_cast<int>(n_q - rows));
    if (t < limit) best = Cut{0, static_cast<int>(rows)};
  }
  return best;
}

// Cuts n_tiles key tiles of each of n_hq query tiles over `wgs` >= n_hq workgroups (block_attn_index.h, "key split").
// As many whole columns as there is room for; the workgroups left over are helpers. A piece costs some 10 us beside its
// tiles (arguments, query rows and first tiles 7, partial result 3, by clock stamps in the kernel), and a helper has
// several. With n_hq / n_help + 1 pieces of rest + kPieceTiles, helpers and columns are done at the same time where
//   col = (n_tiles + kPieceTiles) * n_hq / wgs.
// kPieceTiles = 2 / 6 / 10 / 14 / 20, us: 5 heads x 4680 x 32760 338 / 336 / 334 / 330 / 330, 16 x 4680 x 14040
// 462 / 466 / 465 / 465 / 474, 20 x 4680 x 18720 744 / 752 / 750 / 755 / 763, 13 x 1560 x 9360 111 / 110 / 107 / 105 / 107.
constexpr int kPieceTiles = 10;
inline attn_index::KeySplit cut_keys(int n_hq, int n_tiles, int wgs) {
  attn_index::KeySplit ks{wgs / n_hq, 0, wgs % n_hq, 0};
  const int64_t part = static_cast<int64_t>(n_tiles + (ks.n_help ? kPieceTiles : 0)) * n_hq;
  ks.col = static_cast<int>(ks.n_help ? (part + wgs - 1) / wgs : (n_tiles + ks.cols - 1) / ks.cols);
  const int64_t rest = n_tiles - static_cast<int64_t>(ks.cols) * ks.col;
  if (rest < 1 && ks.cols > 1) {  // nothing for helpers to do
    ks.n_help = 0;
    ks.col = (n_tiles + ks.cols - 1) / ks.cols;
    ks.cols = (n_tiles + ks.col - 1) / ks.col;
    return ks;
  }
  if (rest < 1) {
    // Few workgroups are left over for many query tiles (ALWAYS only): equal runs of all pairs, at most two pieces each. 250
    // query tiles of 220 key tiles, 50 heads x 1250 x 14080: 388 us, 374 unsplit; six helpers would have 42 pieces each.
    const int64_t all = static_cast<int64_t>(n_hq) * n_tiles;
    const int run = static_cast<int>((all + wgs - 1) / wgs);
    return run < n_tiles ? attn_index::KeySplit{0, 0, static_cast<int>((all + run - 1) / run), run} : attn_index::KeySplit{0, 0, 0, 0};
  }
  ks.run = static_cast<int>((n_hq * rest + ks.n_help - 1) / ks.n_help);
  ks.n_help = static_cast<int>((n_hq * rest + ks.run - 1) / ks.run);
  return ks;
}

// SDVG_SPLIT_AUTO considers the split from this share of idle workgroup slots on: with a workspace of the caller's, and
// with the library's own array, which holds fewer partial results and which calls that overlap must not share, so that no
// more shapes split there than have to.
constexpr double kAutoIdle = 0.25, kAutoIdleStatic = 0.6;

// Bytes from the first to the last of n_tokens x n_heads rows of 128 bf16 values, and whether two ranges share a byte.
inline int64_t rows_bytes(int64_t n_tokens, int64_t n_heads, int64_t token_stride, int64_t head_stride) {
  return ((n_tokens - 1) * token_stride + (n_heads - 1) * head_stride + 128) * 2;
}
inline bool ranges_overlap(const void *a, int64_t a_bytes, const void *b, int64_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + static_cast<uintptr_t>(b_bytes) && y < x + static_cast<uintptr_t>(a_bytes);
}

// rows32_ok: the strides are ones that the 32-row kernel takes. in_place: an item's result overlaps its query rows.
inline Plan make_plan(int n_items, int n_q, int n_heads, int64_t n_k, int n_cu, int split_mode, bool rows32_ok = true,
                      double auto_idle = kAutoIdle, bool in_place = false) {
  const Groups unsplit_best = choose_groups(n_items, n_q, n_heads, n_k, n_cu, rows32_ok);
  auto unsplit = [&](int groups, int rows) {
    const int keys = groups == 4 ? 32 : attn_index::kBN;
    Plan pl;
    pl.groups = groups;
    pl.rows = rows;
    pl.n_qtiles = (n_q + rows - 1) / rows;
    pl.n_hq = pl.total_wg = n_items * n_heads * pl.n_qtiles;
    pl.n_tiles = pl.units = static_cast<int>((n_k + keys - 1) / keys);
    pl.split = attn_index::KeySplit{0, 0, 0, 0};
    // 32-row workgroups that leave half of the compute units idle are doubled: each of a pair copies all of K but half of V,
    // and copies are what bounds them (block_attn_rows32.hip). Whole / halves, us in a graph with one set of tensors, four sets in
    // turn, keys from HBM: 12 heads x 312 x 936 keys 9.3 / 8.6, 10.3 / 8.9, 12.5 / 10.5; 4 x 1000 x 4000 22.4 / 21.0, 24.7 / 21.4,
    // 31.9 / 25.8; 3 x 1300 x 9100 50 / 42, 50 / 42, 60 / 48. In a second round every pair would copy K again. Both of a
    // pair read whole query rows and store half of them, at times of their own: not where the result lies over the query.
    pl.halves = rows == 32 && 2 * pl.total_wg <= n_cu && !in_place;
    pl.workspace_bytes = 0;
    pl.us = unsplit_best.us;
    return pl;
  };
  auto plain = [&]() { return unsplit(unsplit_best.groups, unsplit_best.rows); };
  if (split_mode == SDVG_SPLIT_NEVER || n_cu <= 0) return plain();
  Plan pl = unsplit(1, kPlanRows);
  const int rounds = (pl.n_hq + n_cu - 1) / n_cu;
  const double idle = 1.0 - static_cast<double>(pl.n_hq) / (static_cast<double>(rounds) * n_cu);
  // The split costs a second kernel, the partial results' traffic and a slower main kernel, and
  // a chip that is only partly busy clocks higher: 228 busy compute units take a tile in 1.46 us, 256 in 1.61, so
  // that 11 % idle cost nothing. Measured on MI355X, us, the fastest without a split / split, at 4680 rows:
  //   11 % idle  12 heads x 14040 keys 314 / 319, x 32760 710 / 694, 24 x 14040 619 / 637
  //   18 - 26 %  11 x 32760 676 / 641, 20 x 18720 700 / 700
  //   33 - 48 %  8 x 32760 557 / 482, 8 x 14040 242 / 224, 14 x 23400 782 / 631
  // From kAutoIdle on the estimates decide (below).
  if (pl.n_hq % n_cu == 0 || rounds > 4 || pl.n_tiles < 32) return plain();
  if (split_mode == SDVG_SPLIT_AUTO && idle < auto_idle) return plain();
  const int64_t all = static_cast<int64_t>(pl.n_hq) * pl.n_tiles;
  const int64_t wgs = static_cast<int64_t>(rounds) * n_cu;
  const int even = static_cast<int>((all + wgs - 1) / wgs);  // pairs per workgroup; <= n_tiles, because wgs >= n_hq
  if (even < 16 || all > INT32_MAX) return plain();  // (the cut is made in 32 bits)
  const int max_wg = static_cast<int>((all + even - 1) / even);
  pl.workspace_bytes = static_cast<int64_t>(pl.n_hq + max_wg) * kPartialFloats * 4;
  pl.split = cut_keys(pl.n_hq, pl.n_tiles, max_wg);
  if (pl.split.any()) {
    pl.units = pl.split.cols ? pl.split.col : pl.split.run;
    pl.total_wg = pl.n_hq * pl.split.cols + pl.split.n_help;
  }
  // Launch, merge and 1.53 us per key tile of a workgroup, against the estimate without a split. Split /
  // unsplit, us: 1 head x 4680 x 32760 80 / 146, 5 heads 307 / 350; 4 x 4680 x 14040 121 / 139,
  // 5 heads 146 / 153; 12 x 1560 x 4680 57 / 51, 16 x 1031 x 3093 41 / 37, 3 x 4680 x 4680 46 / 38.
  // (Of 299 launches without a batch 10 would gain 3 to 22 % from a split that the estimate does not take, 0.3 % on average.)
  // Below 60 % idle the unsplit estimate, made for a full chip, is a little high for one that is half busy: the split
  // has to win by 11 us there. Of 110 launches drawn at 25 to 60 % idle (1 to 3 items, up to 40 heads, 312 to 4680 rows,
  // 1 to 7 blocks of keys) 31 are split, 4 to 15 % faster each; 10 more would have gained 4 to 11 %. (Against one launch.
  // Against two, choose_cut, which this does not weigh: of 80 drawn launches of more than a round 21 are split, 2.4 % faster on
  // average, the worst 4 % slower; 7 more would have gained 3 to 8 %.)
  const double split_us = 33.0 + 1.53 * rounds * static_cast<double>(even);
  const bool few = idle >= kAutoIdleStatic;
  if (split_mode == SDVG_SPLIT_AUTO && unsplit_best.us < split_us + (few ? 0.0 : 11.0)) {
    Plan g = plain();
    // (from 60 % idle on, what a caller allocates does not depend on this choice)
    if (few) g.workspace_bytes = pl.workspace_bytes;
    return g;
  }
  return pl;
}

// Attention workgroups that an unsplit plan launches.
inline int attention_workgroups(const Plan &pl) { return pl.halves ? 2 * pl.total_wg : pl.total_wg; }

// Copying workgroups of a fused commit of `rows` rows (tokens x heads): as many as the last round of attention workgroups
// leaves compute units idle on every XCD (they then run beside it for its whole length); a full round if none; none
// without a row (32 rows per workgroup and pass). Workgroups go to the XCDs in turn, so that one more than has room on its
// XCD would begin when the round ends, although others have room: 12 heads x 4680 x 9360, 29 of 32 compute units of seven
// XCDs at work, took 28 us longer with 28 copying workgroups than with 24. Workgroups of 32 rows doubled, 16 / 136 beside
// the 240 of 12 x 312 x 312 7.0 / 7.8 us, keys from HBM 6.6 / 7.2; x 936 10.0 / 10.5, 10.4 / 10.8; 16 / 136 beside the
// 240 of 15 x 250 x 500 8.3 / 9.0, 7.9 / 8.8. Behind the full round of 8 x 500 x 1500 (256), 16 / 32 / 64 / 125 / 256
// 15.9 / 14.0 / 13.4 / 12.9 / 13.1 us.
// Copies that would outlast the round are not held up in these few workgroups: a full round of them takes what is left
// when the attention ends. A pass of 32 x 4 rows beside the attention takes 2.5 to 3.6 us (kCopyPass), a full round of
// 256 copies at the rate of HBM, 4.2 us for a pass. Attention alone / copies in the room / by a full round, us:
// 40 x 4680 x 4680 384 / 720 / 411, x 18720 1416 / 1599 / 1436, x 32760 2438 / 2440 / 2457; 13 x 4680 x 4680 130 / 151 / 137,
// x 9360 243 / 244 / 249; 30 x 2000 x 2000 65 / 76 / 72; 24 x 312 x 312 8.0 / 10.6 / 9.2, x 936 12.0 / 12.2 / 12.9.
constexpr int kCopyRows = 32 * 4;  // rows of a copying workgroup and pass
constexpr double kCopyPass = 2.7, kFullPass = 4.2;
inline int copy_workgroups(const Plan &pl, int64_t rows, int n_cu) {
  const int xcd_cus = n_cu > 8 ? n_cu / 8 : 32;
  const int work = attention_workgroups(pl), rounds = (work + 8 * xcd_cus - 1) / (8 * xcd_cus);
  int n = 8 * (xcd_cus - (work + 7) / 8 % xcd_cus);
  const int64_t passes = (rows + int64_t{n} * kCopyRows - 1) / (int64_t{n} * kCopyRows);
  const double late_us = static_cast<double>(passes) * kCopyPass - pl.us / rounds;
  if (late_us > 1.0 + kFullPass * static_cast<double>(rows) / (8.0 * xcd_cus * kCopyRows)) n = 8 * xcd_cus;
  return static_cast<int>(n * int64_t{32} < rows ? n : (rows + 31) / 32);
}

}  // namespace sdvg
