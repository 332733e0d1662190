// Host check of csrc/row_map.h: FastDiv against the division operator at the edges of quotients,
// RowMap against plain loops for token-major, head-major and padded layouts, and the launch shape of
// the row kernels against what a grid dimension can hold. Exit code 0 = passed.
#include <cstdio>
#include <vector>

#include "row_map.h"

using sdvg::FastDiv;
using sdvg::RowMap;

int main() {
  const uint32_t top = (uint32_t{1} << 31) - 1;
  std::vector<uint32_t> divisors;
  for (uint32_t d = 1; d < 5000; ++d) divisors.push_back(d);
  for (int b = 12; b < 31; ++b)
    for (int64_t e = -2; e <= 2; ++e) divisors.push_back(static_cast<uint32_t>((int64_t{1} << b) + e));
  divisors.push_back(top);
  for (uint32_t d : divisors) {
    const FastDiv f = FastDiv::of(d);
    for (uint64_t q : {uint64_t{0}, uint64_t{1}, uint64_t{2}, uint64_t{12345}, uint64_t{top / d}, uint64_t{top / d / 2}})
      for (int64_t e = -1; e <= 1; ++e) {
        const int64_t n = static_cast<int64_t>(q * d) + e;
        if (n < 0 || n > top) continue;
        if (f.div(static_cast<uint32_t>(n)) != static_cast<uint32_t>(n) / d)
          return std::printf("FAIL %lld / %u\n", static_cast<long long>(n), d), 1;
      }
    if (f.div(top) != top / d) return std::printf("FAIL top / %u\n", d), 1;
  }
  struct Case {
    int64_t L, T, H, ls, ts, hs;
  };
  for (const Case &c : {Case{3, 7, 5, 7 * 5 * 128, 5 * 128, 128}, Case{3, 7, 5, 5 * 9 * 128, 128, 9 * 128},
                        Case{2, 1, 1, 4096, 128, 128}, Case{4, 13, 3, 100000, 3 * 136 + 8, 136}, Case{1, 2, 12, 1 << 20, 128, 256}}) {
    const RowMap m = sdvg::row_map(c.T, c.H, c.ls, c.ts, c.hs);
    std::vector<int> seen(c.L * c.T * c.H, 0);
    int64_t last = -1;
    for (uint32_t r = 0; r < seen.size(); ++r) {
      const RowMap::Row row = m.row(r);
      const int64_t t = m.token(row), h = m.token_inner ? row.mid : row.inner, l = row.layer;
      if (t >= c.T || h >= c.H || l >= c.L || seen[(l * c.T + t) * c.H + h]++) return std::printf("FAIL rows\n"), 1;
      if (m.dst(row) != l * c.ls + t * c.ts + h * c.hs || m.src(row) != ((l * c.T + t) * c.H + h) * 128)
        return std::printf("FAIL offsets\n"), 1;
      if (m.dst(row) <= last) return std::printf("FAIL order\n"), 1;
      last = m.dst(row);
    }
  }
  // Every row below the limit is some workgroup's, and no grid dimension holds 2^32 threads.
  const int64_t edge = int64_t{1} << 28;
  for (int64_t n : {int64_t{1}, int64_t{16}, int64_t{17}, sdvg::kSliceRows - 1, sdvg::kSliceRows, sdvg::kSliceRows + 1, edge - 1,
                    edge, edge + 1, 3 * edge + 5, sdvg::kMaxRows - 1}) {
    const sdvg::RowGrid g = sdvg::row_grid(n);
    if (g.x < 1 || g.z < 1 || uint64_t{g.x} * sdvg::kRowThreads >= uint64_t{1} << 32 || g.z > 65535)
      return std::printf("FAIL grid of %lld rows\n", static_cast<long long>(n)), 1;
    int64_t next = 0;  // rows come in order: each slice begins where the one before it ended
    for (uint32_t z = 0; z < g.z; ++z) {
      if (sdvg::row_of(0, z, 0) != next) return std::printf("FAIL first row of a slice\n"), 1;
      next = int64_t{sdvg::row_of(g.x - 1, z, sdvg::kRowThreads - 1)} + 1;
    }
    if (next < n || sdvg::row_of(0, g.z - 1, 0) >= n) return std::printf("FAIL rows of %lld\n", static_cast<long long>(n)), 1;
    for (int t : {0, 15, 16, 255})
      if (sdvg::row_of(3, 0, t) != static_cast<uint32_t>(48 + t / 16)) return std::printf("FAIL row of a thread\n"), 1;
  }
  std::printf("ok\n");
  return 0;
}
