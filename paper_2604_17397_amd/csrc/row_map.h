// Which row (layer, token, head) a thread of the copy kernels works on, and where that row lies.
// Plain integer arithmetic, host and device.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define SDVG_ROW_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define SDVG_ROW_HD inline
#endif

namespace sdvg {

// n / d for 0 <= n < 2^31 and a divisor 1 <= d < 2^31 fixed at launch, by multiplication with a rounded-up
// reciprocal (Granlund and Montgomery, "Division by Invariant Integers using Multiplication", 1994): n * m
// >> (31 + s) with
// s = ceil(log2 d) and m = floor(2^(31+s) / d) + 1. m * d exceeds 2^(31+s) by e <= d <= 2^s, so the
// quotient is exact because n * e < 2^(31+s). (A 64-bit division by a run-time value is some 100
// vector instructions, more than everything else a copying thread does.)
struct FastDiv {
  uint32_t d, m, s;
  static FastDiv of(uint32_t d) {
    uint32_t s = 0;
    while ((uint64_t{1} << s) < d) ++s;
    return FastDiv{d, static_cast<uint32_t>((uint64_t{1} << (31 + s)) / d + 1), s};
  }
  SDVG_ROW_HD uint32_t div(uint32_t n) const { return static_cast<uint32_t>((static_cast<uint64_t>(n) * m) >> (31 + s)); }
};

// Rows numbered ((layer * n_mid) + mid) * n_inner + inner, where (mid, inner) are (token, head) or
// (head, token): whichever of the two has the smaller stride in the destination is the inner one, so
// that neighbouring rows are written to neighbouring addresses.
struct RowMap {
  FastDiv inner, mid;
  int64_t dst_layer, dst_mid, dst_inner;  // elements
  int64_t src_layer, src_mid, src_inner;
  bool token_inner;

  struct Row {
    uint32_t layer, mid, inner;
  };
  SDVG_ROW_HD Row row(uint32_t r) const {
    const uint32_t lm = inner.div(r), l = mid.div(lm);
    return Row{l, lm - l * mid.d, r - lm * inner.d};
  }
  SDVG_ROW_HD int64_t dst(const Row &r) const { return r.layer * dst_layer + r.mid * dst_mid + r.inner * dst_inner; }
  SDVG_ROW_HD int64_t src(const Row &r) const { return r.layer * src_layer + r.mid * src_mid + r.inner * src_inner; }
  SDVG_ROW_HD uint32_t token(const Row &r) const { return token_inner ? r.inner : r.mid; }
};

// Destination strided, source dense [layer][n_tokens][n_heads][128].
inline RowMap row_map(int64_t n_tokens, int64_t n_heads, int64_t layer_stride, int64_t token_stride, int64_t head_stride) {
  const bool token_inner = token_stride < head_stride;
  const int64_t src_t = n_heads * 128, src_h = 128;
  const uint32_t nt = static_cast<uint32_t>(n_tokens), nh = static_cast<uint32_t>(n_heads);
  return RowMap{FastDiv::of(token_inner ? nt : nh), FastDiv::of(token_inner ? nh : nt),
                layer_stride,      token_inner ? head_stride : token_stride, token_inner ? token_stride : head_stride,
                n_tokens * src_t,  token_inner ? src_h : src_t,              token_inner ? src_t : src_h,
                token_inner};
}

// Rows of 256 bytes beyond this many (512 GiB) do not fit the device.
constexpr int64_t kMaxRows = int64_t{1} << 31;

// Launch shape of the kernels that give a row to 16 threads. A grid dimension holds fewer than 2^32
// threads, which is 2^28 rows (64 GiB of one tensor, which does fit the device): x takes slices of
// kSliceRows, z counts the slices. 1 <= n_rows < kMaxRows.
constexpr int kRowThreads = 256;
constexpr int64_t kSliceRows = int64_t{1} << 27;
struct RowGrid {
  uint32_t x, z;
};
inline RowGrid row_grid(int64_t n_rows) {
  const int64_t in_x = n_rows < kSliceRows ? n_rows : kSliceRows;
  return RowGrid{static_cast<uint32_t>((in_x + kRowThreads / 16 - 1) / (kRowThreads / 16)),
                 static_cast<uint32_t>((n_rows + kSliceRows - 1) / kSliceRows)};
}
SDVG_ROW_HD uint32_t row_of(uint32_t block_x, uint32_t block_z, uint32_t thread) {
  return block_z * static_cast<uint32_t>(kSliceRows) + block_x * (kRowThreads / 16) + (thread >> 4);
}

}  // namespace sdvg
