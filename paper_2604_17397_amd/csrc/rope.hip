// Rotary position embedding of q / k rows, alone and fused into the KV commit.
// Paper Sec. 4.1 "Models": the attention backbone caches K/V "via RoPE positional embeddings"; no
// formula is printed. Reading taken: consecutive elements (2i, 2i+1) of a head's vector are the
// real and imaginary part of a complex number that is multiplied by exp(i * angle), the angle of
// (token, pair) being supplied by the caller as fp32 tables cos / sin [token][64] -- so the position
// scheme (1-D, or the 3-D frame / row / column scheme of video transformers) stays the caller's.
// Arithmetic: fp32 in a fixed order (each product and each fma rounded once), result rounded to
// bf16 (RNE):  re' = fma(re, cos, -(im * sin)),  im' = fma(re, sin, im * cos).
//
// Why K is rotated on its way INTO the cache and not "on load" in the attention kernel: K tiles
// go from HBM to LDS without passing through registers, and every one of a head's 19 workgroups
// would have to rotate every tile again. Rotating once, in the bandwidth-bound copy that commits
// the block, costs nothing; q and the current block's K are rotated by the plain kernel (one
// pass over 48 MB in and out per tensor and layer at the target shape, 17 us against 2.4 ms of attention).
#include "row_map.h"
#include "sdvg_common.h"

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Rotates the four pairs held in one 16-byte chunk (8 bf16) by the angles (c[i], s[i]).
__device__ __forceinline__ u32x4 rotate_chunk(u32x4 x, f32x4 c, f32x4 s) {
  u32x4 y;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float re = __uint_as_float(x[i] << 16), im = __uint_as_float(x[i] & 0xffff0000u);
    const float im_sin = __fmul_rn(im, s[i]), im_cos = __fmul_rn(im, c[i]);
    const f32x2 r = {__fmaf_rn(re, c[i], -im_sin), __fmaf_rn(re, s[i], im_cos)};
    const bf16x2 b = __builtin_convertvector(r, bf16x2);
    unsigned int packed;
    __builtin_memcpy(&packed, &b, 4);
    y[i] = packed;
  }
  return y;
}

// One 16-byte chunk per thread: row r = token * n_heads + head.
// Small tensors: a chain of latencies. Every trip to memory for arguments costs 0.3 us, so this file is
// compiled with the first 14 dwords of arguments preloaded into registers (build.py); kDense needs no more than
// those. Two passes and an attention call of 12 heads x 312 rows took 17.8 us in a graph, 17.3 with
// 9 dwords preloaded, 16.4 as it is now (with ordinary stores, below).
// Large ones: HBM bound. q of a target layer (48 MB in, 48 MB out) takes 17.1 us; with ordinary stores, which
// displace what is still to be read, 18.8 to 19.6 (with a nontemporal load as well: 19.0).
template <bool kDense, bool kStream>
__global__ __launch_bounds__(sdvg::kRowThreads) void rope_kernel(
    uint32_t n_rows, uint32_t heads_d, uint32_t heads_m, uint32_t heads_s, const uint16_t *__restrict__ x,
    const float *__restrict__ cos_t, const float *__restrict__ sin_t, uint16_t *out, int64_t x_ts, int64_t x_hs,
    int64_t o_ts, int64_t o_hs) {
  const uint32_t r = sdvg::row_of(blockIdx.x, blockIdx.z, threadIdx.x);
  if (r >= n_rows) return;
  const int ch = threadIdx.x & 15;
  const uint32_t tok = sdvg::FastDiv{heads_d, heads_m, heads_s}.div(r), head = r - tok * heads_d;
  const int64_t from = kDense ? static_cast<int64_t>(r) * 128 : tok * x_ts + head * x_hs;
  const int64_t to = kDense ? static_cast<int64_t>(r) * 128 : tok * o_ts + head * o_hs;
  const u32x4 v = *reinterpret_cast<const u32x4 *>(x + from + ch * 8);
  const f32x4 c = *reinterpret_cast<const f32x4 *>(cos_t + static_cast<int64_t>(tok) * 64 + ch * 4);
  const f32x4 s = *reinterpret_cast<const f32x4 *>(sin_t + static_cast<int64_t>(tok) * 64 + ch * 4);
  const u32x4 y = rotate_chunk(v, c, s);
  u32x4 *dst = reinterpret_cast<u32x4 *>(out + to + ch * 8);
  if (kStream)
    __builtin_nontemporal_store(y, dst);
  else
    *dst = y;
}

// Commit with the rotation of K fused in: grid.y = 0 (K, rotated) / 1 (V, copied), rows in the order
// of their destinations (RowMap). Source dense [L][T][H][128]. The drafter's commit (30 layers x 4680
// tokens x 12 heads): 268 us = 6.45 TB/s, the rate of the plain commit; with a 64-bit division per
// thread to find its row it was bound by the vector units: 287 us.
__global__ __launch_bounds__(sdvg::kRowThreads) void kv_commit_rope_kernel(
    const uint16_t *__restrict__ k_src, const uint16_t *__restrict__ v_src, uint16_t *__restrict__ k_dst,
    uint16_t *__restrict__ v_dst, const float *__restrict__ cos_t, const float *__restrict__ sin_t, sdvg::RowMap m,
    uint32_t n_rows) {
  const uint32_t r = sdvg::row_of(blockIdx.x, blockIdx.z, threadIdx.x);
  if (r >= n_rows) return;
  const bool is_v = blockIdx.y != 0;
  const int ch = threadIdx.x & 15;
  const sdvg::RowMap::Row row = m.row(r);
  const uint16_t *src = (is_v ? v_src : k_src) + m.src(row) + ch * 8;
  uint16_t *dst = (is_v ? v_dst : k_dst) + m.dst(row) + ch * 8;
  u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src));
  if (!is_v) {
    const int64_t t = static_cast<int64_t>(m.token(row)) * 64 + ch * 4;
    v = rotate_chunk(v, *reinterpret_cast<const f32x4 *>(cos_t + t), *reinterpret_cast<const f32x4 *>(sin_t + t));
  }
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
}

// Up to this many rows (4 MiB, an XCD's L2) the result is stored in the ordinary way, and dense tensors take the
// kernel that needs no strides. us, a pair of passes alone / with the attention that reads them, nontemporal and ordinary
// stores: 12 heads x 312 rows 4.27 / 12.1 and 4.27 / 11.4; 12 x 1031 5.2 / 23.5 and 5.3 / 22.8; 12 x 1560 (4.8 MB)
// 5.9 / 34.3 and 6.2 / 33.5; 24 x 1560 8.5 / 52.5 and 9.4 / 52.1. Beyond 16 MB the dense kernel loses to the strided one
// (40 x 4680: 38.0 and 35.1 a pair), presumably because its workgroups start closer together.
constexpr int64_t kCachedRows = 1 << 14;

bool stride_ok(int64_t st) { return st >= 128 && (st & 7) == 0; }

}  // namespace

extern "C" int sdvg_rope(const void *x, const float *cos_table, const float *sin_table, void *out,
                         int64_t n_tokens, int32_t n_heads, int32_t head_dim, int64_t x_token_stride,
                         int64_t x_head_stride, int64_t out_token_stride, int64_t out_head_stride, void *stream) {
  if (n_tokens < 0 || n_heads < 1) return SDVG_ERR_SHAPE;
  if (head_dim != 128) return SDVG_ERR_UNSUPPORTED;
  if (n_tokens == 0) return SDVG_OK;
  if (!x || !cos_table || !sin_table || !out) return SDVG_ERR_NULL;
  if (!stride_ok(x_token_stride) || !stride_ok(x_head_stride) || !stride_ok(out_token_stride) ||
      !stride_ok(out_head_stride))
    return (x_token_stride < 128 || x_head_stride < 128 || out_token_stride < 128 || out_head_stride < 128)
               ? SDVG_ERR_SHAPE
               : SDVG_ERR_ALIGN;
  if (!sdvg::aligned16(x) || !sdvg::aligned16(out) || !sdvg::aligned16(cos_table) || !sdvg::aligned16(sin_table))
    return SDVG_ERR_ALIGN;
  if (n_tokens > (sdvg::kMaxRows - 1) / n_heads) return SDVG_ERR_UNSUPPORTED;
  const int64_t n_rows = n_tokens * n_heads;
  const sdvg::RowGrid g = sdvg::row_grid(n_rows);
  const int64_t row_of_heads = int64_t{128} * n_heads;
  const bool dense = (n_heads == 1 || (x_head_stride == 128 && out_head_stride == 128)) &&
                     (n_tokens == 1 || (x_token_stride == row_of_heads && out_token_stride == row_of_heads));
  const auto kernel = n_rows > kCachedRows ? rope_kernel<false, true> : dense ? rope_kernel<true, false> : rope_kernel<false, false>;
  const sdvg::FastDiv heads = sdvg::FastDiv::of(n_heads);
  hipLaunchKernelGGL(kernel, dim3(g.x, 1, g.z), dim3(sdvg::kRowThreads), 0, static_cast<hipStream_t>(stream),
                     static_cast<uint32_t>(n_rows), heads.d, heads.m, heads.s, static_cast<const uint16_t *>(x),
                     cos_table, sin_table, static_cast<uint16_t *>(out), x_token_stride, x_head_stride,
                     out_token_stride, out_head_stride);
  SDVG_HIP_CHECK(hipGetLastError());
  return SDVG_OK;
}

extern "C" int sdvg_kv_commit_rope(sdvg_kv_cache *cache, const void *k_blk, const void *v_blk, int32_t slot,
                                   const float *cos_table, const float *sin_table, void *stream) {
  if (!cos_table || !sin_table) return SDVG_ERR_NULL;
  if (!sdvg::aligned16(cos_table) || !sdvg::aligned16(sin_table)) return SDVG_ERR_ALIGN;
  // the same checks as the plain commit (descriptor, slot, alignment, aliasing), without a launch
  int st = sdvg::check_commit_args(cache, k_blk, v_blk, slot);
  if (st != SDVG_OK) return st;
  const int64_t T = cache->block_tokens;
  const int64_t n_rows = T * cache->n_heads * cache->n_layers, first = slot * T * cache->token_stride;
  if (n_rows >= sdvg::kMaxRows) return SDVG_ERR_UNSUPPORTED;
  const sdvg::RowGrid g = sdvg::row_grid(n_rows);
  hipLaunchKernelGGL(kv_commit_rope_kernel, dim3(g.x, 2, g.z), dim3(sdvg::kRowThreads), 0,
                     static_cast<hipStream_t>(stream), static_cast<const uint16_t *>(k_blk),
                     static_cast<const uint16_t *>(v_blk), static_cast<uint16_t *>(cache->k) + first,
                     static_cast<uint16_t *>(cache->v) + first, cos_table, sin_table,
                     sdvg::row_map(T, cache->n_heads, cache->layer_stride, cache->token_stride, cache->head_stride),
                     static_cast<uint32_t>(n_rows));
  SDVG_HIP_CHECK(hipGetLastError());
  cache->cache_len = (slot + 1) * T;
  return SDVG_OK;
}
