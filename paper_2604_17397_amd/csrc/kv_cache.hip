// KV-cache commit and rollback: bandwidth-bound copy / zero-fill kernels, one launch for all
// layers and for both K and V. Paper Sec. 3 "Inference flow": an accepted draft is committed
// to the target's KV cache; a rejected one must leave no trace before the target regenerates.
#include "row_map.h"
#include "sdvg_common.h"

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;  // one 16-byte chunk

constexpr int kThreads = 256;

// Contiguous fast path: every layer's destination range is one dense run of chunks_per_layer
// chunks (token-major cache with head_stride == 128, token_stride == H*128).
// grid = (blocks_per_layer, n_layers, 2): z selects K or V. One 16-byte chunk per thread and
// no loop: on MI355X many small workgroups beat grid-stride loops and deeper unrolling for a
// pure copy (measured 6.4 TB/s of read+write traffic against 5.1-5.8 TB/s for the looped forms).
// All copy kernels read with nontemporal loads. Ordinary ones are faster where the memory-side cache (256 MiB) holds the
// source and slower where it does not, which is what a generation loop meets: it reads gigabytes of weights between
// two commits. us, nontemporal / ordinary, three sets in turn and sets of 1.6 GB in turn: 55 MB dense 19.2 / 17.4 and
// 20.2 / 21.0, head-major 19.6 / 17.8 and 20.5 / 21.2, with rotation 19.7 / 18.3 and 20.4 / 21.3; 12 MB head-major
// 5.5 / 5.0 and 5.7 / 6.4; snapshots of 64 MiB 22.2 / 20.3 and 23.3 / 24.1, 4 MiB 2.9 / 2.7 and 2.7 / 3.1.
__global__ __launch_bounds__(kThreads) void kv_commit_dense_kernel(
    const u32x4 *__restrict__ k_src, const u32x4 *__restrict__ v_src, u32x4 *__restrict__ k_dst,
    u32x4 *__restrict__ v_dst, int64_t chunks_per_layer, int64_t dst_layer_stride_chunks,
    int64_t dst_first_chunk) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i >= chunks_per_layer) return;
  const u32x4 *src = (blockIdx.z == 0 ? k_src : v_src) + blockIdx.y * chunks_per_layer;
  u32x4 *dst = (blockIdx.z == 0 ? k_dst : v_dst) + blockIdx.y * dst_layer_stride_chunks +
               dst_first_chunk;
  __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// General strides: one 16-byte chunk per thread, rows in the order of their destinations (RowMap).
// On a head-major cache (30 layers x 12 heads x 1560 tokens, 575 MB moved) 99.5 us = 5.8 TB/s. With
// the rows in the order of the source 103.6, with ordinary stores 113.6, and with 64-bit divisions
// and a loop over chunks 111.
__global__ __launch_bounds__(sdvg::kRowThreads) void kv_commit_strided_kernel(
    const uint16_t *__restrict__ k_src, const uint16_t *__restrict__ v_src, uint16_t *__restrict__ k_dst,
    uint16_t *__restrict__ v_dst, sdvg::RowMap m, uint32_t n_rows) {
  const uint32_t r = sdvg::row_of(blockIdx.x, blockIdx.z, threadIdx.x);
  if (r >= n_rows) return;
  const int ch = (threadIdx.x & 15) * 8;
  const sdvg::RowMap::Row row = m.row(r);
  const uint16_t *src = (blockIdx.y == 0 ? k_src : v_src) + m.src(row) + ch;
  uint16_t *dst = (blockIdx.y == 0 ? k_dst : v_dst) + m.dst(row) + ch;
  __builtin_nontemporal_store(__builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src)),
                              reinterpret_cast<u32x4 *>(dst));
}

__global__ __launch_bounds__(kThreads) void kv_zero_dense_kernel(
    u32x4 *__restrict__ k_dst, u32x4 *__restrict__ v_dst, int64_t chunks_per_layer,
    int64_t dst_layer_stride_chunks, int64_t dst_first_chunk) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i >= chunks_per_layer) return;
  u32x4 *dst = (blockIdx.z == 0 ? k_dst : v_dst) + blockIdx.y * dst_layer_stride_chunks +
               dst_first_chunk;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  __builtin_nontemporal_store(zero, dst + i);
}

__global__ __launch_bounds__(sdvg::kRowThreads) void kv_zero_strided_kernel(
    uint16_t *__restrict__ k_dst, uint16_t *__restrict__ v_dst, sdvg::RowMap m, uint32_t n_rows) {
  const uint32_t r = sdvg::row_of(blockIdx.x, blockIdx.z, threadIdx.x);
  if (r >= n_rows) return;
  uint16_t *dst = (blockIdx.y == 0 ? k_dst : v_dst) + m.dst(m.row(r)) + (threadIdx.x & 15) * 8;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  __builtin_nontemporal_store(zero, reinterpret_cast<u32x4 *>(dst));
}

// Plain device-to-device copy of an opaque buffer: 16-byte chunks, one per thread; the thread
// after the last full chunk moves the 0-15 tail bytes.
__global__ __launch_bounds__(kThreads) void buffer_copy_kernel(const u32x4 *__restrict__ src,
                                                               u32x4 *__restrict__ dst, int64_t chunks,
                                                               int tail_bytes) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (i < chunks) {
    __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
  } else if (i == chunks) {
    const uint8_t *sb = reinterpret_cast<const uint8_t *>(src + chunks);
    uint8_t *db = reinterpret_cast<uint8_t *>(dst + chunks);
    for (int b = 0; b < tail_bytes; ++b) db[b] = sb[b];
  }
}

int validate_cache(const sdvg_kv_cache *c) {
  if (!c) return SDVG_ERR_NULL;
  if (!c->k || !c->v) return SDVG_ERR_NULL;
  if (c->head_dim != 128) return SDVG_ERR_UNSUPPORTED;
  if (c->n_layers <= 0 || c->n_heads <= 0 || c->block_tokens <= 0 || c->capacity_tokens <= 0)
    return SDVG_ERR_SHAPE;
  if (c->cache_len < 0 || c->cache_len > c->capacity_tokens) return SDVG_ERR_RANGE;
  if (c->head_stride < 128 || c->token_stride < 128 || c->layer_stride < 128) return SDVG_ERR_SHAPE;
  if ((c->head_stride | c->token_stride | c->layer_stride) & 7) return SDVG_ERR_ALIGN;
  if (!sdvg::aligned16(c->k) || !sdvg::aligned16(c->v)) return SDVG_ERR_ALIGN;
  // Rows must not overlap: of the token and head strides the larger one has to step over
  // everything the smaller one spans, and (with several layers) a layer over both.
  const bool token_inner = c->token_stride <= c->head_stride;
  const int64_t s_in = token_inner ? c->token_stride : c->head_stride;
  const int64_t n_in = token_inner ? c->capacity_tokens : c->n_heads;
  const int64_t s_out = token_inner ? c->head_stride : c->token_stride;
  const int64_t n_out = token_inner ? c->n_heads : c->capacity_tokens;
  const int64_t span_in = (n_in - 1) * s_in + 128;
  if (n_out > 1 && s_out < span_in) return SDVG_ERR_SHAPE;
  if (c->n_layers > 1 && c->layer_stride < (n_out - 1) * s_out + span_in) return SDVG_ERR_SHAPE;
  return SDVG_OK;
}

// Elements from the first to one past the last element of tokens [first, first + n) of one layer.
int64_t token_range_span(const sdvg_kv_cache *c, int64_t n) {
  return (n - 1) * c->token_stride + (c->n_heads - 1) * c->head_stride + 128;
}

// True if [a, a + a_bytes) and [b, b + b_bytes) share a byte.
bool ranges_overlap(const void *a, int64_t a_bytes, const void *b, int64_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + static_cast<uintptr_t>(b_bytes) && y < x + static_cast<uintptr_t>(a_bytes);
}

bool dense_token_major(const sdvg_kv_cache *c) {
  return c->head_stride == 128 && c->token_stride == static_cast<int64_t>(c->n_heads) * 128;
}

dim3 dense_grid(int64_t chunks_per_layer, int n_layers) {
  return dim3(static_cast<unsigned>((chunks_per_layer + kThreads - 1) / kThreads), n_layers, 2);
}

// Grid of the strided kernels; y selects K or V.
dim3 row_launch(int64_t n_rows) {
  const sdvg::RowGrid g = sdvg::row_grid(n_rows);
  return dim3(g.x, 2, g.z);
}

}  // namespace

namespace sdvg {
// Host-side checks shared by every commit entry point: descriptor, pointers, the append-only slot
// rule, and that the source does not alias the slot it is copied into (in any layer).
int check_commit_args(const sdvg_kv_cache *cache, const void *k_blk, const void *v_blk, int32_t slot) {
  int st = validate_cache(cache);
  if (st != SDVG_OK) return st;
  if (!k_blk || !v_blk) return SDVG_ERR_NULL;
  if (!aligned16(k_blk) || !aligned16(v_blk)) return SDVG_ERR_ALIGN;
  const int64_t T = cache->block_tokens;
  if (slot < 0 || slot * T != cache->cache_len || (slot + 1) * T > cache->capacity_tokens)
    return SDVG_ERR_RANGE;
  const int64_t src_bytes = static_cast<int64_t>(cache->n_layers) * T * cache->n_heads * 128 * 2;
  const int64_t dst_bytes = token_range_span(cache, T) * 2;
  for (int l = 0; l < cache->n_layers; ++l) {
    const int64_t off = (l * cache->layer_stride + slot * T * cache->token_stride) * 2;
    const char *dk = static_cast<const char *>(cache->k) + off, *dv = static_cast<const char *>(cache->v) + off;
    for (const void *src : {k_blk, v_blk})
      if (ranges_overlap(src, src_bytes, dk, dst_bytes) || ranges_overlap(src, src_bytes, dv, dst_bytes))
        return SDVG_ERR_RANGE;
  }
  return SDVG_OK;
}
}  // namespace sdvg

extern "C" int sdvg_kv_commit(sdvg_kv_cache *cache, const void *k_blk, const void *v_blk,
                              int32_t slot, void *stream) {
  int st = sdvg::check_commit_args(cache, k_blk, v_blk, slot);
  if (st != SDVG_OK) return st;
  const int64_t T = cache->block_tokens;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t chunks_per_layer = T * cache->n_heads * 16;
  if (dense_token_major(cache)) {
    hipLaunchKernelGGL(kv_commit_dense_kernel, dense_grid(chunks_per_layer, cache->n_layers),
                       dim3(kThreads), 0, s, static_cast<const u32x4 *>(k_blk),
                       static_cast<const u32x4 *>(v_blk), static_cast<u32x4 *>(cache->k),
                       static_cast<u32x4 *>(cache->v), chunks_per_layer, cache->layer_stride / 8,
                       slot * T * cache->token_stride / 8);
  } else {
    const int64_t n_rows = T * cache->n_heads * cache->n_layers, first = slot * T * cache->token_stride;
    if (n_rows >= sdvg::kMaxRows) return SDVG_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kv_commit_strided_kernel, row_launch(n_rows), dim3(sdvg::kRowThreads), 0, s,
                       static_cast<const uint16_t *>(k_blk), static_cast<const uint16_t *>(v_blk),
                       static_cast<uint16_t *>(cache->k) + first, static_cast<uint16_t *>(cache->v) + first,
                       sdvg::row_map(T, cache->n_heads, cache->layer_stride, cache->token_stride, cache->head_stride),
                       static_cast<uint32_t>(n_rows));
  }
  SDVG_HIP_CHECK(hipGetLastError());
  cache->cache_len = (slot + 1) * T;
  return SDVG_OK;
}

extern "C" int sdvg_kv_commit_mark(sdvg_kv_cache *cache, int32_t slot) {
  int st = validate_cache(cache);
  if (st != SDVG_OK) return st;
  const int64_t T = cache->block_tokens;
  if (slot < 0 || slot * T != cache->cache_len || (slot + 1) * T > cache->capacity_tokens) return SDVG_ERR_RANGE;
  cache->cache_len = (slot + 1) * T;
  return SDVG_OK;
}

extern "C" int sdvg_kv_rollback(sdvg_kv_cache *cache, int64_t new_len, void *stream) {
  int st = validate_cache(cache);
  if (st != SDVG_OK) return st;
  if (new_len < 0 || new_len > cache->cache_len) return SDVG_ERR_RANGE;
  const int64_t n_tok = cache->cache_len - new_len;
  if (n_tok == 0) return SDVG_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t chunks_per_layer = n_tok * cache->n_heads * 16;
  if (dense_token_major(cache)) {
    hipLaunchKernelGGL(kv_zero_dense_kernel, dense_grid(chunks_per_layer, cache->n_layers),
                       dim3(kThreads), 0, s, static_cast<u32x4 *>(cache->k),
                       static_cast<u32x4 *>(cache->v), chunks_per_layer, cache->layer_stride / 8,
                       new_len * cache->token_stride / 8);
  } else {
    const int64_t n_rows = n_tok * cache->n_heads * cache->n_layers, first = new_len * cache->token_stride;
    if (n_rows >= sdvg::kMaxRows) return SDVG_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kv_zero_strided_kernel, row_launch(n_rows), dim3(sdvg::kRowThreads), 0, s,
                       static_cast<uint16_t *>(cache->k) + first, static_cast<uint16_t *>(cache->v) + first,
                       sdvg::row_map(n_tok, cache->n_heads, cache->layer_stride, cache->token_stride, cache->head_stride),
                       static_cast<uint32_t>(n_rows));
  }
  SDVG_HIP_CHECK(hipGetLastError());
  cache->cache_len = new_len;
  return SDVG_OK;
}

extern "C" int sdvg_buffer_snapshot(void *dst, const void *src, int64_t n_bytes, void *stream) {
  if (n_bytes < 0) return SDVG_ERR_SHAPE;
  if (n_bytes == 0) return SDVG_OK;
  if (!dst || !src) return SDVG_ERR_NULL;
  if (!sdvg::aligned16(dst) || !sdvg::aligned16(src)) return SDVG_ERR_ALIGN;
  const uintptr_t d = reinterpret_cast<uintptr_t>(dst), c = reinterpret_cast<uintptr_t>(src);
  if (d < c + static_cast<uintptr_t>(n_bytes) && c < d + static_cast<uintptr_t>(n_bytes)) return SDVG_ERR_RANGE;
  const int64_t chunks = n_bytes / 16;
  const int tail = static_cast<int>(n_bytes % 16);
  const int64_t blocks = (chunks + 1 + kThreads - 1) / kThreads;
  if (blocks > 0x7FFFFFFF) return SDVG_ERR_UNSUPPORTED;  // more than 8 TiB
  hipLaunchKernelGGL(buffer_copy_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0,
                     static_cast<hipStream_t>(stream), static_cast<const u32x4 *>(src),
                     static_cast<u32x4 *>(dst), chunks, tail);
  SDVG_HIP_CHECK(hipGetLastError());
  return SDVG_OK;
}
