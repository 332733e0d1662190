// Internal helpers shared by the translation units of libsdvg (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sdvg.h"

namespace sdvg {

// hipError_t of the last failed runtime call on this thread (sdvg_last_device_error()).
extern thread_local int g_last_device_error;

inline int device_error(hipError_t e) {
  g_last_device_error = static_cast<int>(e);
  return SDVG_ERR_DEVICE;
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// How the copy kernels read. A source of up to 64 MiB (K and V together) that was written or read not long ago is
// still in the memory-side cache (256 MiB, shared by everything that runs), which ordinary loads find and keep it in; beyond
// that, nontemporal loads. us, nontemporal / ordinary, three states in turn: commits with rotation of 46 MB 17.9 / 16.6, 55 MB 21.1 /
// 18.7, head-major 39 MB 15.4 / 12.6; rounds of the drafter (288 MB a commit, 24 MB snapshots) 312.3 / 310.9. With the
// line at 256 MiB, rounds with 157 MB commits and 161 MB snapshots lose: 325.8 / 331.5.
constexpr int64_t kCachedSourceBytes = int64_t{64} << 20;
inline bool streams_in(int64_t bytes) { return bytes > kCachedSourceBytes; }

typedef __attribute__((ext_vector_type(4))) unsigned int chunk_t;  // 16 bytes
template <bool kStream>
__device__ __forceinline__ chunk_t load_chunk(const chunk_t *p) {
  if (kStream) return __builtin_nontemporal_load(p);
  return *p;
}

// kv_cache.hip: host-side checks shared by every commit entry point.
int check_commit_args(const sdvg_kv_cache *cache, const void *k_blk, const void *v_blk, int32_t slot);

}  // namespace sdvg

#define SDVG_HIP_CHECK(expr)                                   \
  do {                                                         \
    hipError_t sdvg_e_ = (expr);                               \
    if (sdvg_e_ != hipSuccess) return sdvg::device_error(sdvg_e_); \
  } while (0)
