// Device-side pieces shared by the bf16 attention kernels: vector types, the global -> LDS copy, the
// workgroup barrier without a fence, the softmax of one tile, the fused commit's copying workgroups.
#pragma once
#include <math.h>
#include <stddef.h>

#include <type_traits>

#include "block_attn_index.h"
#include "block_attn_params.h"

namespace sdvg {
namespace attn_dev {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr float kPSumLimit = 1048576.0f;  // 2^20: a tile whose P sums past this retakes the maximum

// v_permlane32_swap(x, x) returns {own, partner} in the lower half-wave and {partner, own} in
// the upper one (partner = the lane 32 away); only symmetric combinations are used.
__device__ __forceinline__ float lane_max32(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float lane_sum32(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ void wait_vmcnt0() {
  // s_waitcnt vmcnt(0) only (expcnt = 7, lgkmcnt = 15 left unconstrained)
  __builtin_amdgcn_s_waitcnt(0x0F70);
}

// One wave-level 16-byte-per-lane global -> LDS copy: lane i's 16 bytes land at
// lds_addr + 16 * i. Written as inline assembly so that the compiler does not serialise
// successive copies with vmcnt(0) waits; completion is awaited explicitly (wait_vmcnt0)
// before the workgroup barrier that publishes the tile. The statements write M0 and say so in
// their clobber lists, so the compiler never assumes a value of its own survives them (clang
// warns that M0 is a reserved register it will not save; that is the intent).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const void *gptr, uint32_t lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off"
      :
      : "s"(lds_addr), "v"(gptr)
      : "memory", "m0");
}
// Same copy with the pointer step to the next tile (`step` bytes) folded in: the 64-bit add sits between the M0 write
// and the copy (covering the wait state M0 needs) and the stepped pointer is returned.
__device__ __forceinline__ const char *dma16_step(const char *gptr, uint64_t step, uint32_t lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %1\n\t"
      "v_lshl_add_u64 %0, %0, 0, %2\n\t"
      "global_load_lds_dwordx4 %0, off"
      : "+v"(gptr)
      : "s"(lds_addr), "s"(step)
      : "memory", "m0");
  return gptr;
}
#pragma clang diagnostic pop

// Workgroup barrier without the fence of __syncthreads (which would also wait for the
// prefetches still in flight); the compiler-level memory clobbers keep LDS accesses on
// their side of it.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The `items` array of the kernels' by-value AttnParams argument, kParamsAt bytes into the arguments, read from
// the kernel-argument segment (constant memory; the compiler turns the reads into scalar loads).
template <int kParamsAt = 0>
__device__ __forceinline__ const AttnItem *kernarg_items() {
  const char *ka = (const char *)__builtin_amdgcn_kernarg_segment_ptr();
  return reinterpret_cast<const AttnItem *>(ka + kParamsAt + offsetof(AttnParams, items));
}

// Asks for every argument of a launch's first item at once, ahead of the kernel's first branch: a trip to
// memory each otherwise.
__device__ __forceinline__ void load_arguments(const AttnParams &p, const AttnItem &it) {
  asm volatile("" ::"s"(it.q), "s"(it.k_cache), "s"(it.v_cache), "s"(it.k_blk), "s"(it.v_blk), "s"(it.out), "s"(p.q_ts),
               "s"(p.q_hs), "s"(p.kv_ts), "s"(p.kv_hs), "s"(p.blk_ts), "s"(p.blk_hs), "s"(p.cache_len),
               "s"(p.n_blk), "s"(p.copy_first_block), "s"(p.n_q), "s"(p.n_heads), "s"(p.n_qtiles), "s"(p.n_tiles),
               "s"(p.total_work), "s"(p.work_per_xcd), "s"(p.div_qtiles.m), "s"(p.div_qtiles.s), "s"(p.div_heads.m),
               "s"(p.div_heads.s), "s"(p.scale_log2e), "s"(p.o_ts), "s"(p.o_hs));
}

// Rows of O^T held in the accumulator layout (lane = query row lane % 32, half-wave hh), scaled by
// 1 / row sum, rounded to bf16 and stored; rows past n_q are not stored.
__device__ __forceinline__ void store_rows(const AttnParams &p, const AttnItem &it, int head, int q_row,
                                           int hh, const f32x16 (&o_acc)[4], float inv_l) {
  if (q_row >= p.n_q) return;
  uint16_t *op = static_cast<uint16_t *>(it.out) + q_row * p.o_ts + head * p.o_hs + 4 * hh;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 o4 = {o_acc[u][4 * g] * inv_l, o_acc[u][4 * g + 1] * inv_l, o_acc[u][4 * g + 2] * inv_l,
                        o_acc[u][4 * g + 3] * inv_l};
      const bf16x4 ob = __builtin_convertvector(o4, bf16x4);
      *reinterpret_cast<bf16x4 *>(op + 32 * u + 8 * g) = ob;
    }
  }
}

// Fused commit (paper Sec. 3 "Inference flow": the block the target keeps -- an accepted draft or
// its own regeneration -- goes into the target's KV cache): workgroups appended to the attention
// launch copy the block's K and V rows of this layer into cache tokens [cache_len, cache_len +
// n_blk), 16 bytes per lane, while the attention workgroups (which only read tokens below
// cache_len and the block itself) are still running. They are dispatched last and find their
// compute units among those the last round of attention workgroups leaves idle.
// They can be few (copy_workgroups, block_attn_plan.h: 16 beside the 240 of 12 heads x 312 rows) and a copy is then a chain of
// round trips to memory: K and V of four rows are in flight per lane (two / four / eight rows: 12 x 312 x 312 7.2 / 7.1 / 7.1 us,
// 12 x 1031 x 1031 16.0 / 15.7 / 15.7), the last ones too, and a row's token and head follow from the row before
// instead of a 64-bit division each. Ordinary loads, because the attention reads the same rows from the memory-side
// cache then (nontemporal: 12 x 1031 x 1031 17.9 instead of 16.0).
// us of a launch without / with its commit, keys from HBM: 12 x 312 x 312 6.4 / 6.5, 24 x 312 x 936 13.2 / 13.3, 12 x 1031 x
// 1031 17.2 / 15.4, 5 x 1409 x 2818 23.8 / 23.2, 12 x 4680 x 9360 219 / 220.
template <int kParamsAt = 0>
__device__ __forceinline__ void commit_block_rows(const AttnParams &p) {
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  constexpr int kRows = 4;
  const AttnItem it = kernarg_items<kParamsAt>()[0];
  const uint32_t n_heads = p.n_heads, n_blk = p.n_blk;
  const uint32_t row = (blockIdx.x - p.copy_first_block) * 32 + threadIdx.x / 16, step = p.n_copy_blocks * 32;
  const uint32_t step_tok = p.div_heads.div(step), step_head = step - step_tok * n_heads;
  uint32_t tok = p.div_heads.div(row), head = row - tok * n_heads;
  const int ch = threadIdx.x % 16;  // 16-byte chunk of the row
  while (tok < n_blk) {
    u32x4 k[kRows], v[kRows];
    int64_t dst[kRows];
    bool in[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      in[u] = tok < n_blk;
      const int64_t src = tok * p.blk_ts + head * p.blk_hs + ch * 8;
      dst[u] = tok * p.kv_ts + head * p.kv_hs + ch * 8;
      if (in[u]) {
        k[u] = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(it.k_blk) + src);
        v[u] = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(it.v_blk) + src);
      }
      tok += step_tok;
      head += step_head;
      if (head >= n_heads) {
        head -= n_heads;
        ++tok;
      }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      if (in[u]) {
        __builtin_nontemporal_store(k[u], reinterpret_cast<u32x4 *>(static_cast<uint16_t *>(p.k_commit_dst) + dst[u]));
        __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4 *>(static_cast<uint16_t *>(p.v_commit_dst) + dst[u]));
      }
  }
  // Where this path joins the attention's, the compiler would wait there for loads of this one (24 heads x 312 x 936 keys 13.9
  // us instead of 13.2, without any commit).
  __builtin_amdgcn_s_waitcnt(0);
}

// Vector phase: P^T = exp2(scale*log2e * (S^T - m)) rounded to bf16 in B-operand order, plus
// this lane's share of the row sum, taken over the ROUNDED probabilities so that numerator
// and denominator of the softmax use the same weights. The shift by the running maximum m is
// already in the scores (s_init), so forming P costs one multiply and one exp2 per score.
// No maximum is computed on the fast path: m may lag the true maximum, which changes nothing
// (both sides carry the same factor) as long as exp2 stays in range. Only if the tile's sum
// of P comes out huge (a logit more than ~15 above m in log2 units) does the wave take the
// slow path: raise m to the true maximum, rescale O and l, form P again.
// The row sum unpacks the rounded pairs again (a shift and a mask) and adds them as fp32:
// four plain instructions per pair. The one-instruction alternative, v_dot2_f32_bf16 with a
// vector of ones, shares the matrix pipe with the partner wave's MFMAs and, queued behind
// them at lower priority, made the vector phase the longer of the two (measured: 16 of them
// per tile cost 250 cycles per phase; the 64 plain instructions that replace them cost none).
// The work is laid out in stages over all scores (scale, exp2, convert, sum on four
// accumulators): no instruction depends on one issued just before it.
template <int NK>
__device__ __forceinline__ float form_p(const f32x16 (&s_acc)[NK], float scale_log2e, bf16x8 (&pf)[2 * NK]) {
  float pexp[NK][16];
#pragma unroll
  for (int kb = 0; kb < NK; ++kb)
#pragma unroll
    for (int i = 0; i < 16; ++i) pexp[kb][i] = s_acc[kb][i] * scale_log2e;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kb = 0; kb < NK; ++kb)
#pragma unroll
    for (int i = 0; i < 16; ++i) pexp[kb][i] = __builtin_amdgcn_exp2f(pexp[kb][i]);
  __builtin_amdgcn_sched_barrier(0);
  bf16x2 pb[NK][8];
#pragma unroll
  for (int kb = 0; kb < NK; ++kb)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const f32x2 pp = {pexp[kb][2 * i], pexp[kb][2 * i + 1]};
      pb[kb][i] = __builtin_convertvector(pp, bf16x2);
    }
  __builtin_amdgcn_sched_barrier(0);
  float dl[4];
#pragma unroll
  for (int kb = 0; kb < NK; ++kb)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      uint32_t pbits;
      __builtin_memcpy(&pbits, &pb[kb][i], 4);
      const float lo = __uint_as_float(pbits << 16), hi = __uint_as_float(pbits & 0xffff0000u);
      if (kb == 0 && i < 2) {
        dl[2 * i] = lo;
        dl[2 * i + 1] = hi;
      } else {
        dl[(2 * i) & 3] += lo;
        dl[(2 * i + 1) & 3] += hi;
      }
      pf[kb * 2 + (i >> 2)][(i & 3) * 2] = pb[kb][i][0];
      pf[kb * 2 + (i >> 2)][(i & 3) * 2 + 1] = pb[kb][i][1];
    }
  __builtin_amdgcn_sched_barrier(0);
  return (dl[0] + dl[1]) + (dl[2] + dl[3]);
}

// Largest score of the tile for this lane's query (both half-waves), relative to the shift.
template <int NK>
__device__ __forceinline__ float tile_max(const f32x16 (&s_acc)[NK]) {
  float m4[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) m4[c] = NK == 2 ? fmaxf(s_acc[0][c], s_acc[NK - 1][c]) : s_acc[0][c];
#pragma unroll
  for (int kb = 0; kb < NK; ++kb)
#pragma unroll
    for (int i = 4; i < 16; ++i) m4[i & 3] = fmaxf(m4[i & 3], s_acc[kb][i]);
  return lane_max32(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
}

}  // namespace attn_dev
}  // namespace sdvg
