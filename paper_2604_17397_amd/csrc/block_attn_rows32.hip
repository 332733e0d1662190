// Block-causal attention of one video block for the smallest launches, for gfx950 (MI355X).
//
// Same operation and same arithmetic per 32 rows x 32 keys as block_attn_groups.hip with 4 groups (paper
// Sec. 1 / Sec. 4.1 "Models"), for launches whose 32-row workgroups fit one round of the compute units, or need no
// more rounds than 64-row ones (block_attn_plan.h). There a launch is a chain of latencies, and the chain is what this
// kernel cuts:
//   - 32 query rows per workgroup and all 8 waves on different key tiles: twice the workgroups of the 64-row
//     kernel, half the tiles per wave;
//   - a wave copies its tiles into its own part of the LDS and reads nothing else there, so the loop has no
//     barrier; the waves meet at the start (one maximum for all) and at the end (merge);
//   - a tile's K (and V) operands are read into registers at one go, so that the next tile's copies start
//     into the same 8 KB a phase earlier than the products that use the operands end;
//   - no tile holds keys of both sources: copies take a scalar address and a 32-bit offset per lane, four of
//     them with one write of M0, where the 64-bit address of every row costs some ten vector instructions;
//   - the arguments of the first copies are in registers when a wave starts, all others are asked for at once
//     behind those copies; the query rows come through the LDS once per workgroup.
// us among others in a graph, four sets of tensors in turn, with 64 rows / here (profiles/attn_plan_sweep.txt): 12 heads x 312 x
// 936 keys 13.1 / 9.4, 12 x 312 x 312 8.5 / 6.1, 8 x 1024 x 6144 41.1 / 39.3; with keys from HBM 15.9 / 10.6, 9.9 / 6.4, 61.4 / 46.1.
// Where it went at 12 x 312 x 936, one workgroup per 32 rows, while the first copies still waited 0.3 us for their arguments (9.2 us with one set of tensors
// again and again): 0.9 launch, 1.5 until the first tiles have landed, 0.6 first scores, 0.4 common maximum, 4.4 loop, 1.1
// merge and store.
// Where these workgroups are few (block_attn_plan.h) there are two per 32 rows, each with half of the output dims: 96 KB of
// copies per 8 x 32 keys instead of 128, and half of the merge. us in a graph with one set of tensors, four sets in turn, keys from
// HBM: 12 x 312 x 936 9.3 -> 8.6, 10.3 -> 8.9, 12.5 -> 10.5 (9.1 -> 8.3 as calls with one set); 12 x 312 x 312 6.4 -> 5.8, 6.4 -> 5.8,
// 7.2 -> 6.4; 5 x 800 x 5600 32.9 -> 28.1, 33.1 -> 28.1, 40.0 -> 32.8. (The LDS that half a V tile leaves
// free as a second K slot, K copied two tiles ahead: 1 us slower throughout, 9.0 -> 9.8.)
// The loop is bound by the copies: 8 waves bring 128 KB per 8 x 32 keys, which takes 1.13 - 1.18 us, and a
// loop of nothing but such copies from L2 reaches 62 bytes per clock and compute unit, 1.13 us. So
// neither fewer scalar instructions (1 %), nor the copies placed before the products (1 % slower), nor
// wave priorities (-3 to +11 %, by shape) are worth anything.
#include "block_attn_device.h"
#include "block_attn_params.h"
#include "block_attn_rows32_index.h"
#include "sdvg_common.h"

namespace {

using namespace sdvg::attn_dev;
using sdvg::AttnParams;
namespace ix = sdvg::attn_index;
using R = ix::Rows32;

typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) f32x2 lds_f32x2;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

#define SDVG_SB() __builtin_amdgcn_sched_barrier(0)

template <int N>
__device__ __forceinline__ void wait_copies() {  // all but the N most recent copies (or loads) have landed
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Four 1 KB copies (lane i's 16 bytes land at lds_addr + 1024 u + 16 i), each from a scalar address plus
// the lanes' offsets; the immediates count for both addresses.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy4(const uint32_t (&off)[4], const uint64_t *base, uint32_t lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %8\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %4\n\t"
      "global_load_lds_dwordx4 %1, %5 offset:1024\n\t"
      "global_load_lds_dwordx4 %2, %6 offset:2048\n\t"
      "global_load_lds_dwordx4 %3, %7 offset:3072"
      :
      : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base[0]), "s"(base[1]), "s"(base[2]), "s"(base[3]),
        "s"(__builtin_amdgcn_readfirstlane(lds_addr))
      : "memory", "m0");
}
#pragma clang diagnostic pop

// What the first copies of a workgroup need, in the 12 dwords that are in registers when it starts (build.py):
// they are under way before the first trip to memory for the other arguments, 0.3 us, has ended.
struct Early {
  const void *k, *q;               // keys of the first round of tiles (cache or block), and queries
  uint32_t k_ts, k_hs, q_ts, q_hs;  // elements
  int32_t n_q;
  uint32_t div_m, div_s_qtiles;    // by n_qtiles: FastDiv::m, and s << 16 | n_qtiles
  uint32_t work;                   // total_work << 16 | work_per_xcd
};
constexpr int kParamsAt = 48;  // where the AttnParams lie among the kernel's arguments
static_assert(sizeof(Early) == kParamsAt && alignof(AttnParams) == 8, "");

// kEarly: the `Early` arguments hold (early_of). kHalves: two workgroups per 32 query rows, each with half of the output dims.
template <bool kEarly, bool kHalves>
__global__ __launch_bounds__(512) void block_attn_rows32_kernel(
    const void *e_k, const void *e_q, uint32_t e_k_ts, uint32_t e_k_hs, uint32_t e_q_ts, uint32_t e_q_hs, int32_t e_n_q,
    uint32_t e_div_m, uint32_t e_div_s_qtiles, uint32_t e_work, const AttnParams all) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t *)smem));

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r32 = lane & 31, hh = lane >> 5;
  constexpr int kU = kHalves ? 2 : 4;                               // 32-dim blocks of the output
  constexpr int kVCopies = kHalves ? ix::kHalfCopies : R::kCopies;  // copies of a V tile

  // ---- copies
  uint32_t k_chunk[4], v_chunk = ix::rows32_lane_offset(0, lane, 0, 1);
#pragma unroll
  for (int u = 0; u < 4; ++u) k_chunk[u] = ix::rows32_lane_offset(0, lane, u, 0);
  // `keys` rows from `first_row` on
  auto copy_rows = [&](uint64_t first_row, uint32_t pitch, int keys, int is_v) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + ix::rows32_copy_dst(wave, is_v, 0);
    uint64_t base[8];
    base[0] = first_row;
    uint32_t off[4];
    if (kHalves && is_v) {
      if (__builtin_expect(keys == R::kKeys, 1)) {
        off[0] = off[1] = off[2] = off[3] = ix::rows32_half_lane_offset(pitch, lane);
#pragma unroll
        for (int u = 0; u < 3; ++u) base[u + 1] = base[u] + static_cast<int64_t>(ix::rows32_half_copy_step(pitch));
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          off[u] = ix::rows32_half_short_offset(pitch, keys, lane, u);
          base[u] = base[0] - (u > 0 ? 1024 * u : 0);
        }
      }
      copy4(off, base, dst);
      return;
    }
    if (__builtin_expect(keys == R::kKeys, 1)) {
      const uint32_t row_off = static_cast<uint32_t>(lane >> 4) * pitch;
#pragma unroll
      for (int u = 0; u < 4; ++u) off[u] = row_off + (is_v ? v_chunk : k_chunk[u]);
#pragma unroll
      for (int u = 0; u < 7; ++u) base[u + 1] = base[u] + static_cast<int64_t>(ix::rows32_copy_step(pitch, u));
      copy4(off, base, dst);
      copy4(off, base + 4, dst + 4096);
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          off[u] = ix::rows32_short_offset(pitch, keys, lane, 4 * h + u, is_v);
          base[u] = base[0] - (u > 0 ? 1024 * u : 0);
        }
        copy4(off, base, dst + 4096 * h);
      }
    }
  };
  // The query rows (rows past the end re-read the last one and are not stored): four per wave.
  auto copy_query = [&](const void *q, int head, int qt, int n_q, int64_t q_ts, int64_t q_hs) __attribute__((always_inline)) {
    const int row = 4 * wave + (lane >> 4), q_row = qt * 32 + row;
    const uint16_t *qp = static_cast<const uint16_t *>(q) + (q_row < n_q ? q_row : n_q - 1) * q_ts + head * q_hs +
                         ix::swizzled_chunk(row, lane, 0) * 8;
    dma16(qp, lds0 + R::kQ + wave * 1024);
  };

  // Behind the early copies: loads that stood ahead of them would be waited for first.
  auto *arguments = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
  if constexpr (kEarly) {
    const int work = ix::work_of_block(blockIdx.x, static_cast<int>(e_work & 0xffff)), n_qt = static_cast<int>(e_div_s_qtiles & 0xffff);
    if (blockIdx.x < 8 * (e_work & 0xffff) && work < static_cast<int>(e_work >> 16)) {
      const int tile = kHalves ? work >> 1 : work, head = static_cast<int>(sdvg::FastDiv{0, e_div_m, e_div_s_qtiles >> 16}.div(tile));
      const uint32_t pitch = e_k_ts * 2;
      const uint64_t first_row = reinterpret_cast<uint64_t>(e_k) + static_cast<uint64_t>(head) * e_k_hs * 2 +
                                 static_cast<uint64_t>(wave * R::kKeys) * pitch;
      copy_rows(first_row, pitch, R::kKeys, 0);
      copy_query(e_q, head, tile - head * n_qt, e_n_q, e_q_ts, e_q_hs);
    }
    asm volatile("" : "+s"(arguments));
  }
  const AttnParams &p = kEarly ? *(const AttnParams *)(arguments + kParamsAt) : all;
  sdvg::AttnItem it = p.items[0];
  load_arguments(p, it);
  if (static_cast<int>(blockIdx.x) >= p.copy_first_block) {
    commit_block_rows<kParamsAt>(p);
    return;
  }
  const int work = ix::work_of_block(blockIdx.x, p.work_per_xcd);
  if (work >= p.total_work) return;

  const int q_tile = kHalves ? work >> 1 : work, half = kHalves ? work & 1 : 0;
  const int hq = static_cast<int>(p.div_qtiles.div(q_tile)), qt = q_tile - hq * p.n_qtiles;
  const int item = static_cast<int>(p.div_heads.div(hq)), head = hq - item * p.n_heads;
  if (item != 0) it = kernarg_items<kParamsAt>()[item];

  const int c_len = static_cast<int>(p.cache_len), n_blk = p.n_blk;
  const uint32_t c_pitch = static_cast<uint32_t>(p.kv_ts * 2), b_pitch = static_cast<uint32_t>(p.blk_ts * 2);
  const uint64_t kc = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.k_cache) + head * p.kv_hs);
  const uint64_t vc = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.v_cache) + head * p.kv_hs + 64 * half);
  const uint64_t kb = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.k_blk) + head * p.blk_hs);
  const uint64_t vb = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.v_blk) + head * p.blk_hs + 64 * half);
  const int n_it = ix::rows32_tiles_of(wave, p.n_tiles);
  // (a wave past the last tile takes the last one, masked as a whole)
  auto tile_of = [&](int i) __attribute__((always_inline)) {
    const int t = wave + ix::kWaves * i;
    return ix::rows32_tile(c_len, n_blk, t < p.n_tiles ? t : p.n_tiles - 1);
  };

  auto copy_tile = [&](const ix::Rows32Tile &t, int is_v) __attribute__((always_inline)) {
    const uint32_t pitch = t.in_cache ? c_pitch : b_pitch;
    copy_rows((t.in_cache ? (is_v ? vc : kc) : (is_v ? vb : kb)) + static_cast<uint64_t>(static_cast<uint32_t>(t.first)) * pitch,
              pitch, t.keys, is_v);
  };
  if constexpr (!kEarly) {
    copy_tile(tile_of(0), 0);
    copy_query(it.q, head, qt, p.n_q, p.q_ts, p.q_hs);
  }
  copy_tile(tile_of(0), 1);

  uint32_t k_off[8], v_off[kU];  // LDS read addresses
#pragma unroll
  for (int s = 0; s < 8; ++s) k_off[s] = lds0 + ix::k_read_offset(lane, s, 0);
#pragma unroll
  for (int db = 0; db < kU; ++db)
    v_off[db] = lds0 + wave * R::kWavePart + R::kTile +
                (kHalves ? ix::rows32_half_read_offset(lane, 0, db, 0) : ix::v_read_offset(lane, 0, db, 0));
  constexpr int kVRow = kHalves ? ix::kHalfRow : 256;

  f32x16 o_acc[kU];
#pragma unroll
  for (int u = 0; u < kU; ++u)
#pragma unroll
    for (int i = 0; i < 16; ++i) o_acc[u][i] = 0.f;
  float l_run = 0.f, s_shift = 0.f;
  f32x16 s_acc[1], s_init;
  auto set_shift = [&](float v) __attribute__((always_inline)) {
    s_shift = v;
#pragma unroll
    for (int i = 0; i < 16; ++i) s_init[i] = v;
  };
  set_shift(0.f);
  lds_float *const first_max = (lds_float *)static_cast<uintptr_t>(lds0 + R::kMax) + lane;
  // The waves' first maxima meet in LDS: see block_attn_groups.hip for why all start from one.
  auto common_start = [&](float own) __attribute__((always_inline)) {
    first_max[wave * 64] = own;
    wait_lds();
    wg_barrier();
    float mx = fmaxf(first_max[0], first_max[64]), m_all = mx;
#pragma unroll
    for (int w = 2; w < ix::kWaves; ++w) m_all = fmaxf(m_all, first_max[w * 64]);
    if ((m_all - mx) * p.scale_log2e > 20.f) mx = m_all;
    return mx == -INFINITY ? 0.f : mx;
  };

#pragma unroll
  for (int u = 0; u < kU; ++u) asm volatile("" : "+v"(o_acc[u]));  // (ready before the wait)
  asm volatile("" : "+v"(s_init));
  wait_copies<kVCopies>();
  wg_barrier();
  bf16x8 qf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) qf[s] = *(lds_bf16x8 *)static_cast<uintptr_t>(k_off[s] + R::kQ);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    k_off[s] += wave * R::kWavePart;
    asm volatile("" : "+v"(k_off[s]));
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) asm volatile("" : "+v"(v_off[u]));

#pragma unroll 1
  for (int i = 0;; ++i) {
    const bool more = i + 1 < n_it;
    bf16x8 f[8];
    asm volatile("" : "+v"(s_init));
    // ---- S of the tile. Its operands are read at one go, so that the next tile's copies can start
    wait_copies<kVCopies>();  // K of this tile (V may still be on its way)
#pragma unroll
    for (int s = 0; s < 8; ++s) f[s] = *(lds_bf16x8 *)static_cast<uintptr_t>(k_off[s]);
    SDVG_SB();
#pragma unroll
    for (int s = 0; s < 4; ++s)
      s_acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], qf[s], s == 0 ? s_init : s_acc[0], 0, 0, 0);
    SDVG_SB();
    wait_lds();
    if (more) copy_tile(tile_of(i + 1), 0);
    SDVG_SB();
#pragma unroll
    for (int s = 4; s < 8; ++s) s_acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], qf[s], s_acc[0], 0, 0, 0);
    SDVG_SB();
    const int keys = wave + ix::kWaves * i < p.n_tiles ? tile_of(i).keys : 0;
    if (__builtin_expect(keys < R::kKeys, 0)) {
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (4 * hh + 8 * (j >> 2) + (j & 3) >= keys) s_acc[0][j] = -INFINITY;
    }
    if (i == 0) {
      const float mx = common_start(tile_max(s_acc));
#pragma unroll
      for (int j = 0; j < 16; ++j) s_acc[0][j] -= mx;
      set_shift(-mx);
    }
    // ---- softmax with the lazy running maximum of block_attn.hip
    bf16x8 pf[2];
    float dl = form_p(s_acc, p.scale_log2e, pf);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(dl < kPSumLimit)) != 0, 0)) {
      const float d = fmaxf(tile_max(s_acc), 0.f);
      const float alpha = __builtin_amdgcn_exp2f(-d * p.scale_log2e);
#pragma unroll
      for (int u = 0; u < kU; ++u)
#pragma unroll
        for (int j = 0; j < 16; ++j) o_acc[u][j] *= alpha;
      l_run *= alpha;
#pragma unroll
      for (int j = 0; j < 16; ++j) s_acc[0][j] -= d;
      set_shift(s_shift - d);
      dl = form_p(s_acc, p.scale_log2e, pf);
    }
    l_run += dl;
    // ---- O^T += V^T P^T
    if (more)
      wait_copies<R::kCopies>();  // V of this tile (K of the next one may still be on its way)
    else
      wait_copies<0>();
    // The rows past a short tile's keys have P = 0, but 0 times an infinite value would be NaN.
    if (__builtin_expect(keys < R::kKeys, 0)) {
#pragma unroll
      for (int u = 0; u < kVCopies; ++u)
        if ((kHalves ? ix::rows32_half_copy_row(lane, u) : ix::rows32_copy_row(lane, u)) >= keys)
          *(lds_f32x4 *)static_cast<uintptr_t>(lds0 + ix::rows32_copy_dst(wave, 1, 0) + u * 1024 + lane * 16) =
              f32x4{0.f, 0.f, 0.f, 0.f};
      wait_lds();
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint32_t vp = v_off[u] + j * 16 * kVRow;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)static_cast<uintptr_t>(vp));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)static_cast<uintptr_t>(vp + 8 * kVRow));
        const __attribute__((ext_vector_type(8))) short a16 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        __builtin_memcpy(&f[kU * j + u], &a16, sizeof(bf16x8));
      }
    SDVG_SB();
#pragma unroll
    for (int u = 0; u < kU; ++u) o_acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[u], pf[0], o_acc[u], 0, 0, 0);
    SDVG_SB();
    wait_lds();
    if (more) copy_tile(tile_of(i + 1), 1);
    SDVG_SB();
#pragma unroll
    for (int u = 0; u < kU; ++u) o_acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[kU + u], pf[1], o_acc[u], 0, 0, 0);
    SDVG_SB();
    if (!more) break;
  }

  // ---- merge: every wave leaves its O in its own part of the LDS (nobody else reads there) and its row
  // sums and shift where the query rows were (all waves read those two barriers ago); then it combines
  // the eight waves' parts of 4 of the rows: with m the largest running maximum,
  //   O = sum_w 2^((m_w - m) scale*log2e) O_w, l likewise.
  const uint32_t part = lds0 + wave * R::kWavePart;
#pragma unroll
  for (int u = 0; u < kU; ++u)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = 4 * u + g;
      const f32x4 o4 = {o_acc[u][4 * g], o_acc[u][4 * g + 1], o_acc[u][4 * g + 2], o_acc[u][4 * g + 3]};
      const int at = kHalves ? ix::rows32_half_merge_offset(2 * c + hh, r32) : ix::merge_offset(c, hh, r32);
      *(lds_f32x4 *)static_cast<uintptr_t>(part + at) = o4;
    }
  const float l_row = lane_sum32(l_run);
  if (hh == 0) *(lds_f32x2 *)static_cast<uintptr_t>(lds0 + R::kQ + (wave * 32 + r32) * 8) = f32x2{l_row, s_shift};
  wait_lds();
  wg_barrier();
  const int row = 4 * wave + (lane >> 4), q_row = qt * 32 + row, c = lane & 15;
  float l_w[ix::kWaves], shift_w[ix::kWaves];
#pragma unroll
  for (int w = 0; w < ix::kWaves; ++w) {
    const f32x2 v = *(lds_f32x2 *)static_cast<uintptr_t>(lds0 + R::kQ + (w * 32 + row) * 8);
    l_w[w] = v[0];
    shift_w[w] = v[1];
  }
  float shift_min = shift_w[0];
#pragma unroll
  for (int w = 1; w < ix::kWaves; ++w) shift_min = fminf(shift_min, shift_w[w]);
  float l_sum = 0.f;
  f32x4 o_lo = {0.f, 0.f, 0.f, 0.f}, o_hi = o_lo;
#pragma unroll
  for (int w = 0; w < ix::kWaves; ++w) {
    const float factor = __builtin_amdgcn_exp2f((shift_min - shift_w[w]) * p.scale_log2e);
    l_sum += factor * l_w[w];
    const int at = kHalves ? ix::rows32_half_merge_offset(c, row) : ix::merge_offset(c, 0, row);
    const f32x4 lo = *(lds_f32x4 *)static_cast<uintptr_t>(lds0 + w * R::kWavePart + at);
#pragma unroll
    for (int e = 0; e < 4; ++e) o_lo[e] += factor * lo[e];
    if constexpr (!kHalves) {
      const f32x4 hi = *(lds_f32x4 *)static_cast<uintptr_t>(lds0 + w * R::kWavePart + ix::merge_offset(c, 1, row));
#pragma unroll
      for (int e = 0; e < 4; ++e) o_hi[e] += factor * hi[e];
    }
  }
  if (q_row >= p.n_q) return;
  const float inv_l = 1.0f / l_sum;
  if constexpr (kHalves) {
    bf16x4 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = static_cast<__bf16>(o_lo[e] * inv_l);
    *reinterpret_cast<bf16x4 *>(static_cast<uint16_t *>(it.out) + q_row * p.o_ts + head * p.o_hs + 64 * half + 4 * c) = out;
    return;
  }
  bf16x8 out;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    out[e] = static_cast<__bf16>(o_lo[e] * inv_l);
    out[4 + e] = static_cast<__bf16>(o_hi[e] * inv_l);
  }
  *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(it.out) + q_row * p.o_ts + head * p.o_hs + 8 * c) = out;
}

// For one item whose first round of tiles lies wholly in the cache, or in the block if there is no cache, and for
// numbers that fit their fields. (Other launches lose 0.15 us if they take the same way.)
bool early_of(const AttnParams &p, Early &e) {
  const bool in_cache = p.cache_len > 0;
  if (p.n_items != 1 || (in_cache ? p.cache_len : p.n_blk) < ix::kWaves * R::kKeys || p.total_work > 0xffff ||
      p.work_per_xcd > 0xffff || p.n_qtiles > 0xffff)
    return false;
  const sdvg::AttnItem &it = p.items[0];
  e = Early{in_cache ? it.k_cache : it.k_blk,
            it.q,
            static_cast<uint32_t>(in_cache ? p.kv_ts : p.blk_ts),
            static_cast<uint32_t>(in_cache ? p.kv_hs : p.blk_hs),
            static_cast<uint32_t>(p.q_ts),
            static_cast<uint32_t>(p.q_hs),
            p.n_q,
            p.div_qtiles.m,
            p.div_qtiles.s << 16 | static_cast<uint32_t>(p.n_qtiles),
            static_cast<uint32_t>(p.total_work) << 16 | static_cast<uint32_t>(p.work_per_xcd)};
  return true;
}

}  // namespace

namespace sdvg {

hipError_t prepare_block_attn_rows32() {
  for (const auto kernel : {block_attn_rows32_kernel<false, false>, block_attn_rows32_kernel<true, false>,
                            block_attn_rows32_kernel<false, true>, block_attn_rows32_kernel<true, true>}) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, R::kLdsBytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

int launch_block_attn_rows32(AttnParams p, bool halves, hipStream_t s) {
  p.n_tiles = ix::rows32_tiles(static_cast<int>(p.cache_len)) + ix::rows32_tiles(p.n_blk);
  Early e{};
  const bool early = early_of(p, e);
  const auto kernel = halves ? (early ? block_attn_rows32_kernel<true, true> : block_attn_rows32_kernel<false, true>)
                             : (early ? block_attn_rows32_kernel<true, false> : block_attn_rows32_kernel<false, false>);
  hipLaunchKernelGGL(kernel, dim3(8 * p.work_per_xcd + p.n_copy_blocks), dim3(512), R::kLdsBytes, s, e.k, e.q, e.k_ts,
                     e.k_hs, e.q_ts, e.q_hs, e.n_q, e.div_m, e.div_s_qtiles, e.work, p);
  SDVG_HIP_CHECK(hipGetLastError());
  return SDVG_OK;
}

}  // namespace sdvg
