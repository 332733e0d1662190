// Block-causal attention of one video block for launches with few query rows, for gfx950 (MI355X).
//
// Same operation and same per-wave arithmetic as block_attn.hip (paper Sec. 1 / Sec. 4.1 "Models").
// There a workgroup owns 256 query rows and walks all keys; a layer with few heads or a small block
// then has far fewer workgroups than the chip has compute units, each of them one long serial chain
// of key tiles. Here the 8 waves of a workgroup form G key groups: the workgroup owns 8 / G x 32
// query rows and every group walks every G-th key tile, so there are G times as many workgroups and
// the chain is G times shorter. The groups' partial results (O, row sum, maximum) meet in LDS at the
// end, in fp32; nothing goes through memory and no second kernel is needed.
//
// What it costs: a K / V tile in LDS serves 8 / G waves instead of 8, so the L2 -> LDS traffic per
// query row is G times that of the 256-row kernel. Tiles are 64 keys (G = 2) or 32 keys (G = 4),
// because G groups x (3 K + 2 V tiles) have to fit the LDS (160 KB in both cases).
//
// Schedule: ping-pong as in block_attn.hip (waves 0-3 and 4-7 half an iteration apart, vector phase
// of one beside the matrix phase of the other). Matrix phase i of a group computes S(i+1) and
// P(i) V(i) and starts the copies of V(i+1) and K(i+3), one or two behind each second MFMA, into the
// slots last read in matrix phase i - 1 (three K and two V slots per group: all 160 KB of the LDS).
//
// What it went through (12 heads x 1031 x 6186 keys, 4 groups, us per launch; the 256-row kernel takes
// 108):
//   copies started at the head of the vector phase (ring of 2 + 2, 128 KB)         66
//   between the MFMAs, tile kinds told apart by branches at each tile               62
//   one rarely taken branch per tile                                                57
//   slots as offsets in registers instead of a loop unrolled by 6: short launches gain (a KB of
//   code fetched cold costs about 1 us), but its bookkeeping in the vector phase    59
//   bookkeeping moved into the gaps of the matrix phase                              52
//   a shorter way in and out (below)                                                 49
//   copies from a scalar address and 32-bit offsets instead of a 64-bit address per
//   lane; no tile holds keys of both sources, so that only short tiles need new ones 48
// (Scalar addresses, us before / after, 2 groups: 12 x 1560 x 4680 52.9 / 51.3, 9 x 2000 x 8000 81.1 / 78.3, 5 x 4680 x 32760
// 357 / 345. The wave that issues the MFMAs has one instruction in 4 cycles: 200 of them per 32-key tile, now 175, are what
// the loop is short of. All that changes per tile, worked out anew for each, is slower again: 1 to 2 %.)
// (Arguments of the first copies preloaded into registers, as in block_attn_rows32.hip: no gain. 64 rows per wave, every
// wave with key tiles of its own, which halves the LDS reads and needs no barrier: 53, bound by the copies.)
// What bounds it there, by counters: the matrix pipes are busy in 58 % of the SIMD cycles of the
// compute units at work (2 groups 70 %, the 256-row kernel 86 %). With the copies, the softmax or the MFMAs
// left out (not a result, a timing) a launch is 3, 7 and 11 % shorter: no unit is the limit, but the
// hand-over between the phases, some 250 cycles for every 16 MFMAs (512 cycles) of a group's 32-key tile.
// The way in and out: all arguments asked for at once, the work index by multiplication, the query rows
// through the LDS, the first scores as soon as K(0) and those rows have landed, the merge by whole rows (16
// lanes store 256 bytes side by side) take 2.4 to 2.9 us off every launch, us before / after:
//   2 groups  24 heads x 1031 x 1031 keys 23.7 / 21.0   12 x 1560 x 4680 56.1 / 53.7   36 x 449 x 898 20.8 / 18.1
//   4 groups  12 x 1031 x 1031            17.0 / 14.5   8 x 1024 x 6144 45.6 / 43.1    12 x 1031 x 6186 52.0 / 49.1
#include "block_attn_device.h"
#include "block_attn_groups_index.h"
#include "block_attn_params.h"
#include "sdvg_common.h"

namespace {

using namespace sdvg::attn_dev;
using sdvg::AttnParams;
namespace ix = sdvg::attn_index;

typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) f32x2 lds_f32x2;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

#define SDVG_SB() __builtin_amdgcn_sched_barrier(0)

template <int N>
__device__ __forceinline__ void wait_lds() {  // all but the N most recent LDS reads have returned
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// One or two 1 KB copies (lane i's 16 bytes land at dst + kAt + imm + 16 i) from a scalar address plus the lanes' offsets.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int kAt, int kSecondImm>
__device__ __forceinline__ void copy_pair(uint32_t off0, uint32_t off1, uint64_t base, uint32_t dst) {
  if constexpr (kSecondImm == 0)
    asm volatile(
        "s_add_u32 m0, %2, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(off0), "s"(base), "s"(dst), "n"(kAt)
        : "memory", "m0", "scc");
  else
    asm volatile(
        "s_add_u32 m0, %3, %4\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %0, %2\n\t"
        "global_load_lds_dwordx4 %1, %2 offset:%5"
        :
        : "v"(off0), "v"(off1), "s"(base), "s"(dst), "n"(kAt), "n"(kSecondImm)
        : "memory", "m0", "scc");
}
#pragma clang diagnostic pop

// Calls f with 0, kStep, 2 kStep ... below kEnd as constants.
template <int kEnd, int kStep, int kAt = 0, class F>
__device__ __forceinline__ void for_each(F f) {
  if constexpr (kAt < kEnd) {
    f(std::integral_constant<int, kAt>{});
    for_each<kEnd, kStep, kAt + kStep>(f);
  }
}

constexpr int kMergeSums = ix::kWaves * 32 * 512;  // O of all waves; row sums and shifts follow
constexpr int kMergeBytes = kMergeSums + ix::kWaves * 32 * 8;

// kWide: a pitch is too large for 32-bit offsets (ix::group_takes).
template <int G, bool kWide>
__global__ __launch_bounds__(512) void block_attn_groups_kernel(const AttnParams p) {
  using C = ix::Groups<G>;
  constexpr int R = C::kRowWaves, NK = C::kHalves;
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const uint32_t lds_addr0 =
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t *)smem));

  sdvg::AttnItem it = p.items[0];
  load_arguments(p, it);
  if (static_cast<int>(blockIdx.x) >= p.copy_first_block) {
    commit_block_rows(p);
    return;
  }
  const int work = ix::work_of_block(blockIdx.x, p.work_per_xcd);
  if (work >= p.total_work) return;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave / R, wr = wave % R;
  const bool half_b = wave >= 4;
  const int r32 = lane & 31, hh = lane >> 5;

  const int hq = static_cast<int>(p.div_qtiles.div(work)), qt = work - hq * p.n_qtiles;
  const int item = static_cast<int>(p.div_heads.div(hq)), head = hq - item * p.n_heads;
  if (item != 0) it = kernarg_items()[item];

  const int c_len = static_cast<int>(p.cache_len), n_blk = p.n_blk;
  const uint32_t c_pitch = static_cast<uint32_t>(p.kv_ts * 2), b_pitch = static_cast<uint32_t>(p.blk_ts * 2);
  const uint64_t kc = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.k_cache) + head * p.kv_hs);
  const uint64_t vc = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.v_cache) + head * p.kv_hs);
  const uint64_t kb = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.k_blk) + head * p.blk_hs);
  const uint64_t vb = reinterpret_cast<uint64_t>(static_cast<const uint16_t *>(it.v_blk) + head * p.blk_hs);
  const ix::GroupBounds bounds = ix::group_bounds<G>(c_len, n_blk);
  const uint64_t row0[2] = {kc, vc}, block_base[2] = {ix::group_block_base<G>(bounds, kb, b_pitch), ix::group_block_base<G>(bounds, vb, b_pitch)};
  const int n_it = (bounds.end + G - 1) / G;  // the same for all groups: one past its tiles is masked
  auto tile_of = [&](int i) __attribute__((always_inline)) { return grp + G * i; };

  // ---- copies of K [0] and V [1]: where the last tile's first row lies and how far the next one's is from there, the lanes'
  // offsets for this kind of tile, and the first tile that may be of another kind.
  uint64_t base[2], step[2];
  int bound[2] = {0, 0}, keys[2];
  uint32_t pitch[2], off[2][C::kCopies];
  auto set_kind = [&](auto is_v, int t) __attribute__((always_inline)) {
    bound[is_v] = ix::group_next_bound(bounds, t);
    keys[is_v] = ix::group_tile_keys<G>(bounds, c_len, n_blk, t);
    pitch[is_v] = t < bounds.block ? c_pitch : b_pitch;
    step[is_v] = ix::group_step<G>(bounds, t, pitch[is_v]);
    base[is_v] = ix::group_tile_base<G>(bounds, t, row0[is_v], block_base[is_v], pitch[is_v]) - step[is_v] -
                 (kWide ? 0 : ix::group_max_imm<G>());
    if constexpr (!kWide) {
#pragma unroll
      for (int u = 0; u < C::kCopies; ++u) off[is_v][u] = ix::group_lane_offset<G>(wr, lane, u, pitch[is_v], keys[is_v], is_v);
    }
  };
  // Copies u .. u + kTogether - 1 of the tile.
  auto start_copies = [&](auto is_v, auto u_c, uint32_t dst) __attribute__((always_inline)) {
    constexpr int u = decltype(u_c)::value;
    if constexpr (kWide) {
#pragma unroll
      for (int v = u; v < u + C::kTogether; ++v) {
        const int row = ix::group_copy_row<G>(wr, lane, v);
        dma16(reinterpret_cast<const char *>(
                  base[is_v] + static_cast<uint64_t>(static_cast<uint32_t>(ix::clamped_row(row, keys[is_v]))) * pitch[is_v] +
                  ix::swizzled_chunk(row, lane, is_v) * 16),
              dst + v * R * 1024);
      }
    } else {
      copy_pair<u * R * 1024, ix::group_max_imm<G>()>(off[is_v][u], off[is_v][u + C::kTogether - 1], base[is_v], dst);
    }
  };
  auto copy_tile = [&](auto is_v, int i, uint32_t dst) __attribute__((always_inline)) {
    if (tile_of(i) >= bound[is_v]) set_kind(is_v, tile_of(i));
    base[is_v] += step[is_v];
    for_each<C::kCopies, C::kTogether>([&](auto u) __attribute__((always_inline)) { start_copies(is_v, u, dst); });
  };
  constexpr std::integral_constant<int, 0> kK;
  constexpr std::integral_constant<int, 1> kV;
  uint32_t k_dst = lds_addr0 + ix::group_copy_dst<G>(grp, wr, 0, 0, 0);
  uint32_t v_dst = lds_addr0 + ix::group_copy_dst<G>(grp, wr, 0, 0, 1);
  const uint32_t k_dst0 = k_dst, v_dst_sum = 2 * v_dst + C::kTile;
  int wt_count, wt_first;  // (computed behind the first copies)
  ix::group_start_steps([&](auto what) __attribute__((always_inline)) {
    if constexpr (what == ix::kStartK0) {
      copy_tile(kK, 0, k_dst0);
    } else if constexpr (what == ix::kStartQ) {
      // The query rows (rows past the end re-read the last one and are not stored): 4 R per wave.
      wt_count = ix::wave_tiles_of_qtile(qt, p.wt_base, p.wt_rem);
      wt_first = ix::first_wave_tile_of_qtile(qt, p.wt_base, p.wt_rem);
#pragma unroll 1
      for (int r = 0; r < R; ++r) {
        const int row = 4 * wave + (lane >> 4), q_row = (wt_first + r) * 32 + row;
        dma16(static_cast<const uint16_t *>(it.q) + (q_row < p.n_q ? q_row : p.n_q - 1) * p.q_ts + head * p.q_hs +
                  ix::swizzled_chunk(row, lane, 0) * 8,
              lds_addr0 + ix::group_query_tile<G>(r) + wave * 1024);
      }
    } else if constexpr (what == ix::kStartK1K2) {
#pragma unroll 1
      for (int i = 1; i < 3; ++i) copy_tile(kK, i, k_dst0 + i * C::kTile);  // (k_dst: slot of K(3))
    } else {
      copy_tile(kV, 0, v_dst);
      v_dst += C::kTile;  // slot of V(1)
    }
  });

  // ---- LDS read addresses (bytes), with the group's part of the LDS and the slot folded in
  uint32_t k_off[8], v_off[4];
#pragma unroll
  for (int s = 0; s < 8; ++s) k_off[s] = lds_addr0 + grp * C::kGroup + ix::k_read_offset(lane, s, 0);
#pragma unroll
  for (int db = 0; db < 4; ++db) v_off[db] = lds_addr0 + grp * C::kGroup + C::kVSlots + ix::v_read_offset(lane, 0, db, 0);

  f32x16 o_acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int i = 0; i < 16; ++i) o_acc[u][i] = 0.f;
  float l_run = 0.f, s_shift = 0.f;
  f32x16 s_acc[NK];
  f32x16 s_init = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 qf[8], pf[2 * NK];
  bf16x8 f[2][4];  // two groups of 4 MFMA A-operands: one in use, one being fetched
  auto set_shift = [&](float v) __attribute__((always_inline)) {
    s_shift = v;
#pragma unroll
    for (int i = 0; i < 16; ++i) s_init[i] = v;
  };

  // The MFMAs of a matrix phase in groups of 4: groups 0 .. 2 NK - 1 are S^T = K Q^T, groups
  // 2 NK .. 4 NK - 1 are O^T += V^T P^T, one per step of 16 keys.
  auto read_op = [&](bf16x8 &dst, int gi, int i) __attribute__((always_inline)) {
    if (gi < 2 * NK) {
      const int s = NK == 2 ? 2 * gi + (i >> 1) : 4 * gi + i, kb = NK == 2 ? i & 1 : 0;
      dst = *(lds_bf16x8 *)static_cast<uintptr_t>(k_off[s] + kb * 32 * 256);
    } else {
      const uint32_t vp = v_off[i] + (gi - 2 * NK) * 16 * 256;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)static_cast<uintptr_t>(vp));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)static_cast<uintptr_t>(vp + 8 * 256));
      const __attribute__((ext_vector_type(8))) short a16 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      __builtin_memcpy(&dst, &a16, sizeof(bf16x8));
    }
  };
  auto mfma_op = [&](const bf16x8 &a, int gi, int i) __attribute__((always_inline)) {
    if (gi < 2 * NK) {
      const int s = NK == 2 ? 2 * gi + (i >> 1) : 4 * gi + i, kb = NK == 2 ? i & 1 : 0;
      s_acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[s], s == 0 ? s_init : s_acc[kb], 0, 0, 0);
    } else {
      o_acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[gi - 2 * NK], o_acc[i], 0, 0, 0);
    }
  };
  // The first two MFMAs of a group while the operands of the next group (if any) are fetched: half of
  // the reads before the first MFMA, half behind it.
  auto run_group = [&](int gi, bool fetch_next) __attribute__((always_inline)) {
    bf16x8(&cur)[4] = f[gi & 1];
    bf16x8(&nxt)[4] = f[(gi + 1) & 1];
    SDVG_SB();
    if (fetch_next) {
      read_op(nxt[0], gi + 1, 0);
      read_op(nxt[1], gi + 1, 1);
      if (gi + 1 < 2 * NK)
        wait_lds<2>();
      else
        wait_lds<4>();
    } else {
      wait_lds<0>();
    }
    SDVG_SB();
    mfma_op(cur[0], gi, 0);
    SDVG_SB();
    if (fetch_next) {
      read_op(nxt[2], gi + 1, 2);
      read_op(nxt[3], gi + 1, 3);
    }
    SDVG_SB();
    mfma_op(cur[1], gi, 1);
    SDVG_SB();
  };
  // Rows past a tile's keys get -inf (its scores are in hand).
  auto mask_tail = [&](int keys) __attribute__((always_inline)) {
#pragma unroll
    for (int kb = 0; kb < NK; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (4 * hh + kb * 32 + 8 * (i >> 2) + (i & 3) >= keys) s_acc[kb][i] = -INFINITY;
  };
  // They have P = 0, but 0 times an infinite value would be NaN: their V becomes 0 once this wave's copies have landed.
  // Without branches, each of which would be a jump to code that a launch with its keys in HBM fetches from there, too.
  auto clear_v = [&](int keys) __attribute__((always_inline)) {
    const uint32_t at = v_dst_sum - v_dst + lane * 16;
    for_each<C::kCopies, 1>([&](auto u) __attribute__((always_inline)) {
      constexpr int offset = decltype(u)::value * R * 1024;
      const uint64_t past = __ballot(ix::group_copy_row<G>(wr, lane, u) >= keys);
      const uint32_t to = at;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      asm volatile(
          "s_mov_b64 exec, %0\n\t"
          "ds_write_b128 %1, %2 offset:%3\n\t"
          "s_mov_b64 exec, -1"  // (all 64 lanes are active here)
          :
          : "s"(past), "v"(to), "v"(zero), "n"(offset)
          : "memory");
    });
    wait_lds<0>();
  };
  // Softmax with the lazy running maximum of block_attn.hip.
  auto softmax_tile = [&]() __attribute__((always_inline)) {
    float dl = form_p(s_acc, p.scale_log2e, pf);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(dl < kPSumLimit)) != 0, 0)) {
      const float d = fmaxf(tile_max(s_acc), 0.f);
      const float alpha = __builtin_amdgcn_exp2f(-d * p.scale_log2e);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[u][i] *= alpha;
      l_run *= alpha;
#pragma unroll
      for (int kb = 0; kb < NK; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s_acc[kb][i] -= d;
      set_shift(s_shift - d);
      dl = form_p(s_acc, p.scale_log2e, pf);
    }
    l_run += dl;
  };

  int keys_next = ix::group_counted_keys(bounds, tile_of(0), keys[kV]);  // of the tile whose scores come next
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ix::group_left_at_scores<G>()) : "memory");  // K(0) and the query rows
  wg_barrier();
#pragma unroll
  for (int s = 0; s < 8; ++s)
    qf[s] = *(lds_bf16x8 *)static_cast<uintptr_t>(lds_addr0 + ix::group_query_tile<G>(wr) + ix::k_read_offset(lane, s, 0));
  // ---- S of the group's first tile. All groups start from one maximum per row, that of the first 64
  // keys, as the 256-row kernel does: the groups' first-tile maxima meet in LDS (in V slot 1, which is
  // first written in matrix phase 0, a barrier after the values here are read). A group that started
  // from its own tile alone would take its shift from keys that may be masked: with -inf there is
  // nothing to subtract, and a large negative score as the accumulators' initial value leaves no bits
  // for the scores of the group's other tiles. If a first tile past the first 64 keys holds scores
  // that would raise this maximum anyway (2^20, as kPSumLimit), the row starts from those; if all
  // first tiles are masked with -inf, from 0.
  {
#pragma unroll
    for (int i = 0; i < 4; ++i) read_op(f[0][i], 0, i);
#pragma unroll
    for (int gi = 0; gi < 2 * NK; ++gi) {
      run_group(gi, gi + 1 < 2 * NK);
      mfma_op(f[gi & 1][2], gi, 2);
      mfma_op(f[gi & 1][3], gi, 3);
    }
    if (keys_next < C::kKeys) mask_tail(keys_next);
    auto first_max = [&](int g) __attribute__((always_inline)) -> float * {
      return reinterpret_cast<float *>(reinterpret_cast<char *>(smem) + g * C::kGroup + C::kVSlots + C::kTile) +
             wr * 64 + lane;
    };
    const float own = tile_max(s_acc);
    wg_barrier();  // all have read their query rows
    *first_max(grp) = own;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ix::group_left_at_maximum<G>()) : "memory");  // K(1), for the reads below
    __syncthreads();
    float mx = *first_max(0), m_all;
#pragma unroll
    for (int g = 1; g * C::kKeys < ix::kBN; ++g) mx = fmaxf(mx, *first_max(g));
    m_all = mx;
#pragma unroll
    for (int g = ix::kBN / C::kKeys; g < G; ++g) m_all = fmaxf(m_all, *first_max(g));
    if ((m_all - mx) * p.scale_log2e > 20.f) mx = m_all;
    if (mx == -INFINITY) mx = 0.f;
    asm volatile("" : "+v"(mx));  // (all reads of V slot 1 have returned)
#pragma unroll
    for (int kb = 0; kb < NK; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s_acc[kb][i] -= mx;
    set_shift(-mx);
  }
  if (half_b) wg_barrier();  // waves 4-7 run one phase behind waves 0-3

  // ---- one tile: vector phase (softmax of S(i)), barrier, matrix phase (copies of V(i+1) and K(i+3),
  // S(i+1), then O += P(i) V(i)), barrier ahead of the last MFMA.
  // What moves on from tile to tile (LDS offsets of the operands, slots and steps of the copies) is
  // updated in the gaps between the MFMAs: in the vector phase, the longer one for 32-key tiles, the
  // same instructions cost 0.1 us per iteration.
  constexpr int kPerGroup = 2 * C::kCopies / (4 * NK);  // copies started per group of MFMAs
  int k_slot = 0;                                       // slot of the K operands of the next S
  int k_move = C::kTile, v_move = C::kTile;
  auto next_k_slot = [&]() __attribute__((always_inline)) {
    k_slot = k_slot == 2 ? 0 : k_slot + 1;
    k_move = k_slot == 2 ? -2 * C::kTile : C::kTile;
  };
  // Behind the third MFMA of group gi.
  auto chores = [&](int gi, int i) __attribute__((always_inline)) {
    if (gi == 2 * NK - 1) {  // all K operands are on their way
#pragma unroll
      for (int s = 0; s < 8; ++s) k_off[s] += k_move;
    }
    if (gi == 2 * NK) {  // so are the copies of V
      next_k_slot();
      v_dst = v_dst_sum - v_dst;
    }
    if (gi == 4 * NK - 1) {
#pragma unroll
      for (int u = 0; u < 4; ++u) v_off[u] += v_move;
      v_move = -v_move;
      k_dst = k_dst == k_dst0 + 2 * C::kTile ? k_dst0 : k_dst + C::kTile;
    }
  };
#pragma unroll
  for (int s = 0; s < 8; ++s) k_off[s] += k_move;
  next_k_slot();
#pragma unroll 1
  for (int i = 0; i + 1 < n_it; ++i) {
    const int t_k = tile_of(i + 3), t_v = tile_of(i + 1);
    if (__builtin_expect(t_k >= bound[kK] || t_v >= bound[kV], 0)) {
      asm volatile("" ::: "memory");  // a real branch: keep this arithmetic off the fast path
      if (keys_next < C::kKeys) {     // of this tile (behind a short tile comes another kind)
        wait_vmcnt0();
        clear_v(keys_next);
      }
      if (t_k >= bound[kK]) set_kind(kK, t_k);
      if (t_v >= bound[kV]) {
        set_kind(kV, t_v);
        keys_next = ix::group_counted_keys(bounds, t_v, keys[kV]);
      }
    }
    base[kK] += step[kK];
    base[kV] += step[kV];
    softmax_tile();
    asm volatile("" : "+v"(s_init));
#pragma unroll
    for (int a = 0; a < 4; ++a) read_op(f[0][a], 0, a);
#pragma unroll
    for (int j = 0; j < 2 * NK; ++j) asm volatile("" : "+v"(pf[j]));
    asm volatile("" : "+v"(l_run));
    wait_vmcnt0();  // the copies started in the previous matrix phase have landed
    wg_barrier();
    __builtin_amdgcn_s_setprio(1);
    for_each<4 * NK, 1>([&](auto gi_c) __attribute__((always_inline)) {
      constexpr int gi = decltype(gi_c)::value;
      run_group(gi, gi + 1 < 4 * NK);
      for_each<(gi + 1) * kPerGroup, C::kTogether, gi * kPerGroup>([&](auto c) __attribute__((always_inline)) {
        constexpr int n = C::kCopies;
        if constexpr (c < n)
          start_copies(kV, c, v_dst);
        else
          start_copies(kK, std::integral_constant<int, c - n>{}, k_dst);
      });
      SDVG_SB();
      mfma_op(f[gi & 1][2], gi, 2);
      SDVG_SB();
      chores(gi, i);
      SDVG_SB();
      if (gi + 1 < 4 * NK) mfma_op(f[gi & 1][3], gi, 3);
      SDVG_SB();
      if (gi == 2 * NK - 1 && __builtin_expect(keys_next < C::kKeys, 0)) mask_tail(keys_next);
    });
    __builtin_amdgcn_s_setprio(2);
    wg_barrier();
    SDVG_SB();
    mfma_op(f[1][3], 4 * NK - 1, 3);
    SDVG_SB();
    __builtin_amdgcn_s_setprio(0);
  }
  // ---- the last tile: nothing left to copy and no next S
  softmax_tile();
#pragma unroll
  for (int j = 0; j < 2 * NK; ++j) asm volatile("" : "+v"(pf[j]));
  wait_vmcnt0();
  // (A group past the last tile takes no product and clears nothing. That, and this and the mask in line: 12 heads x 780 x 780
  // and 12 x 800 x 800 keys from HBM 14.4 / 14.1 and 14.7 / 14.2 us.)
  if (__builtin_expect(keys_next < C::kKeys && keys_next > 0, 1)) clear_v(keys_next);
  wg_barrier();
  // A group that is past the last tile has only the last key's row there, with P = 0; it adds nothing,
  // because 0 times an infinite value would be NaN.
  if (tile_of(n_it - 1) < bounds.end) {
#pragma unroll
    for (int a = 0; a < 4; ++a) read_op(f[0][a], 2 * NK, a);
#pragma unroll
    for (int gi = 2 * NK; gi < 4 * NK; ++gi) {
      run_group(gi, gi + 1 < 4 * NK);
      mfma_op(f[gi & 1][2], gi, 2);
      mfma_op(f[gi & 1][3], gi, 3);
    }
  }
  wg_barrier();
  if (!half_b) wg_barrier();  // pairs with the extra barrier of waves 4-7: all LDS reads are done

  // ---- merge: every wave leaves its O, row sum and shift in LDS and combines the groups' parts of four
  // rows of each row wave: with m the largest running maximum,
  //   O = sum_g 2^((m_g - m) scale*log2e) O_g, l likewise.
  const uint32_t part = lds_addr0 + wave * 32 * 512;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(lds_f32x4 *)static_cast<uintptr_t>(part + ix::merge_offset(4 * u + g, hh, r32)) =
          f32x4{o_acc[u][4 * g], o_acc[u][4 * g + 1], o_acc[u][4 * g + 2], o_acc[u][4 * g + 3]};
  const float l_row = lane_sum32(l_run);
  if (hh == 0) *(lds_f32x2 *)static_cast<uintptr_t>(lds_addr0 + kMergeSums + (wave * 32 + r32) * 8) = f32x2{l_row, s_shift};
  __syncthreads();
  const int row = 4 * wave + (lane >> 4), c = lane & 15;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r >= wt_count) return;
    float l_g[G], shift_g[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const f32x2 v = *(lds_f32x2 *)static_cast<uintptr_t>(lds_addr0 + kMergeSums + ((g * R + r) * 32 + row) * 8);
      l_g[g] = v[0];
      shift_g[g] = v[1];
    }
    float shift_min = shift_g[0];
#pragma unroll
    for (int g = 1; g < G; ++g) shift_min = fminf(shift_min, shift_g[g]);
    float l_sum = 0.f;
    f32x4 o_lo = {0.f, 0.f, 0.f, 0.f}, o_hi = o_lo;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float factor = __builtin_amdgcn_exp2f((shift_min - shift_g[g]) * p.scale_log2e);
      l_sum += factor * l_g[g];
      const uint32_t from = lds_addr0 + (g * R + r) * 32 * 512;
      const f32x4 lo = *(lds_f32x4 *)static_cast<uintptr_t>(from + ix::merge_offset(c, 0, row));
      const f32x4 hi = *(lds_f32x4 *)static_cast<uintptr_t>(from + ix::merge_offset(c, 1, row));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o_lo[e] += factor * lo[e];
        o_hi[e] += factor * hi[e];
      }
    }
    const float inv_l = 1.0f / l_sum;
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      out[e] = static_cast<__bf16>(o_lo[e] * inv_l);
      out[4 + e] = static_cast<__bf16>(o_hi[e] * inv_l);
    }
    const int q_row = (wt_first + r) * 32 + row;
    if (q_row < p.n_q)
      *reinterpret_cast<bf16x8 *>(static_cast<uint16_t *>(it.out) + q_row * p.o_ts + head * p.o_hs + 8 * c) = out;
  }
}

template <int G>
constexpr size_t lds_bytes() {
  return G * ix::Groups<G>::kGroup > kMergeBytes ? G * ix::Groups<G>::kGroup : kMergeBytes;
}

}  // namespace

namespace sdvg {

hipError_t prepare_block_attn_groups() {
  const struct {
    const void *kernel;
    size_t lds_bytes;
  } kernels[] = {{reinterpret_cast<const void *>(block_attn_groups_kernel<2, false>), lds_bytes<2>()},
                 {reinterpret_cast<const void *>(block_attn_groups_kernel<2, true>), lds_bytes<2>()},
                 {reinterpret_cast<const void *>(block_attn_groups_kernel<4, false>), lds_bytes<4>()},
                 {reinterpret_cast<const void *>(block_attn_groups_kernel<4, true>), lds_bytes<4>()}};
  for (const auto &k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(k.lds_bytes));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int G>
static void launch(const AttnParams &p, hipStream_t s) {
  const bool wide = (p.cache_len > 0 && !ix::group_takes(static_cast<uint64_t>(p.kv_ts) * 2)) ||
                    !ix::group_takes(static_cast<uint64_t>(p.blk_ts) * 2);
  const auto kernel = wide ? block_attn_groups_kernel<G, true> : block_attn_groups_kernel<G, false>;
  hipLaunchKernelGGL(kernel, dim3(8 * p.work_per_xcd + p.n_copy_blocks), dim3(512), lds_bytes<G>(), s, p);
}

int launch_block_attn_groups(const AttnParams &p, int groups, hipStream_t s) {
  if (groups == 2)
    launch<2>(p, s);
  else
    launch<4>(p, s);
  SDVG_HIP_CHECK(hipGetLastError());
  return SDVG_OK;
}

}  // namespace sdvg
