"""GPU parity of the bf16 attention kernels by kernel: the one whose workgroups own 256 query rows (1
group) and the one that splits a workgroup's keys over 2 or 4 groups of waves (few query rows), against
the fp64 oracle. Where a few heads take 4 groups here, the launch is so small that the 32-row kernel runs
it (`rows`); the 64-row kernel of 4 groups has the same cases in test_gpu_attn_rows32.py. Tile and seam edges, a group past the last tile, a running maximum that rises late or
lives in one group only, masked first tiles, infinite values, strides, scale, fused commit. The launch
plan decides which kernel runs, so every case asks it and asserts the answer.
The bounds are the bf16 path's (probabilities and output rounded to bf16, fp32 sums)."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import sdvg_inputs as si
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, MI355X_CUS, attn_errors, attn_plan, bits_of, to_dev_bf16
from test_gpu_attn import structured_case

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_copy_schedule_on_the_host(tmp_path):
    exe = str(tmp_path / "replay")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2604_17397_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_groups_replay.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok:"), res.stdout


def test_plan_by_size():
    """The group count the plan gives on 256 compute units: the shapes it was fitted to, the largest call
    that keeps the 256-row kernel for having few keys, and no group without a tile: that takes 96 keys or
    fewer (64 for 2 groups), where 1 group is the plan at any number of rows."""
    groups = lambda H, n_q, n_k, **kw: attn_plan(H, n_q, n_k, n_cu=MI355X_CUS, **kw).groups
    assert [groups(12, 312, 936), groups(12, 1031, 6186), groups(12, 1560, 4680), groups(5, 4680, 32760)] == [4, 4, 2, 2]
    assert [groups(40, 1031, 3093), groups(16, 4680, 14040), groups(12, 4680, 14040), groups(1, 8, 8)] == [1, 2, 1, 1]
    assert [groups(3, 97, 192), groups(3, 97, 193)] == [1, 4]
    for H in (1, 3, 12, 40, 129, 255, 256, 257, 1000):
        for n_q in (1, 64, 65, 128, 129, 256, 257, 1031, 4680):
            assert all(groups(H, n_q, n_k) == 1 for n_k in (1, 32, 33, 64, 65, 96, 97, 128)), (H, n_q)
    split = attn_plan(1, 4680, 32760, n_cu=MI355X_CUS, split=1)
    assert split.split and split.workgroups <= MI355X_CUS and split.workspace > 0
    auto = attn_plan(16, 1031, 3093, n_cu=MI355X_CUS, split=1)
    assert not auto.split and auto.workspace == attn_plan(16, 1031, 3093, n_cu=MI355X_CUS, split=2).workspace > 0


def run(H, n_q, n_blk, c_len, seed, groups, head_major=False, jitter=False):
    import paper_2604_17397_amd as P
    assert attn_plan(H, n_q, c_len + n_blk).groups == groups
    q, kc, vc, kb, vb = si.attn_inputs(H, max(n_q, n_blk), c_len, seed=seed, jitter=jitter, cache_capacity=c_len + 3)
    q, kb, vb = (np.ascontiguousarray(a) for a in (q[:n_q], kb[:n_blk], vb[:n_blk]))
    d = {k: to_dev_bf16(a) for k, a in dict(q=q, kc=kc, vc=vc, kb=kb, vb=vb).items()}
    if head_major:
        d["kc"], d["vc"] = (d[k].transpose(0, 1).contiguous().transpose(0, 1) for k in ("kc", "vc"))
    out = torch.full_like(d["q"], float("nan"))
    P.block_attn(d["q"], d["kc"], d["vc"], d["kb"], d["vb"], c_len, out=out)
    torch.cuda.synchronize()
    ref = oracle.block_attn(q, kc, vc, kb, vb, c_len)
    max_abs, rel = attn_errors(bits_of(out), ref)
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)


# 3 heads x few rows: 4 groups of 32-key tiles from 193 keys on, the 256-row kernel below; the seam
# inside / at the edge of a tile, in every group in turn
@pytest.mark.gpu
@pytest.mark.parametrize("c_len", [0, 1, 31, 32, 33, 64, 95, 127, 128, 161])
@pytest.mark.parametrize("n_blk,n_q", [(97, 97), (128, 64), (129, 65), (250, 33)])
def test_four_groups_edges(c_len, n_blk, n_q):
    run(3, n_q, n_blk, c_len, seed=500 + c_len, groups=4 if n_blk + c_len > 192 else 1)


@pytest.mark.gpu
@pytest.mark.parametrize("n_blk,n_q,c_len", [(300, 300, 1500), (312, 312, 624)])
@pytest.mark.parametrize("head_major", [False, True])
def test_four_groups_with_jitter_and_strides(n_blk, n_q, c_len, head_major):
    run(5, n_q, n_blk, c_len, seed=520, groups=4, head_major=head_major, jitter=True)


# 36 heads: from 449 rows on workgroups of 64 rows would need two rounds, those of 128 rows fit one
@pytest.mark.gpu
@pytest.mark.parametrize("n_q,n_blk,c_len,groups", [(385, 385, 511, 4), (512, 450, 640, 2), (449, 449, 577, 2)])
def test_two_groups(n_q, n_blk, c_len, groups):
    run(36, n_q, n_blk, c_len, seed=540 + c_len, groups=groups)


# 129 heads x 65 .. 128 rows are more than a round of 64-row workgroups and half a round of 128-row ones;
# with 193 .. 256 rows only 256-row workgroups fit one round.
HEADS = {4: 3, 2: 129, 1: 129}


def run_planned(groups, n_q, n_blk, c_len, seed, head_major=False, jitter=False, scale=None, commit=False):
    """One launch of the kernel with this many groups. The cache has room past cache_len, filled with NaN;
    the first, the middle and the last head are compared with the oracle."""
    import paper_2604_17397_amd as P
    H = HEADS[groups]
    assert attn_plan(H, n_q, c_len + n_blk).groups == groups
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def draw(n, which):
        x = torch.randn((n, H, 128), generator=gen, device="cuda")
        if jitter:
            x *= torch.from_numpy(si.head_scales(seed, H, which).astype(np.float32)).cuda()[None, :, None]
        return x.bfloat16()

    q, kb, vb = draw(n_q, 0), draw(n_blk, 1), draw(n_blk, 2)
    kc, vc = (torch.cat([draw(c_len, w), torch.full((n_blk + 3, H, 128), float("nan"), device="cuda").bfloat16()])
              for w in (1, 2))
    out = torch.full_like(q, float("nan"))
    if head_major:
        q, kc, vc, kb, vb, out = (t.transpose(0, 1).contiguous().transpose(0, 1) for t in (q, kc, vc, kb, vb, out))
    before = kc.clone(), vc.clone()
    P.block_attn(q, kc, vc, kb, vb, c_len, out=out, scale=scale)
    heads = sorted({0, H // 2, H - 1})
    got, *host = (bits_of(t[:, heads]) for t in (out, q, kc[:c_len + 1], vc[:c_len + 1], kb, vb))
    max_abs, rel = attn_errors(got, oracle.block_attn(*host, c_len, scale=scale))
    # Rounding the weights to bf16 moves a row by at most 2 * 2^-9 of the largest value (numerator and row
    # sum use the same weights), rounding the result by 2^-9 of it: heads of larger values are allowed more.
    v_max = max(float(t[:, heads].float().abs().max()) for t in (vc[:max(c_len, 1)], vb) if not t[0].isnan().any())
    assert max_abs <= max(BF16_MAX_ABS, 3 * 2.0 ** -9 * v_max) and rel <= BF16_REL_RMS, (max_abs, rel)
    assert torch.isfinite(out).all()
    if commit:
        fused = P.block_attn_commit(q, kc, vc, kb, vb, c_len, scale=scale)
        assert torch.equal(fused.view(torch.int16), out.view(torch.int16))
        for cache, blk, was in ((kc, kb, before[0]), (vc, vb, before[1])):
            want = torch.cat([was[:c_len], blk, was[c_len + n_blk:]])
            assert torch.equal(cache.view(torch.int16), want.view(torch.int16))


# Key counts about the ends of tiles and of rounds of groups (128 keys; the 256-row kernel: about its
# ring of four tiles), with the seam anywhere in the first rounds: a third of the pairs of the two.
@pytest.mark.gpu
@pytest.mark.parametrize("groups,n_q", [(4, 33), (4, 64), (4, 97), (2, 65), (2, 97), (2, 128), (1, 193), (1, 225), (1, 256)])
@pytest.mark.parametrize("n_k", [193, 224, 225, 256, 257, 320, 385, 641])
def test_edges_by_kernel(groups, n_q, n_k):
    for i, c_len in enumerate([0, 1, 31, 33, 64, 95, 127, 161]):
        if (i + n_q + n_k) % 3 == 0:
            run_planned(groups, n_q, n_k - c_len, c_len, seed=600 + i)


@pytest.mark.gpu
@pytest.mark.parametrize("groups,n_q", [(4, 70), (2, 100), (1, 250)])
@pytest.mark.parametrize("head_major,jitter,scale", [(True, False, None), (False, True, None), (True, True, 0.05)])
def test_strides_scale_and_commit_by_kernel(groups, n_q, head_major, jitter, scale):
    run_planned(groups, n_q, 300, 407, seed=650, head_major=head_major, jitter=jitter, scale=scale, commit=True)
    run_planned(groups, n_q, 333, 0, seed=651, head_major=head_major, jitter=jitter, scale=scale, commit=True)


# The 32-row kernel takes the same profiles from 2 heads x 70 rows in test_gpu_attn.py, the 64-row kernel with 4 groups
# in test_gpu_attn_rows32.py.
@pytest.mark.gpu
@pytest.mark.parametrize("groups,n_q", [(2, 70), (1, 200)])
@pytest.mark.parametrize("pattern", ["rising", "falling", "spike_last"])
@pytest.mark.parametrize("amp", [8.0, 40.0, 150.0])
def test_score_profiles_by_kernel(groups, n_q, pattern, amp):
    assert attn_plan(2, 70, 700).rows == 32 and attn_plan(HEADS[groups], n_q, 700).groups == groups
    max_abs, rel = structured_case(pattern, n_q=n_q, H=HEADS[groups], amp=amp)
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)


@pytest.mark.gpu
@pytest.mark.parametrize("groups", [4, 2])
@pytest.mark.parametrize("n_k,hot", [(300, 299), (300, 0), (300, 40), (1100, 1099), (1100, 700)])
def test_maximum_in_one_group_only(n_k, hot, groups):
    maximum_in_one_group_only({4: 2, 2: 129}[groups], 70, n_k, hot, rows={4: 32, 2: 128}[groups])


def maximum_in_one_group_only(H, n_q, n_k, hot, rows):
    """One key's score towers above the others (by 2^40 in the softmax), so that the other groups'
    shares of the merge vanish; rows below a gain of 1 stay diffuse."""
    import paper_2604_17397_amd as P
    rng = np.random.default_rng(3)
    c_len = 123
    assert attn_plan(H, n_q, n_k).rows == rows
    u = rng.standard_normal(128)
    u /= np.linalg.norm(u)
    q = np.linspace(0.0, 25.0, n_q)[:, None, None] * u[None, None, :].repeat(H, 1)
    k = rng.standard_normal((n_k, H, 128)) * 0.3
    k[hot] = 13.0 * u
    v = rng.standard_normal((n_k, H, 128))
    bits = lambda a: si.f32_to_bf16_bits(a.astype(np.float32))
    q, k, v = bits(q), bits(k), bits(v)
    kc, vc, kb, vb = (np.ascontiguousarray(a) for a in (k[:c_len], v[:c_len], k[c_len:], v[c_len:]))
    out = P.block_attn(*(to_dev_bf16(a) for a in (q, kc, vc, kb, vb)), c_len)
    torch.cuda.synchronize()
    max_abs, rel = attn_errors(bits_of(out), oracle.block_attn(q, kc, vc, kb, vb, c_len))
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)


@pytest.mark.gpu
def test_nan_and_infinite_values_reach_the_rows_that_use_them():
    nan_and_infinite_values(2, 100, rows=32)


def nan_and_infinite_values(H, n_q, rows):
    """A NaN query row is NaN, its neighbours are not; an infinite value is infinite where its weight
    is positive and leaves the other dims alone."""
    import paper_2604_17397_amd as P
    assert attn_plan(H, n_q, 130 + n_q).rows == rows
    q, kc, vc, kb, vb = si.attn_inputs(H, n_q, 130, seed=77)
    dev = [to_dev_bf16(a) for a in (q, kc, vc, kb, vb)]
    dev[0][7, 1] = float("nan")
    dev[2][50, 0, 5] = float("inf")
    out = P.block_attn(*dev, 130)
    torch.cuda.synchronize()
    nan = torch.isnan(out)
    assert nan[7, 1].all() and not nan[8:].any() and not nan[:7].any() and not nan[7, 0].any()
    assert torch.isinf(out[:, 0, 5]).all() and torch.isfinite(out[:, 0, :5]).all() and torch.isfinite(out[8:, 1]).all()


# ---------------------------------------------------------------- masked keys, infinite values

# (heads, query rows): 3 x 70 rows take 4 groups of 32-key tiles at 936 keys (the 32-row kernel), 36 x 449 rows 2 of 64
SHAPES = {4: (3, 70), 2: (36, 449)}
N_K = 936


def masked_inputs(groups, lo, hi, value, seed):
    """Random inputs whose keys lo .. hi - 1 score `value` / sqrt(128) in every head but the first: dim 0
    is 1 in every query and `value` in these keys, 0 in the others."""
    H, n_q = SHAPES[groups]
    assert attn_plan(H, n_q, N_K).groups == groups
    c_len = N_K - n_q
    q, kc, vc, kb, vb = si.attn_inputs(H, n_q, c_len, seed=seed)
    bits = lambda x: si.f32_to_bf16_bits(np.float32([x]))[0]
    k = np.concatenate([kc, kb])
    q[:, :, 0], k[:, :, 0], k[lo:hi, 1:, 0] = bits(1.0), 0, bits(value)
    return q, np.ascontiguousarray(k[:c_len]), vc, np.ascontiguousarray(k[c_len:]), vb, c_len


# One group's first tile (4 groups: 32 keys each; 2 groups: 64), several of them, and later tiles. All
# first tiles only with -inf: a finite maximum of them is the maximum the scores start from.
MASKED = [(lo, hi, value) for lo, hi in [(0, 32), (32, 64), (64, 96), (96, 128), (0, 64), (64, 128), (32, 128), (0, 96),
                                         (128, 256), (904, 936)]
          for value in (float("-inf"), -1e9, -1e30)] + [(0, 128, float("-inf"))]


@pytest.mark.gpu
@pytest.mark.parametrize("groups", [2, 4])
@pytest.mark.parametrize("lo,hi,value", MASKED)
def test_masked_first_tiles(groups, lo, hi, value):
    """A key far below the others has weight 0 and leaves the others as they are, whichever group's tile
    it lies in. The bounds are the bf16 path's: the shift is a score of an unmasked key, or 0."""
    import paper_2604_17397_amd as P
    q, kc, vc, kb, vb, c_len = masked_inputs(groups, lo, hi, value, seed=lo + hi)
    out = P.block_attn(*(to_dev_bf16(a) for a in (q, kc, vc, kb, vb)), c_len)
    torch.cuda.synchronize()
    rows = sorted({0, 1, 31, 32, 63, len(q) - 1})
    max_abs, rel = attn_errors(bits_of(out)[rows], oracle.block_attn(q, kc, vc, kb, vb, c_len, rows=rows))
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)
    assert torch.isfinite(out).all()


# n_k is a whole number of tiles but not of rounds of groups: 10 tiles of 32 keys, 15 of 64
@pytest.mark.gpu
@pytest.mark.parametrize("groups,n_k", [(4, 320), (4, 352), (2, 960)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_infinite_value_in_the_last_key(groups, n_k, value):
    """The last key's value row is also what a group past the last tile has in hand; its weight there is
    no key's weight, and 0 * inf is not part of any row."""
    import paper_2604_17397_amd as P
    H, n_q = SHAPES[groups]
    assert attn_plan(H, n_q, n_k).groups == groups
    c_len = n_k - n_q
    q, kc, vc, kb, vb = si.attn_inputs(H, n_q, c_len, seed=n_k)
    dev = [to_dev_bf16(a) for a in (q, kc, vc, kb, vb)]
    plain = P.block_attn(*dev, c_len)
    dev[4][-1, 0, 5] = value
    out = P.block_attn(*dev, c_len)
    torch.cuda.synchronize()
    want = plain.clone()
    want[:, 0, 5] = value
    assert torch.equal(torch.nan_to_num(out, 1.5, 2.5, 3.5), torch.nan_to_num(want, 1.5, 2.5, 3.5))


# K(1) is read ahead of the loop's first wait and barrier: cold keys beside a commit's copies, many times. Between the
# launches 512 MiB are written, so that neither L2 nor the memory-side cache holds the keys.
@pytest.mark.gpu
@pytest.mark.parametrize("groups,n_q", [(4, 64), (2, 100)])
def test_second_tile_has_landed_when_it_is_read(groups, n_q):
    import paper_2604_17397_amd as P
    H, n_blk, c_len = 129, 300, 407
    assert attn_plan(H, n_q, c_len + n_blk).groups == groups
    gen = torch.Generator(device="cuda").manual_seed(710)
    q, kb, vb = (torch.randn((n, H, 128), generator=gen, device="cuda").bfloat16() for n in (n_q, n_blk, n_blk))
    kc, vc = (torch.randn((c_len + n_blk, H, 128), generator=gen, device="cuda").bfloat16() for _ in range(2))
    flush = torch.empty(512 << 20, dtype=torch.uint8, device="cuda")
    want = P.block_attn(q, kc, vc, kb, vb, c_len)
    for i in range(40):
        flush.fill_(i)
        assert torch.equal(P.block_attn(q, kc, vc, kb, vb, c_len), want)
        flush.fill_(i)
        assert torch.equal(P.block_attn_commit(q, kc, vc, kb, vb, c_len), want)


# The cache's keys end inside a tile (218 = 6 x 32 + 26 = 3 x 64 + 26), and so do the block's: the rows behind them repeat the
# last key with P = 0, which must not meet an infinite value.
@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,n_blk,groups,rows", [(129, 64, 70, 4, 64), (36, 449, 680, 2, 128)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_infinite_value_in_the_last_key_of_each_source(H, n_q, n_blk, groups, rows, value):
    import paper_2604_17397_amd as P
    plan = attn_plan(H, n_q, 218 + n_blk)
    assert plan.groups == groups and plan.rows == rows
    q, kc, vc, kb, vb = si.attn_inputs(H, max(n_q, n_blk), 218, seed=6)
    dev = [to_dev_bf16(np.ascontiguousarray(a)) for a in (q[:n_q], kc, vc, kb[:n_blk], vb[:n_blk])]
    want = P.block_attn(*dev, 218)
    dev[2][217, 0, 5] = dev[4][-1, 1, 7] = value
    out = P.block_attn(*dev, 218)
    want[:, 0, 5] = want[:, 1, 7] = value
    assert torch.equal(torch.nan_to_num(out, 1.5, 2.5, 3.5), torch.nan_to_num(want, 1.5, 2.5, 3.5))
