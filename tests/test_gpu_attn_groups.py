"""GPU parity of the attention launches that split a workgroup's keys over groups of waves (few query
rows), against the fp64 oracle: 2 and 4 groups, tile and seam edges, groups without a single key, a
running maximum that rises late or lives in one group only, batch = single calls, fused commit.
The bounds are the bf16 path's (probabilities and output rounded to bf16, fp32 sums)."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import sdvg_inputs as si
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, attn_errors, bits_of, to_dev_bf16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_copy_schedule_on_the_host(tmp_path):
    exe = str(tmp_path / "replay")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2604_17397_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_groups_replay.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok:"), res.stdout


def run(H, n_q, n_blk, c_len, seed, head_major=False, jitter=False):
    import paper_2604_17397_amd as P
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


# 3 heads x few rows: 4 groups of 32-key tiles; n_k from one tile short of a round of groups to
# just past one, seam inside / at the edge of a tile, in every group in turn
@pytest.mark.gpu
@pytest.mark.parametrize("c_len", [0, 1, 31, 32, 33, 64, 95, 127, 128, 161])
@pytest.mark.parametrize("n_blk,n_q", [(97, 97), (128, 64), (129, 65), (250, 33)])
def test_four_groups_edges(c_len, n_blk, n_q):
    run(3, n_q, n_blk, c_len, seed=500 + c_len)


@pytest.mark.gpu
@pytest.mark.parametrize("n_blk,n_q,c_len", [(300, 300, 1500), (312, 312, 624)])
@pytest.mark.parametrize("head_major", [False, True])
def test_four_groups_with_jitter_and_strides(n_blk, n_q, c_len, head_major):
    run(5, n_q, n_blk, c_len, seed=520, head_major=head_major, jitter=True)


# 32 heads x 400+ rows: workgroups of 128 rows fill one round, those of 64 rows would need two
@pytest.mark.gpu
@pytest.mark.parametrize("n_q,n_blk,c_len", [(385, 385, 511), (512, 450, 640), (449, 449, 577)])
def test_two_groups(n_q, n_blk, c_len):
    run(36, n_q, n_blk, c_len, seed=540 + c_len)


@pytest.mark.gpu
@pytest.mark.parametrize("n_k,hot", [(300, 299), (300, 0), (300, 40), (1100, 1099), (1100, 700)])
def test_maximum_in_one_group_only(n_k, hot):
    """One key's score towers above the others (by 2^40 in the softmax), so that the other groups'
    shares of the merge vanish; rows below a gain of 1 stay diffuse."""
    import paper_2604_17397_amd as P
    rng = np.random.default_rng(3)
    H, n_q, c_len = 2, 70, 123
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
    """A NaN query row is NaN, its neighbours are not; an infinite value is infinite where its weight
    is positive and leaves the other dims alone."""
    import paper_2604_17397_amd as P
    q, kc, vc, kb, vb = si.attn_inputs(2, 100, 130, seed=77)
    dev = [to_dev_bf16(a) for a in (q, kc, vc, kb, vb)]
    dev[0][7, 1] = float("nan")
    dev[2][50, 0, 5] = float("inf")
    out = P.block_attn(*dev, 130)
    torch.cuda.synchronize()
    nan = torch.isnan(out)
    assert nan[7, 1].all() and not nan[8:].any() and not nan[:7].any() and not nan[7, 0].any()
    assert torch.isinf(out[:, 0, 5]).all() and torch.isfinite(out[:, 0, :5]).all() and torch.isfinite(out[8:, 1]).all()


# ---------------------------------------------------------------- masked keys, infinite values

# (heads, query rows): 3 x 70 rows take 4 groups of 32-key tiles at 936 keys, 36 x 449 rows 2 of 64
SHAPES = {4: (3, 70), 2: (36, 449)}
N_K = 936


def masked_inputs(groups, lo, hi, value, seed):
    """Random inputs whose keys lo .. hi - 1 score `value` / sqrt(128) in every head but the first: dim 0
    is 1 in every query and `value` in these keys, 0 in the others."""
    H, n_q = SHAPES[groups]
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
