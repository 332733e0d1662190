"""GPU parity of the 32-row attention kernel (the smallest launches of 4 key groups) at the edges of its
tiles and rounds, and of the 64-row kernel with 4 groups, which keeps the launches of more than one round
of 32-row workgroups. The launch plan is asked which of the two a case runs."""
import os
import subprocess

import pytest
import torch

import test_gpu_attn_groups as by_groups
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, MI355X_CUS, attn_plan_rows
from test_gpu_attn import structured_case

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# 3 heads are one round of 32-row workgroups; 129 heads x 33 .. 64 rows are two, and one of 64 rows
HEADS = {32: 3, 64: 129}


def test_copies_on_the_host(tmp_path):
    exe = str(tmp_path / "replay")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2604_17397_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "attn_rows32_replay.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok:"), res.stdout


def test_plan_by_rounds_and_pitch():
    rows = lambda H, n_q, n_k, **kw: attn_plan_rows(H, n_q, n_k, n_cu=MI355X_CUS, **kw)
    assert [rows(16, 512, 1000), rows(16, 513, 1000), rows(1, 4680, 32760), rows(2, 33, 193), rows(2, 33, 192)] == [32, 64, 32, 32, 256]
    assert rows(16, 512, 1000, rows32_ok=0) == 64
    # whoever does not take 4 groups does not take 32 rows
    assert [rows(12, 1560, 4680), rows(40, 4680, 32760), rows(12, 4680, 14040)] == [128, 256, 256]


def run(rows, monkeypatch, n_q, n_blk, c_len, **kw):
    monkeypatch.setitem(by_groups.HEADS, 4, HEADS[rows])
    assert attn_plan_rows(HEADS[rows], n_q, c_len + n_blk) == rows
    by_groups.run_planned(4, n_q, n_blk, c_len, **kw)


# Tiles of 32 keys, of the cache first, then of the block; eight waves take them in turn. 193 keys leave a
# wave without a tile, 256 are a round, 257 begin the next one.
@pytest.mark.gpu
@pytest.mark.parametrize("n_k", [193, 224, 255, 256, 257, 288, 511, 513, 800])
@pytest.mark.parametrize("c_len", [0, 1, 31, 32, 33, 63, 127, 160, 192])
def test_edges_of_the_tiles(monkeypatch, n_k, c_len):
    run(32, monkeypatch, [1, 31, 32, 33, 97][(n_k + c_len) % 5], n_k - c_len, c_len, seed=n_k + c_len)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,n_q", [(32, 65), (64, 33), (64, 64)])
@pytest.mark.parametrize("head_major,jitter,scale", [(True, False, None), (False, True, None), (True, True, 0.05)])
def test_strides_scale_and_commit(monkeypatch, rows, n_q, head_major, jitter, scale):
    for n_blk, c_len in ((300, 407), (333, 0)):
        run(rows, monkeypatch, n_q, n_blk, c_len, seed=660, head_major=head_major, jitter=jitter, scale=scale, commit=True)


# What the 64-row kernel no longer gets from the cases of 3 heads
@pytest.mark.gpu
@pytest.mark.parametrize("n_k", [193, 224, 225, 256, 257, 320, 385, 641])
def test_edges_of_the_64_row_kernel(monkeypatch, n_k):
    for i, c_len in enumerate([0, 1, 31, 33, 64, 95, 127, 161]):
        if (i + n_k) % 2 == 0:
            run(64, monkeypatch, 33 + i, n_k - c_len, c_len, seed=670 + i)


@pytest.mark.gpu
@pytest.mark.parametrize("lo,hi,value", by_groups.MASKED)
def test_masked_first_tiles_of_the_64_row_kernel(monkeypatch, lo, hi, value):
    monkeypatch.setitem(by_groups.SHAPES, 4, (129, 64))
    assert attn_plan_rows(129, 64, by_groups.N_K) == 64
    by_groups.test_masked_first_tiles(4, lo, hi, value)


# A maximum that rises from tile to tile (the rescaling in the loop), falls, or comes with the last key
@pytest.mark.gpu
@pytest.mark.parametrize("pattern", ["rising", "falling", "spike_last"])
@pytest.mark.parametrize("amp", [8.0, 40.0, 150.0])
def test_score_profiles_of_the_64_row_kernel(pattern, amp):
    assert attn_plan_rows(129, 63, 700) == 64
    max_abs, rel = structured_case(pattern, n_q=63, H=129, amp=amp)
    assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)


# Every group in turn (32-key tiles 0, 1, 2 and 3 of a round), the first round, the last and one between
@pytest.mark.gpu
@pytest.mark.parametrize("n_k,hot", [(300, 299), (300, 0), (300, 40), (300, 70), (300, 100), (1100, 1099), (1100, 700)])
def test_maximum_in_one_group_of_the_64_row_kernel(n_k, hot):
    by_groups.maximum_in_one_group_only(129, 64, n_k, hot, rows=64)


@pytest.mark.gpu
def test_nan_and_infinite_values_in_the_64_row_kernel():
    by_groups.nan_and_infinite_values(129, 64, rows=64)


# Groups 2 and 3 (320 keys), or group 3 alone (352), have no tile in the last round
@pytest.mark.gpu
@pytest.mark.parametrize("n_k", [320, 352])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_infinite_value_in_the_last_key_of_the_64_row_kernel(monkeypatch, n_k, value):
    monkeypatch.setitem(by_groups.SHAPES, 4, (129, 64))
    assert attn_plan_rows(129, 64, n_k) == 64
    by_groups.test_infinite_value_in_the_last_key(4, n_k, value)


# Short tiles repeat their last key; here both have one: the cache's ends at 218 keys, the block's at 70.
@pytest.mark.gpu
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_infinite_value_in_the_last_key_of_a_short_tile(value):
    import paper_2604_17397_amd as P
    import sdvg_inputs as si
    from gpu_util import to_dev_bf16
    assert attn_plan_rows(3, 70, 288) == 32
    dev = [to_dev_bf16(a) for a in si.attn_inputs(3, 70, 218, seed=5)]
    plain = P.block_attn(*dev, 218)
    dev[2][217, 0, 5] = dev[4][-1, 1, 7] = value
    out = P.block_attn(*dev, 218)
    want = plain.clone()
    want[:, 0, 5] = want[:, 1, 7] = value
    assert torch.equal(torch.nan_to_num(out, 1.5, 2.5, 3.5), torch.nan_to_num(want, 1.5, 2.5, 3.5))


@pytest.mark.gpu
def test_several_items():
    """The items of a batch are the same as one call each (both run the 32-row kernel)."""
    import paper_2604_17397_amd as P
    import sdvg_inputs as si
    from gpu_util import to_dev_bf16
    assert attn_plan_rows(3, 100, 430, n_items=3) == 32
    items = [[to_dev_bf16(a) for a in si.attn_inputs(3, 100, 330, seed=s)] for s in (1, 2, 3)]
    outs = P.block_attn_batch(*([it[i] for it in items] for i in range(5)), 330)
    for it, out in zip(items, outs):
        assert torch.equal(out, P.block_attn(*it, 330))


# Whole first rounds of tiles (256 keys) in the cache, or in the block if there is no cache, and one key fewer: what
# the workgroups' first copies are told by. Cache and block have strides of their own.
@pytest.mark.gpu
@pytest.mark.parametrize("c_len,n_blk", [(255, 40), (256, 40), (257, 33), (600, 1), (0, 255), (0, 256), (0, 257), (1, 300)])
@pytest.mark.parametrize("head_major", [False, True])
def test_first_copies(monkeypatch, c_len, n_blk, head_major):
    for n_q in (33, 64):
        run(32, monkeypatch, n_q, n_blk, c_len, seed=690 + c_len, head_major=head_major, commit=c_len > 0)


def test_plan_beyond_one_round():
    """32-row workgroups are taken as long as they need no more rounds than 64-row ones: one round, or any number with
    so few rows that both kernels have the same workgroups."""
    rows = lambda H, n_q, n_k, **kw: attn_plan_rows(H, n_q, n_k, n_cu=MI355X_CUS, **kw)
    assert [rows(300, 64, 256), rows(40, 33, 256, n_items=8), rows(257, 33, 193), rows(129, 64, 480)] == [64] * 4
    assert [rows(37, 1, 256, n_items=7), rows(300, 32, 512), rows(600, 20, 300), rows(128, 64, 480)] == [32] * 4


# Two and three rounds of 32-row workgroups; two rounds of 64-row ones, where 32 rows would need a third
@pytest.mark.gpu
@pytest.mark.parametrize("H,n_q,rows", [(259, 1, 32), (300, 32, 32), (513, 20, 32), (257, 33, 64), (300, 64, 64)])
def test_launches_beyond_one_round(monkeypatch, H, n_q, rows):
    monkeypatch.setitem(HEADS, rows, H)
    run(rows, monkeypatch, n_q, 150, 106, seed=680, commit=True)
