"""The key split under AUTO for launches that leave 25 to 60 % of the workgroup slots idle: which of them the
plan splits, parity of such a launch with the oracle, and that the call with the library's own array splits none."""
import pytest
import torch

import oracle
from gpu_util import BF16_MAX_ABS, BF16_REL_RMS, MI355X_CUS, attn_errors, attn_plan, attn_plan_static_workspace, bits_of


def test_auto_plan_with_a_quarter_to_60_percent_idle():
    plan = lambda H, n_q, n_k, n_items=1, split=1: attn_plan(H, n_q, n_k, n_items=n_items, split=split, n_cu=MI355X_CUS)
    for args in [(8, 4680, 32760), (5, 4680, 32760, 2), (14, 4680, 23400), (13, 1287, 9009, 2)]:
        assert plan(*args).split and plan(*args) == plan(*args, split=2)
    for args in [(11, 4680, 32760), (12, 4680, 14040), (5, 4680, 14040, 2), (20, 4680, 18720), (5, 2383, 7149, 3)]:
        assert not plan(*args).split and plan(*args).workspace == 0


def test_need_of_the_static_call():
    """The query's answer under AUTO is the batch call's: where only that one splits it exceeds the static call's array,
    of which the static call needs nothing. Under ALWAYS the two agree, and under AUTO the static call always fits."""
    limit = 64 << 20
    assert attn_plan(14, 4680, 9360, split=1, n_cu=MI355X_CUS).workspace == 104620032 > limit
    assert attn_plan_static_workspace(14, 4680, 9360) == 0
    for H in list(range(1, 41)) + [257]:
        for n_q in (256, 312, 1031, 1560, 2300, 3100, 4404, 4641, 4680):
            for n_k, n_items in ((n_q, 1), (3 * n_q, 2), (7 * n_q, 1), (65536, 1), (9360, 8)):
                always = attn_plan(H, n_q, n_k, n_items=n_items, split=2, n_cu=MI355X_CUS).workspace
                auto = attn_plan(H, n_q, n_k, n_items=n_items, split=1, n_cu=MI355X_CUS).workspace
                assert attn_plan_static_workspace(H, n_q, n_k, n_items, split=2) == always <= 277 * 10**6
                assert auto <= 182 * 10**6 and attn_plan_static_workspace(H, n_q, n_k, n_items) <= min(limit, always)


@pytest.mark.gpu
def test_auto_split_of_a_half_idle_launch():
    from test_gpu_attn_batch import split_shape_case
    import paper_2604_17397_amd as P
    dev, plain, split = split_shape_case(P, 2, 13, 1287, 6 * 1287, seed=470, jitter=True, split="auto")
    assert attn_plan(13, 1287, 7 * 1287, n_items=2, split=1).split
    rows = [0, 1, 31, 255, 256, 640, 1023, 1024, 1285, 1286]
    for d, a, b in zip(dev, plain, split):
        ref = oracle.block_attn(*[bits_of(d[n]) for n in ("q", "kc", "vc", "kb", "vb")], 6 * 1287, rows=rows)
        for o in (a, b):
            max_abs, rel = attn_errors(bits_of(o)[rows], ref)
            assert max_abs <= BF16_MAX_ABS and rel <= BF16_REL_RMS, (max_abs, rel)


@pytest.mark.gpu
@pytest.mark.parametrize("H", [8, 14])  # 14 heads: the split's partial results would not fit the array
def test_static_call_of_a_half_idle_launch_stays_unsplit(H):
    import paper_2604_17397_amd as P
    d = [torch.randn(4680, H, 128, device="cuda").bfloat16() for _ in range(5)]
    assert attn_plan(H, 4680, 9360, split=2).workspace > (0 if H == 8 else P.lib().sdvg_block_attn_static_workspace_limit())
    outs = [[torch.empty_like(d[0])] for _ in range(2)]
    P.block_attn_batch_static(*[[x] for x in d], 4680, outs[0], split="auto")
    P.block_attn_batch_static(*[[x] for x in d], 4680, outs[1], split="never")
    assert torch.equal(outs[0][0], outs[1][0])
