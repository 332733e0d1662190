"""The rows that the fused commit copies: block sizes and head counts around what one pass of the copying workgroups takes
(32 rows per workgroup, four passes at a time)."""
import pytest
import torch

from gpu_util import MI355X_CUS, attn_plan, attn_plan_commit


def test_copying_workgroups_beside_the_attention():
    """Of the workgroups that are launched, doubled ones counted twice: no more copying ones than the last round leaves room
    for on an XCD, or a full round, and none without a row."""
    assert attn_plan_commit(12, 312, 312, 936) == (240, 16)
    assert attn_plan_commit(8, 312, 312, 936) == (160, 78) and attn_plan_commit(8, 500, 500, 500) == (256, 125)
    n_doubled = 0
    for H in range(3, 17):
        for n_q in (33, 100, 250, 312, 400, 513, 800):
            for n_k in (n_q, 2 * n_q, 5 * n_q):
                work, copies = attn_plan_commit(H, n_q, n_q, n_k)
                plan = attn_plan(H, n_q, n_k, n_cu=MI355X_CUS)
                assert work == plan.workgroups * (2 if plan.rows == 32 and 2 * plan.workgroups <= MI355X_CUS else 1)
                n_doubled += work != plan.workgroups
                per_xcd = -(-work // 8)
                assert 1 <= copies <= -(-H * n_q // 32)
                assert per_xcd % 32 + -(-copies // 8) <= 32 or copies == min(256, -(-H * n_q // 32))
    assert n_doubled > 100


def test_copies_that_would_outlast_the_round_take_a_full_one():
    n = lambda H, T, cached: attn_plan_commit(H, T, T, (cached + 1) * T)[1]
    assert [n(40, 4680, c) for c in (0, 1, 3, 6)] == [256, 256, 256, 8]
    assert [n(13, 4680, c) for c in (0, 1)] == [256, 8] and n(30, 2000, 0) == 256 and n(12, 4680, 0) == 24
    assert [n(24, 312, c) for c in (0, 2)] == [234, 16] and n(12, 312, 0) == 16


@pytest.mark.gpu
@pytest.mark.parametrize("head_major", [False, True])
@pytest.mark.parametrize("H,n_blk,c_len", [(1, 1, 0), (1, 4700, 33), (3, 33, 65), (12, 312, 624), (24, 312, 40), (40, 103, 0),
                                           (257, 40, 8), (1000, 9, 100), (5, 1409, 0)])
def test_every_row_is_copied_and_no_other(H, n_blk, c_len, head_major):
    import paper_2604_17397_amd as P
    g = torch.Generator(device="cuda").manual_seed(H + n_blk)
    mk = lambda t: torch.randn((t, H, 128), device="cuda", generator=g).bfloat16()
    q, kb, vb, kc, vc = mk(min(n_blk, 40)), mk(n_blk), mk(n_blk), mk(c_len + n_blk + 2), mk(c_len + n_blk + 2)
    if head_major:
        kb, vb, kc, vc = [x.transpose(0, 1).contiguous().transpose(0, 1) for x in (kb, vb, kc, vc)]
    k0, v0 = kc.clone(), vc.clone()
    plain = P.block_attn(q, kc, vc, kb, vb, c_len)
    assert torch.equal(P.block_attn_commit(q, kc, vc, kb, vb, c_len), plain)
    for cache, before, blk in ((kc, k0, kb), (vc, v0, vb)):
        assert torch.equal(cache[c_len:c_len + n_blk], blk)
        assert torch.equal(cache[:c_len], before[:c_len]) and torch.equal(cache[c_len + n_blk:], before[c_len + n_blk:])
