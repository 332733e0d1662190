"""The rows that the fused commit copies: block sizes and head counts around what one pass of the copying workgroups takes
(32 rows per workgroup, four passes at a time)."""
import pytest
import torch


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
